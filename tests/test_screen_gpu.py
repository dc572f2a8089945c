"""Packed-table screening of shared rows: the same ids and distance bits as
the tiled scan and the oracle.  Sizes at the edges of a 64-row tile, a
wavefront's block of tiles and a workgroup's chunk; batches that are no whole
group of four; subspace counts on both sides of the prefetched code words (6)
and of a word's four; k at its limit and above the rows selected; tables with
negative, NaN and infinite entries, and lists that overflow (equal rows), which
keep the tiled scan."""
import os
import subprocess
import sys
import time

import numpy as np
import pytest
import torch

import oracle as O
from tests._gpu_util import check_search_row, say

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def B():
    from paper_2607_22922_amd import ifvs
    return ifvs


def _np(t):
    return t.detach().cpu().numpy()


def _index(B, n, m, nq, k, cluster, seed, spread=256, domain=200):
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, spread, size=(n, m), dtype=np.uint8)
    attrs = np.stack([rng.integers(0, domain, n), rng.integers(0, 5, n)]).astype(np.int32)
    idx = B.Index(torch.from_numpy(codes).cuda(), torch.zeros(m, 256, 1, device="cuda"),
                  torch.from_numpy(attrs).cuda(), max_batch=nq, max_k=k, cluster_cols=cluster)
    return idx, codes, attrs, rng


def _preds(rng, nq, domain):
    out = []
    for i in range(nq):
        lo = int(rng.integers(0, domain // 2))
        out.append([(0, lo, lo + domain // 2)])
        if i % 5 == 1:
            out[-1].append((1, 0, 3))
        if i % 11 == 7:
            out[-1] = [(0, lo, lo + 1), (1, 2, 3)]       # few rows: at times fewer than k
        if i % 13 == 12:
            out[-1] = [(0, 5, 5)]                        # none
    return out


def _both(B, idx, preds, lut, k, dt):
    out = []
    for mode in (2, 1):
        idx.set_option(B.OPT_SCREEN, mode)
        ids, dist = idx.search(preds, lut, k, dt)
        torch.cuda.synchronize()
        modes = idx.last_modes(len(preds))
        out.append((_np(ids), _np(dist), modes))
    idx.set_option(B.OPT_SCREEN, 0)
    (ids, dist, modes), (ids1, dist1, modes1) = out
    assert np.array_equal(ids, ids1)
    assert np.array_equal(dist.view(np.uint32), dist1.view(np.uint32))
    assert not (modes1 == 2).any()                       # the tiled scan or row lists
    return ids, dist, modes


def _check(lut, codes, attrs, preds, k, ids, dist, rows):
    for i in rows:
        cand = O.passing_ids(O.predicate_mask(attrs, preds[i]))
        ids_o, dist_o = O.select_topk(O.adc_distances(_np(lut[i]).astype(np.float32), codes, cand), cand, k)
        check_search_row(ids[i], dist[i], ids_o, dist_o, f"q{i} {preds[i]}")


@pytest.mark.parametrize("n,m,nq,k,f16,cluster", [
    (63, 3, 1, 1, False, ()), (65, 4, 5, 7, False, (0,)), (4095, 5, 4, 10, True, ()), (4097, 16, 9, 128, False, (0,)),
    (33_001, 21, 6, 33, True, (0,)), (32_767, 24, 8, 10, False, ()), (40_000, 25, 7, 16, False, (1, 0)),
    (70_001, 48, 13, 10, False, (0,)), (70_001, 48, 37, 100, True, ()), (50_003, 120, 11, 100, False, (0,)),
    (300_007, 16, 40, 10, False, ()), (300_007, 8, 40, 100, False, (0, 1))])
def test_screening_matches_scan_and_oracle(B, n, m, nq, k, f16, cluster):
    say(f"[screen] n={n} m={m} nq={nq} k={k} f16={f16} cluster={cluster}")
    idx, codes, attrs, rng = _index(B, n, m, nq, k, cluster, seed=n + m)
    preds = _preds(rng, nq, 200)
    g = torch.Generator(device="cuda").manual_seed(n)
    # a few near codewords, many far ones, as in a trained quantizer
    lut = torch.rand(nq, m, 256, generator=g, device="cuda") ** 2 * 7 + 0.25 * torch.rand(nq, m, 1, generator=g, device="cuda")
    dt = B.LUT_F16 if f16 else B.LUT_F32
    lut = lut.half() if f16 else lut
    idx.set_option(B.OPT_GATHER, 2)                      # no row lists: screened or left to the scan
    ids, dist, modes = _both(B, idx, preds, lut, k, dt)
    _check(lut, codes, attrs, preds, k, ids, dist, range(min(nq, 13)))
    for i, p in enumerate(preds):
        rows = int(O.predicate_mask(attrs, p).sum())
        if rows * min(1.0, 128 * 64 / n) >= 4 * k + 32:  # plenty in the seed's sample of 128 tiles
            assert modes[i] == 2, (i, p, rows)
        elif rows < k:
            assert modes[i] == 0, (i, p, rows)


def test_screening_leaves_unbounded_queries_to_the_scan(B):
    n, m, nq, k = 50_000, 12, 12, 10
    say("[screen] negative, NaN, infinite, constant and tiny tables, equal rows")
    idx, codes, attrs, rng = _index(B, n, m, nq, k, (), seed=5, spread=4)
    preds = [[(0, 0, 150)]] * nq
    lut = torch.rand(nq, m, 256, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    lut[1, 3, 2] = -0.5
    lut[2, 0, 1] = float("nan")
    lut[3, :, 1] = float("inf")
    lut[4] = float("inf")
    lut[5] = 0.25                      # every row at one distance: its list overflows
    lut[6] = 0.0
    lut[7] *= 1e-38
    lut[8] *= 1e37
    lut[9, 2:] = 0.0
    ids, dist, modes = _both(B, idx, preds, lut, k, B.LUT_F32)
    _check(lut, codes, attrs, preds, k, ids, dist, [0, 1, 3, 5, 6, 7, 8, 9, 10, 11])
    left = [1, 2, 4, 5, 6]                               # negative, NaN, infinite, equal rows
    assert (modes[left] == 0).all() and (modes[[0, 3, 10, 11]] == 2).all(), modes


def test_screening_is_chosen_by_work_and_sharing(B):
    """A large batch over the same rows is screened automatically, a small one
    and every way of asking for the tiled scan are not; the same answer."""
    n, m, nq, k = 400_000, 16, 256, 10
    say("[screen] automatic")
    idx, codes, attrs, rng = _index(B, n, m, nq, k, (), seed=9)
    preds = _preds(rng, nq, 200)
    lut = torch.rand(nq, m, 256, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2)) ** 2
    ids, dist, _ = _both(B, idx, preds, lut, k, B.LUT_F32)
    half = np.array([p[0][2] - p[0][1] > 1 and len(p) == 1 for p in preds])       # half of the rows
    for opt, value in ((None, 0), (B.OPT_QTILE, 2), (B.OPT_GATHER, 2), (B.OPT_SCREEN, 1)):
        if opt:
            idx.set_option(opt, value)
        i2, d2 = idx.search(preds, lut, k)
        torch.cuda.synchronize()
        modes = idx.last_modes(nq)
        if opt:
            idx.set_option(opt, 0)
        assert np.array_equal(_np(i2), ids) and np.array_equal(_np(d2).view(np.uint32), dist.view(np.uint32))
        assert (modes[half] == (0 if opt in (B.OPT_QTILE, B.OPT_SCREEN) else 2)).all(), (opt, modes)
    _check(lut, codes, attrs, preds, k, ids, dist, range(0, nq, 41))
    idx.search(preds[:8], lut[:8].contiguous(), k)                                # little to share
    torch.cuda.synchronize()
    assert not (idx.last_modes(8) == 2).any()


@pytest.mark.parametrize("m,n,nq,k,screened", [
    (21, 800_003, 100, 60, True),        # the scan's and its merge's time grows with k
    (40, 120_001, 72, 2, False),         # short intervals, few neighbours
    (30, 3_000_000, 40, 10, True),       # long intervals
    (4, 1_500_000, 107, 9, False)])      # rows of four subspaces tie
def test_any_subspace_count_is_screened_where_it_pays(B, m, n, nq, k, screened):
    say(f"[screen] automatic, m={m} n={n} nq={nq} k={k}")
    g = torch.Generator(device="cuda").manual_seed(m)
    codes = torch.randint(0, 256, (n, m), generator=g, device="cuda", dtype=torch.uint8)
    attrs = torch.randint(0, 1000, (1, n), generator=g, device="cuda", dtype=torch.int32)
    idx = B.Index(codes, torch.zeros(m, 256, 1, device="cuda"), attrs, max_batch=nq, max_k=k, cluster_cols=(0,))
    preds = [[(0, i * 7 % 900, i * 7 % 900 + 100)] for i in range(nq)]
    lut = torch.rand(nq, m, 256, generator=g, device="cuda") ** 2
    ids, dist = idx.search(preds, lut, k)
    torch.cuda.synchronize()
    assert int((idx.last_modes(nq) == 2).sum()) == (nq if screened else 0)
    idx.set_option(B.OPT_SCREEN, 1)
    ids1, dist1 = idx.search(preds, lut, k)
    torch.cuda.synchronize()
    assert torch.equal(ids, ids1) and torch.equal(dist.view(torch.int32), dist1.view(torch.int32))


@pytest.mark.parametrize("m,n,screened", [(48, 300_007, False), (48, 900_007, True), (16, 900_007, True)])
def test_row_by_row_clauses_are_screened_where_it_pays(B, m, n, screened):
    """Intervals of 67 queries over 42% of the rows, a second clause tested row
    by row: 6.4e6 triples keep the scan for M = 48, 2e7 (M = 16: 6.4e6) do not."""
    nq, k = 67, 2
    say(f"[screen] automatic, row by row, m={m} n={n}")
    g = torch.Generator(device="cuda").manual_seed(m)
    codes = torch.randint(0, 256, (n, m), generator=g, device="cuda", dtype=torch.uint8)
    attrs = torch.randint(0, 1000, (2, n), generator=g, device="cuda", dtype=torch.int32)
    idx = B.Index(codes, torch.zeros(m, 256, 1, device="cuda"), attrs, max_batch=nq, max_k=k, cluster_cols=(0,))
    preds = [[(0, i * 7 % 500, i * 7 % 500 + 422), (1, 10, 990)] for i in range(nq)]
    lut = torch.rand(nq, m, 256, generator=g, device="cuda") ** 2
    ids, dist = idx.search(preds, lut, k)
    torch.cuda.synchronize()
    assert int((idx.last_modes(nq) == 2).sum()) == (nq if screened else 0)
    idx.set_option(B.OPT_SCREEN, 1)
    ids1, dist1 = idx.search(preds, lut, k)
    torch.cuda.synchronize()
    assert torch.equal(ids, ids1) and torch.equal(dist.view(torch.int32), dist1.view(torch.int32))


@pytest.mark.parametrize("nq,cluster,width,screened", [
    (1200, (0,), 500, False), (250, (0,), 900, True), (1700, (), 110, False), (250, (), 400, True)])
def test_large_batches_are_screened_where_each_query_has_work(B, nq, cluster, width, screened):
    """Every query beyond 256 costs the screening its own seed and rerank:
    many queries of few tiles keep the scan or the row lists."""
    n, m, k = (100_003, 48, 5) if screened is False else (400_003, 48, 5)
    say(f"[screen] automatic, nq={nq} cluster={cluster}")
    g = torch.Generator(device="cuda").manual_seed(nq)
    codes = torch.randint(0, 256, (n, m), generator=g, device="cuda", dtype=torch.uint8)
    attrs = torch.randint(0, 1000, (1, n), generator=g, device="cuda", dtype=torch.int32)
    idx = B.Index(codes, torch.zeros(m, 256, 1, device="cuda"), attrs, max_batch=nq, max_k=k, cluster_cols=cluster)
    preds = [[(0, i * 7 % (1000 - width), i * 7 % (1000 - width) + width)] for i in range(nq)]
    lut = torch.rand(nq, m, 256, generator=g, device="cuda") ** 2
    ids, dist = idx.search(preds, lut, k)
    torch.cuda.synchronize()
    assert int((idx.last_modes(nq) == 2).sum()) == (nq if screened else 0)
    idx.set_option(B.OPT_SCREEN, 1)
    ids1, dist1 = idx.search(preds, lut, k)
    torch.cuda.synchronize()
    assert torch.equal(ids, ids1) and torch.equal(dist.view(torch.int32), dist1.view(torch.int32))


def test_equal_rows_cost_little_more_than_the_scan(B):
    """Queries whose every row ties overflow their survivor lists and are left
    to the scan: the screening gives them up early (it took five times the
    scan's time while it counted every row)."""
    n, m, nq, k = 2_000_000, 48, 256, 10
    say("[screen] tied tables, time")
    g = torch.Generator(device="cuda").manual_seed(3)
    codes = torch.randint(0, 256, (n, m), generator=g, device="cuda", dtype=torch.uint8)
    attrs = torch.randint(0, 100, (1, n), generator=g, device="cuda", dtype=torch.int32)
    idx = B.Index(codes, torch.zeros(m, 256, 1, device="cuda"), attrs, max_batch=nq, max_k=k)
    preds = [[(0, i % 50, i % 50 + 50)] for i in range(nq)]
    lut = torch.full((nq, m, 256), 0.25, device="cuda")
    best = _times(B, idx, preds, lut, k, attrs, left=range(nq))
    assert best[0] < 2.5 * best[1]


def _times(B, idx, preds, lut, k, attrs, left):
    """Seconds of a search with and without the screening; `left`: the queries
    it must leave, whose rows all tie (the first k selected ids)."""
    nq, best = len(preds), {}
    pc = B.pack_predicates(preds)
    ids = torch.empty(nq, k, dtype=torch.int32, device="cuda")
    dist = torch.empty(nq, k, device="cuda")
    for mode in (0, 1):
        idx.set_option(B.OPT_SCREEN, mode)
        for _ in range(4):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            idx.search_into(nq, pc, lut, B.LUT_F32, k, ids, dist)
            torch.cuda.synchronize()
            best[mode] = min(best.get(mode, 1e9), time.perf_counter() - t0)
        modes = idx.last_modes(nq) == 2
        assert modes.any() == (mode == 0 and len(left) < nq) and not modes[list(left)].any()
        for i in list(left)[:50]:
            (_, lo, hi), = preds[i]
            assert torch.equal(ids[i].long(), torch.nonzero((attrs[0] >= lo) & (attrs[0] < hi))[:k, 0])
    say(f"[screen] tied: {best[0] * 1e3:.2f} ms automatic, {best[1] * 1e3:.2f} ms without the screening")
    return best


def test_a_tied_query_over_a_long_interval(B):
    """The scan of a query that the screening leaves is cut into chunks enough
    for one query (in 16 it took longer than the whole batch's scan)."""
    n, m, nq, k = 10_000_000, 16, 256, 10
    say("[screen] one tied query over a long interval, time")
    g = torch.Generator(device="cuda").manual_seed(3)
    codes = torch.randint(0, 256, (n, m), generator=g, device="cuda", dtype=torch.uint8)
    attrs = torch.randint(0, 1000, (1, n), generator=g, device="cuda", dtype=torch.int32)
    idx = B.Index(codes, torch.zeros(m, 256, 1, device="cuda"), attrs, max_batch=nq, max_k=k, cluster_cols=(0,))
    preds = [[(0, i % 500, i % 500 + 500)] for i in range(nq)]
    lut = torch.rand(nq, m, 256, device="cuda", generator=g) ** 2
    lut[3] = 0.25
    best = _times(B, idx, preds, lut, k, attrs, left=[3])
    assert best[0] < 1.05 * best[1]


def test_queries_left_by_the_screening_take_row_lists(B):
    """A masked batch is screened before the row lists are made, so a pool of
    up to 30% of the rows that the screening leaves (tied rows) is scored from
    its list, as without the screening, and not by a pass over every tile."""
    n, m, nq, k = 1_500_000, 48, 256, 10
    say("[screen] row lists after the screening")
    g = torch.Generator(device="cuda").manual_seed(4)
    codes = torch.randint(0, 256, (n, m), generator=g, device="cuda", dtype=torch.uint8)
    attrs = torch.randint(0, 100, (1, n), generator=g, device="cuda", dtype=torch.int32)
    idx = B.Index(codes, torch.zeros(m, 256, 1, device="cuda"), attrs, max_batch=nq, max_k=k)
    width = [(2, 10, 50)[i % 3] for i in range(nq)]                   # 2%, 10% and 50% of the rows
    preds = [[(0, i % 50, i % 50 + w)] for i, w in enumerate(width)]
    lut = torch.rand(nq, m, 256, device="cuda", generator=g) ** 2
    tied = torch.arange(nq, device="cuda") % 5 == 0
    lut[tied] = 0.25
    out = []
    for mode in (0, 1):
        idx.set_option(B.OPT_SCREEN, mode)
        ids, dist = idx.search(preds, lut, k)
        torch.cuda.synchronize()
        out.append((ids, dist.view(torch.int32), idx.last_modes(nq)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    for i, w in enumerate(width):
        want = 1 if w == 2 else (2 if not tied[i] else (1 if w == 10 else 0))
        assert out[0][2][i] == want, (i, w, bool(tied[i]), out[0][2][i])
        assert out[1][2][i] == (1 if w <= 10 else 0)


LOAD_WITHOUT = r"""
import sys, torch
sys.path.insert(0, %r)
from paper_2607_22922_amd import ifvs as B
g = torch.Generator(device="cuda").manual_seed(1)
n, m, nq, k, cluster, force = %s
codes = torch.randint(0, 256, (n, m), generator=g, device="cuda", dtype=torch.uint8)
attrs = torch.arange(n, device="cuda", dtype=torch.int32)[None].contiguous()
lut = torch.rand(nq, m, 256, generator=g, device="cuda")
preds = [[(0, 10 * i, 10 * i + n - 1000)] for i in range(nq)]
out = []
for _ in range(2):
    try:
        idx = B.Index(codes, torch.zeros(m, 256, 1, device="cuda"), attrs, max_batch=nq, max_k=k, cluster_cols=cluster)
    except B.IfvsError as e:
        print("REFUSED", e)
        sys.exit(0)
    if force:
        idx.set_option(B.OPT_SCREEN, 2)
    print("LOADED", B.lib().ifvs_last_error().decode())
    ids, dist = idx.search(preds, lut, k)
    torch.cuda.synchronize()
    print("SCREENED", int((idx.last_modes(nq) == 2).sum()))
    out.append((ids, dist))
print("SAME", torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]))
"""


@pytest.mark.parametrize("shape", [(5000, 4, 8, 5, (), True), (400_003, 24, 64, 40, (0,), False)],
                         ids=["forced", "automatic"])
def test_index_works_without_the_screening_workspace(shape):
    """The workspace is the last allocation, of the load where batches can be
    screened automatically, else of asking for it; when it fails, the index
    works all the same and its batches take the scan."""
    nq = shape[2]
    for n in range(34, 0, -1):
        p = subprocess.run([sys.executable, "-c", LOAD_WITHOUT % (ROOT, shape)], capture_output=True, text=True,
                           timeout=100, env=dict(os.environ, IFVS_FAIL_ALLOC=str(n)))
        assert p.returncode == 0, p.stderr[-2000:]
        lines = p.stdout.splitlines()
        say(f"[screen] allocation {n} fails: {lines}")
        if "forced allocation failure" in lines[0]:
            break
    assert lines[0] == "LOADED forced allocation failure: screening workspace", lines
    assert lines[1:] == ["SCREENED 0", lines[0], f"SCREENED {nq}", "SAME True"], lines


def test_small_index_takes_no_screening_workspace(B):
    """No batch of it is screened automatically: the workspace is allocated
    when the screening is asked for."""
    n, m, nq, k = 1000, 16, 4096, 2
    say("[screen] small index")
    codes = torch.randint(0, 256, (n, m), device="cuda", dtype=torch.uint8)
    attrs = torch.arange(n, device="cuda", dtype=torch.int32)[None].contiguous()
    idx = B.Index(codes, torch.zeros(m, 256, 1, device="cuda"), attrs, max_batch=nq, max_k=k)
    preds = [[(0, 0, 900)]] * 8
    lut = torch.rand(8, m, 256, device="cuda")
    out = []
    for mode, screened in ((0, 0), (2, 8), (0, 0)):
        before = torch.cuda.mem_get_info()[0]
        idx.set_option(B.OPT_SCREEN, mode)
        taken = before - torch.cuda.mem_get_info()[0]
        assert (taken > 20 << 20) == (mode == 2), taken                # 16 MB of lists, 16 MiB of tables
        idx.set_option(B.OPT_GATHER, 2)
        ids, dist = idx.search(preds, lut, k)
        torch.cuda.synchronize()
        assert int((idx.last_modes(8) == 2).sum()) == screened
        out.append((ids, dist))
    assert all(torch.equal(o[0], out[0][0]) and torch.equal(o[1], out[0][1]) for o in out)
