"""The Filter stage's value classes against the oracle's predicate masks:
row counts at the edges of a bitmap word, a classified block and a count
part; batches on both sides of a mask word and a query group; clauses on one
to five columns (five take the per-pair tests), several clauses on one
column, bounds at the ends of the int32 range, value tables and searched
bounds, predicates that everything or nothing satisfies."""
import time

import numpy as np
import pytest
import torch

import oracle as O
from tests._gpu_util import say

pytestmark = pytest.mark.gpu
I32 = np.iinfo(np.int32)


@pytest.fixture(scope="module")
def B():
    from paper_2607_22922_amd import ifvs
    return ifvs


def _attrs(n, cols, span, rng):
    a = rng.integers(-span, span, size=(cols, n), dtype=np.int64)
    a[:, rng.integers(0, n, 3)] = [I32.min, I32.max, 0]
    return a.clip(I32.min, I32.max).astype(np.int32)


def _clause(rng, cols, span):
    c = int(rng.integers(0, cols))
    kind = rng.integers(0, 8)
    lo = int(rng.integers(-span, span))
    hi = lo + int(rng.integers(1, span + 1))
    return [(c, lo, hi), (c, lo, lo + 1), (c, I32.min, hi), (c, lo, I32.max + 1), (c, -(1 << 40), hi),
            (c, lo, 1 << 40), (c, I32.max, I32.max + 1), (c, lo, hi)][kind]


@pytest.mark.parametrize("n,nq,cols,span", [
    (1, 1, 1, 5), (31, 3, 1, 40), (33, 33, 2, 40), (2047, 31, 2, 100), (2049, 129, 1, 3000), (4097, 5, 3, 9),
    (16384, 128, 2, 4000), (16385, 64, 4, 1 << 30), (40_001, 257, 4, 50), (40_001, 130, 2, 1 << 31),
    (20_000, 40, 5, 60), (100_003, 300, 3, 6000)])
def test_filter_matches_oracle(B, n, nq, cols, span):
    say(f"[filter] n={n} nq={nq} cols={cols} span={span}")
    rng = np.random.default_rng(n + nq)
    attrs = _attrs(n, cols, span, rng)
    preds = []
    for i in range(nq):
        k = int(rng.integers(0, 5))
        preds.append([_clause(rng, cols, span) for _ in range(k)])
        if i % 9 == 4:
            preds[-1] = [(0, 7, 7)]                       # nothing passes
    codes = torch.zeros(n, 1, dtype=torch.uint8, device="cuda")
    idx = B.Index(codes, torch.zeros(1, 256, 1, device="cuda"), torch.from_numpy(attrs).cuda(), max_batch=nq, max_k=1)
    bm, cnt = idx.filter(preds)
    torch.cuda.synchronize()
    got, cnt = B.bitmap_words_to_numpy(bm), cnt.cpu().numpy()
    for i, p in enumerate(preds):
        mask = O.predicate_mask(attrs, p)
        want = np.packbits(np.pad(mask, (0, -n % 32)), bitorder="little").view("<u4")
        assert np.array_equal(got[i], want), (i, p)
        assert cnt[i] == mask.sum(), (i, p)


def test_filter_bounds_of_one_group_only(B):
    """Groups whose clauses pile up on different columns: more LDS than there
    is for the classes, so the batch takes the per-pair tests."""
    n, nq, cols = 5_000, 512, 4
    rng = np.random.default_rng(1)
    attrs = _attrs(n, cols, 1 << 30, rng)
    preds = []
    for i in range(nq):
        c = i // 128
        preds.append([(c, int(v), int(v) + (1 << 30)) for v in rng.integers(-(1 << 30), 1 << 30, 4)])
    codes = torch.zeros(n, 1, dtype=torch.uint8, device="cuda")
    idx = B.Index(codes, torch.zeros(1, 256, 1, device="cuda"), torch.from_numpy(attrs).cuda(), max_batch=nq, max_k=1)
    bm, cnt = idx.filter(preds)
    torch.cuda.synchronize()
    got, cnt = B.bitmap_words_to_numpy(bm), cnt.cpu().numpy()
    for i, p in enumerate(preds):
        mask = O.predicate_mask(attrs, p)
        want = np.packbits(np.pad(mask, (0, -n % 32)), bitorder="little").view("<u4")
        assert np.array_equal(got[i], want) and cnt[i] == mask.sum(), (i, p)


@pytest.mark.parametrize("n,nq,clauses", [
    (2049, 32, 1), (1, 17, 1), (63, 40, 1), (2047, 129, 1), (16_385, 48, 1), (40_001, 33, "mixed"), (40_001, 60, 1),
    (1_850_003, 33, 1), (30_000, 16, 1), (200_003, 60, 1)])
def test_one_clause_batches(B, n, nq, clauses):
    """Batches of one clause a query: the pair tests of one column (few pairs),
    the classes, and batches where some predicates have none; the oracle's
    bits, and no more time than a pass takes (16 queries of 10K rows took 270
    us where 40 suffice)."""
    say(f"[filter] one clause n={n} nq={nq} clauses={clauses}")
    rng = np.random.default_rng(n + nq)
    attrs = _attrs(n, 2, 300, rng)
    preds = [[(1, int(lo), int(lo) + int(w))] for lo, w in zip(rng.integers(-300, 300, nq), rng.integers(1, 400, nq))]
    preds[0], preds[-1] = [(1, I32.min, 5)], [(1, 5, 1 << 40)]
    if clauses == "mixed":
        preds[3], preds[7] = [], [(1, 9, 9)]
    codes = torch.zeros(n, 1, dtype=torch.uint8, device="cuda")
    idx = B.Index(codes, torch.zeros(1, 256, 1, device="cuda"), torch.from_numpy(attrs).cuda(), max_batch=nq, max_k=1)
    pc = B.pack_predicates(preds)
    bm = torch.full((nq, idx.words()), -1, dtype=torch.int32, device="cuda")
    cnt = torch.empty(nq, dtype=torch.int64, device="cuda")
    best = 1e9
    for _ in range(8):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        idx.filter_into(nq, pc, bm, cnt)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    got, count = B.bitmap_words_to_numpy(bm), cnt.cpu().numpy()
    for i, p in enumerate(preds):
        mask = O.predicate_mask(attrs, p)
        want = np.packbits(np.pad(mask, (0, -n % 32)), bitorder="little").view("<u4")
        assert np.array_equal(got[i], want) and count[i] == mask.sum(), (i, p)
    say(f"[filter] {best * 1e6:.0f} us")
    assert best < 150e-6
