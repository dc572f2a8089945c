"""The exact search's sampled first pass: the screened plan gives the direct
plan's ids and distance bits where pass 1 reads every tile (k of 600), every
second or every eighth one of a wavefront (k, rows and queries decide), for row
lengths with every build, intervals and masks."""
import pytest
import torch

from tests._gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2607_22922_amd import ifvs
    return ifvs


@pytest.mark.parametrize("n,dim,nq,cluster", [(600_001, 96, 256, (0,)), (300_007, 128, 70, ()), (2_500_003, 50, 256, (0,)),
                                           (4_000, 96, 3, (0,))])
def test_sampled_screening_matches_direct(B, n, dim, nq, cluster):
    say(f"[exact] n={n} dim={dim} nq={nq} cluster={cluster}")
    g = torch.Generator(device="cuda").manual_seed(n)
    attrs = torch.randint(0, 1000, (1, n), generator=g, device="cuda", dtype=torch.int32)
    means = torch.rand(20, dim, generator=g, device="cuda") * 2 - 1
    x = means[torch.randint(0, 20, (n,), generator=g, device="cuda")]
    x = x + 0.3 * torch.randn(n, dim, generator=g, device="cuda")
    x[1::2003] = x[0]                                    # equal rows: ties by id
    q = means[torch.randint(0, 20, (nq,), generator=g, device="cuda")] + 0.3 * torch.randn(nq, dim, generator=g,
                                                                                            device="cuda")
    q[0] = x[0]
    codes = torch.zeros(n, 1, dtype=torch.uint8, device="cuda")
    idx = B.Index(codes, torch.zeros(1, 256, dim, device="cuda"), attrs, max_batch=nq, max_k=600, cluster_cols=cluster)
    idx.load_vectors(x)
    preds = [[(0, (7 * i) % 400, (7 * i) % 400 + 500)] for i in range(nq)]
    preds[-1] = [(0, 4, 5)]
    for k in (1, 10, 100, 600):
        out = []
        for plan in (2, 1):
            idx.set_option(B.OPT_EXACT_PLAN, plan)
            ids, dist = idx.exact_search(q, preds, k)
            torch.cuda.synchronize()
            out.append((ids, dist.view(torch.int32)))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]), k


@pytest.mark.parametrize("dim", [1, 16, 17, 33, 64, 65, 96, 97, 112, 113, 128, 129, 144])
def test_every_build_matches_direct(B, dim):
    """Row lengths on both sides of each count of 16-dimension steps with a
    build of its own (1 to 8) and above them."""
    say(f"[exact] dim={dim}")
    n, nq, k = 50_003, 45, 10
    g = torch.Generator(device="cuda").manual_seed(dim)
    attrs = torch.randint(0, 1000, (1, n), generator=g, device="cuda", dtype=torch.int32)
    x = torch.randn(n, dim, generator=g, device="cuda")
    q = torch.randn(nq, dim, generator=g, device="cuda")
    idx = B.Index(torch.zeros(n, 1, dtype=torch.uint8, device="cuda"), torch.zeros(1, 256, dim, device="cuda"), attrs,
                  max_batch=nq, max_k=k, cluster_cols=(0,))
    idx.load_vectors(x)
    preds = [[(0, (7 * i) % 400, (7 * i) % 400 + 500)] for i in range(nq)]
    out = []
    for plan in (2, 1):
        idx.set_option(B.OPT_EXACT_PLAN, plan)
        ids, dist = idx.exact_search(q, preds, k)
        torch.cuda.synchronize()
        out.append((ids, dist.view(torch.int32)))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


def test_intervals_within_the_error_bound(B):
    """Short intervals of long rows, whose distances lie within the screening's
    error bound of each other: nearly every row is a candidate, and the lists
    hold each exactly once."""
    n, dim, nq, k = 20_000, 400, 333, 4
    say("[exact] dense candidates")
    g = torch.Generator(device="cuda").manual_seed(7)
    attrs = torch.randint(0, 1000, (1, n), generator=g, device="cuda", dtype=torch.int32)
    x, q = (torch.randn(r, dim, generator=g, device="cuda") for r in (n, nq))
    idx = B.Index(torch.zeros(n, 1, dtype=torch.uint8, device="cuda"), torch.zeros(1, 256, dim, device="cuda"), attrs,
                  max_batch=nq, max_k=700, cluster_cols=(0,))
    idx.load_vectors(x)
    preds = [[(0, i % 970, i % 970 + 1 + i % 30)] for i in range(nq)]
    for kk in (k, 700):
        out = []
        for plan in (2, 1):
            idx.set_option(B.OPT_EXACT_PLAN, plan)
            ids, dist = idx.exact_search(q, preds, kk)
            torch.cuda.synchronize()
            out.append((ids, dist.view(torch.int32)))
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
