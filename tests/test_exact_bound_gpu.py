"""The screened exact search on values whose bf16 roundings all point one way
(constant or quantized descriptors): the nearest row is screened as far and
the others as near as the rounding allows, and it is still found."""
import pytest
import torch

from tests._gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2607_22922_amd import ifvs
    return ifvs


def both_plans(B, idx, q, preds, k):
    out = []
    for plan in (2, 1):
        idx.set_option(B.OPT_EXACT_PLAN, plan)
        ids, dist = idx.exact_search(q, preds, k)
        torch.cuda.synchronize()
        out.append((ids.cpu(), dist.cpu().view(torch.int32)))
    return out


def exact_index(B, x, nq, k):
    n, dim = x.shape
    attrs = torch.arange(n, device="cuda", dtype=torch.int32)[None]
    idx = B.Index(torch.zeros(n, 1, dtype=torch.uint8, device="cuda"), torch.zeros(1, 256, dim, device="cuda"),
                  attrs.contiguous(), max_batch=nq, max_k=k)
    idx.load_vectors(x)
    return idx


@pytest.mark.parametrize("dim", [50, 96, 97, 128])
@pytest.mark.parametrize("k", [1, 10, 400])
def test_nearest_row_with_one_sided_rounding(B, dim, k):
    say(f"[exact bound] dim={dim} k={k}")
    n, nq, h = 100_000, 40, (dim - 1) // 2
    down, up = 1 + 2.0 ** -8, 1 + 2.0 ** -8 + 2.0 ** -14
    q = torch.zeros(nq, dim, device="cuda")
    q[:, :h], q[:, h:2 * h], q[:, 2 * h] = down, up, 1.0
    x = torch.zeros(n, dim, device="cuda")
    near, others = 70_001, torch.arange(500, device="cuda") * 131
    x[near, :h], x[near, 2 * h] = down, 2.0 ** -4
    x[others, h:2 * h] = up
    idx = exact_index(B, x, nq, k)
    (ids, dist), (ids1, dist1) = both_plans(B, idx, q, [[(0, 0, n)]] * nq, k)
    assert bool((ids1[:, 0] == near).all())              # the direct plan: scored as defined
    assert torch.equal(ids, ids1) and torch.equal(dist, dist1)


@pytest.mark.parametrize("dim", [50, 96])
def test_sums_beyond_fp32(B, dim):
    """Finite values whose |q|^2, |x|^2 or x.q overflow fp32: no row is left
    out for an infinite or undefined screened value."""
    say(f"[exact bound] overflow dim={dim}")
    n, nq, k = 60_000, 36, 10
    g = torch.Generator(device="cuda").manual_seed(dim)
    x = torch.randn(n, dim, generator=g, device="cuda")
    q = torch.randn(nq, dim, generator=g, device="cuda")
    q[1] = 1e20                                          # |q|^2 overflows, every distance too
    q[2, 0] = 2e19                                       # the same in one dimension
    preds = [[(0, 0, n)]] * nq
    for big in (False, True):
        if big:                                          # rows whose own norm overflows, a query near them, the origin
            x[777:30_000:997] = 3e18 * (1 + 0.001 * torch.randn(30, dim, generator=g, device="cuda"))
            q[3], q[4], q[5] = 3e18, -3e18, 0.0
        idx = exact_index(B, x, nq, k)
        (ids, dist), (ids1, dist1) = both_plans(B, idx, q, preds, k)
        assert bool((ids1 >= 0).all())
        for i in range(nq):
            assert torch.equal(ids[i], ids1[i]) and torch.equal(dist[i], dist1[i]), (big, i)
