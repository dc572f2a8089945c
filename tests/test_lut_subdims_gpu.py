"""Distance tables of every sub-dimension count with a fixed build (1 to 16) and
one without (17), conditioned and plain, in both precisions: the oracle's bits."""
import pytest
import torch

import oracle as O
from tests._gpu_util import assert_bitexact, say
from workload import random_index

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dsub", list(range(1, 18)))
def test_tables_match_oracle(dsub):
    from paper_2607_22922_amd import ifvs as B
    M, nq = 6, 18                                        # two query chunks of a workgroup
    say(f"[lut] dsub={dsub}")
    ix = random_index(300, M, dsub, 1, 10, 40 + dsub, device="cuda")
    idx = B.Index(ix["codes"], ix["C_pq"], ix["attrs"], ix["bank"], ix["W"], ix["r"], ix["h"], ix["hash_seed"],
                  max_batch=nq, max_k=4)
    q = torch.randn(nq, M * dsub, generator=torch.Generator(device="cuda").manual_seed(dsub), device="cuda")
    alpha, wf = idx.select_codebook(q, [[(0, 1, 5)]] * nq, 0.5 + 0.1 * q)
    n = lambda t: t.detach().cpu().numpy()
    for dt, name in ((B.LUT_F32, "f32"), (B.LUT_F16, "f16")):
        got, plain = idx.build_lut(q, alpha, wf, dt), idx.build_lut(q, None, wf, dt)
        torch.cuda.synchronize()
        for i in (0, 15, 16, 17):
            ref = O.build_lut(n(q[i]), n(alpha[i]), n(wf[i]), n(ix["C_pq"]), n(ix["W"]), M, ix["r"], lut_dtype=name)
            assert_bitexact(n(got[i]), ref, f"dsub={dsub} {name} q{i}")
            ref = O.build_lut(n(q[i]), 0 * n(alpha[i]), n(wf[i]), n(ix["C_pq"]), 0 * n(ix["W"]), M, ix["r"],
                              lut_dtype=name)
            assert_bitexact(n(plain[i]), ref, f"plain dsub={dsub} {name} q{i}")
