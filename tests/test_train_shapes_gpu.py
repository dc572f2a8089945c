"""The training step at the shapes where its kernels branch: sub-dimension
counts with and without a fixed build (2, 4, 8; 3), candidate lists whose code
words fit the LDS beside the table and ones that do not, more (query, hash)
pairs than the bank update compares at once, query counts below and off the
four quarters of the W update."""
import pytest
import torch

from tests._gpu_util import say
from tests.test_train_gpu import LR, _close, _np, _oracle, _problem

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2607_22922_amd import ifvs
    return ifvs


@pytest.mark.parametrize("M,dsub,nq,n_cand,n_pos,bank_rows", [
    (16, 8, 13, 24, 4, 32), (12, 3, 5, 7, 2, 32), (48, 2, 4, 2900, 6, 32), (5, 2, 150, 12, 2, 7), (9, 4, 4, 8, 1, 3)])
def test_train_step_shapes(B, M, dsub, nq, n_cand, n_pos, bank_rows):
    say(f"[train] M={M} dsub={dsub} nq={nq} n_cand={n_cand} bank={bank_rows}")
    idx, ix, q, w_z, cand, preds, n_pos = _problem(B, 3 + M, M, dsub, (0,), nq=nq, n_cand=n_cand, n_pos=n_pos,
                                                   bank_rows=bank_rows)
    tau, lam = 0.8, 0.05
    ref = _oracle(ix, q, w_z, cand, preds, n_pos, tau, lam)
    bank0, W0 = idx.read_params()
    loss, dwz = idx.train_step(q, preds, w_z, cand, n_pos, tau, lam, LR, want_dwz=True)
    bank1, W1 = idx.read_params()
    torch.cuda.synchronize()
    _close(_np(loss), ref["loss"], "loss", rel=1e-4)
    _close(_np((bank0 - bank1) / LR), ref["bank"], "bank gradient")
    _close(_np((W0 - W1) / LR), ref["W"], "W gradient")
    _close(_np(dwz), ref["w_z"], "w_z gradient")


def test_train_step_at_the_lds_limit(B):
    """The largest candidate list that 160 KB hold beside the table and the
    gradients: (M 256 + n_cand + 4 D + 4 M r) floats; one more is refused."""
    M, dsub, n_cand = 128, 1, 3584
    say(f"[train] LDS limit M={M} n_cand={n_cand}")
    idx, ix, q, w_z, cand, preds, n_pos = _problem(B, 11, M, dsub, (), nq=5, n_cand=n_cand, n_pos=5)
    assert 4 * (M * 256 + n_cand + 4 * M * dsub + 4 * M * ix["r"]) == 160 * 1024
    tau, lam = 0.8, 0.05
    ref = _oracle(ix, q, w_z, cand, preds, n_pos, tau, lam)
    bank0, W0 = idx.read_params()
    loss, dwz = idx.train_step(q, preds, w_z, cand, n_pos, tau, lam, LR, want_dwz=True)
    bank1, W1 = idx.read_params()
    torch.cuda.synchronize()
    _close(_np(loss), ref["loss"], "loss", rel=1e-4)
    _close(_np((bank0 - bank1) / LR), ref["bank"], "bank gradient")
    _close(_np((W0 - W1) / LR), ref["W"], "W gradient")
    _close(_np(dwz), ref["w_z"], "w_z gradient")
    more = torch.cat([cand, cand[:, :1]], 1).contiguous()
    with pytest.raises(B.IfvsError) as e:
        idx.train_step(q, preds, w_z, more, n_pos, tau, lam, LR)
    assert e.value.status == B.E_UNSUPPORTED
