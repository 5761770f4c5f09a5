"""GPU parity of the gradient's way through the inverse for blocks of 128 on either side of the count from which X = P^T G passes
through LDS in parts (two workgroups of 64 rows a block, 256 compute units): evaluations against the oracle (bounds of
tests/parity.py: the arithmetic and its order are the same in both forms) and the update in the same kernel's epilogue."""
import pytest

from oracle import cafeq_oracle as O
from paper_2511_19705_amd import workloads as WL
from tests.test_gpu_prepared import _check_single_prepared
from tests.test_gpu_single import _case, _dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


@pytest.mark.parametrize("nb", [128, 129, 260])
@pytest.mark.parametrize("axis", [O.COL, O.ROW])
def test_evaluation(env, nb, axis):
    W, T, P = _case(axis, 40, nb * 128, 128, 1, 3500 + nb)
    _check_single_prepared(env, W, T, P, 4, 128, axis, 1, want_codes=False)


# one step: gradient and update in one launch equal the two calls bit for bit
@pytest.mark.parametrize("nb", [129, 260])
def test_adam_step(env, nb):
    torch, cafeq = env
    A, B, T0 = (_dev(torch, x) for x in WL.small_pair(40, nb * 128, 128, 1, 3600 + nb, eps=0.03))
    prep = (cafeq.prepare_weights(A, O.COL), cafeq.prepare_weights(B, O.ROW))
    T = T0.clone()
    cafeq.optimize_pair(A, B, T, 4, 128, 1, 5.0, 1e-3, 1, prepared=prep)
    ref, m, v = T0.clone(), torch.zeros_like(T0), torch.zeros_like(T0)
    P, _ = cafeq.block_inverse(ref)
    _, grad, _ = cafeq.dual_proxy_loss_fwd_bwd(A, B, ref, P, 4, 128, 1, 5.0, prepared=prep)
    cafeq.adam_update(ref, grad, m, v, 1, 1e-3, 0.1, 0.999, 1e-8)
    assert float((ref - T0).abs().max()) > 5e-4
    assert torch.equal(T, ref)
