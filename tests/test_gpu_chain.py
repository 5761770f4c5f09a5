"""GPU parity of the gradient's way through the inverse for blocks of 128 on either side of the count from which two workgroups share
a compute unit (two workgroups of 64 rows a block, 256 compute units): evaluations against the oracle (bounds of tests/parity.py) and
the update in the same kernel's epilogue; and gradients near the end of float32's range."""
import numpy as np
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


# a power of two common to the weights: squared in the gradient, whose entries (2^-118 in the root mean square) still are numbers with 24
# bits, and of which bfloat16 (down to 2^-133) would keep 15.  Sums and products keep their bits but for what ends below 2^-149: 2^-31
# of an entry
@pytest.mark.parametrize("nb", [4, 130])
@pytest.mark.parametrize("axis,group", [(O.COL, 128), (O.ROW, 128), (O.COL, 0)])
def test_small_weights(env, nb, axis, group):
    torch, cafeq = env
    W, T, P = _case(axis, 40, nb * 128, 128, 1, 3700 + nb)
    grads = []
    for e in (0, -55):
        losses, grad, _, _ = cafeq.proxy_loss_fwd_bwd(_dev(torch, W * np.float32(2.0 ** e)), _dev(torch, T), _dev(torch, P), 4, group, axis)
        grads.append(grad.double() * 2.0 ** (-2 * e))
    assert float((grads[1] - grads[0]).norm() / grads[0].norm()) < 1e-7
