"""GPU parity where a launch has one workgroup per macro-tile and their number is no multiple of eight: ranges are then dealt in the
order of the workgroups, segments end inside and at the end of a range, and a pair's second member starts at any workgroup.  Against
the oracle, with the bounds of tests/parity.py."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from paper_2511_19705_amd import workloads as WL
from tests import parity
from tests.test_gpu_dual import _check_dual
from tests.test_gpu_prepared import _check_single_prepared
from tests.test_gpu_single import _case, _check_single, _dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


# macro-tiles of 128 lines: 9, 27, 11 x 2, 13 (and 9 of 256 lines, 18 with two a segment, for prepared weights)
@pytest.mark.parametrize("k,group,lines,naxis,axis", [(128, 128, 120, 1152, O.COL), (64, 128, 300, 1152, O.ROW), (32, 32, 132, 1408, O.COL),
                                                      (256, 64, 100, 3328, O.ROW)])
def test_single(env, k, group, lines, naxis, axis):
    W, T, P = _case(axis, lines, naxis, k, 1, 8000 + k)
    _check_single(env, W, T, P, 4, group, axis, 1)
    if k == 128:
        _check_single_prepared(env, W, T, P, 4, group, axis, 1, want_codes=False)


@pytest.mark.parametrize("k,group,lines,naxis", [(128, 128, 200, 1152), (128, 64, 300, 1664), (64, 64, 264, 1152)])
@pytest.mark.parametrize("prepared", [False, True])
def test_pair(env, k, group, lines, naxis, prepared):
    torch, cafeq = env
    A, B, T = WL.small_pair(lines, naxis, k, 1, 8100 + lines, eps=0.05)
    if not prepared:
        _check_dual(env, A, B, T, 3, group, 1, flip_slack=True)
        return
    P = O.block_inverse(T).astype(np.float32)
    Ad, Bd = _dev(torch, A), _dev(torch, B)
    prep = (cafeq.prepare_weights(Ad, O.COL), cafeq.prepare_weights(Bd, O.ROW))
    losses, grad, _ = cafeq.dual_proxy_loss_fwd_bwd(Ad, Bd, _dev(torch, T), _dev(torch, P), 3, group, 1, 5.0, True, False, prepared=prep)
    losses = losses.cpu().numpy().astype(np.float64)
    ref = O.dual_lse(A, B, T, P, 3, group, 1, 5.0)
    for i, name in enumerate(("errU_sq", "errV_sq", "l2A_sq", "l2B_sq", "lse")):
        parity.check_scalar(losses[i], ref[name], what=name)
    slack, n_amb = parity.dual_argmax_flip_slack(A, B, T, P, ref, group, 1, 5.0)
    assert n_amb <= 3
    parity.check_grad_with_slack(grad.cpu().numpy(), ref["gradT"], slack)
