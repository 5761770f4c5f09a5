"""GPU parity of the loss pass over blocks of 32 with groups of 32 where a workgroup walks several macro-tiles: ranges that end inside a
segment, with one and across several, in both axes, shared row-blocks among them, every output it writes; and weights that are not
finite, whose products with the gradient's zeros are not numbers either.  Against the oracle, with the bounds of tests/parity.py."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from paper_2511_19705_amd import workloads as WL
from tests import parity
from tests.test_gpu_dual import _check_dual
from tests.test_gpu_single import _case, _check_single, _dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


# macro-tiles of 128 lines on two workgroups a compute unit (512): 3 a segment x 200, 1 x 550, 14 x 40
@pytest.mark.parametrize("axis,lines,naxis,rep", [(O.COL, 300, 6400, 1), (O.ROW, 100, 17600, 1), (O.ROW, 1700, 1280, 2), (O.COL, 2900, 800, 1)])
def test_single(env, axis, lines, naxis, rep):
    W, T, P = _case(axis, lines, naxis, 32, rep, 9300 + lines)
    _check_single(env, W, T, P, 4, 32, axis, rep)


def test_pair(env):
    A, B, T = WL.small_pair(300, 6400, 32, 1, 9400, eps=0.05)
    _check_dual(env, A, B, T, 3, 32, 1, flip_slack=True)


@pytest.mark.parametrize("axis", [O.COL, O.ROW])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_not_finite(env, axis, value):
    torch, cafeq = env
    W, T, P = _case(axis, 200, 128, 32, 1, 9500)
    W[(70, 45) if axis == O.COL else (45, 70)] = value            # input 13 of block 1
    losses, grad, _, _ = cafeq.proxy_loss_fwd_bwd(_dev(torch, W), _dev(torch, T), _dev(torch, P), 4, 32, axis)
    assert not np.isfinite(losses.cpu().numpy()[1])
    bad = ~np.isfinite(grad.cpu().numpy())
    if axis == O.ROW:
        bad = bad.transpose(0, 2, 1)
    assert bad[1, 13].all() and not bad[[0, 2, 3]].any()


@pytest.mark.parametrize("lr", [0.5, 200.0])
@pytest.mark.parametrize("axis", [O.COL, O.ROW])
def test_loop_against_its_steps(env, axis, lr):
    """The loop's last kernel of a step leaves the next inverse, from the one before (at the larger rate blocks leave Newton's reach and are
    eliminated); each step's losses and transform against calls that take every inverse from scratch.  The two inverses differ by float32
    rounding; a gradient by 1e-6 of itself."""
    torch, cafeq = env
    W, T, _ = _case(axis, 300, 256, 32, 1, 9600, eps=0.2)
    W, T = _dev(torch, W), _dev(torch, T)
    steps, mine = 4, T.clone()
    P, history, status = cafeq.optimize_single(W, mine, 4, 32, axis, lr=lr, steps=steps)
    for s in range(steps):
        Q, st = cafeq.block_inverse(T)
        losses, grad, _, _ = cafeq.proxy_loss_fwd_bwd(W, T, Q, 4, 32, axis)
        np.testing.assert_allclose(history[s, :4].cpu().numpy(), losses.cpu().numpy(), rtol=1e-4)
        cafeq.sgd_update(T, grad, lr, losses[2:3])
    np.testing.assert_allclose(mine.cpu().numpy(), T.cpu().numpy(), rtol=0, atol=1e-4 * float(T.abs().max()))
    Q, st = cafeq.block_inverse(mine)
    assert torch.equal(P, Q) and torch.equal(status, st)


# a group without a number counts as a largest magnitude of zero at its entry 4 (as in the kernel for other blocks and groups): what its line's
# other inputs add to the pair's gradient, by the loss pass itself and, over prepared weights, by records
@pytest.mark.parametrize("prepared", [False, True])
def test_group_without_a_number(env, prepared):
    torch, cafeq = env
    A, B, T = WL.small_pair(136, 128, 32, 1, 9450, eps=0.05)
    P = O.block_inverse(T).astype(np.float32)
    line, block, m0 = 70, 2, 13
    Az = A.copy()
    Az[line, 32 * block:32 * block + 32] = 0.0
    ref = O.dual_lse(Az, B, T, P, 4, 32, 1, 5.0)
    want = ref["gradT"].copy()
    want[block, :, 4] += np.exp(-5.0 * ref["lse"]) * A[line, 32 * block:32 * block + 32].astype(np.float64)
    A[line, 32 * block + m0] = np.nan
    Ad, Bd = _dev(torch, A), _dev(torch, B)
    prep = (cafeq.prepare_weights(Ad, O.COL), cafeq.prepare_weights(Bd, O.ROW)) if prepared else (None, None)
    _, grad, _ = cafeq.dual_proxy_loss_fwd_bwd(Ad, Bd, _dev(torch, T), _dev(torch, P), 4, 32, 1, 5.0, prepared=prep)
    got = grad.cpu().numpy()
    assert np.isnan(got[block, m0]).all() and np.isnan(got).sum() == 32
    got[block, m0] = want[block, m0]
    parity.check_grad(got, want)
