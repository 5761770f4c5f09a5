"""Gradient descent at two bits keeps one gradient pass on every path of the loop -- the update in the gradient's last kernel, updates as
calls of their own beside a regulariser, transform blocks below 32 -- where an evaluation takes the gradient by records.  A
regulariser of weight 1e-30 adds nothing to a gradient that is not zero: its loop's steps equal the plain loop's bit for bit."""
import pytest

from oracle import cafeq_oracle as O
from paper_2511_19705_amd import workloads as WL
from tests.test_gpu_single import _case, _dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


@pytest.mark.parametrize("bits", [2, 3])
@pytest.mark.parametrize("k,group,mode", [(128, 128, 0), (128, 0, 0), (256, 64, 0), (128, 128, 1), (64, 0, 0)])
def test_with_and_without_a_regulariser(env, bits, k, group, mode):
    torch, cafeq = env
    W, T0, _ = _case(O.COL, 333, 768, k, 1, 6100 + k + group)
    ends = []
    for lam in (0.0, 1e-30):
        T = _dev(torch, T0)
        cafeq.optimize_single(_dev(torch, W), T, bits, group, O.COL, 1, 0.5, 1, lam, mode=mode)
        ends.append(T)
    assert torch.equal(ends[0], ends[1]) and not torch.equal(ends[0], _dev(torch, T0))


# from three bits on a loop's step is the evaluation's gradient and the update, bit for bit
@pytest.mark.parametrize("k,group", [(128, 128), (128, 0), (256, 64), (64, 0)])
def test_three_bits_take_the_evaluations_gradient(env, k, group):
    torch, cafeq = env
    W, T0, _ = _case(O.COL, 333, 768, k, 1, 6200 + k + group)
    Wd, T, ref = _dev(torch, W), _dev(torch, T0), _dev(torch, T0)
    cafeq.optimize_single(Wd, T, 3, group, O.COL, 1, 0.5, 1)
    P, _ = cafeq.block_inverse(ref)
    losses, grad, _, _ = cafeq.proxy_loss_fwd_bwd(Wd, ref, P, 3, group, O.COL)
    cafeq.sgd_update(ref, grad / losses[2], 0.5)
    assert torch.equal(T, ref)


# blocks of 16 are run as blocks of 32, whose gradient goes by records from 10 M weights on: a pass over the weights of its own
@pytest.mark.parametrize("bits,passes", [(2, 0), (3, 1)])
def test_small_blocks(env, bits, passes):
    torch, cafeq = env
    W = _dev(torch, WL.student_t3((4888, 2048), 6300))
    T = _dev(torch, WL.perturbed_blocks(128, 16, 6301, 0.03))
    timer = cafeq.LaunchTimer(4, kind=1)
    with timer:
        cafeq.optimize_single(W, T, bits, 64, O.COL, 1, 0.5, 1)
        torch.cuda.synchronize()
    assert timer.table.seen == passes
