"""Which of the ways an evaluation takes (gradient by records or beside the loss pass or as a product; loss pass over prepared weights
or the general one), on either side of the sizes from which one is the faster: the launches that the timing table counts, and
losses and gradient against the oracle on both sides (bounds of tests/parity.py)."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from paper_2511_19705_amd import workloads as WL
from tests import parity
from tests.test_gpu_single import _case, _dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


def _launches(torch, cafeq, kind, call):
    timer = cafeq.LaunchTimer(8, kind=kind)
    with timer:
        out = call()
        torch.cuda.synchronize()
    return out, timer.table.seen


def _single(env, W, T, P, bits, group, axis, prepared, bf16=False):
    torch, cafeq = env
    if bf16:
        b16 = WL.to_bf16_bits(W)
        W, Wd = WL.bf16_bits_to_f32(b16), _dev(torch, b16.view(np.int16)).view(torch.bfloat16)
    else:
        Wd = _dev(torch, W)
    prep = cafeq.prepare_weights(Wd, axis) if prepared else None
    (losses, grad, _, _), n = _launches(torch, cafeq, 1, lambda: cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), _dev(torch, P), bits, group, axis,
                                                                                          prepared=prep))
    sur, g_ref = O.surrogate(W, T, P, bits, group, axis, 1)
    parity.check_scalar(float(losses[3]), sur, what="surrogate")
    parity.check_grad(grad.cpu().numpy(), g_ref)
    return n


# blocks of 32 and 64: the gradient passes over the weights (none: the loss pass forms it on its way).  From 10 M weights on, and
# 2048 axis indices (groups of 128 over prepared weights: 8 M, 1024); 8 bits and plain weights: records of the general kernel.  Blocks of 32 with
# groups of 32, whose loss pass is a kernel of its own: on its way at every size but in bfloat16 along rows from 50 M
@pytest.mark.parametrize("k,group,bits,lines,naxis,axis,prepared,bf16,passes", [
    (32, 32, 4, 4100, 2048, O.COL, True, False, 0), (32, 32, 4, 4888, 2048, O.COL, True, False, 0), (32, 32, 4, 4888, 2048, O.ROW, True, True, 0), (32, 64, 8, 4888, 2048, O.COL, True, False, 1),
    (64, 64, 4, 4888, 2048, O.COL, False, False, 1), (64, 128, 8, 4888, 2048, O.ROW, True, False, 1), (32, 128, 4, 4888, 2048, O.ROW, True, True, 1),
    (64, 64, 4, 9800, 1024, O.COL, False, False, 0), (64, 128, 4, 8200, 1024, O.COL, True, False, 1), (64, 64, 4, 8200, 1024, O.COL, True, True, 1)])
def test_on_the_way_or_by_records(env, k, group, bits, lines, naxis, axis, prepared, bf16, passes):
    W, T, P = _case(axis, lines, naxis, k, 1, 5100 + k + group)
    assert _single(env, W, T, P, bits, group, axis, prepared, bf16) == passes


# ... and where that line lies (the way alone; records of bfloat16 weights along rows against the oracle: above)
@pytest.mark.parametrize("lines,passes", [(24408, 0), (24416, 1)])
def test_rows_in_bfloat16(env, lines, passes):
    torch, cafeq = env
    W = torch.randn((2048, lines), generator=torch.Generator(device="cuda:0").manual_seed(5150), device="cuda:0").to(torch.bfloat16)
    T = _dev(torch, WL.perturbed_blocks(64, 32, 5151, 0.05))
    P, _ = cafeq.block_inverse(T)
    prep = cafeq.prepare_weights(W, O.ROW)
    assert _launches(torch, cafeq, 1, lambda: cafeq.proxy_loss_fwd_bwd(W, T, P, 4, 32, O.ROW, prepared=prep))[1] == passes


# blocks of 256 with groups of 32: eight reads of every line, or the product; blocks of 128: lines and axis indices.  Either way one pass
@pytest.mark.parametrize("k,group,lines,naxis,axis,prepared,bf16", [(256, 32, 200, 512, O.COL, False, False), (256, 32, 200, 512, O.ROW, True, True),
                                                                   (256, 32, 12400, 512, O.COL, False, False), (256, 64, 33000, 256, O.COL, False, False),
                                                                   (128, 128, 16400, 512, O.COL, False, False), (128, 128, 16400, 256, O.ROW, True, False),
                                                                   (128, 128, 16400, 512, O.COL, True, True)])
def test_few_blocks_of_many_lines(env, k, group, lines, naxis, axis, prepared, bf16):
    W, T, P = _case(axis, lines, naxis, k, 1, 5200 + k + group)
    assert _single(env, W, T, P, 4, group, axis, prepared, bf16) == 1


# pairs: a pass per member (product), one for both (records), none (beside the loss passes)
@pytest.mark.parametrize("k,group,rep,lines,d_mid,bits,passes", [(256, 32, 1, 136, 512, 4, 1), (256, 32, 2, 136, 256, 8, 1), (256, 32, 1, 6200, 256, 4, 2),
                                                                 (32, 32, 1, 136, 512, 8, 1), (64, 64, 1, 136, 512, 8, 1), (32, 32, 1, 1544, 256, 4, 0),
                                                                 (32, 64, 1, 1544, 256, 4, 1), (128, 128, 1, 16400, 384, 4, 2)])
def test_pairs(env, k, group, rep, lines, d_mid, bits, passes):
    torch, cafeq = env
    A, B, T = WL.small_pair(lines, d_mid, k, rep, 5300 + k + group, eps=0.05)
    P = O.block_inverse(T).astype(np.float32)
    Ad, Bd, Td, Pd = (_dev(torch, x) for x in (A, B, T, P))
    prep = (cafeq.prepare_weights(Ad, O.COL), cafeq.prepare_weights(Bd, O.ROW))
    (losses, grad, _), n = _launches(torch, cafeq, 1, lambda: cafeq.dual_proxy_loss_fwd_bwd(Ad, Bd, Td, Pd, bits, group, rep, 5.0, prepared=prep))
    assert n == passes
    ref = O.dual_lse(A, B, T, P, bits, group, rep, 5.0)
    for i, name in enumerate(("errU_sq", "errV_sq", "l2A_sq", "l2B_sq", "lse")):
        parity.check_scalar(float(losses[i]), ref[name], what=name)
    slack, _ = parity.dual_argmax_flip_slack(A, B, T, P, ref, group, rep, 5.0)
    parity.check_grad_with_slack(grad.cpu().numpy(), ref["gradT"], slack)


# losses and codes of blocks of 32 and 64: where the general kernel is the faster one a prepared copy changes nothing, bit for bit
@pytest.mark.parametrize("k,group,axis,lines,naxis,bf16", [(32, 32, O.COL, 1152, 512, False), (32, 32, O.COL, 1152, 512, True), (64, 64, O.COL, 1152, 512, False),
                                                           (32, 32, O.ROW, 1152, 512, True), (32, 128, O.COL, 4608, 256, False), (32, 64, O.COL, 304, 4096, False), (64, 128, O.ROW, 4608, 256, False)])
@pytest.mark.parametrize("codes", [False, True])
def test_small_forward(env, k, group, axis, lines, naxis, bf16, codes):
    torch, cafeq = env
    W, T, P = _case(axis, lines, naxis, k, 1, 5400 + k + group)
    Wd = _dev(torch, W)
    if bf16:
        Wd = Wd.to(torch.bfloat16)
    a, b = (cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), _dev(torch, P), 4, group, axis, want_grad=False, want_codes=codes, prepared=p)
            for p in (cafeq.prepare_weights(Wd, axis), None))
    for x, y in zip(a, b):
        assert (x is None) == (y is None) and (x is None or torch.equal(x, y))


# pairs without codes: both members in one launch over prepared weights, or one launch of the general kernel each
@pytest.mark.parametrize("k,group,lines,d_mid,launches", [(32, 32, 600, 512, 2), (32, 32, 4608, 1024, 1), (32, 64, 256, 2304, 2), (32, 64, 136, 512, 1),
                                                          (64, 64, 136, 512, 1), (32, 128, 136, 512, 1)])
def test_small_forward_pairs(env, k, group, lines, d_mid, launches):
    torch, cafeq = env
    A, B, T = WL.small_pair(lines, d_mid, k, 1, 5500 + k + group, eps=0.05)
    P = O.block_inverse(T).astype(np.float32)
    Ad, Bd, Td, Pd = (_dev(torch, x) for x in (A, B, T, P))
    prep = (cafeq.prepare_weights(Ad, O.COL), cafeq.prepare_weights(Bd, O.ROW))
    (losses, _, _), n = _launches(torch, cafeq, 0, lambda: cafeq.dual_proxy_loss_fwd_bwd(Ad, Bd, Td, Pd, 4, group, 1, 5.0, want_grad=False, prepared=prep))
    assert n == launches
    ref = O.dual_lse(A, B, T, P, 4, group, 1, 5.0, want_grad=False)
    for i, name in enumerate(("errU_sq", "errV_sq", "l2A_sq", "l2B_sq", "lse")):
        parity.check_scalar(float(losses[i]), ref[name], what=name)
