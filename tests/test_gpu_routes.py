"""Which of the ways an evaluation takes (loss pass over prepared weights or the general one), on either side of the sizes from which
one is the faster: the launches that the timing table counts, and losses against the oracle on both sides (bounds of tests/parity.py)."""
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
