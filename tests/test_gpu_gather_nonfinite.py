"""A weight that is not a number or infinite makes the gradient of its block not a number at its input, whatever the arg-max of
its line is: the gradient is a product of the weights with a matrix that is zero almost everywhere, and 0 x NaN and 0 x inf
are NaN.  The gradient pass by records leaves those products out, so it has to put this back: groups as long as the block,
groups of several blocks (whose record may lie in another block), blocks of 256 with shorter groups, either axis, both members
of a pair.  The losses of such a call are not finite."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from paper_2511_19705_amd import workloads as WL
from tests.test_gpu_single import _case, _dev

pytestmark = pytest.mark.gpu

BAD = [(3, 5, np.nan), (70, 300, np.inf), (129, 301, -np.inf)]       # (line, input, value)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


def _spoil(W, axis, bad=BAD):
    for line, a, v in bad:
        W[(line, a) if axis == O.COL else (a, line)] = v
    return W


def _mask(nb, k, rep, axis, bad=BAD):
    """Entries that are not numbers: [block][input][output] along columns, [block][output][input] along rows."""
    m = np.zeros((nb, k, k), dtype=bool)
    for _, a, _ in bad:
        b = a // k // rep
        if axis == O.COL:
            m[b, a % k, :] = True
        else:
            m[b, :, a % k] = True
    return m


# 10.6 M weights: blocks of 64 whose gradient goes by records; 0: whole channels
@pytest.mark.parametrize("k,group,lines,naxis,prepared", [(128, 128, 200, 512, False), (128, 128, 200, 512, True), (128, 256, 200, 512, True),
                                                          (128, 0, 200, 512, False), (256, 256, 144, 512, False), (256, 64, 144, 512, True),
                                                          (256, 0, 144, 512, False), (64, 256, 200, 512, False), (64, 0, 200, 512, False),
                                                          (64, 64, 2304, 4608, True)])
@pytest.mark.parametrize("axis", [O.COL, O.ROW])
@pytest.mark.parametrize("bf16", [False, True])
def test_single(env, k, group, lines, naxis, prepared, axis, bf16):
    torch, cafeq = env
    W, T, P = _case(axis, lines, naxis, k, 1, 4100 + k + group)
    Wd = _dev(torch, _spoil(W, axis))
    if bf16:
        Wd = Wd.to(torch.bfloat16)
    losses, grad, _, _ = cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), _dev(torch, P), 4, group, axis,
                                                  prepared=cafeq.prepare_weights(Wd, axis) if prepared else None)
    assert not np.isfinite(float(losses[1]))
    np.testing.assert_array_equal(np.isnan(grad.cpu().numpy()), _mask(naxis // k, k, 1, axis))


@pytest.mark.parametrize("k,group,rep", [(32, 32, 1), (64, 128, 1), (128, 128, 2), (128, 0, 1), (256, 64, 2), (256, 256, 1)])
@pytest.mark.parametrize("member", [0, 1])
def test_pair(env, k, group, rep, member):
    torch, cafeq = env
    A, B, T = WL.small_pair(136, 512, k, rep, 4200 + k + group, eps=0.05)
    P = O.block_inverse(T).astype(np.float32)
    nb = T.shape[0]
    _spoil((A, B)[member], member)
    Ad, Bd = _dev(torch, A), _dev(torch, B)
    prep = (cafeq.prepare_weights(Ad, O.COL), cafeq.prepare_weights(Bd, O.ROW))
    losses, grad, _ = cafeq.dual_proxy_loss_fwd_bwd(Ad, Bd, _dev(torch, T), _dev(torch, P), 4, group, rep, 5.0, prepared=prep)
    assert not np.isfinite(float(losses[member])) and np.isfinite(float(losses[1 - member]))
    got = np.isnan(grad.cpu().numpy())
    if member == 0:
        np.testing.assert_array_equal(got, _mask(nb, k, 1, O.COL))
    else:
        # (multiplied by the inverse on both sides: the whole block)
        np.testing.assert_array_equal(got, np.broadcast_to(_mask(nb, k, rep, O.ROW).any(axis=(1, 2), keepdims=True), got.shape))


# prepared weights, whose loss pass gives the spoiled lines the records of lines of zeros: all other sums keep their terms
def test_other_inputs_keep_their_gradient(env):
    torch, cafeq = env
    W, T, P = _case(O.COL, 200, 512, 128, 1, 4300)
    W[[3, 70]] = 0.0
    bad = [(3, a, np.nan) for a in (1, 130)] + [(70, 140, np.inf)]
    ref, got = (cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), _dev(torch, P), 4, 128, O.COL, prepared=cafeq.prepare_weights(Wd, O.COL))[1].cpu().numpy()
                for Wd in (_dev(torch, W), _dev(torch, _spoil(W.copy(), O.COL, bad))))
    nan = _mask(4, 128, 1, O.COL, bad)
    np.testing.assert_array_equal(np.isnan(got), nan)
    np.testing.assert_array_equal(got[~nan], ref[~nan])
