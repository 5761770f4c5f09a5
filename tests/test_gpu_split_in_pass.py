"""Loss passes over prepared weights that split their operand planes themselves (single matrices at blocks of 64 and pairs at blocks of 64
and 128, without codes) against the calls that write codes, whose planes a launch of its own has split: the same bits where both deal
their tiles alike (single matrices), else what another order of float32 sums leaves.  Blocks of very different magnitude, a block of
zeros, infinite entries of a block."""
import numpy as np
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


def _spread_blocks(T, P, spread):
    """Every other block `spread` times smaller; one block of zeros (its inverse stays what it was: nothing here inverts it)."""
    T, P = T.copy(), P.copy()
    T[::2] /= np.float32(spread)
    P[::2] *= np.float32(spread)
    T[3] = 0.0
    return T, P


@pytest.mark.parametrize("axis,rep,bf16", [(O.COL, 1, False), (O.COL, 1, True), (O.ROW, 1, True), (O.ROW, 2, True)])
@pytest.mark.parametrize("spread", [1.0, 2.0 ** 12, 2.0 ** 30])
def test_single(env, axis, rep, bf16, spread):
    torch, cafeq = env
    W, T, P = _case(axis, 3400, 2048, 64, rep, 9000 + rep)
    T, P = (_dev(torch, x) for x in _spread_blocks(T, P, spread))
    W = _dev(torch, W).to(torch.bfloat16 if bf16 else torch.float32)
    prep = cafeq.prepare_weights(W, axis)
    a, b = (cafeq.proxy_loss_fwd_bwd(W, T, P, 4, 128, axis, rep, want_grad=False, want_codes=codes, prepared=prep)[0].cpu().numpy() for codes in (False, True))
    assert np.isfinite(a).all()
    np.testing.assert_array_equal(a[:3], b[:3])
    np.testing.assert_allclose(a[3], b[3], rtol=1e-6)              # (rho's sums in another order)


@pytest.mark.parametrize("k,group,rep", [(64, 128, 1), (64, 64, 2), (128, 128, 1), (128, 64, 2)])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("spread", [1.0, 2.0 ** 12])
def test_pair(env, k, group, rep, bf16, spread):
    torch, cafeq = env
    A, B, T = WL.small_pair(3400, 2048 // rep, k, rep, 9100 + k + group, eps=0.05)
    P = O.block_inverse(T).astype(np.float32)
    T, P = (_dev(torch, x) for x in _spread_blocks(T, P, spread))
    A, B = (_dev(torch, x).to(torch.bfloat16 if bf16 else torch.float32) for x in (A, B))
    prep = (cafeq.prepare_weights(A, O.COL), cafeq.prepare_weights(B, O.ROW))
    a, b = ([x.cpu().numpy() for x in cafeq.dual_proxy_loss_fwd_bwd(A, B, T, P, 3, group, rep, 5.0, (k, group) == (128, 128), codes, prepared=prep)[:2] if x is not None]
            for codes in (False, True))
    assert all(np.isfinite(x).all() for x in a)
    np.testing.assert_allclose(a[0], b[0], rtol=2e-6)
    if len(a) > 1:
        for x, y in zip(a[1], b[1]):                                # (block by block: their magnitudes differ)
            assert np.abs(x - y).max() <= 1e-5 * np.abs(y).max()


def _infinite_output(T, k):
    """Output 2 of block 3 takes nothing but input 1, at which it has an infinite entry or (the other copy) none."""
    T = T.copy()
    T[3, :, 2] = 0.0
    U = T.copy()
    T[3, 1, 2] = np.inf
    return T, U


# The weights at that input are zeros: the output is 0 x inf, not a number, and no group's largest value; everything else of the block has
# the values that it has without the entry, which would be lost if the entry set the block's scale.
@pytest.mark.parametrize("bf16", [False, True])
def test_infinite_entry_single(env, bf16):
    torch, cafeq = env
    W, T, P = _case(O.COL, 4200, 2048, 64, 1, 9200)
    W[:, 3 * 64 + 1] = 0.0
    W = _dev(torch, W).to(torch.bfloat16 if bf16 else torch.float32)
    prep, P = cafeq.prepare_weights(W, O.COL), _dev(torch, P)
    out = [cafeq.proxy_loss_fwd_bwd(W, _dev(torch, X), P, 4, 128, O.COL, prepared=prep)[:2] for X in _infinite_output(T, 64)]
    assert not torch.isfinite(out[0][0][0]) and torch.isfinite(out[1][0]).all()
    assert torch.equal(out[0][0][2:], out[1][0][2:])                # ||W||^2, the surrogate
    assert torch.equal(out[0][1], out[1][1])                        # the gradient: the groups' largest values and where they are


@pytest.mark.parametrize("k", [64, 128])
@pytest.mark.parametrize("bf16", [False, True])
def test_infinite_entry_pair(env, k, bf16):
    torch, cafeq = env
    A, B, T = WL.small_pair(1400, 1024, k, 1, 9300 + k, eps=0.05)
    P = O.block_inverse(T).astype(np.float32)
    A[:, 3 * k + 1] = 0.0
    A, B = (_dev(torch, x).to(torch.bfloat16 if bf16 else torch.float32) for x in (A, B))
    prep, P = (cafeq.prepare_weights(A, O.COL), cafeq.prepare_weights(B, O.ROW)), _dev(torch, P)
    out = [cafeq.dual_proxy_loss_fwd_bwd(A, B, _dev(torch, X), P, 3, 128, 1, 5.0, True, False, prepared=prep)[:2] for X in _infinite_output(T, k)]
    assert not torch.isfinite(out[0][0][0]) and torch.isfinite(out[1][0]).all()
    assert torch.equal(out[0][0][4], out[1][0][4])                  # LSE
    assert torch.equal(out[0][1], out[1][1])
