"""GPU parity of the pass over blocks of 256 whose groups lie inside a block (csrc/xform256.hip): two waves share a strip of 32
lines, so row counts around its strips and macro-tiles of 128, every group length (256: one group for both waves), both axes, shared
blocks, bfloat16 storage, grids of 2 to 8 bits; lines and blocks of any magnitude, entries far below the rest of their line or block;
transforms that only move weights."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from paper_2511_19705_amd import workloads as WL
from tests import parity
from tests.test_gpu_single import _case, _check_single, _dev

pytestmark = pytest.mark.gpu
K = 256


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


@pytest.mark.parametrize("group,lines,axis,rep,bits,bf16", [
    (32, 4, O.COL, 1, 4, False), (64, 32, O.ROW, 1, 3, False), (128, 36, O.COL, 1, 2, False), (256, 128, O.ROW, 2, 4, False),
    (256, 132, O.COL, 1, 3, False), (64, 260, O.ROW, 2, 8, False), (128, 300, O.COL, 1, 8, True), (32, 392, O.ROW, 1, 2, True),
    (64, 1, O.COL, 1, 4, True), (256, 96, O.COL, 1, 8, False)])
def test_ragged_lines_and_groups(env, group, lines, axis, rep, bits, bf16):
    W, T, P = _case(axis, lines, 1024, K, rep, 7000 + group + lines)
    _check_single(env, W, T, P, bits, group, axis, rep, bf16=bf16)


@pytest.mark.parametrize("axis", [O.COL, O.ROW])
def test_magnitudes(env, axis):
    """Lines of zeros, of one entry and scaled over 24 orders of magnitude; a transform of 1e-6 (bounds relative to each line)."""
    torch, cafeq = env
    W, T, P = _case(axis, 136, 512, K, 1, 7100)
    L = W if axis == O.COL else W.T
    L *= (10.0 ** np.linspace(-12, 12, 136)[:, None]).astype(np.float32)
    L[5], L[6, 1:] = 0.0, 0.0
    T = (T * 1e-6).astype(np.float32)
    P = O.block_inverse(T).astype(np.float32)
    Z = cafeq.apply_transform(_dev(torch, W), _dev(torch, T), _dev(torch, P), axis, cafeq.SIDE_T, 1).cpu().numpy()
    ref = O.blockdiag_apply(W, T, axis, 1)
    bound = O.blockdiag_apply(np.abs(W), np.abs(T), axis, 1) * (K * 2.0 ** -24)
    assert np.all(np.abs(Z - ref) <= bound + 1e-300)
    losses, _, codes, scales = cafeq.proxy_loss_fwd_bwd(_dev(torch, W), _dev(torch, T), _dev(torch, P), 4, 64, axis, want_grad=False, want_codes=True)
    c_ref, s_ref, _ = O.rtn_sym(ref, 4, 64, axis)
    parity.check_scales(scales.cpu().numpy(), s_ref)
    parity.check_codes(codes.cpu().numpy(), c_ref, ref, s_ref, axis, 64, tie_tol=parity.tie_tolerance(W, T, axis, 1, ref, s_ref, 64, parity.forward_unit(K, 64, 4)))
    parity.check_scalar(float(losses[0]), O.proxy_l2(W, T, P, 4, 64, axis, 1)["l2_sq"], what="l2_sq")


@pytest.mark.parametrize("axis,group", [(O.COL, 64), (O.ROW, 256)])
def test_moved_weights_are_moved_exactly(env, axis, group):
    """Signed permutations: the moved weights, their codes and scales are those of the moved matrix, bit for bit."""
    torch, cafeq = env
    rng = np.random.default_rng(7200)
    T = np.stack([np.eye(K)[rng.permutation(K)] * rng.choice([-1.0, 1.0], (K, 1)) for _ in range(2)]).astype(np.float32)
    P = np.ascontiguousarray(T.transpose(0, 2, 1))
    W = WL.student_t3((200, 2 * K) if axis == O.COL else (2 * K, 200), 7201)
    moved = O.blockdiag_apply(W, T, axis, 1).astype(np.float32)
    for side, M in ((cafeq.SIDE_T, T), (cafeq.SIDE_TINV, P)):
        Z = cafeq.apply_transform(_dev(torch, W), _dev(torch, T), _dev(torch, P), axis, side, 1)
        np.testing.assert_array_equal(Z.cpu().numpy(), O.blockdiag_apply(W, M, axis, 1).astype(np.float32))
    _, _, codes, scales = cafeq.proxy_loss_fwd_bwd(_dev(torch, W), _dev(torch, T), _dev(torch, P), 4, group, axis, want_grad=False, want_codes=True)
    c_ref, s_ref, _ = O.rtn_sym(moved, 4, group, axis)
    np.testing.assert_array_equal(scales.cpu().numpy(), s_ref.astype(np.float32))
    np.testing.assert_array_equal(codes.cpu().numpy(), c_ref)


def _spread(shape, axis, unit, seed, lo, hi):
    """Gaussian weights; runs of `unit` indices along the axis are scaled by 2^lo to 2^hi, each by itself, but for the first of a block."""
    rng = np.random.default_rng(seed)
    W = rng.standard_normal(shape).astype(np.float32)
    L = W if axis == O.COL else W.T
    e = rng.integers(lo, hi + 1, (L.shape[0], L.shape[1] // unit))
    e[:, ::K // unit] = 0
    L *= np.exp2(np.repeat(e, unit, axis=1)).astype(np.float32)
    return W


@pytest.mark.parametrize("axis", [O.COL, O.ROW])
def test_entries_far_below_their_line_or_block(env, axis):
    """|err| <= K 2^-24 (|W| . |T|) elementwise (the bound of tests/parity.py) for weights and for rows and columns of a transform block
    down to 2^-60 of the largest beside them; a permutation moves such weights bit for bit."""
    torch, cafeq = env
    rng = np.random.default_rng(7400)
    W = _spread((140, 2 * K) if axis == O.COL else (2 * K, 140), axis, 1, 7401, -60, 0)
    perm = np.stack([np.eye(K)[rng.permutation(K)] for _ in range(2)]).astype(np.float32)
    dense = rng.standard_normal((2, K, K)).astype(np.float32)
    e = np.exp2(rng.integers(-60, 1, (2, K))).astype(np.float32)
    for T in (perm, dense, dense * e[:, :, None], dense * e[:, None, :]):
        T = np.ascontiguousarray(T)
        Z = cafeq.apply_transform(_dev(torch, W), _dev(torch, T), _dev(torch, T), axis, cafeq.SIDE_T, 1).cpu().numpy()
        ref = O.blockdiag_apply(W, T, axis, 1)
        if T is perm or np.array_equal(T, perm):
            np.testing.assert_array_equal(Z, ref.astype(np.float32))
        assert np.all(np.abs(Z - ref) <= O.blockdiag_apply(np.abs(W), np.abs(T), axis, 1) * (K * 2.0 ** -24))


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("axis,group,below", [(O.COL, 32, 45), (O.ROW, 64, 20), (O.COL, 128, 20), (O.ROW, 128, 45)])
def test_groups_far_below_their_line(env, axis, group, below, bf16):
    """Groups 2^-20 or 2^-45 of the line's largest, under rotations that do not mix them with it: codes, scales, losses and gradient.  The
    largest ones lie on the grid, so that the losses are the small ones' errors alone."""
    W = _spread((136, 2 * K) if axis == O.COL else (2 * K, 136), axis, group, 7500 + group, -below - 2, -below)
    sub = WL.haar_blocks(2 * K // group, group, 7501)
    T = np.zeros((2, K, K), dtype=np.float32)
    for i in range(2 * K // group):
        j = slice(i % (K // group) * group, (i % (K // group) + 1) * group)
        T[i // (K // group), j, j] = sub[i] if i % (K // group) else np.eye(group)
    L = W if axis == O.COL else W.T
    for b in range(2):
        head = L[:, b * K:b * K + group]                   # (the unmixed run: multiples of the step, largest 7 of them)
        head[:] = np.clip(np.rint(head * 2), -6, 6) / 8
        head[:, 0] = 7 / 8
    T = np.ascontiguousarray(T if axis == O.COL else T.transpose(0, 2, 1))
    P = np.ascontiguousarray(T.transpose(0, 2, 1))
    _check_single(env, W, T, P, 4, group, axis, 1, bf16=bf16)


@pytest.mark.parametrize("axis,group", [(O.COL, 32), (O.ROW, 64), (O.COL, 128), (O.ROW, 256)])
def test_bfloat16_weights_are_read_as_their_float32_values(env, axis, group):
    """bfloat16 storage multiplies one part where float32 storage multiplies three: of a value that bfloat16 holds the other two are zero, so
    codes, scales and losses are the same bits, for lines whose weights span 36 binades too (the gradient's pass over the weights is
    another one for either storage).  A line with an infinity is not a number in either, and no other line's outputs change by it."""
    torch, cafeq = env
    W, T, P = _case(axis, 136, 512, K, 1, 7300 + group)
    L = W if axis == O.COL else W.T
    L[8:40] *= np.exp2(-np.random.default_rng(7301).integers(0, 37, (32, 512))).astype(np.float32)
    L[40:72] *= np.float32(1e-30)
    def both():
        W16 = _dev(torch, W).to(torch.bfloat16)
        return [[x.cpu().numpy() for x in (*cafeq.proxy_loss_fwd_bwd(w, _dev(torch, T), _dev(torch, P), 4, group, axis, want_grad=True, want_codes=True),
                                           cafeq.apply_transform(w, _dev(torch, T), _dev(torch, P), axis, cafeq.SIDE_T, 1))] for w in (W16, W16.float())]
    got = both()
    for i in (0, 2, 3, 4):
        assert np.isfinite(got[0][i]).all()
        np.testing.assert_array_equal(got[0][i], got[1][i])
    parity.check_grad(got[0][1], got[1][1])
    L[77, 300] = np.inf
    for was, now in zip(got, both()):
        Z0, Z = (x[4] if axis == O.COL else x[4].T for x in (was, now))
        assert not np.isfinite(Z[77, K:]).any()                    # (index 300: block 1)
        for i, per in ((2, 1), (3, group), (4, 1)):
            a, b = ((x[i] if axis == O.COL else x[i].T).copy() for x in (was, now))
            a[77, K // per:] = b[77, K // per:] = 0
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("nb", [16, 17, 33])
@pytest.mark.parametrize("axis", [O.COL, O.ROW])
def test_gradient_through_the_inverse_of_many_blocks(env, nb, axis):
    """Up to 16 blocks (16 tiles each, 256 compute units) take the contraction of P^T G in two halves side by side, more in two turns."""
    W, T, P = _case(axis, 24, nb * K, K, 1, 7600 + nb)
    _check_single(env, W, T, P, 4, 128, axis, 1)
