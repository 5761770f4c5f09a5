"""GPU parity of the loss pass over prepared weights for blocks of 32 and 64: several blocks share a segment of 128, each in
units of its own; groups inside a block and across blocks; ragged line counts; codes, scales and losses against the oracle
(bounds of tests/parity.py, ties by the transform's rounding).  Small matrices take that pass with groups of 128 and the general
kernel, prepared copy or not, with shorter ones; the larger ones below take it throughout.  Gradients: tests/test_gpu_gather.py."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from paper_2511_19705_amd import workloads as WL
from tests import parity
from tests.test_gpu_prepared import _check_single_prepared
from tests.test_gpu_single import _case, _dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


# 296 lines: a macro-tile of 256 and a ragged one; rep 2 and 4: a segment's row-blocks share transform blocks
@pytest.mark.parametrize("k,group", [(32, 32), (32, 64), (32, 128), (64, 32), (64, 64), (64, 128)])
@pytest.mark.parametrize("axis,rep", [(O.COL, 1), (O.ROW, 1), (O.ROW, 2), (O.ROW, 4)])
@pytest.mark.parametrize("bf16", [False, True])
def test_codes_scales_losses(env, k, group, axis, rep, bf16):
    W, T, P = _case(axis, 296, 512, k, rep, 3100 + k + group)
    _check_single_prepared(env, W, T, P, 3 if bf16 else 4, group, axis, rep, bf16=bf16, want_grad=False)
    _check_single_prepared(env, W, T, P, 2, group, axis, rep, bf16=bf16, want_grad=False, want_codes=False)


@pytest.mark.parametrize("k,group", [(32, 32), (32, 128), (64, 64), (64, 128)])
@pytest.mark.parametrize("spread", [2.0, 2.0 ** 12, 2.0 ** 30])
def test_blocks_of_different_magnitude(env, k, group, spread):
    W, T, P = _case(O.COL, 200, 256, k, 1, 3200 + k)
    f = np.where(np.arange(T.shape[0]) % 2 == 0, 1.0, 1.0 / spread).astype(np.float32)[:, None, None]
    T = T * f
    P = O.block_inverse(T).astype(np.float32)
    _check_single_prepared(env, W, T, P, 4, group, O.COL, 1, want_grad=False)


@pytest.mark.parametrize("k,group,rep", [(32, 128, 1), (64, 64, 1), (64, 128, 2)])
def test_pair_with_codes(env, k, group, rep):
    torch, cafeq = env
    A, B, T = WL.small_pair(296, 512 if rep == 1 else 256, k, rep, 3300 + k + group, eps=0.05)
    P = O.block_inverse(T).astype(np.float32)
    Ad, Bd = _dev(torch, A), _dev(torch, B)
    prep = (cafeq.prepare_weights(Ad, O.COL), cafeq.prepare_weights(Bd, O.ROW))
    losses, _, outs = cafeq.dual_proxy_loss_fwd_bwd(Ad, Bd, _dev(torch, T), _dev(torch, P), 3, group, rep, 5.0, False, True,
                                                    prepared=prep)
    torch.cuda.synchronize()
    ref = O.dual_lse(A, B, T, P, 3, group, rep, 5.0)
    for i, name in enumerate(("errU_sq", "errV_sq", "l2A_sq", "l2B_sq", "lse")):
        parity.check_scalar(float(losses[i]), ref[name], what=name)
    cu, su, cv, sv = [x.cpu().numpy() for x in outs]
    cu_ref, su_ref, _ = O.rtn_sym(ref["U"], 3, group, O.COL)
    cv_ref, sv_ref, _ = O.rtn_sym(ref["V"], 3, group, O.ROW)
    parity.check_scales(su, su_ref)
    parity.check_scales(sv, sv_ref)
    parity.check_codes(cu, cu_ref, ref["U"], su_ref, O.COL, group)
    parity.check_codes(cv, cv_ref, ref["V"], sv_ref, O.ROW, group)


# Sizes from which the pass over prepared weights is taken whatever the group (below, groups of 32 and 64 go through the general
# kernel: tests/test_gpu_routes.py): other bits than the general kernel's, the same bounds.  3400 lines: 13 macro-tiles, a ragged one
@pytest.mark.parametrize("k,group", [(32, 32), (32, 64), (32, 128), (64, 32), (64, 64), (64, 128)])
@pytest.mark.parametrize("axis,rep,bf16,codes", [(O.COL, 1, False, True), (O.COL, 1, True, True), (O.ROW, 1, False, False), (O.ROW, 2, True, True),
                                                 (O.ROW, 4, False, False)])
def test_sizes_that_take_the_prepared_pass(env, k, group, axis, rep, bf16, codes):
    torch, cafeq = env
    W, T, P = _case(axis, 3400, 2048, k, rep, 3400 + k + group)
    _check_single_prepared(env, W, T, P, 3 if bf16 else 4, group, axis, rep, bf16=bf16, want_grad=False, want_codes=codes)
    if codes:
        _differs_from_the_general_kernel(torch, cafeq, W, T, P, 3 if bf16 else 4, group, axis, rep, bf16)


def _differs_from_the_general_kernel(torch, cafeq, W, T, P, bits, group, axis, rep, bf16):
    """(in the last bits of some of the scales)"""
    Wd = _dev(torch, W).to(torch.bfloat16 if bf16 else torch.float32)
    a, b = (cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), _dev(torch, P), bits, group, axis, rep, want_grad=False, want_codes=True, prepared=p)[3]
            for p in (cafeq.prepare_weights(Wd, axis), None))
    assert not torch.equal(a, b)


@pytest.mark.parametrize("k", [32, 64])
@pytest.mark.parametrize("spread", [2.0 ** 12, 2.0 ** 30])
def test_blocks_of_different_magnitude_take_the_prepared_pass(env, k, spread):
    torch, cafeq = env
    W, T, P = _case(O.COL, 3400, 2048, k, 1, 3450 + k)
    T = T * np.where(np.arange(T.shape[0]) % 2 == 0, 1.0, 1.0 / spread).astype(np.float32)[:, None, None]
    P = O.block_inverse(T).astype(np.float32)
    _check_single_prepared(env, W, T, P, 4, k, O.COL, 1, want_grad=False)
    _differs_from_the_general_kernel(torch, cafeq, W, T, P, 4, k, O.COL, 1, False)


# member B's codes are byte stores along its rows: from two rounds of the general kernel's workgroups on
@pytest.mark.parametrize("k,group", [(32, 128), (64, 128), (64, 64)])
def test_large_pair_with_codes(env, k, group):
    torch, cafeq = env
    A, B, T = WL.small_pair(4608, 2048, k, 1, 3500 + k + group, eps=0.05)
    P = O.block_inverse(T).astype(np.float32)
    Ad, Bd = _dev(torch, A), _dev(torch, B)
    prep = (cafeq.prepare_weights(Ad, O.COL), cafeq.prepare_weights(Bd, O.ROW))
    losses, _, outs = cafeq.dual_proxy_loss_fwd_bwd(Ad, Bd, _dev(torch, T), _dev(torch, P), 3, group, 1, 5.0, False, True, prepared=prep)
    torch.cuda.synchronize()
    ref = O.dual_lse(A, B, T, P, 3, group, 1, 5.0, want_grad=False)
    for i, name in enumerate(("errU_sq", "errV_sq", "l2A_sq", "l2B_sq", "lse")):
        parity.check_scalar(float(losses[i]), ref[name], what=name)
    for c, s, z, axis in ((outs[0], outs[1], "U", O.COL), (outs[2], outs[3], "V", O.ROW)):
        c_ref, s_ref, _ = O.rtn_sym(ref[z], 3, group, axis)
        parity.check_scales(s.cpu().numpy(), s_ref)
        parity.check_codes(c.cpu().numpy(), c_ref, ref[z], s_ref, axis, group)


# (its own block's transformed values are not numbers; nothing else of the line's 128 inputs depends on it)
@pytest.mark.parametrize("k", [32, 64])
@pytest.mark.parametrize("axis,bf16", [(O.COL, False), (O.COL, True), (O.ROW, True)])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_an_infinite_weight_leaves_its_lines_other_blocks_alone(env, k, axis, bf16, value):
    torch, cafeq = env
    W, T, P = _case(axis, 3400, 2048, k, 1, 3600 + k)
    outs = []
    for v in (value, 0.0):
        W[(70, 300) if axis == O.COL else (300, 70)] = v
        Wd = _dev(torch, W).to(torch.bfloat16 if bf16 else torch.float32)
        _, _, codes, scales = cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), _dev(torch, P), 4, k, axis, want_grad=False, want_codes=True,
                                                       prepared=cafeq.prepare_weights(Wd, axis))
        outs.append([x.cpu().numpy() if axis == O.COL else x.cpu().numpy().T for x in (codes, scales)])
    g = 300 // k
    for codes, scales in outs:
        codes[70, g * k:(g + 1) * k] = 0
        scales[70, g] = 0
    np.testing.assert_array_equal(outs[0][0], outs[1][0])
    np.testing.assert_array_equal(outs[0][1], outs[1][1])


# Blocks of inputs far smaller than their neighbours in the segment of 128: every block's scales and codes are as exact as if it were
# alone.  The first 64 lines only, so that strips of both kinds meet, and one line of strip 40
@pytest.mark.parametrize("k,group", [(32, 32), (32, 64), (32, 128), (64, 32), (64, 64), (64, 128)])
@pytest.mark.parametrize("axis,bf16,factor", [(O.COL, False, 2.0 ** -10), (O.COL, False, 2.0 ** -45), (O.COL, True, 2.0 ** -20),
                                              (O.ROW, False, 2.0 ** -20), (O.ROW, True, 2.0 ** -45)])
def test_inputs_of_different_magnitude(env, k, group, axis, bf16, factor):
    W, T, P = _case(axis, 3400, 2048, k, 1, 3700 + k + group)
    V = W if axis == O.COL else W.T
    small = (np.arange(2048) // k) % 3 != 1
    for line in list(range(64)) + [1285]:
        V[line, small] *= np.float32(factor)
    codes = axis == O.COL or bf16 or (k, group) == (64, 128)          # (along rows from float32 weights: the general kernel's)
    _check_single_prepared(env, W, T, P, 4, group, axis, 1, bf16=bf16, want_grad=False, want_codes=codes)
    if not codes:
        _check_losses_of_the_small_blocks(env, W, T, P, group, k, small)


def _check_losses_of_the_small_blocks(env, W, T, P, group, k, small):
    """Lines of small blocks alone: their errors are the losses (rows, no codes)."""
    torch, cafeq = env
    W = W.copy()
    W[:, 64:1280] = 0.0
    W[:, 1344:] = 0.0
    W[~small] *= np.float32(2.0 ** -3)
    Wd = _dev(torch, W)
    losses, _, _, _ = cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), _dev(torch, P), 4, group, O.ROW, 1, want_grad=False,
                                               prepared=cafeq.prepare_weights(Wd, O.ROW))
    ref = O.proxy_l2(W, T, P, 4, group, O.ROW, 1)
    parity.check_scalar(float(losses[0]), ref["l2_sq"], what="l2_sq")
    parity.check_scalar(float(losses[1]), ref["err_z_sq"], what="err_z_sq")


# (blocks of 128 likewise: their forward operand is two float16 parts with or without a prepared copy)
@pytest.mark.parametrize("k", [32, 64, 128])
@pytest.mark.parametrize("value", [np.inf, -np.inf])
def test_an_infinite_entry_of_a_block_leaves_the_other_outputs_alone(env, k, value):
    torch, cafeq = env
    W, T, P = _case(O.COL, 3400, 2048, k, 1, 3800 + k)
    Wd, Pd = _dev(torch, W), _dev(torch, P)
    prep = cafeq.prepare_weights(Wd, O.COL)
    outs = []
    for v in (value, 0.0):
        T[3, 1, 2] = v
        _, _, codes, scales = cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), Pd, 4, 32, O.COL, want_grad=False, want_codes=True, prepared=prep)
        codes[:, 3 * k:3 * k + 32] = 0                       # (the output's own group)
        scales[:, 3 * k // 32] = 0
        outs.append((codes, scales))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])


# the line's scale at the lower end of float32's range (the losses, squares, are zeros there)
@pytest.mark.parametrize("k", [32, 64, 128])
@pytest.mark.parametrize("factor", [1e-30, 1e-34])
def test_small_weights(env, k, factor):
    torch, cafeq = env
    W, T, P = _case(O.COL, 3400, 2048, k, 1, 3900 + k)
    W = (W * np.float32(factor)).astype(np.float32)
    Wd = _dev(torch, W)
    _, _, codes, scales = cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), _dev(torch, P), 4, 32, O.COL, want_grad=False, want_codes=True,
                                                   prepared=cafeq.prepare_weights(Wd, O.COL))
    Z = O.blockdiag_apply(W, T, O.COL, 1)
    c_ref, s_ref, _ = O.rtn_sym(Z, 4, 32, O.COL)
    parity.check_scales(scales.cpu().numpy(), s_ref)
    tol = parity.tie_tolerance(W, T, O.COL, 1, Z, s_ref, 32, parity.forward_unit(k, 32, 4))
    parity.check_codes(codes.cpu().numpy(), c_ref, Z, s_ref, O.COL, 32, tie_tol=tol)


# a block of values that are not numbers has the codes that it has without a prepared copy (the grid's lowest)
@pytest.mark.parametrize("k,group", [(32, 32), (32, 128), (64, 64), (64, 128)])
@pytest.mark.parametrize("axis,bf16,bits", [(O.COL, False, 4), (O.COL, True, 2), (O.ROW, True, 3)])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_codes_of_a_block_that_is_not_a_number(env, k, group, axis, bf16, bits, value):
    torch, cafeq = env
    rows, cols = (3456, 2048) if axis == O.COL else (2048, 3456)
    W, T, P = _case(axis, rows, cols, k, 1, 4000 + k)
    W[(1700, 700) if axis == O.COL else (700, 1700)] = value
    Wd = _dev(torch, W)
    Wd = Wd.to(torch.bfloat16) if bf16 else Wd
    lo = 700 // k * k
    block = (slice(1700, 1701), slice(lo, lo + k)) if axis == O.COL else (slice(lo, lo + k), slice(1700, 1701))
    codes = [cafeq.proxy_loss_fwd_bwd(Wd, _dev(torch, T), _dev(torch, P), bits, group, axis, want_grad=False, want_codes=True,
                                      prepared=p)[2][block] for p in (None, cafeq.prepare_weights(Wd, axis))]
    assert torch.equal(codes[0], codes[1])
