"""GPU parity of the gradient pass by records (lines gathered row by row of the block): list and window edges, lists that do
not fit LDS, every line's arg-max in one row, blocks of each size, both axes, shared row-blocks, bfloat16 lines.  Tolerances
are those of every other gradient check (tests/parity.py): the pass itself is float32 sums of exact products."""
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


# one line; ends of a batch of 64; lines held in registers while they are sorted (4608) and one more; beyond the list in LDS (5120)
@pytest.mark.parametrize("lines", [4, 60, 64, 68, 4608, 4612, 5124])
@pytest.mark.parametrize("axis", [O.COL, O.ROW])
def test_line_counts(env, lines, axis):
    W, T, P = _case(axis, lines, 256, 128, 1, 2100 + lines)
    _check_single_prepared(env, W, T, P, 4, 128, axis, 1, want_codes=False)


# 8.4 M weights over prepared copies: blocks of 64 with groups of 128 by records; blocks of 32 with groups of 32 still beside the loss
# pass (by records from 10 M on: tests/test_gpu_routes.py)
@pytest.mark.parametrize("k,group,lines,naxis", [(32, 32, 4100, 2048), (64, 128, 4100, 2048), (64, 256, 200, 512), (256, 256, 200, 512),
                                                 (256, 64, 333, 512), (256, 0, 200, 768), (128, 512, 131, 1024)])
@pytest.mark.parametrize("bf16", [False, True])
def test_block_sizes(env, k, group, lines, naxis, bf16):
    W, T, P = _case(O.COL, lines, naxis, k, 1, 2200 + k + group)
    _check_single_prepared(env, W, T, P, 4, group, O.COL, 1, bf16=bf16, want_codes=False)


@pytest.mark.parametrize("axis", [O.COL, O.ROW])
@pytest.mark.parametrize("k,group", [(128, 128), (256, 64)])
def test_one_row_takes_every_line(env, axis, k, group):
    lines = 700
    W, T, P = _case(axis, lines, 2 * k, k, 1, 2300 + k)
    T = np.tile(np.eye(k, dtype=np.float32), (2, 1, 1)) + 0.01 * (T - np.eye(k, dtype=np.float32)[None]).astype(np.float32)
    P = O.block_inverse(T).astype(np.float32)
    ch = slice(None), [5, k + group - 1]
    W[ch if axis == O.COL else ch[::-1]] += 50.0 * np.abs(W).max()
    _check_single_prepared(env, W, T, P, 4, group, axis, 1, want_codes=False)


@pytest.mark.parametrize("k,group,rep,lines", [(32, 64, 1, 200), (64, 64, 2, 200), (128, 128, 2, 152), (256, 64, 2, 136), (256, 128, 1, 136),
                                               (128, 0, 1, 136)])
@pytest.mark.parametrize("bf16", [False, True])
def test_prepared_pairs(env, k, group, rep, lines, bf16):
    torch, cafeq = env
    A, B, T = WL.small_pair(lines, 512, k, rep, 2400 + k + group, eps=0.05)
    P = O.block_inverse(T).astype(np.float32)
    if bf16:
        a16, b16 = WL.to_bf16_bits(A), WL.to_bf16_bits(B)
        A, B = WL.bf16_bits_to_f32(a16), WL.bf16_bits_to_f32(b16)
        Ad, Bd = (_dev(torch, x.view(np.int16)).view(torch.bfloat16) for x in (a16, b16))
    else:
        Ad, Bd = _dev(torch, A), _dev(torch, B)
    prep = (cafeq.prepare_weights(Ad, O.COL), cafeq.prepare_weights(Bd, O.ROW))
    losses, grad, _ = cafeq.dual_proxy_loss_fwd_bwd(Ad, Bd, _dev(torch, T), _dev(torch, P), 4, group, rep, 5.0, True, False,
                                                    prepared=prep)
    torch.cuda.synchronize()
    ref = O.dual_lse(A, B, T, P, 4, group, rep, 5.0)
    for i, name in enumerate(("errU_sq", "errV_sq", "l2A_sq", "l2B_sq", "lse")):
        parity.check_scalar(float(losses[i]), ref[name], what=name)
    slack, _ = parity.dual_argmax_flip_slack(A, B, T, P, ref, group, rep, 5.0)
    parity.check_grad_with_slack(grad.cpu().numpy(), ref["gradT"], slack)


def test_repeated_calls_agree_bit_for_bit(env):
    torch, cafeq = env
    W, T, P = _case(O.COL, 3000, 256, 128, 1, 2500)
    Wd, Td, Pd = (_dev(torch, x) for x in (W, T, P))
    first = cafeq.proxy_loss_fwd_bwd(Wd, Td, Pd, 4, 128, O.COL)[1]
    for _ in range(3):
        assert torch.equal(first, cafeq.proxy_loss_fwd_bwd(Wd, Td, Pd, 4, 128, O.COL)[1])
