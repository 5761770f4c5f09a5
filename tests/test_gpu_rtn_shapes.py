"""GPU parity: the plain quantizer over the lane shapes of its kernels along the contiguous axis -- groups of every power of
two in both storage types, whole channels from one piece per lane to the most a workgroup holds, rows padded and not --
bit-exact codes and scales on both grids."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from paper_2511_19705_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


def _check(env, W, bits, group, bf16, pad, grid):
    torch, cafeq = env
    if bf16:
        b16 = WL.to_bf16_bits(W)
        W = WL.bf16_bits_to_f32(b16)
        Wd = torch.from_numpy(b16.view(np.int16)).to("cuda:0").view(torch.bfloat16)
    else:
        Wd = torch.from_numpy(W).to("cuda:0")
    if pad:
        big = torch.full((Wd.shape[0], Wd.shape[1] + pad), 7.0, dtype=Wd.dtype, device="cuda:0")
        big[:, :Wd.shape[1]] = Wd
        Wd = big[:, :W.shape[1]]
    if grid == "sym":
        codes, scales, err = cafeq.rtn_quantize(Wd, bits, group, O.COL, want_err=True)
        c_ref, s_ref, zh = O.rtn_sym(W, bits, group, O.COL)
    else:
        codes, scales, mins, err = cafeq.rtn_quantize_minmax(Wd, bits, group, O.COL, want_err=True)
        c_ref, s_ref, m_ref, zh = O.rtn_asym(W, bits, group, O.COL, "f32")
        np.testing.assert_array_equal(mins.cpu().numpy(), m_ref.astype(np.float32))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(codes.cpu().numpy().astype(np.int16), c_ref)
    np.testing.assert_array_equal(scales.cpu().numpy(), s_ref.astype(np.float32))
    ref = float(((zh - W.astype(np.float64)) ** 2).sum())
    assert abs(float(err.item()) - ref) <= 1e-5 * ref + 1e-30


@pytest.mark.parametrize("grid", ["sym", "minmax"])
@pytest.mark.parametrize("bf16,pad", [(True, 0), (True, 8), (False, 4)])
@pytest.mark.parametrize("group", [4, 8, 16, 32, 64, 128, 256])
def test_powers_of_two(env, group, bf16, pad, grid):
    W = WL.student_t3((29, 1280), 30 + group)
    W[3, :group] = 0.0
    _check(env, W, 4, group, bf16, pad, grid)


@pytest.mark.parametrize("grid", ["sym", "minmax"])
@pytest.mark.parametrize("bf16,pad", [(True, 0), (False, 12), (False, 0)])
@pytest.mark.parametrize("cols,group", [(2048, 0), (2056, 0), (4096, 2048), (8200, 0), (16392, 0), (36864, 0), (65536, 0), (131080, 0)])
def test_whole_channels(env, cols, group, bf16, pad, grid):
    W = WL.student_t3((5, cols), 60 + cols)
    W[2, cols - 1] = 3.0                             # the largest magnitude at the very end
    _check(env, W, 3, group, bf16, pad, grid)
