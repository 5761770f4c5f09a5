"""GPU parity of each line of Alg. 1 where the Gram matrices take codes on one side (heads of 128 and 256, groups of 64 and more): one and
two versions of the other side, groups of several blocks and whole channels, codes of eight bits, contraction lengths that end inside a
step, groups of 32 next to them (six part products); weights near the ends of what squares in float32 hold.  Against the oracle, with the bounds
of tests/parity.py."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from tests import test_gpu_adaptive as adaptive

pytestmark = pytest.mark.gpu
env = adaptive.env


# (three times as many lines as a block has indices: the bounds are for well conditioned S)
@pytest.mark.parametrize("k,group,rep,bits,extra", [(256, 128, 1, 4, 564), (256, 256, 2, 3, 568), (256, 512, 1, 4, 572), (128, 128, 1, 8, 364),
                                                    (128, 256, 1, 4, 376), (128, 64, 2, 8, 380), (256, 32, 1, 4, 564), (128, 32, 1, 3, 360)])
def test_each_line(env, k, group, rep, bits, extra):
    adaptive.test_each_line_against_oracle(env, k, group, rep, bits, extra)


# (2^-50: products of scales stay numbers, but not their third parts without the scaling of the right operands)
@pytest.mark.parametrize("k,group", [(256, 64), (128, 128)])
@pytest.mark.parametrize("e", [-50, 45])
def test_scaled_pair(env, k, group, e):
    torch, cafeq = env
    U, V = adaptive._pair(330, 296, k, 2, 1, 700 + k)
    cu, su, _ = O.rtn_sym(U, 4, group, O.COL)
    codes = []
    for scale in (1.0, 2.0 ** e):
        Ud, Vd = adaptive._dev(torch, U * np.float32(scale)), adaptive._dev(torch, V)
        dcu, dsu = adaptive._dev(torch, cu), adaptive._dev(torch, (su * scale).astype(np.float32))
        dcv = torch.zeros(V.shape, dtype=torch.int8, device="cuda:0")
        dsv = torch.zeros((V.shape[0] // group, V.shape[1]), device="cuda:0")
        st = cafeq.adaptive_round_step(Ud, Vd, dcu, dsu, dcv, dsv, 4, group, k, 1, half=1)
        assert int(st.abs().sum()) == 0
        codes.append((dcv.cpu().numpy(), dsv.cpu().numpy()))
    np.testing.assert_array_equal(codes[0][0], codes[1][0])       # C does not depend on a power of two common to U and its codes
    np.testing.assert_array_equal(codes[0][1], codes[1][1])
