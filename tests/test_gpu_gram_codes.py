"""GPU parity of each line of Alg. 1 where the Gram matrices take codes on one side (heads of 128 and 256, groups of 64 and more): one and
two versions of the other side, groups of several blocks and whole channels, codes of eight bits, contraction lengths that end inside a
step, groups of 32 next to them (six part products); weights near the ends of what squares in float32 hold.  Against the oracle, with the bounds
of tests/parity.py."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from tests import parity
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


# one line of the head far from the others, a zero, a tiny or a huge one among them; and weights near the end of float32 behind a first line
# of zeros: the correction of the other lines' codes against the oracle
@pytest.mark.parametrize("k,group", [(256, 64), (128, 128)])
@pytest.mark.parametrize("line,factor,rest", [(0, 0.0, 1.0), (0, None, 1.0), (0, None, 64.0), (0, 1e-36, 1.0), (7, None, 64.0), (0, 0.0, 2.0 ** -50), (0, 1e-10, 2.0 ** 30)])
def test_one_line_unlike_the_others(env, k, group, line, factor, rest):
    torch, cafeq = env
    U, V = adaptive._pair(3 * k + 12, 296, k, 2, 1, 720 + k)
    U *= np.float32(rest)
    if factor is None:                            # the head's first scale just above float32's denormal numbers
        factor = 2.0 ** -125.5 / float(O.rtn_sym(U[line:line + 1], 4, group, O.COL)[1][0, 0])
    U[line] *= np.float32(factor)
    cu, su, _ = O.rtn_sym(U, 4, group, O.COL)
    su = su.astype(np.float32)
    Uh = adaptive._dequant(cu, su, group, O.COL)
    _, _, Vt, _ = O.adaptive_round_step(U, V, Uh, 4, group, k, 1, half=0)
    cv, sv, _ = O.rtn_sym(Vt, 4, group, O.ROW)
    dcv = torch.zeros(V.shape, dtype=torch.int8, device="cuda:0")
    dsv = torch.zeros(sv.shape, dtype=torch.float32, device="cuda:0")
    st = cafeq.adaptive_round_step(adaptive._dev(torch, U), adaptive._dev(torch, V), adaptive._dev(torch, cu), adaptive._dev(torch, su), dcv, dsv,
                                   4, group, k, 1, half=1)
    assert int(st.abs().sum()) == 0
    parity.check_scales(dsv.cpu().numpy(), sv)
    parity.check_codes(dcv.cpu().numpy(), cv, Vt, sv, O.ROW, group)
