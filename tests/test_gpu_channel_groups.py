"""GPU parity for groups that span many segments: the records of a group's segments are folded by several threads per
line, its sum of squared inverse norms by a whole workgroup.  Numbers of segments that are no multiple of the runs the
threads take (3, 9, 17), of lines that fill no tile, one group and several."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from tests.test_gpu_minmax_fused import _check_single_minmax
from tests.test_gpu_single import _case, _check_single

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


@pytest.mark.parametrize("k,group,naxis,lines", [(128, 0, 1152, 36), (32, 384, 1152, 4), (64, 0, 2176, 68), (256, 0, 2304, 100)])
@pytest.mark.parametrize("axis,rep", [(O.COL, 1), (O.ROW, 1)])
def test_runs_of_segments(env, k, group, naxis, lines, axis, rep):
    W, T, P = _case(axis, lines, naxis, k, rep, 1500 + k)
    W[3] = 0.0                                             # a line (COL) or an input (ROW) of zeros
    _check_single(env, W, T, P, 4, group, axis, rep)
    _check_single_minmax(env, W, T, P, 3, group, axis, rep)


@pytest.mark.parametrize("k,group,naxis,rep", [(32, 256, 512, 1), (32, 128, 512, 2), (128, 0, 1280, 5), (64, 128, 640, 5)])
def test_sums_of_squared_norms_over_shared_blocks(env, k, group, naxis, rep):
    # rep != 1: the sums come from the kernel over groups; rep == 1 with few whole blocks per group: from the norms' launch
    W, T, P = _case(O.ROW, 40, naxis, k, rep, 1550 + k)
    _check_single(env, W, T, P, 4, group, O.ROW, rep)
