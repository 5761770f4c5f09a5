"""Inverse of blocks of 128 with two workgroups a block (as many blocks as half the compute units or fewer) against one: the same
arithmetic for every column, so the same bits, for rotations, blocks near them, blocks that are eliminated and singular ones."""
import numpy as np
import pytest

from paper_2511_19705_amd import workloads as WL

pytestmark = pytest.mark.gpu


def test_same_bits_as_one_workgroup():
    import torch
    from paper_2511_19705_amd import cafeq
    nb = torch.cuda.get_device_properties(0).multi_processor_count // 2
    T = WL.haar_blocks(nb + 1, 128, 9700)
    rng = np.random.default_rng(9701)
    for b, eps in enumerate((0.0, 1e-6, 1e-3, 0.05, 0.2, 0.5, 3.0)):
        T[b] = T[b] @ (np.eye(128) + rng.standard_normal((128, 128)) * (eps / np.sqrt(128)))
    T[7] *= 1e-4
    T[8, :, 5] = T[8, :, 90]                      # singular
    T[9] = 0.0
    T[10] = np.diag(np.geomspace(1e-3, 1.0, 128)) @ T[10]
    T = torch.from_numpy(np.ascontiguousarray(T, dtype=np.float32)).cuda()
    one, st1 = cafeq.block_inverse(T)
    two, st2 = cafeq.block_inverse(T[:nb].contiguous())
    assert torch.equal(one[:nb], two) and torch.equal(st1[:nb], st2)
    assert st1[8] == 1 and st1[9] == 1 and int(st1.sum()) == 2
    few, st3 = cafeq.block_inverse(T[:11].contiguous())
    assert torch.equal(one[:11], few) and torch.equal(st1[:11], st3)
