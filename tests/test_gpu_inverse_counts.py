"""Inverse of blocks of 128: a block's result does not depend on how many blocks the call has (as many as half the compute units or
fewer, or more): the same bits for rotations, blocks near them, blocks that are eliminated and singular ones.  And the inverse in
T's own memory, which blocks of 32, 64 and 128 allow."""
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


@pytest.mark.parametrize("k", [32, 64, 128])
@pytest.mark.parametrize("nb", [7, 130])
def test_in_place(k, nb):
    import torch
    from paper_2511_19705_amd import cafeq
    T = WL.haar_blocks(nb, k, 9710 + k)
    rng = np.random.default_rng(9711)
    for b, eps in enumerate((0.0, 1e-6, 0.05, 0.2, 0.5, 3.0)):
        T[b] = T[b] @ (np.eye(k) + rng.standard_normal((k, k)) * (eps / np.sqrt(k)))
    T[6, :, 5] = T[6, :, 20]                      # singular
    T = torch.from_numpy(np.ascontiguousarray(T, dtype=np.float32)).cuda()
    P, st = cafeq.block_inverse(T)
    status, ws = torch.empty_like(st), torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    assert cafeq.lib.cafeq_block_inverse(T.data_ptr(), k, nb, T.data_ptr(), None, None, status.data_ptr(), ws.data_ptr(),
                                           cafeq._stream()) == 0
    assert torch.equal(T, P) and torch.equal(status, st) and int(st[6]) == 1
