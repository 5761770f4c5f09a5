"""Equal magnitudes inside a group: the arg-max a prepared loss pass records is the first of them, whatever tile of 32, lane
half or sign it sits in.  With an identity transform and small integers as weights every tie is exact, and the gradient
through the transformed weights (its diagonal scatter) shows which entry was taken."""
import numpy as np
import pytest

from oracle import cafeq_oracle as O
from tests import parity

pytestmark = pytest.mark.gpu
K = 128


@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("bf16", [False, True])
def test_the_first_of_equal_magnitudes(group, axis, bf16):
    import torch
    from paper_2511_19705_amd import cafeq
    rng = np.random.default_rng(group + axis)
    nb, lines = 3, 200
    W = rng.integers(-3, 4, (lines, nb * K)).astype(np.float32)        # every group holds several of each magnitude
    W[5] = 0.0
    W[6:9] = 0.0
    W[6, 127] = W[7, 0] = W[8, 64] = -2.0
    if axis == 1:
        W = np.ascontiguousarray(W.T)
    T = np.tile(np.eye(K, dtype=np.float32), (nb, 1, 1))
    Wd = torch.from_numpy(W).to("cuda:0")
    Wd = Wd.to(torch.bfloat16) if bf16 else Wd
    Td = torch.from_numpy(T).to("cuda:0")
    losses, grad, _, _ = cafeq.proxy_loss_fwd_bwd(Wd, Td, Td, 4, group, axis, prepared=cafeq.prepare_weights(Wd, axis))
    torch.cuda.synchronize()
    value, ref = O.surrogate(W, T, T, 4, group, axis)
    parity.check_scalar(float(losses[3]), value, what="surrogate")
    parity.check_grad(grad.cpu().numpy(), ref)
