"""GPU parity: the update that rides in the epilogue of the gradient's last product (learning loops without a regulariser)
against the gradient from an evaluation and the update as a call of its own: the same arithmetic on the same values, so the
first step is equal bit for bit.  Later steps start from the inverse before them instead of from scratch; both are the
inverse to float32 rounding."""
import numpy as np
import pytest

from paper_2511_19705_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _close(torch, a, b, lr):
    """Entries whose gradient is at the level of rounding may go another way; the others agree far below a step."""
    off = (a - b).abs() > 1e-3 * lr
    assert float(off.float().mean()) <= 2e-3, float(off.float().mean())


@pytest.mark.parametrize("k", [32, 64, 128, 256])
@pytest.mark.parametrize("normalize", [True, False])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("steps", [1, 3])
def test_gradient_descent(env, k, normalize, axis, steps):
    torch, cafeq = env
    W = WL.student_t3((200, 768) if axis == 0 else (768, 200), 11 + k)
    W, T0 = _dev(torch, W), _dev(torch, WL.perturbed_blocks(768 // k, k, 12 + k, 0.03))
    lr = 2.0 if normalize else 2.0 / float(W.double().square().sum())
    T = T0.clone()
    cafeq.optimize_single(W, T, 4, 64, axis, 1, lr, steps, 0.0, normalize)
    ref = T0.clone()
    for _ in range(steps):
        P, _ = cafeq.block_inverse(ref)
        losses, grad, _, _ = cafeq.proxy_loss_fwd_bwd(W, ref, P, 4, 64, axis)
        cafeq.sgd_update(ref, grad / losses[2] if normalize else grad, lr)
    moved = float((ref - T0).abs().max())
    assert moved > 0
    if steps == 1:
        assert torch.equal(T, ref)
    else:
        assert float((T - ref).abs().max()) <= 1e-3 * moved


# 128 blocks of 128 a member, prepared: the gradient pass owns whole blocks; elsewhere partial sums
@pytest.mark.parametrize("k,rep,nb,prepared", [(32, 1, 8, False), (64, 1, 6, True), (64, 2, 6, False), (128, 1, 4, True),
                                               (128, 1, 128, True), (256, 1, 3, False), (256, 2, 3, False)])
@pytest.mark.parametrize("steps", [1, 3])
def test_adam(env, k, rep, nb, prepared, steps):
    torch, cafeq = env
    A, B, T0 = WL.small_pair(136, nb * k, k, rep, 13 + k + rep, eps=0.03)
    A, B, T0 = _dev(torch, A), _dev(torch, B), _dev(torch, T0)
    prep = (cafeq.prepare_weights(A, 0), cafeq.prepare_weights(B, 1)) if prepared else (None, None)
    lr, group = 1e-3, min(k, 64)
    T = T0.clone()
    cafeq.optimize_pair(A, B, T, 4, group, rep, 5.0, lr, steps, prepared=prep)
    ref, m, v = T0.clone(), torch.zeros_like(T0), torch.zeros_like(T0)
    for s in range(steps):
        P, _ = cafeq.block_inverse(ref)
        _, grad, _ = cafeq.dual_proxy_loss_fwd_bwd(A, B, ref, P, 4, group, rep, 5.0, prepared=prep)
        cafeq.adam_update(ref, grad, m, v, s + 1, lr, 0.1, 0.999, 1e-8)
    assert float((ref - T0).abs().max()) > 0.5 * lr
    if steps == 1:
        assert torch.equal(T, ref)
    else:
        _close(torch, T, ref, lr)
