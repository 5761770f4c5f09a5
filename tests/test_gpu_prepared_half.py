"""Prepared copies of bfloat16 weights hold one 16-bit part per weight where those of float32 weights hold two.  The second
part of a bfloat16 value is zero, so every result must equal, bit for bit, the one over a float32 copy of the same values:
single matrices and pairs, either axis, gradients as partial sums and as whole blocks, mixed storage types."""
import numpy as np
import pytest

from paper_2511_19705_amd import workloads as WL

pytestmark = pytest.mark.gpu
K = 128


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


def _weights(torch, shape, seed):
    W = torch.from_numpy(WL.student_t3(shape, seed)).to("cuda:0")
    W[shape[0] // 2] = 0.0
    W.view(-1)[::97] *= 2.0 ** -30                         # far below their line's largest: denormal float16 parts
    return W.to(torch.bfloat16)


def _blocks(torch, cafeq, nb, seed):
    T = torch.from_numpy(WL.perturbed_blocks(nb, K, seed, 0.05)).to("cuda:0")
    return T, cafeq.block_inverse(T)[0]


def _same(torch, a, b):
    assert (a is None) == (b is None)
    if a is not None:
        assert torch.equal(a, b)


# 160 blocks: the gradient pass owns whole blocks; 3 and 8: partial sums.  Lines: one tile, ragged, several
@pytest.mark.parametrize("nb,lines", [(3, 8), (8, 296), (160, 136)])
@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("group,bits,codes", [(128, 3, False), (32, 4, True), (64, 2, False), (0, 4, False)])
def test_single(env, nb, lines, axis, group, bits, codes):
    torch, cafeq = env
    W = _weights(torch, (lines, nb * K) if axis == 0 else (nb * K, lines), 10 * nb + axis)
    T, P = _blocks(torch, cafeq, nb, 5 + nb)
    got = [cafeq.proxy_loss_fwd_bwd(X, T, P, bits, group, axis, want_grad=not codes or nb < 100, want_codes=codes,
                                    prepared=cafeq.prepare_weights(X, axis)) for X in (W, W.float())]
    for a, b in zip(*got):
        _same(torch, a, b)


@pytest.mark.parametrize("nb,d_model", [(5, 200), (80, 136)])
def test_pair_and_mixed_storage(env, nb, d_model):
    torch, cafeq = env
    A, B = _weights(torch, (d_model, nb * K), 31 + nb), _weights(torch, (nb * K, d_model), 32 + nb)
    T, P = _blocks(torch, cafeq, nb, 33 + nb)
    got = []
    for a, b in ((A, B), (A.float(), B.float()), (A, B.float()), (A.float(), B)):
        prep = (cafeq.prepare_weights(a, 0), cafeq.prepare_weights(b, 1))
        got.append(cafeq.dual_proxy_loss_fwd_bwd(a, b, T, P, 4, 128, prepared=prep))
    for other in got[1:2]:
        assert torch.equal(got[0][0], other[0]) and torch.equal(got[0][1], other[1])
    # (mixed types: test_mixed_storage_takes_one_launch)
    for other in got[2:]:
        np.testing.assert_allclose(other[0].cpu().numpy(), got[0][0].cpu().numpy(), rtol=1e-6)
        scale = float(got[0][1].abs().max())
        assert float((other[1] - got[0][1]).abs().max()) <= 1e-5 * scale
    assert cafeq.prepare_weights(A, 0).numel() < 0.55 * cafeq.prepare_weights(A.float(), 0).numel()


@pytest.mark.parametrize("axis", [0, 1])
def test_a_copy_of_the_other_storage_type_is_not_read(env, axis):
    """Its layout and size differ: the result is that over the weights themselves."""
    torch, cafeq = env
    W = _weights(torch, (264, 3 * K) if axis == 0 else (3 * K, 264), 71)
    T, P = _blocks(torch, cafeq, 3, 72)
    for X, other in ((W, W.float()), (W.float(), W)):
        got = cafeq.proxy_loss_fwd_bwd(X, T, P, 4, 128, axis, prepared=cafeq.prepare_weights(other, axis))
        ref = cafeq.proxy_loss_fwd_bwd(X, T, P, 4, 128, axis)
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


def test_a_copy_of_a_smaller_matrix_is_refused(env):
    torch, cafeq = env
    W, small = _weights(torch, (600, 3 * K), 73).float(), _weights(torch, (300, 3 * K), 74).float()
    T, P = _blocks(torch, cafeq, 3, 75)
    prep = cafeq.prepare_weights(small, 0)
    with pytest.raises(cafeq.CafeqError):
        cafeq.proxy_loss_fwd_bwd(W, T, P, 4, 128, 0, prepared=prep)
    B = _weights(torch, (3 * K, 600), 76).float()
    for bad in ((prep, None), (None, cafeq.prepare_weights(B[:, :256].contiguous(), 1))):
        with pytest.raises(cafeq.CafeqError):
            cafeq.dual_proxy_loss_fwd_bwd(W, B, T, P, 4, 128, prepared=bad)
        with pytest.raises(cafeq.CafeqError):
            cafeq.optimize_pair(W, B, T.clone(), 4, 128, prepared=bad, steps=1)
    # a pooled buffer may be larger than the copy in it
    room = torch.zeros(cafeq.prepare_weights(W, 0).numel() + 4096, dtype=torch.uint8, device="cuda:0")
    room[:-4096] = cafeq.prepare_weights(W, 0)
    got, ref = (cafeq.proxy_loss_fwd_bwd(W, T, P, 4, 128, 0, prepared=p) for p in (room, cafeq.prepare_weights(W, 0)))
    assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])


@pytest.mark.parametrize("nb,d_model", [(5, 200), (80, 136)])
@pytest.mark.parametrize("grad", [False, True])
def test_mixed_storage_takes_one_launch(env, nb, d_model, grad):
    """Both members' loss passes, whatever their storage types, and so the same partial sums: equal bit for bit."""
    torch, cafeq = env
    A, B = _weights(torch, (d_model, nb * K), 51 + nb), _weights(torch, (nb * K, d_model), 52 + nb)
    T, P = _blocks(torch, cafeq, nb, 53 + nb)
    ref = None
    for a, b in ((A, B), (A, B.float()), (A.float(), B)):
        prep = (cafeq.prepare_weights(a, 0), cafeq.prepare_weights(b, 1))
        timer = cafeq.LaunchTimer(4)
        with timer:
            losses, g, _ = cafeq.dual_proxy_loss_fwd_bwd(a, b, T, P, 4, 128, want_grad=grad, prepared=prep)
            torch.cuda.synchronize()
        assert timer.table.seen == 1
        ref = ref or (losses, g)
        assert torch.equal(losses, ref[0])
        _same(torch, g, ref[1])


@pytest.mark.parametrize("nb", [4, 160])
@pytest.mark.parametrize("axis", [0, 1])
def test_infinite_weights_act_as_those_of_a_float32_copy(env, nb, axis):
    torch, cafeq = env
    W = _weights(torch, (136, nb * K) if axis == 0 else (nb * K, 136), 81 + axis)
    W.view(-1)[[5, 700, 9001]] = torch.tensor([float("inf"), float("-inf"), float("inf")], dtype=W.dtype, device=W.device)
    W.view(-1)[1234] = float("nan")
    T, P = _blocks(torch, cafeq, nb, 82)
    for grad in (True, False):
        got = [cafeq.proxy_loss_fwd_bwd(X, T, P, 4, 64, axis, want_grad=grad, want_codes=not grad,
                                        prepared=cafeq.prepare_weights(X, axis)) for X in (W, W.float())]
        for a, b in zip(*got):
            if a is not None:
                np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())     # (not-a-numbers in the same places)
