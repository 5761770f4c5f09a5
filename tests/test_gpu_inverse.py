"""GPU parity: cafeq_block_inverse over the distances from a rotation at which its paths change (transpose, Newton's
iteration, float64 elimination) and over numbers of blocks that fill no round of workgroups."""
import numpy as np
import pytest

from paper_2511_19705_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2511_19705_amd import cafeq
    return torch, cafeq


@pytest.mark.parametrize("k", [32, 64, 128])
@pytest.mark.parametrize("nb", [1, 9, 37])
def test_distances_from_a_rotation(env, k, nb):
    torch, cafeq = env
    rng = np.random.default_rng(40 + k + nb)
    H = WL.haar_blocks(nb, k, 41 + k).astype(np.float64)
    scale = 10.0 ** rng.uniform(-3, 3, nb)
    eps = np.resize([0.05, 0.0, 1e-4, 0.01, 0.2, 0.3, 0.4, 0.6, 1.0, 3.0], nb)   # Frobenius distances 0 .. 3 sqrt(k)
    T = np.stack([scale[b] * H[b] @ (np.eye(k) + eps[b] / np.sqrt(k) * rng.standard_normal((k, k))) for b in range(nb)])
    T = T.astype(np.float32)
    Tinv, status = cafeq.block_inverse(torch.from_numpy(T).to("cuda:0"))
    torch.cuda.synchronize()
    assert int(status.abs().sum()) == 0
    got = Tinv.cpu().numpy().astype(np.float64)
    for b in range(nb):
        ref = np.linalg.inv(T[b].astype(np.float64))
        # float32 rounding of the result and of the last step's sum (2^-24 each, of entries up to the largest), and what
        # the iteration leaves: ||I - T X||_F^2 <= 2.5e-9 times ||X||_2 <= sqrt(k) max |x| for these blocks
        tol = (2.0 ** -23 + 2.5e-9 * np.sqrt(k)) * np.abs(ref).max()
        assert np.abs(got[b] - ref).max() <= tol, (b, eps[b], np.abs(got[b] - ref).max() / np.abs(ref).max())
    # reproducible, and a block's result does not depend on its place
    T2 = np.concatenate([T[::-1], T[:1]])
    again, _ = cafeq.block_inverse(torch.from_numpy(np.ascontiguousarray(T2)).to("cuda:0"))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(again.cpu().numpy()[:nb][::-1], Tinv.cpu().numpy())


@pytest.mark.parametrize("k", [32, 64, 128])
def test_flat_and_peaked_blocks(env, k):
    """Near-rotations whose entries are all alike (Hadamard: the inverse is small next to the scaling) or few (signed
    permutations), at several distances and scales."""
    from scipy.linalg import hadamard
    torch, cafeq = env
    rng = np.random.default_rng(50 + k)
    Hd = hadamard(k) / np.sqrt(k)
    Pm = np.eye(k)[rng.permutation(k)] * rng.choice([-1.0, 1.0], k)
    T = np.stack([s * q @ (np.eye(k) + eps / np.sqrt(k) * rng.standard_normal((k, k)))
                  for q in (Hd, Pm) for eps in (0.0, 1e-7 if k == 32 else 1e-5, 1e-4, 0.01, 0.05, 0.3) for s in (1.0, 3.7e4)]).astype(np.float32)
    Tinv, status = cafeq.block_inverse(torch.from_numpy(T).to("cuda:0"))
    torch.cuda.synchronize()
    assert int(status.abs().sum()) == 0
    got = Tinv.cpu().numpy().astype(np.float64)
    for b in range(T.shape[0]):
        ref = np.linalg.inv(T[b].astype(np.float64))
        tol = (2.0 ** -23 + 2.5e-9 * np.sqrt(k)) * np.abs(ref).max()
        assert np.abs(got[b] - ref).max() <= tol, (b, np.abs(got[b] - ref).max() / np.abs(ref).max())


@pytest.mark.parametrize("bad", ["zero", "nan", "inf", "equal rows", "tiny"])
@pytest.mark.parametrize("k", [32, 64, 128])
def test_blocks_without_an_inverse_leave_the_others_alone(env, k, bad):
    torch, cafeq = env
    T = WL.perturbed_blocks(3, k, 60 + k, eps=0.05)
    ref = np.linalg.inv(T.astype(np.float64))
    if bad == "zero":
        T[1] = 0.0
    elif bad == "nan":
        T[1, 3, 5] = np.nan
    elif bad == "inf":
        T[1, 3, 5] = np.inf
    elif bad == "equal rows":
        T[1, 5] = T[1, 9]
    else:
        T[1] *= np.float32(1e-39)                          # denormal entries: an inverse that float32 cannot hold
    Tinv, status = cafeq.block_inverse(torch.from_numpy(T).to("cuda:0"))
    torch.cuda.synchronize()
    st = status.cpu().numpy()
    assert st[0] == 0 and st[2] == 0
    if bad in ("zero", "equal rows"):
        assert st[1] == 1 and float(Tinv[1].abs().max()) == 0.0
    for b in (0, 2):
        np.testing.assert_allclose(Tinv[b].cpu().numpy(), ref[b], rtol=0, atol=2.0 ** -22 * np.abs(ref[b]).max())
