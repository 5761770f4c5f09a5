"""GPU parity: the inverse of a learning loop's iteration, which starts from the one before.  The loops hand back the
inverse of their last transform, made from scratch, so this one is called by its name in the library."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def warm():
    import torch
    from paper_2511_19705_amd import cafeq
    fn = cafeq.lib["_ZN5cafeq25launch_block_inverse_warmEPKfiiPdPfPiP12ihipStream_t"]
    fn.restype = ctypes.c_int
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int] + [ctypes.c_void_p] * 4

    def call(T, X0):
        """(inverse of T from the start X0, status), as float64 and int arrays"""
        nb, k, _ = T.shape
        Td, X = torch.from_numpy(T).to("cuda:0"), torch.from_numpy(X0).to("cuda:0")
        status = torch.full((nb,), 7, dtype=torch.int32, device="cuda:0")
        work = torch.zeros(cafeq.workspace_bytes(4, cafeq.Mat(), x=cafeq.Xform(0, 0, k, nb, 1)), dtype=torch.uint8, device="cuda:0")
        rc = fn(Td.data_ptr(), k, nb, work.data_ptr(), X.data_ptr(), status.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert rc == 0
        return X.cpu().numpy().astype(np.float64), status.cpu().numpy()
    return call


@pytest.mark.parametrize("k", [32, 64, 128, 256])
@pytest.mark.parametrize("entry", [98300.0, 65500.0, 65519.0, 65521.0, 131000.0, 3e5])
def test_entries_beyond_the_range_of_float16(warm, k, entry):
    """A signed permutation with one entry small enough that its inverse's, scaled as the iteration scales it (by 256 for a
    largest |T| of 1), lies about float16's largest number: 98300 is 65504 and 32796, which float16 has not."""
    rng = np.random.default_rng(k)
    T = np.eye(k)[rng.permutation(k)] * rng.choice([-1.0, 1.0], (k, 1))
    T[5] *= 256.0 / entry
    T = T[None].astype(np.float32)
    ref = np.linalg.inv(T.astype(np.float64))
    got, status = warm(T, ref.astype(np.float32))
    assert status[0] == 0
    # (an entry per row and column: float32 rounding of each)
    assert np.abs(got - ref).max(initial=0, where=ref == 0) == 0
    np.testing.assert_allclose(got[ref != 0], ref[ref != 0], rtol=2.0 ** -22)


def _conditioned(k, nb, cond, rng):
    """Blocks of condition number `cond`, singular values evenly spread over their logarithm, 1 in the root mean square."""
    U, V = (np.linalg.qr(rng.standard_normal((nb, k, k)))[0] for _ in range(2))
    s = float(cond) ** (-np.arange(k) / (k - 1))
    return (U * (s / np.sqrt((s * s).mean()))) @ V


@pytest.mark.parametrize("k", [32, 64, 128, 256])
@pytest.mark.parametrize("cond", [1, 3, 10, 30, 100])
@pytest.mark.parametrize("step", [0.0, 1e-6, 1e-4, 1e-3, 1e-2])
def test_the_loops_inverse_carries_its_rounding_alone(warm, k, cond, step):
    """T a step of equal size in every entry (as Adam makes it) from the T whose inverse the iteration starts at."""
    rng = np.random.default_rng(1000 * k + cond)
    T0 = _conditioned(k, 5, cond, rng).astype(np.float32)
    T = (T0 + step / (cond * np.sqrt(k)) * rng.choice([-1.0, 1.0], T0.shape)).astype(np.float32)
    got, status = warm(T, np.linalg.inv(T0.astype(np.float64)).astype(np.float32))
    assert not status.any()
    ref = np.linalg.inv(T.astype(np.float64))
    # rounding to float32 is at most 2^-24 of every entry (and half of that in the root mean square)
    err = np.linalg.norm(got - ref, axis=(1, 2)) / np.linalg.norm(ref, axis=(1, 2))
    assert err.max() <= 2.0 ** -24, err.max()


def test_ill_conditioned_blocks_of_32_are_left_to_the_elimination(warm):
    """Condition 300 and 1000: the digits of the exact residual no longer reach float32 rounding."""
    rng = np.random.default_rng(5)
    for cond in (300, 1000):
        T0 = _conditioned(32, 9, cond, rng).astype(np.float32)
        T = (T0 + 1e-4 / cond * rng.choice([-1.0, 1.0], T0.shape)).astype(np.float32)
        got, status = warm(T, np.linalg.inv(T0.astype(np.float64)).astype(np.float32))
        assert not status.any()
        ref = np.linalg.inv(T.astype(np.float64))
        err = np.linalg.norm(got - ref, axis=(1, 2)) / np.linalg.norm(ref, axis=(1, 2))
        # rounding alone: uniform up to 2^-24 of the leading power of two, 2^-24 / sqrt(3) in the root mean square, of entries
        # of 1.47 leading powers of two (mantissas uniform in their logarithm): 2.35e-8, and a fifth for the spread over the
        # few large entries of a block
        assert err.max() <= 2.8e-8, (cond, err)


@pytest.mark.parametrize("k", [32, 64, 128, 256])
@pytest.mark.parametrize("small", [1.0, 0.1, 0.01, 1e-3, 1e-4])
def test_starts_on_either_side_of_every_bound(warm, k, small):
    """Rotated blocks [[1, 0.7], [0, small]], starts X0 = T^-1 (I - E) with ||E||_F from 0 to 2: residuals on either side of
    the bounds, whose corrections take 16-bit operands of an X that amplifies what they lose by up to 0.7 / small."""
    rng = np.random.default_rng(k)
    size = np.concatenate([[0.0], np.geomspace(1e-3, 2.0, 14), np.geomspace(0.05, 0.6, 9)])
    T = np.linalg.qr(rng.standard_normal((len(size), k, k)))[0] @ np.kron(np.eye(k // 2), [[1.0, 0.7], [0.0, small]])
    T = T.astype(np.float32)
    ref = np.linalg.inv(T.astype(np.float64))
    E = rng.standard_normal(T.shape)
    E *= (size / np.linalg.norm(E, axis=(1, 2)))[:, None, None]
    got, status = warm(T, (ref @ (np.eye(k) - E)).astype(np.float32))
    assert not status.any()
    err = np.linalg.norm(got - ref, axis=(1, 2)) / np.linalg.norm(ref, axis=(1, 2))
    # rounding to float32; k = 256: and the square of a residual ||I - T X||_F of up to 3e-4
    assert err.max() <= 2.0 ** -24 + (9e-8 if k == 256 else 0.0), list(zip(size.round(4), err))


@pytest.mark.parametrize("small", [1e-2, 1e-3, 1e-4])
def test_eliminated_blocks_of_256_carry_their_rounding_alone(small):
    """The same blocks through cafeq_block_inverse: no rotation is near, all are eliminated, in float32."""
    import torch
    from paper_2511_19705_amd import cafeq
    k, rng = 256, np.random.default_rng(9)
    T = np.linalg.qr(rng.standard_normal((3, k, k)))[0] @ np.kron(np.eye(k // 2), [[1.0, 0.7], [0.0, small]])
    T = T.astype(np.float32)
    X, status = cafeq.block_inverse(torch.from_numpy(T).to("cuda:0"))
    assert not status.any()
    ref = np.linalg.inv(T.astype(np.float64))
    err = np.linalg.norm(X.cpu().numpy() - ref, axis=(1, 2)) / np.linalg.norm(ref, axis=(1, 2))
    assert err.max() <= 2.0 ** -24 + 9e-8, err
