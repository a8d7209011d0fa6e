"""The one-launch QR of small and medium matrices (kernel variant 8): LAPACK's
Q element by element for full-rank input at the edges of its forms (one wave
up to 32 x 16, four waves up to 64 x 32, panels up to 128 x 64), and finite,
orthonormal factors of rank-deficient, zero and tiny-noise input."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F32, F64 = 0, 1
SIZES = [(1, 1), (2, 1), (2, 2), (16, 16), (32, 16), (31, 13), (32, 17), (33, 16), (33, 1), (64, 16),
         (64, 32), (63, 31), (64, 33), (65, 32), (65, 3), (90, 45), (96, 48), (128, 64), (127, 63),
         (128, 49), (70, 64), (66, 64), (64, 64), (128, 16), (100, 20)]


@pytest.fixture(scope="module")
def capi():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import capi as c
    return c


def _rand(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _run(capi, f, mode, ct=F64):
    m, n = f.shape
    x = f if mode == 0 else f.conj().T
    q, nrm2 = capi.dcs_test_qr(ct, ct, m, n, mode, 8, np.ascontiguousarray(x).reshape(-1))
    assert abs(nrm2 - np.sum(np.abs(f) ** 2)) <= 1e-10 * max(nrm2, 1e-300)
    return q.reshape(m, n) if mode == 0 else q.reshape(n, m).conj().T


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("m,n", SIZES)
def test_matches_lapack(capi, m, n, mode):
    rng = np.random.default_rng(m * 5 + n)
    f = _rand(rng, m, n)
    ref, _ = np.linalg.qr(f)
    q = _run(capi, f, mode)
    assert np.max(np.abs(q.conj().T @ q - np.eye(n))) < 1e-12
    assert np.max(np.abs(q - ref)) < 1e-10
    f32 = f.astype(np.complex64).astype(np.complex128)
    ref, _ = np.linalg.qr(f32)
    assert np.max(np.abs(_run(capi, f32, mode, F32) - ref)) < 1e-6   # rounding of Q to float


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("kind", ["rank2", "tiny", "zeros", "zero_matrix", "scaled"])
@pytest.mark.parametrize("m,n", [(8, 4), (32, 16), (64, 32), (96, 48), (128, 64), (70, 50)])
def test_deficient(capi, m, n, kind, mode):
    rng = np.random.default_rng(m + n)
    f = _rand(rng, m, 2) @ _rand(rng, 2, n)
    if kind == "tiny":
        f = f + 1e-170 * _rand(rng, m, n)
        f[:, n // 2] *= 1e-170
    elif kind == "zeros":
        f = _rand(rng, m, n)
        f[:, n // 2] = 0.0
        f[m // 2:, 0] = 0.0
    elif kind == "zero_matrix":
        f = np.zeros((m, n), complex)
    elif kind == "scaled":
        f = _rand(rng, m, n) * 10.0 ** rng.integers(-150, 140, size=n)
    q = _run(capi, f, mode)
    assert np.all(np.isfinite(q))
    np.testing.assert_allclose(q.conj().T @ q, np.eye(n), atol=1e-12)
    scale = np.maximum(np.max(np.abs(f), axis=0), 1e-300)
    np.testing.assert_allclose(q @ (q.conj().T @ (f / scale)), f / scale, atol=1e-12 * max(m, n))
    if kind == "scaled":
        ref, _ = np.linalg.qr(f / scale)   # positive column scaling leaves Q as it is
        assert np.max(np.abs(q - ref)) < 1e-9
