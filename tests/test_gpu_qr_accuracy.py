"""Accuracy and range of the one-launch QR (kernel variant 8): the columns of Q
have norm 1 as closely as LAPACK's Householder columns, and columns up to the
largest finite numbers give LAPACK's Q."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F64 = 1


@pytest.fixture(scope="module")
def capi():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import capi as c
    return c


def _rand(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _q(capi, f, mode=0):
    m, n = f.shape
    x = f if mode == 0 else f.conj().T
    q, _ = capi.dcs_test_qr(F64, F64, m, n, mode, 8, np.ascontiguousarray(x).reshape(-1))
    return q.reshape(m, n) if mode == 0 else q.reshape(n, m).conj().T


def _norm_errors(q):
    q = q.astype(np.clongdouble)
    return (q.real ** 2 + q.imag ** 2).sum(0) - 1


@pytest.mark.parametrize("m,n", [(2, 1), (4, 2), (32, 16), (90, 45)])
def test_column_norms(capi, m, n):
    """Root mean square of |q|^2 - 1 over 1000 columns or more, against LAPACK's
    on the same matrices.  Each is known to 1 / sqrt(2 * 1000) = 2.2 %, their
    ratio to 3.2 %; 1.16 is five times that."""
    rng = np.random.default_rng([m, n])
    ours, ref = [], []
    for _ in range(-(-1000 // n)):
        f = _rand(rng, m, n)
        ours.append(_norm_errors(_q(capi, f)))
        ref.append(_norm_errors(np.linalg.qr(f)[0]))
    rms = [float(np.sqrt(np.mean(np.concatenate(e) ** 2))) for e in (ours, ref)]
    assert rms[0] <= 1.16 * rms[1]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("m,n", [(2, 1), (16, 8), (32, 16), (64, 32), (96, 48)])
def test_huge_columns(capi, m, n, mode):
    """Entries up to 1e305, whose squares are infinite.  Scaling a column by a
    power of two leaves Q as it is, so the reference is LAPACK's Q of the
    unscaled matrix; bounds as for the scaled columns of test_gpu_qr_mid.  A
    last column below 1e-280 counts as zero: its column of Q is only
    orthonormal to the others."""
    rng = np.random.default_rng([m, n, 1])
    f = _rand(rng, m, n)
    ref, _ = np.linalg.qr(f)
    e = np.zeros(n, int)
    e[0] = 1013               # 2^1013 = 8.8e304
    if n > 2:
        e[n // 2], e[n - 1] = 999, -999
    q = _q(capi, f * np.ldexp(1.0, e), mode)
    assert np.all(np.isfinite(q))
    np.testing.assert_allclose(q.conj().T @ q, np.eye(n), atol=1e-12)
    k = n - 1 if n > 2 else n
    assert np.max(np.abs(q - ref)[:, :k]) < 1e-9
