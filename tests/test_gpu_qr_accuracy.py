"""Accuracy of the one-launch QR (kernel variant 8): the columns of Q have norm
1 as closely as LAPACK's Householder columns."""
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
