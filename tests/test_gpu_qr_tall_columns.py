"""Column-by-column panels of the large QR path (a panel with an exactly zero
entry is factored that way), at the panel widths and row counts around which
its register shapes change."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F64 = 1
LARGE = 3


@pytest.fixture(scope="module")
def capi():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import capi as c
    return c


@pytest.mark.parametrize("m,n", [(600, 1), (600, 8), (600, 9), (1024, 16), (1025, 16), (1040, 24),
                                 (1041, 33), (2048, 7), (2048, 8), (2048, 9), (2048, 24), (2047, 40)])
def test_zero_entries(capi, m, n):
    rng = np.random.default_rng(3 * m + n)
    f = rng.standard_normal((m, n)) + 1j * rng.standard_normal((m, n))
    f[m // 2, ::3] = 0          # a zero in every panel, off the diagonal
    ref, _ = np.linalg.qr(f)
    q, _ = capi.dcs_test_qr(F64, F64, m, n, 0, LARGE, f.reshape(-1))
    q = q.reshape(m, n)
    # backward stable: a few units of rounding per reflector of a well
    # conditioned matrix, and at least the rounding of sums over m rows
    tol = 40 * 2.0 ** -53 * max(n, np.sqrt(m))
    np.testing.assert_allclose(q.conj().T @ q, np.eye(n), atol=tol)
    assert np.max(np.abs(q - ref)) < 10 * tol
