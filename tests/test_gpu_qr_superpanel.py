"""Q formation of the large QR path, several panels at a time: widths around
one and two superpanels and inside their last one, row counts that give three-
and four-panel superpanels, and one and two row chunks of W."""
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


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("m,n", [(200, 64), (200, 65), (300, 100), (513, 97), (768, 144), (769, 64),
                                 (769, 65), (1024, 79), (1300, 128), (1792, 129), (2048, 200)])
def test_superpanels(capi, m, n, mode):
    rng = np.random.default_rng(m + n)
    f = rng.standard_normal((m, n)) + 1j * rng.standard_normal((m, n))
    ref, _ = np.linalg.qr(f)
    g = f if mode == 0 else f.conj().T.copy()
    q, nrm2 = capi.dcs_test_qr(F64, F64, m, n, mode, LARGE, g.reshape(-1))
    q = q.reshape(m, n) if mode == 0 else q.reshape(n, m).conj().T
    # backward stable: a few units of rounding per reflector of a well
    # conditioned matrix
    tol = 40 * 2.0 ** -53 * n
    assert abs(nrm2 - np.sum(np.abs(f) ** 2)) < 1e-12 * nrm2
    np.testing.assert_allclose(q.conj().T @ q, np.eye(n), atol=tol)
    assert np.max(np.abs(q - ref)) < 10 * tol
