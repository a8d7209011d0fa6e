"""Which QR kernels a call of matrices of one shape takes (no GPU)."""
import pytest

capi = pytest.importorskip("paper_2609_26516_amd.capi")

BLOCKED, LARGE, UNBLOCKED, SPREAD, ONE = range(5)


@pytest.mark.parametrize("m,n,mode,batch,path", [
    (2, 1, 0, 1, ONE), (32, 16, 1, 4096, ONE), (48, 24, 0, 513, ONE), (64, 32, 0, 512, ONE),
    (50, 25, 0, 513, BLOCKED), (64, 32, 0, 513, BLOCKED), (96, 48, 1, 1024, BLOCKED),
    (128, 64, 0, 512, ONE), (128, 64, 0, 513, BLOCKED), (16, 16, 2, 1, BLOCKED), (8, 16, 0, 1, BLOCKED),
    (130, 65, 0, 96, SPREAD), (130, 65, 0, 97, BLOCKED), (512, 256, 1, 1, SPREAD),
    (514, 257, 0, 1, LARGE), (4096, 2048, 0, 1, UNBLOCKED),
])
def test_path(m, n, mode, batch, path):
    assert capi.dcs_test_qr_path(m, n, mode, batch) == path


def test_bad_arguments():
    with pytest.raises(capi.DcsError):
        capi.dcs_test_qr_path(0, 1, 0, 1)
