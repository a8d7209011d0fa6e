"""Rule of the K step of the 32x32 contraction tiles (no GPU): long steps where a
launch leaves room on the CUs and the step does not mostly pad, else 8 columns."""
import pytest

capi = pytest.importorskip("paper_2609_26516_amd.capi")

F32, F64 = 0, 1


@pytest.mark.parametrize("tacc,m,n,k,batch,step", [
    (F32, 1, 1, 1, 1, 8), (F32, 32, 32, 32, 1, 32), (F32, 33, 66, 33, 1, 8), (F32, 40, 80, 40, 75, 8),
    (F32, 90, 45, 180, 1, 32), (F32, 32, 32, 66, 256, 32), (F32, 32, 32, 66, 257, 8),
    (F32, 64, 64, 90, 256, 32), (F32, 64, 64, 90, 257, 8), (F32, 64, 64, 64, 1024, 8),
    (F64, 20, 20, 40, 1, 8), (F64, 20, 20, 48, 1, 16), (F64, 33, 33, 66, 64, 8), (F64, 32, 32, 132, 256, 16),
    (F64, 32, 32, 132, 257, 8), (F64, 32, 32, 64, 1024, 16), (F64, 32, 32, 64, 1025, 8),
])
def test_step(tacc, m, n, k, batch, step):
    assert capi.dcs_test_gemm_step(tacc, m, n, k, batch) == step


def test_bad_arguments():
    with pytest.raises(capi.DcsError):
        capi.dcs_test_gemm_step(7, 1, 1, 1, 1)
    with pytest.raises(capi.DcsError):
        capi.dcs_test_gemm_step(F32, 1, 1, 0, 1)
