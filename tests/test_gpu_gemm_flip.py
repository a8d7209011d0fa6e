"""Contractions with an operand conjugated on top of its op: the same bits as
the product of an operand that was conjugated beforehand."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F32, F64 = 0, 1
OPN, OPT, OPC, OPJ = 0, 1, 2, 3
FLIP_A, FLIP_B = 64, 128


@pytest.fixture(scope="module")
def capi():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import capi as c
    return c


@pytest.mark.parametrize("variant", [0, 1, 4, 1 + 32])
@pytest.mark.parametrize("flip", [FLIP_A, FLIP_B, FLIP_A + FLIP_B])
@pytest.mark.parametrize("combo", [(F32, F32, F32, F32, OPN, OPN), (F32, F32, F32, F32, OPC, OPN),
                                   (F32, F32, F64, F64, OPJ, OPT), (F64, F64, F64, F64, OPN, OPT)])
def test_flip(capi, combo, flip, variant):
    ta, tb, tc, tacc, opa, opb = combo
    if variant == 4 and tacc == F64:
        pytest.skip("the 128 x 128 tile exists for FP32 accumulation only")
    m, n, k, batch = 37, 29, 51, 2
    rng = np.random.default_rng(opa + 4 * flip)

    def rand(*shape, ct):
        x = rng.standard_normal(shape) + 1j * rng.standard_normal(shape)
        return x.astype(np.complex64).astype(np.complex128) if ct == F32 else x

    a = rand(batch, k, m, ct=ta) if opa == OPC else rand(batch, m, k, ct=ta)
    b = rand(batch, n, k, ct=tb) if opb == OPT else rand(batch, k, n, ct=tb)
    got = capi.dcs_test_gemm(ta, tb, tc, tacc, opa, opb, a, b, variant=variant + flip)
    ref = capi.dcs_test_gemm(ta, tb, tc, tacc, opa, opb, a.conj() if flip & FLIP_A else a,
                             b.conj() if flip & FLIP_B else b, variant=1)
    np.testing.assert_array_equal(got, ref)


def test_split_bf16_refuses(capi):
    a = np.ones((1, 4, 4), complex)
    with pytest.raises(RuntimeError):
        capi.dcs_test_gemm(F32, F32, F32, 2, OPN, OPN, a, a, variant=FLIP_A)
