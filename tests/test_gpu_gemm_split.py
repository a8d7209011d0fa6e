"""Contractions whose sum is split into parts that are added afterwards: every
operand layout, parts of unequal length, more than one output tile, against the
product in float64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

F32, F64 = 0, 1
OPN, OPT, OPC, OPJ = 0, 1, 2, 3


@pytest.fixture(scope="module")
def capi():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import capi as c
    return c


@pytest.mark.parametrize("combo", [(F32, F32, F32, F32, OPN, OPN), (F32, F32, F32, F32, OPC, OPN),
                                   (F32, F32, F32, F32, OPJ, OPT), (F64, F64, F64, F64, OPC, OPN),
                                   (F32, F32, F64, F64, OPJ, OPT)])
@pytest.mark.parametrize("mnk,parts", [((1, 1, 512), 4), ((8, 8, 513), 4), ((3, 5, 2047), 16),
                                       ((33, 31, 700), 5), ((128, 8, 640), 5), ((1, 1, 32768), 64)])
def test_split(capi, combo, mnk, parts):
    ta, tb, tc, tacc, opa, opb = combo
    m, n, k = mnk
    rng = np.random.default_rng(k + m)
    batch = 2

    def rand(*shape, ct):
        x = rng.uniform(-1, 1, shape) + 1j * rng.uniform(-1, 1, shape)
        return x.astype(np.complex64).astype(np.complex128) if ct == F32 else x

    a = rand(batch, k, m, ct=ta) if opa == OPC else rand(batch, m, k, ct=ta)
    b = rand(batch, n, k, ct=tb) if opb == OPT else rand(batch, k, n, ct=tb)
    A = {OPN: a, OPC: np.conj(np.swapaxes(a, 1, 2)), OPJ: np.conj(a)}[opa]
    ref = A @ (np.swapaxes(b, 1, 2) if opb == OPT else b)
    u = 2.0 ** -52 if tacc == F64 else 2.0 ** -23
    for v in (0, 1, 2):
        got = capi.dcs_test_gemm(ta, tb, tc, tacc, opa, opb, a, b, variant=v + 256 * parts)
        # three real products of K terms of magnitude up to 2 each, rounded
        # per term
        assert np.max(np.abs(got - ref)) < 8 * u * k
