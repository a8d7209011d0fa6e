"""Tile loads of the contraction kernels: every remainder of a run, a line and
a step, rows that start on 16 bytes and rows that do not, and the form for
far-apart rows, against the product in float64 and against each other (every
tile shape and form adds k in the same order, so results are the same bits)."""
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


def _rand(rng, *shape):
    return rng.uniform(-1, 1, shape) + 1j * rng.uniform(-1, 1, shape)


@pytest.mark.parametrize("combo", [(F32, F32, F32, F32, OPN, OPN), (F32, F32, F32, F32, OPC, OPN),
                                   (F32, F32, F32, F32, OPJ, OPT), (F64, F64, F64, F64, OPN, OPT),
                                   (F64, F32, F64, F64, OPN, OPN), (F32, F64, F64, F64, OPJ, OPT)])
@pytest.mark.parametrize("mnk", [(1, 1, 1), (2, 3, 4), (31, 33, 31), (32, 32, 32), (33, 31, 33),
                                 (34, 66, 36), (65, 2, 95), (3, 65, 130), (129, 127, 17), (8, 8, 513)])
def test_loads(capi, combo, mnk):
    ta, tb, tc, tacc, opa, opb = combo
    m, n, k = mnk
    rng = np.random.default_rng(m * 7 + n * 3 + k)
    batch = 3   # odd sizes: items of the batch start off 16 bytes too
    a = _rand(rng, batch, k, m) if opa == OPC else _rand(rng, batch, m, k)
    b = _rand(rng, batch, n, k) if opb == OPT else _rand(rng, batch, k, n)
    if ta == F32:
        a = a.astype(np.complex64).astype(np.complex128)
    if tb == F32:
        b = b.astype(np.complex64).astype(np.complex128)
    A = {OPN: a, OPC: np.conj(np.swapaxes(a, 1, 2)), OPJ: np.conj(a)}[opa]
    ref = A @ (np.swapaxes(b, 1, 2) if opb == OPT else b)
    c = capi.dcs_test_gemm(ta, tb, tc, tacc, opa, opb, a, b, variant=1)
    # three real products of K terms of magnitude up to 2 each, rounded per term
    u = 2.0 ** -52 if tacc == F64 else 2.0 ** -23
    assert np.max(np.abs(c - ref)) < 8 * u * k + 4 * u
    for v in (0, 2, 3, 4, 1 + 32):
        if v == 4 and tacc == F64:
            continue
        np.testing.assert_array_equal(
            capi.dcs_test_gemm(ta, tb, tc, tacc, opa, opb, a, b, variant=v), c)
