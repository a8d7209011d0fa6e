"""Both K steps of the 32x32 contraction tiles, on either side of the rule's
lines: the product in float64, and the bits of the 64x64 tiles (every tile
shape and step adds k in the same order)."""
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
                                   (F32, F32, F32, F32, OPN, OPT), (F32, F32, F32, F32, OPJ, OPT),
                                   (F64, F64, F64, F64, OPN, OPN), (F32, F64, F64, F64, OPC, OPN),
                                   (F32, F32, F64, F64, OPJ, OPT)])
@pytest.mark.parametrize("m,n,k,batch", [(1, 1, 1, 1), (5, 3, 33, 2), (33, 31, 66, 127), (33, 31, 66, 129),
                                         (31, 33, 96, 511), (31, 33, 96, 513), (20, 40, 20, 140),
                                         (32, 17, 7, 300), (40, 33, 132, 70), (17, 24, 41, 260)])
def test_step(capi, combo, m, n, k, batch):
    ta, tb, tc, tacc, opa, opb = combo
    rng = np.random.default_rng(m * 7 + n * 3 + k)
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
    np.testing.assert_array_equal(capi.dcs_test_gemm(ta, tb, tc, tacc, opa, opb, a, b, variant=0), c)


@pytest.mark.parametrize("ct", [F32, F64])
@pytest.mark.parametrize("direction", [0, 1])
@pytest.mark.parametrize("wl,wr", [(4, 4), (1, 4), (4, 2)])
@pytest.mark.parametrize("d0,d1,k", [(8, 8, 33), (100, 100, 40), (264, 264, 64)])
def test_gate_epilogue(capi, ct, direction, wl, wr, d0, d1, k):
    """Products with the gate operator applied: short steps by padding, by tiles,
    and long ones; the bits of the 64x64 tiles."""
    rng = np.random.default_rng([d0, k, direction])
    m, n = (d0 * wl, 2 * d1) if direction == 0 else (2 * d0, d1 * wr)
    a = _rand(rng, m, k)
    b = _rand(rng, k, n) if direction == 0 else _rand(rng, n, k)
    w = _rand(rng, wl, 2, 2, wr)
    if ct == F32:
        a, b, w = (x.astype(np.complex64).astype(np.complex128) for x in (a, b, w))
    c = capi.dcs_test_gemm_gate(ct, direction, a, b, w, variant=1)
    np.testing.assert_array_equal(capi.dcs_test_gemm_gate(ct, direction, a, b, w, variant=0), c)
