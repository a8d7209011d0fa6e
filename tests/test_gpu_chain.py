"""Compression steps of small branches, which run in one launch, against the
FP64 oracle and against the general path (a call that also holds a branch of a
larger bond cap takes that path for all its branches)."""
import numpy as np
import pytest

from inputs import circuits as C
from inputs.randomness import bra_init_gaussians
from oracle import mps as OM

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eng():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import engine as E
    e = E.Engine(0)
    yield e
    e.close()


def _ket(rng, n, chi, kind):
    d = OM.bond_dims(n, chi)
    out = []
    for j in range(n):
        a = rng.standard_normal((d[j], 2, d[j + 1])) + 1j * rng.standard_normal((d[j], 2, d[j + 1]))
        a /= np.sqrt(4.0 * d[j + 1])
        if kind == "deficient":      # every bond but the first column is noise or zero
            a[:, :, 1:] *= 1e-170 if j % 2 else 0.0
        out.append(a.astype(np.complex64).astype(np.complex128) if kind == "generic" else a)
    return out


def _ops(rng, n, layers, far):
    ops = [((q, q + 1), C.haar_unitary(rng, 4)) for l in range(layers) for q in range(l % 2, n - 1, 2)]
    if far:   # a pair of gates over distance, bond 16 in the middle of the chain
        ops = [((0, n - 1), C.haar_unitary(rng, 4)), ((n - 2, 1), C.haar_unitary(rng, 4))]
    return ops


def _norms(mps, q):
    e, g = np.eye(mps[0].shape[0]), np.eye(mps[-1].shape[2])
    for a in mps[:q]:
        e = np.einsum("ab,asc,bsd->cd", e, a.conj(), a, optimize=True)
    for a in mps[:q:-1]:
        g = np.einsum("asc,bsd,cd->ab", a.conj(), a, g, optimize=True)
    return [float(np.einsum("ab,ac,bd,cd->", e, mps[q][:, m].conj(), mps[q][:, m], g,
                            optimize=True).real) for m in (0, 1)]


CASES = [
    # n, ket cap, bra cap, layers, far, sweeps
    (1, 1, 1, 0, False, 2), (2, 2, 2, 1, False, 3), (3, 1, 2, 2, False, 2), (5, 3, 3, 2, False, 1),
    (6, 8, 5, 2, False, 4), (9, 15, 15, 2, False, 2), (9, 16, 16, 1, False, 3),
    (9, 16, 16, 0, True, 2), (10, 17, 17, 2, False, 2), (11, 16, 31, 2, False, 2),
    (12, 32, 32, 2, False, 1), (12, 32, 32, 1, False, 2), (8, 7, 11, 3, False, 2),
]


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("kind", ["generic", "deficient"])
@pytest.mark.parametrize("n,kcap,bcap,layers,far,sweeps", CASES)
def test_one_launch_step(eng, n, kcap, bcap, layers, far, sweeps, kind, prec):
    from paper_2609_26516_amd import capi
    from paper_2609_26516_amd import engine as E
    rng = np.random.default_rng([n, kcap, bcap, layers, sweeps])
    ket = _ket(rng, n, kcap, kind)
    ops = _ops(rng, n, layers, far) or [((0,), C.haar_unitary(rng, 2))]
    gauss = {c: bra_init_gaussians(n, c, 3) for c in {bcap, 48}}
    st = E.State(eng, prec, n, 3, 48, 16, sorted(gauss), gaussians=gauss.get)
    h = capi.dcs_chunk_compile(eng.ctx, n, [q[0] for q, _ in ops],
                               [q[1] if len(q) == 2 else -1 for q, _ in ops],
                               np.concatenate([m.reshape(-1) for _, m in ops]))
    for i, cap in enumerate((bcap, bcap, 48)):
        capi.dcs_import_mps(st.h, i, cap, ket, eng.stream())
    f = st.compress([0], [h], sweeps)[0]
    got = st.export(0)
    f2 = st.compress([1, 2], [h, h], sweeps)[0]   # n >= 11: cap 48 is wider than 32
    other = st.export(1)
    ref, fr, _ = OM.compress(ket, OM.chunk_mpo(n, ops), OM.generic_bra(gauss[bcap]), sweeps)
    tol_f, tol_s = (1e-9, 1e-9) if prec == "c128" else (1e-5, 1e-6)
    nk = OM.norm_sq(ket) if kind == "deficient" else 1.0   # f scales with the ket's norm
    assert abs(f - fr) <= tol_f * max(nk, fr) and abs(f2 - f) <= tol_f * max(nk, fr)
    for a in (got, other):
        fid = abs(OM.overlap(ref, a)) ** 2 / (OM.norm_sq(ref) * OM.norm_sq(a))
        assert abs(1 - fid) <= tol_s
    if kind == "generic" and prec == "c128" and layers == 2 and kcap == bcap:
        for x, y in zip(got, ref):   # full rank: the tensors themselves, signs of the QR included
            assert np.max(np.abs(x - y)) <= 1e-9
    capi.dcs_chunk_destroy(h)
    st.close()


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("n,cap", [(1, 1), (2, 2), (5, 3), (8, 15), (9, 16), (9, 17)])
def test_one_launch_measurement(eng, n, cap, prec):
    """Outcome norms in one launch (bonds up to 16) and per site (above):
    every qubit order, cached left transfer, states in no canonical form and
    after a compression step.  The reference contracts the exported tensors in
    FP64 over the same sites (transfers are the identity left of the last
    left-canonical site and right of the first right-canonical one), so FP64
    rounding of the contraction is all that separates the two sides."""
    from paper_2609_26516_amd import capi
    from paper_2609_26516_amd import engine as E
    rng = np.random.default_rng([n, cap])
    gauss = bra_init_gaussians(n, cap, 3)
    st = E.State(eng, prec, n, 2, cap, 4, [cap], gaussians=lambda c: gauss)
    ops = [((q, q + 1), C.haar_unitary(rng, 4)) for q in range(n - 1)] or [((0,), C.haar_unitary(rng, 2))]
    h = capi.dcs_chunk_compile(eng.ctx, n, [q[0] for q, _ in ops],
                               [q[1] if len(q) == 2 else -1 for q, _ in ops],
                               np.concatenate([m.reshape(-1) for _, m in ops]))
    for sweeps in (0, 1, 2):   # no canonical form, centre at the end, centre at site 0
        for i in range(2):
            capi.dcs_import_mps(st.h, i, cap, _ket(rng, n, cap, "generic"), eng.stream())
        if sweeps:
            st.compress([0, 1], [h, h], sweeps)
        mps = [st.export(i) for i in range(2)]
        for q in [n // 2, n - 1, 0, n // 2, *range(n)]:
            other = n - 1 - q
            got = st.measure([0, 1], [q, other])
            for g, m, k in zip(got, mps, (q, other)):
                c = None if sweeps == 0 else (n - 1 if sweeps == 1 else 0)   # orthogonality centre
                lo = min(0 if c is None else c, k)
                hi = max(n if c is None else c + 1, k + 1)
                n0, n1 = _norms(m[lo:hi], k - lo)
                assert abs(g - n0 / (n0 + n1)) <= 1e-12
    capi.dcs_chunk_destroy(h)
    st.close()
