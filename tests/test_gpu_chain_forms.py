"""The forms of the one-launch compression step (every intermediate in LDS, only
X, none) in calls of several bond caps, operators and starting states: every
branch against the same branch taken through the general path (a call that
also holds a branch whose bonds go past 32), against its copies in the same
call, and against a second run of the call, bit for bit.  A step turns between
its sweeps, where a visit reads the environment that the visit before it
stored."""
import numpy as np
import pytest

from inputs import circuits as C
from inputs.randomness import bra_init_gaussians
from oracle import mps as OM

pytestmark = pytest.mark.gpu

N = 12   # the middle bond reaches 64, so a cap of 40 takes the general path


@pytest.fixture(scope="module")
def eng():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import engine as E
    e = E.Engine(0)
    yield e
    e.close()


def _ket(rng, cap):
    d = OM.bond_dims(N, cap)
    return [(rng.standard_normal((d[j], 2, d[j + 1])) + 1j * rng.standard_normal((d[j], 2, d[j + 1])))
            / np.sqrt(4.0 * d[j + 1]) for j in range(N)]


def _chunk(eng, rng, bond):
    from paper_2609_26516_amd import capi
    if bond == 16:
        ops = [((0, N - 1), C.haar_unitary(rng, 4)), ((N - 2, 1), C.haar_unitary(rng, 4))]
    else:
        ops = [((q, q + 1), C.haar_unitary(rng, 4)) for l in range(2) for q in range(l, N - 1, 2)]
    return capi.dcs_chunk_compile(eng.ctx, N, [q[0] for q, _ in ops], [q[1] for q, _ in ops],
                                  np.concatenate([m.reshape(-1) for _, m in ops]))


# LDS form taken at these sizes: all (c128 16/4, c64 16/4), X only (c64 16/16,
# c64 28/4, c128 16/4 from 257 branches on), none (c128 16/16, c128 32/4,
# c64 16/16 from 257 branches on)
@pytest.mark.parametrize("prec,cap,bond,branches", [
    ("c128", 16, 4, 13), ("c64", 16, 4, 13), ("c64", 16, 16, 13), ("c64", 28, 4, 13),
    ("c128", 16, 16, 13), ("c128", 32, 4, 13), ("c128", 16, 4, 300), ("c64", 16, 16, 300),
    ("c64", 7, 4, 300)])
@pytest.mark.parametrize("sweeps", [1, 3, 4])
def test_branches_of_a_call(eng, prec, cap, bond, branches, sweeps):
    from paper_2609_26516_amd import capi
    from paper_2609_26516_amd import engine as E
    rng = np.random.default_rng([cap, bond, sweeps])
    caps = (cap, max(2, cap - 3))
    kets = [_ket(rng, caps[0]), _ket(rng, caps[1]), _ket(rng, caps[0])]
    chunks = [_chunk(eng, rng, bond) for _ in range(3)]
    gauss = {c: bra_init_gaussians(N, c, 3) for c in {*caps, 40}}
    st = E.State(eng, prec, N, branches + 1, 40, 16, sorted(gauss), gaussians=gauss.get)
    # interleaved caps, states and operators: 18 kinds of branches
    kind = [(caps[i % 2], i % 3, (i // 2) % 3) for i in range(branches)]

    def load(i, k):
        capi.dcs_import_mps(st.h, i, k[0], kets[k[1]], eng.stream())

    runs = []
    for _ in range(2):
        for i, k in enumerate(kind):
            load(i, k)
        f = st.compress(list(range(branches)), [chunks[k[2]] for k in kind], sweeps)
        runs.append((f, [st.export(i) for i in range(branches)]))
    (f, got), (f2, got2) = runs
    np.testing.assert_array_equal(f, f2)
    for x, y in zip(got, got2):
        for a, b in zip(x, y):
            np.testing.assert_array_equal(a, b)
    # f of a branch is computed in the path precision: the bounds of the
    # one-launch step against the oracle
    tol_f, tol_s = (1e-9, 1e-9) if prec == "c128" else (1e-5, 1e-6)
    first = {}
    for i, k in enumerate(kind):
        if k in first:   # a copy: the same bits
            assert f[i] == f[first[k]]
            for a, b in zip(got[i], got[first[k]]):
                np.testing.assert_array_equal(a, b)
            continue
        first[k] = i
        load(i, k)
        load(branches, (40, k[1]))
        ref_f = st.compress([i, branches], [chunks[k[2]]] * 2, sweeps)[0]
        ref = st.export(i)
        assert abs(f[i] - ref_f) <= tol_f * ref_f
        fid = abs(OM.overlap(ref, got[i])) ** 2 / (OM.norm_sq(ref) * OM.norm_sq(got[i]))
        assert abs(1 - fid) <= tol_s
    for h in chunks:
        capi.dcs_chunk_destroy(h)
    st.close()
