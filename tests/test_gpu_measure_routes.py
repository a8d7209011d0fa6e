"""Outcome norms of a branch of small bonds in one launch and as launches (a call
that also holds a branch of larger bonds): the cached left transfer that one
form leaves is taken up by the other."""
import numpy as np
import pytest

from inputs.randomness import bra_init_gaussians
from oracle import mps as OM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c128", "c64"])
def test_cached_transfer_across_forms(prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import capi
    from paper_2609_26516_amd import engine as E
    n = 12
    eng = E.Engine(0)
    st = E.State(eng, prec, n, 3, 40, 1, [40], gaussians=lambda c: bra_init_gaussians(n, c, 2))
    small = [a / np.sqrt(2.0 * a.shape[2]) for a in bra_init_gaussians(n, 13, 5)]
    large = [a / np.sqrt(2.0 * a.shape[2]) for a in bra_init_gaussians(n, 40, 6)]
    ref_p = {}
    for i, m in ((0, small), (1, small), (2, large)):
        capi.dcs_import_mps(st.h, i, 13 if i < 2 else 40, m, eng.stream())
    exact = st.export(0)

    def p0(q):
        if q not in ref_p:
            n0 = OM.norm_sq([a if j != q else a * np.array([1.0, 0.0])[None, :, None]
                             for j, a in enumerate(exact)])
            ref_p[q] = n0 / OM.norm_sq(exact)
        return ref_p[q]

    # (measured together with the large branch or alone), along the chain and back
    for q, joint in ((2, False), (5, True), (7, False), (7, True), (9, False), (11, True), (4, False),
                     (6, True), (0, True), (3, False)):
        if joint:
            got = st.measure([0, 2], [q, n - 1 - q])[0]
        else:
            got = st.measure([0], [q])[0]
        assert abs(got - p0(q)) <= 1e-12
        assert abs(st.measure([1], [q])[0] - p0(q)) <= 1e-12
    st.close()
    eng.close()
