"""Which compression steps run in one launch: small bonds always, bonds up to 32
where the one launch is the faster form.  A step in one launch is timed as
class 7 alone; as launches it has contraction GEMMs (classes 0 to 3)."""
import numpy as np
import pytest

from inputs import circuits as C
from inputs.randomness import bra_init_gaussians

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


@pytest.mark.parametrize("prec,n,cap,layers,branches,one", [
    ("c128", 28, 16, 2, 1, True), ("c64", 28, 16, 2, 300, True),
    ("c128", 24, 24, 2, 1, True), ("c128", 12, 32, 2, 1, True), ("c64", 16, 32, 2, 1, True),
    ("c128", 24, 32, 1, 1, True),
    # many sites between bonds past 24 under two layers of gates: from some branches on
    ("c128", 16, 32, 2, 1, False), ("c128", 16, 28, 2, 23, False), ("c128", 16, 32, 2, 24, True),
    ("c128", 24, 32, 2, 1, False), ("c128", 24, 26, 2, 55, False), ("c128", 24, 32, 2, 56, True),
    ("c64", 24, 32, 2, 11, False), ("c64", 24, 32, 2, 12, True), ("c64", 28, 32, 2, 1, False),
    ("c64", 16, 32, 2, 257, False), ("c64", 12, 33, 2, 1, False),
])
def test_route(eng, prec, n, cap, layers, branches, one):
    from paper_2609_26516_amd import capi
    from paper_2609_26516_amd import engine as E
    rng = np.random.default_rng([n, cap])
    ops = [((q, q + 1), C.haar_unitary(rng, 4)) for l in range(layers) for q in range(l, n - 1, 2)]
    h = capi.dcs_chunk_compile(eng.ctx, n, [q[0] for q, _ in ops], [q[1] for q, _ in ops],
                               np.concatenate([m.reshape(-1) for _, m in ops]))
    gauss = bra_init_gaussians(n, cap, 3)
    st = E.State(eng, prec, n, branches, cap, 4, [cap], gaussians=lambda c: gauss)
    ids = st.alloc(branches)
    st.init_zero(ids, [cap] * branches)
    eng.timing(True)
    eng.timing_stats(reset=True)
    st.compress(ids, [h] * branches, 1)
    launches = eng.timing_stats(reset=True)[0]
    eng.timing(False)
    st.close()
    capi.dcs_chunk_destroy(h)
    assert (sum(launches[:4]) == 0) == one
