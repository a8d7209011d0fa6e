"""Work that launch timing reports for a compression step in one launch (class
7): the flops that the same step counts as launches, contractions, operators
and QRs together."""
import numpy as np
import pytest

from inputs import circuits as C
from inputs.randomness import bra_init_gaussians

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


@pytest.mark.parametrize("cap,far,sweeps", [(16, False, 1), (16, True, 2), (13, False, 3), (30, False, 4)])
def test_flops_of_one_launch(eng, cap, far, sweeps):
    from paper_2609_26516_amd import capi
    from paper_2609_26516_amd import engine as E
    rng = np.random.default_rng([cap, sweeps])
    ops = [((q, q + 1), C.haar_unitary(rng, 4)) for l in range(2) for q in range(l, N - 1, 2)]
    if far:
        ops = [((0, N - 1), C.haar_unitary(rng, 4)), ((N - 2, 1), C.haar_unitary(rng, 4))]
    h = capi.dcs_chunk_compile(eng.ctx, N, [q[0] for q, _ in ops], [q[1] for q, _ in ops],
                               np.concatenate([m.reshape(-1) for _, m in ops]))
    gauss = {c: bra_init_gaussians(N, c, 3) for c in (cap, 40)}
    st = E.State(eng, "c128", N, 3, 40, 16, sorted(gauss), gaussians=gauss.get)

    def flops(ids, caps):
        st.init_zero(ids, caps)
        st.compress(ids, [h] * len(ids), 1)   # bonds at their caps from here on
        eng.timing(True)
        eng.timing_stats(reset=True)
        st.compress(ids, [h] * len(ids), sweeps)
        launches, _, f, _ = eng.timing_stats(reset=True)
        eng.timing(False)
        capi.dcs_branch_release(st.h, ids)
        return list(launches), list(f)

    one, f_one = flops([0, 1], [cap, cap])
    both, f_both = flops([0, 1, 2], [cap, cap, 40])
    large, f_large = flops([2], [40])
    assert sum(one[:7]) == 0 and one[7] == 1
    assert sum(both[:4]) > 0 and sum(large[:4]) > 0
    ref = sum(f_both) - sum(f_large)
    assert abs(f_one[7] - ref) <= 1e-9 * ref
    capi.dcs_chunk_destroy(h)
    st.close()
