"""Collapse of one branch into a new slot, which goes as copy commands, beside
collapses of several, which take the copy kernel: the child equals the in-place
collapse of the same state bit for bit, with and without a cached left
transfer.  Launch timing (class 7) tells the two apart."""
import numpy as np
import pytest

from inputs.randomness import bra_init_gaussians

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c128", "c64"])
@pytest.mark.parametrize("copied", [1, 2])
@pytest.mark.parametrize("n,chi_max,cap", [(1, 1, 1), (7, 8, 3), (11, 32, 32), (16, 150, 149)])
def test_child_equals_in_place(n, chi_max, cap, copied, prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import capi
    from paper_2609_26516_amd import engine as E
    eng = E.Engine(0)
    eng.tuning(False)   # trials give the two measurements different tile shapes (FP64 rounding)
    st = E.State(eng, prec, n, 5, chi_max, 4, [chi_max],
                 gaussians=lambda c: bra_init_gaussians(n, c, 2))
    src, kids = [0, 1], [2, 3]
    for i in src:
        mps = [a / np.sqrt(2.0 * a.shape[2]) for a in bra_init_gaussians(n, cap, 50 + i)]
        capi.dcs_import_mps(st.h, i, cap, mps, eng.stream())
    for q in dict.fromkeys((n // 2, n - 1)):     # the second time with a cached transfer
        dst = kids[:copied] + src[copied:]       # the rest in place
        p = st.measure(src, [q, q])
        before = [st.export(i) for i in src]
        eng.timing(True)
        eng.timing_stats(reset=True)
        st.collapse(src, [q, q], [1, 1], dst, 1e-10)
        launches = eng.timing_stats(reset=True)[0]
        eng.timing(False)
        assert launches[7] == copied             # the collapse, and the copy kernel for two
        for i in range(copied):                  # the source is as it was
            for x, y in zip(st.export(src[i]), before[i]):
                np.testing.assert_array_equal(x, y)
        np.testing.assert_array_equal(st.measure(src, [q, q])[:copied], p[:copied])
        if copied == 2:
            st.collapse(src, [q, q], [1, 1], src, 1e-10)
        else:
            st.collapse(src[:1], [q], [1], src[:1], 1e-10)
        for a, b in zip(src[:copied], kids):
            for x, y in zip(st.export(a), st.export(b)):
                np.testing.assert_array_equal(x, y)
        np.testing.assert_array_equal(st.measure(src[:copied], [0] * copied),
                                      st.measure(kids[:copied], [0] * copied))
        capi.dcs_branch_release(st.h, kids[:copied])
    st.close()
    eng.close()
