"""Launch timing of tree runs whose contractions split long sums: every launch is
filed under one of the classes, and timing leaves the results as they are."""
import numpy as np
import pytest

from inputs import circuits as C
from inputs.randomness import shot_uniforms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c64", "c128"])
def test_timed_tree_run(prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import engine as E
    circ, prm = C.workload("ttn27_chi32")
    chi, shots = prm["chi"], 3
    k = C.segment_max(circ) + 1
    u = np.stack([shot_uniforms(prm["seed"], s, circ.n_measurements()) for s in range(shots)])
    eng = E.Engine(0)
    st = E.TreeState(eng, prec, prm["tree"], shots, chi, 16, [chi], prm["init_seed"], circ=circ)
    runs = []
    for timed in (False, True, True, False):
        eng.timing(timed)
        eng.timing_stats(reset=True)
        r = E.run_single_path(eng, st, circ, shots, chi, k, 2, uniforms=u)
        st.release(r["ids"])
        runs.append((r["outcomes"], r["p0s"], r["F"]))
        launches, ms, flops, byts = eng.timing_stats(reset=True)
        if timed:
            assert sum(launches[:4]) > 100 and launches[5] > 0 and launches[6] > 0 and launches[7] > 0
            for v in (launches, ms, flops, byts):
                assert all(np.isfinite(x) and x >= 0 for x in v)
            assert 0 < sum(ms) < 60e3
        else:
            assert not any(launches)
    for other in runs[1:]:
        for a, b in zip(runs[0], other):
            np.testing.assert_array_equal(a, b)
    st.close()
    eng.close()
