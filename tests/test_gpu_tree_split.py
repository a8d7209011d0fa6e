"""Split sums of the tree contractions by batch: small batches cut the long sums
of contractions with few tiles into parts (whose sum is a launch more), batches
that fill the chip by themselves do not; the results agree."""
import numpy as np
import pytest

from inputs import circuits as C
from inputs.randomness import shot_uniforms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("c128", 1e-9), ("c64", 1e-5)])
def test_split_by_batch(prec, tol):
    """Launches that a run of 2 and one of 600 shots file under contractions and
    measurements, and the first two shots of both, F within the bounds that the
    parity tests use for the precision."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import engine as E
    circ, prm = C.workload("ttn27_chi32", chi=16)
    k = C.segment_max(circ) + 1
    eng = E.Engine(0)
    eng.tuning(False)
    out = []
    for shots in (2, 600):
        u = np.stack([shot_uniforms(prm["seed"], s % 2, circ.n_measurements()) for s in range(shots)])
        st = E.TreeState(eng, prec, prm["tree"], shots, 16, 16, [16], prm["init_seed"], circ=circ)
        eng.timing(True)
        eng.timing_stats(reset=True)
        r = E.run_single_path(eng, st, circ, shots, 16, k, 2, uniforms=u)
        launches = eng.timing_stats(reset=True)[0]
        eng.timing(False)
        out.append((sum(launches[:4]) + launches[6], r["outcomes"], r["p0s"], r["F"]))
        st.close()
    eng.close()
    assert out[0][0] > out[1][0]
    np.testing.assert_array_equal(out[0][1], out[1][1][:2])
    assert np.max(np.abs(out[0][2] - out[1][2][:2])) <= tol
    assert np.max(np.abs(out[0][3] / out[1][3][:2] - 1)) <= tol
