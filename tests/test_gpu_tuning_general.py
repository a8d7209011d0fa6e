"""Autotuned tile shapes of the compression step's own products: a run whose
steps are launches (bonds above 32) tunes them, plain and with the gate operator
applied, gives the same bits as a run with tuning off and as one that loads the
table."""
import json

import numpy as np
import pytest

from inputs import circuits as C
from inputs.randomness import shot_uniforms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,types", [("c128", [1, 1, 1, 1]), ("c64", [0, 0, 0, 0])])
def test_tuned_step_bit_identical(prec, types, tmp_path):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import engine as E
    circ, prm = C.workload("cfg4_n24_chi64_x1024", n=12, depth=8, chi=40)
    n, chi, shots = prm["n"], prm["chi"], 8
    k = C.segment_max(circ) + 1
    u = np.stack([shot_uniforms(prm["seed"], s, circ.n_measurements()) for s in range(shots)])
    path = str(tmp_path / "tiles.json")

    def run(tuning, load=False, save=False, repeats=1):
        eng = E.Engine(0)
        eng.tuning(tuning, 2)
        if load:
            eng.load_tuning(path)
        st = E.State(eng, prec, n, shots, chi, 4, [chi], prm["init_seed"])
        out = []
        for _ in range(repeats):
            r = E.run_single_path(eng, st, circ, shots, chi, k, 2, uniforms=u)
            out.append((r["p0s"].copy(), r["F"].copy(), [st.export(int(i)) for i in r["ids"]]))
            st.release(r["ids"])
        if save:
            eng.save_tuning(path)
        st.close()
        eng.close()
        return out

    base = run(False)[0]
    tuned = run(True, save=True, repeats=3)
    keys = [e["key"] for e in json.load(open(path))["entries"] if e["key"][:4] == types]
    # key[4]: form of A, plus 4 (8) with the gate operator applied moving right (left)
    assert any(q[4] >= 4 for q in keys) and any(q[4] < 4 for q in keys)
    for p0, f, mps in tuned + run(False, load=True):
        np.testing.assert_array_equal(p0, base[0])
        np.testing.assert_array_equal(f, base[1])
        for a, b in zip(mps, base[2]):
            for x, y in zip(a, b):
                np.testing.assert_array_equal(x, y)
