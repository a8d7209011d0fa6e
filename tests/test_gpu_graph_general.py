"""HIP graph replays of cold-start compression steps that run as many launches:
grouped products with the gate operator, the QR in one launch, the spread QR
and the large-matrix QR.  Every replay equals the eager run bit for bit, with
eager measurements, collapses and synchronisation between the replays."""
import numpy as np
import pytest

from inputs import circuits as C
from inputs.randomness import shot_uniforms

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2609_26516_amd import engine
    return engine


@pytest.mark.parametrize("prec,n,depth,chi,shots", [
    ("c64", 12, 8, 40, 5), ("c128", 12, 8, 40, 5),       # QR of up to 80 x 40 in one launch
    ("c64", 14, 6, 48, 600),                             # two waves per matrix
    ("c64", 16, 4, 100, 3), ("c128", 16, 4, 100, 3),     # spread QR
    ("c64", 20, 4, 300, 1), ("bf16x3", 20, 4, 300, 1),   # large-matrix QR
])
def test_graph_replay_matches_eager(E, prec, n, depth, chi, shots):
    circ, prm = C.workload("cfg4_n24_chi64_x1024", n=n, depth=depth, chi=chi)
    k = C.segment_max(circ) + 1
    u = np.stack([shot_uniforms(prm["seed"], s, circ.n_measurements()) for s in range(shots)])
    kept = range(min(shots, 3))

    def run(graphs, repeats):
        eng = E.Engine(0)
        eng.graphs(graphs)
        # (shape trials move a Hermitian FP64 measurement product by one rounding)
        eng.tuning(False)
        st = E.State(eng, prec, n, shots, chi, 4, [chi], prm["init_seed"])
        out = []
        for _ in range(repeats):
            r = E.run_single_path(eng, st, circ, shots, chi, k, 2, uniforms=u)
            out.append((r, [st.export(int(r["ids"][i])) for i in kept]))
            st.release(r["ids"])
        st.close()
        eng.close()
        return out

    eager = run(False, 1)[0]
    for r, mps in run(True, 4):
        np.testing.assert_array_equal(r["outcomes"], eager[0]["outcomes"])
        np.testing.assert_array_equal(r["p0s"], eager[0]["p0s"])
        np.testing.assert_array_equal(r["F"], eager[0]["F"])
        for a, b in zip(mps, eager[1]):
            for x, y in zip(a, b):
                np.testing.assert_array_equal(x, y)
