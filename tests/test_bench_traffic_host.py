"""The bench's HBM traffic figure of the QR launches stands for every kernel that
they take and for the choice among them (no GPU)."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402

CSRC = os.path.join(ROOT, "paper_2609_26516_amd", "csrc")


def test_every_kernel_file_of_the_choice_is_covered():
    """Files with a kernel that run_qr launches for matrices of up to 512 rows in
    large batches, and the project headers these include."""
    want, todo = set(), ["kernels.hip", "qr_mid.hip"]
    while todo:
        name = todo.pop()
        want.add(name)
        for line in open(os.path.join(CSRC, name)):
            if line.startswith('#include "') and not line.startswith('#include "dcs'):
                inc = line.split('"')[1]
                if inc not in want:
                    todo.append(inc)
    have = {os.path.basename(p) for p in bench.TRAFFIC["qr"]["src"]}
    assert want <= have


def test_a_changed_choice_drops_the_figure(monkeypatch):
    t = dict(bench.TRAFFIC["qr"])
    text = bench.traffic_sources(t)
    assert b"qr_forms" in text and b"launch_qr_mid" in text
    monkeypatch.setitem(bench.TRAFFIC, "qr", t)
    monkeypatch.setattr(bench, "traffic_sources", lambda t: text + b" ")
    assert bench.measured_traffic("qr") is None
