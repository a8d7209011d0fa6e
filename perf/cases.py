"""The work that programs have this framework do, as cases that can be timed.

A case is a dict of plain values.  Five kinds:

  paths  a whole multi-path run (Alg. 2) of the teleportation protocol
  run    a whole batch of single-path shots (Alg. 1) of a circuit
  tree   the same on a tree tensor network
  round  one measurement round of a batch of branches in mid-circuit: measure a
         qubit, collapse every branch into a new slot, compress the next chunk,
         measure and collapse again, measure once more
  state  import a few states, compress one chunk, export the results

Numbers of the complex64 and split-BF16 forms are handed on as float32, their
storage type; those of the complex128 form as float64.
"""
from __future__ import annotations

import math

import numpy as np

from inputs import circuits as C
from inputs.randomness import shot_uniforms

CHECKED = 2          # shots or branches of a batch that exact() works out
FANOUT = 16          # branches of a round made from one imported state
TREES = {27: (1, 3, 9, 27), 16: (1, 2, 4, 8, 16), 9: (1, 3, 9)}


def listed():
    return [
        # the smallest call there is: three qubits, five gates, three
        # measurements with classical control; every launch is latency
        dict(name="teleport_paths", kind="paths", n=3, chi=2, precision="c128"),
        # the sampling study of the dynamic GHZ preparation (13 qubits, bond
        # cap 4): many tiny shots and measurements
        dict(name="ghz13_128shots", kind="run", circuit="ghz", n=13, depth=1, chi=4, shots=128,
             precision="c128", sampling="host"),
        # one shot of a small brickwork circuit, the interactive use
        dict(name="n10_chi16_1shot", kind="run", circuit="brickwork", n=10, depth=10, chi=16,
             shots=1, precision="c128", sampling="host"),
        # the random-circuit study: 27 qubits, gates on any pair of qubits
        # (operator bonds up to 16), a batch of 10 runs
        dict(name="n27_chi16_random", kind="run", circuit="random", n=27, depth=3, chi=16,
             shots=10, precision="c128", sampling="host"),
        # medium bond caps, outcomes drawn on the device; an odd cap and batch
        dict(name="n22_chi45_device", kind="run", circuit="brickwork", n=22, depth=6, chi=45,
             shots=75, precision="c64", sampling="device"),
        # the throughput batch of the 24-qubit circuit: 1024 shots, one-layer chunks
        dict(name="n24_chi64_1024", kind="round", n=24, chi=64, branches=1024, mixed=False,
             layers=1, sweeps=2, precision="c64", warm=-1.0),
        # the headline shape: 256 shots at bond cap 256 in one batch
        dict(name="n26_chi256_256", kind="round", n=26, chi=256, branches=256, mixed=False,
             layers=2, sweeps=2, precision="c64", warm=-1.0),
        # multi-path branches: bond caps from 32 to 256 in one call
        dict(name="n28_mixed_48", kind="round", n=28, chi=256, branches=48, mixed=True,
             layers=2, sweeps=2, precision="c64", warm=-1.0),
        # the plain double-precision path at a ragged cap, started from the ket
        dict(name="n20_chi100_c128", kind="round", n=20, chi=100, branches=30, mixed=False,
             layers=2, sweeps=2, precision="c128", warm=1e-3),
        # the largest bond cap: few sites of 1024, three-layer chunks (operator
        # bond 16), split-BF16 contractions, one branch
        dict(name="n22_chi1024_bf16x3", kind="round", n=22, chi=1024, branches=1, mixed=False,
             layers=3, sweeps=2, precision="bf16x3", warm=-1.0),
        # states in, states out (the tensors themselves come back), one sweep
        dict(name="n14_chi48_states", kind="state", n=14, chi=48, branches=4, layers=2, sweeps=1,
             precision="c128"),
        # the tree of the paper's tree runs
        dict(name="tree27_chi32_64", kind="tree", n=27, chi=32, depth=4, shots=64,
             precision="c64"),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["paths", "run", "run", "run", "round", "round", "round", "state", "tree"])
        prec = rng.choice(["c64", "c64", "c128"])
        if kind == "paths":
            return dict(kind=kind, n=3, chi=rng.choice([2, 3, 4]), precision=prec,
                        salt=rng.randrange(1 << 20))
        if kind == "run":
            circ = rng.choice(["ghz", "brickwork", "brickwork", "random"])
            if circ == "ghz":
                c = dict(kind=kind, circuit=circ, n=2 * rng.randint(2, 8) + 1, depth=1,
                         chi=rng.randint(3, 6), shots=log(1, 300), precision=prec)
            elif circ == "random":
                c = dict(kind=kind, circuit=circ, n=rng.randint(12, 27), depth=rng.randint(2, 4),
                         chi=log(6, 32), shots=log(1, 20), precision=prec,
                         salt=rng.randrange(1 << 20))
            else:
                c = dict(kind=kind, circuit=circ, n=rng.randint(8, 26), depth=2 * rng.randint(2, 5),
                         chi=log(8, 100), shots=log(1, 128), precision=prec)
            c["sampling"] = rng.choice(["host", "host", "device"])
        elif kind == "round":
            prec = rng.choice([prec, prec, prec, "bf16x3"])
            c = dict(kind=kind, n=rng.randint(12, 28), chi=log(12, 400), branches=log(1, 512),
                     mixed=rng.random() < 0.3, layers=rng.choice([1, 2, 2, 3]),
                     sweeps=rng.choice([1, 2, 2, 3]), precision=prec,
                     warm=rng.choice([-1.0, -1.0, 1e-3]))
            if c["mixed"] and c["chi"] < 32:
                continue
        elif kind == "state":
            c = dict(kind=kind, n=rng.randint(6, 16), chi=log(4, 64), branches=rng.randint(1, 6),
                     layers=rng.choice([1, 2]), sweeps=rng.choice([1, 2]), precision="c128")
        else:
            n = rng.choice(sorted(TREES))
            c = dict(kind=kind, n=n, chi=log(3, 32), depth=2 * rng.randint(1, 2),
                     shots=log(1, 64), precision=prec)
        if _cost(c) <= 0.6 * most and _slot_bytes(c) <= 24e9:
            return c


# ---------------------------------------------------------------------------
# Inputs

def _dims(n, chi):
    return [min(chi, 2 ** b, 2 ** (n - b)) for b in range(n + 1)]


def _gaussians(n, chi, seed):
    """Site tensors of the starting guess, as the state takes them."""
    rng = np.random.default_rng([int(seed), n, chi, 1])
    d = _dims(n, chi)
    return [(rng.standard_normal((d[j], 2, d[j + 1])) + 1j * rng.standard_normal((d[j], 2, d[j + 1])))
            / np.sqrt(2.0) for j in range(n)]


def _random_mps(n, chi, seed, precision):
    """A generic state of bond cap chi: Gaussian site tensors whose rows are
    orthonormal on average (full Schmidt rank at every bond, norm near 1)."""
    rng = np.random.default_rng([int(seed), n, chi, 2])
    d = _dims(n, chi)
    out = []
    for j in range(n):
        a = rng.standard_normal((d[j], 2, d[j + 1], 2), dtype=np.float32)
        a = a.view(np.complex64)[..., 0] * np.float32(1.0 / math.sqrt(4.0 * d[j + 1]))
        out.append(a.astype(np.complex128) if precision == "c128" else a)
    return out


def _layers(n, layers, seed):
    """Gates of `layers` Haar brickwork layers, as (qubits, matrix)."""
    rng = np.random.default_rng([int(seed), n, layers, 3])
    ops = []
    for layer in range(layers):
        for q in range(layer % 2, n - 1, 2):
            ops.append(((q, q + 1), C.haar_unitary(rng, 4)))
    return ops


def _caps(case):
    """Bond caps of a round's branches and of the states that they come from."""
    b, chi = case["branches"], case["chi"]
    if not case["mixed"]:
        return [chi] * b, [chi]
    choices = sorted({max(4, chi * k // 8) for k in range(1, 9)})
    rng = np.random.default_rng([b, chi, 4])
    return [int(choices[i]) for i in rng.integers(len(choices), size=b)], choices


def _round_plan(case, seed):
    """Per branch: the imported state it comes from, that measurement's qubit
    and outcome, the outcomes of the round; and the round's qubits."""
    n, b = case["n"], case["branches"]
    rng = np.random.default_rng([int(seed), n, b, 5])
    order = [int(q) for q in rng.permutation(n)]
    q, start = sorted(order[:3]), order[3:3 + FANOUT // 2]   # n >= 12: no qubit twice
    plan = [(i // FANOUT, start[(i % FANOUT) // 2], i % 2) for i in range(b)]
    outcomes = rng.integers(2, size=(2, b)).astype(np.int32)
    outcomes[:, min(2, b - 1)] = outcomes[:, 0]   # a pair whose overlap is not zero
    return plan, q, outcomes


def _circuit(case, seed):
    if case["kind"] == "paths":
        v = np.random.default_rng([int(seed), case.get("salt", 0)]).standard_normal(4)
        return C.teleportation(True, (complex(v[0], v[1]), complex(v[2], v[3])))
    if case["kind"] == "tree":
        return C.brickwork(case["n"], case["depth"], 2, 2, "x_right", int(seed))
    if case["circuit"] == "ghz":
        return C.ghz_dynamic(case["n"])
    if case["circuit"] == "random":
        # one circuit, so that every seed measures as often
        return C.random_dynamic(case["n"], case["depth"], case.get("salt", 0))
    return C.brickwork(case["n"], case["depth"], 2, 2, "x_right", int(seed))


def _chunk_limit(case, circ):
    """Chunk size k and largest operator bond of a run."""
    if case["kind"] == "run" and case["circuit"] in ("ghz", "random"):
        return (25 if case["circuit"] == "ghz" else 20), (4 if case["circuit"] == "ghz" else 16)
    return C.segment_max(circ) + 1, 16 if case["kind"] == "tree" else 4


# ---------------------------------------------------------------------------
# The framework

_ENGINE = []


def _engine():
    """One engine, as a program keeps it."""
    if not _ENGINE:
        from paper_2609_26516_amd import engine
        _ENGINE.append(engine.Engine(0))
    return _ENGINE[0]


class _Holder(dict):
    """A prepared case; gives its branch slots back when it goes."""

    def __del__(self):
        st = self.pop("st", None)
        if st is not None:
            st.close()


def prepare(case, seed):
    from paper_2609_26516_amd import capi
    from paper_2609_26516_amd import engine as E
    eng, kind, n, chi, prec = _engine(), case["kind"], case["n"], case["chi"], case["precision"]
    guess = lambda cap: _gaussians(n, cap, seed)  # noqa: E731
    if kind in ("paths", "run", "tree"):
        circ = _circuit(case, seed)
        k, wmax = _chunk_limit(case, circ)
        s = _Holder(case=case, circ=circ, k=k)
        if kind == "tree":
            s["st"] = E.TreeState(eng, prec, TREES[n], case["shots"], chi, init_chis=[chi],
                                  init_seed=int(seed) % 1000, circ=circ)
        else:
            slots = 2 * 2 ** circ.n_measurements() + 2 if kind == "paths" else case["shots"]
            s["st"] = E.State(eng, prec, n, slots, chi, wmax, [chi], gaussians=guess)
        if kind != "paths":
            nm = circ.n_measurements()
            s["u"] = np.stack([shot_uniforms(int(seed), i, nm) for i in range(case["shots"])])
        return s
    ops = _layers(n, case["layers"], seed)
    wmax = 4 ** ((case["layers"] + 1) // 2)
    x0 = [((q,), C.X) for q in (0, n // 2)]

    def chunk(extra):
        every = ops + extra
        return capi.dcs_chunk_compile(eng.ctx, n, [g[0][0] for g in every],
                                      [g[0][1] if len(g[0]) == 2 else -1 for g in every],
                                      np.concatenate([g[1].reshape(-1) for g in every]))

    b, stream = case["branches"], eng.stream()
    if kind == "state":
        st = E.State(eng, prec, n, b, chi, wmax, [chi], gaussians=guess)
        return _Holder(case=case, st=st, ids=st.alloc(b), chunks=[chunk([])] * b,
                       mps=[_random_mps(n, chi, seed + 1000 * i, prec) for i in range(b)])
    caps, kinds = _caps(case)
    plan, q, outcomes = _round_plan(case, seed)
    bases = plan[-1][0] + 1
    st = E.State(eng, prec, n, 2 * b + bases, chi, wmax, kinds, gaussians=guess)
    if case["warm"] >= 0:
        st.warm_start(case["warm"])
    s = _Holder(case=case, st=st, kets=st.alloc(b), kids=st.alloc(b), caps=caps, q=q,
                out=outcomes, chunks=None)
    for i in range(bases):
        slot = st.alloc(1)[0]
        cap = kinds[-1 - i % len(kinds)]
        capi.dcs_import_mps(st.h, slot, cap, _random_mps(n, cap, seed + 1000 * i, prec), stream)
        for q0 in dict.fromkeys(p[1] for p in plan if p[0] == i):
            mine = [(j, p) for j, p in enumerate(plan) if p[0] == i and p[1] == q0]
            st.measure([slot], [q0])
            st.collapse([slot] * len(mine), [q0] * len(mine), [p[2] for _, p in mine],
                        [s["kets"][j] for j, _ in mine], E.EPS_BRANCH)
    plain, flipped = chunk([]), chunk(x0)
    s["chunks"] = [flipped if m else plain for m in outcomes[0]]
    return s


def _num(x, precision):
    return np.asarray(x, dtype=np.float64 if precision == "c128" else np.float32)


def _split(out):
    """Batch outputs as the items that exact() works out and the others."""
    return {"checked": {k: v[:CHECKED] for k, v in out.items()},
            "others": {k: v[CHECKED:] for k, v in out.items()}}


def run(s):
    from paper_2609_26516_amd import capi
    from paper_2609_26516_amd import engine as E
    case, st, eng = s["case"], s["st"], _engine()
    kind, prec, n = case["kind"], case["precision"], case["n"]
    if kind == "paths":
        r = E.run_multi_path(eng, st, s["circ"], case["chi"], s["k"])
        st.release([b["id"] for b in r["branches"]])
        br = sorted(r["branches"], key=lambda b: b["path"])
        return {"paths": np.array([b["path"] for b in br]), "p": _num([b["p"] for b in br], prec),
                "F": _num([b["F"] for b in br], prec)}
    if kind in ("run", "tree"):
        r = E.run_single_path(eng, st, s["circ"], case["shots"], case["chi"], s["k"],
                              uniforms=s["u"], device_sampling=case.get("sampling") == "device")
        st.release(r["ids"])
        out = {"outcomes": r["outcomes"], "F": _num(r["F"], prec), "p": _num(r["p"], prec)}
        if case.get("sampling") != "device":   # the device form keeps its p_0 to itself
            out["p0"] = _num(r["p0s"], prec)
        return _split(out)
    if kind == "state":
        for i, m in zip(s["ids"], s["mps"]):
            capi.dcs_import_mps(st.h, i, case["chi"], m, eng.stream())
        f = st.compress(s["ids"], s["chunks"], case["sweeps"])
        return {"f": f, "states": [np.concatenate([a.reshape(-1) for a in st.export(i)])
                                   for i in s["ids"]]}
    b, (qa, qb, qc), kids = case["branches"], s["q"], s["kids"]
    p_a = st.measure(s["kets"], [qa] * b)
    st.collapse(s["kets"], [qa] * b, s["out"][0], kids, E.EPS_BRANCH)
    st.set_chi(kids, s["caps"])
    f = st.compress(kids, s["chunks"], case["sweeps"])
    p_b = st.measure(kids, [qb] * b)
    st.collapse(kids, [qb] * b, s["out"][1], kids, E.EPS_BRANCH)
    p_c = st.measure(kids, [qc] * b)
    ov = capi.dcs_overlap(st.h, kids[0], kids[min(2, b - 1)], eng.stream())
    capi.dcs_branch_release(st.h, kids)
    out = _split({"f": _num(f, prec), "p_a": _num(p_a, prec), "p_b": _num(p_b, prec),
                  "p_c": _num(p_c, prec)})
    out["overlap"] = _num([ov.real, ov.imag], prec)
    return out


# ---------------------------------------------------------------------------
# The work that a pass cannot do without

def _step_work(n, ket, bra, w, sweeps, es, warm=False):
    """(bytes, flops) of one compression step: the ket read and the new state
    written once; the contractions and QRs of the sweeps."""
    cm = 8.0
    left = [cm * 2 * ket[j] * bra[j + 1] * w[j + 1] * (ket[j + 1] + 2 * w[j]) for j in range(n)]
    right = [cm * 2 * bra[j] * w[j] * ket[j + 1] * (ket[j] + 2 * w[j + 1]) for j in range(n)]
    env = [cm * bra[j] * w[j] * ket[j] * 2 * bra[j + 1] for j in range(n)]
    envr = [cm * bra[j + 1] * w[j + 1] * ket[j + 1] * 2 * bra[j] for j in range(n)]

    def qr(a, c):
        return cm * (2.0 * a * c * c - 2.0 * c ** 3 / 3.0)

    total = sum(left[j] + env[j] for j in range(1, n))
    for t in range(1, sweeps + 1):
        for j in range(n - 1):
            if t % 2:      # moving right: F, Q, next left environment
                total += right[j] + envr[j] * 2 + qr(2 * bra[j], min(bra[j + 1], 2 * bra[j]))
            else:
                total += left[j + 1] + env[j + 1] * 2 + qr(2 * bra[j + 2], min(bra[j + 1], 2 * bra[j + 2]))
    if warm:
        total += sum(qr(2 * bra[j + 1], min(bra[j], 2 * bra[j + 1])) for j in range(1, n))
    size = sum(2 * ket[j] * ket[j + 1] + 2 * bra[j] * bra[j + 1] for j in range(n)) * es
    return size, total


def _bonds(n, layers):
    """Operator bonds of a brickwork chunk of Haar gates."""
    w = [1] * (n + 1)
    for layer in range(layers):
        for q in range(layer % 2, n - 1, 2):
            w[q + 1] *= 4
    return w


def work(case):
    n, chi, es = case["n"], case["chi"], 16 if case["precision"] == "c128" else 8
    full = _dims(n, chi)
    if case["kind"] in ("round", "state"):
        caps = _caps(case)[0] if case["kind"] == "round" else [chi] * case["branches"]
        kinds = _caps(case)[1] if case["kind"] == "round" else [chi]
        size = flops = 0.0
        for i, cap in enumerate(caps):
            ket = _dims(n, kinds[-1 - (i // FANOUT) % len(kinds)])
            b, f = _step_work(n, ket, _dims(n, cap), _bonds(n, case["layers"]), case["sweeps"], es,
                              case.get("warm", -1.0) >= 0)
            size, flops = size + b, flops + f
        return {"bytes": size, "flops": flops}
    circ = _circuit(case, 0)
    shots = case.get("shots", 4)
    w, ket, size, flops, open_ = [1] * (n + 1), [1] * (n + 1), 0.0, 0.0, False
    for op in list(circ.ops) + [C.Measure(0, 0)]:
        if isinstance(op, C.Measure):
            if open_:
                if case["kind"] == "tree":   # a node is a site of a chain of its own dims
                    nodes = sum(_tree_nodes(n, chi))
                    b, f = nodes * 2 * es, 8.0 * 4 * nodes * chi * 4 * 4   # w = 4, 4 legs, 4 visits
                else:
                    b, f = _step_work(n, ket, full, w, 2, es)
                size, flops = size + b * shots, flops + f * shots
                ket = full
            w, open_ = [1] * (n + 1), False
            continue
        g = op.gate if isinstance(op, C.CGate) else op
        open_ = open_ or not isinstance(op, C.CGate)
        if len(g.qubits) == 2:
            r = 2 if case.get("circuit") == "ghz" or case["kind"] == "paths" else 4
            for b in range(min(g.qubits) + 1, max(g.qubits) + 1):
                w[b] = min(16, w[b] * r)
    return {"bytes": size, "flops": flops}


def _tree_nodes(n, chi):
    """Elements of each node tensor of the tree."""
    lv = TREES[n]
    out = []
    for l in range(len(lv) - 1):
        s, kids = n // lv[l], lv[l + 1] // lv[l]
        up = 1 if l == 0 else min(chi, 2 ** s, 2 ** (n - s))
        down = min(chi, 2 ** (n // lv[l + 1]), 2 ** (n - n // lv[l + 1])) if l + 2 < len(lv) else 2
        out += [up * down ** kids] * lv[l]
    return out


def _cost(case):
    """Rough seconds of a pass, for draw(): arithmetic, latency of the launches."""
    w = work(case)
    rate = {"c64": 4e13, "c128": 2e13, "bf16x3": 4e13}[case["precision"]]
    if case["kind"] == "tree":
        return 0.002 * case["depth"] + case["shots"] * sum(_tree_nodes(case["n"], case["chi"])) * 3e-8
    return w["flops"] / rate + case["n"] * 5e-5


def _slot_bytes(case):
    if case["kind"] == "tree" or case["kind"] == "paths":
        return 0
    d = _dims(case["n"], case["chi"])
    es = 16 if case["precision"] == "c128" else 8
    wmax = 16 if case.get("layers") == 3 or case.get("circuit") == "random" else 4
    one = sum(2 * x * y for x, y in zip(d, d[1:])) * es * 2 + sum(wmax * x * x for x in d) * es
    one += 2 * 2 * max(d) ** 2 * wmax * es + 6 * max(d) ** 2 * 16 * 2
    return one * (2 * case["branches"] + case["branches"] // FANOUT + 1 if "branches" in case
                  else case["shots"])


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain numpy

def _ref_split(m):
    u, s, vh = np.linalg.svd(m.reshape(2, 2, 2, 2).transpose(0, 2, 1, 3).reshape(4, 4))
    r = int(np.sum(s > 1e-14 * s[0]))
    return (u[:, :r] * s[:r]).reshape(2, 2, r), vh[:r].reshape(r, 2, 2)


def _ref_operator(n, ops):
    """One operator per site, W[wl, out, in, wr], of gates in time order."""
    total = [np.eye(2, dtype=complex).reshape(1, 2, 2, 1) for _ in range(n)]

    def then(j, g):   # g[x, s, u, y] after total[j]
        a = total[j]
        c = np.einsum("xsuy,autb->axstby", g, a)
        total[j] = c.reshape(a.shape[0] * g.shape[0], 2, 2, a.shape[3] * g.shape[3])

    for q, m in ops:
        m = np.asarray(m, dtype=complex)
        if len(q) == 1:
            then(q[0], m.reshape(1, 2, 2, 1))
            continue
        a, b = q
        if a > b:
            m, a, b = m.reshape(2, 2, 2, 2).transpose(1, 0, 3, 2).reshape(4, 4), b, a
        left, right = _ref_split(m)
        r = left.shape[2]
        then(a, left.reshape(1, 2, 2, r))
        for j in range(a + 1, b):
            then(j, np.einsum("xy,st->xsty", np.eye(r), np.eye(2)))
        then(b, right.reshape(r, 2, 2, 1))
    return total


def _ref_q(t):
    return np.linalg.qr(t)[0]


def _ref_right(r, bra, ket, w):
    x = np.tensordot(ket, r, axes=(2, 2))                       # x t c v
    x = np.tensordot(x, w, axes=([1, 3], [2, 3]))               # x c w s
    return np.tensordot(bra.conj(), x, axes=([1, 2], [3, 1])).transpose(0, 2, 1)


def _ref_mid(l, ket, w):
    x = np.tensordot(l, ket, axes=(2, 0))                       # a w t y
    return np.tensordot(x, w, axes=([1, 2], [0, 2]))            # a y s v


def _ref_guess(n, chi, gauss):
    return [g if j == 0 else _ref_q(g.reshape(g.shape[0], -1).conj().T).conj().T.reshape(g.shape)
            for j, g in enumerate(gauss)]


def _ref_warm(ket, guess, eta):
    m = []
    for k, g in zip(ket, guess):
        if k.shape[0] > g.shape[0] or k.shape[2] > g.shape[2]:
            return guess
        t = eta * g
        t[:k.shape[0], :, :k.shape[2]] += k
        m.append(t)
    m[0] = ket[0]
    for j in range(len(m) - 1, 0, -1):
        a = m[j].reshape(m[j].shape[0], -1)
        q = _ref_q(a.conj().T).conj().T
        if j > 1:
            m[j - 1] = np.tensordot(m[j - 1], a @ q.conj().T, axes=(2, 0))
        m[j] = q.reshape(m[j].shape)
    return m


def _ref_compress(ket, w, guess, sweeps):
    n = len(ket)
    bra = [b.copy() for b in guess]
    env = [None] * (n + 1)
    env[0] = env[n] = np.ones((1, 1, 1), dtype=complex)
    for j in range(n - 1, 0, -1):
        env[j] = _ref_right(env[j + 1], bra[j], ket[j], w[j])
    visits = []
    for t in range(1, sweeps + 1):
        visits += list(range(0 if t == 1 else 1, n)) if t % 2 else list(range(n - 2, -1, -1))
    for i, j in enumerate(visits):
        mid = _ref_mid(env[j], ket[j], w[j])                                  # a y s v
        t = np.tensordot(mid, env[j + 1], axes=([1, 3], [2, 1]))              # a s c
        f = float(np.vdot(t, t).real)
        t = t / math.sqrt(f)
        if i + 1 == len(visits):
            bra[j] = t
            return bra, f
        if visits[i + 1] > j:
            bra[j] = _ref_q(t.reshape(-1, t.shape[2])).reshape(t.shape)
            env[j + 1] = np.tensordot(bra[j].conj(), mid, axes=([0, 1], [0, 2])).transpose(0, 2, 1)
        else:
            bra[j] = _ref_q(t.reshape(t.shape[0], -1).conj().T).conj().T.reshape(t.shape)
            env[j] = _ref_right(env[j + 1], bra[j], ket[j], w[j])


def _ref_norms(mps, q):
    e = np.ones((1, 1), dtype=complex)
    for a in mps[:q]:
        e = np.tensordot(a.conj(), np.tensordot(e, a, axes=(1, 0)), axes=([0, 1], [0, 1]))
    g = np.ones((1, 1), dtype=complex)
    for a in reversed(mps[q + 1:]):
        g = np.tensordot(a.conj(), np.tensordot(a, g, axes=(2, 1)), axes=([1, 2], [1, 2]))
    z = np.tensordot(np.tensordot(e, mps[q], axes=(1, 0)), g, axes=(2, 1))
    return [float(np.vdot(mps[q][:, m], z[:, m]).real) for m in (0, 1)]


def _ref_collapse(mps, q, m, nm):
    out = list(mps)
    out[q] = out[q].copy()
    out[q][:, 1 - m] = 0.0
    out[q][:, m] /= math.sqrt(nm)
    return out


def _ref_shot(circ, chi, k, wmax, guess, choose):
    """One run; choose(path so far, p_0) gives an outcome.  Returns the
    outcomes, the p_0 of each, their probabilities and the fidelities."""
    n = circ.n_qubits
    psi = [np.array([[[1.0], [0.0]]], dtype=complex) for _ in range(n)]
    bits, chunk, path, p0s, ps, fids = {}, [], [], [], [], []
    w = np.ones(n + 1, dtype=int)

    def close():
        nonlocal psi, chunk
        if chunk:
            psi, f = _ref_compress(psi, _ref_operator(n, chunk), guess, 2)
            fids.append(f)
            chunk = []
            w[:] = 1

    for op in circ.ops:
        if isinstance(op, C.Measure):
            close()
            nm = _ref_norms(psi, op.qubit)
            p0 = nm[0] / sum(nm)
            m = choose(len(path), p0, tuple(path))
            psi = _ref_collapse(psi, op.qubit, m, nm[m])
            bits[op.bit] = m
            path.append(m)
            p0s.append(p0)
            ps.append(nm[m] / sum(nm))
            continue
        if isinstance(op, C.CGate):
            if sum(bits[b] for b in op.cond.bits) % 2 != op.cond.value:
                continue
            op = op.gate
        if len(op.qubits) == 2:
            lo, hi = min(op.qubits) + 1, max(op.qubits) + 1
            r = _ref_split(np.asarray(op.mat, dtype=complex))[0].shape[2]
            if chunk and w[lo:hi].max() * r > wmax:
                close()
            w[lo:hi] *= r
        chunk.append((op.qubits, op.mat))
        if len(chunk) == k:
            close()
    close()
    return path, p0s, ps, fids


def exact(case, seed):
    kind, n, chi, prec = case["kind"], case["n"], case["chi"], case["precision"]
    if kind == "tree":
        return None
    if kind in ("paths", "run"):
        circ = _circuit(case, seed)
        k, wmax = _chunk_limit(case, circ)
        guess = _ref_guess(n, chi, _gaussians(n, chi, seed))
        if kind == "paths":
            todo, done = [()], []
            while todo:
                want = todo.pop()
                path, p0s, ps, fids = _ref_shot(
                    circ, chi, k, wmax, guess,
                    lambda i, p0, _: want[i] if i < len(want) else int(p0 <= 1e-10))
                for i in range(len(want), len(path)):
                    if path[i] == 0 and 1.0 - p0s[i] > 1e-10:
                        todo.append(tuple(path[:i]) + (1,))
                done.append((tuple(path), float(np.prod(ps)), float(np.prod(fids))))
            done.sort()
            return {"paths": None, "p": np.array([d[1] for d in done]),
                    "F": np.array([d[2] for d in done])}
        nm, got = circ.n_measurements(), []
        for i in range(min(CHECKED, case["shots"])):
            u = shot_uniforms(int(seed), i, nm)
            got.append(_ref_shot(circ, chi, k, wmax, guess, lambda j, p0, _: int(u[j] >= p0)))
        out = {"outcomes": None, "F": np.array([np.prod(g[3]) for g in got]),
               "p": np.array([np.prod(g[2]) for g in got])}
        if case["sampling"] != "device":
            out["p0"] = np.array([g[1] for g in got]).reshape(len(got), nm)
        return {"checked": out, "others": {key: None for key in out}}
    ops = _layers(n, case["layers"], seed)
    w = _ref_operator(n, ops)
    if kind == "state":
        guess = _ref_guess(n, chi, _gaussians(n, chi, seed))
        f, states = [], []
        for i in range(case["branches"]):
            psi, fi = _ref_compress(_random_mps(n, chi, seed + 1000 * i, prec), w, guess,
                                    case["sweeps"])
            f.append(fi)
            states.append(np.concatenate([a.reshape(-1) for a in psi]))
        return {"f": np.array(f), "states": states}
    caps, kinds = _caps(case)
    plan, (qa, qb, qc), outcomes = _round_plan(case, seed)
    if chi > 300:
        return None
    flip = _ref_operator(n, ops + [((q,), C.X) for q in (0, n // 2)])
    rows, kids = [], []
    for i in range(min(CHECKED + 1, case["branches"])):
        base, q0, m0 = plan[i]
        cap = kinds[-1 - base % len(kinds)]
        psi = [a.astype(complex) for a in _random_mps(n, cap, seed + 1000 * base, prec)]
        psi = _ref_collapse(psi, q0, m0, _ref_norms(psi, q0)[m0])
        na = _ref_norms(psi, qa)
        m = int(outcomes[0][i])
        psi = _ref_collapse(psi, qa, m, na[m])
        guess = _ref_guess(n, caps[i], _gaussians(n, caps[i], seed))
        if case["warm"] >= 0:
            guess = _ref_warm(psi, guess, case["warm"])
        psi, f = _ref_compress(psi, flip if m else w, guess, case["sweeps"])
        nb = _ref_norms(psi, qb)
        m = int(outcomes[1][i])
        psi = _ref_collapse(psi, qb, m, nb[m])
        nc = _ref_norms(psi, qc)
        rows.append([f, na[0] / sum(na), nb[0] / sum(nb), nc[0] / sum(nc)])
        kids.append(psi)
    e = np.ones((1, 1), dtype=complex)
    for a, b in zip(kids[0], kids[min(2, case["branches"] - 1)]):
        e = np.tensordot(a.conj(), np.tensordot(e, b, axes=(1, 0)), axes=([0, 1], [0, 1]))
    rows = np.array(rows[:CHECKED])
    out = {key: rows[:, j] for j, key in enumerate(("f", "p_a", "p_b", "p_c"))}
    return {"checked": out, "others": {key: None for key in out},
            "overlap": np.array([e[0, 0].real, e[0, 0].imag])}
