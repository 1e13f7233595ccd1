"""Performance cases of the framework's public entry points: sampling, contraction and gradients.

A case is a dict of plain values; `kind` picks the entry point:

  shots       Plan.sample_shots, proportional non-degenerate batched sampling of one circuit
  ragged      RaggedSet.sample_shots, several small circuits in one set, replayed from its graphs
  amplitudes  Plan.contract_batch, the last batch's amplitudes for given prefixes
  populations Plan.contract_batch, one batch's marginals and their totals for given prefixes
  gradient    ExpectZZ forward and backward, the value and all angle gradients of an ansatz

Circuits are the repository's families: chains and grids of Haar two-qubit gates, the
square-root grid with CZ layers and the RY-RZ-CNOT ansatz, with depolarising noise and,
where `gamma` is set, amplitude damping.  Error sets are drawn from the proposals, each
distinct set once with its multiplicity, as trajectory pre-sampling does.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2604_08467_amd as P
from paper_2604_08467_amd.ragged import RaggedSet

I2 = np.eye(2, dtype=np.complex128)
X = np.array([[0, 1], [1, 0]], dtype=np.complex128)
Y = np.array([[0, -1j], [1j, 0]], dtype=np.complex128)
Z = np.diag([1.0, -1.0]).astype(np.complex128)
CZ = np.diag([1.0, 1.0, 1.0, -1.0]).astype(np.complex128)
CNOT = np.array([[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, 0, 1], [0, 0, 1, 0]], dtype=np.complex128)
PRECISIONS = {"c64": 0, "bf16": 1, "f16": 2}


def listed():
    return [
        # a small noisy chain, sampled whole in one batch: launches and latency
        {"name": "chain10_shots", "kind": "shots", "circuit": "chain", "n": 10, "depth": 8, "p": 0.01, "gamma": 0.0,
         "traj": 64, "shots": 100, "batch": 10, "light_cone": False, "precision": "c64"},
        # the 50-qubit chain with the batch size its tuner picks: the headline sampling run
        {"name": "chain50_shots_b5", "kind": "shots", "circuit": "chain", "n": 50, "depth": 6, "p": 0.005,
         "gamma": 0.0, "traj": 4096, "shots": 1000, "batch": 5, "light_cone": True, "precision": "c64"},
        # the same chain with wide batches and the plan's default options: large joins, sweeps through memory
        {"name": "chain50_shots_b10", "kind": "shots", "circuit": "chain", "n": 50, "depth": 6, "p": 0.005,
         "gamma": 0.0, "traj": 384, "shots": 1000, "batch": 10, "light_cone": False, "precision": "c64"},
        # a 2D grid with damping: one statevector per trajectory, weights that differ
        {"name": "grid25_shots", "kind": "shots", "circuit": "sqrt_grid", "n": 25, "depth": 8, "p": 0.01,
         "gamma": 0.02, "traj": 48, "shots": 256, "batch": 10, "light_cone": False, "precision": "c64"},
        # a smaller grid in split precision
        {"name": "grid20_shots_bf16", "kind": "shots", "circuit": "sqrt_grid", "n": 20, "depth": 8, "p": 0.01,
         "gamma": 0.02, "traj": 256, "shots": 256, "batch": 10, "light_cone": False, "precision": "bf16"},
        # a mix of small circuits of several sizes and layouts sampled together, as a job server does
        {"name": "ragged_mix", "kind": "ragged", "circuits": 12, "n_min": 12, "n_max": 20, "depth": 7, "p": 0.005,
         "traj": 128, "shots": 100, "batch": 10},
        # last-batch amplitudes of a long deep chain for a few prefixes
        {"name": "chain100_amplitudes", "kind": "amplitudes", "n": 100, "depth": 12, "p": 0.005, "traj": 4,
         "elems": 4, "batch": 10, "last": 16},
        # marginals of one batch of an odd-sized chain for many prefixes
        {"name": "chain23_populations", "kind": "populations", "n": 23, "depth": 7, "p": 0.01, "traj": 48,
         "elems": 1500, "batch": 6, "which": 1},
        # the 20-qubit ansatz, one optimisation step's value and gradient
        {"name": "ansatz20_gradient", "kind": "gradient", "n": 20, "layers": 10, "p": 0.01, "gamma": 0.0, "traj": 64},
        # a small ansatz, where a step is launches and latency
        {"name": "ansatz8_gradient", "kind": "gradient", "n": 8, "layers": 3, "p": 0.02, "gamma": 0.0, "traj": 16},
        # a middle-sized ansatz with damping (non-unitary operators take another backward form)
        {"name": "ansatz14_damped_gradient", "kind": "gradient", "n": 14, "layers": 5, "p": 0.01, "gamma": 0.02,
         "traj": 64},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["shots_sv", "shots_net", "grid", "ragged", "amplitudes", "populations", "gradient", "gradient"])
    if kind == "shots_sv":        # chains up to 22 qubits, one or several batches
        n = rng.randint(8, 22)
        return {"kind": "shots", "circuit": "chain", "n": n, "depth": rng.randint(4, 10), "p": 0.01, "gamma": 0.0,
                "traj": _log_int(rng, 16, 512), "shots": _log_int(rng, 50, 1000), "batch": rng.randint(4, 11),
                "light_cone": False, "precision": "c64"}
    if kind == "shots_net":       # long chains, narrow and wide batches
        wide = rng.random() < 0.4
        return {"kind": "shots", "circuit": "chain", "n": rng.randint(32, 60), "depth": rng.randint(5, 6), "p": 0.005,
                "gamma": 0.0, "traj": _log_int(rng, 32, 256) if wide else _log_int(rng, 64, 3000),
                "shots": _log_int(rng, 100, 1000), "batch": rng.randint(8, 10) if wide else rng.randint(4, 6),
                "light_cone": rng.random() < 0.5, "precision": "c64"}
    if kind == "grid":            # 2D circuits by the statevector method
        n = rng.choice([12, 15, 16, 18, 20, 21, 24])
        return {"kind": "shots", "circuit": rng.choice(["sqrt_grid", "grid"]), "n": n, "depth": rng.randint(4, 8),
                "p": 0.01, "gamma": rng.choice([0.0, 0.02]), "traj": min(_log_int(rng, 16, 256), 48 << max(0, 25 - n)),
                "shots": _log_int(rng, 64, 512), "batch": rng.randint(5, 10), "light_cone": False,
                "precision": rng.choice(["c64", "bf16", "f16"])}
    if kind == "ragged":
        lo = rng.randint(11, 14)
        return {"kind": "ragged", "circuits": rng.randint(4, 14), "n_min": lo, "n_max": lo + rng.randint(2, 6),
                "depth": rng.randint(4, 8), "p": 0.005, "traj": _log_int(rng, 32, 160), "shots": 100,
                "batch": rng.randint(6, 10)}
    if kind == "amplitudes":
        e = rng.randint(1, 4)
        return {"kind": "amplitudes", "n": rng.randint(40, 100), "depth": rng.randint(8, 12), "p": 0.005, "traj": e,
                "elems": e, "batch": 10, "last": rng.randint(12, 16)}
    if kind == "populations":
        return {"kind": "populations", "n": rng.randint(14, 23), "depth": rng.randint(4, 8), "p": 0.01,
                "traj": _log_int(rng, 8, 48), "elems": _log_int(rng, 64, 1500), "batch": rng.randint(4, 7),
                "which": rng.randint(0, 1)}
    n = rng.randint(7, 19)        # ansatz gradients
    return {"kind": "gradient", "n": n, "layers": rng.randint(2, 8), "p": 0.01, "gamma": rng.choice([0.0, 0.0, 0.02])
            if n <= 14 else 0.0, "traj": _log_int(rng, 8, 64)}


# ------------------------------------------------------------------ circuits
def _depolarizing(p):
    return SimpleNamespace(kraus=np.stack([np.sqrt(1 - p) * I2, np.sqrt(p / 3) * X, np.sqrt(p / 3) * Y,
                                           np.sqrt(p / 3) * Z]), probs=np.array([1 - p, p / 3, p / 3, p / 3]))


def _damping(g):
    return SimpleNamespace(kraus=np.array([[[1, 0], [0, np.sqrt(1 - g)]], [[0, np.sqrt(g)], [0, 0]]],
                                          dtype=np.complex128), probs=None)


def _rot(pauli, angle):
    return np.cos(angle / 2) * I2 - 1j * np.sin(angle / 2) * pauli


def _haar4(rng):
    q, r = np.linalg.qr(rng.standard_normal((4, 4)) + 1j * rng.standard_normal((4, 4)))
    d = np.diag(r)
    q = q * (d / np.abs(d))[None, :]
    return q / np.linalg.det(q) ** 0.25


def _new_circuit(n, p, gamma):
    c = SimpleNamespace(n_qubits=n, gate_qubits=[], gate_mats=[], channels=[_depolarizing(p)], site_gate=[],
                        site_qubits=[], site_channel=[], gate_param=[])
    if gamma:
        c.channels.append(_damping(gamma))
    return c


def _add(c, qubits, mat, param=None):
    g = len(c.gate_qubits)
    c.gate_qubits.append(tuple(qubits))
    c.gate_mats.append(mat)
    c.gate_param.append(param)
    for q in qubits:
        for ch in range(len(c.channels)):
            c.site_gate.append(g)
            c.site_qubits.append((q,))
            c.site_channel.append(ch)


def _chain_layers(n, depth):
    return [[(q, q + 1) for q in range(d % 2, n - 1, 2)] for d in range(depth)]


def _grid_layers(n, depth):
    rows = int(math.isqrt(n))
    cols = -(-n // rows)
    layers = []
    for d in range(depth):
        kind, par = (("h", 0), ("v", 0), ("h", 1), ("v", 1))[d % 4]
        pairs = []
        for q in range(n):
            r, k = divmod(q, cols)
            b = q + 1 if kind == "h" else q + cols
            if (k if kind == "h" else r) % 2 == par and b < n and (kind == "v" or k + 1 < cols):
                pairs.append((q, b))
        layers.append(pairs)
    return layers


def _haar_circuit(n, layers, p, gamma, rng):
    c = _new_circuit(n, p, gamma)
    for layer in layers:
        for pair in layer:
            _add(c, pair, _haar4(rng))
    return c


def _sqrt_grid(n, cycles, p, gamma, rng):
    c = _new_circuit(n, p, gamma)
    roots = [_rot(a, np.pi / 2) for a in (X, Y, (X + Y) / np.sqrt(2.0))]
    for layer in _grid_layers(n, cycles):
        for q in range(n):
            _add(c, (q,), roots[int(rng.integers(0, 3))])
        for pair in layer:
            _add(c, pair, CZ)
    return c


def _ansatz(n, layers, angles, p, gamma):
    c = _new_circuit(n, p, gamma)
    k = 0
    for _ in range(layers):
        for axis, pauli in ((1, Y), (2, Z)):
            for q in range(n):
                _add(c, (q,), _rot(pauli, float(angles[k])), (k, axis))
                k += 1
        for q in range(n - 1):
            _add(c, (q, q + 1), CNOT)
    return c


def _proposal(ch):
    return ch.probs if ch.probs is not None else np.real(np.einsum("kij,kij->k", ch.kraus.conj(), ch.kraus)) / 2


def _error_sets(c, traj, rng):
    """Distinct error sets in first-draw order and how often each was drawn."""
    cum = [np.cumsum(_proposal(ch)) for ch in c.channels]
    site_ch = np.array(c.site_channel)
    rows = np.zeros((0, len(site_ch)), dtype=np.uint8)
    for _ in range(64):
        u = rng.random((2 * traj, len(site_ch)))
        k = np.zeros(u.shape, dtype=np.uint8)
        for ch, cc in enumerate(cum):
            at = site_ch == ch
            k[:, at] = np.minimum(np.searchsorted(cc, u[:, at], side="right"), len(cc) - 1)
        rows = np.concatenate([rows, k])
        distinct, first, count = np.unique(rows, axis=0, return_index=True, return_counts=True)
        if len(distinct) >= traj:
            break
    order = np.argsort(first)[:traj]
    return np.ascontiguousarray(distinct[order]), count[order].astype(np.int64)


def _batches(n, b):
    return [b] * (n // b) + ([n % b] if n % b else [])


def _inputs(case, seed):
    """The circuit, error sets and other host inputs of a case (lists of them for a ragged set)."""
    rng = np.random.default_rng([seed, 7])
    kind = case["kind"]
    n = case.get("n", 0)
    if kind == "shots":
        if case["circuit"] == "sqrt_grid":
            c = _sqrt_grid(n, case["depth"], case["p"], case["gamma"], rng)
        else:
            layers = (_chain_layers if case["circuit"] == "chain" else _grid_layers)(n, case["depth"])
            c = _haar_circuit(n, layers, case["p"], case["gamma"], rng)
        return SimpleNamespace(c=c, batches=_batches(n, case["batch"]), sets=_error_sets(c, case["traj"], rng))
    if kind == "ragged":
        jobs = []
        for k in range(case["circuits"]):
            m = case["n_min"] + int(rng.integers(0, case["n_max"] - case["n_min"] + 1)) if k > 1 else (
                case["n_min"] if k == 0 else case["n_max"])
            layers = (_chain_layers if k % 2 else _grid_layers)(m, max(3, case["depth"] - k % 3))
            c = _haar_circuit(m, layers, case["p"], 0.0, rng)
            jobs.append(SimpleNamespace(c=c, batches=_batches(m, case["batch"]),
                                        sets=_error_sets(c, max(8, case["traj"] >> k % 3), rng)))
        return jobs
    if kind == "gradient":
        angles = rng.uniform(0, 2 * np.pi, 2 * n * case["layers"]).astype(np.float32)
        c = _ansatz(n, case["layers"], angles.astype(np.float64), case["p"], case["gamma"])
        sets = _error_sets(c, case["traj"], rng)
        return SimpleNamespace(c=c, batches=_batches(n, 10), sets=sets, angles=angles,
                               terms=[((q, q + 1), 1.0) for q in range(n - 1)])
    c = _haar_circuit(n, _chain_layers(n, case["depth"]), case["p"], 0.0, rng)
    if kind == "populations":
        batches = _batches(n, case["batch"])
        j = case["which"]
    else:
        batches = _batches(n - case["last"], case["batch"]) + [case["last"]]
        j = len(batches) - 1
    d = SimpleNamespace(c=c, batches=batches, j=j, sets=_error_sets(c, case["traj"], rng))
    start = sum(batches[:j])      # (trajectory, prefix) elements, grouped by trajectory
    d.elem_traj = np.sort(np.arange(case["elems"]) % len(d.sets[0])).astype(np.int32)
    d.bits = rng.integers(0, 2, (case["elems"], start)).astype(np.uint64)
    d.words = np.zeros((case["elems"], (n + 63) // 64), dtype=np.uint64)
    for q in range(start):
        d.words[:, q // 64] |= d.bits[:, q] << np.uint64(q % 64)
    return d


# ------------------------------------------------------------------ the passes
def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _workspace(n_bytes):
    return torch.empty(int(n_bytes), dtype=torch.uint8, device="cuda:0")


def prepare(case, seed):
    kind = case["kind"]
    d = _inputs(case, seed)
    if kind == "ragged":
        jobs, outputs = [], []
        for k, jb in enumerate(d):
            kraus, mult = jb.sets
            per = np.full(len(kraus), case["shots"], dtype=np.int64)
            jobs.append({"plan": P.Plan(jb.c, jb.batches, method="statevector"), "kraus": _dev(kraus),
                         "mult": _dev(mult), "shots_per_traj": per, "seed": seed * 131 + k})
            outputs.append({"shots": torch.empty((int(per.sum()), 1), dtype=torch.int64, device="cuda:0"),
                            "weights": torch.empty(len(kraus), dtype=torch.float64, device="cuda:0"),
                            "norms": torch.empty(len(kraus), dtype=torch.float64, device="cuda:0")})
        rs = RaggedSet()
        return {"kind": kind, "set": rs, "jobs": jobs, "outputs": outputs,
                "stream": torch.cuda.Stream(),    # graphs are captured on a stream of their own
                "workspace": _workspace(rs.workspace_size(jobs))}
    kraus, mult = d.sets
    E = len(kraus)
    s = {"kind": kind, "kraus": _dev(kraus), "mult": _dev(mult), "seed": seed + 17}
    if kind == "shots":
        s["plan"] = P.Plan(d.c, d.batches, light_cone=case["light_cone"], precision=PRECISIONS[case["precision"]])
        s["shots"] = torch.full((E,), case["shots"], dtype=torch.int64, device="cuda:0")
        s["workspace"] = _workspace(s["plan"].sample_workspace_size(E, E * case["shots"]))
    elif kind in ("amplitudes", "populations"):
        s["plan"] = P.Plan(d.c, d.batches, method="network" if kind == "amplitudes" else "auto")
        s["j"] = d.j
        s["elem_traj"] = _dev(d.elem_traj)
        s["elem_prefix"] = _dev(d.words.view(np.int64))
        s["workspace"] = _workspace(s["plan"].contract_workspace_size(d.j, E, len(d.elem_traj)))
    else:
        gp = np.array([-1 if g is None else g[0] for g in d.c.gate_param], dtype=np.int32)
        ga = np.array([0 if g is None else g[1] for g in d.c.gate_param], dtype=np.int32)
        s["plan"] = P.Plan(d.c, d.batches, method="statevector")
        s["spec"] = P.GradSpec(len(d.angles), gp, ga, d.terms)
        s["weights"] = _dev(mult / mult.sum())
        s["angles"] = _dev(d.angles).requires_grad_(True)
    return s


def run(state):
    s = state
    kind = s["kind"]
    if kind == "shots":
        o = s["plan"].sample_shots(s["kraus"], s["shots"], s["seed"], mult_dev=s["mult"], workspace=s["workspace"])
        return {k: o[k] for k in ("shots", "shot_traj", "weights", "norms", "elements_per_batch")}
    if kind == "ragged":
        out, _ = s["set"].sample_shots(s["jobs"], graph=True, workspace=s["workspace"], outputs=s["outputs"],
                                       stamps=False, stream=s["stream"].cuda_stream)
        return [{k: o[k] for k in ("shots", "weights", "norms")} for o in out]
    if kind == "amplitudes":
        return s["plan"].contract_batch(s["j"], s["kraus"], s["elem_traj"], s["elem_prefix"], P.OUT_AMPLITUDE,
                                        workspace=s["workspace"])[0]
    if kind == "populations":
        return s["plan"].contract_batch(s["j"], s["kraus"], s["elem_traj"], s["elem_prefix"],
                                        workspace=s["workspace"])
    s["angles"].grad = None
    value = P.ExpectZZ.apply(s["angles"], s["plan"], s["spec"], s["kraus"], s["weights"])
    value.backward()
    return {"value": value, "grad": s["angles"].grad}


# ------------------------------------------------------------------ work
def _gates(case, n):
    """(one-qubit, two-qubit) gate counts of the case's circuit, by its layout."""
    if case["kind"] == "gradient":
        return 2 * n * case["layers"], (n - 1) * case["layers"]
    pairs = sum(len(x) for x in (_chain_layers if case.get("circuit", "chain") == "chain" else _grid_layers)(
        n, case["depth"]))
    return (n * case["depth"] if case.get("circuit") == "sqrt_grid" else 0), pairs


def _state_work(n, g1, g2):
    """A state evolved through its gates: products, and one write and one read of a state too large for a chip's LDS."""
    flops = (14.0 * g1 + 30.0 * g2) * 2.0 ** n
    return flops, (16.0 * 2.0 ** n if n > 12 else 0.0)


def _distinct(bins_log2, m):
    """Expected distinct values among m uniform draws."""
    return m if bins_log2 > 40 else 2.0 ** bins_log2 * -math.expm1(-m / 2.0 ** bins_log2)


def work(case):
    kind = case["kind"]
    E = case.get("traj", 0)
    n = case.get("n", 0)
    if kind == "ragged":
        flops = moved = 0.0
        for k in range(case["circuits"]):
            m = (case["n_min"] + case["n_max"]) // 2
            e = max(8, case["traj"] >> k % 3)
            f, b = _state_work(m, *_gates({"kind": "shots", "circuit": "chain" if k % 2 else "grid",
                                           "depth": max(3, case["depth"] - k % 3)}, m))
            flops += e * f
            moved += e * (b + 8.0 * case["shots"] + 16.0)
        return {"bytes": moved, "flops": flops}
    g1, g2 = _gates(case, n)
    sites = (g1 + 2 * g2) * (2 if case.get("gamma") else 1)
    moved = float(E * sites)
    if kind == "gradient":
        f, b = _state_work(n, g1, g2)
        return {"bytes": E * 2 * b + moved + 16.0 * n * case["layers"], "flops": E * 3 * f}
    if kind == "populations":
        f, b = _state_work(n, g1, g2)              # by states, or by one bilinear form per element, the smaller
        form = case["elems"] * 2.0 * 4 ** (case["depth"] - 1) * 2 ** case["batch"]
        flops = min(E * f, form)
        return {"bytes": (E * b if flops < form else 0.0) + moved + case["elems"] * 4.0 * 2 ** case["batch"],
                "flops": flops}
    words = (n + 63) // 64
    if kind == "shots":
        moved += E * (case["shots"] * (8.0 * words + 4) + 32)
        if case["circuit"] != "chain" or n <= 22:
            f, b = _state_work(n, g1, g2)
            return {"bytes": E * b + moved, "flops": E * f}
        flops, start = 0.0, 0
        for b in _batches(n, case["batch"]):      # one bilinear form of 2 K^2 flops per element and value
            last = start + b == n
            per = 8.0 * 2 ** (case["depth"] - 1) if last else 2.0 * 4 ** (case["depth"] - 1)
            flops += E * _distinct(start, case["shots"]) * per * 2 ** b
            start += b
        return {"bytes": moved, "flops": flops}
    k = 2.0 ** (case["depth"] - 1)                # wires crossing into the last batch
    flops = (case["elems"] * 8.0 + E * 64.0) * k * 2 ** case["last"]
    return {"bytes": moved + case["elems"] * 8.0 * 2 ** case["last"], "flops": flops}


# ------------------------------------------------------------------ 64-bit values
def _merged(c, kraus, device):
    """Every gate with its trajectory's operators applied after it: a list of (E, d, d) complex128."""
    ops = [np.asarray(ch.kraus) / np.sqrt(np.where(_proposal(ch) > 0, _proposal(ch), 1.0))[:, None, None]
           for ch in c.channels]
    out = [np.broadcast_to(m, (len(kraus),) + m.shape).copy() for m in c.gate_mats]
    for s, g in enumerate(c.site_gate):
        k = ops[c.site_channel[s]][kraus[:, s]]
        if len(c.gate_qubits[g]) == 2:            # the first listed qubit is the matrix index's high bit
            k = (np.einsum("eij,kl->eikjl", k, I2) if c.site_qubits[s][0] == c.gate_qubits[g][0]
                 else np.einsum("ij,ekl->eikjl", I2, k)).reshape(-1, 4, 4)
        out[g] = k @ out[g]
    return [torch.from_numpy(m).to(device) for m in out]


def _legs(psi, n, qubits):
    """psi (E, 2^n, qubit q = bit q) with the gate's qubits as axes, the first listed one first."""
    E = psi.shape[0]
    if len(qubits) == 1:
        q = qubits[0]
        return [psi.view(E, -1, 2, 2 ** q)[:, :, x] for x in range(2)]
    hi, lo = max(qubits), min(qubits)
    v = psi.view(E, -1, 2, 2 ** (hi - lo - 1), 2, 2 ** lo)
    if qubits[0] == hi:
        return [v[:, :, a, :, b] for a in range(2) for b in range(2)]
    return [v[:, :, b, :, a] for a in range(2) for b in range(2)]


def _apply(psi, n, qubits, mats):
    parts = [x.clone() for x in _legs(psi, n, qubits)]
    shape = (-1,) + (1,) * (parts[0].dim() - 1)
    for r, dst in enumerate(_legs(psi, n, qubits)):
        acc = mats[:, r, 0].reshape(shape) * parts[0]
        for k in range(1, len(parts)):
            acc += mats[:, r, k].reshape(shape) * parts[k]
        dst.copy_(acc)


def _states(c, mats, lo, hi, device):
    n = c.n_qubits
    psi = torch.zeros((hi - lo, 2 ** n), dtype=torch.complex128, device=device)
    psi[:, 0] = 1.0
    for g, qubits in enumerate(c.gate_qubits):
        _apply(psi, n, qubits, mats[g][lo:hi])
    return psi


def _exact_norms(c, kraus, device):
    if all(ch.probs is not None for ch in c.channels):
        return np.ones(len(kraus))                # unitary gates and operators
    mats = _merged(c, kraus, device)
    step = max(1, 2 ** 27 >> c.n_qubits)
    return np.concatenate([_states(c, mats, i, min(i + step, len(kraus)), device).abs().square().sum(1).cpu().numpy()
                           for i in range(0, len(kraus), step)])


def _exact_sampling(d, device):
    norms = _exact_norms(d.c, d.sets[0], device)
    w = d.sets[1] * norms
    return {"weights": w / w.sum(), "norms": norms}


def _exact_amplitudes(d, device):
    """Column by column contraction of the projected ket network, one element at a time."""
    c = d.c
    mats = _merged(c, d.sets[0], device)
    n, start = c.n_qubits, sum(d.batches[:d.j])
    order = sorted(range(len(c.gate_qubits)), key=lambda g: (min(c.gate_qubits[g]), g))
    seen, wires = [0] * n, {}
    for g, qubits in enumerate(c.gate_qubits):
        for q in qubits:
            wires[g, q] = ((q, seen[q]), (q, seen[q] + 1))
            seen[q] += 1
    out = []
    for e, t in enumerate(d.elem_traj):
        cur, legs = torch.ones((), dtype=torch.complex128, device=device), []
        for g in order:
            qubits = c.gate_qubits[g]
            m = mats[g][t].reshape((2,) * (2 * len(qubits)))
            names = [wires[g, q][1] for q in qubits] + [wires[g, q][0] for q in qubits]
            for q in qubits:                      # inputs in |0>, outputs of earlier qubits in the prefix's bit
                for name, value in ((wires[g, q][0], 0), (wires[g, q][1], int(d.bits[e][q]) if q < start else None)):
                    if (name[1] == 0 and name == wires[g, q][0]) or (name[1] == seen[q] and value is not None):
                        k = names.index(name)
                        m = m.select(k, value)
                        names.pop(k)
            shared = [x for x in names if x in legs]
            cur = torch.tensordot(cur, m, dims=([legs.index(x) for x in shared], [names.index(x) for x in shared]))
            legs = [x for x in legs if x not in shared] + [x for x in names if x not in shared]
        at = [legs.index((q, seen[q])) for q in range(n - 1, start - 1, -1)]
        out.append(cur.permute(at).reshape(-1))
    return torch.stack(out)


def _exact_populations(d, device):
    mats = _merged(d.c, d.sets[0], device)
    n, start, b = d.c.n_qubits, sum(d.batches[:d.j]), d.batches[d.j]
    prefix = torch.from_numpy(d.words[:, 0].astype(np.int64)).to(device)
    out = torch.zeros((len(d.elem_traj), 2 ** b), dtype=torch.float64, device=device)
    for t in range(len(d.sets[0])):
        p = _states(d.c, mats, t, t + 1, device)[0].abs().square().view(-1, 2 ** b, 2 ** start).sum(0)
        at = torch.from_numpy(np.nonzero(d.elem_traj == t)[0]).to(device)
        out[at] = p[:, prefix[at]].t()
    return out, out.sum(1)


def _exact_gradient(d, device):
    c, (kraus, mult) = d.c, d.sets
    n = c.n_qubits
    mats = _merged(c, kraus, device)
    w = torch.from_numpy(mult / mult.sum()).to(device)
    idx = torch.arange(2 ** n, device=device)
    obs = sum(cf * (1.0 - 2.0 * ((idx >> a ^ idx >> b) & 1).double()) for (a, b), cf in d.terms)
    unitary = len(c.channels) == 1
    step = max(1, 2 ** 26 >> n) if unitary else max(1, 2 ** 28 >> n + len(mats).bit_length())
    value, grad = 0.0, np.zeros(len(d.angles))
    for lo in range(0, len(kraus), step):
        hi = min(lo + step, len(kraus))
        psi = torch.zeros((hi - lo, 2 ** n), dtype=torch.complex128, device=device)
        psi[:, 0] = 1.0
        kept = []
        for g, qubits in enumerate(c.gate_qubits):
            if not unitary:
                kept.append(psi.clone())
            _apply(psi, n, qubits, mats[g][lo:hi])
        value += float((w[lo:hi, None] * psi.abs().square() * obs).sum())
        lam = w[lo:hi, None] * obs * psi
        for g in range(len(mats) - 1, -1, -1):
            back = mats[g][lo:hi].conj().transpose(1, 2)
            _apply(lam, n, c.gate_qubits[g], back)
            if unitary:
                _apply(psi, n, c.gate_qubits[g], back)
            else:
                psi = kept.pop()
            if c.gate_param[g] is not None:       # d/dtheta exp(-i theta P / 2)
                k, axis = c.gate_param[g]
                a0, a1 = _legs(psi, n, c.gate_qubits[g])
                l0, l1 = _legs(lam, n, c.gate_qubits[g])
                if axis == 2:
                    v = (l0.conj() * a0).sum() - (l1.conj() * a1).sum()
                else:
                    v = -1j * (l0.conj() * a1).sum() + 1j * (l1.conj() * a0).sum()
                grad[k] += float(v.imag)
    return {"value": torch.tensor(value, dtype=torch.float64), "grad": grad}


def exact(case, seed):
    device = "cuda:0" if torch.cuda.is_available() else "cpu"
    kind = case["kind"]
    if kind == "amplitudes" and case["elems"] << case["last"] + case["depth"] > 1 << 31:
        return None               # over 20 seconds
    d = _inputs(case, seed)
    if kind == "ragged":
        return [_exact_sampling(jb, device) for jb in d]
    if kind == "shots":
        return _exact_sampling(d, device)
    if kind == "amplitudes":
        return _exact_amplitudes(d, device)
    if kind == "populations":
        return _exact_populations(d, device)
    return _exact_gradient(d, device)
