"""Statevector windows that write the states from |0...0> themselves.

Every workspace is filled with NaN before the call, so that an amplitude that no
window wrote shows.  Circuits of one window, of one qubit more than a window, of
several windows that reach the last qubits late, and circuits that leave qubits
without a gate (whose states are initialised in full)."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _poisoned(torch, dev, nbytes):
    return torch.full(((nbytes + 3) // 4,), float("nan"), dtype=torch.float32, device=dev).view(torch.uint8)


def _idle(n, used, rng):
    """Gates on the qubits `used` only."""
    c = W.Circuit(n_qubits=n)
    ch = c.add_channel(W.depolarizing(0.1))
    for _ in range(6):
        for a, b in zip(used[:-1], used[1:]):
            g = c.add_gate((a, b), W.haar_su4(rng))
            c.add_site(g, (a,), ch)
    return c


CASES = {
    "one_window10": lambda r: (W.random_brickwork(10, 4, r, 0.05), [10]),
    "one_window12": lambda r: (W.random_brickwork(12, 4, r, 0.05), [6, 6]),
    "window_and_one": lambda r: (W.random_brickwork(13, 4, r, 0.05), [5, 8]),
    "grid16": lambda r: (W.sqrt_grid(4, 4, 6, r, p=0.05, gamma=0.1), [8, 8]),
    "late_qubits18": lambda r: (W.random_brickwork(18, 9, r, 0.02), [8, 10]),
    "idle_top": lambda r: (_idle(14, list(range(13)), r), [6, 8]),
    "idle_low": lambda r: (_idle(14, [9, 10, 11, 12, 13], r), [6, 8]),
    "idle_middle": lambda r: (_idle(15, [0, 1, 2, 12, 13, 14], r), [7, 8]),
}


# precision: 0 FP32, 2 fp16 pairs.  factor on the tolerance: a hi + lo pair of fp16 holds 22 bits, two fewer than FP32
@pytest.mark.parametrize("precision, factor", [(0, 1), (2, 4)])
@pytest.mark.parametrize("name", list(CASES))
def test_states_from_zero(name, precision, factor):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    circ, bs = CASES[name](np.random.default_rng(len(name)))
    circ = circ.round_to_complex64()
    plan = P.Plan(circ, bs, method="statevector", precision=precision)
    kr, _, _, _ = plan.sample_trajectories(5, 5)
    E, n, starts = len(kr), circ.n_qubits, sampling.batch_starts(bs)
    psis = oracle_states(circ, kr)
    kd = to_dev(torch, dev, kr)
    rng = np.random.default_rng(1)
    for j, (a, b) in enumerate(zip(starts, bs)):
        traj = np.sort(rng.integers(0, E, size=9)).astype(np.int32)
        # a prefix that idle qubits do not rule out, and random ones
        pre = [0 if i == 0 or a == 0 else int(rng.integers(0, 2 ** a)) for i in range(len(traj))]
        ws = _poisoned(torch, dev, plan.contract_workspace_size(j, E, len(traj)))
        print(f"{name} {precision} batch {j}", flush=True)
        out, tot = plan.contract_batch(j, kd, to_dev(torch, dev, traj), to_dev(torch, dev, prefix_words(pre, plan.n_words)),
                                       P.OUT_POPULATION, workspace=ws)
        torch.cuda.synchronize()
        out, tot = out.cpu().numpy(), tot.cpu().numpy()
        for e, (t, p) in enumerate(zip(traj, pre)):
            ref = sampling.marginal_from_state(psis[t], n, a, b, p)
            # some 10^2 gates in FP32 on a state of norm Z: 1e-6 Z on a marginal, 1e-5 Z on their
            # sum, as everywhere for the statevector method
            Z = np.vdot(psis[t], psis[t]).real
            assert np.abs(out[e] - ref).max() <= factor * 1e-6 * Z, (name, j, e)
            assert abs(tot[e] - ref.sum()) <= factor * 1e-5 * Z, (name, j, e)


def test_ragged_states_from_zero():
    import paper_2604_08467_amd as P
    from paper_2604_08467_amd.ragged import RaggedSet
    torch, dev = torch_dev()
    jobs = []
    for k, name in enumerate(CASES):
        circ, bs = CASES[name](np.random.default_rng(len(name)))
        circ = circ.round_to_complex64()
        plan = P.Plan(circ, bs, method="statevector")
        kr, mult, _, _ = plan.sample_trajectories(50 + k, 6)
        jobs.append({"plan": plan, "kraus": to_dev(torch, dev, kr), "mult": to_dev(torch, dev, mult),
                     "shots_per_traj": np.full(len(kr), 40, dtype=np.int64), "seed": 70 + k,
                     "psis": oracle_states(circ, kr)})
    rs = RaggedSet()
    ws = _poisoned(torch, dev, rs.workspace_size(jobs))
    print("ragged", flush=True)
    outs, _ = rs.sample_shots(jobs, workspace=ws)
    for jb, o in zip(jobs, outs):
        Z = np.array([np.vdot(p, p).real for p in jb["psis"]])
        np.testing.assert_allclose(o["norms"].cpu().numpy(), Z, rtol=1e-5)
        # every shot is an outcome its trajectory can give (one of norm 0 gives none)
        shots = o["shots"].cpu().numpy()
        shots = shots.reshape(len(shots), -1)[:, 0].astype(np.uint64)
        for i, p in enumerate(jb["psis"]):
            assert Z[i] == 0.0 or np.all(np.abs(p[shots[40 * i:40 * i + 40]]) ** 2 > 1e-9 * Z[i])


@pytest.mark.parametrize("damped", [False, True])
@pytest.mark.parametrize("n, idle", [(11, 0), (12, 0), (13, 0), (15, 0), (14, 2)])
def test_gradients_from_zero(n, idle, damped):
    """Value and gradient windows on a poisoned workspace; with idle qubits at the top the
    states are written whole.  Tolerance as for the cluster gradients: under 60 cluster
    products of 32 FP32 terms each way, 1e-5 between the worst and the random case."""
    import ctypes as C

    import paper_2604_08467_amd as P
    from oracle import gradients as gr
    from paper_2604_08467_amd import _lib
    torch, dev = torch_dev()
    rng = np.random.default_rng(n)
    m, layers = n - idle, 3
    theta = rng.uniform(0, 2 * np.pi, size=2 * m * layers)
    inner = W.hea(m, layers, theta, [W.depolarizing(0.05)] + ([W.amplitude_damping(0.1)] if damped else []))
    gp, ga = W.rotation_spec(inner)
    circ = W.Circuit(**{**inner.__dict__, "n_qubits": n})
    terms = W.zz_chain_terms(m)
    plan = P.Plan(circ, [10, n - 10], method="statevector")
    kr, mult, _, _ = plan.sample_trajectories(3, 3)
    w = mult / mult.sum()
    spec = P.GradSpec(len(theta), gp, ga, terms)
    size = C.c_size_t()
    _lib.check(plan._lib.ptsbe_expect_workspace_size(plan._h, C.byref(spec.struct), len(kr), C.byref(size)))
    print(f"gradient n={n} idle={idle} damped={damped}", flush=True)
    out = plan.expect_grad(spec, to_dev(torch, dev, kr), to_dev(torch, dev, w), to_dev(torch, dev, theta),
                           workspace=_poisoned(torch, dev, size.value))
    want = gr.adjoint_gradient(circ, kr, w, theta, gp, ga, terms)
    assert abs(float(out["value"].item()) - gr.value(circ, kr, w, theta, gp, ga, terms)) <= 1e-5 * len(terms)
    assert np.linalg.norm(out["grad"].cpu().numpy() - want) <= 1e-5 * np.linalg.norm(want)
    only = plan.expect_grad(spec, to_dev(torch, dev, kr), to_dev(torch, dev, w), to_dev(torch, dev, theta),
                            want_grad=False, workspace=_poisoned(torch, dev, size.value))
    assert abs(float(only["value"].item()) - gr.value(circ, kr, w, theta, gp, ga, terms)) <= 1e-5 * len(terms)
