"""LDS sweeps of many steps: a launch holds 16 bytes of LDS a step beside its tensors, so that
a run of more steps than 160 KB take is cut into several launches.

Deep brickworks as one last batch (the right part is every gate): 12 qubits (one element a
workgroup, 5,520 steps a launch) and 11, 9, 5 qubits (1, 4, 64 elements a workgroup), around the cuts
and beyond them, some with a run that ends before the rank passes 12.

Tolerance: a gate's entries and its four-term FP32 sums each round at 2^-24 relative; with
random signs the state's error after N gates is about 6 sqrt(N) 2^-24 of its norm."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _circuit(n, steps, seed):
    """A brickwork of exactly `steps` two-qubit gates; a little noise early on."""
    rng = np.random.default_rng(seed)
    c = W.Circuit(n)
    ch = c.add_channel(W.depolarizing(0.1))
    k = layer = 0
    while k < steps:
        for q in range(layer % 2, n - 1, 2):
            if k < steps:
                g = c.add_gate((q, q + 1), W.haar_su4(rng))
                if k < 40:
                    c.add_site(g, (q,), ch)
                k += 1
        layer += 1
    return c.round_to_complex64()


@pytest.mark.parametrize("n,steps,elems", [(12, 5520, 2), (12, 5521, 2), (12, 11100, 3), (11, 9000, 3),
                                           (9, 8000, 9), (5, 15000, 70)])
def test_sweep_of_many_steps(n, steps, elems):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    c = _circuit(n, steps, 10 * n + steps)
    plan = P.Plan(c, [n], method="network", hypersamples=1)
    bi = plan.batch_info(0)
    assert bi["n_right_steps"] == steps and bi["right_peak_rank"] == n and bi["n_right_launches"] == 0
    kr, _, _, _ = plan.sample_trajectories(5, elems)
    E = len(kr)
    print(f"n={n} steps={steps} trajectories={E}", flush=True)
    out, _ = plan.contract_batch(0, to_dev(torch, dev, kr), to_dev(torch, dev, np.arange(E, dtype=np.int32)),
                                 to_dev(torch, dev, prefix_words([0] * E, plan.n_words)), P.OUT_AMPLITUDE)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    for e in range(0, E, 1 if E < 10 else 23):
        ref = oracle_states(c, kr[e:e + 1])[0]
        assert np.linalg.norm(out[e] - ref) <= 6 * np.sqrt(steps) * 2.0 ** -24 * np.linalg.norm(ref), e


def test_long_run_inside_a_larger_part():
    """6,000 steps on 12 qubits, then two qubits more: the run of rank 12 is cut and goes on at
    rank 14."""
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    c = _circuit(12, 6000, 3)
    big = W.Circuit(14)
    for q, m in zip(c.gate_qubits, c.gate_mats):
        big.add_gate(q, m)
    rng = np.random.default_rng(4)
    for q in (11, 12, 10, 11, 12, 0, 5):
        big.add_gate((q, q + 1), W.haar_su4(rng))
    big = big.round_to_complex64()
    plan = P.Plan(big, [14], method="network", hypersamples=1)
    bi = plan.batch_info(0)
    assert bi["n_right_steps"] == 6007 and bi["right_peak_rank"] == 14
    kr = np.zeros((2, max(1, plan.n_sites)), dtype=np.uint8)
    out, _ = plan.contract_batch(0, to_dev(torch, dev, kr), to_dev(torch, dev, np.arange(2, dtype=np.int32)),
                                 to_dev(torch, dev, prefix_words([0, 0], plan.n_words)), P.OUT_AMPLITUDE)
    torch.cuda.synchronize()
    ref = oracle_states(big, kr[:1])[0]
    for row in out.cpu().numpy():
        assert np.linalg.norm(row - ref) <= 6 * np.sqrt(6007) * 2.0 ** -24
