"""Gate groups of the statevector windows: runs of gates applied in registers.

Tiles of 2^10, 2^11 and 2^12 amplitudes hold 4, 8 and 16 of them a thread, so a group
takes two, three or four positions.  Random gates on random pairs in both orders end
groups at every bound; dense, diagonal and permuting gates, with Pauli noise and with
damping (a row of zeros), take each form of the product."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu

_I, _X = np.eye(2), np.array([[0.0, 1.0], [1.0, 0.0]])
_CZ = np.diag([1.0, 1.0, 1.0, -1.0])
_CNOT = np.array([[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, 0, 1], [0, 0, 1, 0]], dtype=float)
_SWAP = np.array([[1, 0, 0, 0], [0, 0, 1, 0], [0, 1, 0, 0], [0, 0, 0, 1]], dtype=float)


def _circuit(n, rng, local):
    """Gates on pairs of nearby qubits (local) or of any, in either order."""
    c = W.Circuit(n_qubits=n)
    noise = [c.add_channel(ch) for ch in (W.depolarizing(0.3), W.amplitude_damping(0.3))]
    two = [lambda: W.haar_su4(rng), lambda: _CZ, lambda: _CNOT, lambda: _SWAP, lambda: np.kron(_X, _X),
           lambda: np.diag(np.exp(2j * np.pi * rng.random(4)))]
    one = [lambda: W.ry(rng.random()) @ W.rz(rng.random()), lambda: _X, lambda: W.rz(rng.random())]
    for _ in range(9 * n):
        a = int(rng.integers(0, n))
        b = (a + int(rng.integers(1, 3))) % n if local else int(rng.integers(0, n))
        if a == b or rng.random() < 0.3:
            g = c.add_gate((a,), np.asarray(one[int(rng.integers(0, len(one)))](), dtype=np.complex128))
        else:
            g = c.add_gate((a, b) if rng.random() < 0.5 else (b, a),
                           np.asarray(two[int(rng.integers(0, len(two)))](), dtype=np.complex128))
        if rng.random() < 0.5:
            c.add_site(g, (a,), noise[int(rng.integers(0, 2))])
    return c.round_to_complex64()


@pytest.mark.parametrize("local", [True, False])
@pytest.mark.parametrize("n, bs", [(10, [4, 6]), (11, [5, 6]), (12, [6, 6]), (14, [6, 8])])
def test_groups(n, bs, local):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    circ = _circuit(n, np.random.default_rng(100 * n + local), local)
    plan = P.Plan(circ, bs, method="statevector")
    kr, _, _, _ = plan.sample_trajectories(9, 24)
    psis = oracle_states(circ, kr)
    kd = to_dev(torch, dev, kr)
    starts = sampling.batch_starts(bs)
    rng = np.random.default_rng(n)
    for j, (a, b) in enumerate(zip(starts, bs)):
        traj = np.arange(len(kr), dtype=np.int32)
        pre = [int(rng.integers(0, 2 ** a)) if a else 0 for _ in traj]
        print(f"n={n} local={local} batch {j}", flush=True)
        out, _ = plan.contract_batch(j, kd, to_dev(torch, dev, traj), to_dev(torch, dev, prefix_words(pre, plan.n_words)),
                                     P.OUT_POPULATION)
        torch.cuda.synchronize()
        out = out.cpu().numpy()
        for t, p in zip(traj, pre):
            ref = sampling.marginal_from_state(psis[t], n, a, b, p)
            # a few products per gate and amplitude in FP32, some 10^2 gates: under 1e-6 of the
            # state's norm on a joint marginal, as everywhere for the statevector method
            Z = np.vdot(psis[t], psis[t]).real
            assert np.abs(out[t] - ref).max() <= 1e-6 * Z, (n, j, t)
