"""Runs of gates on network tensors of rank 13 and more in the window kernel: tensors per
trajectory and per element (several elements of one trajectory next to each other, then a
new trajectory), runs of two gates and of several groups, ranks 14 to 20, against the FP64
oracle's amplitudes."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elems", [1, 37])
@pytest.mark.parametrize("n, depth, bs", [(18, 8, [4, 14]), (20, 10, [6, 14]), (20, 7, [3, 17]), (18, 6, [9, 9]),
                                          (19, 7, [4, 4, 11])])
def test_part_windows(n, depth, bs, elems):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    circ = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.05)
    plan = P.Plan(circ, bs, method="network")
    kr, _, _, _ = plan.sample_trajectories(3, 40)
    E = min(len(kr), (elems + 4) // 5)                      # five elements a trajectory
    kr = kr[:E]
    traj = np.minimum(np.arange(elems) // 5, E - 1).astype(np.int32)
    j, start = len(bs) - 1, sum(bs[:-1])
    pre = [int(x) for x in np.random.default_rng(elems).integers(0, 2 ** start, size=elems)]
    print(f"n={n} depth={depth} batches={bs} elems={elems}", flush=True)
    amp = plan.contract_batch(j, to_dev(torch, dev, kr), to_dev(torch, dev, traj),
                              to_dev(torch, dev, prefix_words(pre, plan.n_words)), P.OUT_AMPLITUDE)[0]
    torch.cuda.synchronize()
    amp = amp.cpu().numpy()
    for e in sorted({0, elems // 2, elems - 1}):
        psi = oracle_states(circ, kr[traj[e]:traj[e] + 1])[0]
        ref = sampling.amplitudes_from_state(psi, n, start, bs[-1], pre[e])
        # some 10^2 gates in FP32: 1e-5 of the element's norm, as everywhere for amplitudes
        assert np.linalg.norm(amp[e] - ref) <= 1e-5 * np.linalg.norm(ref), (e, pre[e])


@pytest.mark.parametrize("light_cone", [False, True])
@pytest.mark.parametrize("n, depth, bs, j", [(16, 6, [8, 8], 0), (18, 6, [6, 6, 6], 1), (18, 7, [5, 6, 7], 1),
                                             (20, 5, [10, 10], 0), (20, 6, [10, 10], 0)])
def test_picked_gates(n, depth, bs, j, light_cone):
    """Marginals of the batches before the last, whose runs hold gates picked by hyper legs
    inside and outside the tile (tensors of rank 13 to 17)."""
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    circ = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.05)
    plan = P.Plan(circ, bs, method="network", light_cone=light_cone)
    kr, _, _, _ = plan.sample_trajectories(3, 40)
    kr = kr[:3]
    traj = np.arange(7, dtype=np.int32) * len(kr) // 7
    start = sum(bs[:j])
    pre = [int(x) for x in np.random.default_rng(n).integers(0, 2 ** start, size=len(traj))]
    print(f"n={n} depth={depth} batches={bs} j={j} light_cone={light_cone}", flush=True)
    pop = plan.contract_batch(j, to_dev(torch, dev, kr), to_dev(torch, dev, traj),
                              to_dev(torch, dev, prefix_words(pre, plan.n_words)), P.OUT_POPULATION)[0]
    torch.cuda.synchronize()
    pop = pop.cpu().numpy()
    for e in range(len(traj)):
        psi = oracle_states(circ, kr[traj[e]:traj[e] + 1])[0]
        ref = sampling.marginal_from_state(psi, n, start, bs[j], pre[e])
        # as for amplitudes: 1e-5 of the element's probability
        assert np.abs(pop[e] - ref).max() <= 1e-5 * ref.sum(), (e, pre[e])
