"""LDS sweeps whose workgroups hold 64 elements of up to 64 different trajectories.

A step's gates are staged once per trajectory of the workgroup's elements: from 33
trajectories on they need more than the 512 entries that were once set aside.  One
element a trajectory (33, 64, 65, 200 of them), and a mix, on sweeps of rank 3 to 5."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(1,) * 33, (1,) * 64, (1,) * 65, (1,) * 200, (20,) + (1,) * 50 + (30, 1, 1)])
@pytest.mark.parametrize("depth", [4, 5, 6])
def test_many_trajectories_a_workgroup(depth, counts):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    n, bs, j = 13, [4, 4, 5], 1
    circ = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.2)
    plan = P.Plan(circ, bs, method="network")
    kr, _, _, _ = plan.sample_trajectories(3, len(counts))
    assert len(kr) == len(counts)
    traj = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    pre = [int(x) for x in np.random.default_rng(1).integers(0, 2 ** bs[0], size=len(traj))]
    print(f"depth={depth} trajectories={len(counts)}", flush=True)
    out, _ = plan.contract_batch(j, to_dev(torch, dev, kr), to_dev(torch, dev, traj),
                                 to_dev(torch, dev, prefix_words(pre, plan.n_words)), P.OUT_POPULATION)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    for e in range(0, len(traj), 3):
        psi = oracle_states(circ, kr[traj[e]:traj[e] + 1])[0]
        ref = sampling.marginal_from_state(psi, n, bs[0], bs[1], pre[e])
        # relative to the element's weight, at the amplitudes' tolerance, as everywhere for the
        # network method's populations
        assert np.abs(out[e] - ref).max() <= 1e-5 * ref.sum() + 1e-12, (e, traj[e])
