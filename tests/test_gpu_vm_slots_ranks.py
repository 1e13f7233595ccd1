"""LDS sweeps of rank 6 to 9 whose workgroups (32 to 4 elements) hold as many different
trajectories as elements: a step's gates then fill, or take an even part of, the 512 entries
that are staged at a time; with few trajectories many steps are staged together."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bs,depth,rank", [(13, [4, 4, 5], 6, 6), (14, [5, 5, 4], 7, 7), (13, [4, 4, 5], 8, 8),
                                             (14, [5, 5, 4], 9, 9)])
@pytest.mark.parametrize("counts", [(1,) * 33, (1, 31, 1, 1, 30), (3,) * 22])
def test_different_trajectories_a_workgroup(n, bs, depth, rank, counts):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    circ = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.2)
    plan = P.Plan(circ, bs, method="network", hypersamples=4)
    assert plan.batch_info(1)["left_peak_rank"] == rank
    kr, _, _, _ = plan.sample_trajectories(3, len(counts))
    assert len(kr) == len(counts)
    traj = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    pre = [int(x) for x in np.random.default_rng(1).integers(0, 2 ** bs[0], size=len(traj))]
    print(f"rank={rank} trajectories={len(counts)}", flush=True)
    out, _ = plan.contract_batch(1, to_dev(torch, dev, kr), to_dev(torch, dev, traj),
                                 to_dev(torch, dev, prefix_words(pre, plan.n_words)), P.OUT_POPULATION)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    for e in range(0, len(traj), 4):
        psi = oracle_states(circ, kr[traj[e]:traj[e] + 1])[0]
        ref = sampling.marginal_from_state(psi, n, bs[0], bs[1], pre[e])
        # relative to the element's weight, at the amplitudes' tolerance, as everywhere for the
        # network method's populations
        assert np.abs(out[e] - ref).max() <= 1e-5 * ref.sum() + 1e-12, (e, traj[e])
