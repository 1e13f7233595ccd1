"""Doubled joins of 16 and 32 crossing values at the edges of their row tiles.

A wavefront takes row tiles of 16, a workgroup 64 or 128 rows of a trajectory: calls
whose trajectories have rows just below, at and above these, and none, for 16 and 32
kept values of x (whose output loops differ) and one or two rows per element."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(1, 0, 15), (16, 17, 3), (63, 0, 64), (65, 8, 0, 32), (127, 128, 1), (129, 33, 0)])
@pytest.mark.parametrize("j", [1, 2])
@pytest.mark.parametrize("depth", [5, 6])
def test_qform_rows(depth, j, counts):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    n, bs = 18, [5, 5, 5, 3]
    circ = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.05)
    plan = P.Plan(circ, bs, method="network")
    info = plan.batch_info(j)
    assert info["doubled"] and info["crossing"] == depth - 1
    kr, _, _, _ = plan.sample_trajectories(3, len(counts))
    assert len(kr) >= len(counts)
    kr = kr[:len(counts)]
    psis = oracle_states(circ, kr)
    rng = np.random.default_rng(sum(counts))
    traj = np.repeat(np.arange(len(counts)), counts)
    a = sampling.batch_starts(bs)[j]
    pre = [int(x) for x in rng.integers(0, 2 ** a, size=len(traj))]
    print(f"depth={depth} batch {j} counts={counts} rows log2 {info['join_rows_log2']}", flush=True)
    out, tot = plan.contract_batch(j, to_dev(torch, dev, kr), to_dev(torch, dev, traj.astype(np.int32)),
                                   to_dev(torch, dev, prefix_words(pre, plan.n_words)), P.OUT_POPULATION)
    torch.cuda.synchronize()
    out, tot = out.cpu().numpy(), tot.cpu().numpy()
    for e, (t, p) in enumerate(zip(traj, pre)):
        ref = sampling.marginal_from_state(psis[t], n, a, bs[j], p)
        # relative to the element's weight, at the amplitudes' tolerance, as everywhere for the
        # network method's populations
        assert np.abs(out[e] - ref).max() <= 1e-5 * ref.sum() + 1e-12, (e, t, p)
        assert abs(tot[e] - ref.sum()) <= 1e-5 * ref.sum() + 1e-12, (e, t, p)
