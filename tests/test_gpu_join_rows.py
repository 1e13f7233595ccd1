"""Doubled joins of 2^6 .. 2^8 crossing values (chains of depth 7 .. 9), row by row.

The join takes 2, 4, 8 or 16 rows of a trajectory at a time by the most rows that one
trajectory has: calls with every trajectory's count below, at and above each of these,
trajectories without elements between them, and one or two rows per element."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu

# n, depth, batches, crossing and rows per element (log2) of batch 1
CASES = [(14, 7, [4, 5, 5], 6, 0), (15, 7, [5, 5, 5], 6, 1), (14, 8, [4, 5, 5], 7, 1), (14, 9, [4, 5, 5], 8, 0)]


@pytest.mark.parametrize("counts", [(1, 0, 2), (3, 1, 0, 4), (7, 0, 8), (9, 1, 16), (17, 33, 0, 5)])
@pytest.mark.parametrize("case", CASES)
def test_join_rows(case, counts):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    n, depth, bs, crossing, rows = case
    circ = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.05)
    plan = P.Plan(circ, bs, method="network")
    info = plan.batch_info(1)
    assert info["doubled"] and info["crossing"] == crossing and info["join_rows_log2"] == rows
    kr, _, _, _ = plan.sample_trajectories(3, len(counts))
    assert len(kr) >= len(counts)
    kr = kr[:len(counts)]
    psis = oracle_states(circ, kr)
    rng = np.random.default_rng(sum(counts))
    traj = np.repeat(np.arange(len(counts)), counts)
    pre = [int(x) for x in rng.integers(0, 2 ** bs[0], size=len(traj))]
    print(f"n={n} depth={depth} counts={counts}", flush=True)
    out, tot = plan.contract_batch(1, to_dev(torch, dev, kr), to_dev(torch, dev, traj.astype(np.int32)),
                                   to_dev(torch, dev, prefix_words(pre, plan.n_words)), P.OUT_POPULATION)
    torch.cuda.synchronize()
    out, tot = out.cpu().numpy(), tot.cpu().numpy()
    for e, (t, p) in enumerate(zip(traj, pre)):
        ref = sampling.marginal_from_state(psis[t], n, bs[0], bs[1], p)
        # 2^8 terms a sum and some 10^2 gates in FP32: under 100 roundings of 6e-8 of the
        # element's weight each way, as everywhere for the network method's populations
        assert np.abs(out[e] - ref).max() <= 1e-5 * ref.sum(), (e, t, p)
        assert abs(tot[e] - ref.sum()) <= 1e-5 * ref.sum(), (e, t, p)
