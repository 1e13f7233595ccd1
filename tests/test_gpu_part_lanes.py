"""Sweeps with one job a lane against the same sweeps in shared workgroups.

A sample of many shots has batches with enough elements for the lane form, a sample of
the first few of them (the draws of a shot do not depend on how many there are) has not;
both add the same products in the same order, so the shots they share are equal, and
they are checked against the FP64 oracle sampler.  Ranks 4 and 5 (chains of depth 5 and
6), with and without a last step that raises the rank, element counts that are no
multiple of a wavefront, and elements of one, few and many trajectories in a wavefront."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_helpers import oracle_shots_sv, oracle_states, shots_to_ints, to_dev, torch_dev

pytestmark = pytest.mark.gpu
MANY = 32768            # elements of a batch from which sweeps take the lane form


@pytest.mark.parametrize("n, bs, n_traj, many, few", [
    (16, [4, 4, 4, 4], 40, 2111, 50), (16, [5, 5, 6], 700, 100, 3), (16, [3, 5, 3, 5], 700, 100, 3),
    (16, [4, 4, 3, 5], 40, 2111, 50), (22, [8, 8, 6], 1, 120000, 400)])
@pytest.mark.parametrize("depth", [5, 6])
def test_lane_sweeps(depth, n, bs, n_traj, many, few):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    circ = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.05)
    plan = P.Plan(circ, bs, method="network")
    kr, _, _, _ = plan.sample_trajectories(4, n_traj)
    E = len(kr)
    print(f"depth={depth} n={n} bs={bs} E={E}", flush=True)

    def sample(m):
        out = plan.sample_shots(to_dev(torch, dev, kr), to_dev(torch, dev, np.full(E, m, dtype=np.int64)), 77)
        torch.cuda.synchronize()
        return out["elements_per_batch"], np.array(shots_to_ints(out["shots"].cpu().numpy())).reshape(E, m)

    el_many, a = sample(many)
    el_few, b = sample(few)
    assert max(int(x) for x in el_many) >= MANY > max(int(x) for x in el_few), (el_many, el_few)
    assert np.array_equal(a[:, :few], b)
    k = min(E, 3)
    want, _ = oracle_shots_sv(circ, oracle_states(circ, kr[:k]), bs, few, 77)
    mism = sum(int(x != y) for i in range(k) for x, y in zip(a[i, :few], want[i]))
    # a draw differs where it falls within the populations' error (1e-5 of the total) of a
    # boundary of the cumulative sums: under 2^8 boundaries x 1e-5 a batch
    assert mism <= 1 + 0.01 * k * few, mism
