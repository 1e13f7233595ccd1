"""A ragged set cut into thousands of waves of one trajectory: the waves' tables stay within
the space set aside for them (16 MB), and the shots are those of one wave."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_helpers import to_dev, torch_dev

pytestmark = pytest.mark.gpu


def test_thousands_of_one_trajectory_waves():
    import paper_2604_08467_amd as P
    from paper_2604_08467_amd.ragged import RaggedSet
    torch, dev = torch_dev()
    E = 2600
    c = W.random_brickwork(16, 32, np.random.default_rng(1), 0.01)
    plan = P.Plan(c, [8, 8], method="statevector")
    assert plan.sv_windows_for(12) >= 8
    kr, _, _, _ = plan.sample_trajectories(2, 16)
    kr = np.tile(kr, (E // len(kr) + 1, 1))[:E].copy()
    job = {"plan": plan, "kraus": to_dev(torch, dev, kr), "mult": to_dev(torch, dev, np.ones(E, dtype=np.int64)),
           "shots_per_traj": np.full(E, 2, dtype=np.int64), "seed": 3}
    rs = RaggedSet()
    whole, _ = rs.sample_shots([job], stamps=False)
    assert rs.info()["n_waves"] == 1
    # one state of 2^16 amplitudes and its arrays to a wave: 16 MB of tables and 1 MB beside them
    small = torch.empty((17 << 20) + (1 << 17), dtype=torch.uint8, device=dev)
    waves, _ = rs.sample_shots([job], workspace=small, stamps=False)
    assert rs.info()["n_waves"] == E
    for k in ("shots", "norms", "weights"):
        assert torch.equal(whole[0][k], waves[0][k]), k
