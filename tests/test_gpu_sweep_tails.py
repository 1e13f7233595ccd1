"""Per-trajectory parts of rank 11 and 12 for many and for few trajectories: sweeps of rank 11
take another workgroup from 513 jobs on, and sweeps that come to rank 12 only at their end are
cut there from 1024 jobs on (one step and several after the cut).  Small calls, which the
oracle tests pin, and large ones are the same bit for bit: products are summed in one order."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bs,j,depth,rank", [(20, [5] * 4, 1, 4, 11), (24, [4] * 6, 2, 5, 12), (20, [5] * 4, 1, 5, 12)])
@pytest.mark.parametrize("E", [513, 1024, 1500])
def test_many_jobs_equal_few(n, bs, j, depth, rank, E):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    c = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.2).round_to_complex64()
    plan = P.Plan(c, bs, method="network", hypersamples=4)
    assert plan.batch_info(j)["right_peak_rank"] == rank
    kr, _, _, _ = plan.sample_trajectories(3, E)
    assert len(np.unique(kr[:, plan.right_sites(j)], axis=0)) == E      # jobs of the per-trajectory part
    pre = [int(x) for x in np.random.default_rng(1).integers(0, 2 ** sum(bs[:j]), size=E)]

    def call(lo, hi):
        return plan.contract_batch(j, to_dev(torch, dev, kr[lo:hi]), to_dev(torch, dev, np.arange(hi - lo, dtype=np.int32)),
                                   to_dev(torch, dev, prefix_words(pre[lo:hi], plan.n_words)), P.OUT_POPULATION)[0]

    print(f"rank={rank} jobs={E}", flush=True)
    whole = call(0, E)
    for lo in range(0, E, 256):
        assert torch.equal(whole[lo:lo + 256], call(lo, min(E, lo + 256)))
    if n == 20:
        for e in (0, E - 1):
            psi = oracle_states(c, kr[e:e + 1])[0]
            ref = sampling.marginal_from_state(psi, n, sum(bs[:j]), bs[j], pre[e])
            assert np.abs(whole[e].cpu().numpy() - ref).max() <= 1e-5 * ref.sum() + 1e-12
