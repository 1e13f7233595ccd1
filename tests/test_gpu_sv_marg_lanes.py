"""Marginals of later batches of many elements (a lane per element) against the FP64 oracle:
2^b from 256 to 4096, prefixes from one cache line (start 4) up, element counts that leave
the last wavefront partly empty, the last batch (no later qubits) and one before it."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elems", [1023, 1024, 1089])
@pytest.mark.parametrize("bs, j", [([4, 8, 3], 1), ([5, 8], 1), ([4, 9, 2], 1), ([4, 10, 1], 1), ([4, 11], 1),
                                   ([4, 12], 1), ([3, 9], 1)])
def test_marginals_of_many_elements(bs, j, elems):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    n = sum(bs)
    circ = W.random_brickwork(n, 4, np.random.default_rng(n), 0.05)
    plan = P.Plan(circ, bs, method="statevector")
    kr, _, _, _ = plan.sample_trajectories(3, 40)
    kr = kr[:5]
    traj = (np.arange(elems) * len(kr) // elems).astype(np.int32)
    start = sum(bs[:j])
    pre = np.random.default_rng(n).integers(0, 2 ** start, size=elems)
    pre = [int(x) for x in pre[np.lexsort((pre, traj))]]
    print(f"batches={bs} elems={elems}", flush=True)
    pop = plan.contract_batch(j, to_dev(torch, dev, kr), to_dev(torch, dev, traj),
                              to_dev(torch, dev, prefix_words(pre, plan.n_words)), P.OUT_POPULATION)[0]
    torch.cuda.synchronize()
    pop = pop.cpu().numpy()
    psi = oracle_states(circ, kr)
    for e in (0, 63, 64, elems // 2, elems - 2, elems - 1):
        ref = sampling.marginal_from_state(psi[traj[e]], n, start, bs[j], pre[e])
        # some 10^2 gates in FP32: 1e-5 of the element's probability
        assert np.abs(pop[e] - ref).max() <= 1e-5 * ref.sum(), (e, pre[e])
