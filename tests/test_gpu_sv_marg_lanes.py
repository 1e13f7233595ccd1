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


@pytest.mark.parametrize("shots", [3, 40])
def test_one_batch_in_chunks(shots):
    """One batch of every qubit: a workspace for a few of the states gives the call's shots
    in several chunks of trajectories, bit for bit those of one chunk."""
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    circ = W.random_brickwork(9, 4, np.random.default_rng(9), 0.05)
    plan = P.Plan(circ, [9], method="statevector")
    kr, mult, _, _ = plan.sample_trajectories(3, 400)
    E = len(kr)
    args = (to_dev(torch, dev, kr), torch.full((E,), shots, dtype=torch.int64, device=dev), 5)
    size = plan.sample_workspace_size(E, E * shots)
    print(f"{E} trajectories x {shots} shots, workspace {size}", flush=True)
    want = plan.sample_shots(*args, mult_dev=to_dev(torch, dev, mult))["shots"].cpu()
    ws = torch.empty(size - (size - (24 << 20)) * 3 // 4, dtype=torch.uint8, device=dev)
    got = plan.sample_shots(*args, mult_dev=to_dev(torch, dev, mult), workspace=ws)["shots"].cpu()
    assert torch.equal(want, got)
