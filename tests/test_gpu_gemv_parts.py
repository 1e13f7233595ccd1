"""Last-batch joins of few elements, whose tiles of x are split over several workgroups:
4 elements of one tile (a sixteenth each), 300 (a quarter), 1100 (whole tiles), for one
and two rows per element, against the FP64 oracle's amplitudes."""
import numpy as np
import pytest

import workloads as W
from oracle import sampling
from tests.gpu_helpers import oracle_states, prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("elems", [4, 300, 1100])
@pytest.mark.parametrize("n, depth, bs", [(18, 4, [4, 14]), (18, 5, [3, 15]), (19, 6, [5, 14]), (20, 7, [6, 14])])
def test_gemv_parts(n, depth, bs, elems):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    circ = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.05)
    plan = P.Plan(circ, bs, method="network")
    kr, _, _, _ = plan.sample_trajectories(3, 4 if elems == 4 else 600)
    E = min(len(kr), elems)
    kr = kr[:E]
    traj = np.sort(np.arange(elems) % E).astype(np.int32)
    pre = [int(x) for x in np.random.default_rng(elems).integers(0, 2 ** bs[0], size=elems)]
    print(f"n={n} depth={depth} elems={elems} rows log2 {plan.batch_info(1)['join_rows_log2']}", flush=True)
    args = (1, to_dev(torch, dev, kr), to_dev(torch, dev, traj), to_dev(torch, dev, prefix_words(pre, plan.n_words)))
    amp = plan.contract_batch(*args, P.OUT_AMPLITUDE)[0]
    pop = plan.contract_batch(*args, P.OUT_POPULATION)[0]
    torch.cuda.synchronize()
    amp, pop = amp.cpu().numpy(), pop.cpu().numpy()
    for e in (0, elems // 2, elems - 1):
        psi = oracle_states(circ, kr[traj[e]:traj[e] + 1])[0]
        ref = sampling.amplitudes_from_state(psi, n, bs[0], bs[1], pre[e])
        # some 10^2 gates and 2^6 terms a sum in FP32: 1e-5 of the element's norm, as everywhere
        # for amplitudes
        nr = np.linalg.norm(ref)
        assert np.linalg.norm(amp[e] - ref) <= 1e-5 * nr, (e, pre[e])
        assert np.abs(pop[e] - np.abs(ref) ** 2).max() <= 1e-5 * nr ** 2, (e, pre[e])
