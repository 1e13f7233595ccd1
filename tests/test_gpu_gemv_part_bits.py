"""Last-batch joins read as matrix-vector products: the same populations and amplitudes bit for
bit whether a workgroup takes a whole tile of 4096 values (1024 elements and more), a quarter
of one or a sixteenth (fewer than 256), with one row an element and with two."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_helpers import prefix_words, to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bs,depth", [(14, [2, 12], 4), (16, [4, 12], 5), (12, [12], 3), (13, [13], 3)])
def test_parts_of_a_tile_round_alike(n, bs, depth):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    E, j = 1100, len(bs) - 1
    c = W.random_brickwork(n, depth, np.random.default_rng(depth), 0.3)
    plan = P.Plan(c, bs, method="network", hypersamples=4)
    kr, _, _, _ = plan.sample_trajectories(2, E)
    assert len(kr) == E
    pre = [int(x) for x in np.random.default_rng(1).integers(0, 2 ** sum(bs[:j]), size=E)]
    for kind in (P.OUT_POPULATION, P.OUT_AMPLITUDE):
        def call(lo, hi):
            return plan.contract_batch(j, to_dev(torch, dev, kr[lo:hi]),
                                       to_dev(torch, dev, np.arange(hi - lo, dtype=np.int32)),
                                       to_dev(torch, dev, prefix_words(pre[lo:hi], plan.n_words)), kind)[0]
        whole = call(0, E)
        assert torch.equal(whole[:300], call(0, 300))
        assert torch.equal(whole[300:340], call(300, 340))
        assert torch.equal(whole[E - 1:], call(E - 1, E))
