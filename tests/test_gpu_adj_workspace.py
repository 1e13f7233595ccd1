"""Adjoint calls in small workspaces: a plan with the cluster tables takes every workspace that
the windows of single gates take (a plan without the tables, for want of budget).

20 qubits with damping, one trajectory: the cluster form has one window, and so one 8 MB
checkpoint, more.  Gradients agree to 1e-5, the cluster windows' tolerance."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_helpers import to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _smallest(P, torch, dev, call, size):
    """The smallest workspace (to 128 KB) that the call takes, and its result there."""
    lo, hi, out = 0, size, None
    while hi - lo > 1 << 17:
        mid = (lo + hi) // 2
        try:
            got = call(torch.empty(mid, dtype=torch.uint8, device=dev))
        except P.PtsbeError as e:
            assert e.status == 3, str(e)
            lo = mid
        else:
            out, hi = got, mid
    return hi, out


@pytest.mark.parametrize("want_grad", [False, True])
@pytest.mark.parametrize("layers,gamma", [(10, 0.02), (3, 0.0)])
def test_small_workspaces_go_to_the_single_gate_windows(layers, gamma, want_grad):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    n = 20
    theta = np.random.default_rng(1).uniform(0, 2 * np.pi, size=2 * n * layers)
    c = W.hea(n, layers, theta, [W.depolarizing(0.01)] + ([W.amplitude_damping(gamma)] if gamma else []))
    gp, ga = W.rotation_spec(c)
    spec = P.GradSpec(len(theta), gp, ga, W.zz_chain_terms(n))
    plan = P.Plan(c, [10, 10], method="statevector")
    tight = P.Plan(c, [10, 10], method="statevector", device_budget_bytes=plan.plan_device_bytes - 1)
    kr, _, _, _ = plan.sample_trajectories(2, 1)
    args = (spec, to_dev(torch, dev, kr), to_dev(torch, dev, np.ones(1)), to_dev(torch, dev, theta))
    full = plan.expect_grad(*args)
    least = []
    for p in (tight, plan):
        size, out = _smallest(P, torch, dev,
                              lambda ws: p.expect_grad(*args, want_grad=want_grad, workspace=ws), 1 << 30)
        least.append(size)
        assert abs(float(out["value"].item() - full["value"].item())) <= 1e-5 * (n - 1)
        if want_grad:
            g, ref = out["grad"].cpu().numpy(), full["grad"].cpu().numpy()
            assert np.linalg.norm(g - ref) <= 1e-5 * np.linalg.norm(ref)
    print("smallest workspaces", least, flush=True)
    assert least[1] <= least[0] + (1 << 17)
