"""Tables of the adjoint cluster windows: they come with the plan (a plan's first gradient
allocates nothing on the device), and a plan whose device_budget_bytes has no room for them
takes the windows of single gates.

Tolerances: as the cluster windows' (1e-5 relative)."""
import numpy as np
import pytest

import workloads as W
from oracle import gradients as gr
from tests.gpu_helpers import to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _case(n, layers, channel, seed, **kw):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    theta = np.random.default_rng(seed).uniform(0, 2 * np.pi, size=2 * n * layers)
    c = W.hea(n, layers, theta, [channel])
    gp, ga = W.rotation_spec(c)
    plan = P.Plan(c, [10] * (n // 10) + ([n % 10] if n % 10 else []), method="statevector", **kw)
    kr, mult, _, _ = plan.sample_trajectories(seed + 1, 3)
    w = mult / mult.sum()
    spec = P.GradSpec(len(theta), gp, ga, W.zz_chain_terms(n))
    args = (spec, to_dev(torch, dev, kr), to_dev(torch, dev, w), to_dev(torch, dev, theta))
    ref = (c, kr, w, theta, gp, ga, W.zz_chain_terms(n))
    return torch, dev, plan, args, ref


def test_first_gradient_allocates_nothing():
    # 5 MB of inserted operators in 64 bits: more than allocations are rounded to
    many = W.Channel(np.concatenate([W.depolarizing(0.05).kraus * np.sqrt(1 / 16)] * 16), None)
    torch, dev, plan, args, _ = _case(9, 20, many, 5)
    ws = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
    warm = _case(9, 2, W.depolarizing(0.05), 6)          # kernels loaded, torch's blocks in its cache
    for want in (False, True):
        warm[2].expect_grad(*warm[3], want_grad=want, workspace=ws)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    plan.expect_grad(*args, want_grad=False, workspace=ws)
    plan.expect_grad(*args, workspace=ws)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] == free


@pytest.mark.parametrize("n", [8, 13])
def test_budget_without_room_for_the_tables(n):
    import paper_2604_08467_amd as P
    torch, dev, plan, args, (c, kr, w, theta, gp, ga, terms) = _case(n, 2, W.depolarizing(0.05), n)
    tight = P.Plan(c, plan.batch_sizes, method="statevector", device_budget_bytes=plan.plan_device_bytes - 1)
    assert tight.plan_device_bytes < plan.plan_device_bytes
    f_ref = gr.value(c, kr, w, theta, gp, ga, terms)
    g_ref = gr.adjoint_gradient(c, kr, w, theta, gp, ga, terms)
    for p in (plan, tight):
        out = p.expect_grad(*args)
        assert abs(float(out["value"].item()) - f_ref) <= 1e-5 * len(terms)
        assert np.linalg.norm(out["grad"].cpu().numpy() - g_ref) <= 1e-5 * np.linalg.norm(g_ref)
