"""Values and gradients of small circuits around the numbers of trajectories from which they
take the windows of single gates, against the FP64 oracle: a few error sets, repeated.

Tolerance: the gradient tests' 1e-5 relative (windows: two FP32 products of a gate's 4 x 4
terms for each of fewer than 100 gates, 200 sqrt(8) 2^-24 = 3e-5 with equal signs)."""
import numpy as np
import pytest

import workloads as W
from oracle import gradients as gr
from tests.gpu_helpers import to_dev, torch_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,layers,damped", [(8, 1, False), (8, 1, True), (8, 2, True), (9, 1, True), (11, 1, False),
                                             (10, 1, False), (11, 2, False), (12, 1, False)])
@pytest.mark.parametrize("E", [1535, 1536, 1920, 2560, 3071, 3072])
def test_many_trajectories(n, layers, damped, E):
    import paper_2604_08467_amd as P
    torch, dev = torch_dev()
    theta = np.random.default_rng(n).uniform(0, 2 * np.pi, size=2 * n * layers)
    c = W.hea(n, layers, theta, [W.depolarizing(0.05)] + ([W.amplitude_damping(0.1)] if damped else []))
    gp, ga = W.rotation_spec(c)
    terms = W.zz_chain_terms(n)
    plan = P.Plan(c, [10] * (n // 10) + ([n % 10] if n % 10 else []), method="statevector")
    few, mult, _, _ = plan.sample_trajectories(n + 1, 3)
    which = np.arange(E) % len(few)
    w = np.linspace(0.5, 1.5, E) / E
    wf = np.array([w[which == k].sum() for k in range(len(few))])
    args = (P.GradSpec(len(theta), gp, ga, terms), to_dev(torch, dev, few[which]), to_dev(torch, dev, w),
            to_dev(torch, dev, theta))
    f_ref = gr.value(c, few, wf, theta, gp, ga, terms)
    g_ref = gr.adjoint_gradient(c, few, wf, theta, gp, ga, terms)
    t_ref = gr.trajectory_values(c, few, theta, gp, ga, terms)
    for want_grad in (False, True):
        out = plan.expect_grad(*args, want_grad=want_grad)
        assert abs(float(out["value"].item()) - f_ref) <= 1e-5 * len(terms)
        np.testing.assert_allclose(out["traj_values"].cpu().numpy(), np.asarray(t_ref)[which], atol=1e-5 * len(terms))
        if want_grad:
            assert np.linalg.norm(out["grad"].cpu().numpy() - g_ref) <= 1e-5 * np.linalg.norm(g_ref)
