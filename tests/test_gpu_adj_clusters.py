"""Cluster form of the adjoint passes (circuits of at least 8 qubits) against the FP64
oracle gradients: tiles of 8..11 qubits, one and several windows, unitary and damped
operators, shared parameters, and small workspaces (one trajectory per chunk, one
workgroup per trajectory).

Tolerance: a pass applies at most 60 cluster matrices of 32-term FP32 sums forward and
back, 120 sqrt(32) 2^-24 = 4e-5 if every rounding error had the same sign, their square
root of that number with random signs; 1e-5 relative lies between."""
import numpy as np
import pytest

import workloads as W
from oracle import gradients as gr
from tests.gpu_helpers import to_dev, torch_dev

pytestmark = pytest.mark.gpu


def _case(n, layers, damped, E, seed):
    import paper_2604_08467_amd as P
    rng = np.random.default_rng(seed)
    theta = rng.uniform(0, 2 * np.pi, size=2 * n * layers)
    chans = [W.depolarizing(0.05)] + ([W.amplitude_damping(0.1)] if damped else [])
    c = W.hea(n, layers, theta, chans)
    gp, ga = W.rotation_spec(c)
    terms = W.zz_chain_terms(n)
    plan = P.Plan(c, [10] * (n // 10) + ([n % 10] if n % 10 else []), method="statevector")
    kr, mult, _, _ = plan.sample_trajectories(seed + 1, E)
    return P, c, plan, kr, mult / mult.sum(), theta, gp, ga, terms


def _check(out, c, kr, w, theta, gp, ga, terms):
    f_ref = gr.value(c, kr, w, theta, gp, ga, terms)
    g_ref = gr.adjoint_gradient(c, kr, w, theta, gp, ga, terms)
    g = out["grad"].cpu().numpy()
    assert abs(float(out["value"].item()) - f_ref) <= 1e-5 * len(terms)
    assert np.linalg.norm(g - g_ref) <= 1e-5 * np.linalg.norm(g_ref)
    np.testing.assert_allclose(out["traj_values"].cpu().numpy(),
                               gr.trajectory_values(c, kr, theta, gp, ga, terms), atol=1e-5 * len(terms))


@pytest.mark.parametrize("damped", [False, True])
@pytest.mark.parametrize("n,layers,E", [(8, 3, 5), (9, 2, 3), (10, 2, 3), (11, 2, 2), (12, 2, 2), (14, 2, 1)])
def test_cluster_gradient_matches_oracle(n, layers, E, damped):
    torch, dev = torch_dev()
    P, c, plan, kr, w, theta, gp, ga, terms = _case(n, layers, damped, E, 100 * n + damped)
    gp[gp == 1] = 0                                    # two rotations share a parameter
    theta[1] = theta[0]
    spec = P.GradSpec(len(theta), gp, ga, terms)
    args = (spec, to_dev(torch, dev, kr), to_dev(torch, dev, w), to_dev(torch, dev, theta))
    _check(plan.expect_grad(*args), c, kr, w, theta, gp, ga, terms)
    only = plan.expect_grad(*args, want_grad=False)    # value-only windows
    assert abs(float(only["value"].item()) - gr.value(c, kr, w, theta, gp, ga, terms)) <= 1e-5 * len(terms)


@pytest.mark.parametrize("damped", [False, True])
def test_cluster_gradient_in_chunks(damped):
    torch, dev = torch_dev()
    P, c, plan, kr, w, theta, gp, ga, terms = _case(13, 2, damped, 3, 77)
    spec = P.GradSpec(len(theta), gp, ga, terms)
    args = (spec, to_dev(torch, dev, kr), to_dev(torch, dev, w), to_dev(torch, dev, theta))
    whole = plan.expect_grad(*args)
    _check(whole, c, kr, w, theta, gp, ga, terms)
    # shrink the workspace until the call refuses it: every accepted size gives the same result
    size, seen = 4 << 20, 0
    while size > 1 << 20:
        try:
            out = plan.expect_grad(*args, workspace=torch.empty(size, dtype=torch.uint8, device=dev))
        except P.PtsbeError:
            break
        _check(out, c, kr, w, theta, gp, ga, terms)
        seen += 1
        size = size * 7 // 8
    assert seen > 0
