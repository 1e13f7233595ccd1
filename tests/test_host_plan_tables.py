"""Plan constants of the adjoint cluster windows and the network windows: counted in
plan_device_bytes, and left out, not refused, where device_budget_bytes has no room for them."""
import numpy as np

import workloads as W


def _plans(c, batches, **kw):
    import paper_2604_08467_amd as P
    full = P.Plan(c, batches, device=-1, **kw).plan_device_bytes
    same = P.Plan(c, batches, device=-1, device_budget_bytes=full, **kw).plan_device_bytes
    less = P.Plan(c, batches, device=-1, device_budget_bytes=full - 1, **kw).plan_device_bytes
    return full, same, less


def test_adjoint_tables_are_counted():
    n, layers = 10, 2
    c = W.hea(n, layers, np.linspace(0.1, 3.0, 2 * n * layers), [W.depolarizing(0.02)])
    full, same, less = _plans(c, [10], method="statevector")
    assert same == full
    # without them: at least the 64-bit gates and inserted operators less (16 entries of 16 bytes)
    assert less <= full - 256 * (c.n_gates + 4 * c.n_sites)


def test_network_windows_are_counted():
    # a chain of 34 qubits (no statevector, so no adjoint tables) with runs of rank 13 and more
    c = W.random_brickwork(34, 6, np.random.default_rng(3), 0.01)
    full, same, less = _plans(c, [10, 10, 14], method="network", hypersamples=4)
    assert same == full and less < full
