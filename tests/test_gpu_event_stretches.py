"""Event-driven iterations of the separable objective, a stretch of them per launch: the same bits as one pass per
iteration, at the vector lengths where the launch changes its form, over rebases and steps of the step size."""
import numpy as np
import pytest

from paper_2307_11617_amd import rfast_set_rebase_interval, rfast_use_blocks
from rfast_workloads import configs, graphs, problems

import harness

pytestmark = pytest.mark.gpu
FIELDS = ("X", "Z", "G", "V_RING", "SIGMA_RING", "RHO_TILDE", "T_NODE", "TAU_R", "TAU_C", "ROUND")


@pytest.mark.parametrize("graph,n,p,momentum", [
    (graphs.directed_ring, 5, 1, 0.0), (graphs.mesh, 12, 255, 0.9), (graphs.tree_pull_star_push, 40, 1028, 0.0),
    (graphs.binary_tree, 9, 65_535, 0.0), (graphs.exponential, 8, 65_536, 0.9), (graphs.tree_pull_star_push, 12, 65_537, 0.0),
    (graphs.bidirectional_ring, 4, 65_539, 0.9), (graphs.mesh, 70, 70_000, 0.0)])
def test_same_bits(graph, n, p, momentum):
    r, c = graph(n)
    gamma = 0.05 if graph in (graphs.mesh, graphs.exponential, graphs.bidirectional_ring) else 0.002
    w = configs._mk(f"events_{n}_{p}", n, p, r, c, 3, gamma, 0, "diag_quadratic", problems.diag_quadratic(n, p, 5), 0.6, 0.3, 5, burst=3)
    a, b = harness.make_gpu(w), harness.make_gpu(w)
    rfast_use_blocks(b.ctx, False)
    x0 = np.random.default_rng(1).standard_normal((n, p)).astype(np.float32)
    for g in (a, b):
        rfast_set_rebase_interval(g.ctx, 23)
        if momentum:
            g.set_optimizer(momentum, 0.01)
        g.set_gamma_schedule(20, 0.8)
        g.init(x0, None)
        for k, iterations in enumerate((70, 1, 33)):
            g.run_events(iterations, 6 + k, None, w.sched.d_max, 0.2, w.gamma)
        g.check()
    for f in FIELDS + (("MOMENTUM",) if momentum else ()):
        assert np.array_equal(a.read(f), b.read(f)), f
    assert np.abs(a.read("X") - x0).max() > 1e-5
