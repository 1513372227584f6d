"""The tile-per-wavefront kernel keeps fewer versions of a node on chip than the ring in memory has slots.  Reads of versions
that have left the chip, versions that somebody holds after the launch, and buffers consumed after their version has left
the ring must give the bits of one pass per round."""
import numpy as np
import pytest

from paper_2307_11617_amd import rfast_set_rebase_interval, rfast_set_tile_group, rfast_use_blocks
from rfast_workloads import configs, graphs, problems
from rfast_workloads.schedule import ScheduleSpec

import harness

pytestmark = pytest.mark.gpu
FIELDS = ("X", "Z", "G", "V_RING", "SIGMA_RING", "RHO_TILDE", "T_NODE", "TAU_R", "TAU_C", "SLOT_R", "SLOT_C", "DELIV_R", "DELIV_C", "T_HIST", "ROUND")


# two, four and six edge slots; up to sixteen, twelve and eight wavefronts per compute unit; from 12 versions down to 5 on chip
@pytest.mark.parametrize("graph,n,p,d_max,burst,group,momentum", [
    ("directed_ring", 8, 4100, 3, 8, 0, 0.0), ("directed_ring", 8, 1027, 2, 6, 0, 0.9), ("bidirectional_ring", 16, 520, 4, 10, 4, 0.0),
    ("bidirectional_ring", 5, 2052, 0, 9, 2, 0.0), ("mesh", 12, 333, 4, 8, 0, 0.0), ("mesh", 16, 1028, 8, 4, 1, 0.9),
    ("exponential", 32, 260, 3, 12, 0, 0.0), ("exponential", 20, 130, 16, 4, 0, 0.0),
    # a lane per node
    ("mesh", 36, 333, 4, 4, 0, 0.0), ("bidirectional_ring", 33, 64, 8, 3, 4, 0.9), ("exponential", 64, 130, 3, 9, 0, 0.0), ("binary_tree", 50, 1001, 2, 2, 0, 0.0)])
def test_versions_that_have_left_the_chip(graph, n, p, d_max, burst, group, momentum):
    wr, wc = getattr(graphs, graph)(n)
    R, C = graphs.from_dense(wr), graphs.from_dense(wc)
    p_act = np.where(np.arange(n) % 4 == 1, 0.06, np.where(np.arange(n) % 4 == 2, 1.0, 0.7))   # stragglers hold old versions
    sched = ScheduleSpec(n, R.nnz_off, C.nnz_off, p_act, d_max, 0.6, seed=n + burst)
    w = configs.Workload(f"on_chip_{graph}", n, p, R, C, d_max + burst - 1, burst, 0.01, 0, "diag_quadratic",
                         problems.diag_quadratic(n, p, 3), sched, 0.1, 50 + n, 1e-4)
    pair = [harness.make_gpu(w), harness.make_gpu(w)]
    rng = np.random.default_rng(n)
    x0 = rng.standard_normal((n, p)).astype(np.float32)
    for g, blocks in zip(pair, (2, 0)):
        rfast_use_blocks(g.ctx, blocks)
        if group:
            rfast_set_tile_group(g.ctx, group)
        rfast_set_rebase_interval(g.ctx, 61)
        if momentum:
            g.set_optimizer(momentum, 1e-3)
        g.init(x0, None)
    _, dev = harness.upload_chunk(pair[0], w, 0, 130)
    for lo, hi in ((0, 3), (3, 50), (50, 130)):   # short, long, across two rebases
        for g in pair:
            g.run(hi - lo, *(dev[k][lo:hi] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")), w.gamma)
            g.check()
        for f in FIELDS:
            assert np.array_equal(pair[0].read(f), pair[1].read(f)), (hi, f)


@pytest.mark.parametrize("graph,n,p,momentum", [("mesh", 36, 333, 0.9), ("bidirectional_ring", 64, 260, 0.0), ("exponential", 40, 1, 0.0), ("binary_tree", 33, 4098, 0.0)])
def test_synchronous_steps_of_more_than_32_nodes(graph, n, p, momentum):
    """Several steps per launch (from two on) and one step per launch: the same bits."""
    wr, wc = getattr(graphs, graph)(n)
    R, C = graphs.from_dense(wr), graphs.from_dense(wc)
    sched = ScheduleSpec(n, R.nnz_off, C.nnz_off, np.ones(n), 1, 0.0, seed=n)
    w = configs.Workload(f"sync_{graph}", n, p, R, C, 1, 1, 0.01, 0, "diag_quadratic", problems.diag_quadratic(n, p, 3), sched, 0.1, 9, 1e-4)
    pair = [harness.make_gpu(w), harness.make_gpu(w)]
    x0 = np.random.default_rng(n).standard_normal((n, p)).astype(np.float32)
    for g, blocks in zip(pair, (1, 0)):
        rfast_use_blocks(g.ctx, blocks)
        if momentum:
            g.set_optimizer(momentum, 1e-3)
        g.init(x0, None)
        for steps in (2, 1, 9):
            g.sync_run(steps, w.gamma)
    for f in ("X", "Z", "T_NODE", "ROUND") + (("MOMENTUM",) if momentum else ()):
        assert np.array_equal(pair[0].read(f), pair[1].read(f)), f
