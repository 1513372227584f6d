"""Vector lengths that are no multiple of four (rows start at any float's address, the last group of a row is short):
the multi-round and multi-step kernels against one pass per round, bit for bit, and the one-pass kernels against the
fp64 oracle."""
import numpy as np
import pytest

from paper_2307_11617_amd import rfast_set_rebase_interval, rfast_use_blocks
from rfast_workloads import configs, graphs, problems
from rfast_workloads.schedule import ScheduleSpec

import harness

pytestmark = pytest.mark.gpu
FIELDS = ("X", "Z", "G", "V_RING", "SIGMA_RING", "RHO_TILDE", "T_NODE", "TAU_R", "TAU_C", "ROUND")


def _workload(n, p, graph=graphs.bidirectional_ring):
    r, c = graph(n)
    R, C = graphs.from_dense(r), graphs.from_dense(c)
    sched = ScheduleSpec(n, R.nnz_off, C.nnz_off, np.where(np.arange(n) % 3 == 1, 0.2, 0.9), 2, 0.3, seed=n)
    return configs.Workload(f"ragged_{n}_{p}", n, p, R, C, 4, 3, 0.02, 0, "diag_quadratic", problems.diag_quadratic(n, p, n),
                            sched, 0.1, 90 + n, 1e-4)


def _pair(w, variant=False):
    a, b = harness.make_gpu(w), harness.make_gpu(w)
    rfast_use_blocks(b.ctx, False)
    x0 = np.random.default_rng(1).standard_normal((w.n, w.p)).astype(np.float32)
    for g in (a, b):
        rfast_set_rebase_interval(g.ctx, 19)
        if variant:
            g.set_optimizer(0.9, 0.01)
        g.init(x0, None)
    return a, b, x0


@pytest.mark.parametrize("n,p,variant", [(16, 1025, False), (16, 1026, True), (16, 1027, False), (5, 1, False), (5, 3, True),
                                         (24, 6, False), (36, 1031, False), (40, 2, True), (16, 131_075, False),
                                         (17, 500_001, False)])
def test_rounds(n, p, variant):
    w = _workload(n, p)
    a, b, _ = _pair(w, variant)
    st, dev = harness.upload_chunk(a, w, 0, 40)
    for lo, hi in ((0, 25), (25, 40)):
        for g in (a, b):
            g.run(hi - lo, *[dev[k][lo:hi].contiguous() for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma)
            g.check()
    for f in FIELDS + (("MOMENTUM",) if variant else ()):
        assert np.array_equal(a.read(f), b.read(f)), f
    da, db = a.diagnostics(), b.diagnostics()
    assert all(abs(da[k] - db[k]) <= 1e-9 * abs(db[k]) for k in ("consensus_sq", "z_sq", "loss_at_xbar"))


@pytest.mark.parametrize("n,p,variant", [(16, 1025, True), (9, 7, False), (32, 515, False)])
def test_synchronous_steps(n, p, variant):
    a, b, _ = _pair(_workload(n, p), variant)
    for steps in (20, 1, 12):
        for g in (a, b):
            g.sync_run(steps, 0.02, None)
            g.check()
        for f in ("X", "Z", "G", "T_NODE"):
            assert np.array_equal(a.read(f), b.read(f)), (steps, f)


@pytest.mark.parametrize("n,p", [(8, 1), (8, 1027), (48, 6)])
def test_one_pass_against_the_oracle(n, p):
    w = _workload(n, p)
    _, b, x0 = _pair(w)
    orc = harness.make_oracle(w, None, x0)
    st, dev = harness.upload_chunk(b, w, 0, 30)
    b.run(30, *[dev[k] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma)
    for r in range(30):
        orc.round(*[st[k][r] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma)
    assert harness.rel_l2(b.read("X"), orc.x) <= 1e-4 and harness.rel_l2(b.read("Z"), orc.z) <= 1e-4
    d = b.diagnostics()
    xbar = orc.x.mean(0)
    assert abs(d["consensus_sq"] - ((orc.x - xbar) ** 2).sum()) <= 1e-3 * d["consensus_sq"]


@pytest.mark.parametrize("floats", [1, 262_143, 262_144, 262_145, 524_289, 5_000_001])
def test_reading_a_field_back(floats):
    """Fields below, at and above one piece of the staged copy, read while rounds are still under way."""
    import torch
    w = _workload(2, floats)
    gpu = harness.make_gpu(w)
    x0 = np.random.default_rng(7).standard_normal((2, floats)).astype(np.float32)
    gpu.init(x0, None)
    assert np.array_equal(gpu.read("X"), x0)
    st, dev = harness.upload_chunk(gpu, w, 0, 5)
    gpu.run(5, *[dev[k] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma)
    got = gpu.read("X")
    torch.cuda.synchronize()
    assert np.array_equal(gpu.read("X"), got) and np.abs(got - x0).max() > 1e-3
