"""Several rounds per launch on graphs that only a part of the nodes is read over: all edges of C lead to one node (its sum is
formed by the senders' lanes), or trees.  Sizes at the edges of the tiling: a lane per node and several, nodes that leave lanes
over, ragged rows, rings from two slots up, launches across rebases, versions that have left the chip."""
import ctypes

import numpy as np
import pytest

from paper_2307_11617_amd import lib, rfast_block_info, rfast_set_rebase_interval, rfast_set_tile_group, rfast_use_blocks
from rfast_workloads import configs, graphs, problems

import harness

pytestmark = pytest.mark.gpu


def _star_at(n, hub):
    """A directed path as R from node `hub` on, and every other node pushes to it."""
    r, c = np.zeros((n, n)), np.zeros((n, n))
    order = [(hub + k) % n for k in range(n)]
    r[hub, hub] = c[hub, hub] = 1.0
    for a, b in zip(order, order[1:]):
        r[b, b], r[b, a] = 0.7, 0.3
        c[hub, b] = 0.3 + 0.5 * b / n
        c[b, b] = 1.0 - c[hub, b]
    return r, c


def _star_and_tree(n):
    """Every node pulls from node 0, and pushes to its parent in a binary tree."""
    r, c = graphs.tree_pull_star_push(n)[0] * 0.0, graphs.binary_tree(n)[1]
    r[0, 0] = 1.0
    r[np.arange(1, n), np.arange(1, n)], r[1:, 0] = 0.5, 0.5
    return r, c


BUILD = {"star_and_tree": _star_and_tree, "directed_ring": graphs.directed_ring, "bidirectional_ring": graphs.bidirectional_ring, "tree_star": graphs.tree_pull_star_push, "binary_tree": graphs.binary_tree, "line_tree": graphs.line_tree, "star_at_2": lambda n: _star_at(n, 2), "star_at_5": lambda n: _star_at(n, 5),
         "star_at_last": lambda n: _star_at(n, n - 1)}
SHAPES = [("tree_star", 64, 1028, 16, 4, 0, 0.0), ("tree_star", 64, 1027, 4, 3, 4, 0.9), ("tree_star", 33, 260, 0, 1, 0, 0.0),
          ("tree_star", 47, 66, 8, 4, 2, 0.0), ("tree_star", 32, 513, 8, 2, 4, 0.9), ("tree_star", 20, 1028, 3, 8, 0, 0.0),
          ("tree_star", 9, 4100, 16, 4, 0, 0.0), ("tree_star", 5, 3, 2, 2, 0, 0.0), ("star_at_5", 17, 516, 5, 2, 1, 0.0),
          ("star_at_5", 50, 129, 3, 3, 0, 0.9), ("star_at_last", 64, 64, 8, 4, 0, 0.0), ("star_at_last", 12, 1, 1, 1, 0, 0.0)]
FEWER = [("tree_star", 64, 8_196, 16, 4, 0, 0.0), ("star_at_5", 20, 20_002, 16, 2, 0, 0.9)]   # fewer versions on chip than the longest delay reads


@pytest.mark.parametrize("graph,n,p,d_max,burst,group,momentum", SHAPES + FEWER)
def test_every_push_to_one_node(graph, n, p, d_max, burst, group, momentum, monkeypatch):
    """Against the oracle: x, z, samples, both rings, buffers, in calls of 2, 3 and 45 rounds; half of the runs with rebases."""
    r, c = BUILD[graph](n)
    w = configs._mk("one_receiver", n, p, r, c, d_max, 0.1 / n, 0, "diag_quadratic", problems.diag_quadratic(n, p, 5), 0.7, 0.4, 5, noise_std=0.1,
                    burst=burst)
    w.sched.p_active[1::4] = 0.1
    make = harness.make_gpu

    def launches(w):
        g = make(w)
        rfast_use_blocks(g.ctx, 2)
        rfast_set_rebase_interval(g.ctx, 25 if n % 2 else 0)
        if group:
            rfast_set_tile_group(g.ctx, group)
        if p % 4 == 0:
            assert rfast_block_info(g.ctx, with_kind=True) == (64 // n, True)
        assert (_versions_on_chip(g) < d_max + min(burst, 2)) == ((graph, n, p, d_max, burst, group, momentum) in FEWER)
        return g
    monkeypatch.setattr(harness, "make_gpu", launches)
    harness.run_parity(w, 100, every=(2, 3, 45, 50), rebase=n % 2 == 1, momentum=momentum, weight_decay=1e-3 if momentum else 0.0)


@pytest.mark.parametrize("graph,n,p,d_max,burst,group,momentum", [
    ("binary_tree", 64, 1028, 16, 4, 0, 0.0), ("binary_tree", 63, 1027, 4, 3, 4, 0.9), ("binary_tree", 21, 516, 8, 4, 2, 0.0), ("binary_tree", 7, 130, 3, 2, 0, 0.9),
    ("star_and_tree", 64, 1028, 9, 4, 0, 0.0), ("star_and_tree", 20, 1027, 12, 2, 4, 0.9),
    ("line_tree", 40, 260, 8, 4, 0, 0.0), ("line_tree", 6, 2052, 2, 6, 4, 0.0), ("binary_tree", 3, 1, 1, 2, 0, 0.0),
    ("bidirectional_ring", 16, 1028, 16, 4, 0, 0.0), ("directed_ring", 30, 519, 20, 3, 0, 0.9), ("bidirectional_ring", 50, 130, 13, 8, 4, 0.0)])
def test_trees(graph, n, p, d_max, burst, group, momentum):
    """The bits of one pass per round."""
    _bits_of_one_pass(graph, n, p, d_max, burst, group, momentum)


# of four and five nodes on edge slots while the chip holds every tile
@pytest.mark.parametrize("graph,n,p,d_max,burst,group,momentum", [
    ("tree_star", 4, 1028, 16, 4, 0, 0.0), ("tree_star", 4, 70_000, 16, 4, 0, 0.0), ("star_at_2", 5, 50_003, 16, 2, 0, 0.9), ("star_at_last", 5, 60_000, 16, 4, 2, 0.0),
    ("tree_star", 7, 2051, 4, 3, 4, 0.9), ("star_at_2", 5, 516, 3, 8, 2, 0.0), ("star_at_5", 6, 1, 1, 1, 0, 0.0), ("star_at_2", 7, 20_000, 8, 4, 1, 0.0),
    ("star_at_last", 4, 130, 0, 2, 0, 0.9)])
def test_stars_of_few_senders(graph, n, p, d_max, burst, group, momentum):
    """The bits of one pass per round."""
    _bits_of_one_pass(graph, n, p, d_max, burst, group, momentum)


@pytest.mark.parametrize("graph,n,p,d_max,burst,group,momentum", [
    ("bidirectional_ring", 16, 20_004, 16, 4, 0, 0.0), ("bidirectional_ring", 16, 17_003, 16, 2, 0, 0.0), ("directed_ring", 30, 7_001, 20, 3, 0, 0.9),
    ("bidirectional_ring", 50, 6_404, 13, 8, 4, 0.0), ("bidirectional_ring", 9, 40_002, 14, 4, 2, 0.0), ("binary_tree", 64, 8_196, 16, 4, 0, 0.0),
    ("line_tree", 40, 9_001, 16, 2, 1, 0.9), ("star_at_2", 5, 80_003, 20, 4, 0, 0.0)])
def test_fewer_versions_on_chip_than_the_longest_delay_reads(graph, n, p, d_max, burst, group, momentum):
    """More tiles than the chip holds with every version: reads of versions that have left it are ordinary then.  The bits of one pass per round."""
    g = _bits_of_one_pass(graph, n, p, d_max, burst, group, momentum)
    assert _versions_on_chip(g) < d_max + min(burst, 2)


def _versions_on_chip(gpu):
    f = lib()._Z16rfast_wave_slotsPK9rfast_ctx   # what a launch takes
    f.argtypes, f.restype = [ctypes.c_void_p], ctypes.c_int
    return f(gpu.ctx)


def _bits_of_one_pass(graph, n, p, d_max, burst, group, momentum):
    r, c = BUILD[graph](n)
    w = configs._mk("trees", n, p, r, c, d_max, 0.01, 0, "diag_quadratic", problems.diag_quadratic(n, p, 5), 0.7, 0.4, 5, noise_std=0.1, burst=burst)
    w.sched.p_active[1::4] = 0.1
    pair = [harness.make_gpu(w), harness.make_gpu(w)]
    x0 = np.random.default_rng(n).standard_normal((n, p)).astype(np.float32)
    for g, blocks in zip(pair, (2, 0)):
        rfast_use_blocks(g.ctx, blocks)
        rfast_set_rebase_interval(g.ctx, 29)
        if group:
            rfast_set_tile_group(g.ctx, group)
        if momentum:
            g.set_optimizer(momentum, 1e-3)
        g.init(x0, None)
    _, dev = harness.upload_chunk(pair[0], w, 0, 90)
    for lo, hi in ((0, 2), (2, 40), (40, 90)):
        for g in pair:
            g.run(hi - lo, *(dev[k][lo:hi] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")), w.gamma)
            g.check()
        for f in ("X", "Z", "G", "V_RING", "SIGMA_RING", "RHO_TILDE", "T_NODE", "TAU_R", "TAU_C", "ROUND"):
            assert np.array_equal(pair[0].read(f), pair[1].read(f)), (hi, f)
    return pair[0]


@pytest.mark.parametrize("graph,n,d_max", [("binary_tree", 64, 16), ("binary_tree", 21, 16), ("line_tree", 40, 16), ("tree_star", 64, 4), ("star_at_5", 17, 5),
                                           ("bidirectional_ring", 30, 4)])
@pytest.mark.parametrize("backwards", [False, True])
def test_infinities_stay_where_edges_lead(graph, n, d_max, backwards):
    """The first node that is read over C or over R has diverged, for longer than the chip keeps its versions and with nobody else active.  An
    infinity takes a round per edge, so two rounds later nobody further away than that has anything but finite values, whatever
    the launch does with the edges that a node has not got."""
    r, c = BUILD[graph](n)
    if backwards:
        r, c = r[::-1, ::-1].copy(), c[::-1, ::-1].copy()
    p = 64
    off = 1 - np.eye(n)
    for m in (c, r):
        bad = int(np.flatnonzero((m * off).any(axis=0))[0])
        w = configs._mk("infinities", n, p, r, c, d_max, 1e-3, 0, "diag_quadratic", problems.diag_quadratic(n, p, 5), 1.0, 0.0, 5, burst=2)
        g = harness.make_gpu(w)
        rfast_use_blocks(g.ctx, 2)
        x0 = np.random.default_rng(n).standard_normal((n, p)).astype(np.float32)
        x0[bad] = np.inf
        g.init(x0, None)
        _, dev = harness.upload_chunk(g, w, 0, 42)
        dev["active"][:40] = 0
        dev["active"][:40, bad] = 1
        for lo, hi in ((0, 40), (40, 42)):
            g.run(hi - lo, *(dev[k][lo:hi] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")), w.gamma)
            g.check()
        assert int(g.read("T_NODE")[bad]) == 42 and not np.isfinite(g.read("X")[bad]).any()
        hop = ((r != 0) | (c != 0)).astype(int)      # [to, from]
        far = np.linalg.matrix_power(hop, 2)[:, bad] == 0
        for f in ("X", "Z"):
            ok = np.isfinite(g.read(f)).all(axis=1)
            assert ok[far].all(), (bad, f, np.flatnonzero(far & ~ok))
