"""The one-pass round of the separable objective at the edges of its batches of in-edges (four and eight): graphs whose
largest in-degree is one batch take another instantiation than graphs with one more."""
import numpy as np
import pytest

from paper_2307_11617_amd import rfast_use_blocks
from rfast_workloads import configs, graphs, problems

import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("momentum", [0.0, 0.9])
@pytest.mark.parametrize("degree,p", [(8, 1001), (9, 1001), (8, 516), (9, 516), (4, 286_000), (5, 286_000), (4, 286_001), (5, 286_001)])
def test_in_degree_of_one_batch_and_one_more(degree, p, momentum, monkeypatch):
    n = 14
    adj = np.eye(n) + np.roll(np.eye(n), 1, axis=0)   # a directed ring, and further in-edges of node 0
    adj[0, :] = 0.0
    adj[0, 0] = adj[0, n - 1] = 1.0
    adj[0, 2:degree + 1] = 1.0
    assert (adj[0] != 0).sum() - 1 == degree   # (batches of eight below 4 M values, of four beyond)
    w = configs._mk("ring_and_hub", n, p, adj / adj.sum(1, keepdims=True), adj / adj.sum(0, keepdims=True), 3, 0.01, 0, "diag_quadratic",
                    problems.diag_quadratic(n, p, 5), 0.7, 0.2, 5, noise_std=0.1, burst=3)
    make = harness.make_gpu

    def one_pass(w):
        g = make(w)
        rfast_use_blocks(g.ctx, False)
        return g
    monkeypatch.setattr(harness, "make_gpu", one_pass)
    coords = None if p < 5000 else np.unique(np.concatenate([np.arange(0, p, 4099), [p - 2, p - 1]]))
    harness.run_parity(w, 60, every=20, coords=coords, momentum=momentum, weight_decay=1e-3 if momentum else 0.0, check_rings=coords is None)


@pytest.mark.parametrize("p", [1001, 64_000, 500_001])
def test_versions_nobody_pulls_are_not_kept(p, monkeypatch):
    """The leaves of a tree that everybody pulls from above: their versions read as zero, everything else as in the oracle."""
    n = 9
    r, c = graphs.tree_pull_star_push(n)
    w = configs._mk("tree_star", n, p, r, c, 3, 0.002, 0, "diag_quadratic", problems.diag_quadratic(n, p, 5), 0.7, 0.2, 5,
                    noise_std=0.1, burst=3)
    make = harness.make_gpu

    def one_pass(w):
        g = make(w)
        rfast_use_blocks(g.ctx, False)
        return g
    monkeypatch.setattr(harness, "make_gpu", one_pass)
    coords = None if p < 5000 else np.unique(np.concatenate([np.arange(0, p, 4099), [p - 2, p - 1]]))
    harness.run_parity(w, 40, every=20, coords=coords, check_rings=coords is None)
    g = one_pass(w)
    g.init(None, None)
    rng = np.random.default_rng(3)
    R, C = w.R, w.C
    import torch
    up = lambda a: torch.as_tensor(a).cuda()  # noqa: E731
    g.run(6, up(np.ones((6, n), np.uint8)), up(rng.integers(0, 4, (6, R.nnz_off), np.int32)), up(rng.integers(0, 4, (6, C.nnz_off), np.int32)),
          up(np.zeros((6, R.nnz_off), np.uint8)), up(np.zeros((6, C.nnz_off), np.uint8)), 0.002, None)
    ring = np.asarray(g.read("V_RING")).reshape(n, -1, p)
    off = r - np.diag(np.diag(r))
    leaves = (off != 0).sum(axis=0) == 0
    assert 0 < leaves.sum() < n
    assert not ring[leaves].any() and all(ring[i].any() for i in np.flatnonzero(~leaves))


def _raw_v_ring(g):
    """The rings of versions as they lie in the workspace (a read of the field returns zeros for what nobody can pick up): behind
    x, z and the two arrays of samples, each on a 256-byte boundary."""
    import torch
    up = lambda b: -(-b // 256) * 256  # noqa: E731
    row = g.n * g.p * 4
    off = 2 * up(row) + up(2 * row)
    return g.workspace[off:off + g.M * row].view(torch.float32).view(g.n, g.M, g.p)


# Which rows stream past the caches: 16 MB per array in calls of fewer than eight rounds, 32 MB (softmax: 24) in longer ones
@pytest.mark.parametrize("kind,n,p,rounds,kept", [
    ("diag_quadratic", 9, 500_000, 6, False), ("diag_quadratic", 9, 500_001, 6, False), ("diag_quadratic", 9, 900_000, 9, False),
    ("diag_quadratic", 9, 900_001, 9, False), ("diag_quadratic", 9, 500_000, 9, True), ("diag_quadratic", 9, 64_000, 6, True),
    ("softmax_bf16", 48, 131_072, 9, False), ("softmax_bf16", 36, 131_072, 3, False)])
def test_rows_nobody_pulls_are_not_written(kind, n, p, rounds, kept):
    """Where the state streams past the caches, the rows of nodes without out-edges over R keep what was there before; x, z and
    everything else are those of a context whose rows held something else, and the oracle's."""
    if kind == "softmax_bf16":
        r, c = graphs.binary_tree(n)
        w = configs._mk("tree_softmax", n, p, r, c, 2, 0.05, 0, kind, problems.softmax_pool(n, 1024, 128, 128, 5), 0.7, 0.1, 5,
                        batch=64, samples=128, burst=2, tol=2e-3, extra={"d": 1024, "K": 128})
    else:
        r, c = graphs.tree_pull_star_push(n)
        w = configs._mk("tree_star", n, p, r, c, 3, 0.002, 0, kind, problems.diag_quadratic(n, p, 5), 0.7, 0.2, 5, noise_std=0.1, burst=3)
    leaves = ((r != 0) & ~np.eye(n, dtype=bool)).sum(axis=0) == 0
    assert 0 < leaves.sum() < n
    pair = [harness.make_gpu(w), harness.make_gpu(w)]
    st, dev = harness.upload_chunk(pair[0], w, 0, rounds)
    for g, mark in zip(pair, (7.5, -3.25)):
        rfast_use_blocks(g.ctx, False)
        g.init(None, w.sched.initial_batch())
        ring = _raw_v_ring(g)
        assert not ring.any()
        for i in np.flatnonzero(leaves):
            ring[i] = mark
        g.run(rounds, *(dev[k] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")), w.gamma, dev["batch_idx"])
        g.check()
        moved = g.read("T_NODE") > 0
        for i in range(n):
            if leaves[i] and moved[i]:
                assert bool((ring[i][:, :p // 4 * 4] == mark).all()) != kept, i   # (the end of a ragged row is written)
            elif moved[i]:
                assert bool(ring[i].any())
        assert not g.read("V_RING")[leaves].any()
    for f in ("X", "Z", "SIGMA_RING", "TAU_R", "TAU_C"):
        assert np.array_equal(pair[0].read(f), pair[1].read(f)), f
    coords = None if kind == "softmax_bf16" else np.unique(np.concatenate([np.arange(0, p, 4099), [p - 2, p - 1]]))
    orc = harness.make_oracle(w, coords)
    for q in range(rounds):
        orc.round(*(st[k][q] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")), w.gamma,
                  None if st["batch_idx"] is None else st["batch_idx"][q])
    sel = slice(None) if coords is None else coords
    assert harness.rel_l2(pair[0].read("X")[:, sel], orc.x) <= w.tol
    assert harness.rel_l2(pair[0].read("Z")[:, sel], orc.z, 1e-3 * float(np.linalg.norm(orc.g))) <= w.tol


# 33, 42 and 43 tiles of 1024 coordinates per node, rounded up to a multiple of eight where rows have several readers or few nodes
# take a single pass; the last tile of the ragged row must be taken once
@pytest.mark.parametrize("kind,graph,n,p", [
    ("diag_quadratic", "mesh", 8, 33_001), ("diag_quadratic", "mesh", 8, 43_008), ("diag_quadratic", "mesh", 8, 43_009),
    ("diag_quadratic", "binary_tree", 20, 33_003), ("softmax_bf16", "exponential", 6, 43_008), ("softmax_bf16", "binary_tree", 6, 43_008)])
def test_tiles_rounded_up(kind, graph, n, p, monkeypatch):
    r, c = getattr(graphs, graph)(n)
    if kind == "softmax_bf16":
        w = configs._mk("tiles_softmax", n, p, r, c, 2, 0.05, 0, kind, problems.softmax_pool(n, 448, 96, 128, 5), 0.7, 0.1, 5, batch=64,
                        samples=128, burst=2, tol=2e-3, extra={"d": 448, "K": 96})
    else:
        w = configs._mk("tiles", n, p, r, c, 2, 0.02, 0, kind, problems.diag_quadratic(n, p, 5), 0.7, 0.2, 5, noise_std=0.1, burst=3)
    make = harness.make_gpu

    def one_pass(w):
        g = make(w)
        rfast_use_blocks(g.ctx, False)
        return g
    monkeypatch.setattr(harness, "make_gpu", one_pass)
    harness.run_parity(w, 20, every=(1, 3, 16))
