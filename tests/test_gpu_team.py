"""Least squares and logistic regression with a team of workgroups per node (several rounds per launch): the same bits
as one chain of kernels per round, at the edges of its chunks, tiles and batches, in every way rounds are asked for."""
import ctypes
import threading
import time

import numpy as np
import pytest
import torch

from paper_2307_11617_amd import RFastError, rfast_set_rebase_interval, rfast_set_wait_limits, rfast_use_blocks
from rfast_workloads import configs, graphs, problems

import harness

pytestmark = pytest.mark.gpu
FIELDS = ("X", "Z", "G", "V_RING", "SIGMA_RING", "RHO_TILDE", "T_NODE", "TAU_R", "TAU_C", "SLOT_R", "SLOT_C", "ROUND",
          "DELIV_R", "DELIV_C", "T_HIST")

# graph, n, p, samples, batch (0: all), objective, momentum
CASES = {
    "chunk_of_one_row_piece": ("exponential", 16, 1001, 96, 0, "least_squares", 0.0),
    "several_chunks_ragged": ("exponential", 32, 4099, 64, 22, "logistic", 0.0),
    "several_chunks_aligned": ("exponential", 32, 4096, 96, 64, "logistic", 0.9),
    "two_tiles_in_turn": ("binary_tree", 31, 784, 80, 32, "logistic", 0.0),
    "rows_from_memory": ("directed_ring", 40, 1030, 310, 300, "logistic", 0.0),
    "rows_from_memory_full_batch": ("mesh", 9, 2050, 261, 0, "least_squares", 0.0),
    "eight_coordinates_per_lane": ("directed_ring", 130, 1795, 40, 7, "least_squares", 0.9),
    "many_in_edges": ("tree_star", 40, 300, 30, 5, "logistic", 0.0),
    "fewer_coordinates_than_a_quad_pair": ("bidirectional_ring", 50, 7, 20, 3, "least_squares", 0.0),
}
BUILD = {"exponential": graphs.exponential, "binary_tree": graphs.binary_tree, "directed_ring": graphs.directed_ring,
         "mesh": graphs.mesh, "tree_star": graphs.tree_pull_star_push, "bidirectional_ring": graphs.bidirectional_ring}


def _workload(case):
    graph, n, p, samples, batch, objective, _ = CASES[case]
    r, c = BUILD[graph](n)
    data = problems.least_squares(n, p, samples, 5) if objective == "least_squares" else problems.logistic(n, p, samples, 5)
    gamma = (0.5 / p if objective == "least_squares" else 0.02) * (1.0 if graph in ("exponential", "mesh", "bidirectional_ring") else 0.1)
    return configs._mk(case, n, p, r, c, 3, gamma, 0, objective, data, 0.6, 0.3, 5, batch=batch, samples=samples, burst=3)


def _pair(case):
    w = _workload(case)
    a, b = harness.make_gpu(w), harness.make_gpu(w)
    rfast_use_blocks(a.ctx, 2)  # stretches of any length
    rfast_use_blocks(b.ctx, False)
    x0 = (0.1 * np.random.default_rng(3).standard_normal((w.n, w.p))).astype(np.float32)
    for g in (a, b):
        rfast_set_rebase_interval(g.ctx, 31)
        if CASES[case][6]:
            g.set_optimizer(CASES[case][6], 0.01)
        g.set_gamma_schedule(20, 0.8)
        g.init(x0, w.sched.initial_batch())
    return w, a, b, x0


def _same(a, b, where, fields=FIELDS):
    for f in fields:
        assert np.array_equal(a.read(f), b.read(f)), (where, f)


@pytest.mark.parametrize("case", list(CASES))
def test_rounds(case):
    w, a, b, x0 = _pair(case)
    st, dev = harness.upload_chunk(a, w, 0, 50)
    names = ("active", "delay_R", "delay_C", "drop_R", "drop_C")
    for lo, hi in ((0, 27), (27, 28), (28, 50)):
        for g in (a, b):
            bi = None if dev["batch_idx"] is None else dev["batch_idx"][lo:hi].contiguous()
            if hi - lo == 1:
                g.round(*[dev[k][lo].contiguous() for k in names], w.gamma, None if bi is None else bi[0].contiguous())
            else:
                g.run(hi - lo, *[dev[k][lo:hi].contiguous() for k in names], w.gamma, bi)
            g.check()
        _same(a, b, (case, hi))
    p_act = torch.full((w.n,), 0.5, dtype=torch.float32)
    for g in (a, b):
        g.run_generated(33, 5, p_act.to(g.device), w.sched.d_max, 0.1, w.gamma)
        g.run_events(40, 6, None, w.sched.d_max, 0.2, w.gamma)
        g.check()
    _same(a, b, (case, "generated and events"))
    if CASES[case][6]:
        _same(a, b, case, ("MOMENTUM",))
    assert np.abs(a.read("X") - x0).max() > 1e-4 and np.isfinite(a.read("X")).all() and np.isfinite(a.read("Z")).all()


@pytest.mark.parametrize("case", ["chunk_of_one_row_piece", "several_chunks_ragged", "several_chunks_aligned", "rows_from_memory",
                                  "many_in_edges", "eight_coordinates_per_lane"])
def test_synchronous_steps(case):
    w, a, b, _ = _pair(case)
    st, dev = harness.upload_chunk(a, w, 0, 45)
    for lo, hi in ((0, 30), (30, 31), (31, 45)):
        for g in (a, b):
            g.sync_run(hi - lo, w.gamma, None if dev["batch_idx"] is None else dev["batch_idx"][lo:hi].contiguous())
            g.check()
        # (two of these lengths leave the counters at 0 and 1 modulo the five slots of a ring)
        _same(a, b, (case, hi), ("X", "Z", "G", "T_NODE", "ROUND", "SIGMA_RING", "RHO_RING", "RHO_TILDE"))
        assert np.array_equal(a.read("V_RING")[:, 0], b.read("V_RING")[:, 0]), (case, hi)
        da, db = a.diagnostics(), b.diagnostics()
        for k in da:
            assert abs(da[k] - db[k]) <= 1e-9 * (abs(db[k]) + db["gsum_sq"] + db["z_sq"]), (case, hi, k, da[k], db[k])


@pytest.mark.parametrize("graph,n,p,samples,batch", [
    # chunks that leave whole wavefronts, lanes of one and second coordinates of a lane over; eight batches of in-edges at one node,
    # whose senders read nothing of it and run ahead
    ("tree_star", 40, 300, 30, 0), ("tree_star", 64, 257, 16, 5), ("tree_star", 60, 5, 24, 0), ("tree_star", 31, 1283, 40, 8),
    ("directed_ring", 16, 1001, 96, 0), ("binary_tree", 20, 65, 20, 4)])
def test_synchronous_steps_of_chunks_that_leave_lanes_over(graph, n, p, samples, batch):
    """A wavefront waits for packets of the same wavefront of its senders only, whichever lanes have a coordinate: long stretches of steps, none of
    whose waits runs out, give the bits of one chain of kernels per step."""
    r, c = BUILD[graph](n)
    w = configs._mk("sync_lanes", n, p, r, c, 3, 0.05 / p, 0, "least_squares", problems.least_squares(n, p, samples, 5), 1.0, 0.0, 5, batch=batch,
                    samples=samples, burst=3)
    a, b = harness.make_gpu(w), harness.make_gpu(w)
    rfast_use_blocks(a.ctx, 2)
    rfast_use_blocks(b.ctx, False)
    x0 = (0.1 * np.random.default_rng(3).standard_normal((n, p))).astype(np.float32)
    for g in (a, b):
        g.init(x0, w.sched.initial_batch())
    st, dev = harness.upload_chunk(a, w, 0, 120)
    for lo, hi in ((0, 100), (100, 102), (102, 120)):
        for g in (a, b):
            g.sync_run(hi - lo, w.gamma, None if dev["batch_idx"] is None else dev["batch_idx"][lo:hi].contiguous())
            g.check()
        _same(a, b, hi, ("X", "Z", "G", "T_NODE", "ROUND"))
    assert np.abs(a.read("X") - x0).max() > 1e-5 and np.isfinite(a.read("Z")).all()


def test_two_streams():
    """Contexts on two streams whose launches overlap: the workgroups of a team wait for each other, so the library
    orders the launches of different streams."""
    w = _workload("several_chunks_ragged")
    st, dev = None, None
    gpus, streams = [], [torch.cuda.Stream(), torch.cuda.Stream()]
    for s in streams:
        with torch.cuda.stream(s):
            g = harness.make_gpu(w)
            g.init(None, w.sched.initial_batch())
            gpus.append(g)
    st, dev = harness.upload_chunk(gpus[0], w, 0, 40)
    torch.cuda.synchronize()
    for _ in range(3):
        for g in gpus:
            g.run(40, *[dev[k] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma, dev["batch_idx"])
    for g in gpus:
        g.check()
    _same(gpus[0], gpus[1], "streams")


def test_stream_of_every_thread():
    """hipStreamPerThread: the same handle in two threads names two streams, whose launches are ordered all the same."""
    w = _workload("several_chunks_ragged")
    st, dev = None, None
    ref = harness.make_gpu(w)
    ref.init(None, w.sched.initial_batch())
    st, dev = harness.upload_chunk(ref, w, 0, 40)
    sched = [dev[k] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")]
    torch.cuda.synchronize()
    for _ in range(5):
        ref.run(40, *sched, w.gamma, dev["batch_idx"])
    ref.check()
    got, gate = {}, threading.Barrier(2)

    def work(key):
        with torch.cuda.stream(torch.cuda.ExternalStream(2)):
            g = harness.make_gpu(w)
            g.init(None, w.sched.initial_batch())
            gate.wait()
            for _ in range(5):
                g.run(40, *sched, w.gamma, dev["batch_idx"])
            g.check()
            got[key] = {f: g.read(f) for f in ("X", "Z", "G", "T_NODE")}
            g.close()
    threads = [threading.Thread(target=work, args=(k,)) for k in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for key in (0, 1):
        for f, v in got[key].items():
            assert np.array_equal(v, ref.read(f)), (key, f)


@pytest.mark.parametrize("units", [128, 8])
def test_stream_with_a_part_of_the_compute_units(units):
    """A team is no larger than the part of the chip its stream may use: every launch finds room, on as few as one
    workgroup's place per node, and a graph with more nodes than that takes the kernels per round."""
    w = _workload("several_chunks_ragged")
    hip = ctypes.CDLL("libamdhip64.so")
    raw = ctypes.c_void_p()
    bits = (ctypes.c_uint32 * 8)(*[min(max(units - 32 * q, 0), 32) and (1 << min(units - 32 * q, 32)) - 1 for q in range(8)])
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(raw), 8, bits) == 0
    got = []
    for stream in (torch.cuda.ExternalStream(raw.value), torch.cuda.current_stream()):
        with torch.cuda.stream(stream):
            g = harness.make_gpu(w)
            # (the chunks of a row's sum go with the size of the team: none for the reference)
            rfast_use_blocks(g.ctx, 2 if not got else False)
            g.init(None, w.sched.initial_batch())
            st, dev = harness.upload_chunk(g, w, 0, 40)
            stream.synchronize()
            began = time.perf_counter()
            for _ in range(3):
                g.run(40, *[dev[k] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma, dev["batch_idx"])
            g.check()
            took = time.perf_counter() - began
            got.append(g)
            if len(got) == 1:
                assert took < 0.2, took   # nobody has waited for a workgroup that found no room
    _close(*got, units, 1e-5)


def test_last_stream_under_capture():
    """The stream of the last team launch is being captured by the program while a context on another stream launches:
    the library's ordering of the two must not reach into the capture."""
    w = _workload("several_chunks_ragged")
    gpus, streams = [], [torch.cuda.Stream(), torch.cuda.Stream()]
    for s in streams:
        with torch.cuda.stream(s):
            g = harness.make_gpu(w)
            g.init(None, w.sched.initial_batch())
            gpus.append(g)
    st, dev = harness.upload_chunk(gpus[0], w, 0, 40)
    buf = torch.zeros(64, device=gpus[0].device)
    torch.cuda.synchronize()
    sched = [dev[k] for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")]
    gpus[0].run(40, *sched, w.gamma, dev["batch_idx"])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=streams[0], capture_error_mode="relaxed"):
        buf.add_(1.0)
        gpus[1].run(40, *sched, w.gamma, dev["batch_idx"])
    for _ in range(3):
        graph.replay()
    torch.cuda.synchronize()
    assert (buf == 3.0).all()
    for g in gpus:
        g.check()
    _same(gpus[0], gpus[1], "captured")


# graph, n, d, K, samples, batch, momentum: feature tiles per chunk, ragged last chunk, class counts, rows per workgroup
SOFTMAX = {
    "one_tile_chunks": ("exponential", 12, 512, 32, 256, 64, 0.9),
    "ragged_last_chunk": ("mesh", 30, 320, 96, 200, 128, 0.0),
    "two_chunks_all_classes": ("directed_ring", 90, 128, 128, 130, 64, 0.0),
    "many_rows": ("binary_tree", 7, 192, 64, 300, 256, 0.0),
    "eight_feature_tiles": ("bidirectional_ring", 128, 448, 32, 100, 64, 0.9),
    "many_in_edges": ("tree_star", 20, 64, 96, 80, 64, 0.0),
    # all rows in every round: they stay in LDS, with and without room for a second copy
    "all_rows": ("exponential", 12, 128, 32, 64, 0, 0.0),
    "all_rows_several_tiles": ("binary_tree", 6, 256, 64, 128, 0, 0.9),
}


def _softmax_workload(case):
    graph, n, d, K, samples, batch, momentum = SOFTMAX[case]
    r, c = BUILD[graph](n)
    gamma = 0.05 if graph in ("exponential", "mesh", "bidirectional_ring") else 0.002
    return configs._mk(case, n, d * K, r, c, 3, gamma, 0, "softmax_bf16", problems.softmax_pool(n, d, K, samples, 4), 0.6, 0.3, 6,
                       batch=batch, samples=samples, burst=3, tol=2e-3, extra={"d": d, "K": K})


def _softmax(case):
    momentum = SOFTMAX[case][-1]
    w = _softmax_workload(case)
    a, b = harness.make_gpu(w), harness.make_gpu(w)
    rfast_use_blocks(a.ctx, 2)  # stretches of any length
    rfast_use_blocks(b.ctx, False)
    x0 = (0.05 * np.random.default_rng(3).standard_normal((w.n, w.p))).astype(np.float32)
    for g in (a, b):
        rfast_set_rebase_interval(g.ctx, 17)
        if momentum:
            g.set_optimizer(momentum, 0.01)
        g.init(x0, w.sched.initial_batch())
    return w, a, b


def _close(a, b, where, tol=2e-3, fields=("X", "Z", "G")):
    for f in ("T_NODE", "TAU_R", "TAU_C", "ROUND"):
        assert np.array_equal(a.read(f), b.read(f)), (where, f)
    for f in fields:
        x, y = a.read(f), b.read(f)
        assert np.isfinite(x).all() and np.linalg.norm(x - y) <= tol * np.linalg.norm(y), (where, f, np.linalg.norm(x - y) / np.linalg.norm(y))


def _tight(a, b, where):
    """State, rings and buffers at the rounding of a sum: logits that differ in their last bits (2^-24) tip the bf16
    rounding (2^-8) of one in some 10^4 entries of E, sqrt(1e-4) * 2^-8 = 4e-5 of a gradient and what is tracked of it at
    most (1.2e-5 is the most measured over the cases); x and v move by gamma times that, with hundredths of z in them
    (4.7e-8).  Running sums right after a rebase are small differences: theirs is taken against the gradients."""
    for f in ("T_NODE", "TAU_R", "TAU_C", "ROUND"):
        assert np.array_equal(a.read(f), b.read(f)), (where, f)
    scale = np.linalg.norm(b.read("G"))
    for f, tol, floor in (("X", 2e-7, 0.0), ("V_RING", 2e-7, 0.0), ("Z", 5e-5, 0.0), ("G", 5e-5, 0.0), ("SIGMA_RING", 5e-5, scale),
                          ("RHO_TILDE", 5e-5, scale)):
        x, y = a.read(f).astype(np.float64), b.read(f).astype(np.float64)
        err, ref = np.linalg.norm(x - y), max(np.linalg.norm(y), floor)
        assert np.isfinite(x).all() and err <= tol * ref, (where, f, err / ref)


@pytest.mark.parametrize("case", list(SOFTMAX))
def test_softmax_rounds(case):
    """The partial logits of a chunk are rounded to fp32 before they are added, so the two forms agree to the rounding of
    a sum (and the bf16 roundings it tips), not bit for bit."""
    w, a, b = _softmax(case)
    st, dev = harness.upload_chunk(a, w, 0, 30)
    for lo, hi in ((0, 20), (20, 21), (21, 30)):
        for g in (a, b):
            g.run(hi - lo, *[dev[k][lo:hi].contiguous() for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma,
                  dev["batch_idx"][lo:hi].contiguous() if dev["batch_idx"] is not None else None)
            g.check()
        _tight(a, b, (case, hi))
    p_act = torch.full((w.n,), 0.5, dtype=torch.float32)
    for g in (a, b):
        g.run_generated(15, 5, p_act.to(g.device), w.sched.d_max, 0.1, w.gamma)
        g.run_events(20, 6, None, w.sched.d_max, 0.2, w.gamma)
        g.check()
    _tight(a, b, (case, "generated and events"))


@pytest.mark.parametrize("softmax,case", [(False, list(CASES)[0]), (True, list(SOFTMAX)[0]), (True, "all_rows")])
def test_forms_alternate(softmax, case):
    """Stretches by the team, single rounds by the kernels per round and what the library chooses, in turn on one context."""
    w, a, b = _softmax(case) if softmax else _pair(case)[:3]
    st, dev = harness.upload_chunk(a, w, 0, 30)
    for lo, hi, blocks in ((0, 9, 2), (9, 10, 0), (10, 12, 2), (12, 15, 0), (15, 16, 2), (16, 17, 1), (17, 19, 1), (19, 30, 1)):
        rfast_use_blocks(a.ctx, blocks)
        for g in (a, b):
            batch = dev["batch_idx"]
            g.run(hi - lo, *[dev[k][lo:hi].contiguous() for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma,
                  None if batch is None else batch[lo:hi].contiguous())
            g.check()
        if softmax:
            _tight(a, b, (case, hi))
        else:
            _same(a, b, (case, hi))


@pytest.mark.parametrize("softmax,case", [(False, "two_tiles_in_turn"), (True, "one_tile_chunks")])
def test_stretch_after_replayed_captures(softmax, case):
    """Two rounds captured by the program and replayed three times, then a stretch in which half of the nodes sit still
    for more rounds than a ring holds: their buffers (S4) have to be saved by the count of rounds that ran, not of calls."""
    w = _softmax_workload(case) if softmax else _workload(case)
    names = ("active", "delay_R", "delay_C", "drop_R", "drop_C")
    x0 = (0.05 * np.random.default_rng(3).standard_normal((w.n, w.p))).astype(np.float32)
    gpus = []
    for blocks in (2, False):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            g = harness.make_gpu(w)
            rfast_use_blocks(g.ctx, blocks)
            rfast_set_rebase_interval(g.ctx, 0)
            g.init(x0, w.sched.initial_batch())
            st, dev = harness.upload_chunk(g, w, 0, 32)
            dev["active"][2:27] = torch.arange(w.n, device=g.device) % 2
            stream.synchronize()
            part = lambda lo, hi: [dev[k][lo:hi].contiguous() for k in names]  # noqa: E731
            rows = lambda lo, hi: dev["batch_idx"][lo:hi].contiguous()  # noqa: E731
            first = [(part(r, r + 1), rows(r, r + 1)) for r in (0, 1)]
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=stream, capture_error_mode="relaxed"):
                for sched, batch in first:
                    g.round(*sched, w.gamma, batch)
            for _ in range(3):
                graph.replay()
            g.run(30, *part(2, 32), w.gamma, rows(2, 32))
            stream.synchronize()
            g.check()
        assert int(g.read("ROUND")[0]) == 36
        gpus.append(g)
    if softmax:
        _tight(*gpus, case)
    else:
        _same(*gpus, case)


@pytest.mark.parametrize("softmax,case", [(False, c) for c in CASES] + [(True, c) for c in ("ragged_last_chunk", "one_tile_chunks", "all_rows")])
def test_one_workgroup_goes_on_alone(softmax, case):
    """The workgroups of a launch do not all find room (one more is expected than there is): one of them computes its
    rounds, later calls take the kernels per round, and rfast_init gives the team another chance."""
    w, a, b = _softmax(case) if softmax else _pair(case)[:3]
    st, dev = harness.upload_chunk(a, w, 0, 30)
    batch = dev["batch_idx"]
    same = (lambda where: _tight(a, b, where)) if softmax else (lambda where: _same(a, b, where))
    for limit in (0, -1):
        rfast_set_wait_limits(a.ctx, limit, -1)
        for lo, hi in ((0, 17), (17, 30)):
            for g in (a, b):
                g.run(hi - lo, *[dev[k][lo:hi].contiguous() for k in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma,
                      None if batch is None else batch[lo:hi].contiguous())
                g.check()
            same((case, limit, hi))
        for g in (a, b):
            g.init(None, w.sched.initial_batch())


@pytest.mark.parametrize("case", ["chunk_of_one_row_piece", "several_chunks_aligned", "eight_coordinates_per_lane"])
def test_one_workgroup_steps_alone(case):
    w, a, b, _ = _pair(case)
    st, dev = harness.upload_chunk(a, w, 0, 18)
    rfast_set_wait_limits(a.ctx, 0, -1)
    for lo, hi in ((0, 15), (15, 18)):
        for g in (a, b):
            g.sync_run(hi - lo, w.gamma, None if dev["batch_idx"] is None else dev["batch_idx"][lo:hi].contiguous())
            g.check()
        _same(a, b, (case, hi), ("X", "Z", "G", "T_NODE", "ROUND", "SIGMA_RING", "RHO_TILDE"))
        assert np.array_equal(a.read("V_RING")[:, 0], b.read("V_RING")[:, 0]), (case, hi)


@pytest.mark.parametrize("softmax,case", [(False, "several_chunks_ragged"), (True, "one_tile_chunks")])
def test_wait_that_runs_out_is_reported_everywhere(softmax, case):
    """Waits within the rounds give up at once: whatever would go on with the state or hand it out says so, whether or not
    a delay has been clamped before, until rfast_init."""
    w, a, b = _softmax(case) if softmax else _pair(case)[:3]
    st, dev = harness.upload_chunk(a, w, 0, 40)
    names = ("active", "delay_R", "delay_C", "drop_R", "drop_C")
    run = lambda g, lo, hi: g.run(hi - lo, *[dev[k][lo:hi].contiguous() for k in names], w.gamma, dev["batch_idx"][lo:hi].contiguous())  # noqa: E731
    dev["active"][0] = 1
    dev["delay_R"][0, 0] = 99
    run(a, 0, 5)
    with pytest.raises(RFastError, match="delay on R edge 0 out of range in round 0"):
        a.check()
    rfast_set_wait_limits(a.ctx, -1, 0)
    run(a, 5, 35)
    calls = [a.check, lambda: a.read("X"), lambda: run(a, 35, 40), lambda: a.run_events(3, 1, None, 1, 0.0, w.gamma),
             lambda: a.run_generated(3, 1, torch.full((w.n,), 0.5, device=a.device), 1, 0.0, w.gamma),
             lambda: a.sync_run(2, w.gamma, dev["batch_idx"][:2].contiguous()), a.diagnostics]
    for call in calls:
        with pytest.raises(RFastError, match="waited in vain") as err:
            call()
        assert err.value.code == -6
    rfast_set_wait_limits(a.ctx, -1, -1)
    dev["delay_R"][0, 0] = 0
    for g in (a, b):
        g.init(None, w.sched.initial_batch())
        run(g, 0, 20)
        g.check()
    (_tight if softmax else _same)(a, b, case)


def test_more_contexts_than_the_shared_page_holds():
    """The words by which the device tells the host about a team's launches: contexts beyond the 64 of the shared page,
    and contexts in places that were given back, see their own and nobody else's."""
    w = _workload("fewer_coordinates_than_a_quad_pair")
    gpus = [harness.make_gpu(w) for _ in range(67)]
    st, dev = harness.upload_chunk(gpus[0], w, 0, 20)
    for k, g in enumerate(gpus):
        g.init(None, w.sched.initial_batch())
        if k in (3, 65):
            rfast_set_wait_limits(g.ctx, -1, 0)
        g.run(20, *[dev[f] for f in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma, dev["batch_idx"])
    for k, g in enumerate(gpus):
        if k in (3, 65):
            with pytest.raises(RFastError, match="waited in vain"):
                g.read("X")
        else:
            g.check()
            assert np.array_equal(g.read("X"), gpus[0].read("X")), k
    for k in (3, 66, 65, 10):
        gpus[k].close()
    for _ in range(3):
        g = harness.make_gpu(w)
        g.init(None, w.sched.initial_batch())
        g.run(20, *[dev[f] for f in ("active", "delay_R", "delay_C", "drop_R", "drop_C")], w.gamma, dev["batch_idx"])
        g.check()
        assert np.array_equal(g.read("X"), gpus[0].read("X"))
        gpus.append(g)
