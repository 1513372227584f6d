"""Diagnostics where the vector is short (the split form: a workgroup per 64 coordinates) and the loss over rows taken
four at a time, at the edges of both, against the fp64 oracle."""
import numpy as np
import pytest
import torch

from rfast_workloads import configs, graphs, problems

import harness

pytestmark = pytest.mark.gpu


# n, p, samples (rows), objective; 2048 coordinates per node, and 65536, are the last lengths of the split form
@pytest.mark.parametrize("n,p,samples,objective", [
    (3, 1, 1, "least_squares"), (5, 3, 5, "logistic"), (17, 63, 15, "logistic"), (18, 65, 16, "least_squares"),
    (16, 257, 17, "logistic"), (40, 1023, 67, "least_squares"), (7, 2, 0, "diag_quadratic"), (33, 130, 0, "diag_quadratic"),
    (3, 6144, 0, "diag_quadratic"), (3, 6145, 6, "logistic"), (33, 65_536, 0, "diag_quadratic"), (33, 65_537, 0, "diag_quadratic")])
def test_against_the_oracle(n, p, samples, objective):
    r, c = graphs.directed_ring(n)
    if objective == "diag_quadratic":
        data = problems.diag_quadratic(n, p, 5)
    else:
        data = (problems.least_squares if objective == "least_squares" else problems.logistic)(n, p, samples, 5)
    w = configs._mk(f"diag_{n}_{p}", n, p, r, c, 3, 1e-3 / max(1, p // 1000), 0, objective, data, 0.6, 0.3, 5, samples=samples)
    x0 = np.random.default_rng(1).standard_normal((n, p)).astype(np.float32)
    gpu, orc = harness.make_gpu(w), harness.make_oracle(w, None, x0)
    gpu.init(x0, None)
    st, dev = harness.upload_chunk(gpu, w, 0, 7)
    names = ("active", "delay_R", "delay_C", "drop_R", "drop_C")
    gpu.run(7, *[dev[k] for k in names], w.gamma, None)
    for k in range(7):
        orc.round(*[st[name][k] for name in names], w.gamma)
    x_star = np.random.default_rng(2).standard_normal(p).astype(np.float32)
    ref = orc.diagnostics(x_star)
    got = gpu.diagnostics(torch.from_numpy(x_star).to(gpu.device))
    for k in ("consensus_sq", "z_sq", "gsum_sq", "xbar_gap_sq", "loss_at_xbar"):
        assert abs(got[k] - ref[k]) <= 1e-4 * abs(ref[k]) + 1e-12, (k, got[k], ref[k])
    assert got["conservation_sq"] <= 1e-9 * (got["gsum_sq"] + got["z_sq"])
