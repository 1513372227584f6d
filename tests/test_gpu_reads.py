"""Reading a field back: sizes at the edges of the staging buffers and of the pieces that threads share (64 KB, 1 MB, 2 MB, 16 MB
and several rounds of it), into fresh memory and into memory that starts anywhere."""
import numpy as np
import pytest

from paper_2307_11617_amd import rfast_read_state
from rfast_workloads import configs, graphs, problems

import harness

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,p", [(2, 8_192), (2, 8_193), (3, 87_381), (3, 87_382), (2, 262_144), (2, 262_145), (5, 262_143), (4, 1_048_576), (9, 1_048_577), (3, 6_000_001)])
@pytest.mark.parametrize("offset", [0, 1, 1023])
def test_read(n, p, offset):
    wr, wc = graphs.directed_ring(n)
    w = configs._mk("reads", n, p, wr, wc, 0, 0.01, 0, "diag_quadratic", problems.diag_quadratic(n, 4, 1), 1.0, 0.0, 1, burst=1)
    w.data = {k: np.ones((n, p), np.float32) for k in w.data}
    g = harness.make_gpu(w)
    x0 = np.arange(n * p, dtype=np.float32).reshape(n, p)
    g.init(x0, None)
    out = np.empty(n * p + offset + 16, np.float32)
    out[offset + n * p:] = -7.0
    out[:offset] = -7.0
    for _ in range(2):   # memory that has never been written, and the same again
        got = rfast_read_state(g.ctx, "X", out[offset:offset + n * p].reshape(n, p))
        assert np.array_equal(got, x0)
        assert (out[:offset] == -7.0).all() and (out[offset + n * p:] == -7.0).all()
    for _ in range(20 if n * p < 4_000_000 else 3):   # new memory each time: its page faults are taken beside the copies
        assert np.array_equal(g.read("X"), x0)
