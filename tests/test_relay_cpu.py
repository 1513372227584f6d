"""The threads that move a large read on to the caller's memory (csrc/rfast_relay.h), with plain memory in place of the device: what
arrives is the source, and a read that fails leaves alone what no piece has reached."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "rfast_relay.h"
// fail_ask, fail_wait: the piece that cannot be asked for, waited for (-1: none)
extern "C" int move(char* dst, const char* src, size_t bytes, size_t piece, size_t unit, int slots, int threads, long fail_ask, long fail_wait) {
  std::vector<char> stage((size_t)slots * piece);
  Relay r;
  r.dst = dst; r.stage = stage.data(); r.bytes = bytes; r.piece = piece; r.unit = unit; r.slots = slots;
  long waited = 0;
  return relay(&r, threads,
               [&](size_t k, int q) {
                 if ((long)k == fail_ask) return false;
                 memcpy(stage.data() + (size_t)q * piece, src + k * piece, r.size(k));
                 return true;
               },
               [&](int) { return waited++ != fail_wait; });
}
"""


@pytest.fixture(scope="module")
def move(tmp_path_factory):
    at = tmp_path_factory.mktemp("relay")
    (at / "move.cpp").write_text(SOURCE)
    out = str(at / "libmove.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-pthread", "-I", os.path.join(ROOT, "paper_2307_11617_amd", "csrc"), str(at / "move.cpp"), "-o", out], check=True)
    f = C.CDLL(out).move
    f.argtypes = [C.c_void_p, C.c_void_p, C.c_size_t, C.c_size_t, C.c_size_t, C.c_int, C.c_int, C.c_long, C.c_long]
    return f


def _call(move, bytes_, piece, unit, slots, threads, offset=0, fail_ask=-1, fail_wait=-1):
    src = np.random.default_rng(bytes_ + threads).integers(1, 255, bytes_, dtype=np.uint8)
    room = np.full(bytes_ + offset + 64, 255, np.uint8)   # no byte of the source is 255 or 0
    dst = room[offset:offset + bytes_]
    ok = move(dst.ctypes.data, src.ctypes.data, bytes_, piece, unit, slots, threads, fail_ask, fail_wait)
    assert (room[:offset] == 255).all() and (room[offset + bytes_:] == 255).all()
    return ok, src, dst


KB = 1 << 10


@pytest.mark.parametrize("bytes_,piece,unit,slots", [(1, 4 * KB, 4 * KB, 2), (4 * KB, 4 * KB, 4 * KB, 2), (4 * KB + 1, 4 * KB, 4 * KB, 2), (1025 * KB + 3, 64 * KB, 32 * KB, 4),
                                                     (600_001, 128 * KB, 128 * KB, 3), (3 << 20, 256 * KB, 64 * KB, 16)])
@pytest.mark.parametrize("threads", [1, 2, 5, 8])
def test_moves_all_of_it(move, bytes_, piece, unit, slots, threads):
    for offset in (0, 7):
        ok, src, dst = _call(move, bytes_, piece, unit, slots, threads, offset)
        assert ok and np.array_equal(src, dst)


@pytest.mark.parametrize("threads", [1, 3, 8])
@pytest.mark.parametrize("what,piece_failed", [("fail_ask", 0), ("fail_ask", 3), ("fail_ask", 9), ("fail_wait", 0), ("fail_wait", 1), ("fail_wait", 11)])
def test_a_read_that_fails_changes_nothing_that_no_piece_has_reached(move, threads, what, piece_failed):
    piece, slots = 64 * KB, 4
    for _ in range(5):
        ok, src, dst = _call(move, 12 * piece - 100, piece, 32 * KB, slots, threads, 0, **{what: piece_failed})
        # a piece is asked for when the one before it in its slot is through; pieces are waited for in turn
        reached = piece_failed if what == "fail_wait" else max(0, piece_failed - slots + 1)
        assert not ok
        assert np.array_equal(dst[:reached * piece], src[:reached * piece])
        assert (dst[reached * piece:] == 255).all()
