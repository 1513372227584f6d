// Large reads: what arrives in pinned memory piece by piece is moved on to pageable memory by several threads.  Host code that knows
// nothing of the device: whoever uses it says how a piece is asked for and how it is waited for.
#pragma once
#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstring>
#include <thread>
#include <vector>

constexpr int kRelaySlots = 16;  // most pieces under way
constexpr size_t kRelayStop = ~(size_t)0;

// The calling thread has pieces copied into the slots in turn, and all threads move each piece on together, a part each, so that
// little is left to move when the last one arrives.
struct Relay {
  char* dst;
  char* stage;                            // [slots][piece]
  size_t bytes, piece;
  size_t unit;                            // bytes touched at a time, a part of a piece
  int slots, threads = 1;
  std::vector<std::atomic<bool>> touched;    // [units]
  std::atomic<size_t> arrived{0};         // pieces that are in their slots (all ones: give up)
  std::atomic<int> done[kRelaySlots] = {};  // threads through with the piece in a slot, counted over all pieces
  size_t pieces() const { return (bytes + piece - 1) / piece; }
  size_t size(size_t k) const { return std::min(piece, bytes - k * piece); }
  // Takes the page faults of a destination that has never been written while the first pieces are on their way: in units of a
  // large page, as two threads that meet a new large page both clear one.  The byte that it exchanges for itself keeps its value, so
  // that a read that fails leaves alone what no piece has reached.  A unit is copied into only when it has been touched.
  void touch(int t) {
    for (size_t u = t; u * unit < bytes; u += threads) {
      for (size_t at = u * unit; at < std::min(bytes, (u + 1) * unit); at += 4096) {
        char same = 0;
        (void)__atomic_compare_exchange_n(dst + at, &same, (char)0, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED);
      }
      touched[u].store(true, std::memory_order_release);
    }
  }
  void part(size_t k, int t) {
    const size_t len = size(k), each = (len / threads + 4095) / 4096 * 4096, from = std::min(len, each * t);
    const size_t end = t == threads - 1 ? len : std::min(len, from + each);
    if (from >= end) {
      done[k % slots].fetch_add(1, std::memory_order_release);
      return;
    }
    for (size_t u = (k * piece + from) / unit; u * unit < k * piece + end; ++u)
      for (int spin = 0; !touched[u].load(std::memory_order_acquire); ++spin)
        if (spin > 64) std::this_thread::yield();
    memcpy(dst + k * piece + from, stage + (k % slots) * piece + from, end - from);
    done[k % slots].fetch_add(1, std::memory_order_release);
  }
};

inline void relay_worker(Relay* r, int t) {
  r->touch(t);
  for (size_t k = 0;; ++k) {
    size_t in;
    for (int spin = 0; (in = r->arrived.load(std::memory_order_acquire)) <= k; ++spin)
      if (spin > 64) std::this_thread::yield();
    if (in == kRelayStop) return;
    r->part(k, t);
    if (k + 1 == r->pieces()) return;
  }
}

// The part of the calling thread.  ask(k, slot): has piece k copied into the slot; wait(slot): until it is there.  Both return
// whether they could; if not, nothing more is asked for, and what is under way is the caller's to wait for.
template <class Ask, class Wait> bool relay_pieces(Relay* r, Ask ask, Wait wait) {
  const size_t pieces = r->pieces();
  bool ok = true;
  auto next = [&](size_t k) {
    if (ok && k < pieces) ok = ask(k, (int)(k % r->slots));
  };
  for (size_t k = 0; k < (size_t)r->slots; ++k) next(k);
  if (ok) r->touch(0);
  for (size_t k = 0; k < pieces && ok; ++k) {
    const size_t q = k % r->slots;
    ok = wait((int)q);
    if (!ok) break;
    r->arrived.store(k + 1, std::memory_order_release);
    r->part(k, 0);
    const int through = (int)(k / r->slots + 1) * r->threads;
    for (int spin = 0; r->done[q].load(std::memory_order_acquire) < through; ++spin)
      if (spin > 64) std::this_thread::yield();
    next(k + r->slots);
  }
  if (!ok) r->arrived.store(kRelayStop, std::memory_order_release);
  return ok;
}

// All of it, by `threads` threads (the calling one among them) or as many as there are to be had.  False: something could not be
// asked for or waited for.  Throws what the vector of units throws.
template <class Ask, class Wait> bool relay(Relay* r, int threads, Ask ask, Wait wait) {
  r->touched = std::vector<std::atomic<bool>>((r->bytes + r->unit - 1) / r->unit);
  std::vector<std::thread> pool;
  std::atomic<int> go{0};  // how many there are is known
  int started = 1;
  try {
    for (; started < threads; ++started)
      pool.emplace_back([&go, r, t = started] {
        for (int spin = 0; go.load(std::memory_order_acquire) == 0; ++spin)
          if (spin > 64) std::this_thread::yield();
        relay_worker(r, t);
      });
  } catch (...) {  // no more threads to be had: those there are do it
  }
  r->threads = started;
  go.store(1, std::memory_order_release);
  const bool ok = relay_pieces(r, ask, wait);
  for (std::thread& t : pool) t.join();
  return ok;
}
