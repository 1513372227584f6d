// What the team kernels share (rfast_team.hip: least squares and logistic regression; rfast_team_softmax.hip): accesses
// that meet behind the L2 caches of the accelerator dies, progress words, packets, bounded waits.
#pragma once
#include "rfast_vec.h"

namespace {

constexpr int kTeamThreads = 512;
constexpr int kFlagWords = 16;             // 32-bit words per progress entry (64 bytes): [0] v, [1] sums
constexpr int kSpin = 1 << 24;             // polls before a wait gives up (some ten seconds)
constexpr size_t kTeamLds = 156 * 1024;

typedef unsigned long long u64;

__device__ inline void put32(unsigned* p, unsigned v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline unsigned get32(const unsigned* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void put64(u64* p, u64 v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline u64 get64(const u64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void put_f(float* p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline float get_f(const float* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Everything this wavefront has loaded or stored so far is done, and nothing below is moved above it.
__device__ inline void drain() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);
  asm volatile("" ::: "memory");
}

__device__ inline int lane_value(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline float lane_value(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }

struct TeamArgs {
  int rounds, W, C, B, buffers;  // buffers: tiles of rows in LDS (two: the next round's rows arrive during this one)
  float gamma;
  unsigned base;              // progress words and packet tags count rounds from here on (they never repeat)
  const int32_t* batch_idx;   // [rounds][n][B], NULL: all rows, in order
  const int32_t* delay_R;     // [rounds][eR] (not the synchronous steps)
  const int32_t* delay_C;     // [rounds][eC]
  u64* packets;
  unsigned* flags;            // [n][owning wavefronts of a node][kFlagWords]
};

// first set bit at or after `from` of a mask of kBlockRounds bits, kBlockRounds if there is none
__device__ inline int next_bit(const u64* mask, int from) {
  int w = from >> 6;
  if (w >= kBlockRounds / 64) return kBlockRounds;
  u64 m = mask[w] & (~0ull << (from & 63));
  while (m == 0) {
    if (++w == kBlockRounds / 64) return kBlockRounds;
    m = mask[w];
  }
  return w * 64 + __ffsll((long long)m) - 1;
}

// Number of the first round of the launch, from the counter on the device (the resolver has moved it past the launch's
// rounds, a synchronous launch moves it behind them): the host's own count does not see the replays of a captured round.
__device__ inline int first_round(const RfastDev& s, const TeamArgs& a, bool sync) { return *s.round_no - (sync ? 0 : a.rounds); }

// a wait of node i has run out
__device__ inline void report_wait(const RfastDev& s, int round0, int i) {
  if (atomicCAS(&s.err[0], 0, RFAST_EHIP) == 0) {
    s.err[1] = round0;
    s.err[2] = 4;
    s.err[3] = i;
  }
}

// A progress word read ahead of the wait for it (an absent one, or one that need not be waited for, reads as round 0).
__device__ inline unsigned peek(const TeamArgs& a, const unsigned* f, int need) { return f != nullptr && need > 0 ? get32(f) : a.base; }

// Waits until the progress words of the lanes that have one (f1, f2, or neither) are at least round `need` of the launch
// whose rounds count from `base`.  v1, v2: the words as read ahead (a.base: not read); where they say enough, the wait
// costs no trip through memory.  dead: an earlier wait has run out, and nothing waits any more.
__device__ inline void wait_progress(const RfastDev& s, const TeamArgs& a, int round0, int i, const unsigned* f1, int need1, const unsigned* f2,
                                     int need2, unsigned v1, unsigned v2, bool* dead) {
  if (need1 <= 0) f1 = nullptr;
  if (need2 <= 0) f2 = nullptr;
  if (!__any(f1 != nullptr || f2 != nullptr) || *dead) return;
  for (int spin = 0;; ++spin) {
    const bool ok = (!f1 || (int)(v1 - a.base) >= need1) && (!f2 || (int)(v2 - a.base) >= need2);
    if (__all(ok)) break;
    if (spin > kSpin) {
      *dead = true;
      report_wait(s, round0, i);
      break;
    }
    v1 = f1 ? get32(f1) : 0;
    v2 = f2 ? get32(f2) : 0;
  }
  // what the words stand for was stored before them; nothing below may be loaded before they were seen
  asm volatile("" ::: "memory");
}

// sampled row b of a round as the caller gave it, clamped into the node's samples and (report) recorded if outside
__device__ inline int team_row(const RfastDev& s, const TeamArgs& a, int round0, int i, int q, int b, bool report) {
  int row = a.batch_idx[((size_t)q * s.n + i) * a.B + b];
  if (row < 0 || row >= s.prob.samples) {
    if (report && atomicCAS(&s.err[0], 0, RFAST_ERANGE) == 0) {
      s.err[1] = round0 + q;
      s.err[2] = 2;
      s.err[3] = i;
    }
    row = row < 0 ? 0 : s.prob.samples - 1;
  }
  return row;
}

}  // namespace
