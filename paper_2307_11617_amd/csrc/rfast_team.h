// What the team kernels share (rfast_team.hip: least squares and logistic regression; rfast_team_softmax.hip): accesses
// that meet behind the L2 caches of the accelerator dies, progress words, packets, bounded waits.
#pragma once
#include "rfast_edge.h"
#include "rfast_vec.h"

namespace {

constexpr int kTeamThreads = 512;
constexpr int kFlagWords = 16;             // 32-bit words per progress entry (64 bytes): the first round of which this is not yet true:
                                           // [0] v is out, [1] the sums are, [2] others' sums are read, [3] others' v is (softmax: [0] and [3] in one)
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
  int rounds, W, C, B, buffers;  // buffers: tiles of rows in LDS (softmax; two: the next round's rows arrive during this one)
  float gamma;
  unsigned base;              // progress words and packet tags count rounds from here on (they never repeat)
  const int32_t* batch_idx;   // [rounds][n][B], NULL: all rows, in order
  const int32_t* delay_R;     // [rounds][eR] (not the synchronous steps)
  const int32_t* delay_C;     // [rounds][eC]
  u64* packets;
  u64* sync;                  // the packets of the synchronous steps
  unsigned* flags;            // [n][owning wavefronts of a node][kFlagWords]
  unsigned* gate;             // kGateWords words: workgroups of this launch that have started (kGone in one of them: the
                              // launch goes on with one workgroup); behind them the word by which one gets to decide that
  unsigned* gate_next;        // those of the next launch, cleared by this one
  // polls before a wait gives up: for the others to start (0: one more is expected than there is), for a word or packet
  int gate_polls, wait_polls;
  unsigned* told;             // pinned host memory: [0] a launch went on with one workgroup, [1] a wait has run out
};

// ---- Are all workgroups of the launch resident?  Nothing else of the device is waited for, but another process, or a
// stream that has been given a part of the compute units, can keep some of them out for as long as the others wait.  So
// nobody touches the state before all have reported; if they do not within about a second, one workgroup (the first to
// swap a word) marks a word on which reports are missing, by a compare-and-swap, so that nobody can find them complete
// any more; the others leave, now or as soon as they start, and it computes the rounds alone: slowly, but what the call
// asked for.  The host sees it in pinned memory and launches no team of this context again before the next rfast_init.
constexpr unsigned kGone = 0x80000000u;

// One lane of every workgroup, first thing.  Eight words, taken in turn: additions to one word follow each other, and
// those of 64 to 256 workgroups to a single one cost a launch 2 us, this way 0.1 to 0.5 (32 words: the same).
__device__ inline void team_arrive(const TeamArgs& a) {
  (void)__hip_atomic_fetch_add(a.gate + (blockIdx.x % kGateWords) * kFlagWords, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The first wavefront of every workgroup, before the first store that anybody else sees.  0: all are there; 1: leave;
// 2: this workgroup is on its own.
__device__ inline int team_complete(const TeamArgs& a, int lane) {
  if (blockIdx.x == 0 && lane <= kGateWords) put32(a.gate_next + lane * kFlagWords, 0);
  const bool mine = lane < kGateWords;
  unsigned* const word = a.gate + lane * kFlagWords;
  const unsigned want = (gridDim.x + kGateWords - 1 - lane) / kGateWords + (a.gate_polls == 0 && lane == 0 ? 1u : 0u);
  bool decide = false;
  for (int poll = 0;; ++poll) {
    const unsigned seen = mine ? get32(word) : 0u;
    if (__any(mine && (seen & kGone))) return 1;
    const unsigned long long missing = __ballot(mine && seen != want);
    if (missing == 0) return 0;
    if (poll == a.gate_polls) {  // one workgroup at most may decide
      unsigned was = 0;
      decide = __any(lane == kGateWords && __hip_atomic_compare_exchange_strong(word, &was, 1u, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    if (decide) {
      unsigned was = seen;
      const bool set = lane == __ffsll((long long)missing) - 1 &&
                       __hip_atomic_compare_exchange_strong(word, &was, seen | kGone, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (__any(set)) {
        if (lane == 0) __hip_atomic_store(a.told, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        return 2;
      }
    }
  }
}

// The host's side of the start and of the bounds of a launch; polls take about a microsecond.
constexpr int kGatePolls = 1 << 20, kWaitPolls = 1 << 24;

inline void team_begin(rfast_ctx* c, TeamArgs* a) {
  a->gate = c->team_gate + (c->team_turn & 1) * kGateBytes / 4;
  a->gate_next = c->team_gate + (~c->team_turn & 1) * kGateBytes / 4;
  a->gate_polls = c->start_polls < 0 ? kGatePolls : c->start_polls;
  a->wait_polls = c->wait_polls < 0 ? kWaitPolls : c->wait_polls;
  a->told = c->team_told;
}
inline hipError_t team_end(rfast_ctx* c, int rounds, hipError_t launched) {
  if (launched != hipSuccess) return launched;
  c->team_base += (unsigned)rounds + 1;
  c->team_turn++;
  return hipSuccess;
}

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

// The arguments of the kernel as a copy of their own in the constant memory they came in, out of the compiler's sight: what
// the rare paths read of them is then not kept in scalar registers through the whole kernel.  (Only a kernel has them:
// whoever asks is inlined.)
static_assert(alignof(RfastDev) == alignof(TeamArgs), "one behind the other");
struct TeamKernelArgs {
  RfastDev s;
  TeamArgs a;
};
__device__ __forceinline__ const TeamKernelArgs& team_kernel_args() {
  const TeamKernelArgs* p = (const TeamKernelArgs*)(const void*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *p;
}

// Number of the first round of the launch, from the counter on the device (the resolver has moved it past the launch's
// rounds, a synchronous launch moves it behind them): the host's own count does not see the replays of a captured round.
__device__ inline int first_round(const RfastDev& s, const TeamArgs& a, bool sync) { return *s.round_no - (sync ? 0 : a.rounds); }

// a wait of node i has run out
__device__ __forceinline__ void report_wait(bool sync, int i) {
  const TeamKernelArgs& k = team_kernel_args();
  if (atomicExch(&k.s.err[0], RFAST_EHIP) != RFAST_EHIP) {  // whatever has been clamped before, this is worse
    k.s.err[1] = first_round(k.s, k.a, sync);
    k.s.err[2] = 4;
    k.s.err[3] = i;
  }
  __hip_atomic_store(k.a.told + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// A progress word read ahead of the wait for it (an absent one, or one that need not be waited for, reads as round 0).
__device__ inline unsigned peek(const TeamArgs& a, const unsigned* f, int need) { return f != nullptr && need > 0 ? get32(f) : a.base; }

// Waits until the progress words of the lanes that have one (f1, f2, or neither) are at least round `need` of the launch
// whose rounds count from `base`.  v1, v2: the words as read ahead (a.base: not read); where they say enough, the wait
// costs no trip through memory.  dead: an earlier wait has run out, and nothing waits any more.
__device__ __forceinline__ void wait_progress(const TeamArgs& a, bool sync, int i, const unsigned* f1, int need1, const unsigned* f2,
                                     int need2, unsigned v1, unsigned v2, bool* dead) {
  if (need1 <= 0) f1 = nullptr;
  if (need2 <= 0) f2 = nullptr;
  if (!__any(f1 != nullptr || f2 != nullptr) || *dead) return;
  for (int spin = 0;; ++spin) {
    const bool ok = (!f1 || (int)(v1 - a.base) >= need1) && (!f2 || (int)(v2 - a.base) >= need2);
    if (__all(ok)) break;
    if (spin >= a.wait_polls) {
      *dead = true;
      report_wait(sync, i);
      break;
    }
    v1 = f1 ? get32(f1) : 0;
    v2 = f2 ? get32(f2) : 0;
  }
  // what the words stand for was stored before them; nothing below may be loaded before they were seen
  asm volatile("" ::: "memory");
}

// a sampled row of round q as the caller gave it, clamped into the node's samples and (report) recorded if outside
__device__ __forceinline__ int team_row(const RfastDev& s, const TeamArgs& a, bool sync, int i, int q, int row, bool report) {
  if (row < 0 || row >= s.prob.samples) {
    const TeamKernelArgs& k = team_kernel_args();
    if (report) record_error(k.s.err, RFAST_ERANGE, first_round(k.s, k.a, sync) + q, 2, i);
    row = row < 0 ? 0 : s.prob.samples - 1;
  }
  return row;
}

// ---- The steps of a round by one workgroup on its own.  Lane `tid` takes coordinates tid, tid + kTeamThreads, ... in
// each of them, so that only the gradient, where coordinates meet, needs barriers.  slots, plan: the parts of the round's
// record that belong to the edges of R and of C.
__device__ inline void alone_mix(const RfastDev& s, int i, int slot_new, float gamma, const int32_t* slots) {
  const int64_t p = s.p;
  for (int64_t k = threadIdx.x; k < p; k += kTeamThreads) {
    const size_t at = (size_t)i * p + k;
    float dir = s.z[at];
    if (s.mom) s.mom[at] = dir = fmaf(s.beta, s.mom[at], dir);
    const float v = fmaf(-gamma, dir, s.x[at]);
    float x = s.r_self[i] * v;
    for (int e = s.r_ptr[i]; e < s.r_ptr[i + 1]; ++e)
      x = fmaf(s.r_w[e], s.v_ring[((size_t)s.r_src[e] * s.M + slots[e]) * p + k], x);
    s.v_ring[((size_t)i * s.M + slot_new) * p + k] = v;
    s.x[at] = x;
  }
}

template <class Gradient>
__device__ inline void alone_track(const RfastDev& s, int i, int t_old, const int32_t* plan, Gradient gradient) {
  const int64_t p = s.p;
  const bool pushes = s.co_ptr[i + 1] > s.co_ptr[i];
  float* sigma = s.sigma_ring + (size_t)i * s.M * p;
  for (int64_t k = threadIdx.x; k < p; k += kTeamThreads) {
    const size_t at = (size_t)i * p + k, half = (size_t)s.n * p;
    float z = s.z[at];
    for (int e = s.c_ptr[i]; e < s.c_ptr[i + 1]; ++e) {
      const int pl = plan[e], prev = (pl >> 8) & 0xFF;
      if (!(pl & (1 << 16))) continue;
      const float* ring = s.sigma_ring + (size_t)s.c_src[e] * s.M * p + k;
      float* saved = s.rho_tilde + (size_t)e * p + k;
      const float cur = ring[(size_t)(pl & 0xFF) * p], last = prev != 0xFF ? ring[(size_t)prev * p] : *saved;
      z = track_edge(z, s.c_w[e], cur, last, prev != 0xFF);
      if (pl & (1 << 17)) *saved = s.c_w[e] * cur;
    }
    const float g = gradient(k), zh = (z + g) - s.g[(t_old & 1) * half + at];
    s.g[((t_old + 1) & 1) * half + at] = g;
    s.z[at] = s.c_self[i] * zh;
    if (pushes) sigma[(size_t)((t_old + 1) % s.M) * p + k] = sigma[(size_t)(t_old % s.M) * p + k] + zh;
  }
}

// S4 for buffers whose version leaves the sender's ring without being consumed
__device__ inline void alone_save(const RfastDev& s, int i, const int32_t* plan) {
  for (int e = s.c_ptr[i]; e < s.c_ptr[i + 1]; ++e)
    if (plan[e] & (1 << 18))
      for (int64_t k = threadIdx.x; k < s.p; k += kTeamThreads)
        s.rho_tilde[(size_t)e * s.p + k] = s.c_w[e] * s.sigma_ring[((size_t)s.c_src[e] * s.M + (plan[e] & 0xFF)) * s.p + k];
}

}  // namespace
