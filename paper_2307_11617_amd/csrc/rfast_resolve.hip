// Integer schedule resolver: turns the masks of a stretch of rounds into ring-slot indices.
//
// For an active receiver i and in-edge e = (j -> i) the stamp picked up is the
// newest one that has arrived on the edge (Algorithm 1, S2a / S2b), i.e. the
// newest version of j that (a) j had published before round r - delay_e and
// (b) was not lost on e, and never older than the stamp already held.  Losses
// are decided when a version is sent (experiments section: a node either sends
// its new packet or discards it).  After burst-1 consecutive losses on an edge
// the next version is delivered regardless, which keeps every read within D
// versions of the sender's counter (Assumption 3 ii).
//
// The same lane decides where the buffer rho~ of step S4 lives for its C edge.  rho~_ij
// equals a_ij * sigma_j[tau_ij], which the sender's ring still holds while
// tau_ij >= t_j - D; only a version about to leave the ring is copied to the rho~ array
// (by the receiver if it consumes exactly that version in this round, else by the sender).
//
// An edge needs nothing of any other edge: its stamp and its delivery bits are its own, and the counter of its
// sender, now and at the start of earlier rounds, is a count of the sender's activity flags.  So one lane takes one
// edge through all rounds of the launch, with its stamp, the sender's counter, the sender's last 64 activity flags and
// the delivery bits in registers (the bits as a shift register, newest version first, so that no remainder by the ring
// length is left in the loop), and a round has no barrier and no LDS.  What bounds it is the dependent instructions of
// one wavefront per edge (0.35 us per round on small graphs), while the inputs of the next eight rounds are on their
// way.  Measured, us per launch of 25 to 32 rounds, against one workgroup in step with three barriers per round: 31
// nodes and 60 edges 51 -> 14, 32 nodes and 320 edges 61 -> 17, 128 nodes and 1792 edges 132 -> 19; a single round
// 6.1 -> 4.1.
#include "rfast_edge.h"
#include "rfast_internal.h"

namespace {

constexpr int kGroupLanes = 1024;  // nodes and edges (each rounded up to wavefronts) one workgroup looks after
constexpr int kChunk = 8;          // rounds whose inputs are fetched ahead together

typedef unsigned long long u64;

// The delivery bits as they are kept between launches, bit s for the version in ring slot s, against the bits the loop
// works with, bit k for version t - k, where t sits in slot st: s and k are each other's mirror, k = (st - s) mod M, so
// that one function goes both ways.
__device__ inline u64 mirror_bits(u64 bits, int st, int M) {
  const u64 rev = __brevll(bits);
  const u64 low = rev >> (63 - st);                                        // slots st .. 0 as k = 0 .. st
  const u64 high = st + 1 < M ? (rev >> (64 - M)) << (st + 1) : 0ull;      // slots M-1 .. st+1 as k = st+1 .. M-1
  return (low | high) & (M == 64 ? ~0ull : (1ull << M) - 1);
}

template <class P> __device__ inline P* shifted(P* ptr, size_t bytes) {
  return reinterpret_cast<P*>(reinterpret_cast<char*>(ptr) + bytes);
}

struct Sched {
  const uint8_t* active;
  const int32_t* delay_R;
  const int32_t* delay_C;
  const uint8_t* drop_R;
  const uint8_t* drop_C;
};

// Where a lane's edge starts from.
struct EdgeState {
  int i, j, old, tj, st;  // receiver, sender, stamp held, the sender's counter and the ring slot of that version (FORM 2: slot on chip)
  u64 dl, hist;           // delivery bits (bit k: version tj - k), activity of the sender (bit k: k+1 rounds ago)
};

template <int KIND>
__device__ inline void edge_begin(const RfastDev& s, int e, int r0, int rounds, const int32_t* delay, EdgeState* q) {
  q->i = (KIND ? s.c_dst : s.r_dst)[e];
  q->j = (KIND ? s.c_src : s.r_src)[e];
  const u64 bits = (KIND ? s.deliv_c : s.deliv_r)[e];
  q->old = (KIND ? s.tau_c : s.tau_r)[e];
  q->tj = s.t[q->j];
  q->st = FastMod(s.M)(q->tj);
  q->dl = mirror_bits(bits, q->st, s.M);
  // activity of the sender before this launch, from the counters at the start of the last H rounds (no delay is
  // longer); a launch of one round looks its one counter up instead, and the bits are any that give that count
  q->hist = 0;
  if (rounds == 1) {
    const int d0 = delay[0], d = d0 < 0 ? 0 : (d0 > s.d_max ? s.d_max : d0);
    if (d > 0) q->hist = (1ull << (q->tj - (d < r0 ? s.t_hist[(size_t)q->j * s.H + FastMod(s.H)(r0 - d)] : 0))) - 1;
  } else {
    const int32_t* h = s.t_hist + (size_t)q->j * s.H;
    int later = q->tj, at = FastMod(s.H)(r0);
    const int back = r0 < s.H - 1 ? r0 : s.H - 1;
    for (int k0 = 0; k0 < back; k0 += kChunk) {
      int t[kChunk];
#pragma unroll
      for (int u = 0; u < kChunk; ++u) {  // all of them before the first use (past the last: one that is not used)
        at = at == 0 ? s.H - 1 : at - 1;
        t[u] = h[at];
      }
#pragma unroll
      for (int u = 0; u < kChunk; ++u)
        if (k0 + u < back) {
          q->hist |= (u64)(later - t[u]) << (k0 + u);
          later = t[u];
        }
    }
  }
}

// What the resolver writes for a round: the per-round plan arrays, a record of ring slots, or a record for the
// wavefront-tile kernel (RfastDev::blk_slots).
enum { kPlans = 0, kRecords = 1, kOnChip = 2 };

// Decides the edge for round r: delay d0 and loss flag as the schedule has them.  Returns the slot read (-1: the
// receiver is idle; kOnChip: 0 otherwise) and the plan word.  *aside: the sender or the receiver saves the buffer (graph C); kOnChip: anything rare.
template <int KIND, int FORM>
__device__ inline int edge_round(const RfastDev& s, int e, int r, int d0, bool dropped, bool act_i, bool act_j, EdgeState& q, int* word, bool* aside) {
  const int M = s.M, tj = q.tj, lo = tj - (M - 2);  // oldest version that stays readable in j's ring during this round
  const int slots = FORM == kOnChip ? s.blk_slots : M;
  const int d = d0 < 0 ? 0 : (d0 > s.d_max ? s.d_max : d0);
  if (act_i && d != d0) record_edge_error(s, r, KIND, e);  // resolved with the clamped delay
  const int seen = tj - __popcll(q.hist & ((1ull << d) - 1));  // the sender's counter at the start of round r - d
  // S2a / S2b: the newest delivered version that is not newer than that: at most burst-1 steps back (a version is
  // delivered by force once the burst-1 before it were all lost; version 0 always counts as delivered)
  const u64 from = q.dl >> (tj - seen);
  int back = from ? __ffsll((long long)from) - 1 : 64;
  back = back < s.burst - 1 ? back : s.burst - 1;
  const int u = seen - back > 0 ? seen - back : 0;
  const int old = q.old;
  const int now = act_i && u > old ? u : old;
  const int sn = q.st - (tj - now), now_slot = sn < 0 ? sn + slots : sn;  // wherever it is used, now lies within the ring
  q.old = now;
  *aside = false;
  if (FORM == kOnChip) {
    const bool far = act_i && tj - now >= slots;               // the version is no longer on chip
    const bool gone = KIND && act_i && now != old && old < lo; // what was consumed last time has left the ring
    *word = act_i ? now_slot : 0;
    *aside = far || gone;
    if (*aside) {
      *word = (far ? 1 << 30 | FastMod(M)(now) << 24 : now_slot) | (gone ? (int)0x80000000 : 0);
      if (far) s.blk_far[(size_t)q.j * kFarWords + now % kFarWords] = now + 1;
    }
  } else if (KIND == 0) {
    *word = act_i ? now_slot : 0;
  } else {
    const bool live = now != old;                // never with an idle receiver
    const bool leaves = act_j && now == lo;      // after this round the ring of an active sender no longer covers version lo
    const bool spill = !live && leaves;          // the receiver does not consume, and the version its buffer holds leaves
    const bool held = old >= lo;                 // what was consumed last time is still in the ring
    const int so = q.st - (tj - old), old_slot = held ? (so < 0 ? so + M : so) : 0xFF;
    // bits 30 and 31 sort the live edges for a consumer that wants one compare per case: the usual one (what was
    // consumed last time is still in the ring, what is consumed now stays there) and the rest;
    // bits 0-7 of a spill word: the slot of the version that leaves (now == lo then)
    const bool usual = live && !leaves && held;
    const int on = now_slot | old_slot << 8 | (live ? 1 << 16 : 0) | (live && leaves ? 1 << 17 : 0) | (spill ? 1 << 18 : 0) |
                   (usual ? 1 << 30 : 0) | (live && !usual ? (int)0x80000000 : 0);
    *word = act_i ? on : (spill ? now_slot | 1 << 18 : 0);
    *aside = spill;
  }
  // the sender publishes version t_j + 1 this round (if it is active): lost only if the schedule says so and not all
  // of the burst-1 versions before it were lost too (versions up to 0 count as delivered)
  const bool all_lost = (q.dl & ((1ull << (s.burst - 1)) - 1)) == 0 && (s.burst == 1 || tj + 2 - s.burst > 0);
  if (act_j) {
    q.dl = (q.dl << 1) | ((!dropped || all_lost) ? 1u : 0u);
    q.tj = tj + 1;
    q.st = q.st + 1 == slots ? 0 : q.st + 1;
  }
  q.hist = (q.hist << 1) | (act_j ? 1u : 0u);
  return !act_i ? -1 : FORM == kOnChip ? 0 : now_slot;
}

// One edge through all rounds.  barrier: called once everything read from the state arrays is in registers.
// FORM: what is written per round; *rare (kOnChip) is set if an edge does anything rare.  The body of the loop is straight-line but for
// the rare spill, and loads nothing but the inputs of the next chunk: memory operations complete in order, so a load
// inside a round would wait for the stores of the rounds before it (0.5 us per round instead of 0.35).
template <int KIND, int FORM, class Barrier>
__device__ inline void edge_rounds(const RfastDev& s, int e, int r0, int rounds, size_t plan_stride, const Sched& sc, bool mine, int* rare,
                                   Barrier barrier) {
  constexpr bool RECORDS = FORM != kPlans;
  EdgeState q;
  const int32_t* delay = (KIND ? sc.delay_C : sc.delay_R) + e;
  if (mine) edge_begin<KIND>(s, e, r0, rounds, delay, &q);
  barrier();
  if (!mine) return;
  const int E = KIND ? s.eC : s.eR;
  const uint8_t* drop = (KIND ? sc.drop_C : sc.drop_R) + e;
  const int W1 = s.n + s.eR + s.eC + 1;
  const int lo0 = q.old, t0 = q.tj;
  if (FORM == kOnChip) q.st = FastMod(s.blk_slots)(t0);
  int d[kChunk];
  uint8_t x[kChunk], ai[kChunk], aj[kChunk];
  auto fetch = [&](int base) {  // (past the last round: the last one again, which is not used)
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const size_t rq = base + u < rounds ? base + u : rounds - 1;
      d[u] = delay[rq * E];
      x[u] = drop[rq * E];
      ai[u] = sc.active[rq * s.n + q.i];
      aj[u] = sc.active[rq * s.n + q.j];
    }
  };
  fetch(0);
  int32_t* rec = RECORDS ? s.blk_plan + s.n + (KIND ? s.eR : 0) + e : nullptr;
  int32_t* slot_out = (KIND ? s.slot_c : s.slot_r) + e;
  int32_t* plan_out = s.plan_c + e;
  int slot = -1, word = 0;
  for (int base = 0; base < rounds; base += kChunk) {
    int dn[kChunk];
    unsigned fl[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      dn[u] = d[u];
      fl[u] = (x[u] ? 1u : 0u) | (ai[u] ? 2u : 0u) | (aj[u] ? 4u : 0u);
    }
    fetch(base + kChunk);
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const int rq = base + u;
      if (rq >= rounds) break;
      bool spilled;
      slot = edge_round<KIND, FORM>(s, e, r0 + rq, dn[u], fl[u] & 1u, fl[u] & 2u, fl[u] & 4u, q, &word, &spilled);
      if (RECORDS) {
        *rec = word;
        rec += W1;
        if ((KIND || FORM == kOnChip) && spilled) {
          s.blk_spill[(size_t)rq * s.n + q.i] = r0 + rq + 1;
          if (FORM == kOnChip) *rare = 1;
        }
      } else {
        *slot_out = slot;
        slot_out = shifted(slot_out, plan_stride);
        if (KIND) {
          *plan_out = word;
          plan_out = shifted(plan_out, plan_stride);
          if (spilled) shifted(s.node_spill, (size_t)rq * plan_stride)[q.j] = q.tj;  // the counter the sender has after this round
        }
      }
    }
  }
  if (FORM == kOnChip) {  // back to slots of the ring in memory
    q.st = FastMod(s.M)(q.tj);
    if (slot >= 0) slot = FastMod(s.M)(q.old);
  }
  if (RECORDS) {  // of the per-round arrays only the last round's slots are looked at (reads of the slot fields)
    *slot_out = slot;
    if (KIND) *plan_out = word;
  }
  (KIND ? s.tau_c : s.tau_r)[e] = q.old;
  (KIND ? s.deliv_c : s.deliv_r)[e] = mirror_bits(q.dl, q.st, s.M);
  if (s.blk_head) {
    // oldest version held on an out-edge of j before and after the rounds; where the S4 buffer lives before and after
    int32_t* H = s.blk_head;
    atomicMin(&H[kHeadWords * q.j + (KIND ? 3 : 2)], lo0);
    atomicMin(&H[kHeadWords * q.j + (KIND ? 5 : 4)], q.old);
    if (KIND) {
      int w = (lo0 < t0 - (s.M - 2) ? 1 : 0) | (q.old < q.tj - (s.M - 2) ? 2 : 0);
      if (FORM == kOnChip) w |= (t0 - lo0 < s.blk_slots ? 4 : 0) | FastMod(s.M)(lo0) << 8 | FastMod(s.blk_slots)(lo0) << 16;
      H[kHeadWords * s.n + e] = w;
    }
  }
}

// The node side: counters, their history, the list of active nodes of every round (or the node words of its record).
// Lane = node; every wavefront counts the active nodes of the others by itself.  Returns the lane's counter at the end.
template <bool CHIP>
__device__ inline int node_rounds(const RfastDev& s, int node, int wave, int lane, int r0, int rounds, size_t plan_stride,
                                  const uint8_t* active, int t, int32_t* hist) {
  const int n = s.n, waves = (n + 63) / 64, W1 = n + s.eR + s.eC + 1;
  const bool mine = node < n;
  const FastMod modH(s.H);
  int at = modH(r0);
  uint8_t a[kChunk];
  auto fetch = [&](int base) {
#pragma unroll
    for (int u = 0; u < kChunk; ++u)  // (past the last round or node: some other flag, which is not used)
      a[u] = active[(size_t)(base + u < rounds ? base + u : rounds - 1) * n + (mine ? node : 0)];
  };
  fetch(0);
  for (int base = 0; base < rounds; base += kChunk) {
    uint8_t an[kChunk];
#pragma unroll
    for (int u = 0; u < kChunk; ++u) an[u] = mine && a[u] != 0;
    fetch(base + kChunk);
#pragma unroll
    for (int u = 0; u < kChunk; ++u) {
      const int rq = base + u;
      if (rq >= rounds) break;
      const bool on = an[u] != 0;
      if (s.blk_plan) {
        int32_t* rec = s.blk_plan + (size_t)rq * W1;
        if (mine) rec[node] = (t & (CHIP ? 0x1FFFFFFF : 0x3FFFFFFF)) | (on ? (CHIP ? (int)0xC0000000 : (int)0x80000000) : 0);
        if (node == 0) rec[W1 - 1] = 0;  // a record ends with a word that is always zero
      }
      if (!s.blk_plan || rq + 1 == rounds) {
        const size_t off_set = s.blk_plan ? 0 : (size_t)rq * plan_stride;
        const u64 mask = __ballot(on);
        int before = 0, total = __popcll(mask);
        for (int w = 0; w < waves; ++w)  // activity of the nodes of the other wavefronts
          if (w != wave) {
            const int m = w * 64 + lane;
            const int c = __popcll(__ballot(m < n && active[(size_t)rq * n + m] != 0));
            total += c;
            before += w < wave ? c : 0;
          }
        if (mine) shifted(s.plan_t, off_set)[node] = t;
        int2* list = shifted(s.active_plan, off_set);
        if (on) list[before + __popcll(mask & ((1ull << lane) - 1))] = make_int2(node, t);
        // what is left of the n + 8 work slots, shared out among the wavefronts
        for (int q = total + wave * 64 + lane; q < n + 8; q += waves * 64) list[q] = make_int2(-1, 0);
        if (node == 0) {
          int32_t* cnt = shifted(s.n_active, off_set);
          cnt[0] = total;
          cnt[1] = r0 + rq + 1;
        }
      }
      if (mine && rq + s.H >= rounds) hist[(size_t)node * s.H + at] = t;
      at = at + 1 == s.H ? 0 : at + 1;
      t += on ? 1 : 0;
    }
  }
  return t;
}

// What a launch of the wavefront-tile kernel finds about the nodes before its first and after its last round
// (RfastDev::blk_head), and, where anything rare happens, the marks in the node words.  By the whole workgroup.
__device__ inline void on_chip_heads(const RfastDev& s, int r0, int rounds, int* rare) {
  const int M = s.M, K = s.blk_slots;
  auto word = [&](int j, int w) { return __hip_atomic_load(&s.blk_head[kHeadWords * j + w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  // Versions that somebody holds after the launch and that are still in the ring of M then: from this one on
  auto kept = [&](int te, int lo_v, int lo_s) {
    const int lo = lo_v < lo_s ? lo_v : lo_s;
    return lo > te - (M - 1) ? lo : te - (M - 1);
  };
  for (int j = threadIdx.x; j < s.n; j += blockDim.x) {
    const int t0 = word(j, 0), te = word(j, 1), lo_v0 = word(j, 2), lo_s0 = word(j, 3), lo_v1 = word(j, 4), lo_s1 = word(j, 5);
    unsigned in_v = 0, in_s = 0, put_v = 0, put_s = 0, sums = 0;
    for (int a = 0; a < M && a < 32; ++a) {
      const unsigned bit = 1u << a;
      if (a < K && t0 - a >= lo_v0) in_v |= bit;
      if (a < K && t0 - a >= lo_s0) in_s |= bit;
      if (a < K && te - a > t0 && te - a >= lo_v1) put_v |= bit;
      if (a < K && te - a > t0 && te - a >= lo_s1) put_s |= bit;
      if (te - a >= lo_s1) sums |= bit;
    }
    int32_t* H = s.blk_head + kHeadWords * j;
    H[6] = (int)sums;
    H[8] = t0 % M;
    H[9] = t0 % K;
    H[10] = (int)in_v;
    H[11] = (int)in_s;
    H[12] = te % M;
    H[13] = te % K;
    H[14] = (int)put_v;
    H[15] = (int)put_s;
    const int first = kept(te, lo_v1, lo_s1);
    if (te - K >= (first > t0 ? first : t0 + 1)) *rare = 1;
  }
  __syncthreads();
  if (!*rare) return;
  const int W1 = s.n + s.eR + s.eC + 1, cells = rounds * s.n;
  constexpr int kAhead = 4;
  for (int c0 = threadIdx.x; c0 < cells; c0 += kAhead * blockDim.x) {
    int w[kAhead], mark[kAhead], j[kAhead];
    int32_t* at[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int c = c0 + u * (int)blockDim.x < cells ? c0 + u * (int)blockDim.x : c0, q = c / s.n;
      j[u] = c - q * s.n;
      at[u] = s.blk_plan + (size_t)q * W1 + j[u];
      w[u] = __hip_atomic_load(at[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      mark[u] = __hip_atomic_load(&s.blk_spill[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == r0 + q + 1;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (w[u] >= 0 || c0 + u * (int)blockDim.x >= cells) continue;
      const int t0 = word(j[u], 0), te = word(j[u], 1);
      const int t = t0 + (((w[u] & 0x1FFFFFFF) - t0) & 0x1FFFFFFF), leaves = t + 1 - K;  // the place of this version is taken
      const bool keep = leaves > t0 && (leaves >= kept(te, word(j[u], 4), word(j[u], 5)) ||
                                        __hip_atomic_load(&s.blk_far[(size_t)j[u] * kFarWords + leaves % kFarWords], __ATOMIC_RELAXED,
                                                          __HIP_MEMORY_SCOPE_AGENT) == leaves + 1);
      if (keep || mark[u]) *at[u] = (w[u] & ~(1 << 30)) | (keep ? 1 << 29 : 0);
    }
  }
}

// rounds > 1: consecutive rounds in one launch, the schedule arrays of round q at offset q of each
// pointer, its plan record (multi-round kernels) behind the previous one, or, without records, its per-round plan
// arrays plan_stride bytes behind those of the previous round.
// lanes_*: lanes (whole wavefronts) of the nodes, the edges of R and those of C, in this order.
// A graph whose lanes fit one workgroup has one barrier, between the last read of the state arrays and the first
// write to them.  Larger graphs take several workgroups, which leave the counters and the history in a second set of
// arrays; the last workgroup to finish copies them over (only there does anybody write what another workgroup reads).
// CHIP: records for the wavefront-tile kernel (a kernel of its own: the others are a hundredth faster without what it needs).
template <bool CHIP>
__global__ void __launch_bounds__(kGroupLanes) rfast_resolve_kernel(RfastDev s, int rounds, size_t plan_stride, Sched sc, int lanes_n,
                                                                    int lanes_R, int lanes_C) {
  const int r0 = *s.round_no;
  const bool single = gridDim.x == 1;
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63;
  __shared__ int rare;
  if (CHIP && threadIdx.x == 0) rare = 0;
  auto barrier = [&] {
    if (single) __syncthreads();
  };
  if (s.blk_head)  // (graphs of one workgroup only)
    for (int j = threadIdx.x; j < s.n; j += blockDim.x) {
      s.blk_head[kHeadWords * j + 2] = s.blk_head[kHeadWords * j + 3] = 0x7fffffff;
      s.blk_head[kHeadWords * j + 4] = s.blk_head[kHeadWords * j + 5] = 0x7fffffff;
    }
  // (the kind of a lane is the same throughout a wavefront)
  if (id < lanes_n) {
    const int t0 = id < s.n ? s.t[id] : 0;
    barrier();
    const int t = node_rounds<CHIP>(s, id, id >> 6, lane, r0, rounds, plan_stride, sc.active, t0, single ? s.t_hist : s.hist_next);
    if (id < s.n) {
      (single ? s.t : s.t_next)[id] = t;
      if (s.blk_head) {
        s.blk_head[kHeadWords * id] = t0;
        s.blk_head[kHeadWords * id + 1] = t;
      }
    }
  } else if (id < lanes_n + lanes_R) {
    const int e = id - lanes_n;
    if (CHIP) edge_rounds<0, kOnChip>(s, e, r0, rounds, plan_stride, sc, e < s.eR, &rare, barrier);
    else if (s.blk_plan) edge_rounds<0, kRecords>(s, e, r0, rounds, plan_stride, sc, e < s.eR, &rare, barrier);
    else edge_rounds<0, kPlans>(s, e, r0, rounds, plan_stride, sc, e < s.eR, &rare, barrier);
  } else {
    const int e = id - lanes_n - lanes_R;
    if (CHIP) edge_rounds<1, kOnChip>(s, e, r0, rounds, plan_stride, sc, e < s.eC, &rare, barrier);
    else if (s.blk_plan) edge_rounds<1, kRecords>(s, e, r0, rounds, plan_stride, sc, e < s.eC, &rare, barrier);
    else edge_rounds<1, kPlans>(s, e, r0, rounds, plan_stride, sc, e < s.eC, &rare, barrier);
  }
  __syncthreads();
  if (!single) {
    __shared__ bool last;
    if (threadIdx.x == 0) {
      __threadfence();
      last = atomicAdd(s.ticket, 1) == (int)gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    const FastMod modH(s.H);
    for (int i = threadIdx.x; i < s.n; i += blockDim.x) {
      s.t[i] = s.t_next[i];
      for (int k = rounds < s.H ? rounds : s.H; k > 0; --k) {
        const int at = modH(r0 + rounds - k);
        s.t_hist[(size_t)i * s.H + at] = s.hist_next[(size_t)i * s.H + at];
      }
    }
    if (threadIdx.x == 0) *s.ticket = 0;
  }
  // what the lanes of a multi-round launch test per ring slot (RfastDev::blk_head), from the counters and stamps
  if (!CHIP && s.blk_head)
    for (int j = threadIdx.x; j < s.n; j += blockDim.x) {
      int32_t* H = s.blk_head + kHeadWords * j;
      const int M = s.M, t0 = H[0], te = H[1];
      const int lo_v0 = __hip_atomic_load(&H[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int lo_s0 = __hip_atomic_load(&H[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int lo_v1 = __hip_atomic_load(&H[4], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int lo_s1 = __hip_atomic_load(&H[5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int s0 = t0 % M, se = te % M;
      unsigned in_v = 0, in_s = 0, written = 0, out_v = 0, out_s = 0;
      for (int m = 0; m < M && m < 32; ++m) {
        // version held by slot m when the latest version t is in slot t mod M (negative: never written)
        const int v0 = t0 - (s0 - m < 0 ? s0 - m + M : s0 - m), v1 = te - (se - m < 0 ? se - m + M : se - m);
        const unsigned bit = 1u << m;
        if (v0 >= lo_v0) in_v |= bit;
        if (v0 >= lo_s0) in_s |= bit;
        if (v1 > t0) written |= bit;
        if (v1 >= lo_v1) out_v |= bit;
        if (v1 >= lo_s1) out_s |= bit;
      }
      H[8] = s0;
      H[9] = se;
      H[10] = (int)in_v;
      H[11] = (int)in_s;
      H[12] = (int)written;
      H[13] = (int)out_v;
      H[14] = (int)out_s;
    }
  if (CHIP) on_chip_heads(s, r0, rounds, &rare);
  if (threadIdx.x == 0) *s.round_no = r0 + rounds;
}

}  // namespace

hipError_t rfast_launch_resolve(rfast_ctx* c, const uint8_t* active, const int32_t* delay_R,
                                const int32_t* delay_C, const uint8_t* drop_R, const uint8_t* drop_C, int rounds,
                                size_t plan_stride) {
  const RfastDev& d = c->d;
  auto whole = [](int v) { return (v + 63) / 64 * 64; };
  const int lanes_n = whole(d.n), lanes_R = whole(d.eR), lanes_C = whole(d.eC);
  const int64_t lanes = (int64_t)lanes_n + lanes_R + lanes_C;
  // One workgroup as long as it holds every lane; beyond, workgroups of two wavefronts, which spread over the chip.
  const bool single = lanes <= kGroupLanes;
  if (!single && (d.blk_head || d.blk_slots)) return hipErrorInvalidValue;  // the kernels that read it take graphs of at most 64 nodes
  const int threads = single ? (int)lanes : 128;
  const int64_t groups = (lanes + threads - 1) / threads;
  if (groups > 0x7fffffffLL) return hipErrorInvalidValue;
  const Sched sc = {active, delay_R, delay_C, drop_R, drop_C};
  if (d.blk_plan && d.blk_slots)
    hipLaunchKernelGGL(rfast_resolve_kernel<true>, dim3((unsigned)groups), dim3(threads), 0, c->stream, d, rounds, plan_stride, sc, lanes_n,
                       lanes_R, lanes_C);
  else
    hipLaunchKernelGGL(rfast_resolve_kernel<false>, dim3((unsigned)groups), dim3(threads), 0, c->stream, d, rounds, plan_stride, sc, lanes_n,
                       lanes_R, lanes_C);
  return hipGetLastError();
}
