// Several rounds per launch for least squares and logistic regression beyond one compute unit: a TEAM of workgroups
// per node, all of them resident for the whole launch.
//
// As a chain of kernels a round of these objectives is 12 to 25 us however little it moves: every kernel of the chain
// starts with a launch and three or four dependent round trips to memory.  Here workgroup (i, w) keeps chunk w of the
// coordinates of node i: x, z, the stored sample, the latest running sum and the heavy-ball buffer stay in registers
// and, where they fit, the sampled rows in LDS; it goes through the rounds in which its node does something and talks
// to the other workgroups through memory:
//   rings   v and the running sums are published by stores and read by loads of agent scope (the L2 caches of the
//           accelerator dies are not coherent with each other; such accesses meet behind them).  The part of a ring
//           that wavefront y of workgroup (j, w) writes is read by wavefronts y of the workgroups (i, w) only, so the
//           progress words of a wavefront (kFlagWords) are all the
//           synchronisation there is between nodes: no barrier over the chip, a node waits for the versions it reads.
//           The longest path through the rounds runs from node to node along these words, each hop 1 to 2 us of travel and
//           what lies between a wait and the word that it lets its owner set.  So every word is set as soon as what it says
//           holds (v is out when the dot products are formed, what a round reads of others when it is read), and running
//           sums that are not out when the dot products are known are waited for behind the gradient.  Us per round with one word per graph,
//           set behind the dot products and with the sums, and now: 31 nodes in a binary tree, p = 784: 5.6 -> 4.7; full gradients of 5
//           nodes in a ring, p = 89, 214 rows: 8.4 -> 8.2.
//   dots    a row's product a_s . x' is the sum of one term per workgroup of the team, exchanged as 8-byte packets of
//           value and round number: the packet is its own flag, one trip through memory (0.8-1.3 us, measured)
//           instead of data, acknowledgement, flag, poll and read.
// What a wavefront may wait for belongs to rounds before the one it is in, or (packets) to the same round of its own
// team, whose members wait for earlier rounds only: by induction over the rounds every wait ends, as long as all
// workgroups of the launch are resident.  They are no more than the compute units (rfast_team_shape), and none of them
// touches the state before all have started (team_complete).  The waits are bounded all the same: a wait that runs
// out reports an error (rfast_check) and no later wait of the workgroup waits at all.
//   A ring slot is overwritten only when every receiver is past the rounds in which its version could be read: the
// slot of version t + 1 held version t - D - 1, which left the readable window with the sender's previous activation,
// so the receivers must have finished the round of that activation.
//
// Four wavefronts own the coordinates (kOwn lanes, kE each); four more fetch the sampled rows of the next active round
// while the others update and mix.  (Loads return in order: a wavefront that polls and fetches rows would poll behind
// the rows.)  All eight form dot products and column sums.
//
// The arithmetic is, operation for operation, that of rfast_state_kernel<MIX>, rfast_rows_kernel, rfast_cols_kernel and
// rfast_state_kernel<TRACK> (same bits); rfast_rows_kernel adds a row's terms by the chunks of RfastDev::row_chunk, the
// chunks of the workgroups here.  SYNC: the synchronous step of eq. (2) instead of a round, every node in every step; v and z
// go from node to node as packets of value and step, like the dot products, in memory of their own (slot 0 of the v ring keeps the last v, as
// with a kernel per step): one trip through memory, where values, acknowledgement, word, poll and read were four.  16 nodes, p = 1001, 96
// rows: 6.5 -> 6.4 us per step.  (v and z apart, so that whoever reads one does not fetch the other, too: interleaved, the lines of the rings took
// twice as long to read where a lane has several coordinates or a node several in-edges: 32 nodes, p = 4096, 64 rows 8.7 -> 7.4 us per step, 7.3 by
// words; 90 nodes of an exponential graph, p = 1600, 64 rows 18.4 -> 16.0, 15.3; binary tree of 100, p = 2000, 6.7 -> 5.4, 6.8.)  The rings of the running sums are not touched: the diagnostics and reads see them as
// rfast_init left them.
//
// Measured, us per round, before (two kernels per round; five for the synchronous step, the heavy-ball buffer and one
// agent per iteration) and now: logistic, 31 nodes in a binary tree, p = 784, batch 32: 12.0 -> 4.7; 32 nodes, p = 4096,
// batch 64: 21.2 -> 8.9; synchronous least squares, 16 nodes, p = 1001, 96 rows: 25.4 -> 6.1; one agent of 55 per
// iteration, p = 208: 18.2 -> 1.6.  What bounds it is the chain of trips through memory of a round (versions in, dot
// products out and in, sums out).
// Registers spilled outside the synchronous steps with a tile of rows: none with one coordinate per lane, 5 and 6 with four and two, 47 with eight (184 B; 22
// without a tile).  That is more than with every wait ahead of the gradient and addresses formed where they are used, and still faster: us per
// 100 rounds then and now, eight per lane: 32 nodes, p = 16384, batch 12 1260 -> 1091 (all active 1486 -> 1353), batch 48 (no tile) 2735 -> 2378; mesh
// of 60, p = 8191, batch 16 1639 -> 1310; tree of 120, p = 4000 1259 -> 1031; four per lane: ring of 100, p = 1900, batch 32 679 -> 627.
#include <type_traits>

#include "rfast_team.h"

namespace {

constexpr int kThreads = kTeamThreads;

// A row of memory in scalar registers, from a pointer of one lane, and a value of it
typedef const __attribute__((address_space(1))) char* Row;
__device__ inline Row lane_row(const float* p, int l) {
  const u64 v = (u64)(uintptr_t)p;
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, l), hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), l);
  return (Row)((u64)hi << 32 | lo);
}
__device__ inline float get_row(Row r, unsigned at) {
  return __hip_atomic_load((const __attribute__((address_space(1))) float*)(r + at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline u64 get_packet(Row r, unsigned at) {
  return __hip_atomic_load((const __attribute__((address_space(1))) u64*)(r + at), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
constexpr int kOwn = 256;                  // lanes that own coordinates
constexpr int kOwnWaves = kOwn / 64;
constexpr int kLoad = kThreads - kOwn;     // lanes that fetch rows
constexpr int kLoadWaves = kLoad / 64;
constexpr int kTileRows = 64 * kLoadWaves; // most sampled rows of a tile: a fetching wavefront holds their numbers, one per lane
// packets: [2][n][W][B]; progress entries: [n][W][kOwnWaves]

// A barrier for what is in LDS: accesses to memory may be under way across it.
__device__ inline void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// value of lane ^ 1, ^ 2 (quad permutes), ^ 4 (half rows reversed, then quads), ^ 8 (rows of 16 rotated by 8)
template <int CTRL> __device__ inline float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ inline float xor1(float v) { return dpp<0xB1>(v); }
__device__ inline float xor2(float v) { return dpp<0x4E>(v); }
__device__ inline float xor4(float v) { return dpp<0x1B>(dpp<0x141>(v)); }
__device__ inline float xor8(float v) { return dpp<0x128>(v); }
// a[l] + a[l ^ 32] in the lower half of the wavefront, b[l] + b[l ^ 32] in the upper; the same with rows of 16 lanes
__device__ inline float fold32(float a, float b) {
  const auto t = __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false);
  return __int_as_float(t[0]) + __int_as_float(t[1]);
}
__device__ inline float fold16(float a, float b) {
  const auto t = __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false);
  return __int_as_float(t[0]) + __int_as_float(t[1]);
}

// The rounds of a launch by one workgroup (see team_complete), in the order of operations of the team: same bits.
// rowi: [B] words of LDS (if rows are sampled), rs: [4][Bq].
template <bool SYNC>
__device__ __forceinline__ void alone(const RfastDev& s, const TeamArgs& a, int* rowi, float* rs) {
  const int n = s.n, B = a.B, Bq = (B + 15) / 16 * 4, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t p = s.p;
  const bool sampled = a.batch_idx != nullptr, logistic = s.prob.kind == RFAST_OBJ_LOGISTIC;
  const float inv = 1.0f / (float)B, lam = (logistic ? s.prob.lambda : 0.f) + s.wd;
  auto residuals = [&](int i, int q) {
    const float* x = s.x + (size_t)i * p;
    const float* data = (const float*)s.prob.data0 + (size_t)i * s.prob.samples * p;
    for (int b = tid; sampled && b < B; b += kTeamThreads) rowi[b] = team_row(s, a, SYNC, i, q, a.batch_idx[((size_t)q * n + i) * B + b], true);
    __syncthreads();  // x and the row numbers
    for (int b = wave; b < B; b += kTeamThreads / 64) {
      const int row = sampled ? rowi[b] : b;
      const float* ar = data + (size_t)row * p;
      float dot = 0.f;
      for (int64_t c0 = 0; c0 < p; c0 += a.C) {
        const int64_t end = c0 + a.C < p ? c0 + a.C : p;
        float acc = 0.f;
        for (int64_t k0 = c0 + 4 * lane; k0 < end; k0 += 256)
          for (int64_t k = k0; k < end && k < k0 + 4; ++k) acc = fmaf(ar[k], x[k], acc);
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
        dot = c0 == 0 ? acc : dot + acc;
      }
      const float y = ((const float*)s.prob.data1)[(size_t)i * s.prob.samples + row];
      if (lane == 0) rs[(b & 3) * Bq + (b >> 2)] = logistic ? 1.0f / (1.0f + expf(-dot)) - y : dot - y;
    }
    __syncthreads();
  };
  auto gradient = [&](int i, int64_t k) {
    const float* col = (const float*)s.prob.data0 + (size_t)i * s.prob.samples * p + k;
    float acc[4];
    for (int rg = 0; rg < 4; ++rg) {
      acc[rg] = 0.f;
      for (int b = rg; b < B; b += 4) acc[rg] = fmaf(rs[rg * Bq + (b >> 2)], col[(size_t)(sampled ? rowi[b] : b) * p], acc[rg]);
    }
    return fmaf(lam, s.x[(size_t)i * p + k], (((acc[0] + acc[1]) + acc[2]) + acc[3]) * inv);
  };
  const size_t half = (size_t)n * p;
  for (int q = 0; q < a.rounds; ++q) {
    if (!SYNC) {
      const int32_t* rec = s.blk_plan + (size_t)q * (n + s.eR + s.eC + 1);
      for (int i = 0; i < n; ++i) {
        const int t_old = rec[i] & 0x3FFFFFFF;
        if (rec[i] < 0) {
          alone_mix(s, i, (t_old + 1) % s.M, a.gamma, rec + n);
          residuals(i, q);
          alone_track(s, i, t_old, rec + n + s.eR, [&](int64_t k) { return gradient(i, k); });
          __syncthreads();  // residuals and row numbers may be overwritten
        }
        alone_save(s, i, rec + n + s.eR);
      }
      continue;
    }
    // all of v (slot 0) before the first x'; the new z waits in slot 1 until nobody needs the old one
    for (int64_t k = tid; k < p; k += kTeamThreads) {
      for (int i = 0; i < n; ++i) {
        float dir = s.z[(size_t)i * p + k];
        if (s.mom) s.mom[(size_t)i * p + k] = dir = fmaf(s.beta, s.mom[(size_t)i * p + k], dir);
        s.v_ring[(size_t)i * s.M * p + k] = fmaf(-a.gamma, dir, s.x[(size_t)i * p + k]);
      }
      for (int i = 0; i < n; ++i) {
        float x = s.r_self[i] * s.v_ring[(size_t)i * s.M * p + k];
        for (int e = s.r_ptr[i]; e < s.r_ptr[i + 1]; ++e) x = fmaf(s.r_w[e], s.v_ring[(size_t)s.r_src[e] * s.M * p + k], x);
        s.x[(size_t)i * p + k] = x;
      }
    }
    for (int i = 0; i < n; ++i) {
      const size_t now = ((s.t[i] + q + 1) & 1) * half, before = ((s.t[i] + q) & 1) * half;
      residuals(i, q);
      for (int64_t k = tid; k < p; k += kTeamThreads) {
        const float g = gradient(i, k);
        s.g[now + (size_t)i * p + k] = g;
        float z = s.c_self[i] * s.z[(size_t)i * p + k];
        for (int e = s.c_ptr[i]; e < s.c_ptr[i + 1]; ++e) z = fmaf(s.c_w[e], s.z[(size_t)s.c_src[e] * p + k], z);
        s.v_ring[((size_t)i * s.M + 1) * p + k] = (z + g) - s.g[before + (size_t)i * p + k];
      }
      __syncthreads();  // residuals and row numbers may be overwritten
    }
    for (int64_t k = tid; k < p; k += kTeamThreads)
      for (int i = 0; i < n; ++i) s.z[(size_t)i * p + k] = s.v_ring[((size_t)i * s.M + 1) * p + k];
  }
}

template <int kE, bool TILE, bool SYNC>
__global__ void __launch_bounds__(kThreads) rfast_team_kernel(RfastDev s, TeamArgs a) {
  constexpr int KB = kE <= 2 ? 8 : (kE == 4 ? 4 : 2);  // in-edges whose ring values are in flight together
  extern __shared__ float4 lds4[];
  __shared__ int verdict;
  if (threadIdx.x == 0) team_arrive(a);
  const int n = s.n, M = s.M, W = a.W, B = a.B, S = s.prob.samples;
  const int64_t p = s.p;
  const int i = blockIdx.x / W, w = blockIdx.x - i * W;
  const int first = w * a.C;                                        // first coordinate of the chunk
  const int Cw = (int)p - first < a.C ? (int)p - first : a.C;       // its coordinates
  const int Q = (Cw + 3) >> 2, Qm = (a.C + 3) >> 2;                 // its groups of four; those of the widest chunk
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool owner = tid < kOwn;
  const bool sampled = a.batch_idx != nullptr;
  // ---- LDS
  float4* const tile = lds4;                                        // TILE: [B][Q]
  float4* xs4 = tile + (TILE ? (size_t)B * Qm : 0);                 // [Q] the mixed x of this round
  float4* cp4 = xs4 + Qm;                                           // [4][Q] column sums of the four groups of rows
  float* rs = reinterpret_cast<float*>(cp4 + 4 * Qm);               // [4][Bq] residuals, row b at [b mod 4][b / 4]
  const int Bq = (B + 15) / 16 * 4;
  int* rowi = reinterpret_cast<int*>(rs + 4 * Bq);                       // [2][B] sampled rows of this active round and the next
  int* nodew = rowi + (sampled ? 2 * B : 0);                        // [kBlockRounds] node words
  __shared__ u64 act_mask[kBlockRounds / 64], ev_mask[kBlockRounds / 64];
  float* xs = reinterpret_cast<float*>(xs4);
  const float* rows_g = (const float*)s.prob.data0 + (size_t)i * S * p + first;   // + row p + coordinate in the chunk
  const float* targets = (const float*)s.prob.data1 + (size_t)i * S;

  // ---- the rounds in which the node does something: it is active, or an S4 buffer of it has to be saved
  const int W1 = n + s.eR + s.eC + 1;
  const int round0 = first_round(s, a, SYNC);
  if (!SYNC) {
    int word = 0;
    bool spill = false;
    if (tid < a.rounds) {
      word = s.blk_plan[(size_t)tid * W1 + i];
      spill = s.blk_spill[(size_t)tid * n + i] == round0 + tid + 1;
    }
    nodew[tid] = word;
    const u64 am = __ballot(word < 0), em = __ballot(word < 0 || spill);
    if (lane == 0) {
      act_mask[wave] = am;
      ev_mask[wave] = em;
    }
  }
  static_assert(kThreads == kBlockRounds, "one lane per round above");

  // ---- graph of the node, one edge per lane; state of the owned coordinates
  // (SYNC: a wavefront without coordinates reads nobody's packets)
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);
  const bool wave_has = wave_s < kOwnWaves && 64 * wave_s < Cw, reads = !SYNC || wave_has;
  const int re0 = s.r_ptr[i], dR = reads ? s.r_ptr[i + 1] - re0 : 0, ce0 = s.c_ptr[i], dI = reads ? s.c_ptr[i + 1] - ce0 : 0;
  const int ro0 = s.ro_ptr[i], dRo = s.ro_ptr[i + 1] - ro0, co0 = s.co_ptr[i], dCo = s.co_ptr[i + 1] - co0;
  const float r_self = s.r_self[i], c_self = s.c_self[i];
  int r_src = 0, c_src = 0, r_dst = 0, c_dst = 0;
  float r_w = 0.f, c_w = 0.f;
  if (lane < dR) { r_src = s.r_src[re0 + lane]; r_w = s.r_w[re0 + lane]; }
  if (lane < dI) { c_src = s.c_src[ce0 + lane]; c_w = s.c_w[ce0 + lane]; }
  if (lane < dRo) r_dst = s.r_dst[s.ro_eid[ro0 + lane]];
  if (lane < dCo) c_dst = s.c_dst[s.co_eid[co0 + lane]];
  // What a round touches, formed once: the progress words of the wavefronts of the same number and chunk ([0] .. [3], see
  // kFlagWords) of the lane's neighbours (nullptr: no such edge), the rings of its senders, and the lane's coordinates as 32-bit
  // byte offsets, so that a load is an address in scalar registers plus such an offset.  (Formed where they were used they cost up
  // to 2000 cycles a round in 64-bit products and, with a branch per coordinate, in masks.)
  auto flag_of = [&](bool there, int node) {
    return there ? a.flags + ((size_t)(node * W + w) * kOwnWaves + wave) * kFlagWords : nullptr;
  };
  unsigned* const f_own = flag_of(true, i);
  const unsigned* const f_r_src = flag_of(lane < dR, r_src);
  const unsigned* const f_r_dst = flag_of(lane < dRo, r_dst);
  const unsigned* const f_c_src = flag_of(lane < dI, c_src);
  const unsigned* const f_c_dst = flag_of(lane < dCo, c_dst);
  auto word_of = [](const unsigned* f, int word) { return f ? f + word : nullptr; };
  const float* const r_ring = s.v_ring + (size_t)r_src * M * p + first;
  const float* const c_ring = s.sigma_ring + (size_t)c_src * M * p + first;
  // SYNC: [2][2][n][p] packets, v and z in the even steps, then in the odd ones; the senders' and the node's own of the even steps
  const size_t sync_z = (size_t)n * p, sync_half = 2 * sync_z;
  const u64* const r_sync = a.sync + (size_t)r_src * p + first;
  const u64* const c_sync = a.sync + sync_z + (size_t)c_src * p + first;
  u64* const own_sync = a.sync + (size_t)i * p + first;
  const float* const c_save = s.rho_tilde + (size_t)(ce0 + (lane < dI ? lane : 0)) * p + first;
  const bool momentum = s.mom != nullptr;
  const float inv = 1.0f / (float)B;
  const bool logistic = s.prob.kind == RFAST_OBJ_LOGISTIC;
  const float lam = (logistic ? s.prob.lambda : 0.f) + s.wd;  // l2 term plus the weight decay of the optimizer variant
  __syncthreads();
  const int t0 = SYNC ? s.t[i] : nodew[0] & 0x3FFFFFFF;
  float x[kE], z[kE], g[kE], sc[kE], m[kE];
  bool has[kE];
  // Byte offset of the coordinate in the chunk.  A lane that has none loads the first one of its wavefront, and nobody looks at the value.  SYNC: the
  // tags of all lanes are looked at, so it must not be another wavefront's: what keeps a sender's wavefront from overwriting a packet
  // is the word of the wavefront of its number here, which may be a step ahead of the others behind the last barrier of a
  // step, and the tag that they wait for would never come.  (A test of the tags that leaves such lanes out costs 16 nodes, p = 1001, 96
  // rows 3 %.)
  unsigned at[kE];
#pragma unroll
  for (int e = 0; e < kE; ++e) {
    const int k = tid + kOwn * e;
    has[e] = owner && k < Cw;
    at[e] = has[e] ? 4u * (unsigned)k : SYNC && wave_has ? 4u * (unsigned)(tid - lane) : 0u;
    x[e] = z[e] = g[e] = sc[e] = m[e] = 0.f;
    if (has[e]) {
      const size_t off = (size_t)i * p + first + k;
      x[e] = s.x[off];
      z[e] = s.z[off];
      g[e] = s.g[(size_t)(t0 & 1) * n * p + off];
      if (!SYNC) sc[e] = s.sigma_ring[((size_t)i * M + t0 % M) * p + first + k];
      if (momentum) m[e] = s.mom[off];
    }
  }
  if (tid < 4 * Q - Cw) xs[Cw + tid] = 0.f;  // the unused end of the last group of four stays zero
  if (TILE)
    for (int f = tid; f < B * (4 * Q - Cw); f += kThreads) {
      const int r = f / (4 * Q - Cw);
      reinterpret_cast<float*>(tile + (size_t)r * Q)[Cw + (f - r * (4 * Q - Cw))] = 0.f;
    }

  bool dead = false;  // a wait has run out
  auto wait2 = [&](const unsigned* f1, int need1, const unsigned* f2, int need2, unsigned v1, unsigned v2) {
    wait_progress(a, SYNC, i, f1, need1, f2, need2, v1, v2, &dead);
  };

  // ---- rows
  // (the lane's first row number as asked for a round ahead)
  auto ask_row = [&](int q) { return q < a.rounds && tid - kOwn < B ? a.batch_idx[((size_t)q * n + i) * B + (tid - kOwn)] : 0; };
  auto keep_rows = [&](int q, int first_row, int* to) {
    for (int b = tid - kOwn; b < B; b += kLoad)
      to[b] = team_row(s, a, SYNC, i, q, b == tid - kOwn ? first_row : a.batch_idx[((size_t)q * n + i) * B + b], w == 0);
  };
  int row_ahead = 0;
  // Four coordinates of a row (unaligned where p is no multiple of four).  At the chunk's ragged end the load starts up
  // to three coordinates early, still inside the row, and whole_quad moves them into place and clears the rest.
  const bool ragged = (Cw & 3) != 0;
  auto row_quad = [&](int row, int quad) {
    const int at = ragged && 4 * quad > Cw - 4 ? Cw - 4 : 4 * quad;
    return V<5>::ld(rows_g + (size_t)row * p + at);
  };
  auto whole_quad = [&](float4 v, int quad) {
    const int by = 4 * quad + 4 - Cw;  // coordinates the load started early
    if (ragged && by > 0) {
      v.x = by == 1 ? v.y : by == 2 ? v.z : v.w;
      v.y = by == 1 ? v.z : by == 2 ? v.w : 0.f;
      v.z = by == 1 ? v.w : 0.f;
      v.w = 0.f;
    }
    return v;
  };
  const unsigned q_magic = 0xFFFFFFFFu / (unsigned)Q;
  auto split = [&](int f, int* b, int* quad) {  // f / Q and f mod Q
    int d = (int)__umulhi((unsigned)f, q_magic);
    int r = f - d * Q;
    if (r >= Q) { r -= Q; ++d; }
    *b = d;
    *quad = r;
  };
  // Rows into LDS, straight from memory: no registers, so that everything is in flight at once.  A wavefront takes every
  // kLoadWaves-th row; the destination of such a load is contiguous over the lanes.
  const bool wide = (p & 3) == 0;  // 16-byte pieces need 16-byte addresses
  auto load_tile = [&](const int* rows) {
    const int lw = wave - kOwnWaves;
    const int mine = sampled && lw + kLoadWaves * lane < B ? rows[lw + kLoadWaves * lane] : 0;
    int r = 0;
    for (int b = lw; b < B; b += kLoadWaves, ++r) {
      const float* src = rows_g + (size_t)(sampled ? lane_value(mine, r) : b) * p;
      float4* to = tile + b * Q;
      if (wide) {
        for (int quad = lane; quad < Q; quad += 64)
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + 4 * quad),
                                           (__attribute__((address_space(3))) void*)(to + (quad - lane)), 16, 0, 0);
      } else {
        for (int k = lane; k < Cw; k += 64)
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + k),
                                           (__attribute__((address_space(3))) void*)(reinterpret_cast<float*>(to) + (k - lane)), 4, 0, 0);
      }
    }
  };
  const int rounds = a.rounds;
  auto next_active = [&](int from) { return SYNC ? from : next_bit(act_mask, from); };
  auto next_event = [&](int from) { return SYNC ? from : next_bit(ev_mask, from); };
  int parity = 0;  // of the active rounds of this launch: packets and row numbers alternate
  {
    const int qa = next_active(0);
    if (!owner && sampled && qa < rounds) {
      keep_rows(qa, ask_row(qa), rowi);
      row_ahead = ask_row(next_active(qa + 1));
    }
    if (sampled) __syncthreads();
    if (TILE && !owner && qa < rounds) load_tile(rowi);
  }

  int q = next_event(0), q_prev = -1;  // this event, and the last round in which the node was active
  // plan words and delays of the event, an edge per lane (of the next event: fetched while this one is computed)
  int rw_n = 0, cw_n = 0, rd_n = 0, cd_n = 0;
  auto fetch_plan = [&](int at) {
    if (SYNC || at >= rounds) return;
    const int32_t* rec = s.blk_plan + (size_t)at * W1;
    if (lane < dR) { rw_n = rec[n + re0 + lane]; rd_n = a.delay_R[(size_t)at * s.eR + re0 + lane]; }
    if (lane < dI) { cw_n = rec[n + s.eR + ce0 + lane]; cd_n = a.delay_C[(size_t)at * s.eC + ce0 + lane]; }
  };
  auto clamped = [&](int d) { return d < 0 ? 0 : (d > s.d_max ? s.d_max : d); };
  if (owner) {
    fetch_plan(q);
  }
  if (wave == 0) {
    const int all = team_complete(a, lane);
    if (lane == 0) verdict = all;
  }
  __syncthreads();
  if (verdict != 0) {
    drain();  // (rows may be on their way into LDS)
    if (verdict == 2) {
      const TeamKernelArgs& k = team_kernel_args();
      alone<SYNC>(k.s, k.a, rowi, rs);
    }
    return;
  }
  if (owner) {
    if (!SYNC && lane == 0) {  // rounds before the first event: nothing to wait for
      put32(f_own, a.base + (unsigned)(q < rounds ? q : rounds));
      put32(f_own + 1, a.base + (unsigned)(q < rounds ? q : rounds));
      put32(f_own + 2, a.base + (unsigned)(q < rounds ? q : rounds));
      put32(f_own + 3, a.base + (unsigned)(q < rounds ? q : rounds));
    }
  }

  unsigned seen_r = a.base, seen_d = a.base;  // the words that the next mix waits for, as read ahead
  // SYNC: asks for the packets of up to KB in-edges from e0 on, an edge's senders in the lanes of `from`; whether
  // all of them are those of the step; and both until they are
  u64 step_tag = 0;
  auto ask_packets = [&](const u64* from, int e0, int edges, u64 (&got)[KB][kE]) {
#pragma unroll
    for (int u = 0; u < KB; ++u)
      if (e0 + u < edges) {
        const Row row = lane_row(reinterpret_cast<const float*>(from), e0 + u);
#pragma unroll
        for (int e = 0; e < kE; ++e) got[u][e] = get_packet(row, 2 * at[e]);
      }
  };
  auto all_there = [&](int e0, int edges, const u64 (&got)[KB][kE]) {
    bool ok = true;
#pragma unroll
    for (int u = 0; u < KB; ++u)
      if (e0 + u < edges) {
#pragma unroll
        for (int e = 0; e < kE; ++e) ok = ok && got[u][e] >> 32 == step_tag >> 32;
      }
    return __all(ok);
  };
  auto until_there = [&](const u64* from, int e0, int edges, u64 (&got)[KB][kE]) {
    for (int spin = 0; !dead && !all_there(e0, edges, got); ++spin) {
      if (spin >= a.wait_polls) {
        dead = true;
        report_wait(SYNC, i);
      }
      ask_packets(from, e0, edges, got);
    }
  };
  while (q < rounds) {
    step_tag = (u64)(a.base + (unsigned)q + 1u) << 32;
    const int q_next = next_event(q + 1);
    const unsigned done_word = a.base + (unsigned)(q_next < rounds ? q_next : rounds);
    const int word = SYNC ? (int)0x80000000 : nodew[q];
    const bool active = word < 0;
    const int t_old = SYNC ? t0 + q : word & 0x3FFFFFFF;
    const int rword = rw_n, cword = cw_n, rneed = q - clamped(rd_n), cneed = q - clamped(cd_n);
    const int slot_new = SYNC ? 0 : (t_old + 1) % M;
    dead = __any(dead);
    if (owner && active) {
      // ---- S1, S2a, S3 (v half)
      if (!SYNC) wait2(f_r_src, rneed, word_of(f_r_dst, 3), q_prev + 1, seen_r, seen_d);
      else wait2(f_r_dst, q, f_c_dst, q, seen_r, seen_d);
      float v[kE], xn[kE];
#pragma unroll
      for (int e = 0; e < kE; ++e) {
        float dir = z[e];
        if (momentum) dir = m[e] = fmaf(s.beta, m[e], z[e]);
        v[e] = fmaf(-a.gamma, dir, x[e]);
        xn[e] = r_self * v[e];
      }
      float* own_v = s.v_ring + ((size_t)i * M + slot_new) * p + first + tid;
      if (SYNC) {
        // Everybody's v and z of this step, as packets: each is its own flag, so that a step has no other word to wait for than the
        // one that says that the readers of the packets overwritten here are through (a wavefront that publishes step q has read all that it
        // reads of step q - 1, which is what the sender's wavefronts of its number have written).
        u64* own = own_sync + (q & 1 ? sync_half : 0) + tid;
#pragma unroll
        for (int e = 0; e < kE; ++e)
          if (has[e]) {
            put64(own + kOwn * e, step_tag | __float_as_uint(v[e]));
            put64(own + sync_z + kOwn * e, step_tag | __float_as_uint(z[e]));
            if (q == rounds - 1) own_v[kOwn * e] = v[e];
          }
        if (lane == 0) put32(f_own, a.base + (unsigned)(q + 1));
        for (int e0 = 0; e0 < dR; e0 += KB) {
          u64 got[KB][kE];
          const u64* from = r_sync + (q & 1 ? sync_half : 0);
          ask_packets(from, e0, dR, got);
          until_there(from, e0, dR, got);
#pragma unroll
          for (int u = 0; u < KB; ++u)
            if (e0 + u < dR) {
              const float wt = lane_value(r_w, e0 + u);
#pragma unroll
              for (int e = 0; e < kE; ++e) xn[e] = fmaf(wt, __uint_as_float((unsigned)got[u][e]), xn[e]);
            }
        }
      }
      const float* const v_from = r_ring + (size_t)(unsigned)rword * (size_t)p;
      for (int e0 = 0; !SYNC && e0 < dR; e0 += KB) {
        float vb[KB][kE];
#pragma unroll
        for (int u = 0; u < KB; ++u)
          if (e0 + u < dR) {
            const Row src = lane_row(v_from, e0 + u);
#pragma unroll
            for (int e = 0; e < kE; ++e) vb[u][e] = get_row(src, at[e]);
          }
#pragma unroll
        for (int u = 0; u < KB; ++u)
          if (e0 + u < dR) {
            const float wt = lane_value(r_w, e0 + u);
#pragma unroll
            for (int e = 0; e < kE; ++e) xn[e] = fmaf(wt, vb[u][e], xn[e]);
          }
      }
#pragma unroll
      for (int e = 0; e < kE; ++e)
        if (has[e]) {
          if (!SYNC) put_f(own_v + kOwn * e, v[e]);
          x[e] = xn[e];
          xs[tid + kOwn * e] = xn[e];
        }
    }
    if (active) {
      if (TILE && !owner) drain();  // the rows on their way into LDS have arrived
      __syncthreads();  // the mixed x and the sampled rows are in LDS
      unsigned seen_c = a.base, seen_o = a.base;  // the words that the running sums wait for travel during the dot products
      if (owner && !SYNC) {
        asm volatile("" ::: "memory");
        if (lane == 0) put32(f_own + 3, done_word);  // what this round reads of others' v has been used
        seen_c = peek(a, word_of(f_c_src, 1), cneed);
        seen_o = peek(a, word_of(f_c_dst, 2), q_prev + 1);
      }
      // ---- gradient, rows: eight (four) rows per wavefront at a time; lane c sums coordinates 4c .. 4c+3 (+ 256 m) of the
      // chunk, and the lanes' sums are added as a butterfly from distance 32 down to 1 whose first steps halve the rows
      const int* rows = rowi + (parity ? B : 0);
      const float target = tid < B ? targets[sampled ? rows[tid] : tid] : 0.f;  // of the lane's first row
      u64* const packets = a.packets + (size_t)(unsigned)((parity * n + i) * W) * (unsigned)B;  // of the team and the round
      u64* const out = packets + w * B;
      auto dots = [&](auto rb) {
        constexpr int RB = decltype(rb)::value;
        for (int b0 = wave * RB; b0 < B; b0 += RB * (kThreads / 64)) {
          float acc[RB];
          const float4* trow[RB];
          int grow[RB];
#pragma unroll
          for (int r = 0; r < RB; ++r) {
            acc[r] = 0.f;
            const int b = b0 + r < B ? b0 + r : B - 1;
            if (TILE) trow[r] = tile + b * Q;
            else grow[r] = sampled ? rows[b] : b;
          }
          for (int quad = lane; quad < Q; quad += 64) {
            const float4 xv = xs4[quad];
            float4 av[RB];
#pragma unroll
            for (int r = 0; r < RB; ++r) av[r] = TILE ? trow[r][quad] : row_quad(grow[r], quad);
            if (!TILE && ragged) {
#pragma unroll
              for (int r = 0; r < RB; ++r) av[r] = whole_quad(av[r], quad);
            }
#pragma unroll
            for (int r = 0; r < RB; ++r) {
              acc[r] = fmaf(av[r].x, xv.x, acc[r]);
              acc[r] = fmaf(av[r].y, xv.y, acc[r]);
              acc[r] = fmaf(av[r].z, xv.z, acc[r]);
              acc[r] = fmaf(av[r].w, xv.w, acc[r]);
            }
          }
          // distances 32 and 16 halve the rows: one swap of half-wavefronts (rows of 16 lanes) brings both terms of two
          // rows' sums together, the lower lanes going on with the first row; 8 .. 1 through the data-parallel moves
          int row = 0;
          if constexpr (RB == 8) {
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = fold32(acc[r], acc[r + 4]);
            row += lane & 32 ? 4 : 0;
#pragma unroll
            for (int r = 0; r < 2; ++r) acc[r] = fold16(acc[r], acc[r + 2]);
            row += lane & 16 ? 2 : 0;
            const bool up = lane & 8;
            const float keep = up ? acc[1] : acc[0], send = up ? acc[0] : acc[1];
            acc[0] = keep + xor8(send);
            row += up ? 1 : 0;
          } else {
#pragma unroll
            for (int r = 0; r < 2; ++r) acc[r] = fold32(acc[r], acc[r + 2]);
            row += lane & 32 ? 2 : 0;
            acc[0] = fold16(acc[0], acc[1]);
            row += lane & 16 ? 1 : 0;
            acc[0] += xor8(acc[0]);
          }
          float sum = acc[0];
          sum += xor4(sum);
          sum += xor2(sum);
          sum += xor1(sum);
          if (!SYNC && b0 == wave * RB && owner) {  // v has gone out meanwhile
            drain();
            if (lane == 0) put32(f_own, done_word);
          }
          const int b = b0 + row;
          if ((lane & (64 / RB - 1)) == 0 && b < B) {
            if (W == 1) rs[(b & 3) * Bq + (b >> 2)] = sum;
            else
              put64(out + b, (u64)(a.base + (unsigned)q + 1u) << 32 | __float_as_uint(sum));
          }
        }
      };
      if (B >= 64) dots(std::integral_constant<int, 8>());
      else dots(std::integral_constant<int, 4>());
      // ---- the owners ask for the ring values of the tracker update; the others look up the rows of the next round
      float sg[KB][kE], rt[KB][kE];
      u64 zp[KB][kE];  // SYNC
      const int qa = next_active(q + 1);
      const bool late_sums = !SYNC && __any(lane < dI && (cword & (1 << 18)));
      // (a batch of in-edges from e0 on; as many loads as there are live edges)
      const unsigned c_prev = (unsigned)cword >> 8 & 0xFFu;
      const float* const c_now = c_ring + (size_t)((unsigned)cword & 0xFFu) * (size_t)p;
      const float* const c_last = c_prev != 0xFFu ? c_ring + (size_t)c_prev * (size_t)p : c_save;
      auto ask_sums = [&](int e0) {
#pragma unroll
        for (int u = 0; u < KB; ++u)
          if (e0 + u < dI && (lane_value(cword, e0 + u) & (1 << 16))) {
            const Row now = lane_row(c_now, e0 + u), last = lane_row(c_last, e0 + u);
#pragma unroll
            for (int e = 0; e < kE; ++e) {
              sg[u][e] = get_row(now, at[e]);
              rt[u][e] = get_row(last, at[e]);
            }
          }
      };
      bool early = false;
      if (owner) {
        if (SYNC) {
          seen_r = peek(a, f_r_dst, q + 1);
          seen_d = peek(a, f_c_dst, q + 1);
          ask_packets(c_sync + (q & 1 ? sync_half : 0), 0, dI, zp);
        }
        fetch_plan(q_next);
      } else if (sampled && qa < rounds) {
        keep_rows(qa, row_ahead, rowi + (parity ? 0 : B));
      }
      // ---- residuals: the terms of the team in order
      if (W == 1) __syncthreads();
      for (int b = tid; b < B && (W == 1 || owner); b += W == 1 ? kThreads : kOwn) {
        float dot;
        if (W == 1) {
          dot = rs[(b & 3) * Bq + (b >> 2)];
        } else {
          dot = 0.f;
          const u64* src = packets + b;
          const unsigned tag = a.base + (unsigned)q + 1u;
          for (int w0 = 0; w0 < W; w0 += 8) {
            u64 got[8];
            for (int spin = 0;; ++spin) {
              bool ok = true;
#pragma unroll
              for (int u = 0; u < 8; ++u)
                if (w0 + u < W) got[u] = get64(src + (size_t)(w0 + u) * B);
#pragma unroll
              for (int u = 0; u < 8; ++u)
                if (w0 + u < W) ok = ok && (unsigned)(got[u] >> 32) == tag;
              if (ok || dead) break;
              if (spin >= a.wait_polls) {
                dead = true;
                report_wait(SYNC, i);
                break;
              }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (w0 + u < W) dot = w0 + u == 0 ? __uint_as_float((unsigned)got[u]) : dot + __uint_as_float((unsigned)got[u]);
          }
        }
        const float y = b == tid ? target : targets[sampled ? rows[b] : b];
        rs[(b & 3) * Bq + (b >> 2)] = logistic ? 1.0f / (1.0f + expf(-dot)) - y : dot - y;
      }
      if (owner && !SYNC) {
        if (wave * (B >= 64 ? 8 : 4) >= B) {  // (a wavefront without rows)
          drain();
          if (lane == 0) put32(f_own, done_word);
        }
        // The running sums of the in-edges, if the words say that they are out and that the place of this round's own is free.  (Here, where
        // the words have returned with the packets: waited for before them they cost 1500 cycles more.)
        early = !__any((lane < dI && cneed > 0 && (int)(seen_c - a.base) < cneed) || (lane < dCo && (int)(seen_o - a.base) <= q_prev));
        if (early) ask_sums(0);
      }
      __syncthreads();  // residuals, and the row numbers of the next active round
      // The words of the sums again, which travel during the column sums: read behind them only, the wait was a trip of its own wherever all nodes
      // are active and their words come a little late (us per 100 rounds: 16 nodes, p = 1000, 200 rows 884 -> 853; 31 nodes, p = 784, 200 rounds 957 -> 940).
      if (owner && !SYNC && !early) {
        seen_c = peek(a, word_of(f_c_src, 1), cneed);
        seen_o = peek(a, word_of(f_c_dst, 2), q_prev + 1);
      }
      // ---- gradient, columns: group rg sums rows rg, rg + 4, ... for four coordinates; for two where four would leave half of
      // the wavefronts without any (a SIMD issues for one wavefront every other time only: 16 nodes, p = 1001, 96 rows, synchronous, 6.4 -> 6.25 us per step)
      if (TILE && 8 * Q <= kThreads) {
        if (tid < 8 * Q) {
          int rg, quad;
          split(tid >> 1, &rg, &quad);
          float2 acc = make_float2(0.f, 0.f);
          const float* rq = rs + rg * Bq;
          const float2* half = reinterpret_cast<const float2*>(tile + quad) + (tid & 1);
          auto row_of_group = [&](int b, float r) {
            const float2 av = half[2 * b * Q];
            acc.x = fmaf(r, av.x, acc.x);
            acc.y = fmaf(r, av.y, acc.y);
          };
          int b = rg;
#pragma unroll 2
          for (; b + 12 < B; b += 16) {
            const float4 r4 = *reinterpret_cast<const float4*>(rq + (b >> 2));
            row_of_group(b, r4.x);
            row_of_group(b + 4, r4.y);
            row_of_group(b + 8, r4.z);
            row_of_group(b + 12, r4.w);
          }
          for (; b < B; b += 4) row_of_group(b, rq[b >> 2]);
          reinterpret_cast<float2*>(cp4)[tid] = acc;
        }
      }
      for (int f = TILE && 8 * Q <= kThreads ? 4 * Q : tid; f < 4 * Q; f += kThreads) {
        int rg, quad;
        split(f, &rg, &quad);
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
        const float* rq = rs + rg * Bq;
        auto row_of_group = [&](int b, float r) {
          const float4 av = TILE ? tile[b * Q + quad] : whole_quad(row_quad(sampled ? rows[b] : b, quad), quad);
          acc.x = fmaf(r, av.x, acc.x);
          acc.y = fmaf(r, av.y, acc.y);
          acc.z = fmaf(r, av.z, acc.z);
          acc.w = fmaf(r, av.w, acc.w);
        };
        int b = rg;
#pragma unroll 2
        for (; b + 12 < B; b += 16) {  // four rows of the group, their residuals in one read
          const float4 r4 = *reinterpret_cast<const float4*>(rq + (b >> 2));
          row_of_group(b, r4.x);
          row_of_group(b + 4, r4.y);
          row_of_group(b + 8, r4.z);
          row_of_group(b + 12, r4.w);
        }
        for (; b < B; b += 4) row_of_group(b, rq[b >> 2]);
        cp4[f] = acc;
      }
      // (loads on their way into LDS would be waited for by a barrier that orders memory, and by reads of LDS behind them: the rows
      // of the next round are asked for when the column sums are done, their numbers a round ahead of that: 31 nodes, p = 784: 5.6 -> 5.4 us.  A second tile would have nothing to
      // hold: without it 8 nodes of a mesh, p = 8192, batch 128, 9.6 -> 9.3; 16 nodes, p = 2048, batch 128, 8.8 -> 8.6)
      lds_barrier();  // column sums; the tile may be overwritten
      if (!owner) {
        if (sampled && qa < rounds) {
          const int ahead = next_active(qa + 1);  // (looked up before the rows go out: 12 nodes, p = 6000, 6.46 -> 6.40)
          if (TILE) load_tile(rowi + (parity ? 0 : B));
          row_ahead = ask_row(ahead);
        }
      } else {
        // ---- S2b, S2c, S3 (rho half), S4; or eq. (2)
        float g_new[kE], z_half[kE];
        const float* cp = reinterpret_cast<const float*>(cp4);
#pragma unroll
        for (int e = 0; e < kE; ++e) {
          const unsigned k = at[e] / 4;
          const float acc = ((cp[k] + cp[4 * Q + k]) + cp[8 * Q + k]) + cp[12 * Q + k];
          g_new[e] = fmaf(lam, x[e], acc * inv);
          z_half[e] = SYNC ? c_self * z[e] : z[e];
        }
        // (waited for here where they were not out when the dot products were: nothing before needs them)
        if (!SYNC && !early) {
          wait2(word_of(f_c_src, 1), cneed, word_of(f_c_dst, 2), q_prev + 1, seen_c, seen_o);
          ask_sums(0);
        }
        for (int e0 = 0; e0 < dI; e0 += KB) {
          if (SYNC) {
            const u64* from = c_sync + (q & 1 ? sync_half : 0);
            if (e0 > 0) ask_packets(from, e0, dI, zp);
            until_there(from, e0, dI, zp);
          } else if (e0 > 0) {
            ask_sums(e0);  // in-degree above one batch
          }
#pragma unroll
          for (int u = 0; u < KB; ++u)
            if (e0 + u < dI) {
              const float wt = lane_value(c_w, e0 + u);
              if (SYNC) {
#pragma unroll
                for (int e = 0; e < kE; ++e) z_half[e] = fmaf(wt, __uint_as_float((unsigned)zp[u][e]), z_half[e]);
              } else {
                const int pl = lane_value(cword, e0 + u);
                if (pl & (1 << 16)) {
                  const bool in_ring = ((pl >> 8) & 0xFF) != 0xFF;
#pragma unroll
                  for (int e = 0; e < kE; ++e) z_half[e] = track_edge(z_half[e], wt, sg[u][e], rt[u][e], in_ring);
                  if (pl & (1 << 17)) {
                    float* saved = s.rho_tilde + (size_t)(ce0 + e0 + u) * p + first + tid;
#pragma unroll
                    for (int e = 0; e < kE; ++e)
                      if (has[e]) saved[kOwn * e] = wt * sg[u][e];
                  }
                }
              }
            }
        }
        // what this round reads of others' sums is read, unless a buffer is still to be saved
        if (!SYNC && !late_sums) {
          drain();
          if (lane == 0) put32(f_own + 2, done_word);
        }
        float* own_s = s.sigma_ring + ((size_t)i * M + slot_new) * p + first + tid;
#pragma unroll
        for (int e = 0; e < kE; ++e)
          if (has[e]) {
            const float zh = (z_half[e] + g_new[e]) - g[e];
            g[e] = g_new[e];
            if (SYNC) {
              z[e] = zh;
            } else {
              z[e] = c_self * zh;
              if (dCo > 0) {
                sc[e] += zh;
                put_f(own_s + kOwn * e, sc[e]);
              }
            }
          }
      }
      parity ^= 1;
      q_prev = q;
    } else if (owner) {
      // an S4 buffer is about to lose its version: its sender must have published it (long ago) and may overwrite it
      // only after this
      fetch_plan(q_next);
    }
    if (owner && !SYNC) {
      // S4 for buffers whose version leaves the sender's ring in this round without being consumed
      u64 leaving = __ballot(lane < dI && (cword & (1 << 18)));
      if (!active && leaving) wait2(word_of(f_c_src, 1), cneed, nullptr, 0, a.base, a.base);
      while (leaving) {
        const int u = __ffsll((long long)leaving) - 1;
        leaving &= leaving - 1;
        const float* ring = s.sigma_ring + ((size_t)lane_value(c_src, u) * M + (lane_value(cword, u) & 0xFF)) * p + first + tid;
        float* saved = s.rho_tilde + (size_t)(ce0 + u) * p + first + tid;
        const float wt = lane_value(c_w, u);
#pragma unroll
        for (int e = 0; e < kE; ++e)
          if (has[e]) saved[kOwn * e] = wt * get_f(ring + kOwn * e);
      }
      // the words that the next mix waits for are read on the trip that the stores take anyway
      seen_r = peek(a, f_r_src, q_next - clamped(rd_n));
      seen_d = peek(a, word_of(f_r_dst, 3), q_prev + 1);
      drain();
      if (lane == 0) {
        if (!active) put32(f_own, done_word);
        put32(f_own + 1, done_word);
        put32(f_own + 2, done_word);
        if (!active) put32(f_own + 3, done_word);
      }
    }
    q = q_next;
  }

  // ---- write-back
  const int t_end = SYNC ? t0 + rounds : s.t[i];
  if (owner && (SYNC ? rounds > 0 : q_prev >= 0)) {
#pragma unroll
    for (int e = 0; e < kE; ++e)
      if (has[e]) {
        const size_t off = (size_t)i * p + first + tid + kOwn * e;
        s.x[off] = x[e];
        s.z[off] = z[e];
        s.g[(size_t)(t_end & 1) * n * p + off] = g[e];
        if (momentum) s.mom[off] = m[e];
      }
  }
}

size_t team_lds(const RfastDev& d, int C, int B, bool tile) {
  const size_t Qm = (size_t)(C + 3) / 4;
  return ((tile ? (size_t)B : 0) * Qm + 5 * Qm) * 16 + ((size_t)B + 15) / 16 * 64 + (d.prob.batch > 0 ? 2 * (size_t)B * 4 : 0) + kBlockRounds * 4;
}

template <int kE, bool TILE, bool SYNC>
hipError_t launch_team(rfast_ctx* c, const TeamArgs& a) {
  static bool raised = false;
  if (!raised) {  // more than 64 KB of dynamic LDS has to be asked for once per kernel
    const hipError_t e = hipFuncSetAttribute((const void*)rfast_team_kernel<kE, TILE, SYNC>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTeamLds);
    if (e != hipSuccess) return e;
    raised = true;
  }
  hipLaunchKernelGGL((rfast_team_kernel<kE, TILE, SYNC>), dim3((unsigned)(c->d.n * a.W)), dim3(kThreads), team_lds(c->d, a.C, a.B, TILE),
                     c->stream, c->d, a);
  return hipGetLastError();
}

template <bool SYNC>
hipError_t launch_team(rfast_ctx* c, const TeamArgs& a) {
  const RfastTeam& t = c->team;
  if (t.tiles > 0) {
    switch (t.per_lane) {
      case 1: return launch_team<1, true, SYNC>(c, a);
      case 2: return launch_team<2, true, SYNC>(c, a);
      case 4: return launch_team<4, true, SYNC>(c, a);
      default: return launch_team<8, true, SYNC>(c, a);
    }
  }
  switch (t.per_lane) {
    case 1: return launch_team<1, false, SYNC>(c, a);
    case 2: return launch_team<2, false, SYNC>(c, a);
    case 4: return launch_team<4, false, SYNC>(c, a);
    default: return launch_team<8, false, SYNC>(c, a);
  }
}

int rows_per_gradient(const rfast_problem* prob) { return prob->batch > 0 ? prob->batch : prob->samples; }

}  // namespace

// The team of a problem: workgroups per node, and their chunk of the coordinates.  `compute_units` workgroups can be
// resident at once, one each.  More workgroups mean fewer rows' bytes for each and one more trip through memory for the
// dot products; the estimate is that of a round in which every node is active.
RfastTeam rfast_team_shape(const RfastDev& d, int max_degree, int max_out_degree_r, int compute_units) {
  RfastTeam best;
  if ((d.prob.kind != RFAST_OBJ_LEAST_SQUARES && d.prob.kind != RFAST_OBJ_LOGISTIC) || d.p < 4 || d.p > (1 << 22)) return best;
  if (max_degree > 64 || max_out_degree_r > 64 || d.n > compute_units || d.M > 254) return best;  // one edge per lane
  const int B = rows_per_gradient(&d.prob), p = (int)d.p;
  double best_us = 1e30;
  for (int W = 1; W <= compute_units / d.n && W <= 32; ++W) {
    const int C = W == 1 ? p : ((p + W - 1) / W + 255) / 256 * 256;
    if ((p + C - 1) / C != W || C > 8 * kOwn) continue;
    const int64_t quads = (int64_t)B * ((C + 3) / 4);
    const bool fits = d.prob.batch == 0 || B <= kTileRows;
    const bool tile = fits && team_lds(d, C, B, true) <= kTeamLds;
    if (!tile && (quads * 16 > 512 * 1024 || team_lds(d, C, B, false) > kTeamLds)) continue;
    const double kb = quads * 16 / 1024.0;
    double us = 3.0 + (W > 1 ? 1.0 + 0.05 * W : 0.0) + 0.15 * C / kOwn;
    if (!tile) us += kb / 20.0;  // read twice, through the L2
    else us += kb / 120.0 + (d.prob.batch > 0 && kb > 64 ? (kb - 64) / 40.0 : 0.0);  // the next rows arrive beside the update and the mix
    if (us < best_us) {
      best_us = us;
      best.W = W;
      best.C = C;
      best.tiles = tile ? 1 : 0;
      const int per = (C + kOwn - 1) / kOwn;
      best.per_lane = per <= 1 ? 1 : per <= 2 ? 2 : per <= 4 ? 4 : 8;
    }
  }
  return best;
}

size_t rfast_team_packet_bytes(const RfastTeam& t, int32_t n, const rfast_problem* prob) {
  return t.W > 0 ? (size_t)2 * n * t.W * rows_per_gradient(prob) * sizeof(u64) : 0;
}
// (a team holds kTeamMost chunks of 8 kOwn coordinates at most)
size_t rfast_team_sync_bytes(int32_t n, int64_t p, const rfast_problem* prob) {
  const bool any = (prob->kind == RFAST_OBJ_LEAST_SQUARES || prob->kind == RFAST_OBJ_LOGISTIC) && n * p <= (int64_t)kTeamMost * 8 * kOwn;
  return any ? (size_t)2 * n * p * 2 * sizeof(u64) : 0;
}
size_t rfast_team_flag_bytes(const RfastTeam& t, int32_t n) { return (size_t)n * t.W * kOwnWaves * kFlagWords * 4; }

// rounds: at most kBlockRounds with sync = false (their plan records are in c->d.blk_plan)
hipError_t rfast_launch_team(rfast_ctx* c, bool sync, int rounds, float gamma, const int32_t* d_batch_idx,
                             const int32_t* d_delay_R, const int32_t* d_delay_C) {
  const RfastTeam& t = c->team;
  if (t.W <= 0 || rounds < 1 || (!sync && (rounds > kBlockRounds || !c->d.blk_plan))) return hipErrorInvalidValue;
  TeamArgs a;
  a.rounds = rounds;
  a.W = t.W;
  a.C = t.C;
  a.B = rows_per_gradient(&c->d.prob);
  a.buffers = 1;
  a.gamma = gamma;
  a.base = c->team_base;
  a.batch_idx = c->d.prob.batch > 0 ? d_batch_idx : nullptr;
  a.delay_R = d_delay_R;
  a.delay_C = d_delay_C;
  a.packets = (u64*)c->team_packets;
  a.sync = (u64*)c->team_sync;
  a.flags = c->team_flags;
  team_begin(c, &a);
  return team_end(c, rounds, sync ? launch_team<true>(c, a) : launch_team<false>(c, a));
}
