// Several rounds per launch for softmax regression of small and moderate size: a team of workgroups per node, as in
// rfast_team.hip (residency, progress words, packets and why every wait ends are explained there).
//
// Workgroup (i, w) keeps FT tiles of 32 features (all K classes) of node i.  A wavefront owns a tile of 32 features x 32
// classes, in the very layout in which v_mfma_f32_32x32x16_bf16 leaves a 32 x 32 result (lane l: class l % 32, features
// 8 (v / 4) + 4 (l / 32) + v % 4 for v = 0 .. 15): the gradient comes out of the matrix cores where x, z, the stored
// sample and the running sum of the same coordinates already are.  A round of an active node:
//   mix          x' in registers; its bf16 rounding to LDS, class-major (8 consecutive features per operand)
//   forward      partial logits of all B sampled rows over the chunk's features, 32 x 32 tiles shared out over the
//                wavefronts; to the workgroup that looks after the row, as packets
//   sums         while they travel, or behind the backward product where they are not out yet: the running sums of the
//                in-neighbours, z + sum of a (sigma - sigma~)
//   softmax      workgroup w' adds the partial logits of its B / W rows (in the order of the chunks), forms
//                E = bf16((softmax - onehot) / B) and sends it to all of the team, two classes per packet
//   backward     G = X^T E from the rows in LDS (8 rows of one feature gathered per operand), then the tracker update
// Two exchanges of about a microsecond each, against four kernels of 4 to 14 us and the gaps between them.
//
// The partial logits are rounded to fp32 per chunk where the one-kernel form keeps one accumulator over all features;
// nothing else differs from rfast_softmax.hip.  Measured, us per round, before (four kernels) and now: 16 nodes, d 512,
// K 32, batch 64, heavy-ball buffer: 33.6 -> 12.2 (13.5 with one word for the sums that are out and those that are read, 12.9 with the sums waited for before the softmax); one agent of 16 per iteration, d 192: 20.6 -> 5.0.
//
// With 256 registers per lane the five arrays of a tile (x, z, sample, running sum, heavy-ball buffer: 64 or 80 registers)
// and the ring values in flight beside them do not all fit: 60 to 119 registers are spilled over the eight instantiations
// (184 to 328 B of scratch per lane), some of them reloaded between the parts of a round.
//
// What bounds it is the chain of trips through memory in the wavefronts that own tiles, so everything else is kept out of
// them as long as there are others (15.7 -> 13.6 us per round in the first case): the forward product, the softmax, row
// numbers and rows of the next round go to the wavefronts without a tile first; the barrier for the weights does not
// wait for the stores of v; progress words are read ahead on trips that are made anyway.
#include "rfast_team.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned short u16;
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

constexpr int kWaves = kTeamThreads / 64;
constexpr int kPad = 8;  // bf16 elements between the rows of Wt and Et in LDS

// bf16 elements of LDS: X tiles, Wt, Et
__host__ __device__ inline size_t x_elems(int B, int FT) { return (size_t)B * 32 * FT; }
__host__ __device__ inline size_t wt_elems(int K, int FT) { return (size_t)K * (32 * FT + kPad); }
__host__ __device__ inline size_t et_elems(int K, int B) { return (size_t)K * (B + kPad); }

// The rounds of a launch by one workgroup (see team_complete).  rowi: [B] words of LDS, et: [K][B + kPad].
template <int K>
__device__ __forceinline__ void alone(const RfastDev& s, const TeamArgs& a, int* rowi, u16* et) {
  const int n = s.n, B = a.B, d = s.prob.d, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool sampled = a.batch_idx != nullptr;
  const float inv_b = 1.0f / (float)B;
  auto value = [](u16 h) { return __uint_as_float((uint32_t)h << 16); };
  for (int q = 0; q < a.rounds; ++q) {
    const int32_t* rec = s.blk_plan + (size_t)q * (n + s.eR + s.eC + 1);
    for (int i = 0; i < n; ++i) {
      const int t_old = rec[i] & 0x3FFFFFFF;
      if (rec[i] < 0) {
        const u16* pool = (const u16*)s.prob.data0 + (size_t)i * s.prob.samples * d;
        const float* x = s.x + (size_t)i * s.p;
        alone_mix(s, i, (t_old + 1) % s.M, a.gamma, rec + n);
        for (int b = tid; b < B; b += kTeamThreads) rowi[b] = sampled ? team_row(s, a, false, i, q, a.batch_idx[((size_t)q * n + i) * B + b], true) : b;
        __syncthreads();  // x and the row numbers
        // logits in the packets' place (as packets of round 0, which nobody waits for)
        for (int f = tid; f < B * K; f += kTeamThreads) {
          const int b = f / K, k = f - b * K;
          float acc = 0.f;
          for (int c = 0; c < d; ++c) acc = fmaf(value(pool[(size_t)rowi[b] * d + c]), value(rfast_f32_to_bf16(x[(size_t)c * K + k])), acc);
          a.packets[f] = __float_as_uint(acc);
        }
        __syncthreads();
        for (int b = wave; b < B; b += kTeamThreads / 64) {
          int lab = ((const int32_t*)s.prob.data1)[(size_t)i * s.prob.samples + rowi[b]];
          if (lab < 0 || lab >= K) {
            if (lane == 0) record_error(s.err, RFAST_ERANGE, first_round(s, a, false) + q, 3, i);
            lab = lab < 0 ? 0 : K - 1;
          }
          float lg[2], mx = -INFINITY, sum = 0.f;
          for (int u = 0; u < 2; ++u) {
            lg[u] = lane + 64 * u < K ? __uint_as_float((unsigned)a.packets[b * K + lane + 64 * u]) : -INFINITY;
            mx = fmaxf(mx, lg[u]);
          }
          for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
          for (int u = 0; u < 2; ++u) {
            lg[u] = lane + 64 * u < K ? __expf(lg[u] - mx) : 0.f;
            sum += lg[u];
          }
          for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
          for (int u = 0; u < 2; ++u) {
            const int k = lane + 64 * u;
            if (k < K) et[(size_t)k * (B + kPad) + b] = rfast_f32_to_bf16((lg[u] * (1.0f / sum) - (k == lab ? 1.0f : 0.0f)) * inv_b);
          }
        }
        __syncthreads();
        alone_track(s, i, t_old, rec + n + s.eR, [&](int64_t at) {
          const int f = (int)(at / K), k = (int)(at - (int64_t)f * K);
          float acc = 0.f;
          for (int b = 0; b < B; ++b) acc = fmaf(value(pool[(size_t)rowi[b] * d + f]), value(et[(size_t)k * (B + kPad) + b]), acc);
          return s.wd != 0.f ? fmaf(s.wd, x[at], acc) : acc;
        });
        __syncthreads();  // E and the row numbers may be overwritten
      }
      alone_save(s, i, rec + n + s.eR);
    }
  }
}

// a.C: feature tiles per chunk (1, 2, 4 or 8)
template <int KT, bool MOM>
__global__ void __launch_bounds__(kTeamThreads) rfast_team_softmax_kernel(RfastDev s, TeamArgs a) {
  constexpr int K = 32 * KT;
  extern __shared__ float4 lds4[];
  __shared__ u64 act_mask[kBlockRounds / 64], ev_mask[kBlockRounds / 64];
  __shared__ int verdict;
  if (threadIdx.x == 0) team_arrive(a);
  const int n = s.n, M = s.M, W = a.W, B = a.B, FT = a.C, d = s.prob.d;
  const int64_t p = s.p;
  const int i = blockIdx.x / W, w = blockIdx.x - i * W;
  const int DT = d / 32, ft0 = w * FT, FTw = DT - ft0 < FT ? DT - ft0 : FT;  // feature tiles of the node, first and number of this chunk's
  const int Fc = 32 * FT, nc = 4 * FT;                                       // features of a chunk, 16-byte pieces of a row of it
  const int R = (B + W - 1) / W;                                             // rows a workgroup looks after
  const int r0 = w * R, r1 = r0 + R < B ? r0 + R : B;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lo = lane & 31, hi = lane >> 5;
  const bool sampled = a.batch_idx != nullptr;
  u16* const xt = reinterpret_cast<u16*>(lds4);                              // [buffers][B][Fc]
  u16* const wt = xt + a.buffers * x_elems(B, FT);                           // [K][Fc + kPad]
  u16* const et = wt + wt_elems(K, FT);                                      // [K][B + kPad]
  int* const rowi = reinterpret_cast<int*>(et + et_elems(K, B));             // [2][B] sampled rows of this active round and the next
  int* const nodew = rowi + 2 * B;                                             // [kBlockRounds] node words
  const int ftw = wave / KT, kt = wave - ftw * KT;                           // the wavefront's tile
  const bool owner = ftw < FTw;
  const u16* const pool = (const u16*)s.prob.data0 + (size_t)i * s.prob.samples * d + 32 * ft0;
  const int32_t* const labels = (const int32_t*)s.prob.data1 + (size_t)i * s.prob.samples;

  // ---- the rounds in which the node does something
  const int W1 = n + s.eR + s.eC + 1;
  const int round0 = first_round(s, a, false);
  {
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
  const int re0 = s.r_ptr[i], dR = s.r_ptr[i + 1] - re0, ce0 = s.c_ptr[i], dI = s.c_ptr[i + 1] - ce0;
  const int ro0 = s.ro_ptr[i], dRo = s.ro_ptr[i + 1] - ro0, co0 = s.co_ptr[i], dCo = s.co_ptr[i + 1] - co0;
  const float r_self = s.r_self[i], c_self = s.c_self[i];
  int r_src = 0, c_src = 0, r_dst = 0, c_dst = 0;
  float r_w = 0.f, c_w = 0.f;
  if (lane < dR) { r_src = s.r_src[re0 + lane]; r_w = s.r_w[re0 + lane]; }
  if (lane < dI) { c_src = s.c_src[ce0 + lane]; c_w = s.c_w[ce0 + lane]; }
  if (lane < dRo) r_dst = s.r_dst[s.ro_eid[ro0 + lane]];
  if (lane < dCo) c_dst = s.c_dst[s.co_eid[co0 + lane]];
  auto flag_of = [&](int node, int word) { return a.flags + ((size_t)(node * DT + ft0 + ftw) * KT + kt) * kFlagWords + word; };
  const float wd = s.wd, inv_b = 1.0f / (float)B;
  __syncthreads();
  const int t0 = nodew[0] & 0x3FFFFFFF;

  // ---- the tile: element v of a lane is coordinate tile0 + step(v) + at, the first two the same for all lanes
  const size_t tile0 = (size_t)(32 * (ft0 + ftw)) * K + 32 * kt;
  const unsigned at = (unsigned)(4 * hi * K + lo);
  auto step = [&](int v) { return (size_t)((8 * (v >> 2) + (v & 3)) * K); };
  float x[16], z[16], g[16], sc[16], m[16];
  if (owner) {
    const size_t off = (size_t)i * p + tile0;
    const float* ring = s.sigma_ring + ((size_t)i * M + t0 % M) * p + tile0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      x[v] = (s.x + off + step(v))[at];
      z[v] = (s.z + off + step(v))[at];
      g[v] = (s.g + (size_t)(t0 & 1) * n * p + off + step(v))[at];
      sc[v] = (ring + step(v))[at];
      if (MOM) m[v] = (s.mom + off + step(v))[at];
    }
  }
  bool dead = false;
  auto wait2 = [&](const unsigned* f1, int need1, const unsigned* f2, int need2, unsigned v1, unsigned v2) {
    wait_progress(a, false, i, f1, need1, f2, need2, v1, v2, &dead);
  };

  // ---- rows of X into LDS, straight from memory: 16-byte piece q of the tile is piece pos = q mod nc of row q / nc and
  // holds features 8 c .. 8 c + 7 of the chunk, c = pos ^ swz(row), so that the 32 rows that an operand of the forward
  // product takes at one c lie on different banks
  const int nc_sh = 2 + (FT == 1 ? 0 : FT == 2 ? 1 : FT == 4 ? 2 : 3);
  const int sw_sh = nc_sh >= 4 ? 0 : 4 - nc_sh, sw_mask = nc < 16 ? nc - 1 : 15;
  auto swz = [&](int b) { return (b >> sw_sh) & sw_mask; };
  // Wavefronts without a tile fetch them, if there are any: loads return in order, and one that polls would poll behind
  // the rows.
  const int busy = FTw * KT < kWaves ? FTw * KT : 0, idle = kWaves - busy;
  auto load_x = [&](const int* rows, u16* dst) {
    const int total = wave >= busy ? B << nc_sh : 0;
    for (int q0 = 64 * (wave - busy); q0 < total; q0 += 64 * idle) {
      const int q = q0 + lane;
      const int b = q >> nc_sh, c = (q & (nc - 1)) ^ swz(b);
      if (q < total && c < 4 * FTw) {
        const int row = sampled ? rows[b] : b;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(pool + (size_t)row * d + 8 * c),
                                         (__attribute__((address_space(3))) void*)(dst + (size_t)q0 * 8), 16, 0, 0);
      }
    }
  };
  const int rounds = a.rounds;
  auto next_active = [&](int from) { return next_bit(act_mask, from); };
  auto next_event = [&](int from) { return next_bit(ev_mask, from); };
  auto fetch_rows = [&](int q, int* to) {
    for (int b = kTeamThreads - 1 - tid; b < B; b += kTeamThreads) to[b] = team_row(s, a, false, i, q, a.batch_idx[((size_t)q * n + i) * B + b], w == 0);
  };
  int parity = 0;
  {
    const int qa = next_active(0);
    if (sampled && qa < rounds) fetch_rows(qa, rowi);
    if (sampled) __syncthreads();
    if (qa < rounds) load_x(rowi, xt);
  }
  int q = next_event(0), q_prev = -1;
  int rw_n = 0, cw_n = 0, rd_n = 0, cd_n = 0;
  auto fetch_plan = [&](int at) {
    if (at >= rounds) return;
    const int32_t* rec = s.blk_plan + (size_t)at * W1;
    if (lane < dR) { rw_n = rec[n + re0 + lane]; rd_n = a.delay_R[(size_t)at * s.eR + re0 + lane]; }
    if (lane < dI) { cw_n = rec[n + s.eR + ce0 + lane]; cd_n = a.delay_C[(size_t)at * s.eC + ce0 + lane]; }
  };
  auto clamped = [&](int dl) { return dl < 0 ? 0 : (dl > s.d_max ? s.d_max : dl); };
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
      alone<K>(k.s, k.a, rowi, et);
    }
    return;
  }
  if (owner) {
    if (lane == 0) {
      put32(flag_of(i, 0), a.base + (unsigned)(q < rounds ? q : rounds));
      put32(flag_of(i, 1), a.base + (unsigned)(q < rounds ? q : rounds));
      put32(flag_of(i, 2), a.base + (unsigned)(q < rounds ? q : rounds));
    }
  }
  unsigned seen_r = a.base, seen_d = a.base;  // the words that the next mix waits for, as read ahead
  const unsigned r_magic = 0xFFFFFFFFu / (unsigned)R;
  u64* const e_packets = a.packets + (size_t)2 * n * W * W * R * K;  // behind the partial logits

  while (q < rounds) {
    dead = __any(dead);
    const int q_next = next_event(q + 1);
    const unsigned done_word = a.base + (unsigned)(q_next < rounds ? q_next : rounds), tag = a.base + (unsigned)q + 1u;
    const int word = nodew[q];
    const bool active = word < 0;
    const int t_old = word & 0x3FFFFFFF;
    const int rword = rw_n, cword = cw_n, rneed = q - clamped(rd_n), cneed = q - clamped(cd_n);
    const int slot_new = (t_old + 1) % M;
    float z_half[16];
    if (owner && active) {
      // ---- S1, S2a, S3 (v half)
      wait2(lane < dR ? flag_of(r_src, 0) : nullptr, rneed, lane < dRo ? flag_of(r_dst, 0) : nullptr, q_prev + 1, seen_r, seen_d);
      float vn[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float dir = z[v];
        if (MOM) dir = m[v] = fmaf(s.beta, m[v], z[v]);
        vn[v] = fmaf(-a.gamma, dir, x[v]);
        x[v] = r_self * vn[v];
      }
      float* own_v = s.v_ring + ((size_t)i * M + slot_new) * p + tile0;
      constexpr int KB = 4;
      for (int e0 = 0; e0 < dR; e0 += KB) {
        float vb[KB][16];
#pragma unroll
        for (int u = 0; u < KB; ++u)
          if (e0 + u < dR) {
            const float* src = s.v_ring + ((size_t)lane_value(r_src, e0 + u) * M + lane_value(rword, e0 + u)) * p + tile0;
#pragma unroll
            for (int v = 0; v < 16; ++v) vb[u][v] = get_f(src + step(v) + at);
          }
#pragma unroll
        for (int u = 0; u < KB; ++u)
          if (e0 + u < dR) {
            const float wt_e = lane_value(r_w, e0 + u);
#pragma unroll
            for (int v = 0; v < 16; ++v) x[v] = fmaf(wt_e, vb[u][v], x[v]);
          }
      }
      // the weights as bf16, class-major: four consecutive features of the lane's class per store
      u16* to = wt + (size_t)(32 * kt + lo) * (Fc + kPad) + 32 * ftw + 4 * hi;
#pragma unroll
      for (int v = 0; v < 16; v += 4) {
        uint2 pk;
        pk.x = rfast_f32_to_bf16(x[v]) | ((uint32_t)rfast_f32_to_bf16(x[v + 1]) << 16);
        pk.y = rfast_f32_to_bf16(x[v + 2]) | ((uint32_t)rfast_f32_to_bf16(x[v + 3]) << 16);
        *reinterpret_cast<uint2*>(to + 2 * v) = pk;
      }
      drain();  // (rows that this wavefront fetched are in LDS; the loads of the mix were issued behind them)
#pragma unroll
      for (int v = 0; v < 16; ++v) put_f(own_v + step(v) + at, vn[v]);
    }
    if (active) {
      const int* rows = rowi + (parity ? B : 0);
      const u16* X = xt + (a.buffers > 1 && parity ? x_elems(B, FT) : 0);
      u16* X_next = xt + (a.buffers > 1 && !parity ? x_elems(B, FT) : 0);
      const int qa = next_active(q + 1);
      if (!owner) drain();  // the rows on their way into LDS have arrived
      __syncthreads();  // weights and rows are in LDS
      const int back = kWaves - 1 - wave;  // forward and softmax: the wavefronts without a tile first
      unsigned seen_c = a.base, seen_o = a.base;
      if (owner) {
        // v is out; the words that the running sums wait for are read on the same trip
        seen_c = peek(a, lane < dI ? flag_of(c_src, 1) : nullptr, cneed);
        seen_o = peek(a, lane < dCo ? flag_of(c_dst, 2) : nullptr, q_prev + 1);
        drain();
        if (lane == 0) put32(flag_of(i, 0), done_word);
      }
      // ---- forward: partial logits, 32 rows x 32 classes at a time
      for (int tl = back; tl < (B / 32) * KT; tl += kWaves) {
        const int bt = tl / KT, k2 = tl - bt * KT;
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        const int b = 32 * bt + lo;
        const u16* xr = X + (size_t)b * Fc;
        const u16* wr = wt + (size_t)(32 * k2 + lo) * (Fc + kPad) + 8 * hi;
        const int sw = swz(b);
        for (int st = 0; st < 2 * FTw; ++st) {
          const bf16x8 af = *reinterpret_cast<const bf16x8*>(xr + 8 * ((2 * st + hi) ^ sw));
          const bf16x8 bf = *reinterpret_cast<const bf16x8*>(wr + 16 * st);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bf, acc, 0, 0, 0);
        }
        // packet of row b and class k for the workgroup that looks after b
        u64* base = a.packets + (((size_t)parity * n + i) * W * W + w) * R * K + 32 * k2 + lo;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int bb = 32 * bt + 8 * (v >> 2) + 4 * hi + (v & 3);
          int dest = (int)__umulhi((unsigned)bb, r_magic);
          if (bb - dest * R >= R) ++dest;
          put64(base + ((size_t)dest * W * R + (bb - dest * R)) * K, (u64)tag << 32 | __float_as_uint(acc[v]));
        }
      }
      // ---- S2b without the gradient, S4: z + sum over the in-edges of C, two live edges at a time; where the words say that they are
      // not out yet, behind the gradient
      auto sums = [&] {
#pragma unroll
        for (int v = 0; v < 16; ++v) z_half[v] = z[v];
        u64 live = __ballot(lane < dI && (cword & (1 << 16)));
        while (live) {
          float sg[2][16], rt[2][16];
          int eu[2] = {0, 0};
          bool have[2] = {false, false};
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (live) {
              const int e = __ffsll((long long)live) - 1;
              live &= live - 1;
              eu[u] = e;
              have[u] = true;
              const int pl = lane_value(cword, e), prev = (pl >> 8) & 0xFF;
              const float* ring = s.sigma_ring + (size_t)lane_value(c_src, e) * M * p + tile0;
              const float* cur = ring + (size_t)(pl & 0xFF) * p;
              const float* last = prev != 0xFF ? ring + (size_t)prev * p : s.rho_tilde + (size_t)(ce0 + e) * p + tile0;
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                sg[u][v] = get_f(cur + step(v) + at);
                rt[u][v] = get_f(last + step(v) + at);
              }
            }
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (have[u]) {
              const int pl = lane_value(cword, eu[u]);
              const float ce = lane_value(c_w, eu[u]);
              const bool in_ring = ((pl >> 8) & 0xFF) != 0xFF;
#pragma unroll
              for (int v = 0; v < 16; ++v) z_half[v] = track_edge(z_half[v], ce, sg[u][v], rt[u][v], in_ring);
              if (pl & (1 << 17)) {  // consumed, and leaving its sender's ring
                float* saved = s.rho_tilde + (size_t)(ce0 + eu[u]) * p + tile0;
#pragma unroll
                for (int v = 0; v < 16; ++v) put_f(saved + step(v) + at, ce * sg[u][v]);
              }
            }
        }
        // what this round reads of others' sums is read, unless a buffer is still to be saved
        if (!__any(lane < dI && (cword & (1 << 18)))) {
          drain();
          if (lane == 0) put32(flag_of(i, 2), done_word);
        }
      };
      bool early = false;
      if (owner) {
        early = !__any((lane < dI && cneed > 0 && (int)(seen_c - a.base) < cneed) || (lane < dCo && (int)(seen_o - a.base) <= q_prev));
        if (early) sums();
        fetch_plan(q_next);
      }
      // ---- softmax of the workgroup's rows: K lanes (two classes per lane above 64) per row
      {
        constexpr int G = K <= 32 ? 32 : 64, PL = K > 64 ? 2 : 1;  // lanes of a row, classes of a lane
        const int per = 64 / G, gl = lane & (G - 1);
        for (int r = r0 + back * per + lane / G; r < r1; r += kWaves * per) {
          int lab = labels[sampled ? rows[r] : r];
          float lg[PL];
          const u64* src = a.packets + (((size_t)parity * n + i) * W + w) * W * R * K + (size_t)(r - r0) * K + gl;
#pragma unroll
          for (int u = 0; u < PL; ++u) {
            lg[u] = -INFINITY;
            if (gl + 64 * u < K) {
              float sum = 0.f;
              for (int w0 = 0; w0 < W; w0 += 8) {
                u64 got[8];
                for (int spin = 0;; ++spin) {
                  bool ok = true;
#pragma unroll
                  for (int c = 0; c < 8; ++c)
                    if (w0 + c < W) got[c] = get64(src + (size_t)(w0 + c) * R * K + 64 * u);
#pragma unroll
                  for (int c = 0; c < 8; ++c)
                    if (w0 + c < W) ok = ok && (unsigned)(got[c] >> 32) == tag;
                  if (ok || dead) break;
                  if (spin >= a.wait_polls) {
                    dead = true;
                    report_wait(false, i);
                    break;
                  }
                }
#pragma unroll
                for (int c = 0; c < 8; ++c)
                  if (w0 + c < W) sum = w0 + c == 0 ? __uint_as_float((unsigned)got[c]) : sum + __uint_as_float((unsigned)got[c]);
              }
              lg[u] = sum;
            }
          }
          float mx = PL == 2 ? fmaxf(lg[0], lg[PL - 1]) : lg[0];
#pragma unroll
          for (int o = G / 2; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
          float ex[PL], sum = 0.f;
#pragma unroll
          for (int u = 0; u < PL; ++u) {
            ex[u] = gl + 64 * u < K ? __expf(lg[u] - mx) : 0.f;
            sum += ex[u];
          }
#pragma unroll
          for (int o = G / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
          const float inv = 1.0f / sum;
          if (lab < 0 || lab >= K) {  // clamped and reported, like a sample row
            const TeamKernelArgs& k = team_kernel_args();
            if (gl == 0) record_error(k.s.err, RFAST_ERANGE, first_round(k.s, k.a, false) + q, 3, i);
            lab = lab < 0 ? 0 : K - 1;
          }
#pragma unroll
          for (int u = 0; u < PL; ++u) {
            const int k = gl + 64 * u;
            const uint32_t mine = rfast_f32_to_bf16((ex[u] * inv - (k == lab ? 1.0f : 0.0f)) * inv_b);
            const uint32_t other = __shfl_xor(mine, 1, 64);
            if ((k & 1) == 0 && k < K)
              put64(e_packets + (((size_t)parity * n + i) * B + r) * (K / 2) + k / 2, (u64)tag << 32 | mine | other << 16);
          }
        }
      }
      if (sampled && qa < rounds) fetch_rows(qa, rowi + (parity ? 0 : B));  // while E travels
      // ---- E of all rows, class-major into LDS
      {
        const u64* src = e_packets + ((size_t)parity * n + i) * B * (K / 2);
        const int total = B * (K / 2);
        for (int f0 = 0; f0 < total; f0 += 8 * kTeamThreads) {
          u64 got[8];
          for (int spin = 0;; ++spin) {
            bool ok = true;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
              const int f = f0 + c * kTeamThreads + tid;
              if (f < total) got[c] = get64(src + f);
            }
#pragma unroll
            for (int c = 0; c < 8; ++c)
              if (f0 + c * kTeamThreads + tid < total) ok = ok && (unsigned)(got[c] >> 32) == tag;
            if (ok || dead) break;
            if (spin >= a.wait_polls) {
              dead = true;
              report_wait(false, i);
              break;
            }
          }
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            const int f = f0 + c * kTeamThreads + tid;
            if (f < total) {
              const int b = f / (K / 2), k = 2 * (f - b * (K / 2));
              et[(size_t)k * (B + kPad) + b] = (u16)got[c];
              et[(size_t)(k + 1) * (B + kPad) + b] = (u16)(got[c] >> 16);
            }
          }
        }
      }
      __syncthreads();  // E, and the row numbers of the next active round
      if (sampled && qa < rounds && a.buffers > 1) load_x(rowi + (parity ? 0 : B), X_next);
      if (owner) {
        // ---- backward: G of the tile, 16 rows at a time
        f32x16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        const int f = 32 * ftw + lo, c = f >> 3, fo = f & 7;
        const u16* er = et + (size_t)(32 * kt + lo) * (B + kPad) + 8 * hi;
        for (int b0 = 0; b0 < B; b0 += 16) {
          u16x8 col;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int b = b0 + 8 * hi + j;
            col[j] = X[(size_t)b * Fc + 8 * (c ^ swz(b)) + fo];
          }
          const bf16x8 bf = *reinterpret_cast<const bf16x8*>(er + b0);
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, col), bf, acc, 0, 0, 0);
        }
        if (!early) {
          wait2(lane < dI ? flag_of(c_src, 1) : nullptr, cneed, lane < dCo ? flag_of(c_dst, 2) : nullptr, q_prev + 1, a.base, a.base);
          sums();
        }
        // ---- S2b, S2c, S3 (rho half)
        float* own_s = s.sigma_ring + ((size_t)i * M + slot_new) * p + tile0;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float g_new = wd != 0.f ? fmaf(wd, x[v], acc[v]) : acc[v];
          const float zh = (z_half[v] + g_new) - g[v];
          g[v] = g_new;
          z[v] = c_self * zh;
          if (dCo > 0) {
            sc[v] += zh;
            put_f(own_s + step(v) + at, sc[v]);
          }
        }
      }
      if (a.buffers == 1 && sampled && qa < rounds) {
        __syncthreads();  // nobody reads the rows of this round any more
        load_x(rowi + (parity ? 0 : B), X_next);
      }
      parity ^= 1;
      q_prev = q;
    } else if (owner) {
      fetch_plan(q_next);
    }
    if (owner) {
      // S4 for buffers whose version leaves the sender's ring in this round without being consumed
      u64 leaving = __ballot(lane < dI && (cword & (1 << 18)));
      if (!active && leaving) wait2(lane < dI ? flag_of(c_src, 1) : nullptr, cneed, nullptr, 0, a.base, a.base);
      while (leaving) {
        const int e = __ffsll((long long)leaving) - 1;
        leaving &= leaving - 1;
        const float* ring = s.sigma_ring + ((size_t)lane_value(c_src, e) * M + (lane_value(cword, e) & 0xFF)) * p + tile0;
        float* saved = s.rho_tilde + (size_t)(ce0 + e) * p + tile0;
        const float ce = lane_value(c_w, e);
        float val[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) val[v] = get_f(ring + step(v) + at);
#pragma unroll
        for (int v = 0; v < 16; ++v) put_f(saved + step(v) + at, ce * val[v]);
      }
      // the words that the next mix waits for are read on the trip that the stores take anyway
      seen_r = peek(a, lane < dR ? flag_of(r_src, 0) : nullptr, q_next - clamped(rd_n));
      seen_d = peek(a, lane < dRo ? flag_of(r_dst, 0) : nullptr, q_prev + 1);
      drain();
      if (lane == 0) {
        if (!active) put32(flag_of(i, 0), done_word);
        put32(flag_of(i, 1), done_word);
        put32(flag_of(i, 2), done_word);
      }
    }
    q = q_next;
  }

  // ---- write-back
  const int t_end = s.t[i];
  if (owner && q_prev >= 0) {
    const size_t off = (size_t)i * p + tile0;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      (s.x + off + step(v))[at] = x[v];
      (s.z + off + step(v))[at] = z[v];
      (s.g + (size_t)(t_end & 1) * n * p + off + step(v))[at] = g[v];
      if (MOM) (s.mom + off + step(v))[at] = m[v];
    }
  }
}

size_t softmax_lds(const rfast_problem* prob, int B, int FT, int buffers) {
  return 2 * (buffers * x_elems(B, FT) + wt_elems(prob->K, FT) + et_elems(prob->K, B)) + ((size_t)2 * B + kBlockRounds) * 4;
}

int rows_per_gradient(const rfast_problem* prob) { return prob->batch > 0 ? prob->batch : prob->samples; }

template <int KT, bool MOM>
hipError_t launch(rfast_ctx* c, const TeamArgs& a) {
  static bool raised = false;
  if (!raised) {  // more than 64 KB of dynamic LDS has to be asked for once per kernel
    const hipError_t e = hipFuncSetAttribute((const void*)rfast_team_softmax_kernel<KT, MOM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kTeamLds);
    if (e != hipSuccess) return e;
    raised = true;
  }
  hipLaunchKernelGGL((rfast_team_softmax_kernel<KT, MOM>), dim3((unsigned)(c->d.n * a.W)), dim3(kTeamThreads),
                     softmax_lds(&c->d.prob, a.B, a.C, a.buffers), c->stream, c->d, a);
  return hipGetLastError();
}
template <int KT>
hipError_t launch(rfast_ctx* c, const TeamArgs& a) {
  return c->d.mom ? launch<KT, true>(c, a) : launch<KT, false>(c, a);
}

}  // namespace

// The team of a softmax problem: W workgroups of C feature tiles each, as many as the compute units hold but no more than
// eight tiles of 32 x 32 per workgroup, one per wavefront.  More workgroups: fewer tiles to move for each, more partial
// logits to add up.
RfastTeam rfast_team_softmax_shape(const RfastDev& d, int max_degree, int max_out_degree_r, int compute_units) {
  RfastTeam best;
  if (d.prob.kind != RFAST_OBJ_SOFTMAX_BF16) return best;
  if (max_degree > 64 || max_out_degree_r > 64 || d.n > compute_units || d.M > 254) return best;  // one edge per lane
  const int B = rows_per_gradient(&d.prob), KT = d.prob.K / 32, DT = d.prob.d / 32;
  double best_us = 1e30;
  for (int FT = 1; FT * KT <= kWaves; FT *= 2) {
    const int W = (DT + FT - 1) / FT;
    if ((int64_t)W * d.n > compute_units || W > B) continue;
    int buffers = d.prob.batch > 0 ? 2 : 1;  // two: the rows of the next round arrive during this one (all rows: they stay)
    while (buffers > 0 && softmax_lds(&d.prob, B, FT, buffers) > kTeamLds) --buffers;
    if (buffers == 0) continue;
    const double us = 6.0 + 0.1 * W + 0.5 * FT * KT;
    if (us < best_us) {
      best_us = us;
      best.W = W;
      best.C = FT;
      best.tiles = buffers;
      best.per_lane = 16;
    }
  }
  return best;
}

// partial logits [2][n][destination W][source W][rows][K], then E [2][n][B][K / 2]
size_t rfast_team_softmax_packet_bytes(const RfastTeam& t, int32_t n, const rfast_problem* prob) {
  if (t.W <= 0) return 0;
  const size_t B = rows_per_gradient(prob), R = (B + t.W - 1) / t.W;
  return ((size_t)2 * n * t.W * t.W * R * prob->K + (size_t)2 * n * B * (prob->K / 2)) * sizeof(u64);
}
size_t rfast_team_softmax_flag_bytes(const RfastTeam& t, int32_t n, const rfast_problem* prob) {
  return t.W > 0 ? (size_t)n * (prob->d / 32) * (prob->K / 32) * kFlagWords * 4 : 0;
}

hipError_t rfast_launch_team_softmax(rfast_ctx* c, int rounds, float gamma, const int32_t* d_batch_idx,
                                     const int32_t* d_delay_R, const int32_t* d_delay_C) {
  const RfastTeam& t = c->team;
  if (t.W <= 0 || rounds < 1 || rounds > kBlockRounds || !c->d.blk_plan) return hipErrorInvalidValue;
  TeamArgs a;
  a.rounds = rounds;
  a.W = t.W;
  a.C = t.C;
  a.B = rows_per_gradient(&c->d.prob);
  a.buffers = t.tiles;
  a.gamma = gamma;
  a.base = c->team_base;
  a.batch_idx = c->d.prob.batch > 0 ? d_batch_idx : nullptr;
  a.delay_R = d_delay_R;
  a.delay_C = d_delay_C;
  a.packets = (u64*)c->team_packets;
  a.flags = c->team_flags;
  team_begin(c, &a);
  switch (c->d.prob.K / 32) {
    case 1: return team_end(c, rounds, launch<1>(c, a));
    case 2: return team_end(c, rounds, launch<2>(c, a));
    case 3: return team_end(c, rounds, launch<3>(c, a));
    default: return team_end(c, rounds, launch<4>(c, a));
  }
}
