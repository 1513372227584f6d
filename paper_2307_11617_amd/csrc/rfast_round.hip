// State-update kernels of one activation round (Algorithm 1, steps S1-S5).
//
// One work item = (active node, tile of coordinates).  Everything is
// elementwise in the coordinate k, has no reuse and moves 4 bytes per ~1 flop,
// so the kernels are pure HBM streams: every access is a float4 per lane
// (1 KiB per wavefront instruction), loads of one phase are issued back to back
// before their first use, and inactive nodes cost nothing.
//
//   FUSED  separable objective (diagonal quadratic): S1, S2a, gradient, S2b,
//          S2c, S3, S4 in one pass.
//   MIX    S1, S2a and the v half of S3; the gradient kernels run next.
//   TRACK  S2b, S2c, the rho half of S3, S4.
//
// The per-edge running sums rho_li of S2c are kept as ONE running sum per sender,
// sigma_i = sum of z_half, with rho_li = a_li * sigma_i formed by the receiver:
// algebraically identical to the per-edge recursion, bit-identical when a_li is
// a power of two, and it replaces dO reads + dO writes per coordinate by 1 + 1.
#include "rfast_internal.h"
#include "rfast_vec.h"

namespace {

constexpr int kThreads = 256;

// ------------------------------------------------------------------- kernel
// A value that is the same in all lanes, as the compiler should know (it takes what is read after a store through a
// vector load, and would form every address and branch per lane).
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// An element of the graph or of the round's plan.  No kernel here writes these, which the compiler cannot see past the
// stores of the state; said through the address space they are scalar loads wherever the index is uniform.
template <class T> __device__ inline T fixed(const T* p) {
  return *(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

// What is read from another node's ring.  Its other readers run beside this one, and find the line in L2 or behind it if
// it came there by an ordinary load; everything else a pass touches once, and streams past (V<-4>, V<-5>).  Measured, us
// per round, rings streamed too -> rings cached -> also the rings' stores and z cached -> everything: 128 nodes of an
// exponential graph, p 100000: 100.7 -> 81.5 -> 82.5 -> 87.4; softmax 128 x 131072: 176.8 -> 161.7 -> 168.0 -> 173.6;
// mesh of 36, p 250001: 51.9 -> 45.9 -> 46.4 -> 47.6; tree of 64, p 1 M (little to share): 272 -> 264 -> 281 -> 291;
// 16 nodes of a bidirectional ring, p 11.2 M: 1529 -> 1514 -> 1571 -> 1648.
template <int VEC> using Ring = V<(VEC == -4 ? 4 : VEC == -5 ? 5 : VEC)>;

// Loads of one live in-edge of C (plan word pl): the running sum being consumed and the one
// consumed last time (rho~ of S4), which is read from the sender's ring while it is still there.
template <int VEC>
__device__ inline void load_edge(const RfastDev& s, int e, int src, int pl, int M, int64_t p, int64_t k, typename V<VEC>::T* sg,
                                 typename V<VEC>::T* rt) {
  const float* ring = s.sigma_ring + (size_t)src * M * p + k;
  const int prev = (pl >> 8) & 0xFF;
  const float* last = prev != 0xFF ? ring + (size_t)prev * p : s.rho_tilde + (size_t)e * p + k;
  *sg = Ring<VEC>::ld(ring + (size_t)(pl & 0xFF) * p);
  *rt = Ring<VEC>::ld(last);
}

// Softmax objective: the GEMMs read the weights as bf16, 8 consecutive features of one class per
// 16-byte unit (layout [d/8][K][8]).  The 1024 coordinates of one tile are 1024/K whole features
// x K classes, i.e. exactly the elements [1024*tile, 1024*tile + 1024) of that layout in another
// order: permute through LDS and write them out coalesced, instead of a pass that re-reads x.
template <int VEC>
__device__ inline void emit_bf16_blocked(const RfastDev& s, int i, int tile, typename V<VEC>::T x_new) {
  __shared__ unsigned short perm[kThreads * 4];
  const int K = s.prob.K;
  const int l = threadIdx.x * 4, f = l / K, k0 = l % K;
  unsigned short* dst = perm + (f >> 3) * (8 * K) + k0 * 8 + (f & 7);
  const float4 w = *reinterpret_cast<const float4*>(&x_new);
  dst[0] = rfast_f32_to_bf16(w.x);
  dst[8] = rfast_f32_to_bf16(w.y);
  dst[16] = rfast_f32_to_bf16(w.z);
  dst[24] = rfast_f32_to_bf16(w.w);
  __syncthreads();
  unsigned short* wt = (unsigned short*)s.gscratch + (size_t)i * s.p + (size_t)tile * (kThreads * 4);
  *reinterpret_cast<uint2*>(wt + l) = *reinterpret_cast<const uint2*>(perm + l);
}

// MOM: the optimizer variant's heavy-ball buffer is in use (a template flag so that the
// plain method carries neither the branch nor the registers).
// KB: in-edge loads kept in flight per phase.  8 costs 146 registers (3 wavefronts per SIMD), 4 costs
// 91 (5 wavefronts): graphs with many in-edges per node want the deeper batch, graphs with few want
// the wavefronts (measured: bidirectional ring 1.53 vs 1.59 ms with 8 vs 4, tree/star 0.293 vs 0.274).
// DEEP: nodes may have more in-edges than one batch.  What the loop over further batches reads ahead costs the one-pass
// form up to 31 registers (heavy-ball buffer, batches of eight: 179 against 148, 2 against 3 wavefronts per SIMD), so
// graphs without such nodes go without it: 16 nodes of a bidirectional ring, p 11.2 M, heavy-ball: 1845 -> 1799 us per
// round.  The two-pass forms lose nothing by it (128 nodes, in-degree 7, softmax: 177.5 us per round with, 178.7 without).
template <int MODE, int VEC, bool MOM, int KB, bool DEEP, bool MANY = false>
__device__ inline void state_update(const RfastDev& s, float gamma, int2 slot, int tile, int64_t k) {
  using T = typename V<VEC>::T;
  constexpr bool kMix = MODE != RFAST_MODE_TRACK, kTrack = MODE != RFAST_MODE_MIX;
  const int i = slot.x;
  auto at = [](auto* q) {  // (the one-pass kernels have no stores ahead of most of these, and fewer registers to spare)
    if constexpr (MANY) return fixed(q);
    else return *q;
  };
  const int64_t p = s.p;
  const int M = s.M;
  const int t_old = slot.y;
  const int slot_new = (t_old + 1) % M;
  const int slot_cur = t_old % M;
  const size_t node_off = (size_t)i * p + k;
  float* g_old_p = s.g + (size_t)(t_old & 1) * s.n * p + node_off;
  float* g_new_p = s.g + (size_t)((t_old + 1) & 1) * s.n * p + node_off;
  const int re0 = at(s.r_ptr + i), re1 = at(s.r_ptr + i + 1);
  const int ce0 = at(s.c_ptr + i), ce1 = at(s.c_ptr + i + 1);
  // The running sums of S2c share one factor per sender: rho_li = a_li * sigma_i with
  // sigma_i = sum of every z_half node i produced (1 read + 1 write instead of dO + dO).
  const bool pushes = at(s.co_ptr + i + 1) > at(s.co_ptr + i);

  // Whether anybody pulls from this node.  Only where the state streams past the caches is a row not written worth the look:
  // small rounds wait for it (binary tree of 120 nodes, p 1392: 6.29 us per round without it, 6.75 with it), and so do
  // stretches of single activations (1.2 %).  A graph without such nodes is spared it too.
  constexpr bool kLook = VEC <= -4 && !MANY;
  const bool pulled = !kLook || !s.leaves || at(s.ro_ptr + i + 1) > at(s.ro_ptr + i);

  // ---- every load of the first batch of each phase is issued before its first use:
  //      with few wavefronts per CU this is what keeps enough bytes in flight
  T x_i, z_i, g_old, g_new, h, c, sig_cur, m_i;
  T vb[KB], sg[KB], rt[KB];
  float vw[KB], ca[KB];
  int pl[KB];  // plan words of the C in-edges of the current batch (0: nothing to do)
  const bool spills = pushes && at(s.node_spill + i) == t_old + 1;
  z_i = V<VEC>::ld(s.z + node_off);
  if (kMix) {
    x_i = V<VEC>::ld(s.x + node_off);
    if (MOM) m_i = V<VEC>::ld(s.mom + node_off);
#pragma unroll
    for (int q = 0; q < KB; ++q)
      if (re0 + q < re1) {
        vb[q] = Ring<VEC>::ld(s.v_ring + ((size_t)at(s.r_src + re0 + q) * M + at(s.slot_r + re0 + q)) * p + k);
        vw[q] = at(s.r_w + re0 + q);
      }
  }
  if (kTrack) {
    if (MODE == RFAST_MODE_FUSED) {
      h = V<VEC>::ld((const float*)s.prob.data0 + node_off);
      c = V<VEC>::ld((const float*)s.prob.data1 + node_off);
    } else {
      g_old = V<VEC>::ld(g_old_p);
      g_new = V<VEC>::ld(g_new_p);
    }
    if (pushes) sig_cur = V<VEC>::ld(s.sigma_ring + ((size_t)i * M + slot_cur) * p + k);
#pragma unroll
    for (int q = 0; q < KB; ++q) {
      const int e = ce0 + q;
      pl[q] = e < ce1 ? at(s.plan_c + e) : 0;
      if (pl[q] & (1 << 16)) {
        load_edge<VEC>(s, e, at(s.c_src + e), pl[q], M, p, k, &sg[q], &rt[q]);
        ca[q] = at(s.c_w + e);
      }
    }
  }

  T x_new;
  if (kMix) {
    // S1: local descent; with the optimizer variant along the heavy-ball buffer m <- beta m + z
    T dir = z_i;
    if (MOM) {
      dir = fma_s(s.beta, m_i, z_i);
      V<VEC>::st(s.mom + node_off, dir);
    }
    const T v = fma_s(-gamma, dir, x_i);
    // S2a: pull the stamped neighbour copies and mix with row-stochastic weights
    x_new = mul_s(at(s.r_self + i), v);
#pragma unroll
    for (int q = 0; q < KB; ++q)
      if (re0 + q < re1) x_new = fma_s(vw[q], vb[q], x_new);
    if (DEEP && re0 + KB < re1) {  // in-degree above one batch: what the loads of a batch need is read during the batch before
      int src[KB], ver[KB];
      auto look = [&](int eb) {  // (past the last edge: the last one, which is not used)
#pragma unroll
        for (int q = 0; q < KB; ++q) {
          const int e = eb + q < re1 ? eb + q : re1 - 1;
          src[q] = at(s.r_src + e);
          ver[q] = at(s.slot_r + e);
          vw[q] = at(s.r_w + e);
        }
      };
      look(re0 + KB);
      for (int eb = re0 + KB; eb < re1; eb += KB) {
        float w_now[KB];
#pragma unroll
        for (int q = 0; q < KB; ++q) {
          if (eb + q < re1) vb[q] = Ring<VEC>::ld(s.v_ring + ((size_t)uniform(src[q]) * M + uniform(ver[q])) * p + k);
          w_now[q] = vw[q];
        }
        look(eb + KB);
#pragma unroll
        for (int q = 0; q < KB; ++q)
          if (eb + q < re1) x_new = fma_s(w_now[q], vb[q], x_new);
      }
    }
    // S3 (v half): publish version t+1, unless nobody pulls from this node (the leaves of an in-tree: tree/star of 64 nodes,
    // p 1 M, half of them leaves: 258.5 -> 248.3 us per round; softmax over a binary tree of 128: 115.7 -> 112.8)
    if (pulled) V<VEC>::st(s.v_ring + ((size_t)i * M + slot_new) * p + k, v);
    V<VEC>::st(s.x + node_off, x_new);
    if (MODE == RFAST_MODE_MIX) {
      if constexpr (VEC == 4 || VEC == -4) {  // p is a multiple of 2048 for this objective: every tile is full
        if (s.prob.kind == RFAST_OBJ_SOFTMAX_BF16 && (1024 % s.prob.K) == 0) emit_bf16_blocked<VEC>(s, i, tile, x_new);
      }
      return;
    }
  }

  if (MODE == RFAST_MODE_FUSED) {
    // New sample at the new point; the old sample is the same function of the old x and the
    // old counter, so it is recomputed rather than kept in memory (2 words per coordinate less).
    g_new = diag_sample<VEC>(s, h, c, x_new, i, t_old + 1, k);
    g_old = diag_sample<VEC>(s, h, c, x_i, i, t_old, k);
  }

  // S2b: tracker sum over the in-edges of C; S4: buffer what was consumed.
  // An edge whose stamp did not move holds rho == rho~ exactly and is skipped.
  T z_half = z_i;
#pragma unroll
  for (int q = 0; q < KB; ++q)
    if (pl[q] & (1 << 16)) {
      z_half = track_edge(z_half, ca[q], sg[q], rt[q], ((pl[q] >> 8) & 0xFF) != 0xFF);
      if (pl[q] & (1 << 17)) V<VEC>::st(s.rho_tilde + (size_t)(ce0 + q) * p + k, mul_s(ca[q], sg[q]));
    }
  if (DEEP && ce0 + KB < ce1) {  // in-degree above one batch, in the same way
    int src[KB];
    auto look = [&](int eb) {
#pragma unroll
      for (int q = 0; q < KB; ++q) {
        const int e = eb + q < ce1 ? eb + q : ce1 - 1;
        src[q] = at(s.c_src + e);
        pl[q] = eb + q < ce1 ? at(s.plan_c + e) : 0;
        ca[q] = at(s.c_w + e);
      }
    };
    look(ce0 + KB);
    for (int eb = ce0 + KB; eb < ce1; eb += KB) {
      int now[KB];
      float a_now[KB];
#pragma unroll
      for (int q = 0; q < KB; ++q) {
        now[q] = uniform(pl[q]);
        a_now[q] = ca[q];
        if (now[q] & (1 << 16)) load_edge<VEC>(s, eb + q, uniform(src[q]), now[q], M, p, k, &sg[q], &rt[q]);
      }
      look(eb + KB);
#pragma unroll
      for (int q = 0; q < KB; ++q)
        if (now[q] & (1 << 16)) {
          z_half = track_edge(z_half, a_now[q], sg[q], rt[q], ((now[q] >> 8) & 0xFF) != 0xFF);
          if (now[q] & (1 << 17)) V<VEC>::st(s.rho_tilde + (size_t)(eb + q) * p + k, mul_s(a_now[q], sg[q]));
        }
    }
  }
  z_half = sub(add(z_half, g_new), g_old);

  // S2c: keep a_ii; push: sigma_i grows by z_half.  S3 (rho half): new version t+1
  V<VEC>::st(s.z + node_off, mul_s(at(s.c_self + i), z_half));
  if (pushes) {
    V<VEC>::st(s.sigma_ring + ((size_t)i * M + slot_new) * p + k, add(sig_cur, z_half));
    // S4 for receivers that do not do it themselves in this round: version t - D of this node's
    // running sum leaves the ring with this activation; a receiver whose buffer rho~ is that
    // version gets it copied to the rho~ array now (the slot read here is not the one written above).
    if (spills) {
      const T leaving = V<VEC>::ld(s.sigma_ring + ((size_t)i * M + (t_old - (M - 2)) % M) * p + k);
      for (int o = at(s.co_ptr + i); o < at(s.co_ptr + i + 1); ++o)
        if (at(s.plan_c + at(s.co_eid + o)) & (1 << 18)) V<VEC>::st(s.rho_tilde + (size_t)at(s.co_eid + o) * p + k, mul_s(at(s.co_w + o), leaving));
    }
  }
}

template <int MODE, int VEC, bool MOM, int KB, bool DEEP>
__global__ void __launch_bounds__(kThreads) rfast_state_kernel(RfastDev s, float gamma, int tiles_per_node) {
  const int a = blockIdx.x / tiles_per_node;
  const int2 slot = s.active_plan[a];  // {node, its counter at the start of the round}, node < 0: no work
  if (slot.x < 0) return;
  const int tile = blockIdx.x - a * tiles_per_node;
  // A tile past the end (the launch rounds their number up) finds no coordinates, but for the last ones of a ragged row,
  // which must not be taken twice.  (Tested on every row it cost 0.2 us per pass: 64 nodes of softmax, p 49152, 52.1 -> 51.8 us per round.)
  if constexpr (VEC == 5 || VEC == -5)
    if (tile >= (int)group_tiles(s.p)) return;
  each_group<VEC>(tile, s.p, [&](auto vec, int64_t k) { state_update<MODE, decltype(vec)::value, MOM, KB, DEEP>(s, gamma, slot, tile, k); });
}

// Consecutive iterations of the event-driven mode, one active node each.  A pass over one node's vectors is bound by
// memory, but the next iterations read much of it again (this node's neighbours read the versions it has just written), so
// a lane takes its coordinates through all of the iterations: nothing of theirs depends on another coordinate, and
// what the coordinates under way touch stays in the caches.  16 nodes of a mesh, p 1e6: 15.1 us per iteration as a launch
// of its own, 8.9 this way (bound by the caches behind L2: 72 MB per iteration); 11 nodes, p 144988: 7.0 -> 3.2.
template <int VEC, bool MOM, int KB>
__global__ void __launch_bounds__(kThreads) rfast_events_kernel(RfastDev s, float gamma, int rounds, size_t set_bytes) {
  auto next = [&](auto*& q) { q = reinterpret_cast<std::remove_reference_t<decltype(q)>>(reinterpret_cast<char*>(q) + set_bytes); };
  each_group<VEC>(blockIdx.x, s.p, [&](auto vec, int64_t k) {
    RfastDev r = s;
    for (int q = 0; q < rounds; ++q) {
      for (int a = 0; a < s.n; ++a) {
        const unsigned long long w = fixed(reinterpret_cast<const unsigned long long*>(r.active_plan + a));
        const int2 slot = make_int2((int)(unsigned)w, (int)(w >> 32));
        if (slot.x < 0) break;
        state_update<RFAST_MODE_FUSED, decltype(vec)::value, MOM, KB, true, true>(r, gamma, slot, 0, k);
      }
      next(r.active_plan); next(r.slot_r); next(r.plan_c); next(r.node_spill);
    }
  });
}

// Writes the current sample of every node, g_i = sample(x_i, t_i), into g[t_i & 1][i]: the
// initial gradient g^0 (t = 0, initialisation of Algorithm 1) and the copy that reads of
// the G field return.
template <int VEC>
__global__ void __launch_bounds__(kThreads) rfast_diag_sample_kernel(RfastDev s) {
  const int i = blockIdx.y;
  const int t = s.t[i];
  each_group<VEC>(blockIdx.x, s.p, [&](auto vec, int64_t k) {
    using Vk = V<decltype(vec)::value>;
    const size_t off = (size_t)i * s.p + k;
    const auto h = Vk::ld((const float*)s.prob.data0 + off);
    const auto c = Vk::ld((const float*)s.prob.data1 + off);
    Vk::st(s.g + (size_t)(t & 1) * s.n * s.p + off, diag_sample<decltype(vec)::value>(s, h, c, Vk::ld(s.x + off), i, t, k));
  });
}

// Rebase of the running sums.  sigma_j only ever enters as a_ij*sigma_j - rho~_ij, so
// subtracting c_j = sigma_j(latest) from every ring slot of sender j and a_ij*c_j from
// every buffer rho~_ij fed by j changes nothing in exact arithmetic; in fp32 it
// removes the ever-growing common offset that the difference otherwise has to cancel.
template <int VEC>
__global__ void __launch_bounds__(kThreads) rfast_rebase_kernel(RfastDev s) {
  const int j = blockIdx.y;
  const int o0 = s.co_ptr[j], o1 = s.co_ptr[j + 1];
  if (o0 == o1) return;  // nobody reads this sender's sums
  const int slot = s.t[j] % s.M;
  each_group<VEC>(blockIdx.x, s.p, [&](auto vec, int64_t k) {
    using Vk = V<decltype(vec)::value>;
    float* ring = s.sigma_ring + (size_t)j * s.M * s.p + k;
    const auto c = Vk::ld(ring + (size_t)slot * s.p);
    for (int m = 0; m < s.M; ++m) Vk::st(ring + (size_t)m * s.p, sub(Vk::ld(ring + (size_t)m * s.p), c));
    for (int o = o0; o < o1; ++o) {
      float* rt = s.rho_tilde + (size_t)s.co_eid[o] * s.p + k;
      Vk::st(rt, sub(Vk::ld(rt), mul_s(s.co_w[o], c)));
    }
  });
}

// ---------------------------------------------------------------------------
// Synchronous push-pull step, eq. (2) of the paper (the recursion R-FAST is built on):
//   x_i' = sum_j w_ij (x_j - gamma z_j),   z_i' = sum_j a_ij z_j + grad f_i(x_i') - grad f_i(x_i)
// Every node steps at once, so the v_j = x_j - gamma z_j of all nodes are formed
// first (slot 0 of the v ring serves as the buffer) and z is double-buffered
// (parity 0: the z array, parity 1: slot 1 of the v ring).
// ---------------------------------------------------------------------------
__device__ inline float* sync_z(const RfastDev& s, int parity, int i) {
  return parity == 0 ? s.z + (size_t)i * s.p : s.v_ring + ((size_t)i * s.M + 1) * s.p;
}

// rounds: steps taken at once (the plan arrays are left as the last of them leaves them)
__global__ void __launch_bounds__(256) rfast_sync_plan_kernel(RfastDev s, int rounds) {
  for (int i = threadIdx.x; i < s.n; i += blockDim.x) {
    const int ti = s.t[i] + rounds - 1;
    s.plan_t[i] = ti;
    s.active_plan[i] = make_int2(i, ti);
    s.t[i] = ti + 1;
  }
  if (threadIdx.x == 0) {
    *s.n_active = s.n;
    for (int q = 0; q < 8; ++q) s.active_plan[s.n + q] = make_int2(-1, 0);
    *s.round_no = *s.round_no + rounds;
    s.n_active[1] = *s.round_no;
  }
}

template <int VEC>
__global__ void __launch_bounds__(kThreads) rfast_sync_descent_kernel(RfastDev s, float gamma, int parity) {
  const int i = blockIdx.y;
  each_group<VEC>(blockIdx.x, s.p, [&](auto vec, int64_t k) {
    using Vk = V<decltype(vec)::value>;
    const auto x = Vk::ld(s.x + (size_t)i * s.p + k);
    auto dir = Vk::ld(sync_z(s, parity, i) + k);
    if (s.mom) {
      dir = fma_s(s.beta, Vk::ld(s.mom + (size_t)i * s.p + k), dir);
      Vk::st(s.mom + (size_t)i * s.p + k, dir);
    }
    Vk::st(s.v_ring + (size_t)i * s.M * s.p + k, fma_s(-gamma, dir, x));
  });
}

// acc += sum of w_e row(src_e) over the edges e0 .. e1-1, in order: eight loads in flight, and what the next eight need
// is read meanwhile (edge by edge, the root of a star of 44 nodes took 61 us a step).
template <int VEC, class Row>
__device__ inline void sum_edges(const int32_t* src, const float* w, int e0, int e1, Row row, typename V<VEC>::T* acc) {
  constexpr int KB = 8;
  typename V<VEC>::T vb[KB];
  int from[KB];
  float wt[KB];
  if (e0 >= e1) return;
  auto look = [&](int eb) {  // (past the last edge: the last one, which is not used)
#pragma unroll
    for (int q = 0; q < KB; ++q) {
      const int e = eb + q < e1 ? eb + q : e1 - 1;
      from[q] = src[e];
      wt[q] = w[e];
    }
  };
  look(e0);
  for (int eb = e0; eb < e1; eb += KB) {
    float w_now[KB];
#pragma unroll
    for (int q = 0; q < KB; ++q) {
      if (eb + q < e1) vb[q] = Ring<VEC>::ld(row(uniform(from[q])));
      w_now[q] = wt[q];
    }
    look(eb + KB);
#pragma unroll
    for (int q = 0; q < KB; ++q)
      if (eb + q < e1) *acc = fma_s(w_now[q], vb[q], *acc);
  }
}

// PHASE 0: mix only (x').  PHASE 1: tracker only (reads g' written by the gradient
// kernels).  PHASE 2: mix + diagonal-quadratic gradient + tracker in one pass.
template <int VEC, int PHASE>
__device__ inline void sync_step(const RfastDev& s, int parity, int i, int t_old, int64_t k) {
  using T = typename V<VEC>::T;
  const int64_t p = s.p;
  const size_t off = (size_t)i * p + k;
  float* g_old_p = s.g + (size_t)(t_old & 1) * s.n * p + off;
  float* g_new_p = s.g + (size_t)((t_old + 1) & 1) * s.n * p + off;
  T x_new, g_new, g_old;
  if (PHASE != 1) {
    const T x_old = V<VEC>::ld(s.x + off);
    x_new = mul_s(s.r_self[i], V<VEC>::ld(s.v_ring + (size_t)i * s.M * p + k));
    sum_edges<VEC>(s.r_src, s.r_w, s.r_ptr[i], s.r_ptr[i + 1], [&](int j) { return s.v_ring + (size_t)j * s.M * p + k; }, &x_new);
    V<VEC>::st(s.x + off, x_new);
    if (PHASE == 0) return;
    const T h = V<VEC>::ld((const float*)s.prob.data0 + off);
    const T c = V<VEC>::ld((const float*)s.prob.data1 + off);
    g_new = diag_sample<VEC>(s, h, c, x_new, i, t_old + 1, k);
    g_old = diag_sample<VEC>(s, h, c, x_old, i, t_old, k);
  } else {
    g_new = V<VEC>::ld(g_new_p);
    g_old = V<VEC>::ld(g_old_p);
  }
  T z_new = mul_s(s.c_self[i], V<VEC>::ld(sync_z(s, parity, i) + k));
  sum_edges<VEC>(s.c_src, s.c_w, s.c_ptr[i], s.c_ptr[i + 1], [&](int j) { return sync_z(s, parity, j) + k; }, &z_new);
  z_new = sub(add(z_new, g_new), g_old);
  V<VEC>::st(sync_z(s, parity ^ 1, i) + k, z_new);
}

template <int VEC, int PHASE>
__global__ void __launch_bounds__(kThreads) rfast_sync_step_kernel(RfastDev s, int parity) {
  const int i = blockIdx.y, t_old = s.plan_t[i];
  each_group<VEC>(blockIdx.x, s.p, [&](auto vec, int64_t k) { sync_step<decltype(vec)::value, PHASE>(s, parity, i, t_old, k); });
}

template <int VEC>
__global__ void __launch_bounds__(kThreads) rfast_sync_fold_kernel(RfastDev s) {
  const int i = blockIdx.y;
  each_group<VEC>(blockIdx.x, s.p, [&](auto vec, int64_t k) {
    using Vk = V<decltype(vec)::value>;
    Vk::st(s.z + (size_t)i * s.p + k, Vk::ld(sync_z(s, 1, i) + k));
  });
}

// Bytes per array from which on the passes stream past the caches (but for the rings, see Ring): 16 MB, or more where the
// rounds before this one have left the state in the caches (`warm`: a call of eight or more rounds).  Time streamed over time
// cached, contexts in turn (the caches hold somebody else's state) and one context over and over: single rounds, 24 to 28 MB: mesh of 16 0.92 and
// 1.01, star of 20 0.93 and 1.02, ring of 128 0.96 and 1.04; calls of four, 17 to 28 MB: 0.95 to 1.0 and 1.0 to 1.07.  Calls of eight, 17 to
// 31 MB: star of 64 0.99 to 1.05 and 1.01 to 1.14, ring of 16 1.01 to 1.04 and 1.01 to 1.03, tree of 64 0.99 to 1.03 and 1.01 to 1.08, at 60 MB all
// 0.91 to 0.98; where a row has several readers even from 17 to 24 MB and 0.96 to 0.99 from there on (mesh of 30, exponential graph of 16).  The
// softmax passes: 1.01 to 1.05 at 17 to 22 MB, 0.97 at 27 to 29.  Least squares and logistic regression read their data between the
// passes, which leaves the caches cold: 0.95 at 18 MB.
double stream_from(const RfastDev& d, bool warm) {
  if (!warm || (d.prob.kind != RFAST_OBJ_SOFTMAX_BF16 && d.prob.kind != RFAST_OBJ_DIAG_QUADRATIC)) return 16.0e6;
  return d.prob.kind == RFAST_OBJ_SOFTMAX_BF16 || (int64_t)d.eR + d.eC >= 6 * (int64_t)d.n ? 24.0e6 : 32.0e6;
}

template <int MODE, bool MOM, int KB, bool DEEP>
hipError_t launch_deep(rfast_ctx* c, float gamma, bool warm) {
  const RfastDev& d = c->d;
  const bool vec4 = (d.p % 4) == 0;
  const bool streaming = (double)d.n * (double)d.p * 4.0 >= stream_from(d, warm);
  // Consecutive workgroups go round the eight dies, each with an L2 of its own: a multiple of eight tiles per node puts
  // a tile of every node, which shares its neighbours' rows, on one die.  The price is up to seven workgroups per node that find
  // nothing, and dies that get up to a fifth more than others.  Time with it over time without:
  // Three and more in-edges per graph on average: mesh of 8, p 256248, 0.93; exponential graph of 100, p 70000, 0.92; softmax on 64 nodes
  // of one, p 43008, 0.98.  Of 36 to 52 tiles every other node shares a die as it is: mesh of 100, p 36000, 1.02, so only from five in-edges on.
  // Fewer in-edges: a single pass of few nodes gains (tree of 30, p 68332: 0.95; of 64, p 33052: 0.95; star of 20, p 300000: 0.99), of many it
  // does not (star of 100, p 42500: 1.02), nor from 49 nodes on where it streams (tree of 64, p 156248: 1.04); two passes with
  // matrix products between them do not (softmax, 36 tiles: tree of 100, 1.03; ring of 120, 1.02).
  // Event-driven iterations have one active node at a time, which shares with nobody.
  int64_t tiles = group_tiles(d.p);
  const bool half = tiles % 8 == 4 && tiles < 56;
  const bool shared = (int64_t)d.eR + d.eC >= (half ? 10 : 6) * (int64_t)d.n;
  const bool few = MODE == RFAST_MODE_FUSED && !half && d.n <= (streaming ? 48 : 64);
  if (tiles >= 32 && !c->no_tiles && (shared || few)) tiles = (tiles + 7) / 8 * 8;
  const int64_t blocks = tiles * d.n;
  if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
  // Wavefronts per SIMD matter: the bidirectional ring (about 15 streams per node-update) is fastest at 3, slower at
  // 2 (capped through reserved LDS: +11 %) and at 4 or 5 (+2 %, +4 %); the register count of KB sets it.
  if (vec4 && streaming)
    hipLaunchKernelGGL((rfast_state_kernel<MODE, -4, MOM, KB, DEEP>), dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, d, gamma, (int)tiles);
  else if (vec4)
    hipLaunchKernelGGL((rfast_state_kernel<MODE, 4, MOM, KB, DEEP>), dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, d, gamma, (int)tiles);
  else if (streaming)
    hipLaunchKernelGGL((rfast_state_kernel<MODE, -5, MOM, KB, DEEP>), dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, d, gamma, (int)tiles);
  else
    hipLaunchKernelGGL((rfast_state_kernel<MODE, 5, MOM, KB, DEEP>), dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, d, gamma, (int)tiles);
  return hipGetLastError();
}

template <int MODE, bool MOM, int KB>
hipError_t launch(rfast_ctx* c, float gamma, bool warm) {
  if constexpr (MODE == RFAST_MODE_FUSED)
    if (c->max_in_degree <= KB) return launch_deep<MODE, MOM, KB, false>(c, gamma, warm);
  return launch_deep<MODE, MOM, KB, true>(c, gamma, warm);
}

}  // namespace

hipError_t rfast_diag_init_gradient(rfast_ctx* c) {
  const RfastDev& d = c->d;
  const bool vec4 = (d.p % 4) == 0;
  const unsigned gx = (unsigned)group_tiles(d.p);
  if (vec4)
    hipLaunchKernelGGL(rfast_diag_sample_kernel<4>, dim3(gx, d.n), dim3(kThreads), 0, c->stream, d);
  else
    hipLaunchKernelGGL(rfast_diag_sample_kernel<5>, dim3(gx, d.n), dim3(kThreads), 0, c->stream, d);
  return hipGetLastError();
}

// phase: 0 plan + descent + mix, 1 tracker, 2 plan + descent + fused step, 3 fold z back into its array
hipError_t rfast_launch_sync(rfast_ctx* c, int phase, float gamma, int parity) {
  const RfastDev& d = c->d;
  const bool vec4 = (d.p % 4) == 0;
  const dim3 grid((unsigned)group_tiles(d.p), d.n), blk(kThreads);
  const bool streaming = vec4 && (double)d.n * (double)d.p * 4.0 >= 32.0e6;
  if (phase == 0 || phase == 2) {
    hipLaunchKernelGGL(rfast_sync_plan_kernel, dim3(1), dim3(256), 0, c->stream, d, 1);
    if (streaming) hipLaunchKernelGGL(rfast_sync_descent_kernel<-4>, grid, blk, 0, c->stream, d, gamma, parity);
    else if (vec4) hipLaunchKernelGGL(rfast_sync_descent_kernel<4>, grid, blk, 0, c->stream, d, gamma, parity);
    else hipLaunchKernelGGL(rfast_sync_descent_kernel<5>, grid, blk, 0, c->stream, d, gamma, parity);
  }
  if (streaming) {
    if (phase == 0) hipLaunchKernelGGL((rfast_sync_step_kernel<-4, 0>), grid, blk, 0, c->stream, d, parity);
    if (phase == 1) hipLaunchKernelGGL((rfast_sync_step_kernel<-4, 1>), grid, blk, 0, c->stream, d, parity);
    if (phase == 2) hipLaunchKernelGGL((rfast_sync_step_kernel<-4, 2>), grid, blk, 0, c->stream, d, parity);
    if (phase == 3) hipLaunchKernelGGL(rfast_sync_fold_kernel<-4>, grid, blk, 0, c->stream, d);
  } else if (vec4) {
    if (phase == 0) hipLaunchKernelGGL((rfast_sync_step_kernel<4, 0>), grid, blk, 0, c->stream, d, parity);
    if (phase == 1) hipLaunchKernelGGL((rfast_sync_step_kernel<4, 1>), grid, blk, 0, c->stream, d, parity);
    if (phase == 2) hipLaunchKernelGGL((rfast_sync_step_kernel<4, 2>), grid, blk, 0, c->stream, d, parity);
    if (phase == 3) hipLaunchKernelGGL(rfast_sync_fold_kernel<4>, grid, blk, 0, c->stream, d);
  } else {
    if (phase == 0) hipLaunchKernelGGL((rfast_sync_step_kernel<5, 0>), grid, blk, 0, c->stream, d, parity);
    if (phase == 1) hipLaunchKernelGGL((rfast_sync_step_kernel<5, 1>), grid, blk, 0, c->stream, d, parity);
    if (phase == 2) hipLaunchKernelGGL((rfast_sync_step_kernel<5, 2>), grid, blk, 0, c->stream, d, parity);
    if (phase == 3) hipLaunchKernelGGL(rfast_sync_fold_kernel<5>, grid, blk, 0, c->stream, d);
  }
  return hipGetLastError();
}

// the integer side of `rounds` synchronous steps taken by one launch of the multi-step kernel
hipError_t rfast_launch_sync_plan(rfast_ctx* c, int rounds) {
  hipLaunchKernelGGL(rfast_sync_plan_kernel, dim3(1), dim3(256), 0, c->stream, c->d, rounds);
  return hipGetLastError();
}

hipError_t rfast_launch_rebase(rfast_ctx* c) {
  const RfastDev& d = c->d;
  const bool vec4 = (d.p % 4) == 0;
  const unsigned gx = (unsigned)group_tiles(d.p);
  if (vec4)
    hipLaunchKernelGGL(rfast_rebase_kernel<4>, dim3(gx, d.n), dim3(kThreads), 0, c->stream, d);
  else
    hipLaunchKernelGGL(rfast_rebase_kernel<5>, dim3(gx, d.n), dim3(kThreads), 0, c->stream, d);
  return hipGetLastError();
}

hipError_t rfast_launch_events(rfast_ctx* c, float gamma, int rounds) {
  const RfastDev& d = c->d;
  auto go = [&](auto vec, auto mom, int64_t blocks) {
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    // (loads in batches of four: eight cost more registers than they hide, 2636 -> 3143 us over 200 iterations)
    hipLaunchKernelGGL((rfast_events_kernel<decltype(vec)::value, decltype(mom)::value, 4>), dim3((unsigned)blocks), dim3(kThreads),
                       0, c->stream, d, gamma, rounds, c->plan_set_bytes);
    return hipGetLastError();
  };
  auto with = [&](auto vec, int64_t blocks) {
    return d.mom ? go(vec, std::integral_constant<bool, true>(), blocks) : go(vec, std::integral_constant<bool, false>(), blocks);
  };
  // Four coordinates per lane as soon as that leaves a wavefront for every compute unit (p 1e6: 2124 us against 2636
  // with one), one per lane below (p 45746: 68 against 71).
  if (d.p < 65536) return with(std::integral_constant<int, 1>(), (d.p + kThreads - 1) / kThreads);
  if (d.p % 4 == 0) return with(std::integral_constant<int, 4>(), group_tiles(d.p));
  return with(std::integral_constant<int, 5>(), group_tiles(d.p));
}

hipError_t rfast_launch_state(rfast_ctx* c, int mode, float gamma, bool warm) {
  const bool mom = c->d.mom != nullptr;
  // three or more in-edges per node on average (both graphs together), or a state so small that wavefronts are few
  // anyway and only the trips through memory count: the deeper load batch
  const bool deep = (int64_t)c->d.eR + c->d.eC >= 3 * (int64_t)c->d.n || (double)c->d.n * (double)c->d.p < 4.0e6;
  switch (mode) {
    case RFAST_MODE_FUSED:
      if (deep) return mom ? launch<RFAST_MODE_FUSED, true, 8>(c, gamma, warm) : launch<RFAST_MODE_FUSED, false, 8>(c, gamma, warm);
      return mom ? launch<RFAST_MODE_FUSED, true, 4>(c, gamma, warm) : launch<RFAST_MODE_FUSED, false, 4>(c, gamma, warm);
    case RFAST_MODE_MIX:
      if (deep) return mom ? launch<RFAST_MODE_MIX, true, 8>(c, gamma, warm) : launch<RFAST_MODE_MIX, false, 8>(c, gamma, warm);
      return mom ? launch<RFAST_MODE_MIX, true, 4>(c, gamma, warm) : launch<RFAST_MODE_MIX, false, 4>(c, gamma, warm);
    default:  // S1 is not part of this pass
      return deep ? launch<RFAST_MODE_TRACK, false, 8>(c, gamma, warm) : launch<RFAST_MODE_TRACK, false, 4>(c, gamma, warm);
  }
}
