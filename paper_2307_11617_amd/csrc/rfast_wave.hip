// Several activation rounds per launch with the tile of one WAVEFRONT resident in LDS.
//
// Like rfast_block.hip (every step of Algorithm 1 is elementwise in the coordinate, so a tile of
// coordinates of every node can stay on chip over many rounds), with one difference that removes
// every barrier from the round loop: a tile belongs to a single wavefront.  The 64 lanes of a
// wavefront are split among ALL nodes (16 nodes: 4 lanes per node, 4 coordinates per lane, a tile of
// 16 coordinates), so every neighbour read of S2a / S2b and every publication of S3 stays within the
// wavefront, whose LDS operations execute in program order: a round needs no synchronisation with
// any other wavefront, the wavefronts of a CU drift out of step, and while one waits for its LDS
// reads another computes.  The plan words of a round are read from global memory one round ahead
// (the records of all rounds are a few KB that every wavefront of the chip reads, so they stay in the
// caches), which leaves LDS to the rings and takes the plan reads out of the critical path.  What was
// consumed last time over an edge (S4) lives in the registers of the receiving node's lanes, and so does a
// node's own latest sum, so a round reads one value per edge from LDS and touches global memory for the
// plan words only.
//
// LDS holds the latest K versions of a node, not the M = D + 2 of the ring in memory: the reads of a round come before its
// publications in the program of the wavefront, so that the oldest version gives its place to the new one (M - 1 versions
// always suffice), and a version older than the longest delay is read only after several losses in a row.  Such a read
// is marked in the plan; the version goes to the ring in memory when it loses its place on chip, if anybody
// reads it later or holds it after the launch, and comes from there.  The fewer versions, the more
// wavefronts: that decides (500 rounds of 16 nodes, p 11.2 M, us per round: 192.7 with nine versions of which eight
// wavefronts fit a CU, 167 with the same eight and the round's work cut, 139.5 with twelve at six versions, 137.8 with sixteen at
// five; a SIMD is busy with its vector ALU only from three wavefronts on).
//
// The arithmetic is, operation for operation, that of rfast_state_kernel<FUSED> and of
// rfast_block_kernel: the three paths give the same bits (but for kC = 0, below).  (One liberty: where those skip a missing
// or idle edge, this kernel runs it through the multiply-add with weight zero or a difference of zero, which spares the round
// loop most of its branches.  Adding zero changes nothing but the sign of a sum that is exactly zero,
// as long as the ring values are finite; an infinity of a node with fewer edges than the kernel has slots can turn to NaN here
// an activation before it does elsewhere, where infinity minus infinity follows in the next tracker sum.)
#include <algorithm>

#include "rfast_vec.h"

namespace {

constexpr int kWaveMaxDeg = 6;  // most in-edges of R, in-edges of C and out-edges of C a node may have on this path
                                // (kernels for 2, 4 and 6 edge slots per node: an exponential graph on 32 nodes has 5
                                // edges per node and kind; 8 slots would not fit the registers of two wavefronts per SIMD)
constexpr int kWaveMaxNodes = 64;  // at least one lane (4 coordinates, 16 B of a row) per node
constexpr unsigned kXcds = 8;      // accelerator dies; consecutive workgroups go round them
constexpr unsigned kTileRun = 64;  // neighbouring tiles that one XCD takes in a row
constexpr unsigned kSyncTileRun = 4;  // the same for the multi-step synchronous kernel (measured: 4 is 3 % faster there than 64)

// Orders the LDS and global accesses of the lanes of one wavefront: everything before it is done
// (in program order of the wavefront) before anything after it starts.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The sum over the nodes of a value per lane, column by column (lane = node * lw + column; lanes past the last node bring
// zeros), in all lanes of a column.
__device__ inline float4 sum_of_nodes(float4 t, int lane, int n, int i, int ln, int lw) {
  if (lw == 1) {
    // Halves, then rows of 16 lanes are added so that two, then all four coordinates share a register, a row each; then
    // within the rows: 14 instructions where a butterfly over four registers takes 48.
    auto u = [](float v) { return __float_as_uint(v); };
    auto f = [](unsigned v) { return __uint_as_float(v); };
    const auto xz = __builtin_amdgcn_permlane32_swap(u(t.x), u(t.z), false, false);
    const auto yw = __builtin_amdgcn_permlane32_swap(u(t.y), u(t.w), false, false);
    const auto r = __builtin_amdgcn_permlane16_swap(u(f(xz[0]) + f(xz[1])), u(f(yw[0]) + f(yw[1])), false, false);
    float v = f(r[0]) + f(r[1]);  // rows: x, y, z, w
    auto ror = [](float a, auto by) {
      return a + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), 0x120 + decltype(by)::value, 0xF, 0xF, false));
    };
    v = ror(v, std::integral_constant<int, 8>());
    v = ror(v, std::integral_constant<int, 4>());
    v = ror(v, std::integral_constant<int, 2>());
    v = ror(v, std::integral_constant<int, 1>());
    auto at = [&](int from) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), from)); };
    return make_float4(at(0), at(16), at(32), at(48));
  }
  int step = 1;
  while (2 * step < n) step *= 2;
  for (; step > 0; step >>= 1) {
    const int from = lane + step * lw;
    const float4 o = make_float4(__shfl(t.x, from), __shfl(t.y, from), __shfl(t.z, from), __shfl(t.w, from));
    if (i < step && i + step < n) t = add(t, o);
  }
  return make_float4(__shfl(t.x, ln), __shfl(t.y, ln), __shfl(t.z, ln), __shfl(t.w, ln));
}

// lw: lanes per node (64 / n, rounded down); kR, kC: edge slots per node over R and over C; MOM: the optimizer
// variant is in use, heavy-ball buffer, weight decay or both (a template flag, so that the plain method
// carries neither the registers and the copies at the join nor the tests).
// ANY: p is not a multiple of four: rows start at any float's address, and the last group of a row may be short (its
// missing coordinates are zeros on chip and are not stored).
// W: wavefronts per workgroup.  Every wavefront still owns a tile of 4 lw coordinates and runs its
// rounds without looking at the others; the W tiles of a workgroup are neighbours, and the workgroup
// moves their rings between HBM and LDS together, so that a row segment is W times as wide (16 nodes,
// W = 2: 128 B, a whole cache line per row; with one wavefront per workgroup every load and store
// instruction touched 16 half lines).  The barriers this costs stand before and after the round loop,
// not in it.
// (A persistent grid, as many workgroups as the chip holds with each streaming through a region of
// its own, was measured and dropped: its workgroups run in step, so that all of them move tiles at one
// time and compute at another, and a launch of 20 rounds took 10.9 ms against 8.6 ms.  With a delay of
// its own for every workgroup at the start, up to 14 us, and what depends on the node alone set up once
// per wavefront, 10 rounds took 5.1 ms against 5.3, but 20 rounds 7.4 against 7.1 and 500 rounds 101.8
// against 93.9: the same round loop, instruction for instruction, ran 8 % slower.)
// kC = 0: every edge of C leads to one node (a star, at most one in-edge of R per node: any tree), which as a lane of its own
// would need a slot per sender.  Instead the lanes of every sender, which have its sums in their own column, form its term
// a (sigma - what was consumed last) and keep what belongs to the edge (S4), and the terms are added up across the wavefront.  That is
// another order of a sum of up to 63 terms than that of one pass per round (the depth of the tree, not the number of terms, bounds its
// error: against 64 bits, stars of 12 to 64 nodes after 200 to 600 rounds, x 1.4 to 3 times closer, z 1.0 to 1.8), so these launches agree with
// it to the rounding of that sum and not bit for bit.  kC = -1: the same with at most kStarInOrder nodes, whose few terms the lanes of
// the hub read one after the other, in the order of one pass per round, so that the bits are the same.  (Six edge slots would hold these stars
// as well, with two wavefronts per SIMD and every ring: star of 7, p 600000, 100 rounds, delays of up to 4 / 16: 762 / 1385 us with slots,
// 490 / 750 this way, 1700 / 1750 one pass per round.)  Tree and star of 64 nodes, p 1 M, delays of up to 16, 100 rounds: 25.2 ms one pass per
// round (6.0 TB/s), 10.2 this way, 80 to 94 us per round and 2 ms of tile movement.
// kC = -1 is there for four wavefronts per SIMD only: it takes no more registers than that leaves with fewer of them.
// FEW: only nodes with readers have rings on chip: a tree is read over half of its nodes, the others publish no v.
// PER: wavefronts per SIMD, to which the registers are cut: 4 at two edge slots (120 to 128 registers), 3 at four (164 to 168), 2 at six (three
// would spill 45 registers in the round loop: 75 -> 239 us per round on 32 nodes of an exponential graph, p 1 M).  At four edge slots
// the heavy-ball buffer and several wavefronts per workgroup spill up to 6 registers, and three still win: us per round in
// calls of 20 / 60 / 200 at two and three wavefronts, heavy-ball buffer in use: mesh of 16, p 1 M, 34.8 / 27.7 / 22.1 and 29.0 / 19.7 / 17.6; mesh of
// 40, p 300000, 45.2 / 36.2 / 28.7 and 38.1 / 26.2 / 23.3.  The forms for three and four at two edge slots take the same registers, but order
// their loads and rounds differently: three wavefronts of the form for four are 1 to 4 % slower (500 rounds of 16 nodes, p 11.2 M: 69.8 -> 72.3 ms).
//
// Only what can matter is moved.  Stamps never go back (S2a / S2b take the largest stamp received), so
// a version older than every stamp held on its sender's out-edges will never be read again: such a
// slot is neither loaded (LDS gets zeros, which the multiply-adds with weight zero need to be finite)
// nor, if the launch wrote it and it is out of reach again by the end, stored; slots the launch did
// not write are not stored either, nor x and z of a node it never activated, and an S4 buffer is moved
// only while its version is outside its sender's ring.  With the delays of the bidirectional-ring
// workload that is 30 rows per node instead of 46.
//
// Multipliers for the two divisions of a lane number that the kernel starts with, by the lanes per node and by the
// lanes of a row segment: x / d = (x * ceil(2^16 / d)) >> 16 for x < 256 and d <= 256 (the error of the quotient,
// x (d ceil(2^16 / d) - 2^16) / (2^16 d), stays below 1 / d).  The division itself is some 25 instructions, which
// every wavefront of a launch would run.
struct WaveDiv {
  unsigned lanes, segment;
};
static WaveDiv wave_div(int lw, int W) {
  WaveDiv dv;
  dv.lanes = (65536u + (unsigned)lw - 1) / (unsigned)lw;
  dv.segment = (65536u + (unsigned)(lw * W) - 1) / (unsigned)(lw * W);
  return dv;
}

template <int kR, int kC, bool FEW, bool MOM, int W, bool ANY, int PER>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(PER, PER))) rfast_wave_kernel(RfastDev s, RfastBlock blk, int lw, WaveDiv dv) {
  constexpr int VEC = 4;
  constexpr bool HUB = kC <= 0, ORDERED = kC < 0;
  extern __shared__ float4 lds4[];
  const int n = s.n, M = s.M, K = blk.slots;
  const int64_t p = s.p;
  const int W1 = n + s.eR + s.eC + 1;  // words of a plan record; the last one is always zero
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = (int)(((unsigned)lane * dv.lanes) >> 16), ln = lane - i * lw;  // lane / lw
  // Workgroup b runs on XCD b mod 8, each with an L2 of its own.  Neighbouring workgroups go to the same
  // XCD, one right after the other, in runs that cover kTileRun tiles (4 KB of every row on 16 nodes):
  // that keeps the rows an XCD moves at one time on few pages (a launch of 10 rounds, which is all moving,
  // took 8.1 ms with such runs and 9.3 ms with runs of 4 tiles), and where a row segment is less than a
  // cache line the neighbour finds the other part in that L2.
  constexpr unsigned kRun = kTileRun / W;
  const unsigned xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int64_t group = ((int64_t)(slot / kRun) * kXcds + xcd) * kRun + slot % kRun;
  const int64_t k_wg = group * (4 * lw * W);  // first coordinate of the workgroup
  if (k_wg >= p) return;  // a workgroup past the end (the grid is whole runs): all of its wavefronts leave
  const int64_t k = k_wg + (wave * lw + ln) * 4;
  const bool wave_has = k_wg + (int64_t)wave * lw * 4 < p;  // this wavefront has a tile (the last workgroup may be ragged)
  const bool mine = i < n && k < p;
  const int left = p - k < 4 ? (int)(p - k) : 4;  // ANY: coordinates of the row from the lane's first one on
  // float4 of the rings of v of one wavefront's tile, [rows][K][lw]; the rings of sums follow.  FEW: only nodes whose v or
  // sums somebody reads have a ring, in the order of their numbers (bit lw j of a mask: node j has one).
  const int v_rows = FEW ? blk.v_rows : n, s_rows = FEW ? blk.s_rows : n;
  const size_t ring_f4 = (size_t)v_rows * K * lw;
  unsigned long long has_v = 0, has_s = 0;
  bool pulled = true;
  if (FEW) {
    int out_r = 0, out_c = 0;
    if (i < n) {
      out_r = s.ro_ptr[i + 1] - s.ro_ptr[i];
      out_c = s.co_ptr[i + 1] - s.co_ptr[i];
    }
    pulled = out_r > 0;
    has_v = __ballot(pulled && ln == 0);
    has_s = __ballot(out_c > 0 && ln == 0);
  }
  auto has = [&](unsigned long long rows, int j) { return !FEW || (rows >> (j * lw) & 1) != 0; };
  auto row = [&](unsigned long long rows, int j) { return FEW ? __popcll(rows & ((1ull << (j * lw)) - 1)) : j; };
  // LDS addresses proper (32 bits, the start of the array included): column of the lane in a node's ring + slot * bytes
  // per slot, one 24-bit multiply-add each, which leaves the high byte of a plan word to its flags.
  const unsigned slot_bytes = (unsigned)lw * sizeof(float4);
  typedef float Vec4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) Vec4 LdsVec4;
  auto lds_ld = [&](unsigned a) {
    const Vec4 t = *(LdsVec4*)(uintptr_t)a;
    return make_float4(t.x, t.y, t.z, t.w);
  };
  auto lds_st = [&](unsigned a, float4 w) {
    const Vec4 t = {w.x, w.y, w.z, w.w};
    *(LdsVec4*)(uintptr_t)a = t;
  };
  const unsigned sg_off = (unsigned)v_rows * K * slot_bytes;  // from the rings of v to those of sums
  const unsigned tile_f4 = (unsigned)(v_rows + s_rows) * K * lw + (ORDERED ? (unsigned)(n * lw) : 0u);  // ORDERED: a term per lane behind the rings
  const unsigned tile = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds4 + (unsigned)wave * tile_f4 * (unsigned)sizeof(float4);
  const unsigned terms = tile + (unsigned)(v_rows + s_rows) * K * slot_bytes;
  // Moving the rings: lane T of the workgroup moves column cT (of the lw W columns of a row segment) of
  // node iT, i.e. column lT of the tile of wavefront wT.  With W = 1 that is the lane's own column.
  const int seg = lw * W;
  const int iT = W == 1 ? i : (int)((threadIdx.x * dv.segment) >> 16), cT = (int)threadIdx.x - iT * seg;  // threadIdx.x / seg
  const int wT = W == 1 ? 0 : (int)(((unsigned)cT * dv.lanes) >> 16), lT = cT - wT * lw;                  // cT / lw
  const int64_t kT = k_wg + 4 * cT;
  const bool moves = iT < n && kT < p;
  const int leftT = p - kT < 4 ? (int)(p - kT) : 4;
  const bool mv_has_v = has(has_v, iT), mv_has_s = has(has_s, iT);
  float4* mv_v = lds4 + (size_t)wT * tile_f4 + (size_t)row(has_v, iT) * K * lw + lT;  // + slot * lw
  float4* mv_s = lds4 + (size_t)wT * tile_f4 + ring_f4 + (size_t)row(has_s, iT) * K * lw + lT;
  // What the resolver, which has been through all rounds of the launch already, left about the moved node: the places of
  // its latest version before the launch, in memory and on chip, and, one bit per version counted back from it, which
  // versions a receiver can still pick up (the others are not loaded); and the same for after the launch, where a version
  // goes back if the launch wrote it, still holds it and somebody can still read it, and with a rebase every readable sum
  // is shifted, whether the launch wrote it or not and wherever it is.
  int4 head = make_int4(0, 0, 0, 0), tail = head;
  if (moves) {
    head = *reinterpret_cast<const int4*>(s.blk_head + kHeadWords * iT + 8);
    tail = *reinterpret_cast<const int4*>(s.blk_head + kHeadWords * iT + 12);
    if (blk.rebase) tail.w = s.blk_head[kHeadWords * iT + 6];
  }

  float4 x, z, g, h, c, m = make_float4(0.f, 0.f, 0.f, 0.f);
  const bool momentum = MOM && s.mom != nullptr;  // the heavy-ball buffer of the optimizer variant is in use
  int ce0 = 0, dR = 0, dI = 0, dO = 0;
  // What was consumed last time over each in-edge of C, in registers: the sender's running sum of that version, or (bit u of
  // `prod`) its product with the weight, which is what the array of S4 buffers holds.  So a round reads one sum per edge from LDS,
  // and a buffer is written only at the end of a launch, if its version is outside the sender's ring then.
  // HUB: every edge of C leads to one node.  A sender's lanes hold this for their edge to it (in place 0), form its term of the
  // sum in their own columns and add the terms up across the wavefront.
  constexpr int kL = kC > 0 ? kC : 1;
  float4 last[kL];
  unsigned prod = 0, outside = 0;  // outside: the same for after the launch, edge by edge (RfastDev::blk_head)
  int where[kL];
  float4 sig = make_float4(0.f, 0.f, 0.f, 0.f);  // the node's own latest running sum
  float r_self = 0.f, c_self = 0.f;
  // the node's edges, in registers for the whole launch: LDS column of the sender's ring, weight,
  // position of the edge's plan word in a record; a missing edge has weight zero, the node's own
  // column and the zero word of the record.  (FEW: in a ring that the node has, as zero times another node's infinity would be NaN wherever
  // it is in the graph.  A node without in-edges of R is the root of R, which is read; one without a ring of sums is the root of C,
  // which is that of R and has a ring of v.)
  unsigned r_col[kR], c_col[kL];
  // positions of plan words as unsigned byte offsets: a 32-bit offset from a uniform base, no 64-bit address arithmetic
  unsigned r_pw[kR], c_pw[kL];
  float r_w[kR], c_w[kL];
#pragma unroll
  for (int u = 0; u < kR; ++u) {
    r_col[u] = tile;
    r_pw[u] = 4u * (W1 - 1);
    r_w[u] = 0.f;
  }
#pragma unroll
  for (int u = 0; u < kL; ++u) {
    c_col[u] = tile;
    where[u] = 0;
    c_pw[u] = 4u * (W1 - 1);
    c_w[u] = 0.f;
    last[u] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // this lane's column in the ring of v of its node, and from there to its column in the node's ring of sums
  const unsigned a_own = tile + (unsigned)(row(has_v, i) * K * lw + ln) * sizeof(float4);
  const unsigned to_sum = FEW ? sg_off + (unsigned)((row(has_s, i) - row(has_v, i)) * K * lw) * (unsigned)sizeof(float4) : sg_off;
  unsigned node_pw = 4u * (W1 - 1);
  if (mine) {
    node_pw = 4u * i;
    const int re0 = s.r_ptr[i];
    dR = s.r_ptr[i + 1] - re0;
    ce0 = s.c_ptr[i];
    dI = s.c_ptr[i + 1] - ce0;
    dO = s.co_ptr[i + 1] - s.co_ptr[i];
    r_self = s.r_self[i];
    c_self = s.c_self[i];
    if (HUB) {  // the node's edge to the hub, if it has one
      dI = dO;
      ce0 = dO > 0 ? s.co_eid[s.co_ptr[i]] : 0;
    }
#pragma unroll
    for (int u = 0; u < kR; ++u) {
      const bool hr = u < dR;
      r_col[u] = tile + (unsigned)(row(has_v, hr ? s.r_src[re0 + u] : i) * K * lw + ln) * sizeof(float4);
      r_w[u] = hr ? s.r_w[re0 + u] : 0.f;
      r_pw[u] = 4u * (hr ? n + re0 + u : W1 - 1);
    }
    if (HUB && dI > 0) {
      c_col[0] = a_own + to_sum;
      c_w[0] = s.c_w[ce0];
      c_pw[0] = 4u * (n + s.eR + ce0);
    }
#pragma unroll
    for (int u = 0; u < kC; ++u) {
      const bool hc = u < dI;
      c_col[u] = FEW && !hc && dO == 0 ? a_own : tile + sg_off + (unsigned)(row(has_s, hc ? s.c_src[ce0 + u] : i) * K * lw + ln) * sizeof(float4);
      c_w[u] = hc ? s.c_w[ce0 + u] : 0.f;
      c_pw[u] = 4u * (hc ? n + s.eR + ce0 + u : W1 - 1);
    }
  }
  // Plan words are read through a buffer descriptor over the records of this launch: the address is
  // descriptor + uniform record offset + 32-bit lane offset, formed by the load itself (no 64-bit
  // address arithmetic per word), and a read past the records returns zero instead of faulting.
  // First those of round 0 (every lane: the lanes of a wavefront without a node read the zero word).
  const __amdgpu_buffer_rsrc_t plans = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<int*>(s.blk_plan), 0, blk.rounds * W1 * (int)sizeof(int), 0x00020000);
  const int rec_bytes = W1 * (int)sizeof(int);
  auto word = [&](int round, unsigned byte_offset) {
    return __builtin_amdgcn_raw_buffer_load_b32(plans, byte_offset, round * rec_bytes, 0);
  };
  struct Plan {
    int node, r[kR], c[kL], hub;
  };
  auto fetch = [&](int round, Plan& P) {
    P.node = word(round, node_pw);
#pragma unroll
    for (int u = 0; u < kR; ++u) P.r[u] = word(round, r_pw[u]);
#pragma unroll
    for (int u = 0; u < kL; ++u) P.c[u] = word(round, c_pw[u]);
    if (HUB) P.hub = word(round, 4u * (unsigned)blk.hub);
  };
  Plan plan_a, plan_b;  // two register sets that take turns: one in use, one arriving
  fetch(0, plan_a);
  if (mine) {
    const size_t off = (size_t)i * p + k;
    x = ld_group<ANY>(s.x + off, left);
    z = ld_group<ANY>(s.z + off, left);
    h = ld_group<ANY>((const float*)s.prob.data0 + off, left);
    c = ld_group<ANY>((const float*)s.prob.data1 + off, left);
    if (momentum) m = ld_group<ANY>(s.mom + off, left);
    // (a version that neither the array of S4 buffers nor the part of the ring on chip holds comes from the ring in memory)
#pragma unroll
    for (int u = 0; u < kL; ++u)
      if (u < dI) {
        where[u] = s.blk_head[kHeadWords * n + ce0 + u];
        outside |= (unsigned)(where[u] >> 1 & 1) << u;
        if (where[u] & 1) {
          last[u] = ld_group<ANY>(s.rho_tilde + (size_t)(ce0 + u) * p + k, left);
          prod |= 1u << u;
        } else if (!(where[u] & 4)) {
          last[u] = ld_group<ANY>(s.sigma_ring + ((size_t)(HUB ? i : s.c_src[ce0 + u]) * M + (where[u] >> 8 & 0xFF)) * p + k, left);
        }
      }
  }
  // rings, from the latest version back: kBatch versions of both in flight at a time, then into LDS; a version
  // that nobody can read any more is zeros instead (the multiply-adds with weight zero need finite values)
  constexpr int kBatch = PER >= 4 ? 5 : PER >= 3 ? 6 : kR <= 2 ? 12 : (kR <= 4 ? 10 : 8);
  const int64_t back_to_last = (int64_t)(M - 1) * p, to_sums = s.sigma_ring - s.v_ring;
  if (moves) {
    int at_g = head.x, at_l = head.y;
    const float* vg = s.v_ring + ((size_t)iT * M + at_g) * p + kT;
    for (int a0 = 0; a0 < K; a0 += kBatch) {
      float4 tv[kBatch], ts[kBatch];
      const unsigned get_v = (unsigned)head.z >> a0, get_s = (unsigned)head.w >> a0;  // bits past the oldest are clear
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        tv[u] = ts[u] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (get_v & (1u << u)) tv[u] = ld_group<ANY>(vg, leftT);
        if (get_s & (1u << u)) ts[u] = ld_group<ANY>(vg + to_sums, leftT);
        vg += at_g == 0 ? back_to_last : -p;
        at_g = at_g == 0 ? M - 1 : at_g - 1;
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (a0 + u < K) {
          if (mv_has_v) mv_v[__umul24((unsigned)at_l, (unsigned)lw)] = tv[u];
          if (mv_has_s) mv_s[__umul24((unsigned)at_l, (unsigned)lw)] = ts[u];
          at_l = at_l == 0 ? K - 1 : at_l - 1;
        }
    }
  }
  // The stored sample of S2b is a function of (x_i, t_i); from here on it lives in registers, and so
  // does the LDS address of the node's current version in its v ring (advanced by one slot per activation,
  // back to the first slot after the last: no division, no multiplication).
  unsigned a_cur = a_own;
  int ver_next = 1, ver_first = 1;  // version of the node's next activation (counted here: the plan's copy would need a mask and an add)
  const unsigned a_end = a_own + __umul24((unsigned)K, slot_bytes);
  if (mine) {
    const int t0 = s.blk_head[kHeadWords * i];
    g = diag_sample<VEC, MOM>(s, h, c, x, i, t0, k);
    a_cur = a_own + __umul24((unsigned)s.blk_head[kHeadWords * i + 9], slot_bytes);  // the place of version t0
    ver_next = ver_first = t0 + 1;
  }
  if (W > 1) __syncthreads();  // the tiles of the workgroup are in LDS
  else wave_sync();

  if (mine) {
    if (!FEW || dO > 0) sig = lds_ld(a_cur + to_sum);
#pragma unroll
    for (int u = 0; u < kL; ++u)
      if (where[u] & 4) last[u] = lds_ld(c_col[u] + __umul24((unsigned)(where[u] >> 16 & 0xFF), slot_bytes));
  }

  // one round with the plan words P, while those of the round after it arrive in N
  auto round = [&](int q, const Plan& P, Plan& N) {
    // the plan words of the next round, from global memory, used one round from now
    fetch(min(q + 1, blk.rounds - 1), N);
    float4 inbox = make_float4(0.f, 0.f, 0.f, 0.f);
    if (HUB) {
      const int hub = __builtin_amdgcn_readfirstlane(P.hub);
      if (hub < 0) {  // the hub is activated: what every sender adds to its sum, formed by the sender's lanes
        float4 term = make_float4(0.f, 0.f, 0.f, 0.f);
        float weight = c_w[0];  // ORDERED: that of the term
        if (dI > 0) {
          float4 sum = lds_ld(c_col[0] + __umul24((unsigned)P.c[0], slot_bytes));
          if (hub < (int)0xC0000000 && (P.c[0] & 1 << 30) != 0) {
            sum = ld_group<ANY>(s.sigma_ring + ((size_t)i * M + (P.c[0] >> 24 & 0x3F)) * p + k, left);
            __builtin_amdgcn_s_waitcnt(0x0F70);
          }
          term = ORDERED ? sub(sum, last[0]) : mul_s(c_w[0], sub(sum, last[0]));
          if (hub < (int)0xC0000000 && P.c[0] < 0) {
            term = sub(mul_s(c_w[0], sum), prod ? last[0] : mul_s(c_w[0], last[0]));
            weight = 1.f;
            prod = 0;
          }
          last[0] = sum;
        }
        if (ORDERED) {
          // z + a (sigma - sigma~) + ..., by the lanes of the hub (what the others form is of no use); the terms travel through LDS
          if (i < n) lds_st(terms + (unsigned)lane * (unsigned)sizeof(float4), term);
          wave_sync();
          inbox = z;
          float4 t[kStarInOrder - 1];
#pragma unroll
          for (int u = 0; u < kStarInOrder - 1; ++u)
            if (u < n - 1) t[u] = lds_ld(terms + (unsigned)((u + (u >= blk.hub ? 1 : 0)) * lw + ln) * (unsigned)sizeof(float4));
#pragma unroll
          for (int u = 0; u < kStarInOrder - 1; ++u)
            if (u < n - 1) inbox = fma_s(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(weight), (u + (u >= blk.hub ? 1 : 0)) * lw)), t[u], inbox);
        } else {
          inbox = sum_of_nodes(term, lane, n, i, ln, lw);
          if (i != blk.hub) inbox = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
    }
    if (P.node < 0) {  // bit 31: node i is activated in this round (never set in the zero word)
      float4 nb[kR], cur[kL];
      const unsigned a_new = a_cur + slot_bytes == a_end ? a_own : a_cur + slot_bytes;
      // every ring value of the round in one batch of LDS reads (what a missing edge reads is a valid address; its value
      // is multiplied by zero)
#pragma unroll
      for (int u = 0; u < kR; ++u) nb[u] = lds_ld(r_col[u] + __umul24((unsigned)P.r[u], slot_bytes));
#pragma unroll
      for (int u = 0; u < kC; ++u) cur[u] = lds_ld(c_col[u] + __umul24((unsigned)P.c[u], slot_bytes));
      const bool rare = P.node < (int)0xC0000000;  // bit 30 clear: one test for whatever is not the usual round
      if (rare) {
        // a version that the chip no longer holds: from the ring in memory, where it has been all along or was put when
        // it lost its place
        const int re0 = s.r_ptr[i];
#pragma unroll
        for (int u = 0; u < kR; ++u)
          if (P.r[u] & (1 << 30)) nb[u] = ld_group<ANY>(s.v_ring + ((size_t)s.r_src[re0 + u] * M + (P.r[u] >> 24 & 0x3F)) * p + k, left);
#pragma unroll
        for (int u = 0; u < kC; ++u)
          if (P.c[u] & (1 << 30)) cur[u] = ld_group<ANY>(s.sigma_ring + ((size_t)s.c_src[ce0 + u] * M + (P.c[u] >> 24 & 0x3F)) * p + k, left);
        // vmcnt(0), here: with these loads under way on one of two paths, every round waited for the plan words just asked for
        // (20 rounds of 16 nodes, p 11.2 M: 296 -> 263 us per round)
        __builtin_amdgcn_s_waitcnt(0x0F70);
        if (P.node & (1 << 29)) {  // the version whose place this round takes
          float* to = s.v_ring + ((size_t)i * M + (unsigned)(ver_next - K) % (unsigned)M) * p + k;
          if (pulled) st_group<ANY>(to, left, lds_ld(a_new));
          if (dO > 0) st_group<ANY>(to + to_sums, left, lds_ld(a_new + to_sum));
        }
      }
      // S1: local descent; with the optimizer variant along the heavy-ball buffer m <- beta m + z
      if (momentum) m = fma_s(s.beta, m, z);
      const float4 v = fma_s(-blk.gamma, momentum ? m : z, x);
      // S2a: pull the stamped neighbour copies and mix with row-stochastic weights
      float4 x_new = mul_s(r_self, v);
      // (a missing edge has weight zero and reads the node's own ring: it adds zero, without a branch)
#pragma unroll
      for (int u = 0; u < kR; ++u) x_new = fma_s(r_w[u], nb[u], x_new);
      const float4 g_new = diag_sample<VEC, MOM>(s, h, c, x_new, i, ver_next, k);
      ++ver_next;
      // S2b: tracker sum over the in-edges of C; S4: keep what was consumed.  An idle edge, whose stamp did not move, reads
      // the sum it holds already and adds zero: no branch.
      float4 z_half = ORDERED ? (i == blk.hub ? inbox : z) : HUB ? add(z, inbox) : z;
#pragma unroll
      for (int u = 0; u < kC; ++u) z_half = track_edge(z_half, c_w[u], cur[u], last[u], true);
      if (kC > 0 && rare) {  // once more, with what left the sender's ring of M before it was consumed as the product it was kept as
        z_half = z;
#pragma unroll
        for (int u = 0; u < kC; ++u) {
          if (P.c[u] < 0) {
            z_half = track_edge(z_half, c_w[u], cur[u], prod >> u & 1 ? last[u] : mul_s(c_w[u], last[u]), false);
            prod &= ~(1u << u);
          } else {
            z_half = track_edge(z_half, c_w[u], cur[u], last[u], true);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kC; ++u) last[u] = cur[u];
      z_half = sub(add(z_half, g_new), g);
      // S3: publish version t+1 (in the place of the oldest one, whose readers of this round are through); S2c: keep a_ii, push
      if (pulled) lds_st(a_new, v);
      sig = add(sig, z_half);
      if (dO > 0) lds_st(a_new + to_sum, sig);
      x = x_new;
      z = mul_s(c_self, z_half);
      g = g_new;
      a_cur = a_new;
    }
    wave_sync();  // S5: the round is over, its publications are visible to the lanes of this wavefront
  };
  // (two rounds at a time, so that the two sets of plan words stay where they are)
  if (wave_has) {
    for (int q = 0; q < blk.rounds; q += 2) {
      round(q, plan_a, plan_b);
      if (q + 1 < blk.rounds) round(q + 1, plan_b, plan_a);
    }
  }
  // The last plan words asked for are not used.  They are looked at here all the same, on every path: memory
  // operations complete in order, and as long as the compiler has to assume that a load may still be under way on
  // some path, each wait it places for that load in the write-back is a wait for every store issued before it.
  auto settle = [](const Plan& P) {
    asm volatile("" ::"v"(P.node));
#pragma unroll
    for (int u = 0; u < kR; ++u) asm volatile("" ::"v"(P.r[u]));
#pragma unroll
    for (int u = 0; u < kL; ++u) asm volatile("" ::"v"(P.c[u]));
    if (HUB) asm volatile("" ::"v"(P.hub));
  };
  settle(plan_a);
  settle(plan_b);

  // Write-back.  With blk.rebase the running sums are rebased on the way (what rfast_rebase_kernel does, and with
  // its operations): sender j's latest sum leaves every slot of its ring, and a_ij times it every buffer it feeds.
  if (mine) {
    const size_t off = (size_t)i * p + k;
    if (ver_next != ver_first) {  // x and z of a node that was not activated are what they were
      st_group<ANY>(s.x + off, left, x);
      st_group<ANY>(s.z + off, left, z);
      if (momentum) st_group<ANY>(s.mom + off, left, m);
    }
#pragma unroll
    for (int u = 0; u < kL; ++u)
      // the buffer lives in the array only if its version is outside the sender's ring now
      if (outside >> u & 1) {
        float4 rt = prod >> u & 1 ? last[u] : mul_s(c_w[u], last[u]);
        if (HUB && blk.rebase) {
          rt = sub(rt, mul_s(c_w[u], sig));
        } else if (blk.rebase) {
          const int end = s.blk_head[kHeadWords * s.c_src[ce0 + u] + 13];  // of the sender's latest version
          rt = sub(rt, mul_s(c_w[u], lds_ld(c_col[u] + __umul24((unsigned)end, slot_bytes))));
        }
        st_group<ANY>(s.rho_tilde + (size_t)(ce0 + u) * p + k, left, rt);
      }
  }
  if (W > 1) __syncthreads();  // every wavefront of the workgroup is through with its rounds
  else wave_sync();
  if (moves) {
    const unsigned put_v = (unsigned)tail.z, put_s = (unsigned)tail.w;
    float4 base = make_float4(0.f, 0.f, 0.f, 0.f);
    const bool shift = blk.rebase && put_s != 0;  // nobody reads the sums of a node without out-edges
    if (shift) base = mv_s[__umul24((unsigned)tail.y, (unsigned)lw)];
    int at_g = tail.x, at_l = tail.y;
    float* vg = s.v_ring + ((size_t)iT * M + at_g) * p + kT;
    for (int a0 = 0; a0 < K; a0 += kBatch) {
      float4 tv[kBatch], ts[kBatch];
      const unsigned back_v = put_v >> a0, back_s = put_s >> a0;  // bits past the oldest are clear
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (a0 + u < K) {
          if (back_v & (1u << u)) tv[u] = mv_v[__umul24((unsigned)at_l, (unsigned)lw)];
          if (back_s & (1u << u)) {
            ts[u] = mv_s[__umul24((unsigned)at_l, (unsigned)lw)];
            if (shift) ts[u] = sub(ts[u], base);
          }
          at_l = at_l == 0 ? K - 1 : at_l - 1;
        }
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (a0 + u < K) {
          if (back_v & (1u << u)) st_group<ANY>(vg, leftT, tv[u]);
          if (back_s & (1u << u)) st_group<ANY>(vg + to_sums, leftT, ts[u]);
          vg += at_g == 0 ? back_to_last : -p;
          at_g = at_g == 0 ? M - 1 : at_g - 1;
        }
    }
    if (shift)
      for (int a = K; a < M; ++a) {  // sums that are no longer on chip
        if (put_s >> a & 1) st_group<ANY>(vg + to_sums, leftT, sub(ld_group<ANY>(vg + to_sums, leftT), base));
        vg += at_g == 0 ? back_to_last : -p;
        at_g = at_g == 0 ? M - 1 : at_g - 1;
      }
  }
}

// ---------------------------------------------------------------------------
// The synchronous push-pull step of eq. (2), several steps per launch, on the same tiling: every
// node steps at once and reads its neighbours' current x - gamma z and z, which the lanes of the
// wavefront exchange through two LDS rows per node.  x, z, the stored sample and the objective data
// stay in registers; the arithmetic is that of rfast_sync_descent_kernel + rfast_sync_step_kernel
// (the stored sample of a step is the new sample of the step before: the same function of the same
// arguments that the one-step kernels recompute).  On return z is in its own array and slot 0 of
// the v ring holds the last x - gamma z, as after the one-step kernels.
// ---------------------------------------------------------------------------
template <int kDeg, bool MOM, bool ANY>
__global__ void __launch_bounds__(64) rfast_sync_wave_kernel(RfastDev s, float gamma, int rounds, int lw) {
  constexpr int VEC = 4;
  extern __shared__ float4 lds4[];
  const int n = s.n;
  const int64_t p = s.p;
  const int lane = threadIdx.x;
  const int i = lane / lw, ln = lane - i * lw;
  const unsigned xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int64_t tile = ((int64_t)(slot / kSyncTileRun) * kXcds + xcd) * kSyncTileRun + slot % kSyncTileRun;
  const int64_t k = tile * (4 * lw) + ln * 4;
  const bool mine = i < n && k < p;
  float4* v_l = lds4;                   // [n][lw]
  float4* z_l = v_l + (size_t)n * lw;   // [n][lw]
  if (!mine) return;  // no barrier below: the lanes of a wavefront without coordinates may leave
  const int left = p - k < 4 ? (int)(p - k) : 4;  // ANY: coordinates of the row from the lane's first one on
  const int own = i * lw + ln;
  const size_t off = (size_t)i * p + k;
  float4 x = ld_group<ANY>(s.x + off, left), z = ld_group<ANY>(s.z + off, left);
  const float4 h = ld_group<ANY>((const float*)s.prob.data0 + off, left), c = ld_group<ANY>((const float*)s.prob.data1 + off, left);
  float4 m = make_float4(0.f, 0.f, 0.f, 0.f);
  if (MOM) m = ld_group<ANY>(s.mom + off, left);
  const int re0 = s.r_ptr[i], ce0 = s.c_ptr[i];
  const int dR = s.r_ptr[i + 1] - re0, dI = s.c_ptr[i + 1] - ce0;
  const float r_self = s.r_self[i], c_self = s.c_self[i];
  int r_col[kDeg], c_col[kDeg];
  float r_w[kDeg], c_w[kDeg];
#pragma unroll
  for (int u = 0; u < kDeg; ++u) {
    r_col[u] = (u < dR ? s.r_src[re0 + u] : i) * lw + ln;
    r_w[u] = u < dR ? s.r_w[re0 + u] : 0.f;
    c_col[u] = (u < dI ? s.c_src[ce0 + u] : i) * lw + ln;
    c_w[u] = u < dI ? s.c_w[ce0 + u] : 0.f;
  }
  int t = s.t[i];
  float4 g = diag_sample<VEC>(s, h, c, x, i, t, k), v = x;
  for (int q = 0; q < rounds; ++q) {
    if (MOM) m = fma_s(s.beta, m, z);
    v = fma_s(-gamma, MOM ? m : z, x);
    v_l[own] = v;
    z_l[own] = z;
    wave_sync();  // every node's v and z of this step are out
    float4 nb[kDeg], zb[kDeg];
#pragma unroll
    for (int u = 0; u < kDeg; ++u) {
      nb[u] = v_l[r_col[u]];
      zb[u] = z_l[c_col[u]];
    }
    float4 x_new = mul_s(r_self, v);
#pragma unroll
    for (int u = 0; u < kDeg; ++u) x_new = fma_s(r_w[u], nb[u], x_new);  // a missing edge: weight zero, own row
    const float4 g_new = diag_sample<VEC>(s, h, c, x_new, i, t + 1, k);
    float4 z_new = mul_s(c_self, z);
#pragma unroll
    for (int u = 0; u < kDeg; ++u) z_new = fma_s(c_w[u], zb[u], z_new);
    z_new = sub(add(z_new, g_new), g);
    wave_sync();  // every read of this step is done before the next one overwrites the rows
    x = x_new;
    z = z_new;
    g = g_new;
    ++t;
  }
  st_group<ANY>(s.x + off, left, x);
  st_group<ANY>(s.z + off, left, z);
  if (MOM) st_group<ANY>(s.mom + off, left, m);
  st_group<ANY>(s.v_ring + (size_t)i * s.M * p + k, left, v);
}

constexpr int kUnits = 256;
constexpr size_t kCuLds = 160 * 1024, kLdsGrain = 1280;  // LDS of a compute unit, and what it is handed out in

// LDS of one wavefront's tile with `slots` versions per node
size_t wave_lds_bytes(const rfast_ctx* c, int slots, int rings) { return (size_t)rings * slots * (64 / c->d.n) * sizeof(float4); }
size_t wave_lds_bytes(const rfast_ctx* c, int slots) {
  const bool in_order = c->hub >= 0 && c->d.n <= kStarInOrder;  // (and a term per lane)
  return wave_lds_bytes(c, slots, c->v_rows + c->s_rows) + (in_order ? (size_t)c->d.n * (64 / c->d.n) * sizeof(float4) : 0);
}
// Wavefronts of that size that a compute unit holds, `per` to a SIMD at most.
int wave_resident(const rfast_ctx* c, int slots, int per, int rings) {
  const size_t one = (wave_lds_bytes(c, slots, rings) + kLdsGrain - 1) / kLdsGrain * kLdsGrain;
  return (int)std::min<size_t>(kCuLds / one, (size_t)(4 * per));
}
int wave_resident(const rfast_ctx* c, int slots, int per) { return wave_resident(c, slots, per, c->v_rows + c->s_rows); }


}  // namespace

// The separable objective, at most 64 nodes with at most kWaveMaxDeg edges of a
// kind each or one receiver of all edges of C, rings of at most 32 slots (one bit per version in the records of the resolver; the LDS of one
// wavefront's tile is 64 KB at most then).
bool rfast_wave_eligible(const rfast_ctx* c) {
  const RfastDev& d = c->d;
  return d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC && (c->max_degree <= kWaveMaxDeg || c->hub >= 0) && d.n <= kWaveMaxNodes && d.M <= 32;
}

int rfast_wave_lanes(const rfast_ctx* c) { return 64 / c->d.n; }

// (Stars and graphs with at most two edges of a kind: fewer versions than the longest delay reads where that gives more wavefronts, until there
// are two per SIMD, down to three quarters of it.  A wavefront has few edges to read over then, so that a read from the ring in memory is
// rare, and delays count rounds, versions only the sender's active ones.  Delays of up to 16, 20 % lost, 132 rounds, ms with 18 / 14 / 13 / 12 / 10
// versions, half of the nodes active and all (13 is what this takes: as many as fit beside the wavefronts that 12 allow): bidirectional ring
// of 16, p 1 M, 4.30 / 3.50 / 3.00 / 3.00 / 2.62 and 4.27 / 3.51 / 3.11 / 3.57 / 5.05; of 32, p 524288, 4.52 / 4.02 / 3.36 / 3.42 / 3.08 and 4.59 / 4.29 /
// 3.63 / 4.16 / 6.16; binary tree of 64, p 262144, 3.84 / 2.93 / 2.44 / 2.48 / 2.97 and 4.00 / 3.30 / 2.81 / 3.21 / 5.86; star of 64, p 524288, 9.26 / 7.43 /
// 5.86 / 5.80 / 6.48 and 10.5 / 8.53 / 6.97 / 7.46 / 11.2.  With 2 % lost 13 take up to 6 % less, with half lost up to
// 16 % more, and are the best of them there with all active.  Not where the chip holds every tile as it is: fewer versions only
// cost then (ring of 32, p 8192, all active: 0.86).  With more edges all nodes active lose what half of them
// gain: mesh of 64, 5.61 / 5.21 / 4.46 / 4.97 and 5.73 / 8.91 / 8.19 / 11.5.)
// Wavefronts per SIMD (the instantiation) and versions of a node on chip.  At least as many versions as the longest delay
// reads, and one more: with none to spare the reads of versions that have left the chip cost more than the wavefronts bring
// (16 nodes, p 11.2 M, delays of up to 4, five versions and sixteen wavefronts against six and twelve, us per round of
// 20: 255 against 263 where 2 % of the packets are lost, 353 against 274 where 20 % are).  Then as many more as
// LDS has room for at that number of wavefronts.
struct WaveShape {
  int per, slots;
};
static int wave_most(const rfast_ctx* c) { return c->hub >= 0 || c->max_degree <= 2 ? 4 : c->max_degree <= 4 ? 3 : 2; }
static WaveShape wave_shape(const rfast_ctx* c) {
  const RfastDev& d = c->d;
  int least = std::min(d.M - 1, d.d_max + 2);
  const bool in_order = c->hub >= 0 && d.n <= kStarInOrder;  // (has one form, for four wavefronts per SIMD)
  const int64_t tiles = (d.p + 4 * (64 / d.n) - 1) / (4 * (64 / d.n));
  if (c->hub >= 0 || c->max_degree <= 2)
    while (least > (3 * d.d_max + 3) / 4 && wave_resident(c, least, 2) < 8 && tiles > (int64_t)kUnits * wave_resident(c, least, 2)) --least;
  WaveShape w;
  for (w.per = wave_most(c); !in_order && w.per > 2 && wave_resident(c, least, w.per) < 4 * w.per;) --w.per;
  w.slots = least;
  while (w.slots < d.M - 1 && wave_resident(c, w.slots + 1, w.per) == wave_resident(c, least, w.per)) ++w.slots;
  return w;
}
int rfast_wave_slots(const rfast_ctx* c) { return wave_shape(c).slots; }
int rfast_wave_held(const rfast_ctx* c) {
  const int reach = std::min(c->d.M - 1, c->d.d_max + 2), rings = 2 * c->d.n;
  int per = wave_most(c);
  while (per > 2 && wave_resident(c, reach, per, rings) < 4 * per) --per;
  return wave_resident(c, reach, per, rings);
}

// Wavefronts per workgroup, as many as LDS holds without losing a resident wavefront.  Short launches, which are
// mostly tile movement, gain from row segments of whole cache lines; in long ones the barriers of a workgroup weigh as much.
// Measured with 1 / 2 / 4 wavefronts, us per round: 16 nodes x 11.2 M, 8 rounds 530 / 496 / 486, 20 rounds 260 / 250 /
// 244, 32 rounds 206 / 202 / 202, 64 and more even; from 22 nodes on, where the segment of one tile is 16 or 32 bytes, at any length: mesh of 64, p 1 M, 20
// rounds 6.3 / 5.0 / 4.4 ms, 100 rounds 11.6 / 10.6 / 9.9, 400 rounds 36.4 / 34.4 / 33.0, ring of 64 8.0 / 7.1 / 6.8 of 100, mesh of 32 4.18 / 4.09 / 3.99; 32 nodes x 1 M, six edge slots, 10 rounds 149 / 138 / 140, 20 rounds 93 / 88 / 87; 8 nodes
// x 3 M, 20 rounds 26.3 / 26.4 / 25.4.
static int wave_group(const rfast_ctx* c, int rounds, WaveShape shape) {
  const RfastDev& d = c->d;
  const size_t one = wave_lds_bytes(c, shape.slots);
  if (c->wave_group == 1 || c->wave_group == 2 || c->wave_group == 4) return (size_t)c->wave_group * one <= kCuLds ? c->wave_group : 1;
  if (rounds > 64 && 64 / d.n > 2) return 1;
  const size_t most = (size_t)(4 * shape.per), resident = (size_t)wave_resident(c, shape.slots, shape.per);
  int w = 1;
  // (a resident wavefront fewer is no loss where the chip holds all tiles even so: binary tree of 64, p 4096, delays of up to 16, calls of 8: 26 -> 23 us)
  const size_t tiles = (size_t)((d.p + 4 * (64 / d.n) - 1) / (4 * (64 / d.n)));
  auto enough = [&](size_t held) { return held >= resident || (held > 0 && tiles <= (size_t)kUnits * held); };
  while (w < 4 && enough(std::min<size_t>(kCuLds / (2 * w * one) * (2 * w), most))) w *= 2;
  return w;
}

template <class Form, bool MOM, int W, bool ANY, int PER>
static hipError_t launch_wave(rfast_ctx* c, const RfastBlock& blk) {
  static bool raised = false;
  if (!raised) {  // more than 64 KB of dynamic LDS has to be asked for once per kernel
    const hipError_t e = hipFuncSetAttribute((const void*)rfast_wave_kernel<Form::r, Form::c, Form::few, MOM, W, ANY, PER>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    raised = true;
  }
  const RfastDev& d = c->d;
  if (!d.blk_plan || !d.blk_head || blk.slots < 1 || blk.slots > d.M - 1 || blk.slots != d.blk_slots) return hipErrorInvalidValue;
  const int lw = 64 / d.n;
  const int64_t run = (int64_t)kXcds * (kTileRun / W), per = (int64_t)4 * lw * W;
  const int64_t groups = ((d.p + per - 1) / per + run - 1) / run * run;  // whole runs: a workgroup past the end leaves at once
  if (groups > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((rfast_wave_kernel<Form::r, Form::c, Form::few, MOM, W, ANY, PER>), dim3((unsigned)groups), dim3(64 * W),
                     (size_t)W * wave_lds_bytes(c, blk.slots), c->stream, c->d, blk, lw, wave_div(lw, W));
  return hipGetLastError();
}

// A launch that does nothing (one workgroup that finds no coordinates and leaves): the first launch of a kernel
// pays for loading its code, about 0.7 ms, which belongs to setting a context up and not to its first run.
template <class Form, bool MOM, int W, bool ANY, int PER>
static hipError_t prime_wave(rfast_ctx* c) {
  const hipError_t e = hipFuncSetAttribute((const void*)rfast_wave_kernel<Form::r, Form::c, Form::few, MOM, W, ANY, PER>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e != hipSuccess) return e;
  RfastDev none = c->d;
  none.p = 0;
  RfastBlock blk;
  blk.gamma = 0.f;
  blk.rounds = 0;
  blk.rebase = 0;
  blk.slots = 1;
  blk.hub = 0;
  blk.v_rows = blk.s_rows = 0;
  hipLaunchKernelGGL((rfast_wave_kernel<Form::r, Form::c, Form::few, MOM, W, ANY, PER>), dim3(1), dim3(64 * W), 0, c->stream, none, blk, 64 / c->d.n, wave_div(64 / c->d.n, W));
  return hipGetLastError();
}

// (the forms of long and of short launches: a third that rfast_set_tile_group may choose cost every context 0.2 ms)
template <class Form, bool MOM, int PER>
static hipError_t prime_wave_w(rfast_ctx* c, WaveShape shape) {
  const int brief = wave_group(c, 1, shape);
  if (c->d.p % 4 != 0) {
    const hipError_t e = prime_wave<Form, MOM, 1, true, PER>(c);
    return e == hipSuccess && brief == 4 ? prime_wave<Form, MOM, 4, true, PER>(c) : e;
  }
  const hipError_t e = prime_wave<Form, MOM, 1, false, PER>(c);
  if (e == hipSuccess && brief == 2) return prime_wave<Form, MOM, 2, false, PER>(c);
  return e == hipSuccess && brief == 4 ? prime_wave<Form, MOM, 4, false, PER>(c) : e;
}

// Edge slots of a node over R and over C (0, -1: the edges of C all lead to one node), and whether only nodes with readers have rings.
template <int kR, int kC, bool FEW> struct WaveForm {
  static constexpr int r = kR, c = kC;
  static constexpr bool few = FEW;
};

// The instantiation for the edges of this context, its optimizer and a launch of that many rounds: f(form, optimizer, per SIMD).
template <class F> static hipError_t with_wave_form(const rfast_ctx* c, int per, F f) {
  using T = std::true_type;
  using N = std::false_type;
  const int deg = c->max_degree;
  auto by_per = [&](auto form, auto mom) {
    if (per == 4) return f(form, mom, std::integral_constant<int, 4>());
    return per == 3 ? f(form, mom, std::integral_constant<int, 3>()) : f(form, mom, std::integral_constant<int, 2>());
  };
  auto by_deg = [&](auto mom) {
    if (c->hub >= 0 && c->d.n <= kStarInOrder) return f(WaveForm<1, -1, true>(), mom, std::integral_constant<int, 4>());
    if (c->hub >= 0) return by_per(WaveForm<1, 0, true>(), mom);
    // (a tree takes this form only where its rings leave no room for sixteen wavefronts: more than 640 slots of 16 bytes each)
    if (c->tree)
      return per >= 3 ? f(WaveForm<1, 2, true>(), mom, std::integral_constant<int, 3>()) : f(WaveForm<1, 2, true>(), mom, std::integral_constant<int, 2>());
    if (deg > 4) return f(WaveForm<kWaveMaxDeg, kWaveMaxDeg, false>(), mom, std::integral_constant<int, 2>());
    if (deg > 2)
      return per == 3 ? f(WaveForm<4, 4, false>(), mom, std::integral_constant<int, 3>())
                      : f(WaveForm<4, 4, false>(), mom, std::integral_constant<int, 2>());
    return by_per(WaveForm<2, 2, false>(), mom);
  };
  return c->d.mom || c->d.wd != 0.f ? by_deg(T()) : by_deg(N());
}

// Loads the instantiations of the multi-round kernel that this context can launch (rfast_create,
// rfast_set_optimizer).
hipError_t rfast_wave_prime(rfast_ctx* c) {
  if (!rfast_wave_eligible(c) || rfast_block_takes(c, kBlockRounds)) return hipSuccess;
  const WaveShape shape = wave_shape(c);
  return with_wave_form(c, shape.per, [&](auto form, auto mom, auto per) { return prime_wave_w<decltype(form), mom.value, per.value>(c, shape); });
}

hipError_t rfast_launch_wave(rfast_ctx* c, const RfastBlock& blk) {
  const WaveShape shape = wave_shape(c);
  if (shape.slots != blk.slots) return hipErrorInvalidValue;
  return with_wave_form(c, shape.per, [&](auto form, auto mom, auto per) {
    if (c->d.p % 4 != 0)
      return c->wave_group == 0 && wave_group(c, blk.rounds, shape) == 4 ? launch_wave<decltype(form), mom.value, 4, true, per.value>(c, blk)
                                                                         : launch_wave<decltype(form), mom.value, 1, true, per.value>(c, blk);
    switch (wave_group(c, blk.rounds, shape)) {
      case 4: return launch_wave<decltype(form), mom.value, 4, false, per.value>(c, blk);
      case 2: return launch_wave<decltype(form), mom.value, 2, false, per.value>(c, blk);
      default: return launch_wave<decltype(form), mom.value, 1, false, per.value>(c, blk);
    }
  });
}

// The synchronous mode through the multi-step kernel: the separable objective,
// at most 64 nodes with at most kWaveMaxDeg in-edges of a kind each (64 nodes of a mesh, p 500000, calls of 50: 367 us per
// step one launch each, 25 this way; calls of 4: 367 / 135).
bool rfast_sync_wave_eligible(const rfast_ctx* c) {
  const RfastDev& d = c->d;
  return d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC && c->max_degree <= kWaveMaxDeg && d.n <= kWaveMaxNodes;
}

template <int kDeg, bool MOM>
static hipError_t launch_sync_wave(rfast_ctx* c, float gamma, int rounds) {
  const RfastDev& d = c->d;
  const int lw = 64 / d.n;
  const int64_t run = (int64_t)kXcds * kSyncTileRun;
  const int64_t tiles = ((d.p + 4 * lw - 1) / (4 * lw) + run - 1) / run * run;
  if (tiles > 0x7fffffffLL) return hipErrorInvalidValue;
  if (d.p % 4 != 0)
    hipLaunchKernelGGL((rfast_sync_wave_kernel<kDeg, MOM, true>), dim3((unsigned)tiles), dim3(64),
                       (size_t)2 * d.n * lw * sizeof(float4), c->stream, c->d, gamma, rounds, lw);
  else
    hipLaunchKernelGGL((rfast_sync_wave_kernel<kDeg, MOM, false>), dim3((unsigned)tiles), dim3(64),
                       (size_t)2 * d.n * lw * sizeof(float4), c->stream, c->d, gamma, rounds, lw);
  return hipGetLastError();
}

hipError_t rfast_launch_sync_wave(rfast_ctx* c, float gamma, int rounds) {
  const int deg = c->max_degree;
  if (c->d.mom)
    return deg <= 2 ? launch_sync_wave<2, true>(c, gamma, rounds)
                    : (deg <= 4 ? launch_sync_wave<4, true>(c, gamma, rounds) : launch_sync_wave<kWaveMaxDeg, true>(c, gamma, rounds));
  return deg <= 2 ? launch_sync_wave<2, false>(c, gamma, rounds)
                  : (deg <= 4 ? launch_sync_wave<4, false>(c, gamma, rounds) : launch_sync_wave<kWaveMaxDeg, false>(c, gamma, rounds));
}
