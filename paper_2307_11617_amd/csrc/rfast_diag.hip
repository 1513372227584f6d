// Diagnostics of the current state as wavefront reductions:
//   consensus error ||x - 1 xbar^T||^2 and optimality gap ||xbar - x*||^2 (the
//   quantities of Theorem 1 and the merit function of Theorem 2), ||z||^2, and
//   the residual of the tracking-conservation identity of Lemma 3,
//   sum_i z_i + sum_e (rho_e latest - rho~_e) - sum_i g_i  (zero in exact arithmetic).
// One lane owns four consecutive coordinates
// and walks over the nodes once, then over the edges of C (coalesced along k, the arrays of the nodes read once);
// partial sums are kept in fp64, reduced across the 64 lanes with shuffles
// then across the workgroup through LDS, and added to the result with one fp64 atomic per workgroup.
#include "rfast_vec.h"

namespace {

constexpr int kThreads = 256;

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__global__ void rfast_diag_zero(double* out) {
  if (threadIdx.x < 8) out[threadIdx.x] = 0.0;
}

template <int VEC>
__device__ inline float comp(const typename V<VEC>::T& v, int u) { return reinterpret_cast<const float*>(&v)[u]; }

// The coordinates of one lane (one Philox call per node for a group of four), added to acc.
template <int VEC>
__device__ inline void diag_group(const RfastDev& s, const float* xstar, int64_t k, double (&acc)[7]) {
  using T = typename V<VEC>::T;
  constexpr int W = V<VEC>::W;
  const int64_t p = s.p;
  const bool separable = s.prob.kind == RFAST_OBJ_DIAG_QUADRATIC;
  const float* hp = (const float*)s.prob.data0;
  const float* cp = (const float*)s.prob.data1;
  // One walk over the nodes, their arrays read once.  What needs the average xbar, which is known only after
  // the walk, is accumulated about a reference that is known from the start, node 0's own value:
  //   sum_i (x_i - xbar)^2 = sum_i d_i^2 - 2 dx sum_i d_i + n dx^2,       d_i = x_i - x_0, dx = xbar - x_0
  //   sum_i h_i (xbar - c_i)^2 = dc^2 sum_i h_i - 2 dc sum_i h_i f_i + sum_i h_i f_i^2,  f_i = c_i - c_0, dc = xbar - c_0
  // (differences of fp32 values, exact in fp64; whatever cancels in these sums is of the size of the spread of
  // the x_i, or of the c_i, not of the values themselves).
  double gs[W], flight[W], sd[W], sd2[W], sh[W], shf[W], shf2[W];  // flight: sum of the z_i, then what is on the edges too
  float x0[W], c0[W];
#pragma unroll
  for (int u = 0; u < W; ++u) {
    gs[u] = flight[u] = sd[u] = sd2[u] = sh[u] = shf[u] = shf2[u] = 0.0;
    x0[u] = c0[u] = 0.f;
  }
#pragma unroll 1
  for (int i = 0; i < s.n; ++i) {
    const size_t off = (size_t)i * p + k;
    const int ti = s.t[i];
    const T x = V<VEC>::ld(s.x + off), z = V<VEC>::ld(s.z + off);
    T h, c, g;
    if (separable) {
      // the separable objective keeps no sample in memory: it is a function of (x_i, t_i)
      h = V<VEC>::ld(hp + off);
      c = V<VEC>::ld(cp + off);
      g = diag_sample<VEC>(s, h, c, x, i, ti, k);
    } else {
      g = V<VEC>::ld(s.g + (size_t)(ti & 1) * s.n * p + off);
    }
#pragma unroll
    for (int u = 0; u < W; ++u) {
      const double zi = comp<VEC>(z, u);
      if (i == 0) x0[u] = comp<VEC>(x, u);
      const double d = (double)comp<VEC>(x, u) - (double)x0[u];
      sd[u] += d;
      sd2[u] += d * d;
      flight[u] += zi;
      acc[1] += zi * zi;
      gs[u] += comp<VEC>(g, u);
      if (separable) {
        const double hi = comp<VEC>(h, u);
        if (i == 0) c0[u] = comp<VEC>(c, u);
        const double f = (double)comp<VEC>(c, u) - (double)c0[u];
        sh[u] += hi;
        shf[u] += hi * f;
        shf2[u] += hi * f * f;
      }
    }
  }
#pragma unroll 2
  for (int e = 0; e < s.eC; ++e) {
    const int j = s.c_src[e];
    const int tj = s.t[j], tau = s.tau_c[e];
    const float a = s.c_w[e];
    const float* ring = s.sigma_ring + (size_t)j * s.M * p + k;
    const T latest = V<VEC>::ld(ring + (size_t)(tj % s.M) * p);
    // rho~ is read from the sender's ring while its version is still there (tau >= t_j - D)
    const bool in_ring = tau >= tj - (s.M - 2);
    const T last = V<VEC>::ld(in_ring ? ring + (size_t)(tau % s.M) * p : s.rho_tilde + (size_t)e * p + k);
#pragma unroll
    for (int u = 0; u < W; ++u) {
      const float rt = in_ring ? a * comp<VEC>(last, u) : comp<VEC>(last, u);
      flight[u] += (double)(a * comp<VEC>(latest, u)) - (double)rt;
    }
  }
  T xbar_f, xs_f;
  if (xstar) xs_f = V<VEC>::ld(xstar + k);
#pragma unroll
  for (int u = 0; u < W; ++u) {
    const double dx = sd[u] / s.n, xbar = (double)x0[u] + dx;
    reinterpret_cast<float*>(&xbar_f)[u] = (float)xbar;
    acc[6] += xbar * xbar;
    acc[0] += sd2[u] - 2.0 * dx * sd[u] + s.n * dx * dx;
    if (separable) {
      const double dc = xbar - (double)c0[u];
      acc[5] += 0.5 * (dc * dc * sh[u] - 2.0 * dc * shf[u] + shf2[u]);
    }
    const double res = flight[u] - gs[u];
    acc[2] += res * res;
    acc[3] += gs[u] * gs[u];
    if (xstar) acc[4] += (xbar - comp<VEC>(xs_f, u)) * (xbar - comp<VEC>(xs_f, u));
  }
  if (s.xbar) V<VEC>::st(s.xbar + k, xbar_f);  // staged for the loss kernels of the objectives that need it
}

// VEC = 4: four coordinates per lane and step; VEC = 5: the same where p is not a multiple of four.
template <int VEC>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) rfast_diag_kernel(RfastDev s, const float* xstar, double* out) {
  double acc[7] = {0, 0, 0, 0, 0, 0, 0};
  const int64_t tiles = group_tiles(s.p);
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x)
    each_group<VEC>(tile, s.p, [&](auto vec, int64_t k) { diag_group<decltype(vec)::value>(s, xstar, k, acc); });
  // one fp64 atomic per quantity and workgroup: the seven results are single addresses, and
  // tens of thousands of atomics on them would serialise
  __shared__ double part[kThreads / 64][7];
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    const double w = wave_sum(acc[q]);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][q] = w;
  }
  __syncthreads();
  if (threadIdx.x < 7) {
    double w = 0.0;
    for (int v = 0; v < kThreads / 64; ++v) w += part[v][threadIdx.x];
    atomicAdd(&out[threadIdx.x], w);
  }
}

// The same sums where p is small: with four coordinates per lane a vector of 4096 is four workgroups, each of which goes
// through the nodes and edges one after the other (105.6 us on 32 nodes with 160 edges).  Here a workgroup takes 64
// coordinates, and its sixteen wavefronts share out the nodes and the edges; the partial sums of a coordinate meet in
// LDS, and the seven results, one cache line, take one atomic instruction per workgroup (n 48, p 4096, 96 edges: 68.4 ->
// 14.7 us; with an atomic of its own for each, some 9 ns apiece, it was 23.8).
constexpr int kSplitWaves = 16;
__global__ void __launch_bounds__(64 * kSplitWaves) rfast_diag_split_kernel(RfastDev s, const float* xstar, double* out) {
  __shared__ double part[kSplitWaves][8][64];  // flight, gs, sd, sd2, sh, shf, shf2, z_sq of a coordinate
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t p = s.p, k = (int64_t)blockIdx.x * 64 + lane;
  const bool separable = s.prob.kind == RFAST_OBJ_DIAG_QUADRATIC, mine = k < p;
  const float* hp = (const float*)s.prob.data0;
  const float* cp = (const float*)s.prob.data1;
  double flight = 0, gs = 0, sd = 0, sd2 = 0, sh = 0, shf = 0, shf2 = 0, z_sq = 0;
  float x0 = 0.f, c0 = 0.f;
  if (mine) {
    x0 = s.x[k];
    if (separable) c0 = cp[k];
#pragma unroll 4
    for (int i = wave; i < s.n; i += kSplitWaves) {
      const size_t off = (size_t)i * p + k;
      const int ti = s.t[i];
      const float x = s.x[off], z = s.z[off];
      float g;
      if (separable) {
        const float h = hp[off], c = cp[off];
        g = diag_sample<1>(s, h, c, x, i, ti, k);
        const double f = (double)c - (double)c0;
        sh += h;
        shf += h * f;
        shf2 += h * f * f;
      } else {
        g = s.g[(size_t)(ti & 1) * s.n * p + off];
      }
      const double d = (double)x - (double)x0;
      sd += d;
      sd2 += d * d;
      flight += z;
      z_sq += (double)z * z;
      gs += g;
    }
#pragma unroll 8
    for (int e = wave; e < s.eC; e += kSplitWaves) {
      const int j = s.c_src[e];
      const int tj = s.t[j], tau = s.tau_c[e];
      const float a = s.c_w[e];
      const float* ring = s.sigma_ring + (size_t)j * s.M * p + k;
      const bool in_ring = tau >= tj - (s.M - 2);
      const float latest = ring[(size_t)(tj % s.M) * p];
      const float last = *(in_ring ? ring + (size_t)(tau % s.M) * p : s.rho_tilde + (size_t)e * p + k);
      flight += (double)(a * latest) - (double)(in_ring ? a * last : last);
    }
  }
  double* mail = &part[wave][0][lane];
  mail[0] = flight; mail[64] = gs; mail[128] = sd; mail[192] = sd2; mail[256] = sh; mail[320] = shf; mail[384] = shf2; mail[448] = z_sq;
  __syncthreads();
  if (wave != 0) return;
  for (int w = 1; w < kSplitWaves; ++w) {
    const double* m = &part[w][0][lane];
    flight += m[0]; gs += m[64]; sd += m[128]; sd2 += m[192]; sh += m[256]; shf += m[320]; shf2 += m[384]; z_sq += m[448];
  }
  double acc[7] = {0, 0, 0, 0, 0, 0, 0};
  if (mine) {
    const double dx = sd / s.n, xbar = (double)x0 + dx;
    acc[6] = xbar * xbar;
    acc[0] = sd2 - 2.0 * dx * sd + s.n * dx * dx;
    if (separable) {
      const double dc = xbar - (double)c0;
      acc[5] = 0.5 * (dc * dc * sh - 2.0 * dc * shf + shf2);
    }
    const double res = flight - gs;
    acc[2] = res * res;
    acc[3] = gs * gs;
    if (xstar) acc[4] = (xbar - xstar[k]) * (xbar - xstar[k]);
    if (s.xbar) s.xbar[k] = (float)xbar;
  }
  acc[1] = z_sq;
  double sum = 0.0;  // the results lie in one cache line: seven lanes add to it with one instruction
#pragma unroll
  for (int q = 0; q < 7; ++q) {
    const double w = wave_sum(acc[q]);
    if (lane == q) sum = w;
  }
  if (lane < 7) atomicAdd(&out[lane], sum);
}

// sum_i f_i(xbar) for least squares and logistic regression over each node's FULL local data.  The rows are read once
// (the bound: 1 GB on 32 nodes x 2048 rows x 4096); a wavefront takes four rows at a time, so that the average is read
// once for four, and a workgroup goes through many before it adds its sum to the one result (with one row per wavefront,
// one float per lane and one fp64 atomic per row on that one address the same took 851 us; now 192, 5.6 TB/s).
constexpr int kLossRows = 4;
__global__ void __launch_bounds__(kThreads) rfast_loss_rows_kernel(RfastDev s, double* out) {
  const int i = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t p = s.p;
  const int S = s.prob.samples;
  const float* rows = (const float*)s.prob.data0 + (size_t)i * S * p;
  const float* ys = (const float*)s.prob.data1 + (size_t)i * S;
  double total = 0.0;
  for (int r0 = (blockIdx.x * (kThreads / 64) + wave) * kLossRows; r0 < S; r0 += gridDim.x * (kThreads / 64) * kLossRows) {
    double acc[kLossRows] = {0.0, 0.0, 0.0, 0.0};
    const float* a_row[kLossRows];
#pragma unroll
    for (int u = 0; u < kLossRows; ++u) a_row[u] = rows + (size_t)(r0 + u < S ? r0 + u : S - 1) * p;
    const int64_t full = p & ~(int64_t)3;
#pragma unroll 2
    for (int64_t k = 4 * lane; k < full; k += 256) {  // (no branch in here: every load of a step is in flight at once)
      float4 a[kLossRows];
#pragma unroll
      for (int u = 0; u < kLossRows; ++u) a[u] = V<5>::ld(a_row[u] + k);
      const float4 x = V<5>::ld(s.xbar + k);
#pragma unroll
      for (int u = 0; u < kLossRows; ++u)
        acc[u] += (double)a[u].x * x.x + (double)a[u].y * x.y + (double)a[u].z * x.z + (double)a[u].w * x.w;
    }
    if (full + lane < p) {
#pragma unroll
      for (int u = 0; u < kLossRows; ++u) acc[u] += (double)a_row[u][full + lane] * s.xbar[full + lane];
    }
#pragma unroll
    for (int u = 0; u < kLossRows; ++u) {
      const double dot = wave_sum(acc[u]);
      if (lane == u && r0 + u < S) {
        const double y = ys[r0 + u];
        if (s.prob.kind == RFAST_OBJ_LOGISTIC) total += (dot > 0 ? dot + log1p(exp(-dot)) : log1p(exp(dot))) - y * dot;
        else total += 0.5 * (dot - y) * (dot - y);
      }
    }
  }
  __shared__ double part[kThreads / 64];
  total = wave_sum(total);
  if (lane == 0) part[wave] = total;
  __syncthreads();
  if (threadIdx.x == 0) {
    double w = 0.0;
    for (int v = 0; v < kThreads / 64; ++v) w += part[v];
    if (w != 0.0) atomicAdd(&out[5], w / S);
  }
}

// The six results in the order of rfast_diag, from the accumulators (what rfast_diagnostics does on the host).
__global__ void rfast_diag_finish(const double* acc, double l2_half_n, int has_xstar, double* out) {
  if (threadIdx.x == 0) {
    out[0] = acc[0];
    out[1] = acc[1];
    out[2] = acc[2];
    out[3] = acc[3];
    out[4] = has_xstar ? acc[4] : -1.0;
    out[5] = acc[5] + l2_half_n * acc[6];
  }
}

// Scratch of rfast_diagnostics_static, the entry point that allocates nothing: the fp64 accumulators of the
// reductions, then the node average xbar that the loss kernels of the non-separable objectives read.  One copy per
// GPU, held until the process ends; every call on a GPU shares it.
constexpr size_t kStaticAccBytes = 256;
constexpr int64_t kStaticMaxCoords = 1 << 20;
__device__ __align__(256) unsigned char scratch[kStaticAccBytes + kStaticMaxCoords * sizeof(float)];
constexpr int kMaxDevices = 64;
void* g_scratch[kMaxDevices] = {};  // device address of `scratch` on each GPU (the array's name is no device address in host code)

}  // namespace

// Looks up the address of the static scratch array on the current device, once per device.
hipError_t rfast_static_scratch_init() {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  if (g_scratch[dev]) return hipSuccess;
  void* ptr = nullptr;
  e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!ptr) return hipErrorInvalidSymbol;
  g_scratch[dev] = ptr;
  return hipSuccess;
}

int64_t rfast_static_max_coords() { return kStaticMaxCoords; }

// rfast_launch_diag with the accumulators and xbar in the static scratch of the current device, and the six
// results written to d_out (device) by a last small kernel.  The caller has checked the size.
hipError_t rfast_launch_diag_static(rfast_ctx* c, const float* d_xstar, double* d_out, double l2_half_n) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices || !g_scratch[dev]) return hipErrorNotInitialized;
  unsigned char* base = static_cast<unsigned char*>(g_scratch[dev]);
  double* acc = reinterpret_cast<double*>(base);
  float* keep = c->d.xbar;
  c->d.xbar = c->d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC ? nullptr : reinterpret_cast<float*>(base + kStaticAccBytes);
  e = rfast_launch_diag(c, d_xstar, acc);  // clears the accumulators with a kernel first
  c->d.xbar = keep;
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(rfast_diag_finish, dim3(1), dim3(64), 0, c->stream, acc, l2_half_n, d_xstar ? 1 : 0, d_out);
  return hipGetLastError();
}

hipError_t rfast_launch_diag(rfast_ctx* c, const float* d_xstar, double* d_out) {
  hipLaunchKernelGGL(rfast_diag_zero, dim3(1), dim3(64), 0, c->stream, d_out);
  const bool vec4 = (c->d.p % 4) == 0 && ((uintptr_t)d_xstar % 16) == 0;
  int64_t blocks = group_tiles(c->d.p);
  if (blocks > 2048) blocks = 2048;  // grid-stride beyond that: 8 workgroups per CU
  const bool streaming = (double)c->d.n * (double)c->d.p * 4.0 >= 32.0e6;  // far beyond the caches: non-temporal loads
  // The other form's time is its serial chain, which grows with n and hardly with p; the split form's is its p / 64
  // workgroups.  us, other form -> split: n 4: p 8192 11.0 -> 9.7, 16384 10.9 -> 12.8; n 8: 16384 16.2 -> 13.3, 24576
  // 16.4 -> 20.3; n 16: 32768 27.0 -> 23.8, 49152 27.2 -> 35.0; n 48: 65536 96 -> 67; n 128: 65536 364 -> 125; and with
  // n 48 it is the slower one again at 131072 (100 -> 131).
  if (c->d.p <= 65536 && c->d.p <= (int64_t)2048 * c->d.n)
    hipLaunchKernelGGL(rfast_diag_split_kernel, dim3((unsigned)((c->d.p + 63) / 64)), dim3(64 * kSplitWaves), 0, c->stream, c->d,
                       d_xstar, d_out);
  else if (vec4 && streaming)
    hipLaunchKernelGGL(rfast_diag_kernel<-4>, dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, c->d, d_xstar, d_out);
  else if (vec4)
    hipLaunchKernelGGL(rfast_diag_kernel<4>, dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, c->d, d_xstar, d_out);
  else if (streaming)
    hipLaunchKernelGGL(rfast_diag_kernel<-5>, dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, c->d, d_xstar, d_out);
  else
    hipLaunchKernelGGL(rfast_diag_kernel<5>, dim3((unsigned)blocks), dim3(kThreads), 0, c->stream, c->d, d_xstar, d_out);
  const int kind = c->d.prob.kind;
  if (kind == RFAST_OBJ_LEAST_SQUARES || kind == RFAST_OBJ_LOGISTIC) {
    const int per = kThreads / 64 * kLossRows, most = (c->d.prob.samples + per - 1) / per;
    const int each = (2048 + c->d.n - 1) / c->d.n;  // eight workgroups per compute unit over all nodes
    hipLaunchKernelGGL(rfast_loss_rows_kernel, dim3(most < each ? most : each, c->d.n), dim3(kThreads), 0, c->stream, c->d, d_out);
  }
  if (kind == RFAST_OBJ_SOFTMAX_BF16) {
    const hipError_t e = rfast_softmax_loss(c, d_out + 5);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}
