// C-ABI entry points of librfast: argument checks, workspace layout, launch order.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

#include "rfast_internal.h"
#include "rfast_relay.h"

size_t rfast_gemv_scratch_floats(int32_t n, const rfast_problem* prob);
size_t rfast_softmax_scratch_bytes(int32_t n, const rfast_problem* prob);
bool rfast_softmax_shape_ok(const rfast_problem* prob);

namespace {

std::string g_create_error;

constexpr size_t kAlign = 256;
inline size_t up(size_t b) { return (b + kAlign - 1) / kAlign * kAlign; }

// Sizes of every carve-out, in the order they are laid out.
struct Layout {
  size_t total = 0;
  size_t take(size_t bytes) {
    const size_t off = total;
    total += up(bytes);
    return off;
  }
};

struct Offsets {
  size_t x, z, g, v_ring, sigma_ring, rho_tilde;
  size_t r_ptr, r_src, r_dst, r_w, r_self, c_ptr, c_src, c_dst, c_w, c_self, co_ptr, co_eid, co_w, ro_ptr, ro_eid;
  size_t t, t_hist, tau_r, tau_c, deliv_r, deliv_c, round_no, err;
  size_t n_active, active_plan, plan_t, slot_r, slot_c, plan_c, node_spill, plan_set_bytes, blk_plan, blk_spill, blk_far, blk_head, t_next, hist_next, ticket;
  size_t gen_active, gen_delay_r, gen_delay_c, gen_drop_r, gen_drop_c, gen_batch, gen_cdf;
  int32_t gen_depth;
  size_t xbar, resid, gscratch, diag, team_packets, team_sync, team_gate, team_flags;  // (flags right behind the gate)
  size_t total;
};

bool sizes_ok(int32_t n, int64_t p, int32_t nnzR, int32_t nnzC, int32_t D, const rfast_problem* prob) {
  if (n < 1 || n > 65535 || p < 1 || nnzR < n || nnzC < n || D < 0 || D + 2 > 64 || prob == nullptr) return false;  // n rides in gridDim.y
  if (prob->kind < 0 || prob->kind > RFAST_OBJ_SOFTMAX_BF16) return false;
  if (prob->kind != RFAST_OBJ_DIAG_QUADRATIC && (prob->samples < 1 || prob->batch < 0 || prob->batch > prob->samples))
    return false;
  if ((prob->kind == RFAST_OBJ_LEAST_SQUARES || prob->kind == RFAST_OBJ_LOGISTIC) &&
      (prob->batch > 0 ? prob->batch : prob->samples) > 4096)
    return false;  // the sampled residuals of one node are staged in LDS
  if (prob->kind == RFAST_OBJ_SOFTMAX_BF16 &&
      (prob->d < 1 || prob->K < 1 || (int64_t)prob->d * prob->K != p || !rfast_softmax_shape_ok(prob)))
    return false;  // MFMA tiling: d % 64 == 0, K in {32, 64, 96, 128}, rows per gradient % 64 == 0
  return true;
}

Offsets layout(int32_t n, int64_t p, int32_t nnzR, int32_t nnzC, int32_t D, const rfast_problem* prob) {
  const size_t eR = (size_t)(nnzR - n), eC = (size_t)(nnzC - n), M = (size_t)D + 2, H = (size_t)D + 1;
  const size_t vec = (size_t)p * sizeof(float);
  Layout L;
  Offsets o;
  o.x = L.take(n * vec);
  o.z = L.take(n * vec);
  o.g = L.take(2 * n * vec);
  o.v_ring = L.take(n * M * vec);
  o.sigma_ring = L.take(n * M * vec);
  o.rho_tilde = L.take(eC * vec);
  o.r_ptr = L.take((n + 1) * 4);
  o.r_src = L.take(eR * 4);
  o.r_dst = L.take(eR * 4);
  o.r_w = L.take(eR * 4);
  o.r_self = L.take(n * 4);
  o.c_ptr = L.take((n + 1) * 4);
  o.c_src = L.take(eC * 4);
  o.c_dst = L.take(eC * 4);
  o.c_w = L.take(eC * 4);
  o.c_self = L.take(n * 4);
  o.co_ptr = L.take((n + 1) * 4);
  o.co_eid = L.take(eC * 4);
  o.co_w = L.take(eC * 4);
  o.ro_ptr = L.take((n + 1) * 4);
  o.ro_eid = L.take(eR * 4);
  o.t = L.take(n * 4);
  o.t_hist = L.take(n * H * 4);
  o.tau_r = L.take(eR * 4);
  o.tau_c = L.take(eC * 4);
  o.deliv_r = L.take(eR * 8);
  o.deliv_c = L.take(eC * 8);
  o.round_no = L.take(4);
  o.err = L.take(24);
  o.n_active = L.take(8);
  o.active_plan = L.take(((size_t)n + 8) * 8);
  o.plan_t = L.take(n * 4);
  o.slot_r = L.take(eR * 4);
  o.slot_c = L.take(eC * 4);
  o.plan_c = L.take(eC * 4);
  o.node_spill = L.take(n * 4);
  // the seven arrays above are the plan of one round; kResolveAhead - 1 more such sets follow, so that the
  // resolver can run that many rounds ahead of the kernels that read the plans
  o.plan_set_bytes = L.total - o.n_active;
  (void)L.take((size_t)(kResolveAhead - 1) * o.plan_set_bytes);
  o.blk_plan = L.take((size_t)kBlockRounds * ((size_t)n + eR + eC + 1) * 4);
  o.blk_spill = L.take((size_t)kBlockRounds * n * 4);
  o.blk_far = L.take(prob->kind == RFAST_OBJ_DIAG_QUADRATIC && n <= 64 ? (size_t)n * kFarWords * 4 : 0);
  o.blk_head = L.take((kHeadWords * (size_t)n + eC) * 4);
  o.t_next = L.take(n * 4);
  o.hist_next = L.take(n * H * 4);
  o.ticket = L.take(4);
  // the generator draws the schedule of up to gen_depth rounds per launch (as many as fit 64 MB, at most kBlockRounds)
  const size_t gen_rows = (size_t)n * (size_t)(prob->kind == RFAST_OBJ_DIAG_QUADRATIC ? 0 : prob->batch);
  const size_t gen_round = (size_t)n + 5 * (eR + eC) + 4 * gen_rows;
  const size_t G = std::max<size_t>(1, std::min<size_t>(kBlockRounds, ((size_t)64 << 20) / gen_round));
  o.gen_depth = (int32_t)G;
  o.gen_active = L.take(G * n);
  o.gen_delay_r = L.take(G * eR * 4);
  o.gen_delay_c = L.take(G * eC * 4);
  o.gen_drop_r = L.take(G * eR);
  o.gen_drop_c = L.take(G * eC);
  o.gen_batch = L.take(G * gen_rows * 4);
  o.gen_cdf = L.take(n * 4);
  o.xbar = L.take(vec);
  o.resid = L.take(rfast_gemv_scratch_floats(n, prob) * 4);
  o.gscratch = L.take(rfast_softmax_scratch_bytes(n, prob));
  o.diag = L.take(64 * sizeof(double));
  // the team kernels' packets and progress words: which team a problem gets depends on the graph and the device, so
  // room for the largest one (at most kTeamMost workgroups)
  RfastTeam most;
  if (prob->kind == RFAST_OBJ_SOFTMAX_BF16) {
    RfastDev shape{};
    shape.n = n;
    shape.p = p;
    shape.M = D + 2;
    shape.prob = *prob;
    most = rfast_team_softmax_shape(shape, 0, 0, kTeamMost);
    o.team_packets = L.take(rfast_team_softmax_packet_bytes(most, n, prob));
    o.team_gate = L.take(2 * kGateBytes + rfast_team_softmax_flag_bytes(most, n, prob));
  } else {
    if (prob->kind != RFAST_OBJ_DIAG_QUADRATIC && n <= kTeamMost) most.W = std::min(32, kTeamMost / n);
    o.team_packets = L.take(rfast_team_packet_bytes(most, n, prob));
    o.team_gate = L.take(2 * kGateBytes + rfast_team_flag_bytes(most, n));
  }
  o.team_flags = o.team_gate + 2 * kGateBytes;
  o.team_sync = L.take(rfast_team_sync_bytes(n, p, prob));
  o.total = L.total;
  return o;
}

struct HostGraph {
  std::vector<int32_t> ptr, src, dst, out_ptr, out_eid;
  std::vector<float> w, self, out_w;
};

// Splits a CSR (row = receiver, diagonal included) into off-diagonal in-edge and
// out-edge lists and checks Assumption 1: positive diagonal, non-negative
// weights, rows (row_stochastic) or columns summing to one.
int split_graph(const char* name, int32_t n, const int32_t* rowptr, const int32_t* col, const float* w,
                bool row_stochastic, HostGraph* g, std::string* err) {
  if (rowptr[0] != 0) { *err = std::string(name) + ": rowptr[0] != 0"; return RFAST_EGRAPH; }
  g->ptr.assign(n + 1, 0);
  g->self.assign(n, 0.f);
  std::vector<double> colsum(n, 0.0);
  for (int i = 0; i < n; ++i) {
    if (rowptr[i + 1] < rowptr[i]) { *err = std::string(name) + ": rowptr not monotone"; return RFAST_EGRAPH; }
    double rowsum = 0.0;
    int prev = -1;
    bool diag = false;
    for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) {
      const int j = col[k];
      if (j < 0 || j >= n || j <= prev) {
        *err = std::string(name) + ": column indices must be in range, ascending and unique (row " + std::to_string(i) + ")";
        return RFAST_EGRAPH;
      }
      prev = j;
      if (!(w[k] > 0.f) || !std::isfinite(w[k])) {
        *err = std::string(name) + ": stored weights must be positive (row " + std::to_string(i) + ")";
        return RFAST_ESTOCH;
      }
      rowsum += w[k];
      colsum[j] += w[k];
      if (j == i) {
        diag = true;
        g->self[i] = w[k];
      } else {
        g->src.push_back(j);
        g->dst.push_back(i);
        g->w.push_back(w[k]);
      }
    }
    if (!diag) { *err = std::string(name) + ": missing self-loop at node " + std::to_string(i); return RFAST_ESTOCH; }
    if (row_stochastic && fabs(rowsum - 1.0) > 1e-6) {
      *err = std::string(name) + ": row " + std::to_string(i) + " does not sum to 1";
      return RFAST_ESTOCH;
    }
    g->ptr[i + 1] = (int32_t)g->src.size();
  }
  if (!row_stochastic)
    for (int j = 0; j < n; ++j)
      if (fabs(colsum[j] - 1.0) > 1e-6) {
        *err = std::string(name) + ": column " + std::to_string(j) + " does not sum to 1";
        return RFAST_ESTOCH;
      }
  // out-edge lists (sender-major)
  const size_t E = g->src.size();
  g->out_ptr.assign(n + 1, 0);
  for (size_t e = 0; e < E; ++e) g->out_ptr[g->src[e] + 1]++;
  for (int j = 0; j < n; ++j) g->out_ptr[j + 1] += g->out_ptr[j];
  g->out_eid.assign(E, 0);
  g->out_w.assign(E, 0.f);
  std::vector<int32_t> fill(g->out_ptr.begin(), g->out_ptr.end() - 1);
  for (size_t e = 0; e < E; ++e) {
    const int pos = fill[g->src[e]]++;
    g->out_eid[pos] = (int32_t)e;
    g->out_w[pos] = g->w[e];
  }
  return RFAST_OK;
}

// Nodes from which every node can be reached along `forward` edges sender->receiver
// (forward = true) or receiver->sender (forward = false).
std::vector<char> roots_of(int32_t n, const HostGraph& g, bool forward) {
  std::vector<std::vector<int>> adj(n);
  for (int i = 0; i < n; ++i)
    for (int e = g.ptr[i]; e < g.ptr[i + 1]; ++e) {
      if (forward) adj[g.src[e]].push_back(i);
      else adj[i].push_back(g.src[e]);
    }
  std::vector<char> is_root(n, 0);
  std::vector<int> stack;
  std::vector<char> seen;
  for (int r = 0; r < n; ++r) {
    seen.assign(n, 0);
    stack.assign(1, r);
    seen[r] = 1;
    int cnt = 1;
    while (!stack.empty()) {
      const int u = stack.back();
      stack.pop_back();
      for (int v : adj[u])
        if (!seen[v]) { seen[v] = 1; ++cnt; stack.push_back(v); }
    }
    is_root[r] = cnt == n;
  }
  return is_root;
}

template <class T>
hipError_t upload(rfast_ctx* c, char* base, size_t off, const std::vector<T>& v) {
  if (v.empty()) return hipSuccess;
  return hipMemcpyAsync(base + off, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, c->stream);
}

int fail(rfast_ctx* c, int code, const std::string& msg) {
  if (c) c->err = msg; else g_create_error = msg;
  return code;
}
int hipfail(rfast_ctx* c, hipError_t e, const char* what) {
  return fail(c, RFAST_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

size_t field_bytes(const rfast_ctx* c, int32_t field) {
  const RfastDev& d = c->d;
  const size_t vec = (size_t)d.p * 4;
  switch (field) {
    case RFAST_X: case RFAST_Z: case RFAST_G: return d.n * vec;
    case RFAST_V_RING: return (size_t)d.n * d.M * vec;
    case RFAST_RHO_RING: return (size_t)d.eC * d.M * vec;
    case RFAST_SIGMA_RING: return (size_t)d.n * d.M * vec;
    case RFAST_RHO_TILDE: return (size_t)d.eC * vec;
    case RFAST_T_NODE: return (size_t)d.n * 4;
    case RFAST_TAU_R: case RFAST_SLOT_R: return (size_t)d.eR * 4;
    case RFAST_TAU_C: case RFAST_SLOT_C: return (size_t)d.eC * 4;
    case RFAST_ROUND: return 4;
    case RFAST_DELIV_R: return (size_t)d.eR * 8;
    case RFAST_DELIV_C: return (size_t)d.eC * 8;
    case RFAST_T_HIST: return (size_t)d.n * d.H * 4;
    case RFAST_SCHED_ACTIVE: return (size_t)d.n;
    case RFAST_SCHED_DELAY_R: return (size_t)d.eR * 4;
    case RFAST_SCHED_DELAY_C: return (size_t)d.eC * 4;
    case RFAST_SCHED_DROP_R: return (size_t)d.eR;
    case RFAST_SCHED_DROP_C: return (size_t)d.eC;
    case RFAST_SCHED_BATCH: return (size_t)d.n * (d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC ? 0 : d.prob.batch) * 4;
    case RFAST_MOMENTUM: return d.mom ? d.n * vec : (size_t)-1;
    default: return (size_t)-1;
  }
}

// Ring slots whose version no receiver can pick up any more: stamps never go back, so a version older
// than every stamp held on its sender's out-edges (all versions, if the sender has none) is dead.  The
// kernels are free not to keep such slots up to date; reads of the ring fields return them as zeros.
// `ring` is a host copy of `rings` rings of [M][p] floats, ring q belonging to sender sender_of[q].
hipError_t zero_dead_slots(const rfast_ctx* c, bool sums, float* ring, int rings, const int32_t* sender_of) {
  const RfastDev& d = c->d;
  const int E = sums ? d.eC : d.eR;
  std::vector<int32_t> t(d.n), src(E), tau(E), lo(d.n, 0x7fffffff);
  hipError_t e = hipMemcpy(t.data(), d.t, (size_t)d.n * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess && E) e = hipMemcpy(src.data(), sums ? d.c_src : d.r_src, (size_t)E * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess && E) e = hipMemcpy(tau.data(), sums ? d.tau_c : d.tau_r, (size_t)E * 4, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return e;
  for (int q = 0; q < E; ++q) lo[src[q]] = std::min(lo[src[q]], tau[q]);
  for (int q = 0; q < rings; ++q) {
    const int j = sender_of ? sender_of[q] : q;
    for (int m = 0; m < d.M; ++m) {
      const int back = ((t[j] - m) % d.M + d.M) % d.M, ver = t[j] - back;  // version held by slot m
      if (ver < lo[j]) memset(ring + ((size_t)q * d.M + m) * d.p, 0, (size_t)d.p * 4);
    }
  }
  return hipSuccess;
}

void time_begin(rfast_ctx* c, int which) {
  if (!c->profiling || c->ev_used[which] >= c->ev[which][0].size()) return;
  (void)hipEventRecord(c->ev[which][0][c->ev_used[which]], c->stream);
}
void time_end(rfast_ctx* c, int which) {
  if (!c->profiling || c->ev_used[which] >= c->ev[which][0].size()) return;
  (void)hipEventRecord(c->ev[which][1][c->ev_used[which]], c->stream);
  c->ev_used[which]++;
}

// the synchronous mode double-buffers z; bring it back into its own array before anything else looks at it
int fold_sync(rfast_ctx* c) {
  if (c->sync_parity == 0) return RFAST_OK;
  const hipError_t e = rfast_launch_sync(c, 3, 0.f, 1);
  if (e != hipSuccess) return hipfail(c, e, "fold launch");
  c->sync_parity = 0;
  return RFAST_OK;
}

constexpr int32_t kGraphRounds = 16;

// Which team of workgroups a node gets for the several-rounds-per-launch form of the objectives that are not separable,
// and the chunks in which every kernel sums a row's dot product.  A problem that fits the LDS of one compute unit keeps
// its rows in one chunk (the one-workgroup kernel sums them so).
void choose_team(rfast_ctx* c, int max_out_r) {
  RfastDev& d = c->d;
  int units = 0;
  d.row_chunk = (int32_t)std::min<int64_t>(d.p, 0x7fffffff);
  if (hipGetDevice(&c->device) != hipSuccess ||
      hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess)
    return;
  units = std::min(units, kTeamMost);
  // a stream may have been given a part of the compute units (one bit each)
  uint32_t mask[(kTeamMost + 31) / 32 * 2] = {};
  if (hipExtStreamGetCUMask(c->stream, sizeof(mask) / sizeof(mask[0]), mask) == hipSuccess) {
    int given = 0;
    for (uint32_t m : mask) given += __builtin_popcount(m);
    if (given > 0) units = std::min(units, given);
  } else {
    (void)hipGetLastError();
  }
  if (rfast_tiny_eligible(c)) units = std::min(units, d.n);  // one workgroup per node at most
  if (d.prob.kind == RFAST_OBJ_SOFTMAX_BF16) {
    c->team = rfast_team_softmax_shape(d, c->max_degree, max_out_r, units);
    return;
  }
  c->team = rfast_team_shape(d, c->max_degree, max_out_r, units);
  if (c->team.W > 1) d.row_chunk = c->team.C;
}

hipError_t launch_team(rfast_ctx* c, bool sync, int rounds, float gamma, const int32_t* d_batch_idx, const int32_t* d_delay_R,
                       const int32_t* d_delay_C) {
  return c->d.prob.kind == RFAST_OBJ_SOFTMAX_BF16
             ? rfast_launch_team_softmax(c, rounds, gamma, d_batch_idx, d_delay_R, d_delay_C)
             : rfast_launch_team(c, sync, rounds, gamma, d_batch_idx, d_delay_R, d_delay_C);
}

// The workgroups of a team launch wait for each other to start, so two such launches that each hold a part of the chip
// would both wait until they give up (team_complete).  Launches on one stream follow each other; a launch on another stream
// than the last one first waits for the event recorded behind that one.  (Behind the launch and not when the next one
// comes: the other stream may by then be gone.)  hipStreamPerThread is one handle for a stream of every thread's own.
// The order is for speed, the result does not depend on it: where the runtime refuses a wait or a record, as it does
// while the other stream is under capture, the launch goes out without.
struct TeamOrder {
  bool used = false;
  hipStream_t stream = nullptr;
  hipEvent_t event = nullptr;
};
std::mutex g_team_mutex;
TeamOrder g_team_order[64];

bool same_stream(hipStream_t a, hipStream_t b) { return a == b && a != hipStreamPerThread; }

template <class Launch> hipError_t in_team_order(rfast_ctx* c, Launch launch) {
  if (c->device < 0 || c->device >= 64) return hipErrorInvalidDevice;
  const std::lock_guard<std::mutex> lock(g_team_mutex);
  TeamOrder& o = g_team_order[c->device];
  if (!o.event && hipEventCreateWithFlags(&o.event, hipEventDisableTiming) != hipSuccess) o.event = nullptr;
  if (o.event && o.used && !same_stream(o.stream, c->stream)) (void)hipStreamWaitEvent(c->stream, o.event, 0);
  (void)hipGetLastError();
  const hipError_t e = launch();
  if (e != hipSuccess) return e;
  o.used = o.event && hipEventRecord(o.event, c->stream) == hipSuccess;
  o.stream = c->stream;
  (void)hipGetLastError();
  return hipSuccess;
}

// Pinned words through which the device speaks to the host, a cache line per context: a page that all contexts of the
// process share and that stays (like the events above; allocating pinned memory takes some 100 us, a fifth of what making
// a small context does), and an allocation of its own for each context beyond the 64 that it holds.
std::mutex g_told_mutex;
char* g_told = nullptr;
uint64_t g_told_used = 0;

hipError_t take_told(rfast_ctx* c) {
  const std::lock_guard<std::mutex> lock(g_told_mutex);
  hipError_t e = hipSuccess;
  if (!g_told) e = hipHostMalloc((void**)&g_told, 64 * 64, hipHostMallocPortable);
  if (e != hipSuccess) {
    g_told = nullptr;
  } else if (~g_told_used != 0) {
    const int slot = __builtin_ctzll(~g_told_used);
    g_told_used |= 1ull << slot;
    c->team_told = (unsigned*)(g_told + 64 * slot);
  } else {
    e = hipHostMalloc((void**)&c->team_told, 64, hipHostMallocPortable);
    if (e != hipSuccess) c->team_told = nullptr;
  }
  if (c->team_told) c->team_told[0] = c->team_told[1] = 0;
  return e;
}

// (nothing on the device writes to it any more)
void drop_told(rfast_ctx* c) {
  if (!c->team_told) return;
  const std::lock_guard<std::mutex> lock(g_told_mutex);
  const ptrdiff_t at = g_told ? (char*)c->team_told - g_told : -1;
  if (at >= 0 && at < 64 * 64) g_told_used &= ~(1ull << (at / 64));
  else (void)hipHostFree(c->team_told);
  c->team_told = nullptr;
}

// the context's stream has been waited for and is about to be given up
void leave_team_order(rfast_ctx* c) {
  if (c->device < 0 || c->device >= 64) return;
  const std::lock_guard<std::mutex> lock(g_team_mutex);
  TeamOrder& o = g_team_order[c->device];
  if (o.used && same_stream(o.stream, c->stream)) o.used = false;
}

// Copies to pageable host memory.  The runtime's own copy of such memory reaches 4-9 GB/s and 18 us at the least; a
// copy into pinned memory takes 54 GB/s and 6 us.  So what is read goes through a pinned buffer that all contexts
// share (lazily allocated, given back with the last context; one of its own for small reads, which need not pay for the
// 16 MB of the other), and, where it is large, several threads move it on:
// most of their time goes into the page faults of a destination that has never been written.  Measured, a field of
// 9 KB 30 -> 17 us, 36 MB 3.6 -> 1.4 ms, 128 MB 12.4 -> 5.0 ms with pieces of 1 MB, one to a thread; 36 MB 1.05 ms, 128 MB 4.3 ms with pieces of up to 4
// MB that the threads share and the page faults taken before the first arrives (1.78 ms without: several threads then meet in a large page).
constexpr size_t kStageSlot = (size_t)1 << 20;
constexpr size_t kStageSmall = (size_t)64 << 10;
constexpr size_t kStageMost = (size_t)4 << 20;
constexpr int kStageThreads = 8;
std::mutex g_stage_mutex;   // whoever holds it owns the buffers; others copy without them
char* g_stage = nullptr;
char* g_stage_small = nullptr;
std::atomic<int> g_contexts{0};

hipError_t stage_ready(char** stage, size_t bytes) {
  if (*stage) return hipSuccess;
  void* p = nullptr;
  const hipError_t e = hipHostMalloc(&p, bytes, hipHostMallocPortable);
  if (e == hipSuccess) *stage = (char*)p;
  return e;
}

// Copies to host memory behind everything on the context's stream and waits for it.
hipError_t to_host(rfast_ctx* c, void* dst, const void* src, size_t bytes) {
  std::unique_lock<std::mutex> own(g_stage_mutex, std::try_to_lock);
  const bool small = bytes <= kStageSmall;
  if (!own.owns_lock() || (small ? stage_ready(&g_stage_small, kStageSmall) : stage_ready(&g_stage, kRelaySlots * kStageSlot)) != hipSuccess) {
    (void)hipGetLastError();
    const hipError_t e = hipStreamSynchronize(c->stream);
    return e == hipSuccess ? hipMemcpy(dst, src, bytes, hipMemcpyDeviceToHost) : e;
  }
  if (bytes <= kStageSlot) {
    char* stage = small ? g_stage_small : g_stage;
    hipError_t e = hipMemcpyAsync(stage, src, bytes, hipMemcpyDeviceToHost, c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e == hipSuccess) memcpy(dst, stage, bytes);
    return e;
  }
  const int cores = (int)std::thread::hardware_concurrency();
  Relay r;
  r.dst = (char*)dst;
  r.stage = g_stage;
  r.bytes = bytes;
  // a copy into pinned memory costs some 8 us of its own: pieces of 1, 2 and 4 MB reach 37, 45 and 50 GB/s
  r.piece = bytes >= 32 * kStageSlot ? kStageMost : bytes >= 16 * kStageSlot ? kStageMost / 2 : kStageSlot;
  r.unit = std::min(r.piece, 2 * kStageSlot);
  r.slots = (int)(kRelaySlots * kStageSlot / r.piece);
  // a thread is worth starting (15 us) for 2 MB and more
  const int threads = (int)std::max<size_t>(1, std::min({(size_t)kStageThreads, bytes / (2 * kStageSlot), (size_t)std::max(cores, 1)}));
  hipError_t e = hipSuccess;
  hipEvent_t ev[kRelaySlots] = {};
  for (int q = 0; q < r.slots && e == hipSuccess; ++q) e = hipEventCreateWithFlags(&ev[q], hipEventDisableTiming);
  try {
    if (e == hipSuccess)
      relay(&r, threads,
            [&](size_t k, int q) {
              e = hipMemcpyAsync(g_stage + (size_t)q * r.piece, (const char*)src + k * r.piece, r.size(k), hipMemcpyDeviceToHost, c->stream);
              if (e == hipSuccess) e = hipEventRecord(ev[q], c->stream);
              return e == hipSuccess;
            },
            [&](int q) { return (e = hipEventSynchronize(ev[q])) == hipSuccess; });
  } catch (...) {
    e = hipErrorOutOfMemory;
  }
  if (e != hipSuccess) (void)hipStreamSynchronize(c->stream);  // nothing is under way into the buffer afterwards
  for (hipEvent_t x : ev)
    if (x) (void)hipEventDestroy(x);
  return e;
}

void context_made() { g_contexts++; }
void context_gone() {
  if (--g_contexts > 0) return;
  const std::lock_guard<std::mutex> lock(g_stage_mutex);
  if (g_contexts != 0) return;
  for (char** stage : {&g_stage, &g_stage_small})
    if (*stage) {
      (void)hipHostFree(*stage);
      *stage = nullptr;
    }
}

// A captured launch would be replayed with the progress words of its capture, so captured rounds take the kernels per round; so do
// profiled ones, whose state and gradient kernels are to be timed apart, and rounds that would have to wait for a stream
// that is under capture just now (the runtime allows no such dependency, whatever the event was recorded behind).
bool team_usable(const rfast_ctx* c) {
  if (!c->use_blocks || c->team.W <= 0 || c->capturing || c->profiling) return false;
  if (((volatile unsigned*)c->team_told)[0] != 0) return false;  // the workgroups of a team of this context do not all find room
  if (c->stream != nullptr) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &st) == hipSuccess && st != hipStreamCaptureStatusNone) return false;
  }
  if (c->device < 0 || c->device >= 64) return false;
  const std::lock_guard<std::mutex> lock(g_team_mutex);
  const TeamOrder& o = g_team_order[c->device];
  if (o.used && o.stream != c->stream && o.stream != nullptr) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(o.stream, &st) == hipSuccess && st != hipStreamCaptureStatusNone) return false;
  }
  return true;
}

// The fewest rounds of a team launch that are faster than the kernels per round (bit for bit the same for least squares
// and logistic regression), from both timed side by side.
// Least squares, logistic: two rounds (1.03 to 1.6 times as fast over 16 sizes).  A single one only where rows are longer
// than the rows kernel takes in one step (p 4096, 32 nodes: 25.9 against 29.4 us; 16384, 8 nodes: 25.2 against 35.7; 16384,
// 16 nodes: 45.6 against 50.0; 8192, 4 nodes: 46.5 against 47.8): below, the kernels of a round are through before the
// workgroups of a team have fetched what they keep (p 784, 31 nodes: 20.1 against 18.8; 1001, 16 nodes: 27.0 against 21.7;
// 3000, 64 nodes: 35.9 against 34.4; 600, 36 nodes, 300 rows: 30.5 against 31.1, the only one of twelve the other way).
// Softmax regression: with R = B / W rows per workgroup a team's round is about 12.5 us + 3 ns R K + 0.85 ns B K (the
// softmax of its rows, E received by everybody), the four kernels 18 to 35 us.  R K 128 and 512: 16 to 20 against 19
// to 23 us a round, and about 20 us at its start, even from 5 rounds on; R K 1024, B K 8192: 24.5 against 24.6 with
// every node active, 21.4 against 23.1 with half of them, even from about 16; beyond (64 nodes, d 64, K 64, batch 128:
// 34 against 22; 8 nodes, d 1024, K 128, batch 256: 45 against 35) never.  With one agent per iteration only one node
// pays for that: 3 iterations at any size (two: 0.94 to 1.3 times as fast, six: 1.4 to 2.3).
int32_t team_least_rounds(const rfast_ctx* c) {
  const RfastDev& d = c->d;
  const int64_t B = d.prob.batch > 0 ? d.prob.batch : d.prob.samples;
  if (c->use_blocks == 2) return 1;
  if (d.prob.kind != RFAST_OBJ_SOFTMAX_BF16) return d.p >= 4096 ? 1 : 2;
  if (c->no_tiles) return 3;
  const int64_t RK = (B + c->team.W - 1) / c->team.W * d.prob.K;
  if (RK > 1024 || B * d.prob.K > 8192) return kBlockRounds + 1;
  return RK <= 512 ? 5 : 16;
}

// step size of round `round`: gamma * factor^(round div step_rounds)
float gamma_at(const rfast_ctx* c, float gamma, int64_t round) {
  if (c->gamma_step <= 0) return gamma;
  return gamma * powf(c->gamma_factor, (float)(round / c->gamma_step));
}
// ... of the round about to run
float gamma_now(const rfast_ctx* c, float gamma) { return gamma_at(c, gamma, c->host_round); }

void drop_graph(rfast_ctx* c) {
  if (c->graph_exec) (void)hipGraphExecDestroy(c->graph_exec);
  c->graph_exec = nullptr;
}

// automatic rebase of the running sums whenever the round counter reaches a multiple of
// `rebase_interval` (0 = never): a function of the round number, so a restored run repeats it
int after_round(rfast_ctx* c) {
  c->host_round++;
  if (c->rebase_interval > 0 && c->host_round % c->rebase_interval == 0) {
    const hipError_t e = rfast_launch_rebase(c);
    if (e != hipSuccess) return hipfail(c, e, "rebase launch");
  }
  return RFAST_OK;
}

}  // namespace

extern "C" int rfast_round(rfast_ctx* c, const uint8_t* d_active, const int32_t* d_delay_R, const int32_t* d_delay_C,
                           const uint8_t* d_drop_R, const uint8_t* d_drop_C, float gamma, const int32_t* d_batch_idx);

namespace {

// Captures kGraphRounds generated rounds on a private stream (capture is not allowed on
// the legacy default stream, which is what callers usually hand over) and instantiates them.
int build_graph(rfast_ctx* c, uint64_t seed, const float* d_p_active, int32_t max_delay, float p_drop, float gamma) {
  drop_graph(c);
  if (!c->capture_stream) {
    const hipError_t e = hipStreamCreateWithFlags(&c->capture_stream, hipStreamNonBlocking);
    if (e != hipSuccess) return hipfail(c, e, "hipStreamCreateWithFlags");
  }
  const RfastDev& d = c->d;
  hipStream_t user = c->stream;
  hipError_t e = hipStreamBeginCapture(c->capture_stream, hipStreamCaptureModeThreadLocal);
  if (e != hipSuccess) return hipfail(c, e, "hipStreamBeginCapture");
  c->stream = c->capture_stream;
  c->capturing = true;
  const int64_t round_before = c->host_round;  // capture enqueues nothing: the counter moves when the graph is launched
  int rc = RFAST_OK;
  for (int32_t r = 0; r < kGraphRounds && rc == RFAST_OK; ++r) {
    const hipError_t g = rfast_launch_generate(c, seed, d_p_active, max_delay, p_drop, false);
    if (g != hipSuccess) rc = hipfail(c, g, "schedule generator launch");
    else rc = rfast_round(c, d.gen_active, d.gen_delay_r, d.gen_delay_c, d.gen_drop_r, d.gen_drop_c, gamma, d.gen_batch);
  }
  c->stream = user;
  c->capturing = false;
  c->host_round = round_before;
  hipGraph_t graph = nullptr;
  e = hipStreamEndCapture(c->capture_stream, &graph);
  if (rc != RFAST_OK) {
    if (graph) (void)hipGraphDestroy(graph);
    return rc;
  }
  if (e != hipSuccess) return hipfail(c, e, "hipStreamEndCapture");
  e = hipGraphInstantiate(&c->graph_exec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) {
    c->graph_exec = nullptr;
    return hipfail(c, e, "hipGraphInstantiate");
  }
  c->graph_seed = seed;
  c->graph_p_active = d_p_active;
  c->graph_max_delay = max_delay;
  c->graph_p_drop = p_drop;
  c->graph_gamma = gamma_now(c, gamma);
  return RFAST_OK;
}

}  // namespace

extern "C" {

int rfast_common_roots(int32_t n, const int32_t* R_rowptr, const int32_t* R_col, const int32_t* C_rowptr,
                       const int32_t* C_col, uint8_t* host_is_root) {
  if (n < 1 || !R_rowptr || !R_col || !C_rowptr || !C_col) return fail(nullptr, RFAST_EINVAL, "NULL argument or n < 1");
  HostGraph g[2];
  const int32_t* ptrs[2] = {R_rowptr, C_rowptr};
  const int32_t* cols[2] = {R_col, C_col};
  for (int q = 0; q < 2; ++q) {
    if (ptrs[q][0] != 0) return fail(nullptr, RFAST_EGRAPH, "rowptr[0] != 0");
    g[q].ptr.assign(n + 1, 0);
    for (int i = 0; i < n; ++i) {
      if (ptrs[q][i + 1] < ptrs[q][i]) return fail(nullptr, RFAST_EGRAPH, "rowptr not monotone");
      for (int k = ptrs[q][i]; k < ptrs[q][i + 1]; ++k) {
        const int j = cols[q][k];
        if (j < 0 || j >= n) return fail(nullptr, RFAST_EGRAPH, "column index out of range");
        if (j != i) g[q].src.push_back(j);
      }
      g[q].ptr[i + 1] = (int32_t)g[q].src.size();
    }
  }
  const std::vector<char> rr = roots_of(n, g[0], true), rc = roots_of(n, g[1], false);
  int count = 0;
  for (int i = 0; i < n; ++i) {
    const bool both = rr[i] && rc[i];
    if (host_is_root) host_is_root[i] = both ? 1 : 0;
    count += both;
  }
  return count;
}

size_t rfast_workspace_bytes(int32_t n, int64_t p, int32_t nnzR, int32_t nnzC, int32_t D, const rfast_problem* prob) {
  if (!sizes_ok(n, p, nnzR, nnzC, D, prob)) return 0;
  return layout(n, p, nnzR, nnzC, D, prob).total;
}

int rfast_create(rfast_ctx** out, int32_t n, int64_t p, const int32_t* R_rowptr, const int32_t* R_col, const float* R_w,
                 const int32_t* C_rowptr, const int32_t* C_col, const float* C_w, int32_t D, int32_t burst,
                 const rfast_problem* prob, void* d_workspace, size_t workspace_bytes, void* hip_stream) {
  if (out == nullptr) return fail(nullptr, RFAST_EINVAL, "out is NULL");
  *out = nullptr;
  if (!R_rowptr || !R_col || !R_w || !C_rowptr || !C_col || !C_w || !prob || !d_workspace)
    return fail(nullptr, RFAST_EINVAL, "NULL argument");
  if (n < 1 || n > 65535 || p < 1) return fail(nullptr, RFAST_EINVAL, "need 1 <= n <= 65535 and p >= 1");
  if (D < 0 || D + 2 > 64) return fail(nullptr, RFAST_ERANGE, "D + 2 must be in [2, 64]");
  if (burst < 1 || burst - 1 > D) return fail(nullptr, RFAST_ERANGE, "burst must be in [1, D+1]");
  const int32_t nnzR = R_rowptr[n], nnzC = C_rowptr[n];
  if (!sizes_ok(n, p, nnzR, nnzC, D, prob)) return fail(nullptr, RFAST_EINVAL, "sizes or problem description out of range");
  if (!prob->data0 || !prob->data1) return fail(nullptr, RFAST_EINVAL, "problem data pointers are NULL");
  if (((uintptr_t)d_workspace % kAlign) != 0) return fail(nullptr, RFAST_EINVAL, "workspace must be 256-byte aligned");
  if ((p % 4) == 0 && ((((uintptr_t)prob->data0) | ((uintptr_t)prob->data1)) % 16) != 0)
    return fail(nullptr, RFAST_EINVAL, "problem data must be 16-byte aligned");

  HostGraph gr, gc;
  std::string msg;
  int rc = split_graph("R", n, R_rowptr, R_col, R_w, true, &gr, &msg);
  if (rc != RFAST_OK) return fail(nullptr, rc, msg);
  rc = split_graph("C", n, C_rowptr, C_col, C_w, false, &gc, &msg);
  if (rc != RFAST_OK) return fail(nullptr, rc, msg);
  {
    // Assumption 2: G(R) and G(C^T) each contain a spanning tree and share a root.
    // In G(R) information flows sender -> receiver; in G(C^T) the edges of C are reversed.
    const std::vector<char> rr = roots_of(n, gr, true), rc2 = roots_of(n, gc, false);
    bool common = false;
    for (int i = 0; i < n; ++i) common = common || (rr[i] && rc2[i]);
    if (!common) return fail(nullptr, RFAST_EGRAPH, "G(R) and G(C^T) share no spanning-tree root (Assumption 2)");
  }
  const Offsets o = layout(n, p, nnzR, nnzC, D, prob);
  if (workspace_bytes < o.total)
    return fail(nullptr, RFAST_ENOMEM, "workspace too small: need " + std::to_string(o.total) + " bytes");

  rfast_ctx* c = new (std::nothrow) rfast_ctx();
  if (!c) return fail(nullptr, RFAST_ENOMEM, "host allocation failed");
  c->stream = (hipStream_t)hip_stream;
  c->nnzR = nnzR;
  c->nnzC = nnzC;
  char* b = (char*)d_workspace;
  RfastDev& d = c->d;
  d.n = n; d.p = p; d.M = D + 2; d.H = D + 1; d.eR = nnzR - n; d.eC = nnzC - n;
  d.burst = burst; d.d_max = D - (burst - 1);
  d.x = (float*)(b + o.x); d.z = (float*)(b + o.z); d.g = (float*)(b + o.g);
  d.v_ring = (float*)(b + o.v_ring); d.sigma_ring = (float*)(b + o.sigma_ring); d.rho_tilde = (float*)(b + o.rho_tilde);
  d.r_ptr = (int32_t*)(b + o.r_ptr); d.r_src = (int32_t*)(b + o.r_src); d.r_dst = (int32_t*)(b + o.r_dst); d.r_w = (float*)(b + o.r_w);
  d.r_self = (float*)(b + o.r_self);
  d.c_ptr = (int32_t*)(b + o.c_ptr); d.c_src = (int32_t*)(b + o.c_src); d.c_dst = (int32_t*)(b + o.c_dst); d.c_w = (float*)(b + o.c_w); d.c_self = (float*)(b + o.c_self);
  d.co_ptr = (int32_t*)(b + o.co_ptr); d.co_eid = (int32_t*)(b + o.co_eid); d.co_w = (float*)(b + o.co_w);
  d.ro_ptr = (int32_t*)(b + o.ro_ptr); d.ro_eid = (int32_t*)(b + o.ro_eid);
  d.t = (int32_t*)(b + o.t); d.t_hist = (int32_t*)(b + o.t_hist);
  d.tau_r = (int32_t*)(b + o.tau_r); d.tau_c = (int32_t*)(b + o.tau_c);
  d.deliv_r = (unsigned long long*)(b + o.deliv_r); d.deliv_c = (unsigned long long*)(b + o.deliv_c);
  d.round_no = (int32_t*)(b + o.round_no); d.err = (int32_t*)(b + o.err);
  d.n_active = (int32_t*)(b + o.n_active); d.active_plan = (int2*)(b + o.active_plan);
  d.plan_t = (int32_t*)(b + o.plan_t); d.slot_r = (int32_t*)(b + o.slot_r); d.slot_c = (int32_t*)(b + o.slot_c);
  d.plan_c = (int32_t*)(b + o.plan_c); d.node_spill = (int32_t*)(b + o.node_spill);
  d.blk_plan = nullptr;
  d.blk_spill = (int32_t*)(b + o.blk_spill);
  d.t_next = (int32_t*)(b + o.t_next); d.hist_next = (int32_t*)(b + o.hist_next); d.ticket = (int32_t*)(b + o.ticket);
  d.blk_head = nullptr;
  d.blk_slots = 0;
  d.blk_far = (int32_t*)(b + o.blk_far);
  c->blk_plan_base = (int32_t*)(b + o.blk_plan);
  c->blk_head_base = (int32_t*)(b + o.blk_head);
  c->plan_set0 = b + o.n_active;
  c->plan_set_bytes = o.plan_set_bytes;
  c->plan_set = 0;
  d.gen_active = (uint8_t*)(b + o.gen_active); d.gen_delay_r = (int32_t*)(b + o.gen_delay_r);
  d.gen_delay_c = (int32_t*)(b + o.gen_delay_c); d.gen_drop_r = (uint8_t*)(b + o.gen_drop_r);
  d.gen_drop_c = (uint8_t*)(b + o.gen_drop_c); d.gen_batch = (int32_t*)(b + o.gen_batch);
  d.gen_cdf = (uint32_t*)(b + o.gen_cdf);
  c->gen_depth = o.gen_depth;
  d.xbar = (float*)(b + o.xbar);
  c->team_packets = (void*)(b + o.team_packets); c->team_flags = (unsigned*)(b + o.team_flags);
  c->team_gate = (unsigned*)(b + o.team_gate);
  c->team_sync = (void*)(b + o.team_sync);
  d.mom = nullptr; d.beta = 0.f; d.wd = 0.f;
  d.resid = (float*)(b + o.resid); d.gscratch = (void*)(b + o.gscratch);
  c->d_diag = (double*)(b + o.diag);
  d.prob = *prob;

  hipError_t e = rfast_static_scratch_init();  // for rfast_diagnostics_static, which may not look anything up later
  auto chk = [&](hipError_t r) { if (e == hipSuccess) e = r; };
  chk(upload(c, b, o.r_ptr, gr.ptr)); chk(upload(c, b, o.r_src, gr.src)); chk(upload(c, b, o.r_dst, gr.dst)); chk(upload(c, b, o.r_w, gr.w));
  chk(upload(c, b, o.r_self, gr.self));
  chk(upload(c, b, o.c_ptr, gc.ptr)); chk(upload(c, b, o.c_src, gc.src)); chk(upload(c, b, o.c_dst, gc.dst)); chk(upload(c, b, o.c_w, gc.w)); chk(upload(c, b, o.c_self, gc.self));
  chk(upload(c, b, o.co_ptr, gc.out_ptr)); chk(upload(c, b, o.co_eid, gc.out_eid)); chk(upload(c, b, o.co_w, gc.out_w));
  chk(upload(c, b, o.ro_ptr, gr.out_ptr)); chk(upload(c, b, o.ro_eid, gr.out_eid));
  for (int i = 0; i < n; ++i) c->max_in_degree = std::max({c->max_in_degree, gr.ptr[i + 1] - gr.ptr[i], gc.ptr[i + 1] - gc.ptr[i]});
  for (int i = 0; i < n; ++i)
    c->max_degree = std::max({c->max_degree, gr.ptr[i + 1] - gr.ptr[i], gc.ptr[i + 1] - gc.ptr[i], gc.out_ptr[i + 1] - gc.out_ptr[i]});
  int max_in_r = 0, max_in_c = 0, v_rows = 0, s_rows = 0;
  bool one_receiver = true;
  for (int i = 0; i < n; ++i) {
    max_in_r = std::max(max_in_r, gr.ptr[i + 1] - gr.ptr[i]);
    max_in_c = std::max(max_in_c, gc.ptr[i + 1] - gc.ptr[i]);
    v_rows += gr.out_ptr[i + 1] > gr.out_ptr[i] ? 1 : 0;
    s_rows += gc.out_ptr[i + 1] > gc.out_ptr[i] ? 1 : 0;
  }
  for (int32_t to : gc.dst) one_receiver = one_receiver && to == gc.dst[0];
  c->v_rows = c->s_rows = n;
  if (v_rows > 0 && s_rows > 0 && max_in_r <= 1) {
    // (stars of four and five nodes stay on edge slots while the chip holds every tile that way: p 20000, 100 rounds, 106 and 107 us against 110 and
    // 113; p 1 M 471 and 597 against 458 and 531; six and seven nodes need six slots: p 20000, 117 against 112.  The same bits.)
    const int64_t columns = 4 * (64 / std::min(n, 64)), tiles = (p + columns - 1) / columns;
    if (one_receiver && max_in_c > 2 && !(n <= 5 && tiles <= 256 * (int64_t)rfast_wave_held(c))) c->hub = gc.dst[0];
    // (rings of nodes without readers left out: only where all of them would leave fewer than eight wavefronts to a compute unit.  What
    // finding the rings costs a launch, half a microsecond, weighs more elsewhere: binary tree of 12, p 1664, delays of up to 4, calls of four
    // 0.93, of 40 0.98; of 64, delays of up to 16, p 1 M, 1.8 times as fast.)
    else if (n <= 64) c->tree = max_in_c <= 2 && c->max_degree <= 2 && v_rows + s_rows < 2 * n && n * (64 / n) * std::min(d.M - 1, d.d_max + 2) > 640;
    if (c->hub >= 0 || c->tree) {
      c->v_rows = v_rows;
      c->s_rows = s_rows;
    }
  }
  int max_out_r = 0;
  d.leaves = 0;
  for (int i = 0; i < n; ++i) {
    max_out_r = std::max(max_out_r, gr.out_ptr[i + 1] - gr.out_ptr[i]);
    if (gr.out_ptr[i + 1] == gr.out_ptr[i]) d.leaves = 1;
  }
  chk(hipMemsetAsync(d.ticket, 0, 4, c->stream));
  choose_team(c, max_out_r);
  if (c->team.W > 0) {
    const bool softmax = prob->kind == RFAST_OBJ_SOFTMAX_BF16;
    chk(hipMemsetAsync(c->team_packets, 0, softmax ? rfast_team_softmax_packet_bytes(c->team, n, prob) : rfast_team_packet_bytes(c->team, n, prob), c->stream));
    chk(hipMemsetAsync(c->team_gate, 0, 2 * kGateBytes + (softmax ? rfast_team_softmax_flag_bytes(c->team, n, prob) : rfast_team_flag_bytes(c->team, n)), c->stream));
    if (const size_t sync = rfast_team_sync_bytes(n, p, prob)) chk(hipMemsetAsync(c->team_sync, 0, sync, c->stream));
    chk(take_told(c));
  }
  chk(rfast_wave_prime(c));
  chk(hipStreamSynchronize(c->stream));  // the host vectors die with this scope
  if (e != hipSuccess) {
    const int r = hipfail(nullptr, e, "uploading graph");
    drop_told(c);
    delete c;
    return r;
  }
  context_made();
  *out = c;
  return RFAST_OK;
}

// RFAST_EHIP if a wait within a team launch has run out since the last rfast_init: the state is not that of any run.  The
// device leaves word of it in pinned memory, so that a call asks the device itself (and waits for it) only then.
static int state_usable(rfast_ctx* c) {
  volatile unsigned* told = c->team_told;
  if (!told || told[1] == 0 || c->capturing) return RFAST_OK;
  int32_t code = 0;
  const hipError_t e = to_host(c, &code, c->d.err, 4);
  if (e != hipSuccess) return hipfail(c, e, "reading device status");
  if (code == RFAST_EHIP) return rfast_check(c);
  told[1] = 0;  // from before an rfast_init
  return RFAST_OK;
}

int rfast_init(rfast_ctx* c, const float* d_x0, const int32_t* d_batch_idx0) {
  if (!c) return RFAST_EINVAL;
  RfastDev& d = c->d;
  if (d.prob.kind != RFAST_OBJ_DIAG_QUADRATIC && d.prob.batch > 0 && !d_batch_idx0)
    return fail(c, RFAST_EINVAL, "initial sample rows are required when batch > 0");
  const size_t vec = (size_t)d.p * 4;
  c->sync_parity = 0;
  c->host_round = 0;
  c->needs_init = false;
  if (c->team_told) ((volatile unsigned*)c->team_told)[0] = 0;  // a team may find room again
  hipError_t e = hipSuccess;
  auto chk = [&](hipError_t r) { if (e == hipSuccess) e = r; };
  if (d.mom) chk(hipMemsetAsync(d.mom, 0, d.n * vec, c->stream));
  if (d_x0) chk(hipMemcpyAsync(d.x, d_x0, d.n * vec, hipMemcpyDeviceToDevice, c->stream));
  else chk(hipMemsetAsync(d.x, 0, d.n * vec, c->stream));
  chk(hipMemsetAsync(d.g, 0, 2 * d.n * vec, c->stream));
  chk(hipMemsetAsync(d.v_ring, 0, (size_t)d.n * d.M * vec, c->stream));
  chk(hipMemsetAsync(d.sigma_ring, 0, (size_t)d.n * d.M * vec, c->stream));
  if (d.eC) {
    chk(hipMemsetAsync(d.rho_tilde, 0, (size_t)d.eC * vec, c->stream));
    chk(hipMemsetAsync(d.tau_c, 0, (size_t)d.eC * 4, c->stream));
    chk(hipMemsetAsync(d.slot_c, 0xff, (size_t)d.eC * 4, c->stream));
    chk(hipMemsetAsync(d.plan_c, 0, (size_t)d.eC * 4, c->stream));
    // only version 0 (slot 0) counts as delivered
    chk(hipMemsetAsync(d.deliv_c, 0, (size_t)d.eC * 8, c->stream));
  }
  if (d.eR) {
    chk(hipMemsetAsync(d.tau_r, 0, (size_t)d.eR * 4, c->stream));
    chk(hipMemsetAsync(d.slot_r, 0xff, (size_t)d.eR * 4, c->stream));
    chk(hipMemsetAsync(d.deliv_r, 0, (size_t)d.eR * 8, c->stream));
  }
  chk(hipMemsetAsync(d.t, 0, (size_t)d.n * 4, c->stream));
  chk(hipMemsetAsync(d.t_hist, 0, (size_t)d.n * d.H * 4, c->stream));
  chk(hipMemsetAsync(d.plan_t, 0, (size_t)d.n * 4, c->stream));
  chk(hipMemsetAsync(d.round_no, 0, 4, c->stream));
  chk(hipMemsetAsync(d.err, 0, 16, c->stream));
  chk(hipMemsetAsync(d.err + 4, 0xff, 8, c->stream));
  chk(hipMemsetAsync(d.ticket, 0, 4, c->stream));
  chk(hipMemsetAsync(d.n_active, 0, 8, c->stream));
  if (e != hipSuccess) return hipfail(c, e, "rfast_init clears");
  e = rfast_launch_init_grad(c, d_batch_idx0);
  if (e != hipSuccess) return hipfail(c, e, "initial gradient");
  return RFAST_OK;
}

// Points the per-round plan arrays of c->d at set q (the resolver writes the rounds it takes in one
// launch into consecutive sets; the kernels of a round read the set of that round).
static void use_plan_set(rfast_ctx* c, int32_t q) {
  RfastDev& d = c->d;
  const ptrdiff_t shift = (ptrdiff_t)(q - c->plan_set) * (ptrdiff_t)c->plan_set_bytes;
  auto move = [shift](auto*& ptr) { ptr = reinterpret_cast<std::remove_reference_t<decltype(ptr)>>(reinterpret_cast<char*>(ptr) + shift); };
  move(d.n_active); move(d.active_plan); move(d.plan_t); move(d.slot_r); move(d.slot_c); move(d.plan_c); move(d.node_spill);
  c->plan_set = q;
}

static int check_round_args(rfast_ctx* c, const uint8_t* d_active, const int32_t* d_delay_R, const int32_t* d_delay_C,
                            const uint8_t* d_drop_R, const uint8_t* d_drop_C, float gamma, const int32_t* d_batch_idx) {
  const RfastDev& d = c->d;
  if (!d_active || (d.eR && (!d_delay_R || !d_drop_R)) || (d.eC && (!d_delay_C || !d_drop_C)))
    return fail(c, RFAST_EINVAL, "NULL schedule pointer");
  const bool separable = d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC;
  if (!separable && d.prob.batch > 0 && !d_batch_idx) return fail(c, RFAST_EINVAL, "sample rows are required when batch > 0");
  if (!std::isfinite(gamma)) return fail(c, RFAST_EINVAL, "gamma is not finite");
  if (c->needs_init) return fail(c, RFAST_EINVAL, "rfast_init must follow rfast_set_optimizer");
  return state_usable(c);
}

static int float_round(rfast_ctx* c, float gamma, const int32_t* d_batch_idx, bool warm);
static int32_t block_length(const rfast_ctx* c, int32_t rounds, int64_t at_round = -1);
static int run_block(rfast_ctx* c, int32_t len, const uint8_t* d_active, const int32_t* d_delay_R, const int32_t* d_delay_C,
                     const uint8_t* d_drop_R, const uint8_t* d_drop_C, float gamma, const int32_t* d_batch_idx);

int rfast_round(rfast_ctx* c, const uint8_t* d_active, const int32_t* d_delay_R, const int32_t* d_delay_C,
                const uint8_t* d_drop_R, const uint8_t* d_drop_C, float gamma, const int32_t* d_batch_idx) {
  if (!c) return RFAST_EINVAL;
  const int rc = check_round_args(c, d_active, d_delay_R, d_delay_C, d_drop_R, d_drop_C, gamma, d_batch_idx);
  if (rc != RFAST_OK) return rc;
  if (c->d.prob.kind != RFAST_OBJ_DIAG_QUADRATIC && block_length(c, 1) > 0)
    return run_block(c, 1, d_active, d_delay_R, d_delay_C, d_drop_R, d_drop_C, gamma, d_batch_idx);
  if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
  time_begin(c, 2);
  const hipError_t e = rfast_launch_resolve(c, d_active, d_delay_R, d_delay_C, d_drop_R, d_drop_C);
  time_end(c, 2);
  if (e != hipSuccess) return hipfail(c, e, "resolver launch");
  return float_round(c, gamma, d_batch_idx, c->capturing);  // (a graph holds several rounds)
}

// The floating-point part of a round whose plan the resolver has written into the current plan set.  warm: a round of a call
// of many.
static int float_round(rfast_ctx* c, float gamma, const int32_t* d_batch_idx, bool warm) {
  const bool separable = c->d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC;
  gamma = gamma_now(c, gamma);
  hipError_t e;
  if (separable) {
    time_begin(c, 0);
    e = rfast_launch_state(c, RFAST_MODE_FUSED, gamma, warm);
    time_end(c, 0);
    if (e != hipSuccess) return hipfail(c, e, "fused round launch");
    return after_round(c);
  }
  time_begin(c, 0);
  e = rfast_launch_state(c, RFAST_MODE_MIX, gamma, warm);
  time_end(c, 0);
  if (e != hipSuccess) return hipfail(c, e, "mix launch");
  time_begin(c, 1);
  e = rfast_launch_gradient(c, d_batch_idx);
  time_end(c, 1);
  if (e != hipSuccess) return hipfail(c, e, "gradient launch");
  time_begin(c, 0);
  e = rfast_launch_state(c, RFAST_MODE_TRACK, gamma, warm);
  time_end(c, 0);
  if (e != hipSuccess) return hipfail(c, e, "track launch");
  return after_round(c);
}

// `count` consecutive rounds of least squares or logistic regression whose plans the resolver has written into plan
// sets 0 .. count-1: two kernels per round instead of four (the lane that tracks a coordinate in one round mixes it for
// the next).  d_active, d_batch_idx: the activity flags and the rows of the first of these rounds, those of the others
// behind them.
static int chained_rounds(rfast_ctx* c, int32_t count, float gamma, const uint8_t* d_active, const int32_t* d_batch_idx) {
  const RfastDev& d = c->d;
  const size_t rows = (size_t)d.n * (size_t)d.prob.batch;
  use_plan_set(c, 0);
  time_begin(c, 0);
  hipError_t e = rfast_launch_state(c, RFAST_MODE_MIX, gamma_now(c, gamma), true);
  time_end(c, 0);
  if (e != hipSuccess) return hipfail(c, e, "mix launch");
  for (int32_t q = 0; q < count; ++q) {
    use_plan_set(c, q);
    const int32_t* bi = d_batch_idx ? d_batch_idx + (size_t)q * rows : nullptr;
    const uint8_t* act = d_active + (size_t)q * d.n;
    time_begin(c, 1);
    e = rfast_launch_rows(c, bi, act);
    time_end(c, 1);
    if (e != hipSuccess) return hipfail(c, e, "rows launch");
    time_begin(c, 0);
    e = rfast_launch_cols_track_mix(c, bi, act, q + 1 < count ? act + d.n : nullptr, c->plan_set_bytes,
                                    gamma_at(c, gamma, c->host_round + 1));
    time_end(c, 0);
    if (e != hipSuccess) return hipfail(c, e, "columns, track and mix launch");
    const int rc = after_round(c);
    if (rc != RFAST_OK) return rc;
  }
  return RFAST_OK;
}

// Rounds from which on a launch of the wavefront-tile kernel pays.  It moves every live ring slot, a pass per round only what the
// round reads, so it takes the more rounds the larger the state and the longer the delays, that is, the more versions are live; and
// the fewer, the more nodes are active, which the host does not know: with all of them active a launch is even after little more than
// half as many rounds as with half of them.  One pass per round over a launch, contexts in turn, half / all active:
// Up to 32 nodes, by the wavefronts of the launch that a compute unit holds (12 or more, 8, fewer: delays of up to 4, 8, 16 rounds):
//   to 1 MB per array   mesh of 16, p 14840: 0.96 / 1.07 in calls of 2; delays of up to 8 0.88 / 0.98 of 2, 1.15 / 1.25 of 3 (a ring with
//                       one edge of a kind, p 6248, 1.05 / 1.03 of 2); of up to 16 0.95 / 1.01 of 3
//   to 2 MB             mesh of 16, p 26560: 1.16 / 1.30 of 3; 1.04 / 1.17 of 3; 0.96 / 0.99 of 5
//   to 8 MB             p 62500: 0.84 / 1.27 of 3, 1.05 / 1.47 of 4; 0.93 / 1.31 of 4, 1.11 / 1.49 of 5; 0.90 / 1.24 of 8, 1.01 / 1.45 of 10
//   beyond              p 937500: 0.98 / 1.60 of 4, 1.20 / 1.90 of 5; 0.94 / 1.5 of 5, 1.10 / 1.7 of 6; 0.77 / 1.36 of 12, 0.95 / 1.6 of 16
// 33 to 64 nodes, a lane each (rows in segments of 16 bytes), by the versions that the longest delay reads (delays of up to 4, 8, 16; between
// them by interpolation), ring and mesh of 36, mesh of 60, tree of 64:
//   to 1 MB             0.82 to 0.95 / 0.88 to 1.02 of 2, 1.1 to 1.3 of 3; the same; 0.62 to 0.89 / 0.66 to 0.98 of 3, 0.76 to 1.1 of 4
//   to 2 MB             0.98 to 1.17 / 1.06 to 1.25 of 3; 0.95 to 1.05 / 1.02 to 1.11 of 3; 0.94 to 1.05 of 6
//   to 8 MB             0.83 to 1.3 / 1.3 to 1.8 of 5; 0.78 to 1.1 / 1.2 to 1.5 of 5, 0.88 to 1.3 of 6; 0.82 to 1.02 / 1.2 to 1.4 of 10
//   to 20 MB            0.88 to 1.2 / 1.3 of 6, 0.99 and more of 7; 0.88 to 1.1 / 1.4 of 7; 0.95 to 1.02 / 1.5 of 16, 1.1 to 1.25 of 20
//   to 50 MB            0.89 to 1.2 / 1.5 of 7; 0.77 to 0.92 / 1.2 to 1.4 of 7, 0.86 to 0.98 of 8; 0.93 to 0.97 / 1.4 of 20, 1.0 to 1.1 of 24
//   beyond              0.82 to 1.02 / 1.4 of 7; 0.82 to 0.87 / 1.4 of 8, 0.94 to 1.01 of 10; 0.8 to 0.9 / 1.4 of 20, 0.9 to 0.99 of 24
// and with five and six edges of a kind (exponential graph of 40) 0.93 / 1.07 of 4 to 2 MB, 0.88 to 1.0 / 1.3 of 6 and 7 to 8 MB, 0.9 to 1.04 /
// 1.4 of 9 and 10 beyond.
// One receiver of all edges of C, half of the nodes active (one pass has a node with up to 63 in-edges to wait for, so a launch pays earlier
// where the state is small), delays of up to 4 / 16, even at: 4 to 7 nodes, to 0.5 MB 2 / 3.5 rounds, 2 MB 2 / 5, 5 MB 3.5 / 8, 12 MB 4 / 10, 30 MB 5 / 12
// (7 nodes, 17 MB: 75 us in 4 passes, 68 in a launch of 4; 99 and 76 of 6); 12 and 24 nodes, 0.2 MB 2 / 3 rounds, 2 MB 3 / 5, 16 MB 7.5 / 11.5, 48 MB 11 / 19;
// 48 and 64 nodes, to 2 MB 2 / 2, 16 MB 3.5 / 6, 48 MB 7 / 10, 268 MB 10 / 14; 64 nodes, 2 MB, 20 rounds 6.2 / 5.2 times as fast.
static int32_t wave_least_rounds(const rfast_ctx* c) {
  const RfastDev& d = c->d;
  const double mb = (double)d.n * (double)d.p * 4.0e-6;
  if (c->hub >= 0) {
    static const float star[3][5][2] = {{{2, 4}, {3, 5}, {4, 8}, {5, 10}, {5, 12}}, {{2, 3}, {3, 5}, {5, 8}, {8, 12}, {12, 19}}, {{2, 2}, {2, 2}, {3, 4}, {4, 6}, {8, 10}}};
    const int size = mb > 20.0 ? 4 : mb > 8.0 ? 3 : mb > 2.5 ? 2 : mb > 0.5 ? 1 : 0;
    const float* v = star[d.n <= kStarInOrder ? 0 : d.n <= 32 ? 1 : 2][size];
    const int reach = std::min(d.M - 1, d.d_max + 2);
    const float at = std::min(std::max((float)(reach - 6) / 12.f, 0.f), 1.f), more = d.n > 32 && mb > 100.0 ? 4.f : 0.f;
    return (int32_t)(v[0] + (v[1] - v[0]) * at + more + 0.5f);
  }
  int row = mb > 8.0 ? 3 : mb > 2.0 ? 2 : mb > 1.0 || d.p % 4 != 0 ? 1 : 0;
  if (d.n <= 32) {
    static const int32_t few[4][3] = {{2, 3, 3}, {3, 3, 6}, {4, 5, 10}, {5, 6, 12}};
    const int held = rfast_wave_held(c), col = held >= 12 ? 0 : held >= 8 ? 1 : 2;
    return row == 0 && col == 1 && c->max_degree < 2 ? 2 : few[row][col];
  }
  static const float many[6][3] = {{3, 3, 4}, {3, 3, 6}, {5, 6, 10}, {7, 7, 16}, {7, 8, 20}, {7, 9, 22}};
  static const float many_edges[6][3] = {{3, 3, 4}, {4, 4, 6}, {6, 7, 10}, {9, 9, 16}, {9, 10, 20}, {9, 10, 22}};
  if (row == 3) row += mb > 50.0 ? 2 : mb > 20.0 ? 1 : 0;
  const float* v = c->max_degree > 4 ? many_edges[row] : many[row];
  const int reach = std::min(d.M - 1, d.d_max + 2);  // versions that the longest delay reads, and one more
  const float least = reach <= 6 ? v[0] : reach <= 10 ? v[0] + (v[1] - v[0]) * (float)(reach - 6) / 4.f : v[1] + (v[2] - v[1]) * (float)(reach - 10) / 8.f;
  return (int32_t)(least + 0.5f);
}

// How many of the next `rounds` rounds one launch of the LDS-resident kernel should take (0: run
// the next round as one pass).  A launch holds no rebase, so it must end at the latest on the next
// multiple of the rebase interval, and it runs with one step size, so it must end with the current
// step of the step-size schedule; and it reads and writes every ring slot once, which a large
// state earns back only over enough rounds.
static int32_t block_length(const rfast_ctx* c, int32_t rounds, int64_t at_round) {
  if (!c->use_blocks || c->capturing) return 0;
  const bool gemv = rfast_tiny_eligible(c) || c->team.W > 0;  // (every round of these takes the multi-round kernels)
  if (!gemv && (c->no_tiles || !rfast_wave_eligible(c))) return 0;
  if (gemv && !rfast_tiny_eligible(c) && !team_usable(c)) return 0;
  const int64_t now = at_round >= 0 ? at_round : c->host_round;  // the round the launch would start with
  int32_t len = rounds < kBlockRounds ? rounds : kBlockRounds;
  if (c->rebase_interval > 0) {
    const int64_t to_boundary = c->rebase_interval - now % c->rebase_interval;
    if (to_boundary < len) len = (int32_t)to_boundary;
  }
  if (c->gamma_step > 0) {  // one step size per launch
    const int64_t to_decay = c->gamma_step - now % c->gamma_step;
    if (to_decay < len) len = (int32_t)to_decay;
  }
  if (gemv) return rfast_tiny_eligible(c) || len >= team_least_rounds(c) ? len : 0;
  const double bytes = (double)c->d.n * (double)c->d.p * 4.0;
  int32_t least;
  if (!rfast_block_eligible(c)) {
    least = wave_least_rounds(c);
  } else {  // (the longer launches that take the other kernel do so because it is faster still)
    // (one pass per round / a launch, rings of two or three slots: ring of 36, p 416664, 73 / 77 us per round in calls of 4, 74 / 59 of
    // 6; p 97220: 22.6 / 26.4 of 3, 22.0 / 22.0 of 4; p 27776: 11.2 / 12.5 of 2, 10.2 / 9.7 of 3; p 6944: 9.0 / 7.5 of 2; ring of 48 and
    // tree of 64 alike)
    least = bytes > 20.0e6 ? 5 : bytes > 8.0e6 ? 4 : bytes > 2.0e6 || c->d.p % 4 != 0 ? 3 : 2;
  }
  if (c->use_blocks == 2) least = 2;
  return len >= least ? len : 0;
}

// Resolves `len` rounds (schedule arrays of round q at offset q of each pointer) into plan records,
// one launch, and advances them with one launch.
static int run_block(rfast_ctx* c, int32_t len, const uint8_t* d_active, const int32_t* d_delay_R,
                     const int32_t* d_delay_C, const uint8_t* d_drop_R, const uint8_t* d_drop_C, float gamma,
                     const int32_t* d_batch_idx) {
  RfastDev& d = c->d;
  if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
  RfastBlock blk;
  blk.rounds = len;
  // a rebase that falls due when these rounds are done costs the wavefront-tile kernel nothing: it shifts the
  // running sums while it writes its tiles back (the other kernels are followed by the rebase kernel)
  const bool tiny = rfast_tiny_eligible(c), team = !tiny && c->team.W > 0, wave = !tiny && !team && !rfast_block_takes(c, len);
  const bool rebase_due = c->rebase_interval > 0 && (c->host_round + len) % c->rebase_interval == 0;
  blk.rebase = rebase_due && wave ? 1 : 0;
  blk.gamma = gamma_now(c, gamma);  // of the first round: a launch does not straddle a decay step
  const bool own_resolver = rfast_tiny_resolves(c);  // the one-workgroup kernel resolves its rounds itself
  hipError_t e = hipSuccess;
  d.blk_plan = c->blk_plan_base;
  d.blk_head = tiny || team ? nullptr : c->blk_head_base;
  blk.slots = d.blk_slots = wave ? rfast_wave_slots(c) : 0;
  blk.hub = c->hub;
  blk.v_rows = c->v_rows;
  blk.s_rows = c->s_rows;
  if (!own_resolver) {
    time_begin(c, 2);
    e = rfast_launch_resolve(c, d_active, d_delay_R, d_delay_C, d_drop_R, d_drop_C, len);
    time_end(c, 2);
  }
  c->host_round += len;
  if (e == hipSuccess) {
    time_begin(c, 0);
    if (team)
      e = in_team_order(c, [&] { return launch_team(c, false, len, blk.gamma, d_batch_idx, d_delay_R, d_delay_C); });
    else if (tiny)
      e = rfast_launch_tiny(c, blk, d_batch_idx, (int)(c->host_round - len), d_active, d_delay_R, d_delay_C, d_drop_R, d_drop_C);
    else e = wave ? rfast_launch_wave(c, blk) : rfast_launch_block(c, blk);
    time_end(c, 0);
  }
  d.blk_plan = nullptr;
  d.blk_head = nullptr;
  d.blk_slots = 0;
  if (e != hipSuccess) return hipfail(c, e, "multi-round launch");
  if (rebase_due && !blk.rebase) {
    e = rfast_launch_rebase(c);
    if (e != hipSuccess) return hipfail(c, e, "rebase launch");
  }
  return RFAST_OK;
}

int rfast_block_info(rfast_ctx* c, int32_t* lanes_per_node, int32_t* tile_per_wavefront) {
  if (!c || !lanes_per_node) return RFAST_EINVAL;
  const bool taken = block_length(c, kBlockRounds) > 0 && c->d.p % 4 == 0 && (rfast_tiny_eligible(c) || c->team.W <= 0), wave = rfast_wave_eligible(c) && !rfast_block_eligible(c);
  if (taken && rfast_tiny_eligible(c)) {  // one workgroup holds the whole problem
    *lanes_per_node = 1024 / c->d.n > 0 ? 1024 / c->d.n : 1;
    if (tile_per_wavefront) *tile_per_wavefront = 0;
    return RFAST_OK;
  }
  *lanes_per_node = taken ? (wave ? rfast_wave_lanes(c) : rfast_block_lanes(c)) : 0;
  if (tile_per_wavefront) *tile_per_wavefront = taken && wave ? 1 : 0;
  return RFAST_OK;
}

int rfast_set_tile_group(rfast_ctx* c, int32_t wavefronts) {
  if (!c) return RFAST_EINVAL;
  if (wavefronts != 0 && wavefronts != 1 && wavefronts != 2 && wavefronts != 4)
    return fail(c, RFAST_EINVAL, "wavefronts per workgroup must be 0 (automatic), 1, 2 or 4");
  c->wave_group = wavefronts;
  return RFAST_OK;
}

int rfast_set_wait_limits(rfast_ctx* c, int32_t start_polls, int32_t wait_polls) {
  if (!c) return RFAST_EINVAL;
  c->start_polls = start_polls;
  c->wait_polls = wait_polls;
  return RFAST_OK;
}

int rfast_use_blocks(rfast_ctx* c, int32_t on) {
  if (!c) return RFAST_EINVAL;
  c->use_blocks = on == 2 ? 2 : (on != 0 ? 1 : 0);
  return RFAST_OK;
}

int rfast_run(rfast_ctx* c, int32_t rounds, const uint8_t* d_active, const int32_t* d_delay_R, const int32_t* d_delay_C,
              const uint8_t* d_drop_R, const uint8_t* d_drop_C, float gamma, const int32_t* d_batch_idx) {
  if (!c) return RFAST_EINVAL;
  if (rounds < 0) return fail(c, RFAST_EINVAL, "rounds < 0");
  if (const int rc = state_usable(c)) return rc;
  const RfastDev& d = c->d;
  const size_t B = d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC ? 0 : (size_t)d.prob.batch;
  for (int32_t r = 0; r < rounds; ++r) {
    // the separable objective on a small graph: tiles of coordinates stay in LDS over up to kBlockRounds rounds
    const int32_t len = block_length(c, rounds - r);
    if (len > 0) {
      if (!d_active || (d.eR && (!d_delay_R || !d_drop_R)) || (d.eC && (!d_delay_C || !d_drop_C)))
        return fail(c, RFAST_EINVAL, "NULL schedule pointer");
      if (!std::isfinite(gamma)) return fail(c, RFAST_EINVAL, "gamma is not finite");
      if (c->needs_init) return fail(c, RFAST_EINVAL, "rfast_init must follow rfast_set_optimizer");
      if (B > 0 && !d_batch_idx) return fail(c, RFAST_EINVAL, "sample rows are required when batch > 0");
      const int rc = run_block(c, len, d_active + (size_t)r * d.n, d_delay_R ? d_delay_R + (size_t)r * d.eR : nullptr,
                               d_delay_C ? d_delay_C + (size_t)r * d.eC : nullptr,
                               d_drop_R ? d_drop_R + (size_t)r * d.eR : nullptr,
                               d_drop_C ? d_drop_C + (size_t)r * d.eC : nullptr, gamma,
                               d_batch_idx ? d_batch_idx + (size_t)r * d.n * B : nullptr);
      if (rc != RFAST_OK) return rc;
      r += len - 1;
      continue;
    }
    // One pass per round: the resolver takes up to kResolveAhead rounds in one launch, into as many
    // plan sets (integer state only, so it may run ahead of the kernels); a stretch ends where a
    // multi-round launch may start and, because the rebase reads the counters, on the multiples of
    // the rebase interval.
    int32_t ahead = rounds - r < kResolveAhead ? rounds - r : kResolveAhead;
    for (int32_t q = 1; q < ahead; ++q) {
      const int64_t then = c->host_round + q;
      const bool boundary = c->rebase_interval > 0 && then % c->rebase_interval == 0;
      if (boundary || block_length(c, rounds - r - q, then) > 0) { ahead = q; break; }
    }
    int rc = check_round_args(c, d_active + (size_t)r * d.n, d_delay_R, d_delay_C, d_drop_R, d_drop_C, gamma, d_batch_idx);
    if (rc != RFAST_OK) return rc;
    if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
    use_plan_set(c, 0);
    time_begin(c, 2);
    const hipError_t e = rfast_launch_resolve(c, d_active + (size_t)r * d.n, d_delay_R ? d_delay_R + (size_t)r * d.eR : nullptr,
                                              d_delay_C ? d_delay_C + (size_t)r * d.eC : nullptr,
                                              d_drop_R ? d_drop_R + (size_t)r * d.eR : nullptr,
                                              d_drop_C ? d_drop_C + (size_t)r * d.eC : nullptr, ahead, c->plan_set_bytes);
    time_end(c, 2);
    if (e != hipSuccess) return hipfail(c, e, "resolver launch");
    if (c->use_blocks && rfast_chain_eligible(c)) {
      rc = chained_rounds(c, ahead, gamma, d_active + (size_t)r * d.n, d_batch_idx ? d_batch_idx + (size_t)r * d.n * B : nullptr);
      if (rc != RFAST_OK) return rc;
    } else if (c->no_tiles && c->use_blocks && !c->profiling && d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC) {
      for (int32_t q = 0; q < ahead;) {
        use_plan_set(c, q);
        int32_t len = ahead - q;  // one step size per launch (and no rebase inside: the stretch ends there)
        if (c->gamma_step > 0) len = (int32_t)std::min<int64_t>(len, c->gamma_step - c->host_round % c->gamma_step);
        const hipError_t g = rfast_launch_events(c, gamma_now(c, gamma), len);
        if (g != hipSuccess) return hipfail(c, g, "event-driven iterations launch");
        c->host_round += len - 1;
        rc = after_round(c);
        if (rc != RFAST_OK) return rc;
        q += len;
      }
      use_plan_set(c, ahead - 1);
    } else {
      for (int32_t q = 0; q < ahead; ++q) {
        use_plan_set(c, q);
        rc = float_round(c, gamma, d_batch_idx ? d_batch_idx + (size_t)(r + q) * d.n * B : nullptr, rounds >= 8);
        if (rc != RFAST_OK) return rc;
      }
    }
    r += ahead - 1;
  }
  return RFAST_OK;
}

int rfast_use_graphs(rfast_ctx* c, int32_t on) {
  if (!c) return RFAST_EINVAL;
  c->use_graphs = on != 0;
  if (!on) drop_graph(c);
  return RFAST_OK;
}

int rfast_run_generated(rfast_ctx* c, int32_t rounds, uint64_t seed, const float* d_p_active, int32_t max_delay,
                        float p_drop, float gamma) {
  if (!c || !d_p_active) return RFAST_EINVAL;
  if (rounds < 0) return fail(c, RFAST_EINVAL, "rounds < 0");
  const RfastDev& d = c->d;
  if (max_delay < 0 || max_delay > d.d_max) return fail(c, RFAST_ERANGE, "max_delay must lie in [0, D - burst + 1]");
  if (!(p_drop >= 0.f && p_drop <= 1.f)) return fail(c, RFAST_ERANGE, "p_drop must lie in [0, 1]");
  if (!std::isfinite(gamma)) return fail(c, RFAST_EINVAL, "gamma is not finite");
  // A generated round takes no host argument that varies from round to round (the
  // generator reads the round number on the device), so kGraphRounds of them are
  // captured once into a HIP graph and replayed: one launch per kGraphRounds rounds.
  if (c->needs_init) return fail(c, RFAST_EINVAL, "rfast_init must follow rfast_set_optimizer");
  if (const int rc = state_usable(c)) return rc;
  const bool graphs = c->use_graphs && !c->profiling;
  while (rounds > 0) {
    // a graph bakes the step size in, so a replay must not straddle a decay step of the schedule,
    // and it must hold no rebase, so it must end before the next multiple of the rebase interval
    const bool one_step_size = c->gamma_step <= 0 || c->host_round % c->gamma_step + kGraphRounds <= c->gamma_step;
    const bool no_rebase_inside =
        c->rebase_interval <= 0 || c->host_round % c->rebase_interval + kGraphRounds < c->rebase_interval;
    if (graphs && rounds >= kGraphRounds && one_step_size && no_rebase_inside) {
      if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
      const bool same = c->graph_exec && c->graph_seed == seed && c->graph_p_active == d_p_active &&
                        c->graph_max_delay == max_delay && c->graph_p_drop == p_drop && c->graph_gamma == gamma_now(c, gamma);
      if (!same) {
        const int rc = build_graph(c, seed, d_p_active, max_delay, p_drop, gamma);
        if (rc != RFAST_OK) return rc;
      }
      const hipError_t e = hipGraphLaunch(c->graph_exec, c->stream);
      if (e != hipSuccess) return hipfail(c, e, "hipGraphLaunch");
      c->host_round += kGraphRounds;
      c->gen_last = 0;
      rounds -= kGraphRounds;
      continue;
    }
    // no replay: the schedule of the next stretch of rounds in one launch, then as an uploaded one
    // (several rounds per launch where that applies, else the resolver ahead of the round kernels)
    int32_t len = rounds < c->gen_depth ? rounds : c->gen_depth;
    if (graphs && len > kGraphRounds) len = kGraphRounds;  // a replay may become possible again after a boundary
    const hipError_t e = rfast_launch_generate(c, seed, d_p_active, max_delay, p_drop, false, len);
    if (e != hipSuccess) return hipfail(c, e, "schedule generator launch");
    const int rc = rfast_run(c, len, d.gen_active, d.gen_delay_r, d.gen_delay_c, d.gen_drop_r, d.gen_drop_c, gamma, d.gen_batch);
    if (rc != RFAST_OK) return rc;
    c->gen_last = len - 1;
    rounds -= len;
  }
  return RFAST_OK;
}

int rfast_run_events(rfast_ctx* c, int32_t iterations, uint64_t seed, const float* host_weights, int32_t max_delay,
                     float p_drop, float gamma) {
  if (!c) return RFAST_EINVAL;
  if (iterations < 0) return fail(c, RFAST_EINVAL, "iterations < 0");
  const RfastDev& d = c->d;
  if (max_delay < 0 || max_delay > d.d_max) return fail(c, RFAST_ERANGE, "max_delay must lie in [0, D - burst + 1]");
  if (!(p_drop >= 0.f && p_drop <= 1.f)) return fail(c, RFAST_ERANGE, "p_drop must lie in [0, 1]");
  if (!std::isfinite(gamma)) return fail(c, RFAST_EINVAL, "gamma is not finite");
  if (c->needs_init) return fail(c, RFAST_EINVAL, "rfast_init must follow rfast_set_optimizer");
  if (const int rc = state_usable(c)) return rc;
  // selection thresholds: node i is drawn when cdf[i-1] <= u < cdf[i], u a 32-bit word
  std::vector<uint32_t> cdf(d.n);
  double total = 0.0;
  for (int i = 0; i < d.n; ++i) {
    const double w = host_weights ? (double)host_weights[i] : 1.0;
    if (!(w >= 0.0) || !std::isfinite(w)) return fail(c, RFAST_ERANGE, "selection weights must be finite and >= 0");
    total += w;
  }
  if (!(total > 0.0)) return fail(c, RFAST_ERANGE, "selection weights sum to zero");
  double cum = 0.0;
  for (int i = 0; i < d.n; ++i) {
    cum += host_weights ? (double)host_weights[i] : 1.0;
    const double thr = std::floor(cum / total * 4294967296.0);
    cdf[i] = thr >= 4294967295.0 ? 0xFFFFFFFFu : (uint32_t)thr;
  }
  hipError_t e = hipMemcpyAsync(d.gen_cdf, cdf.data(), (size_t)d.n * 4, hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);  // the host vector dies with this scope
  if (e != hipSuccess) return hipfail(c, e, "uploading selection thresholds");
  // A stretch of iterations drawn by one launch, then, for the separable objective, up to kResolveAhead of them per launch
  // (not on tiles in LDS, where one lane in n would work); the kernels of least squares and logistic regression skip the rounds of nodes that are not active.
  c->no_tiles = true;
  int rc = RFAST_OK;
  for (int32_t k = 0; k < iterations && rc == RFAST_OK;) {
    const int32_t len = iterations - k < c->gen_depth ? iterations - k : c->gen_depth;
    e = rfast_launch_generate(c, seed, nullptr, max_delay, p_drop, true, len);
    if (e != hipSuccess) {
      rc = hipfail(c, e, "schedule generator launch");
      break;
    }
    rc = rfast_run(c, len, d.gen_active, d.gen_delay_r, d.gen_delay_c, d.gen_drop_r, d.gen_drop_c, gamma, d.gen_batch);
    c->gen_last = len - 1;
    k += len;
  }
  c->no_tiles = false;
  return rc;
}

int rfast_sync_round(rfast_ctx* c, float gamma, const int32_t* d_batch_idx) {
  if (!c) return RFAST_EINVAL;
  const RfastDev& d = c->d;
  const bool separable = d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC;
  if (!separable && d.prob.batch > 0 && !d_batch_idx) return fail(c, RFAST_EINVAL, "sample rows are required when batch > 0");
  if (!std::isfinite(gamma)) return fail(c, RFAST_EINVAL, "gamma is not finite");
  if (c->needs_init) return fail(c, RFAST_EINVAL, "rfast_init must follow rfast_set_optimizer");
  if (const int rc = state_usable(c)) return rc;
  if (d.prob.kind != RFAST_OBJ_SOFTMAX_BF16 && team_usable(c)) return rfast_sync_run(c, 1, gamma, d_batch_idx);
  gamma = gamma_now(c, gamma);
  hipError_t e;
  time_begin(c, 0);
  e = rfast_launch_sync(c, separable ? 2 : 0, gamma, c->sync_parity);
  time_end(c, 0);
  if (e != hipSuccess) return hipfail(c, e, "synchronous step launch");
  if (!separable) {
    time_begin(c, 1);
    e = rfast_launch_gradient(c, d_batch_idx);
    time_end(c, 1);
    if (e != hipSuccess) return hipfail(c, e, "gradient launch");
    time_begin(c, 0);
    e = rfast_launch_sync(c, 1, gamma, c->sync_parity);
    time_end(c, 0);
    if (e != hipSuccess) return hipfail(c, e, "synchronous tracker launch");
  }
  c->sync_parity ^= 1;
  c->host_round++;
  return RFAST_OK;
}

int rfast_sync_run(rfast_ctx* c, int32_t rounds, float gamma, const int32_t* d_batch_idx) {
  if (!c) return RFAST_EINVAL;
  if (rounds < 0) return fail(c, RFAST_EINVAL, "rounds < 0");
  if (const int rc = state_usable(c)) return rc;
  const RfastDev& d = c->d;
  const size_t B = d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC ? 0 : (size_t)d.prob.batch;
  const bool multi = c->use_blocks && rfast_sync_wave_eligible(c);
  const bool team = d.prob.kind != RFAST_OBJ_SOFTMAX_BF16 && team_usable(c);
  for (int32_t r = 0; r < rounds;) {
    if (team) {  // least squares / logistic regression: the steps up to the next decay of the step size in one launch
      int32_t len = std::min(rounds - r, 1 << 20);
      if (c->gamma_step > 0) len = (int32_t)std::min<int64_t>(len, c->gamma_step - c->host_round % c->gamma_step);
      if (!std::isfinite(gamma)) return fail(c, RFAST_EINVAL, "gamma is not finite");
      if (c->needs_init) return fail(c, RFAST_EINVAL, "rfast_init must follow rfast_set_optimizer");
      if (B > 0 && !d_batch_idx) return fail(c, RFAST_EINVAL, "sample rows are required when batch > 0");
      if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
      time_begin(c, 0);
      hipError_t e = in_team_order(c, [&] {
        return launch_team(c, true, len, gamma_now(c, gamma), d_batch_idx ? d_batch_idx + (size_t)r * d.n * B : nullptr, nullptr, nullptr);
      });
      time_end(c, 0);
      if (e == hipSuccess) e = rfast_launch_sync_plan(c, len);
      if (e != hipSuccess) return hipfail(c, e, "multi-step synchronous launch");
      c->host_round += len;
      r += len;
      continue;
    }
    // several steps per launch for the separable objective on a small graph, with one step size
    int32_t len = multi ? rounds - r : 0;
    if (len > 0 && c->gamma_step > 0) {
      const int64_t to_decay = c->gamma_step - c->host_round % c->gamma_step;
      if (to_decay < len) len = (int32_t)to_decay;
    }
    if (len >= 2) {
      if (!std::isfinite(gamma)) return fail(c, RFAST_EINVAL, "gamma is not finite");
      if (c->needs_init) return fail(c, RFAST_EINVAL, "rfast_init must follow rfast_set_optimizer");
      if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
      time_begin(c, 0);
      hipError_t e = rfast_launch_sync_wave(c, gamma_now(c, gamma), len);
      time_end(c, 0);
      if (e == hipSuccess) e = rfast_launch_sync_plan(c, len);
      if (e != hipSuccess) return hipfail(c, e, "multi-step synchronous launch");
      c->host_round += len;
      r += len;
      continue;
    }
    const int rc = rfast_sync_round(c, gamma, d_batch_idx ? d_batch_idx + (size_t)r * d.n * B : nullptr);
    if (rc != RFAST_OK) return rc;
    ++r;
  }
  return RFAST_OK;
}

int rfast_set_optimizer(rfast_ctx* c, float momentum, float weight_decay, float* d_momentum) {
  if (!c) return RFAST_EINVAL;
  if (!(momentum >= 0.f && momentum < 1.f)) return fail(c, RFAST_ERANGE, "momentum must lie in [0, 1)");
  if (!(weight_decay >= 0.f) || !std::isfinite(weight_decay)) return fail(c, RFAST_ERANGE, "weight_decay must be finite and >= 0");
  if (momentum != 0.f && !d_momentum) return fail(c, RFAST_EINVAL, "momentum != 0 needs a buffer of n*p floats");
  if (d_momentum && ((uintptr_t)d_momentum % 16) != 0) return fail(c, RFAST_EINVAL, "momentum buffer must be 16-byte aligned");
  drop_graph(c);  // a captured graph holds the old kernel arguments
  c->d.beta = momentum;
  c->d.wd = weight_decay;
  c->d.mom = momentum != 0.f ? d_momentum : nullptr;
  c->needs_init = true;
  const hipError_t e = rfast_wave_prime(c);  // the variant has instantiations of its own
  if (e != hipSuccess) return hipfail(c, e, "loading the multi-round kernel");
  return RFAST_OK;
}

int rfast_set_gamma_schedule(rfast_ctx* c, int32_t step_rounds, float factor) {
  if (!c) return RFAST_EINVAL;
  if (step_rounds < 0) return fail(c, RFAST_EINVAL, "step_rounds < 0");
  if (!(factor > 0.f) || !std::isfinite(factor)) return fail(c, RFAST_ERANGE, "factor must be finite and > 0");
  c->gamma_step = step_rounds;
  c->gamma_factor = factor;
  return RFAST_OK;
}

int rfast_set_rebase_interval(rfast_ctx* c, int32_t rounds) {
  if (!c || rounds < 0) return RFAST_EINVAL;
  c->rebase_interval = rounds;
  return RFAST_OK;
}

int rfast_rebase(rfast_ctx* c) {
  if (!c) return RFAST_EINVAL;
  const hipError_t e = rfast_launch_rebase(c);
  if (e != hipSuccess) return hipfail(c, e, "rebase launch");
  return RFAST_OK;
}

int rfast_check(rfast_ctx* c) {
  if (!c) return RFAST_EINVAL;
  int32_t err[6];
  const hipError_t e = to_host(c, err, c->d.err, 24);
  if (e != hipSuccess) return hipfail(c, e, "reading device status");
  const uint64_t edge = (uint64_t)(uint32_t)err[5] << 32 | (uint32_t)err[4];  // the earliest delay out of range
  if (edge != ~0ull && err[0] != RFAST_EHIP && (err[0] == 0 || (int32_t)(edge >> 32) <= err[1])) {
    err[0] = RFAST_ERANGE;
    err[1] = (int32_t)(edge >> 32);
    err[2] = (int32_t)(edge >> 31 & 1);
    err[3] = (int32_t)(edge & 0x7fffffff);
  }
  if (err[0] == 0) return RFAST_OK;
  static const char* kinds[] = {"delay on R edge", "delay on C edge", "sample row of node", "class label of a sample of node"};
  if (err[0] == RFAST_EHIP)
    return fail(c, RFAST_EHIP, "a workgroup waited in vain for another one in the rounds from " + std::to_string(err[1]) +
                                   " on: the state is not valid before the next rfast_init");
  const char* what = err[2] >= 0 && err[2] <= 3 ? kinds[err[2]] : "value";
  return fail(c, err[0], std::string(what) + " " + std::to_string(err[3]) + " out of range in round " + std::to_string(err[1]) +
                             " (clamped on the device)");
}

int rfast_read_state(rfast_ctx* c, int32_t field, void* host_dst, size_t bytes) {
  if (!c || !host_dst) return RFAST_EINVAL;
  const size_t want = field_bytes(c, field);
  if (want == (size_t)-1) return fail(c, RFAST_EINVAL, "unknown field");
  if (bytes != want) return fail(c, RFAST_EINVAL, "field holds " + std::to_string(want) + " bytes");
  const RfastDev& d = c->d;
  if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
  hipError_t e = hipSuccess;
  if (bytes == 0) {
    e = hipStreamSynchronize(c->stream);
    return e == hipSuccess ? RFAST_OK : hipfail(c, e, "stream synchronize");
  }
  const void* src = nullptr;
  switch (field) {
    case RFAST_X: src = d.x; break;
    case RFAST_Z: src = d.z; break;
    case RFAST_V_RING: src = d.v_ring; break;
    case RFAST_SIGMA_RING: src = d.sigma_ring; break;
    case RFAST_RHO_TILDE: src = d.rho_tilde; break;
    case RFAST_T_NODE: src = d.t; break;
    case RFAST_TAU_R: src = d.tau_r; break;
    case RFAST_TAU_C: src = d.tau_c; break;
    case RFAST_SLOT_R: src = d.slot_r; break;
    case RFAST_SLOT_C: src = d.slot_c; break;
    case RFAST_ROUND: src = d.round_no; break;
    case RFAST_DELIV_R: src = d.deliv_r; break;
    case RFAST_DELIV_C: src = d.deliv_c; break;
    case RFAST_T_HIST: src = d.t_hist; break;
    // the generator's arrays hold a stretch of rounds; these fields are the last round executed
    case RFAST_SCHED_ACTIVE: src = d.gen_active + (size_t)c->gen_last * d.n; break;
    case RFAST_SCHED_DELAY_R: src = d.gen_delay_r + (size_t)c->gen_last * d.eR; break;
    case RFAST_SCHED_DELAY_C: src = d.gen_delay_c + (size_t)c->gen_last * d.eC; break;
    case RFAST_SCHED_DROP_R: src = d.gen_drop_r + (size_t)c->gen_last * d.eR; break;
    case RFAST_SCHED_DROP_C: src = d.gen_drop_c + (size_t)c->gen_last * d.eC; break;
    case RFAST_SCHED_BATCH:
      src = d.gen_batch + (size_t)c->gen_last * d.n * (d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC ? 0 : d.prob.batch);
      break;
    case RFAST_MOMENTUM: src = d.mom; break;
    default: break;
  }
  if (field == RFAST_RHO_RING) {
    // rho_ij = a_ij * sigma_j: expand the per-sender rings into per-edge rings
    // (fp32 product, the value the kernels consume)
    std::vector<int32_t> src_h(d.eC);
    std::vector<float> w_h(d.eC);
    e = hipStreamSynchronize(c->stream);
    if (e == hipSuccess && d.eC) e = hipMemcpy(src_h.data(), d.c_src, (size_t)d.eC * 4, hipMemcpyDeviceToHost);
    if (e == hipSuccess && d.eC) e = hipMemcpy(w_h.data(), d.c_w, (size_t)d.eC * 4, hipMemcpyDeviceToHost);
    const size_t ring = (size_t)d.M * d.p;
    for (int q = 0; q < d.eC && e == hipSuccess; ++q) {
      float* dst = (float*)host_dst + (size_t)q * ring;
      e = to_host(c, dst, d.sigma_ring + (size_t)src_h[q] * ring, ring * 4);
      for (size_t k = 0; k < ring; ++k) dst[k] = w_h[q] * dst[k];
    }
    if (e == hipSuccess) e = zero_dead_slots(c, true, (float*)host_dst, d.eC, src_h.data());
  } else if (field == RFAST_RHO_TILDE) {
    // rho~_ij = a_ij * sigma_j[tau_ij] lives in the sender's ring while tau_ij >= t_j - D and in the
    // array otherwise: put the two together
    std::vector<int32_t> src_h(d.eC), tau_h(d.eC), t_h(d.n);
    std::vector<float> w_h(d.eC);
    e = to_host(c, host_dst, d.rho_tilde, bytes);
    if (e == hipSuccess) e = hipMemcpy(src_h.data(), d.c_src, (size_t)d.eC * 4, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(w_h.data(), d.c_w, (size_t)d.eC * 4, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(tau_h.data(), d.tau_c, (size_t)d.eC * 4, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(t_h.data(), d.t, (size_t)d.n * 4, hipMemcpyDeviceToHost);
    for (int q = 0; q < d.eC && e == hipSuccess; ++q) {
      const int j = src_h[q];
      if (tau_h[q] < t_h[j] - (d.M - 2)) continue;
      float* dst = (float*)host_dst + (size_t)q * d.p;
      e = to_host(c, dst, d.sigma_ring + ((size_t)j * d.M + tau_h[q] % d.M) * d.p, (size_t)d.p * 4);
      for (int64_t k = 0; k < d.p; ++k) dst[k] = w_h[q] * dst[k];
    }
  } else if (field == RFAST_G) {
    // the separable objective keeps no sample in memory: write the current ones out first
    if (d.prob.kind == RFAST_OBJ_DIAG_QUADRATIC) {
      e = rfast_diag_init_gradient(c);
      if (e != hipSuccess) return hipfail(c, e, "forming the gradient samples");
    }
    // the stored sample of node i is the one of version t_i: g[t_i & 1][i]
    std::vector<int32_t> t(d.n);
    e = to_host(c, t.data(), d.t, (size_t)d.n * 4);
    const size_t vec = (size_t)d.p * 4;
    for (int i = 0; i < d.n && e == hipSuccess; ++i)
      e = to_host(c, (char*)host_dst + i * vec, (const char*)d.g + ((size_t)(t[i] & 1) * d.n + i) * vec, vec);
  } else {
    e = to_host(c, host_dst, src, bytes);
    if (e == hipSuccess && (field == RFAST_V_RING || field == RFAST_SIGMA_RING))
      e = zero_dead_slots(c, field == RFAST_SIGMA_RING, (float*)host_dst, d.n, nullptr);
  }
  if (e != hipSuccess) return hipfail(c, e, "copying state to host");
  return state_usable(c);
}

int rfast_write_state(rfast_ctx* c, int32_t field, const void* host_src, size_t bytes) {
  if (!c || !host_src) return RFAST_EINVAL;
  if (field == RFAST_RHO_RING || field == RFAST_SLOT_R || field == RFAST_SLOT_C ||
      (field >= RFAST_SCHED_ACTIVE && field <= RFAST_SCHED_BATCH))
    return fail(c, RFAST_EINVAL, "this field is derived and cannot be written");
  const size_t want = field_bytes(c, field);
  if (want == (size_t)-1) return fail(c, RFAST_EINVAL, "unknown field");
  if (bytes != want) return fail(c, RFAST_EINVAL, "field holds " + std::to_string(want) + " bytes");
  const RfastDev& d = c->d;
  if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
  hipError_t e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hipfail(c, e, "stream synchronize");
  if (bytes == 0) return RFAST_OK;
  void* dst = nullptr;
  switch (field) {
    case RFAST_X: dst = d.x; break;
    case RFAST_Z: dst = d.z; break;
    case RFAST_V_RING: dst = d.v_ring; break;
    case RFAST_SIGMA_RING: dst = d.sigma_ring; break;
    case RFAST_RHO_TILDE: dst = d.rho_tilde; break;
    case RFAST_T_NODE: dst = d.t; break;
    case RFAST_TAU_R: dst = d.tau_r; break;
    case RFAST_TAU_C: dst = d.tau_c; break;
    case RFAST_ROUND: dst = d.round_no; break;
    case RFAST_DELIV_R: dst = d.deliv_r; break;
    case RFAST_DELIV_C: dst = d.deliv_c; break;
    case RFAST_T_HIST: dst = d.t_hist; break;
    case RFAST_MOMENTUM: dst = d.mom; break;
    default: break;
  }
  if (field == RFAST_ROUND) c->host_round = *(const int32_t*)host_src;
  if (field == RFAST_G) {
    // both parities receive the sample, so the order of restoring G and T_NODE does not matter
    e = hipMemcpy(d.g, host_src, bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy((char*)d.g + bytes, host_src, bytes, hipMemcpyHostToDevice);
  } else {
    e = hipMemcpy(dst, host_src, bytes, hipMemcpyHostToDevice);
  }
  if (e != hipSuccess) return hipfail(c, e, "copying state to the device");
  return RFAST_OK;
}

int rfast_diagnostics(rfast_ctx* c, const float* d_xstar, rfast_diag* host_out) {
  if (!c || !host_out) return RFAST_EINVAL;
  if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
  hipError_t e = rfast_launch_diag(c, d_xstar, c->d_diag);
  if (e != hipSuccess) return hipfail(c, e, "diagnostics launch");
  double h[8];
  e = to_host(c, h, c->d_diag, sizeof(h));
  if (e != hipSuccess) return hipfail(c, e, "copying diagnostics");
  host_out->consensus_sq = h[0];
  host_out->z_sq = h[1];
  host_out->conservation_sq = h[2];
  host_out->gsum_sq = h[3];
  host_out->xbar_gap_sq = d_xstar ? h[4] : -1.0;
  // sum_i f_i(xbar); the l2 term of the logistic objective and the weight decay of the optimizer
  // variant each add n * coefficient/2 * ||xbar||^2
  const double l2 = (c->d.prob.kind == RFAST_OBJ_LOGISTIC ? (double)c->d.prob.lambda : 0.0) + (double)c->d.wd;
  host_out->loss_at_xbar = h[5] + 0.5 * l2 * c->d.n * h[6];
  return state_usable(c);
}

int rfast_diagnostics_static(rfast_ctx* c, const float* d_xstar, double* d_out) {
  if (!c || !d_out) return RFAST_EINVAL;
  if (c->d.prob.kind != RFAST_OBJ_DIAG_QUADRATIC && c->d.p > rfast_static_max_coords())
    return fail(c, RFAST_ERANGE, "rfast_diagnostics_static: p = " + std::to_string(c->d.p) + " exceeds the " +
                                     std::to_string(rfast_static_max_coords()) +
                                     " coordinates its static scratch holds for this objective (use rfast_diagnostics)");
  if (const int rc = state_usable(c)) return rc;
  if (fold_sync(c) != RFAST_OK) return RFAST_EHIP;
  const double l2 = (c->d.prob.kind == RFAST_OBJ_LOGISTIC ? (double)c->d.prob.lambda : 0.0) + (double)c->d.wd;
  const hipError_t e = rfast_launch_diag_static(c, d_xstar, d_out, 0.5 * l2 * c->d.n);
  if (e != hipSuccess) return hipfail(c, e, "diagnostics launch (static scratch)");
  return RFAST_OK;
}

int rfast_profile_enable(rfast_ctx* c, int32_t on) {
  if (!c) return RFAST_EINVAL;
  constexpr size_t kMax = 4096;
  if (on && c->ev[0][0].empty()) {
    for (int w = 0; w < 3; ++w)
      for (int s = 0; s < 2; ++s) {
        const size_t cnt = (w == 0 ? 2 : 1) * kMax;
        c->ev[w][s].resize(cnt);
        for (size_t k = 0; k < cnt; ++k)
          if (hipEventCreate(&c->ev[w][s][k]) != hipSuccess) return fail(c, RFAST_EHIP, "hipEventCreate failed");
      }
  }
  for (int w = 0; w < 3; ++w) c->ev_used[w] = 0;
  c->profiling = on != 0;
  return RFAST_OK;
}

int rfast_kernel_time(rfast_ctx* c, int32_t which, double* ms_sum, int64_t* launches) {
  if (!c || which < 0 || which > 2 || !ms_sum || !launches) return RFAST_EINVAL;
  hipError_t e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hipfail(c, e, "stream synchronize");
  double tot = 0.0;
  for (size_t k = 0; k < c->ev_used[which]; ++k) {
    float ms = 0.f;
    e = hipEventElapsedTime(&ms, c->ev[which][0][k], c->ev[which][1][k]);
    if (e != hipSuccess) return hipfail(c, e, "hipEventElapsedTime");
    tot += ms;
  }
  *ms_sum = tot;
  *launches = (int64_t)c->ev_used[which];
  return RFAST_OK;
}

const char* rfast_last_error(const rfast_ctx* c) { return c ? c->err.c_str() : g_create_error.c_str(); }

void rfast_destroy(rfast_ctx* c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  leave_team_order(c);
  drop_graph(c);
  if (c->capture_stream) (void)hipStreamDestroy(c->capture_stream);
  for (int w = 0; w < 3; ++w)
    for (int s = 0; s < 2; ++s)
      for (hipEvent_t ev : c->ev[w][s]) (void)hipEventDestroy(ev);
  drop_told(c);
  context_gone();
  delete c;
}

}  // extern "C"
