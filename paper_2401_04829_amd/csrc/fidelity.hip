// Fidelity of an explanation (eq. 7-8, Sec. 4.3; protocol of Sec. 4.6).
//
// Importance of a player is |phi| (Sec. 2.3), larger first, equal values by
// lower player index.  G_S keeps all players but the floor(s M) least
// important, G_{C \ S} all but the min(k, M) most important; both are
// evaluated as two deterministic coalitions by the coalition kernels, and a
// target's terms are |f(G_C) - f(G_S)| and |f(G_C) - f(G_{C\S})| for the
// explained output.
//
// The two player sets come from one workgroup per target: the n-th largest
// key (the float bits of |phi|, which order like the values) by a radix
// selection, eight bits at a time, for both sets together (a histogram in LDS
// and a suffix sum over its bins per step; a binary search over the bits, a
// count over the players each, took 36 us for 20 to 400 players); then one
// pass in player order that ranks the players equal to that key by a prefix
// count (wave ballots) and writes the mask words with ballots.
//
// Targets of models that the batched evaluation takes run together (with the
// kernels that the single call takes), one
// launch per step (each alone is a chain of four one-workgroup kernels).
// Bound by launch latency and the chain of dependent steps in a workgroup:
// 40 Cora-shaped targets 2565 us one target after the other, 145 us now.
#include <algorithm>
#include <cmath>
#include <vector>

#include "batch.h"

namespace {

constexpr int kFidThreads = 1024;
constexpr int kFidWaves = kFidThreads / 64;

__device__ __forceinline__ uint32_t key_of(const float* __restrict__ phi, int64_t j) {
  return __float_as_uint(phi[j]) & 0x7FFFFFFFu;   // |phi| as ordered bits
}

// A set of the n most important players: key > thr, and the first `need`
// players with key == thr.
struct Cut {
  uint32_t thr, need;
};

// The cuts of two sets of n[0] and n[1] players, 0 < n < M (others are left
// undefined): the keys' bytes from the highest down; each step counts the
// keys that share the bytes found so far by their next byte and takes the
// largest byte that leaves at least the wanted number at or above it.
__device__ void select_cuts(const float* __restrict__ phi, int64_t M, const int64_t (&n)[2], Cut (&cut)[2]) {
  __shared__ uint32_t hist[2][256];
  __shared__ uint32_t found[2], left[2];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  if (tid < 2) {
    found[tid] = 0;
    left[tid] = static_cast<uint32_t>(n[tid]);
  }
  for (int shift = 24; shift >= 0; shift -= 8) {
    if (tid < 512) hist[tid >> 8][tid & 255] = 0;
    __syncthreads();
    const uint32_t f0 = found[0], f1 = found[1];
    const uint32_t above = shift == 24 ? 0u : ~0u << (shift + 8);
    for (int64_t j = tid; j < M; j += kFidThreads) {
      const uint32_t k = key_of(phi, j);
      if ((k & above) == f0) atomicAdd(&hist[0][(k >> shift) & 255], 1u);
      if ((k & above) == f1) atomicAdd(&hist[1][(k >> shift) & 255], 1u);
    }
    __syncthreads();
    if (wv < 2) {   // wavefront s: set s; lane l: bins 255 - 4 l .. 252 - 4 l
      uint32_t c[4], sum = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c[q] = hist[wv][255 - 4 * lane - q];
        sum += c[q];
      }
      uint32_t upto = sum;   // keys in this lane's bins and the larger ones
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t x = __shfl_up(upto, off);
        if (lane >= off) upto += x;
      }
      const uint32_t want = left[wv];
      uint32_t over = upto - sum;
      if (over < want && want <= upto) {   // one lane (none when n is not in (0, M])
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (over < want && want <= over + c[q]) {
            found[wv] |= static_cast<uint32_t>(255 - 4 * lane - q) << shift;
            left[wv] = want - over;
          }
          over += c[q];
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) cut[q] = Cut{found[q], left[q]};
}

// Row `out` of masks: bit j set iff player j is among the n most important
// (complemented within the M players when `complement`).
__device__ void write_top(const float* __restrict__ phi, int64_t M, int64_t n, Cut cut, bool complement, int64_t wpr,
                          uint64_t* __restrict__ out, uint32_t* red) {
  const bool all = n >= M, none = n <= 0;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint32_t carry = 0;
  for (int64_t base = 0; base < M; base += kFidThreads) {
    const int64_t j = base + threadIdx.x;
    const bool valid = j < M;
    const uint32_t k = valid ? key_of(phi, j) : 0u;
    const bool eq = valid && !all && !none && k == cut.thr;
    const bool gt = valid && !all && !none && k > cut.thr;
    const uint64_t eqb = __ballot(eq);
    const uint32_t before = __popcll(eqb & ((1ull << lane) - 1ull));
    __syncthreads();
    if (lane == 0) red[wv] = __popcll(eqb);
    __syncthreads();
    uint32_t wave_off = 0, total = 0;
    for (int i = 0; i < kFidWaves; ++i) {
      if (i < wv) wave_off += red[i];
      total += red[i];
    }
    const bool in = all ? valid : (gt || (eq && carry + wave_off + before < cut.need));
    const bool bit = valid && (complement ? !in : in);
    const uint64_t word = __ballot(bit);
    const int64_t w = (base >> 6) + wv;
    if (lane == 0 && w < wpr) out[w] = word;
    carry += total;
  }
}

// One target of a launch.
struct FidJob {
  const float* phi;
  int64_t M, n_keep, n_top, wpr;
  uint64_t* masks;   // G_S, then G_{C \ S}
  const float* y;    // their values
  const float* fef;
  float* out;
};

__device__ __forceinline__ void masks_body(const FidJob& J) {
  __shared__ uint32_t red[kFidWaves];
  const int64_t n[2] = {J.n_keep, J.n_top};
  Cut cut[2];
  select_cuts(J.phi, J.M, n, cut);
  write_top(J.phi, J.M, J.n_keep, cut[0], false, J.wpr, J.masks, red);          // G_S
  write_top(J.phi, J.M, J.n_top, cut[1], true, J.wpr, J.masks + J.wpr, red);    // G_{C \ S}
}

__global__ void __launch_bounds__(kFidThreads) k_fid_masks(FidJob J) { masks_body(J); }
__global__ void __launch_bounds__(kFidThreads) k_fid_masks_batch(const FidJob* __restrict__ jobs) {
  masks_body(jobs[blockIdx.x]);
}

// out[0] = |f(G_C) - f(G_S)|, out[1] = |f(G_C) - f(G_{C\S})|, out[2] = f(G_C).
__device__ __forceinline__ void terms_body(const float* __restrict__ y, const float* __restrict__ fef,
                                           float* __restrict__ out) {
  const double full = fef[1];
  out[0] = static_cast<float>(fabs(full - static_cast<double>(y[0])));
  out[1] = static_cast<float>(fabs(full - static_cast<double>(y[1])));
  out[2] = fef[1];
}
__global__ void k_fid_terms(const float* __restrict__ y, const float* __restrict__ fef, float* __restrict__ out) {
  if (threadIdx.x == 0) terms_body(y, fef, out);
}
__global__ void __launch_bounds__(64) k_fid_terms_batch(const FidJob* __restrict__ jobs, int64_t n) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 64 + threadIdx.x;
  if (t < n) terms_body(jobs[t].y, jobs[t].fef, jobs[t].out);
}

// avg[c] = mean over t of terms[t * stride + c], c = 0, 1 (fp64 sums in a fixed order).
__global__ void __launch_bounds__(256) k_fid_average(const float* __restrict__ terms, int64_t n, int64_t stride,
                                                     float* __restrict__ avg) {
  __shared__ double red[2][4];
  double s0 = 0.0, s1 = 0.0;
  for (int64_t t = threadIdx.x; t < n; t += 256) {
    s0 += terms[t * stride];
    s1 += terms[t * stride + 1];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    s0 += __shfl_xor(s0, off);
    s1 += __shfl_xor(s1, off);
  }
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = s0;
    red[1][threadIdx.x >> 6] = s1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double a = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
    const double b = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
    avg[0] = static_cast<float>(a / static_cast<double>(n));
    avg[1] = static_cast<float>(b / static_cast<double>(n));
  }
}

struct FidWs {
  uint64_t* masks;
  float* y;
  float* fef;
  void* eval;
  size_t eval_bytes;
};

int fid_carve(const gnnshap_subgraph* sg, const gnnshap_gcn* m, void* base, FidWs* w, size_t* bytes) {
  size_t eb = 0;
  if (int st = gnnshap_eval_workspace(sg, m, 2, &eb)) return st;
  gnnshap::Carver c(base);
  const int64_t wpr = gnnshap::ceil_div(sg->num_edges, 64);
  w->masks = c.take<uint64_t>(2 * wpr);
  w->y = c.take<float>(2);
  w->fef = c.take<float>(2);
  w->eval = c.take<char>(eb);
  w->eval_bytes = eb;
  *bytes = c.bytes();
  return GNNSHAP_OK;
}

void set_players(FidJob* J, const float* phi, int64_t M, double sparsity, int64_t top_k) {
  const int64_t n_drop = static_cast<int64_t>(std::floor(sparsity * static_cast<double>(M)));
  J->phi = phi;
  J->M = M;
  J->n_keep = M - (n_drop < M ? n_drop : M);
  J->n_top = top_k < M ? top_k : M;
  J->wpr = gnnshap::ceil_div(M, 64);
}

// The workspace of a batch: the job tables, then a slice per target; targets
// that are not batched run one after the other in one slice of the largest.
struct FidBatchWs {
  bool batched = true;
  FidJob* fid = nullptr;
  gnnshap::EvalJob* eval = nullptr;
  char* shared = nullptr;
  size_t shared_bytes = 0;
  std::vector<FidWs> slice;
};

int fid_batch_carve(const gnnshap_subgraph* sgs, int64_t n, const gnnshap_gcn* m, gnnshap::Carver& c,
                    FidBatchWs* w) {
  w->batched = n <= 65535;
  for (int64_t t = 0; t < n && w->batched; ++t) w->batched = gnnshap::eval_batch_same(&sgs[t], m, 2);
  gnnshap::clear_error();
  if (!w->batched) {
    for (int64_t t = 0; t < n; ++t) {
      size_t b = 0;
      if (int st = gnnshap_fidelity_workspace(&sgs[t], m, &b)) return st;
      w->shared_bytes = std::max(w->shared_bytes, b);
    }
    w->shared = c.take<char>(w->shared_bytes);
    return GNNSHAP_OK;
  }
  w->fid = c.take<FidJob>(n);
  w->eval = c.take<gnnshap::EvalJob>(n);
  w->slice.resize(static_cast<size_t>(n));
  for (int64_t t = 0; t < n; ++t) {
    FidWs& s = w->slice[static_cast<size_t>(t)];
    s.masks = c.take<uint64_t>(2 * gnnshap::ceil_div(sgs[t].num_edges, 64));
    s.y = c.take<float>(2);
    s.fef = c.take<float>(2);
    s.eval_bytes = gnnshap::eval_slice_bytes(&sgs[t], m, 2);
    s.eval = c.take<char>(s.eval_bytes);
  }
  return GNNSHAP_OK;
}

int fid_batch_check(const gnnshap_subgraph* sgs, int64_t n, const gnnshap_gcn* m) {
  if (!sgs || !m || n < 1) return gnnshap::fail(GNNSHAP_EINVAL, "null argument or n < 1");
  for (int64_t t = 0; t < n; ++t)
    if (sgs[t].num_edges < 1)
      return gnnshap::fail(GNNSHAP_EINVAL, "the subgraph of target %lld has no players", static_cast<long long>(t));
  return GNNSHAP_OK;
}

}  // namespace

extern "C" int gnnshap_fidelity_batch_workspace(const gnnshap_subgraph* sgs, int64_t n, const gnnshap_gcn* m,
                                                size_t* bytes) {
  GS_TRY_BEGIN
  gnnshap::clear_error();
  if (!bytes) return gnnshap::fail(GNNSHAP_EINVAL, "bytes is NULL");
  if (int st = fid_batch_check(sgs, n, m)) return st;
  gnnshap::Carver c(nullptr);
  FidBatchWs w;
  if (int st = fid_batch_carve(sgs, n, m, c, &w)) return st;
  *bytes = c.bytes();
  return GNNSHAP_OK;
  GS_TRY_END
}

extern "C" int gnnshap_fidelity_batch(const gnnshap_subgraph* sgs, const float* const* phi, int64_t n,
                                      const gnnshap_gcn* m, const float* X, int32_t target_class, double sparsity,
                                      int64_t top_k, float* out, void* ws, size_t ws_bytes, void* stream) {
  GS_TRY_BEGIN
  gnnshap::clear_error();
  if (int st = fid_batch_check(sgs, n, m)) return st;
  if (!phi || !X || !out || !ws) return gnnshap::fail(GNNSHAP_EINVAL, "null argument");
  for (int64_t t = 0; t < n; ++t)
    if (!phi[t]) return gnnshap::fail(GNNSHAP_EINVAL, "null argument");
  if (!(sparsity >= 0.0 && sparsity <= 1.0)) return gnnshap::fail(GNNSHAP_EINVAL, "sparsity must be in [0, 1]");
  if (top_k < 0) return gnnshap::fail(GNNSHAP_EINVAL, "top_k must be >= 0");
  gnnshap::Carver need(nullptr);
  FidBatchWs w;
  if (int st = fid_batch_carve(sgs, n, m, need, &w)) return st;
  if (ws_bytes < need.bytes())
    return gnnshap::fail(GNNSHAP_ECAPACITY, "fidelity workspace needs %zu bytes", need.bytes());
  gnnshap::Carver cv(ws);
  w = FidBatchWs{};
  if (int st = fid_batch_carve(sgs, n, m, cv, &w)) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (!w.batched) {
    for (int64_t t = 0; t < n; ++t)
      if (int st = gnnshap_fidelity(&sgs[t], m, X, target_class, phi[t], sparsity, top_k, out + 3 * t, w.shared,
                                    w.shared_bytes, stream))
        return st;
    return GNNSHAP_OK;
  }
  if (target_class >= m->dims[2] || target_class < -1)
    return gnnshap::fail(GNNSHAP_EINVAL, "target_class out of range");
  // Under stream capture the jobs go by value in the launches, one target at a
  // time (as gnnshap_fidelity's do): the staging buffer of the job tables is
  // used again by later calls, so a replay would read another call's tables.
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &capture) != hipSuccess) {
    (void)hipGetLastError();
    capture = hipStreamCaptureStatusActive;
  }
  if (capture != hipStreamCaptureStatusNone) {
    for (int64_t t = 0; t < n; ++t) {
      const FidWs& sl = w.slice[static_cast<size_t>(t)];
      if (int e = gnnshap_fidelity_masks(phi[t], sgs[t].num_edges, sparsity, top_k, sl.masks, stream)) return e;
      if (int e = gnnshap_eval_coalitions(&sgs[t], m, X, target_class, sl.masks, 2,
                                          gnnshap::ceil_div(sgs[t].num_edges, 64), sl.y, sl.fef, nullptr, sl.eval,
                                          sl.eval_bytes, stream))
        return e;
      k_fid_terms<<<1, 64, 0, s>>>(sl.y, sl.fef, out + 3 * t);
      GS_LAUNCHED();
    }
    return GNNSHAP_OK;
  }
  // the job tables reach the front of the workspace in one copy
  char* const base = static_cast<char*>(ws);
  const size_t front = static_cast<size_t>(reinterpret_cast<char*>(w.eval + n) - base);
  gnnshap::HostStage* stage = gnnshap::host_stage(front, 0);
  if (!stage) return gnnshap::fail(GNNSHAP_EHIP, "page-locked staging allocation failed");
  FidJob* fj = reinterpret_cast<FidJob*>(stage->buf + (reinterpret_cast<char*>(w.fid) - base));
  gnnshap::EvalJob* ej = reinterpret_cast<gnnshap::EvalJob*>(stage->buf + (reinterpret_cast<char*>(w.eval) - base));
  int64_t max_nodes = 0, max_ndst = 0, max_n1 = 0, max_wpr = 0, rows_jobs = 0;
  size_t rows_lds = 0;
  for (int64_t t = 0; t < n; ++t) {
    const gnnshap_subgraph& g = sgs[t];
    if (!g.node_gid || !g.dst_ptr || !g.edge_src) return gnnshap::fail(GNNSHAP_EINVAL, "null subgraph arrays");
    const FidWs& sl = w.slice[static_cast<size_t>(t)];
    FidJob J{};
    set_players(&J, phi[t], g.num_edges, sparsity, top_k);
    J.masks = sl.masks;
    J.y = sl.y;
    J.fef = sl.fef;
    J.out = out + 3 * t;
    fj[t] = J;
    gnnshap::EvalJob E{};
    E.node_gid = g.node_gid;
    E.dst_ptr = g.dst_ptr;
    E.edge_src = g.edge_src;
    E.n_nodes = g.num_nodes;
    E.n_dst = g.num_dst;
    E.n1 = g.hop_ptr[2];
    E.M = g.num_edges;
    E.wpr = J.wpr;
    E.k = 2;
    E.masks = sl.masks;
    E.y = sl.y;
    E.fef = sl.fef;
    gnnshap::eval_carve_slice(sl.eval, &g, m, 2, &E);
    const size_t rl = gnnshap::eval_rows_lds(&g, m);
    E.rows_ok = rl > 0 ? 1 : 0;
    ej[t] = E;
    rows_jobs += E.rows_ok;
    rows_lds = std::max(rows_lds, rl);
    max_nodes = std::max(max_nodes, E.n_nodes);
    max_ndst = std::max(max_ndst, E.n_dst);
    max_n1 = std::max(max_n1, E.n1);
    max_wpr = std::max(max_wpr, E.wpr);
  }
  if (int st = gnnshap::copy_by_kernel(ws, stage->buf, front, s)) return st;
  GS_HIP(hipEventRecord(stage->done, s));
  stage->pending = true;
  {
    GS_TIMED("k_fid_masks_batch", s);
    k_fid_masks_batch<<<static_cast<unsigned>(n), kFidThreads, 0, s>>>(w.fid);
  }
  GS_LAUNCHED();
  const gnnshap::EvalModel md{m->XW1, m->b ? m->b[0] : nullptr, m->W[1], m->b ? m->b[1] : nullptr,
                              m->dims[1], m->dims[2], target_class};
  const int st = gnnshap::launch_eval_batch(w.eval, n, md, max_nodes, max_ndst, max_n1, max_wpr, 2, rows_jobs,
                                            rows_lds, s);
  if (st == GNNSHAP_EUNSUPPORTED) {
    // the largest shapes of the batch together need more LDS than a workgroup
    // has: one by one, each in its own slice
    gnnshap::clear_error();
    for (int64_t t = 0; t < n; ++t) {
      const FidWs& sl = w.slice[static_cast<size_t>(t)];
      if (int e = gnnshap_eval_coalitions(&sgs[t], m, X, target_class, sl.masks, 2, ej[t].wpr, sl.y, sl.fef, nullptr,
                                          sl.eval, sl.eval_bytes, stream))
        return e;
    }
  } else if (st != GNNSHAP_OK) {
    return st;
  }
  k_fid_terms_batch<<<static_cast<unsigned>(gnnshap::ceil_div(n, 64)), 64, 0, s>>>(w.fid, n);
  GS_LAUNCHED();
  return GNNSHAP_OK;
  GS_TRY_END
}

extern "C" int gnnshap_fidelity_workspace(const gnnshap_subgraph* sg, const gnnshap_gcn* m, size_t* bytes) {
  gnnshap::clear_error();
  if (!sg || !m || !bytes) return gnnshap::fail(GNNSHAP_EINVAL, "null argument");
  if (sg->num_edges < 1) return gnnshap::fail(GNNSHAP_EINVAL, "the subgraph has no players");
  FidWs w;
  return fid_carve(sg, m, nullptr, &w, bytes);
}

extern "C" int gnnshap_fidelity(const gnnshap_subgraph* sg, const gnnshap_gcn* m, const float* X,
                                int32_t target_class, const float* phi, double sparsity, int64_t top_k, float* out,
                                void* ws, size_t ws_bytes, void* stream) {
  GS_TRY_BEGIN
  gnnshap::clear_error();
  if (!sg || !m || !X || !phi || !out || !ws) return gnnshap::fail(GNNSHAP_EINVAL, "null argument");
  if (sg->num_edges < 1) return gnnshap::fail(GNNSHAP_EINVAL, "the subgraph has no players");
  if (!(sparsity >= 0.0 && sparsity <= 1.0)) return gnnshap::fail(GNNSHAP_EINVAL, "sparsity must be in [0, 1]");
  if (top_k < 0) return gnnshap::fail(GNNSHAP_EINVAL, "top_k must be >= 0");
  FidWs w;
  size_t need = 0;
  if (int st = fid_carve(sg, m, nullptr, &w, &need)) return st;
  if (ws_bytes < need) return gnnshap::fail(GNNSHAP_ECAPACITY, "fidelity workspace needs %zu bytes", need);
  if (int st = fid_carve(sg, m, ws, &w, &need)) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int64_t M = sg->num_edges;
  const int64_t wpr = gnnshap::ceil_div(M, 64);
  if (int st = gnnshap_fidelity_masks(phi, M, sparsity, top_k, w.masks, stream)) return st;
  if (int st = gnnshap_eval_coalitions(sg, m, X, target_class, w.masks, 2, wpr, w.y, w.fef, nullptr, w.eval,
                                       w.eval_bytes, stream))
    return st;
  k_fid_terms<<<1, 64, 0, s>>>(w.y, w.fef, out);
  GS_LAUNCHED();
  return GNNSHAP_OK;
  GS_TRY_END
}

extern "C" int gnnshap_fidelity_masks(const float* phi, int64_t M, double sparsity, int64_t top_k, uint64_t* masks,
                                      void* stream) {
  GS_TRY_BEGIN
  gnnshap::clear_error();
  if (!phi || !masks) return gnnshap::fail(GNNSHAP_EINVAL, "null argument");
  if (M < 1) return gnnshap::fail(GNNSHAP_EINVAL, "M must be >= 1");
  if (!(sparsity >= 0.0 && sparsity <= 1.0)) return gnnshap::fail(GNNSHAP_EINVAL, "sparsity must be in [0, 1]");
  if (top_k < 0) return gnnshap::fail(GNNSHAP_EINVAL, "top_k must be >= 0");
  FidJob J{};
  set_players(&J, phi, M, sparsity, top_k);
  J.masks = masks;
  {
    GS_TIMED("k_fid_masks", static_cast<hipStream_t>(stream));
    k_fid_masks<<<1, kFidThreads, 0, static_cast<hipStream_t>(stream)>>>(J);
  }
  GS_LAUNCHED();
  return GNNSHAP_OK;
  GS_TRY_END
}

extern "C" int gnnshap_fidelity_average(const float* terms, int64_t n, int64_t stride, float* avg, void* stream) {
  GS_TRY_BEGIN
  gnnshap::clear_error();
  if (!terms || !avg) return gnnshap::fail(GNNSHAP_EINVAL, "null argument");
  if (n < 1 || stride < 2) return gnnshap::fail(GNNSHAP_EINVAL, "need n >= 1 targets and stride >= 2");
  k_fid_average<<<1, 256, 0, static_cast<hipStream_t>(stream)>>>(terms, n, stride, avg);
  GS_LAUNCHED();
  return GNNSHAP_OK;
  GS_TRY_END
}
