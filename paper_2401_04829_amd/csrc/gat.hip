// Coalition values of a two-layer graph attention network (App. E of the
// GNNShap paper: the explainer treats the model as a black box and is shown
// on a GAT with 8 heads).
//
// A coalition keeps its edges and every self loop.  Layer 1 (H heads of
// width F, concatenated, then ELU) at node x of H_1 under coalition S:
//     out1_h[x] = sum_{u in N_S(x) + x} a_h(u -> x) z_h[u] / sum a_h(u -> x)
// with z = X W_1 and a_h(u -> x) = exp(LeakyReLU(s_h[u] + d_h[x]) - m_h[x]),
// s_h = a_src,h . z_h, d_h = a_dst,h . z_h.  The logits, and therefore the
// unnormalised weights a_h, do not depend on the coalition: they are
// computed once per target (m_h[x] is the largest logit among all of x's
// candidate edges, so every weight is at most 1); a coalition only decides
// which of them enter the sums, i.e. the softmax is renormalised over the
// present edges.  Layer 2 (one head of width C) is needed at the target v
// only, and only through the class explained: with u2_src = W_2 a_src,2 and
// u2_dst = W_2 a_dst,2, the layer-2 logit of edge x -> v is
// LeakyReLU(out1[x] . u2_src + out1[v] . u2_dst) and the class value of x is
// out1[x] . W_2[:, c]; their softmax is accumulated online (running maximum).
// Layer 1 is computed only at v and at the in-neighbours of v whose edge to
// v is present (the others do not reach v).  A coalition without an in-edge
// of v has the value f(empty) (Sec. 3.4.1 holds for any message-passing
// model).
#include <algorithm>
#include <cmath>

#include "batch.h"

namespace {

constexpr int kGatMaxFeat = 256;              // heads * head_dim
constexpr int kGatSlots = kGatMaxFeat / 64;   // features per lane
constexpr int kRowsWaves = 4;                 // coalitions per workgroup of the per-coalition kernel

using gnnshap::GatDev;
using gnnshap::GatJob;

__device__ __forceinline__ float leaky(float x, float slope) { return x > 0.f ? x : slope * x; }
__device__ __forceinline__ float elu(float x) { return x > 0.f ? x : expm1f(x); }

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}

// z1 rows of the subgraph's nodes and the per-head attention terms s (every
// node) and d (nodes of H_1).  Grid-stride over (node, feature) and (node, head).
__device__ __forceinline__ void gather_body(const GatDev& g) {
  const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = tid; i < g.n_nodes * g.nf; i += stride) {
    const int64_t u = i / g.nf, f = i % g.nf;
    g.z1[i] = g.XW1[static_cast<int64_t>(g.gid[u]) * g.nf + f];
  }
  for (int64_t i = tid; i < g.n_nodes * g.H; i += stride) {
    const int64_t u = i / g.H, h = i % g.H;
    const float* z = g.XW1 + static_cast<int64_t>(g.gid[u]) * g.nf + h * g.F;
    float s = 0.f, d = 0.f;
    for (int f = 0; f < g.F; ++f) {
      s += g.att_src1[h * g.F + f] * z[f];
      d += g.att_dst1[h * g.F + f] * z[f];
    }
    g.ss1[i] = s;
    if (u < g.n1) g.sd1[i] = d;
  }
}

// Unnormalised layer-1 weights of every candidate edge (players into H_1 and
// the self loops), shifted by each destination's largest logit; the layer-2
// attention vectors folded through W_2.
__device__ __forceinline__ void weights_body(const GatDev& g) {
  const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t i = tid; i < g.n1 * g.H; i += stride) {
    const int64_t x = i / g.H, h = i % g.H;
    const float d = g.sd1[i];
    const float lself = leaky(g.ss1[x * g.H + h] + d, g.slope);
    float m = lself;
    // eight edges at a time, their loads in flight together
    const int32_t p0 = g.dst_ptr[x], p1 = g.dst_ptr[x + 1];
    for (int32_t p = p0; p < p1; p += 8) {
      int64_t u[8];
      float l[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) u[q] = g.esrc[p + q < p1 ? p + q : p1 - 1];
#pragma unroll
      for (int q = 0; q < 8; ++q) l[q] = g.ss1[u[q] * g.H + h];
#pragma unroll
      for (int q = 0; q < 8; ++q) m = fmaxf(m, leaky(l[q] + d, g.slope));
    }
    for (int32_t p = p0; p < p1; p += 8) {
      int64_t u[8];
      float l[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) u[q] = g.esrc[p + q < p1 ? p + q : p1 - 1];
#pragma unroll
      for (int q = 0; q < 8; ++q) l[q] = g.ss1[u[q] * g.H + h];
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (p + q < p1) g.w[static_cast<int64_t>(p + q) * g.H + h] = expf(leaky(l[q] + d, g.slope) - m);
    }
    g.wself[i] = expf(lself - m);
  }
  for (int64_t f = tid; f < g.nf; f += stride) {
    float s = 0.f, d = 0.f;
    for (int c = 0; c < g.C; ++c) {
      s += g.W2[f * g.C + c] * g.att_src2[c];
      d += g.W2[f * g.C + c] * g.att_dst2[c];
    }
    g.u2s[f] = s;
    g.u2d[f] = d;
  }
}

// Layer-1 output of node x for this lane's features (f = lane + 64 i), under
// the coalition whose presence test is `present(p)`.
template <class Present>
__device__ __forceinline__ void layer1(const GatDev& g, int64_t x, Present present, float (&out)[kGatSlots]) {
  const int lane = threadIdx.x & 63;
  float num[kGatSlots], den[kGatSlots];
#pragma unroll
  for (int i = 0; i < kGatSlots; ++i) {
    const int f = lane + 64 * i;
    if (f < g.nf) {
      const float ws = g.wself[x * g.H + f / g.F];
      num[i] = ws * g.z1[x * g.nf + f];
      den[i] = ws;
    } else {
      num[i] = 0.f;
      den[i] = 1.f;
    }
  }
  const int32_t p0 = g.dst_ptr[x], p1 = g.dst_ptr[x + 1];
  for (int32_t p = p0; p < p1; ++p) {
    if (!present(p)) continue;
    const int64_t u = g.esrc[p];
#pragma unroll
    for (int i = 0; i < kGatSlots; ++i) {
      const int f = lane + 64 * i;
      if (f < g.nf) {
        const float wp = g.w[static_cast<int64_t>(p) * g.H + f / g.F];
        num[i] += wp * g.z1[u * g.nf + f];
        den[i] += wp;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < kGatSlots; ++i) {
    const int f = lane + 64 * i;
    out[i] = f < g.nf ? elu(num[i] / den[i] + g.b1[f]) : 0.f;
  }
}

// Dot product of a lane-distributed layer-1 output with a vector of nf (sum over the wave).
__device__ __forceinline__ float dot_nf(const GatDev& g, const float (&o)[kGatSlots], const float* v, int64_t stride) {
  const int lane = threadIdx.x & 63;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kGatSlots; ++i) {
    const int f = lane + 64 * i;
    if (f < g.nf) s += o[i] * v[f * stride];
  }
  return wave_sum_f(s);
}

// Layer-2 output at v for class c under a coalition (one wave): online
// softmax over the self loop and the present in-edges of v.
template <class Present>
__device__ float value_at_v(const GatDev& g, int32_t c, Present present) {
  float o[kGatSlots];
  layer1(g, 0, present, o);
  const float sdv = dot_nf(g, o, g.u2d, 1);
  float mx = leaky(dot_nf(g, o, g.u2s, 1) + sdv, g.slope);
  float sum = 1.f;
  float acc = dot_nf(g, o, g.W2 + c, g.C);
  for (int64_t e = 0; e < g.indeg_v; ++e) {
    if (!present(static_cast<int32_t>(e))) continue;
    const int64_t x = g.esrc[e];
    layer1(g, x, present, o);
    const float lx = leaky(dot_nf(g, o, g.u2s, 1) + sdv, g.slope);
    const float yx = dot_nf(g, o, g.W2 + c, g.C);
    if (lx > mx) {
      const float r = expf(mx - lx);
      sum = sum * r + 1.f;
      acc = acc * r + yx;
      mx = lx;
    } else {
      const float wx = expf(lx - mx);
      sum += wx;
      acc += wx * yx;
    }
  }
  return acc / sum + g.b2[c];
}

// f(empty) and f(E_c) for every class, then the explained class and
// f_empty_full.  One workgroup of 16 wavefronts per target: under E_c they
// share v's in-neighbours, each accumulating its own online softmax of their
// layer-1 rows; the layer-2 output of class c is then the softmax-weighted
// row times W_2[:, c] (one row sum instead of one pass over the neighbours
// per class: 89 us per Cora-shaped target before).
constexpr int kEndsWaves = 16;

__device__ __forceinline__ float pair_sum(float (&t)[kEndsWaves]) {
#pragma unroll
  for (int n = kEndsWaves / 2; n > 0; n >>= 1)
#pragma unroll
    for (int w = 0; w < n; ++w) t[w] += t[w + n];
  return t[0];
}

__device__ __forceinline__ void ends_body(const GatJob& J) {
  __shared__ float rows[kEndsWaves + 1][kGatMaxFeat];   // the wavefronts' sums; the last one: the row under the empty coalition
  __shared__ float mxs[kEndsWaves], sums[kEndsWaves];
  const GatDev& g = J.g;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  float o[kGatSlots], acc[kGatSlots];
  if (wv == 0) {
    layer1(g, 0, [](int32_t) { return false; }, o);
#pragma unroll
    for (int i = 0; i < kGatSlots; ++i)
      if (lane + 64 * i < g.nf) rows[kEndsWaves][lane + 64 * i] = o[i];
  }
  const auto all = [](int32_t) { return true; };
  layer1(g, 0, all, o);
  const float sdv = dot_nf(g, o, g.u2d, 1);
  float mx = -INFINITY, sum = 0.f;
  auto first = [&](float lx) {
    mx = lx;
    sum = 1.f;
#pragma unroll
    for (int i = 0; i < kGatSlots; ++i) acc[i] = o[i];
  };
#pragma unroll
  for (int i = 0; i < kGatSlots; ++i) acc[i] = 0.f;
  if (wv == 0) first(leaky(dot_nf(g, o, g.u2s, 1) + sdv, g.slope));
  for (int64_t e = wv; e < g.indeg_v; e += kEndsWaves) {
    layer1(g, g.esrc[e], all, o);
    const float lx = leaky(dot_nf(g, o, g.u2s, 1) + sdv, g.slope);
    if (sum == 0.f) {
      first(lx);
    } else if (lx > mx) {
      const float r = expf(mx - lx);
      sum = sum * r + 1.f;
#pragma unroll
      for (int i = 0; i < kGatSlots; ++i) acc[i] = acc[i] * r + o[i];
      mx = lx;
    } else {
      // (two logits of -inf without v among them: their weight is taken below)
      const float wx = wv > 0 && lx == -INFINITY && mx == -INFINITY ? 1.f : expf(lx - mx);
      sum += wx;
#pragma unroll
      for (int i = 0; i < kGatSlots; ++i) acc[i] += wx * o[i];
    }
  }
#pragma unroll
  for (int i = 0; i < kGatSlots; ++i)
    if (lane + 64 * i < g.nf) rows[wv][lane + 64 * i] = acc[i];
  if (lane == 0) {
    mxs[wv] = mx;
    sums[wv] = sum;
  }
  __syncthreads();
  // The wavefronts' sums at the largest logit of all.  As in the kernels of
  // the coalitions, one logit of +inf takes all the weight and a second one
  // leaves no number.
  float top = mxs[0];
  int infs = 0;
#pragma unroll
  for (int w = 0; w < kEndsWaves; ++w) {
    top = fmaxf(top, mxs[w]);
    infs += mxs[w] == INFINITY ? 1 : 0;
  }
  float scale[kEndsWaves], t[kEndsWaves];
#pragma unroll
  for (int w = 0; w < kEndsWaves; ++w) {
    // (a wavefront without neighbours has no sum)
    scale[w] = sums[w] == 0.f ? 0.f : mxs[w] == top && infs < 2 ? 1.f : expf(mxs[w] - top);
    t[w] = sums[w] * scale[w];
  }
  const float total = pair_sum(t);
#pragma unroll
  for (int i = 0; i < kGatSlots; ++i) {
    const int f = lane + 64 * i;
    acc[i] = o[i] = 0.f;
    if (f < g.nf) {
#pragma unroll
      for (int w = 0; w < kEndsWaves; ++w) t[w] = rows[w][f] * scale[w];
      acc[i] = pair_sum(t) / total;
      o[i] = rows[kEndsWaves][f];
    }
  }
  for (int32_t c = wv; c < g.C; c += kEndsWaves) {
    const float fe = dot_nf(g, o, g.W2 + c, g.C) + g.b2[c], ff = dot_nf(g, acc, g.W2 + c, g.C) + g.b2[c];
    if (lane == 0) {
      J.scratch[c] = fe;
      J.scratch[g.C + c] = ff;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t c = J.target_class;
    if (c < 0) {
      c = 0;
      for (int32_t i = 1; i < g.C; ++i)
        if (J.scratch[g.C + i] > J.scratch[g.C + c]) c = i;
    }
    *g.cls = c;
    J.fef[0] = J.scratch[c];
    J.fef[1] = J.scratch[g.C + c];
    if (J.class_out) *J.class_out = c;
  }
}

// Whether any in-edge of v is in a coalition.
__device__ __forceinline__ bool reaches_v(const GatDev& g, const uint64_t* row) {
  bool live = false;
  for (int64_t w = 0; w * 64 < g.indeg_v; ++w) {
    const int64_t n = g.indeg_v - w * 64;
    live |= (row[w] & (n >= 64 ? ~0ull : ((1ull << n) - 1ull))) != 0;
  }
  return live;
}

// y[b] for coalition b: one wave per coalition, features over the lanes (head
// widths that are no multiple of 16).
__device__ __forceinline__ void rows_body(const GatJob& J) {
  const GatDev& g = J.g;
  const int64_t b = static_cast<int64_t>(blockIdx.x) * kRowsWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (b >= J.k) return;
  const uint64_t* row = J.masks + b * J.wpr;
  auto present = [row](int32_t p) { return ((row[p >> 6] >> (p & 63)) & 1ull) != 0; };
  float v;
  if (!reaches_v(g, row)) v = J.fef[0];   // no in-edge of v: the target alone (Sec. 3.4.1)
  else v = value_at_v(g, *g.cls, present);
  if ((threadIdx.x & 63) == 0) J.y[b] = v;
}

// y[b] of 64 coalitions per workgroup, one per lane (head widths that are
// multiples of 16): wavefront w holds features 16 w .. 16 w + 15 of every
// lane's layer-1 row, which belong to one head.  An edge's weight and source
// features are the same for all lanes and stay in scalar registers, and its
// 17 multiply-adds run under the lanes whose coalition holds it, in edge
// order as above; so 64 coalitions share every load and the loop control,
// where one wavefront per coalition spent ~15 instructions per edge on one
// coalition.  Bound by VALU issue, most of it the ELU and the division of
// the rows.  40 Cora-shaped targets x 10,000 coalitions: 3.2 ms of kernel
// time one target after the other before, 0.76 ms for the larger group now
// (0.97 ms with the edges' values in vector registers).
constexpr int kSlice = 16;
constexpr int kEdges = 4;
constexpr int kMaxSlices = kGatMaxFeat / kSlice;

// Arrays that no wavefront of the kernel writes, read at addresses that are
// the same for all lanes: through the constant address space they are loaded
// by scalar loads, also behind barriers.
template <class T>
using Uniform = const __attribute__((address_space(4))) T*;
template <class T>
__device__ __forceinline__ Uniform<T> uniform(const T* p) {
  return (Uniform<T>)(reinterpret_cast<uintptr_t>(p));
}

// Sum of o[q] u(q) over a wavefront's 16 features, and a lane's sum over the
// wavefronts: pairs of features first, then pairs of sums, as deep as the tree
// over the lanes of a wavefront per coalition (a chain over the features and
// then the wavefronts put the values of 40 Cora-shaped targets 7.91e-8 off
// their 64-bit results instead of 7.64e-8).
template <class U>
__device__ __forceinline__ float dot_slice(const float (&o)[kSlice], U u) {
  float v[kSlice / 2];
#pragma unroll
  for (int q = 0; q < kSlice / 2; ++q) v[q] = fmaf(o[2 * q + 1], u(2 * q + 1), o[2 * q] * u(2 * q));
#pragma unroll
  for (int n = kSlice / 4; n > 0; n >>= 1)
#pragma unroll
    for (int q = 0; q < n; ++q) v[q] += v[q + n];
  return v[0];
}

__device__ __forceinline__ float sum_slices(const float (&part)[kMaxSlices][64], int slices, int lane) {
  constexpr int kHalf = kMaxSlices / 2;
  float v[kHalf];
#pragma unroll
  for (int w = 0; w < kHalf; ++w) {
    const float x = part[w < slices ? w : 0][lane];
    v[w] = w < slices ? x : 0.f;
  }
  if (slices > kHalf) {
#pragma unroll
    for (int w = 0; w < kHalf; ++w) {
      const float x = part[w + kHalf < slices ? w + kHalf : 0][lane];
      v[w] += w + kHalf < slices ? x : 0.f;
    }
  }
#pragma unroll
  for (int n = kHalf / 2; n > 0; n >>= 1)
#pragma unroll
    for (int w = 0; w < n; ++w) v[w] += v[w + n];
  return v[0];
}

__device__ __forceinline__ void rows_lanes_body(const GatJob& J) {
  __shared__ float part[2][2][kMaxSlices][64];
  const GatDev& g = J.g;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), slices = blockDim.x >> 6;
  const int64_t tile = blockIdx.x;
  if (tile * 64 >= J.k) return;
  const int64_t b = tile * 64 + lane;
  const uint64_t* row = J.masks + (b < J.k ? b : J.k - 1) * J.wpr;
  const bool live = reaches_v(g, row);
  const float f_empty = J.fef[0];
  if (!__any(live)) {
    if (wave == 0 && b < J.k) J.y[b] = f_empty;
    return;   // the same outcome in every wavefront
  }
  const int32_t c = *g.cls;
  const int f0 = wave * kSlice, h = f0 / g.F;
  const auto z1 = uniform(g.z1), w1 = uniform(g.w), wself = uniform(g.wself), b1 = uniform(g.b1), u2s = uniform(g.u2s),
             u2d = uniform(g.u2d), W2 = uniform(g.W2);
  const auto esrc = uniform(g.esrc), dst_ptr = uniform(g.dst_ptr);
  float mx = 0.f, sum = 0.f, acc = 0.f, sdv = 0.f;
  uint64_t word_e = 0;
  int buf = 0;   // the sums of one node are written while those of the node before are read
  for (int64_t i = -1; i < g.indeg_v; ++i) {   // v itself, then its in-neighbours
    bool on = live;
    int64_t x = 0;
    if (i >= 0) {
      if ((i & 63) == 0) word_e = row[i >> 6];
      on = live && ((word_e >> (i & 63)) & 1ull);
      if (!__any(on)) continue;
      x = esrc[i];
    }
    float num[kSlice];
    float den = wself[x * g.H + h];
    const auto z = z1 + x * g.nf + f0;
#pragma unroll
    for (int q = 0; q < kSlice; ++q) num[q] = den * z[q];
    const int32_t p0 = dst_ptr[x], p1 = dst_ptr[x + 1];
    uint64_t word = p0 < p1 ? row[p0 >> 6] : 0;
    // four edges at a time, so that their (scalar) loads overlap
    for (int32_t p = p0; p < p1; p += kEdges) {
      float wp[kEdges];
      Uniform<float> zu[kEdges];
#pragma unroll
      for (int k = 0; k < kEdges; ++k) {
        const int32_t pk = p + k < p1 ? p + k : p1 - 1;
        wp[k] = w1[static_cast<int64_t>(pk) * g.H + h];
        zu[k] = z1 + static_cast<int64_t>(esrc[pk]) * g.nf + f0;
      }
#pragma unroll
      for (int k = 0; k < kEdges; ++k) {
        if (p + k >= p1) break;
        if (((p + k) & 63) == 0) word = row[(p + k) >> 6];
        if (on && ((word >> ((p + k) & 63)) & 1ull)) {
          den += wp[k];
#pragma unroll
          for (int q = 0; q < kSlice; ++q) num[q] += wp[k] * zu[k][q];
        }
      }
    }
    float o[kSlice];
#pragma unroll
    for (int q = 0; q < kSlice; ++q) o[q] = elu(num[q] / den + b1[f0 + q]);
    buf ^= 1;
    part[buf][0][wave][lane] = dot_slice(o, [&](int q) { return u2s[f0 + q]; });
    part[buf][1][wave][lane] = dot_slice(o, [&](int q) { return W2[static_cast<int64_t>(f0 + q) * g.C + c]; });
    __syncthreads();
    float sl = 0.f, sy = 0.f;
    if (wave == 0) {
      sl = sum_slices(part[buf][0], slices, lane);
      sy = sum_slices(part[buf][1], slices, lane);
    }
    if (i < 0) {
      part[buf ^ 1][0][wave][lane] = dot_slice(o, [&](int q) { return u2d[f0 + q]; });
      __syncthreads();
      if (wave == 0) {
        sdv = sum_slices(part[buf ^ 1][0], slices, lane);
        mx = leaky(sl + sdv, g.slope);
        sum = 1.f;
        acc = sy;
      }
      __syncthreads();
    } else if (wave == 0 && on) {
      const float lx = leaky(sl + sdv, g.slope);
      if (lx > mx) {
        const float r = expf(mx - lx);
        sum = sum * r + 1.f;
        acc = acc * r + sy;
        mx = lx;
      } else {
        const float wx = expf(lx - mx);
        sum += wx;
        acc += wx * sy;
      }
    }
  }
  if (wave == 0 && b < J.k) J.y[b] = live ? acc / sum + g.b2[c] : f_empty;
}

// One target (its job by value) and a batch (job blockIdx.y of a table).
__global__ void __launch_bounds__(256) k_gat_gather(GatJob J) { gather_body(J.g); }
__global__ void __launch_bounds__(256) k_gat_gather_batch(const GatJob* __restrict__ jobs) { gather_body(jobs[blockIdx.y].g); }
__global__ void __launch_bounds__(256) k_gat_weights(GatJob J) { weights_body(J.g); }
__global__ void __launch_bounds__(256) k_gat_weights_batch(const GatJob* __restrict__ jobs) { weights_body(jobs[blockIdx.y].g); }
__global__ void __launch_bounds__(kEndsWaves * 64) k_gat_ends(GatJob J) { ends_body(J); }
__global__ void __launch_bounds__(kEndsWaves * 64) k_gat_ends_batch(const GatJob* __restrict__ jobs) { ends_body(jobs[blockIdx.y]); }
__global__ void __launch_bounds__(kRowsWaves * 64) k_gat_rows(GatJob J) { rows_body(J); }
__global__ void __launch_bounds__(kRowsWaves * 64) k_gat_rows_batch(const GatJob* __restrict__ jobs) { rows_body(jobs[blockIdx.y]); }
__global__ void __launch_bounds__(kMaxSlices * 64) k_gat_rows_lanes(GatJob J) { rows_lanes_body(J); }
__global__ void __launch_bounds__(kMaxSlices * 64) k_gat_rows_lanes_batch(const GatJob* __restrict__ jobs) { rows_lanes_body(jobs[blockIdx.y]); }

struct GatWs {
  float *z1, *ss1, *sd1, *w, *wself, *u2s, *u2d, *scratch;
  int32_t* cls;
};

GatWs gat_carve(gnnshap::Carver& c, const gnnshap_subgraph* sg, const gnnshap_gat* m) {
  const int64_t nf = static_cast<int64_t>(m->heads) * m->head_dim;
  GatWs w;
  w.z1 = c.take<float>(sg->num_nodes * nf);
  w.ss1 = c.take<float>(sg->num_nodes * m->heads);
  w.sd1 = c.take<float>(sg->num_dst * m->heads);
  w.w = c.take<float>(sg->num_edges * m->heads);
  w.wself = c.take<float>(sg->num_dst * m->heads);
  w.u2s = c.take<float>(nf);
  w.u2d = c.take<float>(nf);
  w.scratch = c.take<float>(2 * static_cast<int64_t>(m->num_classes));
  w.cls = c.take<int32_t>(1);
  return w;
}

int gat_check(const gnnshap_subgraph* sg, const gnnshap_gat* m) {
  if (!sg || !m) return gnnshap::fail(GNNSHAP_EINVAL, "null subgraph or model");
  if (sg->num_hops != 2) return gnnshap::fail(GNNSHAP_EINVAL, "the two-layer GAT needs a 2-hop subgraph");
  if (sg->num_edges < 1 || sg->num_dst < 1 || sg->num_nodes < sg->num_dst)
    return gnnshap::fail(GNNSHAP_EINVAL, "subgraph sizes are inconsistent");
  if (m->heads < 1 || m->head_dim < 1 || static_cast<int64_t>(m->heads) * m->head_dim > kGatMaxFeat)
    return gnnshap::fail(GNNSHAP_EINVAL, "heads * head_dim must be in [1, %d]", kGatMaxFeat);
  if (m->num_classes < 1 || m->num_classes > GNNSHAP_MAX_CLASSES)
    return gnnshap::fail(GNNSHAP_EINVAL, "num_classes out of range");
  if (!(m->negative_slope >= 0.0 && m->negative_slope < 1.0))
    return gnnshap::fail(GNNSHAP_EINVAL, "negative_slope must be in [0, 1)");
  if (!m->XW1 || !m->att_src1 || !m->att_dst1 || !m->W2 || !m->att_src2 || !m->att_dst2)
    return gnnshap::fail(GNNSHAP_EINVAL, "null model array");
  return GNNSHAP_OK;
}

}  // namespace

extern "C" int gnnshap_gat_eval_workspace(const gnnshap_subgraph* sg, const gnnshap_gat* m, int64_t k,
                                          size_t* bytes) {
  gnnshap::clear_error();
  if (!bytes || k < 1) return gnnshap::fail(GNNSHAP_EINVAL, "bad arguments");
  if (int st = gat_check(sg, m)) return st;
  gnnshap::Carver c(nullptr);
  gat_carve(c, sg, m);
  *bytes = c.bytes();
  return GNNSHAP_OK;
}

int gnnshap::gat_fill_job(const gnnshap_subgraph* sg, const gnnshap_gat* m, int32_t target_class,
                          const uint64_t* masks, int64_t k, int64_t words_per_row, float* y, float* f_empty_full,
                          int32_t* class_out, void* ws, size_t ws_bytes, GatJob* job) {
  if (int st = gat_check(sg, m)) return st;
  if (!masks || !y || !f_empty_full || !ws || k < 1) return gnnshap::fail(GNNSHAP_EINVAL, "null argument or k < 1");
  if (!sg->node_gid || !sg->dst_ptr || !sg->edge_src) return gnnshap::fail(GNNSHAP_EINVAL, "null subgraph arrays");
  if (words_per_row != gnnshap::ceil_div(sg->num_edges, 64))
    return gnnshap::fail(GNNSHAP_EINVAL, "words_per_row != ceil(M/64)");
  if (target_class < -1 || target_class >= m->num_classes)
    return gnnshap::fail(GNNSHAP_EINVAL, "target_class out of range");
  gnnshap::Carver need(nullptr);
  gat_carve(need, sg, m);
  if (ws_bytes < need.bytes()) return gnnshap::fail(GNNSHAP_ECAPACITY, "GAT workspace needs %zu bytes", need.bytes());
  if (!m->b1 || !m->b2) return gnnshap::fail(GNNSHAP_EINVAL, "the GAT needs both biases (zero arrays for none)");
  gnnshap::Carver cv(ws);
  const GatWs w = gat_carve(cv, sg, m);
  *job = GatJob{};
  GatDev& g = job->g;
  g.gid = sg->node_gid;
  g.dst_ptr = sg->dst_ptr;
  g.esrc = sg->edge_src;
  g.n_nodes = sg->num_nodes;
  g.n1 = sg->num_dst;
  g.M = sg->num_edges;
  // hop-1 nodes are exactly v's in-neighbours, so v has hop_ptr[2] - 1 players
  g.indeg_v = sg->hop_ptr[2] - sg->hop_ptr[1];
  g.H = m->heads;
  g.F = m->head_dim;
  g.nf = m->heads * m->head_dim;
  g.C = m->num_classes;
  g.XW1 = m->XW1;
  g.att_src1 = m->att_src1;
  g.att_dst1 = m->att_dst1;
  g.b1 = m->b1;
  g.W2 = m->W2;
  g.att_src2 = m->att_src2;
  g.att_dst2 = m->att_dst2;
  g.b2 = m->b2;
  g.slope = static_cast<float>(m->negative_slope);
  g.z1 = w.z1;
  g.ss1 = w.ss1;
  g.sd1 = w.sd1;
  g.w = w.w;
  g.wself = w.wself;
  g.u2s = w.u2s;
  g.u2d = w.u2d;
  g.cls = w.cls;
  job->masks = masks;
  job->k = k;
  job->wpr = words_per_row;
  job->fef = f_empty_full;
  job->y = y;
  job->class_out = class_out;
  job->scratch = w.scratch;
  job->target_class = target_class;
  return GNNSHAP_OK;
}

// Head widths that are multiples of 16 take the kernel with one coalition per
// lane, whose wavefronts hold 16 features of one head each.
static bool takes_lanes(const gnnshap_gat* m) { return m->head_dim % kSlice == 0; }

int gnnshap::launch_gat_batch(const GatJob* jobs, int64_t n, const gnnshap_gat* m, int64_t max_nodes, int64_t max_ndst,
                              int64_t max_k, hipStream_t s) {
  if (n < 1) return GNNSHAP_OK;
  const unsigned nn = static_cast<unsigned>(n);
  const int64_t nf = static_cast<int64_t>(m->heads) * m->head_dim;
  k_gat_gather_batch<<<dim3(grid_for(max_nodes * nf, 256, 1024), nn), 256, 0, s>>>(jobs);
  GS_LAUNCHED();
  k_gat_weights_batch<<<dim3(grid_for(std::max<int64_t>(max_ndst * m->heads, nf), 256, 256), nn), 256, 0, s>>>(jobs);
  GS_LAUNCHED();
  {
    GS_TIMED("k_gat_ends_batch", s);
    k_gat_ends_batch<<<dim3(1, nn), kEndsWaves * 64, 0, s>>>(jobs);
  }
  GS_LAUNCHED();
  {
    GS_TIMED("k_gat_rows_batch", s);
    if (takes_lanes(m))
      k_gat_rows_lanes_batch<<<dim3(static_cast<unsigned>(ceil_div(max_k, 64)), nn),
                               static_cast<unsigned>(nf / kSlice * 64), 0, s>>>(jobs);
    else
      k_gat_rows_batch<<<dim3(static_cast<unsigned>(ceil_div(max_k, kRowsWaves)), nn), kRowsWaves * 64, 0, s>>>(jobs);
  }
  GS_LAUNCHED();
  return GNNSHAP_OK;
}

extern "C" int gnnshap_gat_eval_coalitions(const gnnshap_subgraph* sg, const gnnshap_gat* m, int32_t target_class,
                                           const uint64_t* masks, int64_t k, int64_t words_per_row, float* y,
                                           float* f_empty_full, int32_t* class_out, void* ws, size_t ws_bytes,
                                           void* stream) {
  GS_TRY_BEGIN
  gnnshap::clear_error();
  GatJob J;
  if (int st = gnnshap::gat_fill_job(sg, m, target_class, masks, k, words_per_row, y, f_empty_full, class_out, ws,
                                     ws_bytes, &J))
    return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  k_gat_gather<<<gnnshap::grid_for(sg->num_nodes * J.g.nf, 256, 1024), 256, 0, s>>>(J);
  GS_LAUNCHED();
  k_gat_weights<<<gnnshap::grid_for(std::max<int64_t>(sg->num_dst * J.g.H, J.g.nf), 256, 256), 256, 0, s>>>(J);
  GS_LAUNCHED();
  {
    GS_TIMED("k_gat_ends", s);
    k_gat_ends<<<1, kEndsWaves * 64, 0, s>>>(J);
  }
  GS_LAUNCHED();
  {
    GS_TIMED("k_gat_rows", s);
    if (takes_lanes(m))
      k_gat_rows_lanes<<<static_cast<unsigned>(gnnshap::ceil_div(k, 64)), static_cast<unsigned>(J.g.nf / kSlice * 64),
                         0, s>>>(J);
    else
      k_gat_rows<<<static_cast<unsigned>(gnnshap::ceil_div(k, kRowsWaves)), kRowsWaves * 64, 0, s>>>(J);
  }
  GS_LAUNCHED();
  return GNNSHAP_OK;
  GS_TRY_END
}
