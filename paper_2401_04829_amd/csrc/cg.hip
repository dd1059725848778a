// Matrix-free conjugate gradients for the projected Kernel-SHAP normal
// equations (Sec. 3.5 of the GNNShap paper: above 5000 players the regression
// is fitted iteratively rather than by a direct solve).
//
// Unknown psi in 1-perp, phi = Delta/M + psi.  With R the random
// representative rows (each stands for itself and its complement) and P the
// centring projector, the operator on 1-perp is
//     A v = alpha v + 2 w_r P R^T (R v),
// alpha collecting the enumerated classes (their projected Gram is a multiple
// of P).  No Gram matrix is formed: every iteration applies R and R^T to the
// residual straight from the packed bits.
//
// The recurrences are those of Chronopoulos and Gear's conjugate gradients
// (SIAM J. Sci. Stat. Comput. 1989), which apply A to the residual r and
// carry s = A p along: with w = A r, gamma = r.r and delta = r.w,
//     beta = gamma / gamma_prev, a = gamma / (delta - beta gamma / a_prev),
//     p = r + beta p, s = w + beta s, x += a p, r -= a s.
// Every vector a pass reads was finished by an earlier kernel.  delta needs no
// extra reduction: r.A r = alpha |r|^2 + 2 w_r |R r|^2 for r in 1-perp.
//
// Products with the bits run on the matrix cores, exactly.  A vector v is
// held as integers rint(|v_j| 2^e) < 2^62 (e from a bound on |v|), split into 16
// base-16 digits with the sign of v_j.  A digit is exact in fp6 (e2m3 holds
// 0..15 eighths), a mask bit left in place in its nibble is an fp4 number
// (0001 = 0.5, 0010 = 1.0; e2m1), so v_mfma_f32_16x16x128_f8f6f4 contracts
// 16 bit rows x 128 entries with the 16 digits in one instruction: every
// product is a whole number of eighths and every sum stays below 2^24 of
// them, so fp32 accumulation loses nothing (segments of kSegGroups groups per
// wavefront keep it so for any number of rows).  The digit sums are combined in fp64.
// What rounds is the integer, by 2^-63 of the bound, and the last 16-term fp64
// combination, where a direct sum has thousands of fp64 additions; and the
// result does not depend on how the work is split over wavefronts.  The bounds
// are sqrt(M) |r| for u = R r (Cauchy-Schwarz), and for the new r the largest
// old |r| plus the step times what |R^T u| <= sqrt(kr) |u| allows; nothing
// bounds how far above the largest entry they lie.  In a model of the iteration
// (64 to 6,000 players, 9,700 to 95,840 rows) it was a factor of 2^2 to 2^5 for
// u and about sqrt(kr), 2^7 to 2^9, for r: up to 2^9 the largest entries keep
// all 53 bits of their fp64 value.
//
// Rows of small coalitions are mostly zero bits: the random rows whose size
// is at most M / kSparseDiv (the first ones: the plan orders random classes
// by ascending size), in whole blocks of 64 rows, are kept as lists of their
// players instead (sparse rows), built once per solve from the bits: for pass
// A padded to the largest row of their block (its rows' sizes are nearly
// equal), entry i of the 64 rows contiguous, so a workgroup reads a block's
// lists and the entries of r they name without following pointers; for pass
// B by player, in ascending row order, eight lanes summing one player's list.
//
// Per iteration t, two launches (three where pass B's products are split over
// parts of the rows, whose digit sums pass B adds: exact, so the same bits):
//   pass A   stopping test on gamma_t; u = R r of the bit rows (a workgroup
//            per 64 rows, its wavefronts sharing the players), the digits of
//            u, partial |u|^2 and |m|.u; in workgroups of their own the same
//            for the sparse rows (u itself, no digits);
//   pass B   a workgroup per 64 players, its wavefronts sharing the bit rows:
//            R^T u plus the sparse rows' R_s^T u, then w = alpha r +
//            2 w_r (R^T u - mean), the scalars, the vector steps of these
//            players, the digits of the new r and the partial sums of the
//            new gamma.
// Vectors and sums of products are fp64; partial sums are kept per 64 rows
// or players and reduced in a fixed order, so repeated solves give the same
// bits, alone or in a group.  The iteration stops when
// |r| <= kTol |r_0| or after kMaxIt iterations; the host queues iterations in
// chunks and checks a flag the device writes to mapped host memory, so at
// most one chunk runs idle.
//
// What bounds an iteration: the mask words are read once per pass (52 MB at
// 18,001 players x 100,000 coalitions, 17-23 us a pass: 5-7 TB/s of words
// that stay in the 256 MB last-level cache while streaming) plus ~6 us of
// fixed latency per launch (the launch, a chain of dependent loads behind
// the kernel boundary, the reduction over the wavefronts).  Against fp64
// subset-sum tables in LDS (16 reads of 512 B per 64-bit word and wavefront,
// near the LDS limit) and four launches, per iteration of a single solve:
// 10,793 players x 60,000 coalitions 39 -> 25 us, 18,001 x 100,000 63 -> 41,
// 30,000 x 100,000 81 -> 51.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <vector>

#include "cg.h"

namespace {

// Relative residual at which the iteration stops.  On the Reddit-shaped
// targets (10,793-30,000 players, 100,000 coalitions) phi then differs from
// a solve to 1e-10 by at most 4.6e-6 of max|phi| (1e-7: 4.9e-7; 1e-8:
// 6e-8), far inside the 1e-3 bar that the solution is held to, at 3/4 of
// the iterations that 1e-8 takes.
constexpr double kTol = 1e-6;
constexpr int64_t kMaxIt = 4000;
constexpr int64_t kChunk = 8;        // iterations queued between stopping checks
constexpr int kWaves = 8;            // waves per workgroup of both passes
constexpr int kThreads = kWaves * 64;
constexpr int kSegGroups = 512;      // K groups (256 entries) a wavefront accumulates in fp32 before an fp64 sum
// a segment's sum over its wavefronts, in eighths, is exact in fp32
static_assert(int64_t(kSegGroups) * kWaves * 256 * 15 < (int64_t(1) << 24));
constexpr int64_t kSparseDiv = 128;   // sparse rows: coalition size at most M / kSparseDiv
constexpr int kFixedBits = 62;        // |fixed-point entries| stay below 2^62
constexpr uint64_t kSign = uint64_t(1) << 63;

struct Args {
  const uint64_t* blocked;   // the random rows in row blocks (pass A)
  const uint64_t* T;         // the random rows transposed (pass B)
  const int32_t* sz;
  int64_t M, wpr, kr, nrb;
  int64_t rs, rbd0, nbits;   // sparse rows, their blocks (the first bit block), bit blocks
  const int64_t* ell_ptr;
  const int32_t* ell_idx;
  const int64_t* csc_ptr;
  const int32_t* csc_row;
  double alpha, wr2, tol2;
  int64_t maxit;
  double* x;
  double* r;       // M + 1 (r[M] = 0: the lists' padding)
  double* p;
  double* s;
  double* us;      // rs: R r of the sparse rows
  char* rdig;      // digits of r (digit_bytes(wpr))
  char* udig;      // digits of R r of the bit rows (digit_bytes(nbits))
  double* uu;      // 2 x (2 nbits + rbd0): partial |u|^2 and |m|.u
  double* rr;      // 3 x 2 wpr: partial r.r of iterations t mod 3
  double* mx;      // 2 x 2 x 2 wpr: largest |r| and |s| per 32 players, by iteration parity
  double* hist;    // step length of even and odd iterations
  int32_t* ex;     // fixed-point exponents: r of even and odd iterations, u
  gnnshap::CgState* st;
  int32_t* host_flag;  // mapped host memory: [0] done, [1] iterations
  double* qd;          // parts x the digit sums of R^T u (parts > 1)
  int64_t parts;       // parts of the bit rows in pass B's products
};

// The members of one launch of a pass: member m owns workgroups
// [blk[m], blk[m + 1]) of the flat grid and runs iteration t[m].
struct GroupArgs {
  Args a[gnnshap::kCgGroupMax];
  int64_t t[gnnshap::kCgGroupMax];
  uint32_t blk[gnnshap::kCgGroupMax + 1];
  int32_t n;
};

// The member of this workgroup and the workgroup's index within it.
__device__ __forceinline__ int member_of(const GroupArgs& g, int64_t& bid) {
  const uint32_t b = blockIdx.x;
  int m = 0;
  while (m + 1 < g.n && b >= g.blk[m + 1]) ++m;
  bid = static_cast<int64_t>(b - g.blk[m]);
  return m;
}

// v of the lane that DPP control CTRL (within rows of 16 lanes) selects.
template <int CTRL>
__device__ __forceinline__ double row_move(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, true));
}

// Sum over rows of 16 lanes, in every lane: lanes xor 1, xor 2 (quad_perm),
// then the mirrored half row and the mirrored row, whose sums the earlier
// steps have made equal within their quads and halves.
__device__ __forceinline__ double row_sum_d(double v) {
  v += row_move<0xB1>(v);
  v += row_move<0x4E>(v);
  v += row_move<0x141>(v);
  return v + row_move<0x140>(v);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum and maximum over each half wavefront, in its first lane.
__device__ __forceinline__ double half_sum_d(double v) {
  v = row_sum_d(v);
  return v + __shfl_xor(v, 16);
}

__device__ __forceinline__ double half_max_d(double v) {
  v = fmax(v, row_move<0xB1>(v));
  v = fmax(v, row_move<0x4E>(v));
  v = fmax(v, row_move<0x141>(v));
  v = fmax(v, row_move<0x140>(v));
  return fmax(v, __shfl_xor(v, 16));
}

// Sum and maximum over a wavefront, in every lane.
__device__ __forceinline__ double wave_sum_d(double v) {
  v = row_sum_d(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

__device__ __forceinline__ double wave_max_d(double v) {
  v = fmax(v, row_move<0xB1>(v));
  v = fmax(v, row_move<0x4E>(v));
  v = fmax(v, row_move<0x141>(v));
  v = fmax(v, row_move<0x140>(v));
  return fmax(fmax(lane_value(v, 0), lane_value(v, 16)), fmax(lane_value(v, 32), lane_value(v, 48)));
}

// Sum (or maximum) of n values a[stride * i] by one whole wave in a fixed
// order, sixteen loads in flight; every lane gets the same bits.
template <bool MAX = false>
__device__ __forceinline__ double wave_fixed(const double* __restrict__ a, int64_t n, int64_t stride = 1) {
  const int lane = threadIdx.x & 63;
  double s = 0.0;
  for (int64_t i = 0; i < n; i += 1024) {
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int64_t k = i + 64 * q + lane;
      v[q] = k < n ? a[k * stride] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) s = MAX ? fmax(s, v[q]) : s + v[q];
  }
  return MAX ? wave_max_d(s) : wave_sum_d(s);
}

// ---- fixed-point vectors and their digits ---------------------------------------------------

// Exponent e with bound * 2^e < 2^kFixedBits, for a finite bound >= every |v_j|.
__device__ __forceinline__ int fixed_exponent(double bound) {
  const int lg = static_cast<int>(__double_as_longlong(bound > 1e-270 ? bound : 1e-270) >> 52) - 1023;
  const int e = kFixedBits - 1 - lg;
  return e > 960 ? 960 : (e < -900 ? -900 : e);
}

// rint(|v| 2^e) with the sign of v in bit 63.
__device__ __forceinline__ uint64_t to_fixed(double v, int e) {
  const double m = __builtin_rint(__builtin_ldexp(__builtin_fabs(v), e));
  return static_cast<uint64_t>(m < 4.6e18 ? m : 4.6e18) | (v < 0.0 ? kSign : 0);
}

// A digit array holds, for every group of 256 entries (four 64-entry blocks)
// and half h of its blocks (a unit: 32 entries), one MFMA operand: lane g * 16 + d has digit d of
// the 32 entries h of block g as 32 fp6 numbers (24 bytes), the first 16
// bytes of the 64 lanes first, then their last 8.  Operand element 8 t + i is
// entry 4 i + t of the 32: the order in which the bits of a 32-bit mask word,
// taken as w & 0x11111111, w & 0x22222222 and the same of w >> 2, fill an fp4
// operand.  Bits taken as 0001 weigh 0.5, as 0010 1.0, so their digits are
// stored as quarters and eighths: every product is an eighth.
constexpr int64_t kOperand = 1536;
constexpr int64_t digit_bytes(int64_t nblocks) { return (nblocks + 3) / 4 * 2 * kOperand; }

// Thread (d, t) = (q / 4 % 16, q % 4), q < 64: the eight elements 8 t .. 8 t +
// 7 (48 bits) of digit d of unit `u` (half u % 2 of block u / 2) from its 32
// fixed-point entries.
__device__ __forceinline__ void store_digits(const uint64_t* fixed, int q, int64_t u, char* dig) {
  const int t = q & 3, d = q >> 2;
  uint64_t bits = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint64_t v = fixed[4 * i + t];
    const uint32_t n = static_cast<uint32_t>((v & ~kSign) >> (4 * d)) & 15u;
    const uint32_t mag = (t & 1) ? n : n + (n < 8u ? n : 8u);   // e2m3 codes of n / 8 and n / 4
    bits |= static_cast<uint64_t>(mag | static_cast<uint32_t>(v >> 63) << 5) << (6 * i);
  }
  char* op = dig + ((u >> 3) * 2 + (u & 1)) * kOperand;
  const int lane = static_cast<int>((u >> 1) & 3) * 16 + d;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int hw = 3 * t + k;   // halfword of the lane's 24 bytes
    char* at = hw < 8 ? op + lane * 16 + 2 * hw : op + 1024 + lane * 8 + 2 * (hw - 8);
    *reinterpret_cast<uint16_t*>(at) = static_cast<uint16_t>(bits >> (16 * k));
  }
}

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

// The digit operand of half h of group q.
__device__ __forceinline__ v8i load_operand(const char* __restrict__ dig, int q, int h) {
  const char* op = dig + (static_cast<int64_t>(q) * 2 + h) * kOperand;
  const int lane = threadIdx.x & 63;
  const v4i lo = *reinterpret_cast<const v4i*>(op + lane * 16);
  const v2i hi = *reinterpret_cast<const v2i*>(op + 1024 + lane * 8);
  return v8i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, 0, 0};
}

// acc += the bits of 32-bit mask words m times the digit operand b.
__device__ __forceinline__ v4f mma_half(uint32_t m, v8i b, v4f acc) {
  const uint32_t m2 = m >> 2;
  const v8i a = {static_cast<int>(m & 0x11111111u), static_cast<int>(m & 0x22222222u),
                 static_cast<int>(m2 & 0x11111111u), static_cast<int>(m2 & 0x22222222u), 0, 0, 0, 0};
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, acc, 4, 2, 0, 0, 0, 0);
}

// Blocks of 64 bit rows per part of pass B's products, whole groups of four.
__host__ __device__ __forceinline__ int64_t part_blocks(int64_t nbits, int64_t parts) {
  return ((nbits + 3) / 4 + parts - 1) / parts * 4;
}

// A workgroup's product of 16 TW bit rows (or players' columns) with the
// digits in dig, over nk 64-entry blocks: TW tiles of 16, tile t's words of
// block k at src[base[t] + 64 k + lane % 16].  Its wavefronts take groups of
// four blocks in turn; block g of a group is read by lanes 16 g .. (beyond nk
// the last one, whose digits are zero).
template <int TW>
struct BitProducts {
  // the registers of one group: words of the tiles, digits of both halves
  struct Stage {
    uint64_t w[TW];
    v8i b0, b1;
  };
  const char* src[TW];
  const char* dig;
  int nk;
  Stage s;   // the next group

  // Tiles t0 .. t0 + TW - 1 (beyond nt the last one, whose results are not
  // used) of `words`: blocks of four tiles, `len` 64-word blocks of entries
  // each, of which `first` .. first + nkb - 1 are multiplied.
  __device__ __forceinline__ void set(const uint64_t* words, int64_t first, int64_t t0, int64_t nt, int64_t len,
                                      int64_t nkb, const char* digits) {
    nk = static_cast<int>(nkb);
    dig = digits;
#pragma unroll
    for (int t = 0; t < TW; ++t) {
      const int64_t g = t0 + t < nt ? t0 + t : nt - 1;
      src[t] = reinterpret_cast<const char*>(words + ((g >> 2) * len + first) * 64 + (g & 3) * 16);
    }
  }

  __device__ __forceinline__ void load(int q) {
    const int lane = threadIdx.x & 63;
    const uint32_t at = static_cast<uint32_t>(min(4 * q + (lane >> 4), nk - 1)) * 512u + (lane & 15) * 8u;
#pragma unroll
    for (int t = 0; t < TW; ++t) s.w[t] = *reinterpret_cast<const uint64_t*>(src[t] + at);
    s.b0 = load_operand(dig, q, 0);
    s.b1 = load_operand(dig, q, 1);
  }

  __device__ __forceinline__ void multiply(v4f (&a)[TW]) const {
#pragma unroll
    for (int t = 0; t < TW; ++t) a[t] = mma_half(static_cast<uint32_t>(s.w[t]), s.b0, a[t]);
#pragma unroll
    for (int t = 0; t < TW; ++t) a[t] = mma_half(static_cast<uint32_t>(s.w[t] >> 32), s.b1, a[t]);
  }

  // this wavefront's first group, so that its loads run under whatever comes before sums()
  __device__ __forceinline__ void start(int wave) { load(min(wave, (nk + 3) / 4 - 1)); }

  // row[c] (wavefronts 0 .. TW - 1), lane 16 g + d: the sum of digit d over
  // row 16 wave + 4 g + c, in eighths: a whole number, exact.  The wavefronts'
  // sums are added (whole eighths).  buf: kWaves * TW * 256 floats.  Every
  // thread calls it; it ends behind a barrier that covers all LDS writes
  // before it.
  __device__ __forceinline__ void sums(int wave, float* buf, double (&row)[4]) {
    const int lane = threadIdx.x & 63;
    const int nq = (nk + 3) / 4;
    row[0] = row[1] = row[2] = row[3] = 0.0;
    for (int seg = 0; seg < nq; seg += kSegGroups * kWaves) {
      const int end = min(seg + kSegGroups * kWaves, nq);
      v4f a[TW] = {};
      int q = seg + wave;
      if (seg > 0) load(min(q, end - 1));
      // one group in registers: the next one is loaded into them as soon as
      // they are multiplied, and the other wavefronts of the CU (three
      // workgroups fit) multiply meanwhile; two groups in flight with half
      // the workgroups per CU measured the same
      for (; q < end; q += kWaves) {
        multiply(a);
        __builtin_amdgcn_sched_barrier(0);
        load(min(q + kWaves, end - 1));
      }
      if (seg > 0) __syncthreads();
      v4f* out = reinterpret_cast<v4f*>(buf) + wave * TW * 64 + lane;
#pragma unroll
      for (int t = 0; t < TW; ++t) out[64 * t] = a[t];
      __syncthreads();
      if (wave < TW) {
        const v4f* in = reinterpret_cast<const v4f*>(buf) + wave * 64 + lane;
        v4f sum = in[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) sum += in[w * TW * 64];
#pragma unroll
        for (int c = 0; c < 4; ++c) row[c] += static_cast<double>(sum[c]);
      }
    }
  }
};

// 2^-e times the product of row 4 (lane / 16) + c from its digits' sums, in all
// 16 lanes of a row of lanes: lane 16 g + d holds digit d, times 16^d (and 8:
// the sums are in eighths), then over the digits in fp64.
__device__ __forceinline__ void combine_digits(double (&row)[4], int e) {
  const double weight = __longlong_as_double(static_cast<long long>(1023 + 4 * (threadIdx.x & 15) + 3) << 52);
#pragma unroll
  for (int c = 0; c < 4; ++c) row[c] = __builtin_ldexp(row_sum_d(row[c] * weight), -e);
}

// The value of lane 16 g + d, d < 4: row[d].
__device__ __forceinline__ double pick_row(const double (&row)[4], int lane) {
  const double lo = (lane & 1) ? row[1] : row[0], hi = (lane & 1) ? row[3] : row[2];
  return (lane & 2) ? hi : lo;
}

// r = dv - mean(dv), x = p = s = 0, partial gamma_0 and largest |r| per 32
// players; digit arrays cleared; sizes of the random rows.
// Grid: ceil(wpr / 4) workgroups of 256.
__global__ void __launch_bounds__(256) k_cg_init(Args a, const double* __restrict__ dv,
                                                 const double* __restrict__ bsum, int64_t nb,
                                                 const gnnshap_class* __restrict__ cls, int64_t ncls, int64_t rb0,
                                                 int32_t* sz) {
  __shared__ double mean;
  if (threadIdx.x == 0) {
    double sm = 0.0;
    for (int64_t i = 0; i < nb; ++i) sm += bsum[i];
    mean = sm / static_cast<double>(a.M);
  }
  __syncthreads();
  const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const double rj = j < a.M ? dv[j] - mean : 0.0;
  if (j < a.M) {
    a.r[j] = rj;
    a.x[j] = 0.0;
    a.p[j] = 0.0;
    a.s[j] = 0.0;
  }
  const double r2 = half_sum_d(rj * rj), rm = half_max_d(__builtin_fabs(rj));
  if ((threadIdx.x & 31) == 0 && j < a.wpr * 64) {
    a.rr[j / 32] = r2;   // gamma_0: slot 0
    a.mx[j / 32] = rm;
    a.mx[2 * a.wpr + j / 32] = 0.0;
  }
  if (j == 0) {
    a.r[a.M] = 0.0;
    a.st->last = INT32_MAX;
    a.st->iters = 0;
    a.st->status = 0;
  }
  const int64_t stride = static_cast<int64_t>(gridDim.x) * 256;
  const uint4 zero = {0, 0, 0, 0};
  for (int64_t i = j; i < digit_bytes(a.wpr) / 16; i += stride) reinterpret_cast<uint4*>(a.rdig)[i] = zero;
  for (int64_t i = j; i < digit_bytes(a.nbits) / 16; i += stride) reinterpret_cast<uint4*>(a.udig)[i] = zero;
  // row sizes: class of row rb0 + b by binary search over row_begin
  for (int64_t b = j; b < a.kr; b += stride) {
    const int64_t row = rb0 + b;
    int64_t lo = 0, hi = ncls - 1;
    while (lo < hi) {
      const int64_t mid = (lo + hi + 1) >> 1;
      if (cls[mid].row_begin <= row) lo = mid; else hi = mid - 1;
    }
    sz[b] = cls[lo].size;
  }
}

// The digits of r_0, one workgroup per 64 players.
__global__ void __launch_bounds__(128) k_cg_digits(Args a) {
  __shared__ uint64_t fixed[64];
  const int64_t w = blockIdx.x, j = w * 64 + threadIdx.x;
  const int e = fixed_exponent(wave_fixed<true>(a.mx, 2 * a.wpr));
  if (threadIdx.x < 64) fixed[threadIdx.x] = to_fixed(j < a.M ? a.r[j] : 0.0, e);
  __syncthreads();
  store_digits(fixed + 32 * (threadIdx.x >> 6), threadIdx.x & 63, 2 * w + (threadIdx.x >> 6), a.rdig);
  if (w == 0 && threadIdx.x == 0) a.ex[0] = e;
}

// Stopping test of iteration t on g = gamma_t, by one thread; records the stop.
__device__ __forceinline__ void cg_stop(const Args& a, int64_t t, double g) {
  const double g0 = t == 0 ? g : a.st->rr0;
  const bool bad = !(g == g) || g > 1e300;
  const bool conv = !bad && g <= a.tol2 * g0;
  if (conv || bad || t >= a.maxit) {
    a.st->last = static_cast<int32_t>(t) - 1;
    a.st->iters = static_cast<int32_t>(t);
    a.st->status = conv ? 0 : (bad ? 2 : 1);
    __hip_atomic_store(a.host_flag + 1, static_cast<int32_t>(t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(a.host_flag, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  } else if (t == 0) {
    a.st->rr0 = g;
  }
}

// Tiles of 16 rows (pass A) or players (pass B) per workgroup.  Per group of
// 256 entries a wavefront loads 512 bytes of bits per tile and 3 KiB of
// digits, through a path of 64 bytes per clock and CU that bounds the loop:
// more tiles use each digit operand more often, fewer give more workgroups.
// The launch takes the number (4 or 6) that leaves the busiest CU the least
// to load (18,001 players, pass B: 4 tiles are 282 workgroups, two on 26 of
// the 256 CUs; 6 tiles 188).  2 tiles were slower throughout, 8 need more
// registers than three workgroups per CU leave.  The results do not depend on it.
// Pass A.  Workgroup x < nxa: u = R r of bit rows 16 TW x .., the digits of
// their u, partial |u|^2 and |m|.u per 32 rows; workgroup 0 also takes the
// stopping test (the others' results are not read after a stop).  Workgroup
// nxa + x: u_b of the 64 sparse rows of block x, lane = row, the wavefronts
// sharing the entries of their lists; the block's partial sums.
template <int TW>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(6))) k_cg_pass_a(GroupArgs g) {
  __shared__ alignas(16) float buf[kWaves * TW * 256];
  __shared__ uint64_t fixed[16 * TW];
  __shared__ double red[2 * kWaves];
  __shared__ double gamma;
  int64_t bid;
  const int m = member_of(g, bid);
  const Args& a = g.a[m];
  const int64_t t = g.t[m];
  // workgroup 0 may set this while others start: a wavefront that sees it ends
  // (barriers wait for the wavefronts that are left), the rest computes values
  // that nobody reads
  if (a.st->last < static_cast<int32_t>(t)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t nx = std::max<int64_t>((4 * a.nbits + TW - 1) / TW, 1);
  if (bid >= nx) {                  // sparse rows
    const int64_t x = bid - nx;
    const int64_t e0 = a.ell_ptr[x];
    const int n = static_cast<int>(a.ell_ptr[x + 1] - e0);   // entries per row
    const int i1 = n * (wave + 1) / kWaves;
    const int32_t* __restrict__ idx = a.ell_idx + e0 * 64 + lane;
    const double* __restrict__ r = a.r;
    const double size = static_cast<double>(a.sz[x * 64 + lane]);
    double v = 0.0;
    for (int i = n * wave / kWaves; i < i1; i += 8) {
      int32_t p[8];
      double e[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) p[k] = i + k < i1 ? idx[(i + k) * 64] : static_cast<int32_t>(a.M);
#pragma unroll
      for (int k = 0; k < 8; ++k) e[k] = r[p[k]];
#pragma unroll
      for (int k = 0; k < 8; ++k) v += e[k];
    }
    double* part = reinterpret_cast<double*>(buf);
    part[wave * 64 + lane] = v;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int w = 1; w < kWaves; ++w) v += part[w * 64 + lane];
      a.us[x * 64 + lane] = v;
      const double s1 = wave_sum_d(v * v), s2 = wave_sum_d(size * v);
      if (lane == 0) {
        a.uu[2 * (2 * a.nbits + x)] = s1;
        a.uu[2 * (2 * a.nbits + x) + 1] = s2;
      }
    }
    return;
  }
  BitProducts<TW> bp;
  if (a.nbits > 0) {
    bp.set(a.blocked + a.rbd0 * a.wpr * 64, 0, bid * TW, 4 * a.nbits, a.wpr, a.wpr, a.rdig);
    bp.start(wave);
  }
  // this lane's row in wavefronts 0 .. TW - 1
  const int i = 16 * wave + 4 * (lane >> 4) + (lane & 3);
  const int64_t b = (a.rbd0 * 4 + bid * TW) * 16 + i;
  const bool mine = wave < TW && (lane & 15) < 4;
  const double size = mine && b < a.kr ? static_cast<double>(a.sz[b]) : 0.0;
  const int er = a.ex[t & 1];
  if (wave == kWaves - 1) {
    const double v = wave_fixed(a.rr + (t % 3) * 2 * a.wpr, 2 * a.wpr);
    if (lane == 0) {
      gamma = v;
      if (bid == 0) cg_stop(a, t, v);
    }
  }
  if (a.nbits == 0) return;
  double row[4];
  bp.sums(wave, buf, row);
  combine_digits(row, er);
  // |u_b| <= sqrt(M) |r| (Cauchy-Schwarz) gives the digits of u their exponent
  const int eu = fixed_exponent(1.0000001 * __builtin_sqrt(static_cast<double>(a.M) * gamma));
  if (wave < TW) {
    // rows beyond kr have no bits (zero), those beyond the last block belong to none
    const double v = mine && bid * TW + wave < 4 * a.nbits ? pick_row(row, lane) : 0.0;
    if (mine) fixed[i] = to_fixed(v, eu);
    const double s1 = wave_sum_d(v * v), s2 = wave_sum_d(size * v);
    if (lane == 0) {
      red[wave] = s1;
      red[kWaves + wave] = s2;
    }
  }
  __syncthreads();
  if (tid < 32 * TW) {
    const int64_t u = bid * (TW / 2) + wave;
    if (u < 2 * a.nbits) {
      store_digits(fixed + 32 * wave, lane, u, a.udig);
      if (lane == 0) {
        a.uu[2 * u] = red[2 * wave] + red[2 * wave + 1];
        a.uu[2 * u + 1] = red[kWaves + 2 * wave] + red[kWaves + 2 * wave + 1];
      }
    }
  }
  if (bid == 0 && tid == 0) a.ex[2] = eu;
}

// The products of pass B for part y of the bit rows and players 16 TW x ..,
// workgroup y ceil(4 wpr / TW) + x: the digits' sums, for pass B to add.  For
// systems of few players and so many rows that pass B's own workgroups, one
// per 64 or 96 players, would leave most CUs idle for long.
template <int TW>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) k_cg_pass_b_part(GroupArgs g) {
  __shared__ alignas(16) float buf[kWaves * TW * 256];
  int64_t bid;
  const int m = member_of(g, bid);
  const Args& a = g.a[m];
  const int64_t t = g.t[m];
  if (a.st->last < static_cast<int32_t>(t)) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nx = (4 * a.wpr + TW - 1) / TW, x = bid % nx, y = bid / nx;
  const int64_t per = part_blocks(a.nbits, a.parts), b0 = y * per;
  const int64_t nb = a.nbits - b0 < per ? a.nbits - b0 : per;
  double row[4] = {};
  if (nb > 0) {   // (the last parts may be empty)
    BitProducts<TW> bp;
    bp.set(a.T, a.rbd0 + b0, x * TW, 4 * a.wpr, a.nrb, nb, a.udig + b0 / 4 * (2 * kOperand));
    bp.start(wave);
    bp.sums(wave, buf, row);
  }
  if (wave < TW)
    reinterpret_cast<v4d*>(a.qd)[((y * nx + x) * TW + wave) * 64 + (threadIdx.x & 63)] = v4d{row[0], row[1], row[2], row[3]};
}

// Pass B.  Workgroup x: players 16 TW x .. (see the recurrences above).  PARTS:
// some of the members have their products in parts (the branch costs the others
// 1 %).
template <int TW, bool PARTS>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) k_cg_pass_b(GroupArgs g) {
  __shared__ alignas(16) float buf[kWaves * TW * 256];
  __shared__ double sparse[16 * TW];
  __shared__ uint64_t fixed[16 * TW];
  __shared__ double sums[6];
  __shared__ double red[3][kWaves];
  int64_t bid;
  const int m = member_of(g, bid);
  const Args& a = g.a[m];
  const int64_t t = g.t[m];
  // set by an earlier launch, or to t by this one: all wavefronts go the same
  // way, as they must before x is written
  if (a.st->last < static_cast<int32_t>(t)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool whole = a.nbits > 0 && !(PARTS && a.parts > 1);
  BitProducts<TW> bp;
  if (whole) {
    bp.set(a.T, a.rbd0, bid * TW, 4 * a.wpr, a.nrb, a.nbits, a.udig);
    bp.start(wave);
  }
  // this lane's player in wavefronts 0 .. TW - 1
  const int i = 16 * wave + 4 * (lane >> 4) + (lane & 3);
  const int64_t j = bid * (16 * TW) + i;
  const bool mine = wave < TW && (lane & 15) < 4 && j < a.M;
  double rj = 0.0, pj = 0.0, sj = 0.0, xj = 0.0;
  if (mine) {
    rj = a.r[j];
    pj = a.p[j];
    sj = a.s[j];
    xj = a.x[j];
  }
  // the sparse rows' lists of this thread's players
  constexpr int kLists = (TW + 3) / 4;
  int64_t le0[kLists], le1[kLists];
#pragma unroll
  for (int h = 0; h < kLists; ++h) {
    const int ps = 64 * h + (tid >> 3);
    const int64_t js = bid * (16 * TW) + ps;
    const bool any = a.rs > 0 && js < a.M && ps < 16 * TW;
    le0[h] = any ? a.csc_ptr[js] + (tid & 7) : 0;
    le1[h] = any ? a.csc_ptr[js + 1] : 0;
  }
  const int eu = a.ex[2];
  const double before = t > 0 ? a.hist[(t + 1) & 1] : 1.0;   // the step before this one
  // the scalars' partial sums, one wavefront each: gamma, the gamma before,
  // |u|^2, |m|.u, largest |r| and |s|
  if (wave < 6) {
    const int64_t n = 2 * a.wpr;   // units of 32 players
    double v;
    if (wave == 0) v = wave_fixed(a.rr + (t % 3) * n, n);
    else if (wave == 1) v = t > 0 ? wave_fixed(a.rr + ((t + 2) % 3) * n, n) : 1.0;
    else if (wave < 4) v = wave_fixed(a.uu + (wave - 2), 2 * a.nbits + a.rbd0, 2);
    else v = wave_fixed<true>(a.mx + ((t & 1) * 2 + wave - 4) * n, n);
    if (lane == 0) sums[wave] = v;
  }
  // sparse rows: eight lanes per player, eight entries of each lane in flight
#pragma unroll
  for (int h = 0; h < kLists; ++h) {
    double v = 0.0;
    for (int64_t e = le0[h]; e < le1[h]; e += 64) {
      int32_t p[8];
      double u[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) p[k] = e + 8 * k < le1[h] ? a.csc_row[e + 8 * k] : -1;
#pragma unroll
      for (int k = 0; k < 8; ++k) u[k] = p[k] >= 0 ? a.us[p[k]] : 0.0;
#pragma unroll
      for (int k = 0; k < 8; ++k) v += u[k];
    }
    v += row_move<0xB1>(v);
    v += row_move<0x4E>(v);
    v += row_move<0x141>(v);
    if ((tid & 7) == 0 && 64 * h + (tid >> 3) < 16 * TW) sparse[64 * h + (tid >> 3)] = v;
  }
  double row[4] = {};
  if (whole) {
    bp.sums(wave, buf, row);
  } else {
    if (PARTS && a.parts > 1 && wave < TW) {
      // the parts' sums (whole numbers below 2^53 together: any order is exact)
      const v4d* qd = reinterpret_cast<const v4d*>(a.qd) + (bid * TW + wave) * 64 + lane;
      const int64_t stride = ((4 * a.wpr + TW - 1) / TW) * TW * 64;
      for (int64_t q = 0; q < a.parts; q += 8) {
        v4d v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = q + k < a.parts ? qd[(q + k) * stride] : v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 8; ++k)
#pragma unroll
          for (int c = 0; c < 4; ++c) row[c] += v[k][c];
      }
    }
    __syncthreads();
  }
  combine_digits(row, eu);
  const double gamma = sums[0], uu = sums[2];
  double beta = 0.0, den = a.alpha * gamma + a.wr2 * uu;
  if (t > 0) {
    beta = gamma / sums[1];
    den -= beta * gamma / before;
  }
  const double step = gamma / den;
  const double mq = sums[3] / static_cast<double>(a.M);
  if (!(den > 0.0 && step < 1e300 && beta == beta)) {   // identical in every workgroup
    if (bid == 0 && tid == 0) {
      a.st->last = static_cast<int32_t>(t);
      a.st->iters = static_cast<int32_t>(t);
      a.st->status = 2;
      __hip_atomic_store(a.host_flag + 1, static_cast<int32_t>(t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __hip_atomic_store(a.host_flag, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
  // |(R^T u)_j| <= sqrt(kr) |u| bounds the new s and r, and so gives the
  // digits of r their exponent (either weight may be negative)
  const double bw = __builtin_fabs(a.alpha) * sums[4] +
                    __builtin_fabs(a.wr2) * (__builtin_sqrt(static_cast<double>(a.kr) * uu) + __builtin_fabs(mq));
  const int e = fixed_exponent(1.0000001 * (sums[4] + step * (bw + beta * sums[5])));
  if (wave < TW) {
    double rn = 0.0, sn = 0.0;
    if (mine) {
      const double wj = a.alpha * rj + a.wr2 * ((sparse[i] + pick_row(row, lane)) - mq);
      const double pn = rj + beta * pj;
      sn = wj + beta * sj;
      rn = rj - step * sn;
      a.p[j] = pn;
      a.s[j] = sn;
      a.x[j] = xj + step * pn;
      a.r[j] = rn;
    }
    if ((lane & 15) < 4) fixed[i] = to_fixed(rn, e);
    const double r2 = wave_sum_d(rn * rn), rm = wave_max_d(__builtin_fabs(rn)), sm = wave_max_d(__builtin_fabs(sn));
    if (lane == 0) {
      red[0][wave] = r2;
      red[1][wave] = rm;
      red[2][wave] = sm;
    }
  }
  __syncthreads();
  if (tid < 32 * TW) {
    const int64_t u = bid * (TW / 2) + wave, n = 2 * a.wpr;
    if (u < n) {
      store_digits(fixed + 32 * wave, lane, u, a.rdig);
      if (lane == 0) {
        a.rr[((t + 1) % 3) * n + u] = red[0][2 * wave] + red[0][2 * wave + 1];
        double* mx = a.mx + ((t + 1) & 1) * 2 * n;
        mx[u] = fmax(red[1][2 * wave], red[1][2 * wave + 1]);
        mx[n + u] = fmax(red[2][2 * wave], red[2][2 * wave + 1]);
      }
    }
  }
  if (bid == 0 && tid == 0) {
    a.hist[t & 1] = step;
    a.ex[(t + 1) & 1] = e;
  }
}

// The instance of a pass for `tiles` tiles per workgroup (4 or 6).
using PassFn = void (*)(GroupArgs);
PassFn pass_a(int tiles) { return tiles == 4 ? k_cg_pass_a<4> : k_cg_pass_a<6>; }
PassFn pass_b_part(int tiles) { return tiles == 4 ? k_cg_pass_b_part<4> : k_cg_pass_b_part<6>; }
PassFn pass_b(int tiles, bool parts) {
  return tiles == 4 ? (parts ? k_cg_pass_b<4, true> : k_cg_pass_b<4, false>)
                    : (parts ? k_cg_pass_b<6, true> : k_cg_pass_b<6, false>);
}

// ---- the sparse rows' lists, built once per solve ------------------------------------------

// Inclusive prefix sum of v over the 1024 threads of a workgroup.
__device__ int64_t block_scan(int64_t v) {
  __shared__ int64_t part[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int64_t x = __shfl_up(static_cast<long long>(v), off);
    if (lane >= off) v += x;
  }
  if (lane == 63) part[wave] = v;
  __syncthreads();
  for (int w = 0; w < wave; ++w) v += part[w];
  return v;
}

// Row lists: ptr[x] = entries per row of the blocks before x (block x's rows
// have as many as its last, largest row), at most 1024 blocks.
__global__ void __launch_bounds__(1024) k_cg_ell_ptr(const int32_t* __restrict__ sz, int64_t nblk,
                                                     int64_t* __restrict__ ptr) {
  const int x = threadIdx.x;
  const int64_t n = x < nblk ? sz[64 * x + 63] : 0;
  const int64_t end = block_scan(n);
  if (x == 0) ptr[0] = 0;
  if (x < nblk) ptr[x + 1] = end;
}

// The lists are built in kSeg segments at once: of the player words for the
// row lists, of the row blocks for the player lists.  A count pass gives each
// (row or player, segment) its number of entries, so the fill pass of a
// segment starts at the list's start plus the counts of the segments before
// it; every list comes out in ascending order.
constexpr int kSeg = 8;

// Row lists, counts: wavefront (g, s) reads the words of segment s of its
// 64 rows from the row-blocked copy (lane = row): cnt[s][b].
__global__ void __launch_bounds__(64) k_cg_ell_count(const uint64_t* __restrict__ blocked, int64_t wpr, int64_t rs,
                                                     int32_t* __restrict__ cnt) {
  const int64_t g = blockIdx.x;
  const int sg = blockIdx.y;
  const int64_t b = g * 64 + threadIdx.x;
  if (b >= rs) return;
  const int64_t w0 = wpr * sg / kSeg, w1 = wpr * (sg + 1) / kSeg;
  const uint64_t* src = blocked + g * wpr * 64 + threadIdx.x;
  int c = 0;
  for (int64_t w = w0; w < w1; ++w) c += __popcll(src[w * 64]);
  cnt[sg * rs + b] = c;
}

// Row lists, fill: the players of segment s of row b in order; the last
// segment pads the row with M.
__global__ void __launch_bounds__(64) k_cg_ell_fill(const uint64_t* __restrict__ blocked, int64_t wpr, int64_t rs,
                                                    const int64_t* __restrict__ ptr, const int32_t* __restrict__ cnt,
                                                    int32_t M, int32_t* __restrict__ idx) {
  const int64_t g = blockIdx.x;
  const int sg = blockIdx.y;
  const int64_t b = g * 64 + threadIdx.x;
  if (b >= rs) return;
  int64_t pos = ptr[g];
  const int64_t end = ptr[g + 1];
  for (int q = 0; q < sg; ++q) pos += cnt[q * rs + b];
  const int64_t w0 = wpr * sg / kSeg, w1 = wpr * (sg + 1) / kSeg;
  const uint64_t* src = blocked + g * wpr * 64 + threadIdx.x;
  idx += threadIdx.x;
  for (int64_t w = w0; w < w1; ++w) {
    uint64_t word = src[w * 64];
    while (word && pos < end) {
      idx[64 * pos++] = static_cast<int32_t>(w * 64 + __builtin_ctzll(word));
      word &= word - 1;
    }
  }
  if (sg == kSeg - 1)
    for (; pos < end; ++pos) idx[64 * pos] = M;
}

// Player-major lists, counts: cnt[s][j] = the sparse rows of segment s (row
// blocks nrb_s s / kSeg .. of the bit-transposed rows T[rb, j]) holding j.
__global__ void __launch_bounds__(256) k_cg_csc_count(const uint64_t* __restrict__ T, int64_t M, int64_t nrb, int64_t nrb_s,
                                                      int32_t* __restrict__ cnt) {
  const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int sg = blockIdx.y;
  if (j >= M) return;
  const int64_t r0 = nrb_s * sg / kSeg, r1 = nrb_s * (sg + 1) / kSeg;
  int c = 0;
  for (int64_t rb = r0; rb < r1; ++rb) c += __popcll(T[((j >> 6) * nrb + rb) * 64 + (j & 63)]);
  cnt[sg * M + j] = c;
}

// ptr[j] = total of player j's segment counts (fixed order), then the
// exclusive prefix sums over j in place (ptr[M] = the total).
__global__ void __launch_bounds__(256) k_cg_csc_total(const int32_t* __restrict__ cnt, int64_t M,
                                                      int64_t* __restrict__ ptr) {
  const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (j >= M) return;
  int64_t v = 0;
#pragma unroll
  for (int q = 0; q < kSeg; ++q) v += cnt[q * M + j];
  ptr[j] = v;
}

// (in place: each thread reads each of its entries before writing it)
__global__ void __launch_bounds__(1024) k_cg_csc_scan(int64_t M, int64_t* ptr) {
  const int t = threadIdx.x;
  const int64_t per = (M + 1023) / 1024;
  const int64_t i0 = t * per, i1 = i0 + per < M ? i0 + per : M;
  int64_t s = 0;
  for (int64_t i = i0; i < i1; ++i) s += ptr[i];
  int64_t run = block_scan(s) - s;
  if (t == 1023) ptr[M] = run + s;
  for (int64_t i = i0; i < i1; ++i) {
    const int64_t x = ptr[i];
    ptr[i] = run;
    run += x;
  }
}

__global__ void __launch_bounds__(256) k_cg_csc_fill(const uint64_t* __restrict__ T, int64_t M, int64_t nrb, int64_t nrb_s,
                                                     const int64_t* __restrict__ ptr, const int32_t* __restrict__ cnt,
                                                     int64_t nnz, int32_t* __restrict__ rows) {
  const int64_t j = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int sg = blockIdx.y;
  if (j >= M) return;
  int64_t pos = ptr[j];
  for (int q = 0; q < sg; ++q) pos += cnt[q * M + j];
  const int64_t end = ptr[j + 1] < nnz ? ptr[j + 1] : nnz;
  const int64_t r0 = nrb_s * sg / kSeg, r1 = nrb_s * (sg + 1) / kSeg;
  for (int64_t rb = r0; rb < r1; ++rb) {
    uint64_t word = T[((j >> 6) * nrb + rb) * 64 + (j & 63)];
    while (word && pos < end) {
      rows[pos++] = static_cast<int32_t>(rb * 64 + __builtin_ctzll(word));
      word &= word - 1;
    }
  }
}

// Sum of v over the 1024 threads of a workgroup, in every thread.
__device__ __forceinline__ double block_sum_d(double v) {
  __shared__ double red[16];
  v = wave_sum_d(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < 16; ++i) s += red[i];
  return s;
}

// phi = Delta/M + x - mean(x) (the projection made exact), info from the state.
__global__ void __launch_bounds__(1024) k_cg_finish(const double* __restrict__ x, int64_t M,
                                                    const gnnshap::CgState* __restrict__ st,
                                                    const float* __restrict__ fef, float* __restrict__ phi,
                                                    int32_t* info, int32_t undetermined) {
  double sm = 0.0;
  for (int64_t j = threadIdx.x; j < M; j += 1024) sm += x[j];
  const double mean = block_sum_d(sm) / static_cast<double>(M);
  const double base = (static_cast<double>(fef[1]) - static_cast<double>(fef[0])) / static_cast<double>(M);
  for (int64_t j = threadIdx.x; j < M; j += 1024) phi[j] = static_cast<float>(base + (x[j] - mean));
  if (threadIdx.x == 0) *info = (st->status == 0 && !undetermined) ? 0 : static_cast<int32_t>(M + 1);
}

// Mapped page-locked stopping flags of the calling thread and their device
// addresses: one slot per solve in flight (created on first use, kept until
// the process ends).
struct HostFlag {
  int32_t* host = nullptr;
  int32_t* dev = nullptr;
  bool busy = false;
};

constexpr int kFlagSlots = 16;

HostFlag* acquire_flag() {
  static thread_local HostFlag pool[kFlagSlots];
  for (HostFlag& f : pool) {
    if (f.busy) continue;
    if (!f.host) {
      void* h = nullptr;
      if (hipHostMalloc(&h, 256, hipHostMallocMapped | hipHostMallocCoherent) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
      }
      void* d = nullptr;
      if (hipHostGetDevicePointer(&d, h, 0) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipHostFree(h);
        return nullptr;
      }
      f.host = static_cast<int32_t*>(h);
      f.dev = static_cast<int32_t*>(d);
    }
    f.busy = true;
    return &f;
  }
  return nullptr;
}

// The two events of a group's chunk ring, per calling thread (created on
// first use, kept until the process ends).
struct EventPair {
  hipEvent_t ev[2] = {nullptr, nullptr};
  bool busy = false;
};

constexpr int kPairSlots = 8;

EventPair* acquire_pair() {
  static thread_local EventPair pool[kPairSlots];
  for (EventPair& e : pool) {
    if (e.busy) continue;
    for (int i = 0; i < 2; ++i)
      if (!e.ev[i] && hipEventCreateWithFlags(&e.ev[i], hipEventDisableTiming) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
      }
    e.busy = true;
    return &e;
  }
  return nullptr;
}

// Whether the work recorded by ev has completed, without waiting; a query
// that finds it pending leaves no error behind for the next launch check.
bool event_done(hipEvent_t ev) {
  const hipError_t e = hipEventQuery(ev);
  if (e == hipErrorNotReady) {
    (void)hipGetLastError();
    return false;
  }
  return true;   // complete, or an error that the wait on it reports
}

// Pass B in parts: up to 128 word columns (two workgroups of 64 players per
// CU are 512) and from 196,608 bit rows on, whose products take a workgroup
// 32 us and more, against the ~12 us that another launch and the parts' sums
// cost.  The solve of 5,001 players x 1,600,000 coalitions 4.29 -> 3.32 ms,
// x 800,000 2.65 -> 2.12, 2,000 x 1,600,000 3.36 -> 2.14; 12,000 x 1,600,000
// (188 workgroups) is left whole at 7.2 ms.
int64_t parts_of(int64_t wpr, int64_t nbits) {
  return wpr <= 128 && nbits >= 3072 ? std::min<int64_t>({512 / wpr, nbits / 512, 64}) : 1;
}

}  // namespace

gnnshap::CgShape gnnshap::cg_shape(int64_t M, int64_t wpr, int64_t kr, int64_t rb0, const gnnshap_class* classes,
                                   int64_t ncls) {
  CgShape s{};
  s.M = M;
  s.wpr = wpr;
  s.kr = kr;
  s.nrb = ceil_div(kr, 64);
  // sparse rows: the longest run of random rows from the first whose sizes are
  // at most M / kSparseDiv and ascend (a block's last row is its largest, as
  // its padded lists need; other orders of a caller's class table end the
  // run), cut to whole 64-row groups
  if (kr > 0 && classes) {
    const int64_t tmax = M / kSparseDiv;
    std::vector<int32_t> sz;
    sz.reserve(static_cast<size_t>(kr));
    for (int64_t i = 0; i < ncls && static_cast<int64_t>(sz.size()) < kr; ++i) {
      if (classes[i].row_begin + classes[i].row_count <= rb0) continue;
      if (classes[i].size > tmax || (!sz.empty() && classes[i].size < sz.back())) break;
      const int64_t from = std::max<int64_t>(classes[i].row_begin, rb0);
      for (int64_t r = from; r < classes[i].row_begin + classes[i].row_count; ++r) sz.push_back(classes[i].size);
    }
    s.rs = (std::min<int64_t>(static_cast<int64_t>(sz.size()), kr) / 64) * 64;
    if (s.rs > 64 * 1024) s.rs = 64 * 1024;   // the row lists' scan holds 1024 blocks
    for (int64_t b = 0; b < s.rs; ++b) s.nnz += sz[b];
    // the padded lists: a block's rows have the entries of its last one, and the
    // sizes ascend to tmax, so this holds them for any order of the classes
    if (s.rs > 0) s.nell = s.nnz + 64 * tmax;
  }
  s.rbd0 = s.rs / 64;
  s.nbits = s.nrb - s.rbd0;
  s.parts = parts_of(wpr, s.nbits);
  return s;
}

gnnshap::CgWs gnnshap::cg_carve(Carver& c, const CgShape& sh) {
  CgWs w;
  const int64_t kr = sh.kr > 0 ? sh.kr : 1;
  w.x = c.take<double>(sh.M);
  w.r = c.take<double>(sh.M + 1);
  w.p = c.take<double>(sh.M);
  w.s = c.take<double>(sh.M);
  w.us = c.take<double>(sh.rs > 0 ? sh.rs : 1);
  w.rdig = c.take<char>(digit_bytes(sh.wpr));
  // (the digits, the partial sums and the parts are sized for no sparse rows, so
  // that a table with fewer of them than the plan's own, which workspace
  // queries assume, needs no more)
  w.udig = c.take<char>(std::max<int64_t>(digit_bytes(sh.nrb), 1));
  w.uu = c.take<double>(2 * std::max<int64_t>(2 * sh.nrb, 1));
  const int64_t parts = parts_of(sh.wpr, sh.nrb);
  w.qd = c.take<double>(parts > 1 ? parts * (4 * sh.wpr + 5) * 256 : 1);
  w.rr = c.take<double>(3 * 2 * sh.wpr);
  w.mx = c.take<double>(4 * 2 * sh.wpr);
  w.hist = c.take<double>(2);
  w.ex = c.take<int32_t>(3);
  w.sz = c.take<int32_t>(kr);
  w.blocked = c.take<uint64_t>((sh.nrb > 0 ? sh.nrb : 1) * sh.wpr * 64);
  w.st = c.take<CgState>(1);
  w.ell_ptr = c.take<int64_t>(sh.rbd0 + 1);
  w.ell_idx = c.take<int32_t>(sh.nell > 0 ? sh.nell : 1);
  w.csc_ptr = c.take<int64_t>(sh.M + 1);
  w.csc_row = c.take<int32_t>(sh.nnz > 0 ? sh.nnz : 1);
  w.segcnt = c.take<int32_t>(kSeg * std::max<int64_t>(std::max<int64_t>(sh.rs, sh.M), 1));
  return w;
}

// One member of a group: its arguments, shape, problem and flag, the
// iteration its next launch runs and its grids.
struct Member {
  Args a;
  gnnshap::CgShape sh;
  gnnshap::CgProblem pr;
  gnnshap::CgWs w;
  HostFlag* hf = nullptr;
  int64_t t = 0;
};

struct gnnshap::CgGroup::State {
  std::vector<Member> mem;
  EventPair* ev = nullptr;
  int64_t chunk = 0;
};

gnnshap::CgGroup::CgGroup() : st_(new State()) {}

gnnshap::CgGroup::~CgGroup() {
  for (Member& m : st_->mem)
    if (m.hf) m.hf->busy = false;
  if (st_->ev) st_->ev->busy = false;
}

int gnnshap::CgGroup::size() const { return static_cast<int>(st_->mem.size()); }

int gnnshap::CgGroup::add(const CgProblem& pr, const CgShape& sh, const CgWs& w) {
  State& S = *st_;
  if (full()) return fail(GNNSHAP_EINVAL, "solver group already holds %d systems", kCgGroupMax);
  if (!S.ev) {
    S.ev = acquire_pair();
    if (!S.ev) return fail(GNNSHAP_EHIP, "could not create the solver's events (or more than %d groups)", kPairSlots);
  }
  HostFlag* hf = acquire_flag();
  if (!hf) return fail(GNNSHAP_EHIP, "could not allocate the solver's host flag (or more than %d solves in flight)",
                       kFlagSlots);
  hipStream_t s = s_;
  Member m;
  m.hf = hf;
  m.sh = sh;
  m.pr = pr;
  m.w = w;
  Args& a = m.a;
  a = Args{};
  a.blocked = pr.blocked;
  a.T = pr.T;
  a.sz = w.sz;
  a.M = sh.M;
  a.wpr = sh.wpr;
  a.kr = sh.kr;
  a.nrb = sh.nrb;
  a.alpha = pr.alpha;
  a.wr2 = sh.kr > 0 ? 2.0 * pr.wr : 0.0;
  a.tol2 = kTol * kTol;
  a.maxit = kMaxIt;
  a.x = w.x;
  a.r = w.r;
  a.p = w.p;
  a.s = w.s;
  a.us = w.us;
  a.qd = w.qd;
  a.parts = sh.parts;
  a.rdig = w.rdig;
  a.udig = w.udig;
  a.uu = w.uu;
  a.rr = w.rr;
  a.mx = w.mx;
  a.hist = w.hist;
  a.ex = w.ex;
  a.st = w.st;
  a.rs = sh.rs;
  a.rbd0 = sh.rbd0;
  a.nbits = sh.nbits;
  a.ell_ptr = w.ell_ptr;
  a.ell_idx = w.ell_idx;
  a.csc_ptr = w.csc_ptr;
  a.csc_row = w.csc_row;
  a.host_flag = hf->dev;
  // no kernel of an earlier solve that used this flag writes it any more:
  // a solve stops writing it at its stopping iteration, which had completed
  // before the flag was released
  __atomic_store_n(hf->host, 0, __ATOMIC_RELEASE);
  __atomic_store_n(hf->host + 1, -1, __ATOMIC_RELEASE);
  {
    GS_TIMED("k_cg_init", s);
    k_cg_init<<<static_cast<unsigned>(ceil_div(sh.wpr, 4)), 256, 0, s>>>(a, pr.dv, pr.bsum, pr.nb, pr.classes,
                                                                         pr.ncls, pr.rb0, w.sz);
    GS_LAUNCHED();
    k_cg_digits<<<static_cast<unsigned>(sh.wpr), 128, 0, s>>>(a);
  }
  GS_LAUNCHED();
  if (sh.rs > 0) {
    // the sparse rows' lists (row sizes from k_cg_init)
    const int64_t nrb_s = sh.rs / 64;
    const dim3 gr(static_cast<unsigned>(nrb_s), kSeg), gp(static_cast<unsigned>(ceil_div(sh.M, 256)), kSeg);
    GS_TIMED("k_cg_sparse_build", s);
    k_cg_ell_ptr<<<1, 1024, 0, s>>>(w.sz, nrb_s, w.ell_ptr);
    GS_LAUNCHED();
    k_cg_ell_count<<<gr, 64, 0, s>>>(pr.blocked, sh.wpr, sh.rs, w.segcnt);
    GS_LAUNCHED();
    k_cg_ell_fill<<<gr, 64, 0, s>>>(pr.blocked, sh.wpr, sh.rs, w.ell_ptr, w.segcnt, static_cast<int32_t>(sh.M),
                                    w.ell_idx);
    GS_LAUNCHED();
    k_cg_csc_count<<<gp, 256, 0, s>>>(pr.T, sh.M, sh.nrb, nrb_s, w.segcnt);
    GS_LAUNCHED();
    k_cg_csc_total<<<static_cast<unsigned>(ceil_div(sh.M, 256)), 256, 0, s>>>(w.segcnt, sh.M, w.csc_ptr);
    GS_LAUNCHED();
    k_cg_csc_scan<<<1, 1024, 0, s>>>(sh.M, w.csc_ptr);
    GS_LAUNCHED();
    k_cg_csc_fill<<<gp, 256, 0, s>>>(pr.T, sh.M, sh.nrb, nrb_s, w.csc_ptr, w.segcnt, sh.nnz, w.csc_row);
    GS_LAUNCHED();
  }
  S.mem.push_back(m);
  return GNNSHAP_OK;
}

bool gnnshap::CgGroup::ready() const {
  const State& S = *st_;
  return S.chunk < 2 || event_done(S.ev->ev[S.chunk & 1]);   // step() waits for the chunk before last
}

namespace {

// Fills g with the members selected by `take` (grid of member m: grid(m)),
// each at iteration t + dt; returns the total number of workgroups.
template <class Take, class Grid>
uint32_t fill_group(GroupArgs& g, const std::vector<Member>& mem, int64_t dt, Take take, Grid grid) {
  g.n = 0;
  uint32_t total = 0;
  for (const Member& m : mem) {
    if (!take(m, m.t + dt)) continue;
    g.a[g.n] = m.a;
    g.t[g.n] = m.t + dt;
    g.blk[g.n] = total;
    total += grid(m);
    ++g.n;
  }
  g.blk[g.n] = total;
  return total;
}

}  // namespace

namespace {

// Workgroups of `tiles` tiles each: of pass A's bit rows (at least one, which
// takes the stopping test) and of pass B.
int64_t blocks_a(const gnnshap::CgShape& sh, int tiles) {
  return std::max<int64_t>(gnnshap::ceil_div(4 * sh.nbits, tiles), 1);
}
int64_t blocks_b(const gnnshap::CgShape& sh, int tiles) { return gnnshap::ceil_div(4 * sh.wpr, tiles); }

// Tiles per workgroup of a pass over the members: the number that leaves the
// busiest of 256 CUs the least to load (see the passes), taking the
// workgroups as spread evenly.
template <class Blocks, class Groups>
int choose_tiles(const std::vector<Member>& mem, Blocks blocks, Groups groups) {
  int best = 4;
  double least = 0.0;
  for (int tiles = 4; tiles <= 6; tiles += 2) {
    double count = 0.0, work = 0.0;
    for (const Member& m : mem) {
      const double n = static_cast<double>(blocks(m.sh, tiles));
      count += n;
      work += n * static_cast<double>(groups(m.sh)) * (8 * tiles + 48);   // clocks of 64 bytes
    }
    const double busiest = std::ceil(count / 256.0) * (work / count);
    if (tiles == 4 || busiest < least) {
      best = tiles;
      least = busiest;
    }
  }
  return best;
}

}  // namespace

// Waits for the chunk before the last one queued; every member whose stop
// flag is set gets phi and info queued (after the chunks already queued,
// whose launches it leaves at once) and leaves the group.  Then queues
// iterations t .. t + kChunk - 1 of every member left (pass A alone of
// iteration kMaxIt, which always stops; nothing beyond it) and records the
// chunk's event.  The ring has two events: chunk n reuses the event of chunk
// n - 2, which has completed by then.
int gnnshap::CgGroup::step() {
  State& S = *st_;
  if (S.mem.empty()) return GNNSHAP_OK;
  hipStream_t s = s_;
  if (S.chunk >= 2) {
    GS_HIP(hipEventSynchronize(S.ev->ev[S.chunk & 1]));
    for (size_t i = 0; i < S.mem.size();) {
      Member& m = S.mem[i];
      if (__atomic_load_n(m.hf->host, __ATOMIC_ACQUIRE) == 0) {
        ++i;
        continue;
      }
      const int64_t iters = __atomic_load_n(m.hf->host + 1, __ATOMIC_ACQUIRE);
      last_iters_ = iters;
      const CgShape& sh = m.sh;
      timing_note_solve(sh.M, sh.wpr, sh.kr, iters, sh.rs, sh.nnz);
      {
        GS_TIMED("k_cg_finish", s);
        // without enumerated classes, fewer than M - 1 random rows cannot
        // determine psi (1-perp has M - 1 dimensions): reported like a failed pivot
        const int32_t undetermined = (m.pr.alpha == 0.0 && sh.kr < sh.M - 1) ? 1 : 0;
        k_cg_finish<<<1, 1024, 0, s>>>(m.w.x, sh.M, m.w.st, m.pr.fef, m.pr.phi, m.pr.info, undetermined);
      }
      GS_LAUNCHED();
      m.hf->busy = false;
      S.mem.erase(S.mem.begin() + static_cast<std::ptrdiff_t>(i));
    }
    if (S.mem.empty()) return GNNSHAP_OK;
  }
  GroupArgs g;
  const int ta = choose_tiles(S.mem, blocks_a, [](const CgShape& sh) { return ceil_div(sh.wpr, 4); });
  const int tb = choose_tiles(S.mem, blocks_b, [](const CgShape& sh) { return ceil_div(sh.nbits, 4) + 1; });
  for (int64_t dt = 0; dt < kChunk; ++dt) {
    uint32_t n = fill_group(g, S.mem, dt, [](const Member&, int64_t t) { return t <= kMaxIt; },
                            [ta](const Member& m) { return static_cast<uint32_t>(blocks_a(m.sh, ta) + m.sh.rbd0); });
    if (g.n == 0) break;
    {
      GS_TIMED("k_cg_pass_a", s);
      pass_a(ta)<<<n, kThreads, 0, s>>>(g);
    }
    GS_LAUNCHED();
    n = fill_group(g, S.mem, dt, [](const Member& m, int64_t t) { return t < kMaxIt && m.sh.parts > 1; },
                   [tb](const Member& m) { return static_cast<uint32_t>(blocks_b(m.sh, tb) * m.sh.parts); });
    const bool parts = g.n > 0;
    if (parts) {
      GS_TIMED("k_cg_pass_b_part", s);
      pass_b_part(tb)<<<n, kThreads, 0, s>>>(g);
    }
    GS_LAUNCHED();
    n = fill_group(g, S.mem, dt, [](const Member&, int64_t t) { return t < kMaxIt; },
                   [tb](const Member& m) { return static_cast<uint32_t>(blocks_b(m.sh, tb)); });
    if (g.n > 0) {
      {
        GS_TIMED("k_cg_pass_b", s);
        pass_b(tb, parts)<<<n, kThreads, 0, s>>>(g);
      }
      GS_LAUNCHED();
    }
  }
  for (Member& m : S.mem) m.t = std::min(m.t + kChunk, kMaxIt + 1);
  GS_HIP(hipEventRecord(S.ev->ev[S.chunk & 1], s));
  ++S.chunk;
  return GNNSHAP_OK;
}

int gnnshap::cg_solve(const CgProblem& pr, const CgShape& sh, const CgWs& w, hipStream_t s, int64_t* iters_out) {
  CgGroup grp;
  grp.set_stream(s);
  if (int st = grp.add(pr, sh, w)) return st;
  while (!grp.empty())
    if (int st = grp.step()) return st;
  if (iters_out) *iters_out = grp.last_iters();
  return GNNSHAP_OK;
}
