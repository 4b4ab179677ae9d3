// Compress path on gfx950: v_max scan, stratified subsample and the bucketed
// kernel-halving round (KH(1/2) under kappa_att), one launch per round.
#include <math.h>

#include <algorithm>

#include "common.hpp"
#include "launch.hpp"
#include "score_plan.hpp"

namespace thin {

namespace {

constexpr double kLn2 = 0.69314718055994530942;
constexpr double kLog2e = 1.44269504088896340736;

// Row strides of the index lists (0 = packed: n_r in, n_r / 2 out) and the
// first uniform of bucket t's P pairs within its slice.
__device__ __forceinline__ int64_t in_stride(const HalveArgs& a) {
  return a.in_stride ? a.in_stride : a.n_r;
}
__device__ __forceinline__ int64_t out_stride(const HalveArgs& a) {
  return a.out_stride ? a.out_stride : (a.n_r >> 1);
}
__device__ __forceinline__ int64_t bucket_u(const HalveArgs& a, int64_t t, int P) {
  return a.u_bucket ? a.u_bucket[t] : a.u_off + t * (int64_t)P;
}

__device__ __forceinline__ float wave_max_f(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}
__device__ __forceinline__ uint32_t wave_max_u(uint32_t v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off));
  return v;
}
__device__ __forceinline__ double wave_max_d(double v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  return v;
}

// ---------------------------------------------------------------------------
// v_max = max_i ||v_i||_inf over the n thinned rows of a slice (Sec. 2.1, eq.
// katt); consecutive slices start slice_words 16-byte words apart.
// grid (chunks, S); the per-slice maximum is merged with an integer atomicMax
// on the float's bit pattern (valid for non-negative floats).
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void vmax_kernel(const T* V, int64_t words_per_slice,
                                                   int64_t slice_words, int64_t words_per_block,
                                                   uint32_t* vmax_bits) {
  const int64_t s = blockIdx.y;
  const uint4* base = reinterpret_cast<const uint4*>(V) + s * slice_words;
  int64_t w0 = (int64_t)blockIdx.x * words_per_block;
  int64_t w1 = w0 + words_per_block;
  if (w1 > words_per_slice) w1 = words_per_slice;
  // The magnitude bits of a (non-NaN) float order like the magnitudes
  // themselves, so max |x| is taken on the bit patterns as unsigned integers
  uint32_t m = 0u;
  auto fold = [&](const u32x4& x) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (Elem<T>::bytes == 4) {
        m = max(m, x[c] & 0x7fffffffu);
      } else {
        m = max(m, (x[c] << 16) & 0x7fffffffu);
        m = max(m, x[c] & 0x7fff0000u);
      }
    }
  };
  // eight independent 16-byte loads in flight per thread
  constexpr int U = 8;
  const u32x4* vb = reinterpret_cast<const u32x4*>(base);
  int64_t w = w0 + threadIdx.x;
  for (; w + (U - 1) * (int64_t)blockDim.x < w1; w += U * (int64_t)blockDim.x) {
    u32x4 x[U];
#pragma unroll
    for (int k = 0; k < U; ++k) x[k] = vb[w + k * (int64_t)blockDim.x];
#pragma unroll
    for (int k = 0; k < U; ++k) fold(x[k]);
  }
  for (; w < w1; w += blockDim.x) fold(vb[w]);
  const float mf = wave_max_f(__uint_as_float(m));
  __shared__ float part[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) part[wave] = mf;
  __syncthreads();
  if (threadIdx.x == 0) {
    float r = part[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = fmaxf(r, part[i]);
    atomicMax(vmax_bits + s, __float_as_uint(r));
  }
}

// p[0..count) = 0, and *also = 0 (nullable).
__global__ void zero_u32_kernel(uint32_t* p, int64_t count, int32_t* also) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = 0u;
  if (also && i == 0) *also = 0;
}

__global__ void zero_u8_kernel(uint8_t* p, int64_t count) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = 0;
}

// ---------------------------------------------------------------------------
// Stratified subsample (Alg. 3 / App. H Algorithm H.1 with unequal strata):
// stratum t = [floor(t n / n_kept), floor((t+1) n / n_kept)), pick
// start + floor(u len) computed in integers from k = floor(u 2^24).
// ---------------------------------------------------------------------------
// Also clears zero[0..zero_words) and *also (nullable): what the v_max launch
// after it would else need a launch of its own for.
__global__ void subsample_kernel(int64_t n, int64_t n_kept, const float* U, int64_t u_slice,
                                 int32_t* idx0, uint32_t* zero, int64_t zero_words,
                                 int32_t* also) {
  const int64_t s = blockIdx.y;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t threads = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = s * threads + t; i < zero_words; i += gridDim.y * threads) zero[i] = 0u;
  if (also && s == 0 && t == 0) *also = 0;
  if (t >= n_kept) return;
  const int64_t start = (t * n) / n_kept;
  const int64_t len = ((t + 1) * n) / n_kept - start;
  int64_t k = (int64_t)(U[s * u_slice + t] * 16777216.0f);
  k = k < 0 ? 0 : (k > 16777215 ? 16777215 : k);
  int64_t pick = (k * len) >> 24;
  if (pick > len - 1) pick = len - 1;
  idx0[s * n_kept + t] = (int32_t)(start + pick);
}

// dst[s, j] = src ? src[s * src_stride + j] : j   (j < n_out)
__global__ void fill_rows_kernel(int64_t n_out, const int32_t* src, int64_t src_stride,
                                 int32_t* dst) {
  const int64_t s = blockIdx.y;
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n_out) return;
  dst[s * n_out + j] = src ? src[s * src_stride + j] : (int32_t)j;
}

// Output of a compress with exact sink and window rows: row j of slice s is
// sink j (j < ns), then coreset row ns + src[s * src_stride + j - ns] (src
// null = the identity) for n_out rows, then window row n - nw + ...; its
// log-weight (logw nullable) is 0 for exact rows and lw_core for coreset rows.
__global__ void assemble_kernel(int64_t n, int64_t ns, int64_t n_out, int64_t nw,
                                const int32_t* src, int64_t src_stride, int32_t* dst,
                                float* logw, float lw_core) {
  const int64_t s = blockIdx.y;
  const int64_t m = ns + n_out + nw;
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= m) return;
  int64_t r = j;
  float w = 0.0f;
  if (j >= ns + n_out) {
    r = n - nw + (j - ns - n_out);
  } else if (j >= ns) {
    r = ns + (src ? (int64_t)src[s * src_stride + j - ns] : j - ns);
    w = lw_core;
  }
  dst[s * m + j] = (int32_t)r;
  if (logw) logw[s * m + j] = w;
}

// ---------------------------------------------------------------------------
// Cross-lane helpers (VALU only, no LDS crossbar).
// ---------------------------------------------------------------------------

// Value of lane l ^ 1 (DPP quad_perm [1,0,3,2]).
__device__ __forceinline__ uint32_t from_partner(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);
}
__device__ __forceinline__ float from_partner(float v) {
  return __uint_as_float(from_partner(__float_as_uint(v)));
}
__device__ __forceinline__ double from_partner(double v) {
  const uint64_t u = (uint64_t)__double_as_longlong(v);
  const uint64_t r = (uint64_t)from_partner((uint32_t)u) |
                     ((uint64_t)from_partner((uint32_t)(u >> 32)) << 32);
  return __longlong_as_double((long long)r);
}

// Inclusive prefix maximum over lanes 0..31 (rows of 16 by DPP row shifts,
// then lane 15 carried into the second row).  Lanes >= 32 are ignored.
__device__ __forceinline__ double dpp_row_shr_max(double x, int n_ctrl) {
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  const uint64_t ninf = (uint64_t)__double_as_longlong(-INFINITY);
  uint32_t lo, hi;
  switch (n_ctrl) {
    case 1:
      lo = __builtin_amdgcn_update_dpp((int)(uint32_t)ninf, (int)(uint32_t)u, 0x111, 0xF, 0xF, false);
      hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(ninf >> 32), (int)(uint32_t)(u >> 32), 0x111, 0xF, 0xF, false);
      break;
    case 2:
      lo = __builtin_amdgcn_update_dpp((int)(uint32_t)ninf, (int)(uint32_t)u, 0x112, 0xF, 0xF, false);
      hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(ninf >> 32), (int)(uint32_t)(u >> 32), 0x112, 0xF, 0xF, false);
      break;
    case 4:
      lo = __builtin_amdgcn_update_dpp((int)(uint32_t)ninf, (int)(uint32_t)u, 0x114, 0xF, 0xF, false);
      hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(ninf >> 32), (int)(uint32_t)(u >> 32), 0x114, 0xF, 0xF, false);
      break;
    default:
      lo = __builtin_amdgcn_update_dpp((int)(uint32_t)ninf, (int)(uint32_t)u, 0x118, 0xF, 0xF, false);
      hi = __builtin_amdgcn_update_dpp((int)(uint32_t)(ninf >> 32), (int)(uint32_t)(u >> 32), 0x118, 0xF, 0xF, false);
      break;
  }
  return fmax(x, __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32))));
}

__device__ __forceinline__ double prefix_max32(double x, int lane) {
  x = dpp_row_shr_max(x, 1);
  x = dpp_row_shr_max(x, 2);
  x = dpp_row_shr_max(x, 4);
  x = dpp_row_shr_max(x, 8);
  const uint64_t u = (uint64_t)__double_as_longlong(x);
  const uint64_t r15 = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 15) |
                       ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), 15) << 32);
  const double m15 = __longlong_as_double((long long)r15);
  return (lane >= 16 && lane < 32) ? fmax(x, m15) : x;
}

// exp(x) for float64 x: 2^n * 2^f with n = floor(x log2 e), 2^f from the
// float32 exp2 (about 1e-7 relative), so the range is that of float64.
__device__ __forceinline__ double exp_fast(double x) {
  const double y = x * kLog2e;
  const double n = floor(y);
  const float f = (float)(y - n);
  return ldexp((double)__builtin_amdgcn_exp2f(f), (int)n);
}

// Sum over the four lanes l, l^16, l^32, l^48 (the four column quarters of
// a row fragment); every lane receives the sum.
__device__ __forceinline__ float sum_quarters(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const uint32_t w = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ double sum_quarters(double x) {
  uint64_t u = (uint64_t)__double_as_longlong(x);
  auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
  auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  double y = __longlong_as_double((long long)((uint64_t)lo[0] | ((uint64_t)hi[0] << 32))) +
             __longlong_as_double((long long)((uint64_t)lo[1] | ((uint64_t)hi[1] << 32)));
  u = (uint64_t)__double_as_longlong(y);
  lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
  hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  return __longlong_as_double((long long)((uint64_t)lo[0] | ((uint64_t)hi[0] << 32))) +
         __longlong_as_double((long long)((uint64_t)lo[1] | ((uint64_t)hi[1] << 32)));
}

// ---------------------------------------------------------------------------
// Row-pair terms.  For a 16-row tile held as fragments (lane l: row l%16,
// column quarter l/16): float64 self dots <k,k>, <v,v> of every row and the
// cross dots <k,k'>, <v,v'> of every pair (rows 2q, 2q+1).  bf16: each
// v_dot2 gives two exact products summed in fp32, a partial covers 8
// elements and is accumulated in fp64; fp32: fp64 FMAs.  The cross dots use
// the partner lane's words (DPP).
// ---------------------------------------------------------------------------
// This lane's quarter of <k,k>.  Every place that forms a pair's scale h
// runs this same instruction sequence, so all of them see identical bits.
template <typename T, int D>
__device__ __forceinline__ double quarter_self_dot(const uint4* f) {
  constexpr int NW = Frag<T, D>::NV * 4;
  const uint32_t* w = reinterpret_cast<const uint32_t*>(f);
  double s = 0.0;
  if constexpr (Elem<T>::bytes == 2) {
#pragma unroll
    for (int c = 0; c < NW / 4; ++c) {
      float a = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bf16x2_t b = __builtin_bit_cast(bf16x2_t, w[4 * c + q]);
        a = __builtin_amdgcn_fdot2_f32_bf16(b, b, a, false);
      }
      s += (double)a;
    }
  } else {
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const double x = (double)__uint_as_float(w[i]);
      s = fma(x, x, s);
    }
  }
  return s;
}

// This lane's quarters of <v,v>, <k,k'> and <v,v'> (k', v' = partner row).
template <typename T, int D>
__device__ __forceinline__ void quarter_pair_dots(const uint4* fk, const uint4* fv, double& sv,
                                                  double& ck, double& cv) {
  constexpr int NW = Frag<T, D>::NV * 4;
  const uint32_t* wk = reinterpret_cast<const uint32_t*>(fk);
  const uint32_t* wv = reinterpret_cast<const uint32_t*>(fv);
  sv = 0.0; ck = 0.0; cv = 0.0;
  if constexpr (Elem<T>::bytes == 2) {
#pragma unroll
    for (int c = 0; c < NW / 4; ++c) {
      float a1 = 0.f, a2 = 0.f, a3 = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t xk = wk[4 * c + q], xv = wv[4 * c + q];
        const bf16x2_t bk = __builtin_bit_cast(bf16x2_t, xk);
        const bf16x2_t bv = __builtin_bit_cast(bf16x2_t, xv);
        const bf16x2_t pk = __builtin_bit_cast(bf16x2_t, from_partner(xk));
        const bf16x2_t pv = __builtin_bit_cast(bf16x2_t, from_partner(xv));
        a1 = __builtin_amdgcn_fdot2_f32_bf16(bv, bv, a1, false);
        a2 = __builtin_amdgcn_fdot2_f32_bf16(bk, pk, a2, false);
        a3 = __builtin_amdgcn_fdot2_f32_bf16(bv, pv, a3, false);
      }
      sv += (double)a1;
      ck += (double)a2;
      cv += (double)a3;
    }
  } else {
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const double xk = (double)__uint_as_float(wk[w]), xv = (double)__uint_as_float(wv[w]);
      const double pk = (double)__uint_as_float(from_partner(wk[w]));
      const double pv = (double)__uint_as_float(from_partner(wv[w]));
      sv = fma(xv, xv, sv);
      ck = fma(xk, pk, ck);
      cv = fma(xv, pv, cv);
    }
  }
}

// Scale exponent of a row: its diagonal exponent ||k||^2/sqrt(d) in base 2,
// rounded up to an integer (sk = <k,k>).  The scale of a pair is the larger
// of its two rows' values; that value is used wherever the pair's kappa
// values are scaled by 2^-h.  Integer scales keep every shifted scale
// (below) exact, and 2^(shifted - h) an exact power of two.
__device__ __forceinline__ float row_h2f(double sk, double inv_sqrt_d) {
  return (float)ceil((sk * inv_sqrt_d) * kLog2e);
}

// Extra scale of the scores of a block of rows i against pair p.  By
// Cauchy-Schwarz, <k_i,k_q>/sqrt(d) <= (e_i + e_q)/2 for the diagonal
// exponents e, so every cross exponent of a row of the block against a row q
// of pair p is at most (m_B + h_p)/2, m_B = the block's largest row scale.
// Scaling those kappa values by 2^-(h_p + shift) with
// shift = max(0, ceil((m_B - h_p)/2)) keeps every exponent <= 0 (no float32
// overflow, whatever the keys); the block's scores are then 2^-shift times
// their value at scale h_p, which the decisions undo exactly (ldexp) when
// they add the block's sums in float64.  Both arguments are integers, so
// every kernel that forms the shift gets the same value.
__device__ __forceinline__ float scale_shift(float mB, float h2) {
  return fmaxf(0.0f, ceilf(0.5f * (mB - h2)));
}
__device__ __forceinline__ float pair_h2f(float row_h2) {
  return fmaxf(row_h2, from_partner(row_h2));
}

// Row-pair terms of the 16-row tile: the row's scale exponent rh2 and its
// pair's h2f (above), and lbt = log of the RKHS distance b (Algorithm A.1)
// scaled by exp(-h/2).  The exponentials and the log are float32 (about 1e-7
// relative) on float64 arguments; the sums are float64.
template <typename T, int D>
__device__ __forceinline__ void frag_pair_terms(const uint4* fk, const uint4* fv, double vm2d,
                                                double inv_sqrt_d, float& rh2, float& h2f,
                                                float& lbt) {
  double sv, ck, cv;
  const double sk = sum_quarters(quarter_self_dot<T, D>(fk));
  quarter_pair_dots<T, D>(fk, fv, sv, ck, cv);
  sv = sum_quarters(sv);
  ck = sum_quarters(ck);
  cv = sum_quarters(cv);
  rh2 = row_h2f(sk, inv_sqrt_d);
  h2f = pair_h2f(rh2);
  const double svp = from_partner(sv);
  const double ex = sk * inv_sqrt_d, exp_ = from_partner(sk) * inv_sqrt_d, exx = ck * inv_sqrt_d;
  const double h2 = (double)h2f;
  const double t1 = (double)__builtin_amdgcn_exp2f((float)(ex * kLog2e - h2)) * (sv + vm2d);
  const double t2 = (double)__builtin_amdgcn_exp2f((float)(exp_ * kLog2e - h2)) * (svp + vm2d);
  const double t3 = (double)__builtin_amdgcn_exp2f((float)(exx * kLog2e - h2)) * (cv + vm2d);
  const double bt2 = t1 + t2 - 2.0 * t3;
  if (bt2 >= 1e-30) {
    lbt = (float)(0.5 * kLn2) * __builtin_amdgcn_logf((float)bt2);
  } else if (bt2 > 0.0) {
    // below float range: bt2 = m 2^e (hardware frexp), log2 bt2 = log2 m + e
    const float m = (float)__builtin_amdgcn_frexp_mant(bt2);
    const int e = __builtin_amdgcn_frexp_exp(bt2);
    lbt = (float)(0.5 * kLn2) * (__builtin_amdgcn_logf(m) + (float)e);
  } else {
    lbt = -INFINITY;
  }
}

// ---------------------------------------------------------------------------
// One Halve round: KH(1/2) (App. A, Algorithm A.1) on every bucket, in two
// launches.
//
// Bucket rows y_0..y_{N-1}; pair p = (y_{2p}, y_{2p+1}).  The score of
// Algorithm A.1, alpha_p = sum_{S2} f_p - sum_{S1} f_p, is the signed sum
//     alpha_p = sum_{i<p} sgn_i E(i,p),
//     E(i,p) = k(y'_i,y_p) - k(y_i,y_p) - k(y'_i,y'_p) + k(y_i,y'_p),
// sgn_i = -1 if pair i was swapped, else +1 (the same sum, regrouped by
// earlier pair).  E does not depend on any decision, so:
//   1. pair_scores_kernel evaluates every E(i,p), i < p, of every bucket at
//      once (MFMA Gram tiles + exp), plus the per-pair terms b_i and h_i;
//   2. halve_pass_kernel takes the decisions pair by pair, in blocks of BP
//      pairs: one wavefront decides a block (ballot on alpha < a (1 - 2u),
//      the exact form of "u < min(1, (1 - alpha/a)_+ / 2)"), then every
//      wavefront adds the block's signed scores to the later pairs' alpha.
// Scaling: alpha_p is accumulated at the scale 2^h_p (h_p as in pair_h2f),
// the scale of pair p's own terms b and a; the decision only depends on
// alpha/a, which a common factor leaves unchanged.  The scores of the rows of
// one 64-row block B against p are stored at the scale 2^(h_p + shift(B,p))
// (scale_shift), which keeps every float32 exponent of the Gram epilogue at
// or below 0 whatever the keys (kappa_att overflows float32 for large keys);
// the decisions multiply each block's signed sum by 2^shift (exact) when they
// add it to alpha.  E is float32; alpha accumulates in float64.
//
// Score layout of one bucket (BR = 16 RT rows = BP pairs per block, NT =
// ceil(N/16) row tiles): panel B (the block's BP pairs as i) holds every pair
// p of the column tiles jt = B RT .. NT-1 (8 pairs each) in runs of 16 pairs
// (8 in the last one when NT is odd), each run the block's pairs i = 0..15 as
// [p][16 i], then i = 16..31, so a pair's scores are two pieces of 64 bytes
// and a wave of the score kernel, which forms the scores of one half-block
// against 16 pairs at a time, writes 1 KiB in a row with one 16-byte store per
// lane.  Panel B starts panel_tiles(B) KiB into the bucket's array.
// ---------------------------------------------------------------------------
__host__ __device__ inline int64_t panel_tiles(int64_t B, int64_t NT, int64_t RT) {
  return B * NT - RT * B * (B - 1) / 2;
}

// Floats from i = 0..15 to i = 16..31 in the run of pairs 16 u .. (whole
// bucket; RT is even).
__host__ __device__ inline int half_run(int u, int NT) { return 2 * u + 1 < NT ? 256 : 128; }

// Work decomposition of pair_scores_kernel.  A group is BLOCKS = W / 2
// consecutive decision blocks (64 rows each) of one bucket; each of the
// group's W waves holds one half-block (32 rows) of it as MFMA fragments.
// W = 8 where a half-block's fragments take at most four words per lane and
// row tile (bf16, and fp32 up to d = 64: at most 128 registers per wave, four
// waves per SIMD, two workgroups per CU, whose latencies hide each other's),
// else W = 4 (fp32, d = 128).  Every launch of a bucket size uses the same W,
// so own and streamed chunks share their groups.  A workgroup handles one
// (bucket, group, chunk): the own chunk covers the group's own column tiles,
// which the owning waves write to LDS from their registers (so the bucket's
// rows are read from HBM once); a streamed chunk the column tiles after the
// group in one of the bucket's stretches of ch tiles of 32 rows (kScoreChunk,
// more in launches of many workgroups, fewer in launches of few), copied from
// global memory straight into LDS.
//   What bounds it: a 32-row tile takes the four waves of a SIMD 2700 cycles
// (s_memtime; 65536 rows x 32 slices), of which their 32 MFMAs each need 2048
// and their vector instructions (about 75 and 16 exponentials each) about
// 2200; a workgroup's row loads before the loop take about
// a quarter of its time.  Tiles of 32 columns with one barrier each, copied
// straight to LDS, and scores stored from the registers, against tiles of 16
// columns staged through registers with the scores turned in LDS: score
// launches of 65536 rows x 32 slices (d = 128, bf16) 3.40 -> 3.04 ms, of 16384
// rows x 64 slices 455 -> 383 us.
constexpr int kScoreChunk = 16;
constexpr int kScoreChunkMax = 32;
constexpr int64_t kScoreMinWorkgroups = 128;  // half the CUs
constexpr int64_t kScoreSets = 16;  // buckets of an XCD whose workgroups are interleaved
constexpr int64_t kScoreLongWorkgroups = 1024;         // four per CU
constexpr int kScoreRowsStaged = kScoreChunkMax * 32;  // rows of a streamed chunk, at most
// A score tile (8 column pairs x 32 row pairs) in the local kernel's LDS:
// column stride 36 floats, so that the decisions' reads of whole columns by
// consecutive lanes fall in different banks.
constexpr int kETileStride = 36;
constexpr int kETileLds = 8 * kETileStride;
constexpr size_t kCuLds = (size_t)160 << 10;  // LDS of a gfx950 CU

template <typename T, int D, int W>
struct ScoreShape {
  static constexpr int NV = Frag<T, D>::NV;
  static constexpr int BLOCKS = W / 2;         // decision blocks per group
  static constexpr int GT = 4 * BLOCKS;        // 16-row tiles per group
  static constexpr int CHUNKS = 2 * NV;        // 1 KB fragment chunks per 16-row tile (K, then V)
  // own chunks: a ring of 16-row tiles, one ahead of the other's readers
  static constexpr int OWN_STAGES = 3;
  static constexpr int OWN_RING = OWN_STAGES * CHUNKS * 1024;
  // streamed chunks: a ring of 32-row tiles; three where two workgroups per
  // CU have room for them, else two (and one more barrier per tile)
  static constexpr int STAGES = 6 * CHUNKS <= 48 ? 3 : 2;
  static constexpr int STAGE = 2 * CHUNKS * 1024;
  static constexpr int LPT = (2 * CHUNKS + W - 1) / W;  // copies per wave and tile
  // ring, scales of the column rows per block, column row indices, the
  // half-blocks' largest row scales
  static constexpr int lds_stream(int ch) {
    return STAGES * STAGE + ch * 32 * 4 * (BLOCKS + 1) + 2 * BLOCKS * 4;
  }
  // ring, pair scale exponents of the group's rows, the half-blocks' maxima
  static constexpr int LDS_OWN = OWN_RING + GT * 16 * 4 + 2 * BLOCKS * 4;
};

// Waves of every score launch and of the local kernel (see above).
template <typename T, int D>
constexpr int score_waves() {
  return Frag<T, D>::NV < 8 ? 8 : 4;
}

// The decisions of one block of 32 pairs (lane p: pair p of the block, with
// alpha = its score from earlier blocks, thr = a(1 - 2u), ef[i] = E(i, p)).
// One decision per step: the ballot of alpha < thr gives pair i's decision
// (swap: -E(i,.), else +E(i,.)), and every lane adds its signed score as one
// fused multiply-add by a uniform +-1 (the product is exact, so the result
// is the rounded sum alpha +- E).  Between the ballot and the add there are
// only scalar operations: the wave's instruction stream per decision is a
// handful of instructions, which sets this loop's speed.  No masking: lane
// p's alpha is read only at its own decision (step p), before any score of a
// pair i >= p has been added; decisions past the block's npb pairs are
// dropped.  With NEAR, en[i] = E(i, q) for a pair q of the next block, and
// near receives q's signed sum over the block (float32, in ascending i).
template <bool NEAR>
__device__ __forceinline__ uint32_t decide_block(double alpha, double thr, const float* ef,
                                                 const float* en, int npb, float& near) {
  // One step: compare (vector, into VCC), test bit i of VCC (scalar, into
  // SCC), select +-1.0 as a float64 pair on SCC, FMA; then, off the chain,
  // the float32 +-1 for the signed sum and the decision shifted into a
  // scalar mask (decision i at bit 31 - i: mask + mask + SCC).  Four
  // instructions on the chain against five to six for the same arithmetic
  // in compiled C++, which builds the sign with shifts and masks.
  uint32_t rmask = 0;
  const double one = 1.0, mone = -1.0;
#pragma unroll
  for (int i = 0; i < 32; ++i) {
    const double e = (double)ef[i];
    double sg;
    float sf;
    asm volatile(
        "v_cmp_lt_f64_e32 vcc, %[a], %[t]\n\t"
        "s_bitcmp1_b32 vcc_lo, %[i]\n\t"
        "s_cselect_b64 %[sg], %[mo], %[o]\n\t"
        "v_fmac_f64_e32 %[a], %[sg], %[e]\n\t"
        "s_cselect_b32 %[sf], -1.0, 1.0\n\t"
        "s_addc_u32 %[m], %[m], %[m]"
        : [a] "+v"(alpha), [sg] "=&s"(sg), [sf] "=&s"(sf), [m] "+s"(rmask)
        : [t] "v"(thr), [e] "v"(e), [i] "n"(i), [mo] "s"(mone), [o] "s"(one)
        : "vcc", "scc");
    if (NEAR) near = __builtin_fmaf(en[i], sf, near);
  }
  uint32_t smask = __builtin_bitreverse32(rmask);
  if (npb < 32) smask &= (1u << npb) - 1u;
  return smask;
}

// Threshold a(1 - 2u) of the pair of lane l < 32 in a block of npb pairs
// (Algorithm A.1: a = b b_max (1/2 + log(2N/delta))), in the log domain:
// lbt = log of the pair's scaled b (-inf if b = 0), h2 = its scale exponent
// (base 2), carry = log b_max over the bucket's earlier blocks (updated to
// include this block).  a = 0 (b = 0 or b_max = 0) gives p = 1/2: swap iff
// u < 1/2.  Lanes >= 32 return values of no meaning.
__device__ __forceinline__ double block_threshold(float lbt, float h2, float u, int npb, int lane,
                                                  double log_c, double& carry) {
  const bool act = lane < npb;
  const float lbtf = act ? lbt : -INFINITY;
  const float h2f = act ? h2 : 0.0f;
  const double half_h = (double)h2f * (0.5 * kLn2);
  const double pm = prefix_max32(act ? (double)lbtf + half_h : -INFINITY, lane);
  const double lbmax = fmax(carry, pm);
  double thr;
  if (!(lbtf > -INFINITY) || !(lbmax > -INFINITY))
    thr = (u < 0.5f) ? INFINITY : -INFINITY;
  else
    thr = exp_fast((double)lbtf + lbmax + log_c - half_h) * (1.0 - 2.0 * (double)u);
  carry = __shfl(lbmax, npb - 1);
  return thr;
}

// The largest |x| of this lane's words of RT row fragments, as the float's bits
// (magnitude bits order like magnitudes; bf16 pairs by packed 16-bit maxima).
template <typename T, int NV, int RT>
__device__ __forceinline__ uint32_t frag_absmax(const uint4 (&f)[RT][NV]) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  uint32_t m = 0u;
  u16x2 m2 = {0, 0};
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const uint32_t w[4] = {f[rt][v].x, f[rt][v].y, f[rt][v].z, f[rt][v].w};
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if constexpr (Elem<T>::bytes == 4) {
          m = max(m, w[c] & 0x7fffffffu);
        } else {
          const uint32_t x = w[c] & 0x7fff7fffu;
          m2 = __builtin_elementwise_max(m2, __builtin_bit_cast(u16x2, x));
        }
      }
    }
  return Elem<T>::bytes == 4 ? m : (uint32_t)max(m2[0], m2[1]) << 16;
}

// Row of a half-block's (or column tile's) 32 rows that lane m16 of 16-row
// tile rt holds.  MFMA outputs put rows 4g..4g+3 of a tile in lane group g;
// with this order the group holds eight consecutive rows over both tiles,
// i.e. four consecutive pairs, whose scores against one pair it can store as
// 16 bytes.  Pairs stay in adjacent lanes.
__device__ __forceinline__ int frag_row(int rt, int m16) {
  return 8 * (m16 >> 2) + 4 * rt + (m16 & 3);
}

// F of two 16 x 16 Gram tiles (rows of the wave's 16 pairs) at scale 2^-he.
__device__ __forceinline__ void score_kappa(const floatx4_t* gk, const floatx4_t* gv, float c2,
                                            float he, float* f) {
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    float kap[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      kap[e] = __builtin_amdgcn_exp2f(gk[rt][e] * c2 - he) * gv[rt][e];
    f[2 * rt] = kap[1] - kap[0];
    f[2 * rt + 1] = kap[3] - kap[2];
  }
}
// F = kappa(y'_i, x) - kappa(y_i, x) of the wave's 16 pairs i against the
// column rows x of one 16-row tile, whose fragments (CHUNKS KiB) start at st:
// lane (g, m16) gets f[k] for the pairs i = 4g + k against row m16, at the
// scale 2^-he of that row.  The column fragments are read word by word beside
// the MFMAs that use them.
template <typename T, int NV>
__device__ __forceinline__ void score_f(const uint4 (&Ak)[2][NV], const uint4 (&Av)[2][NV],
                                        const unsigned char* st, int lane, float vm2f, float c2,
                                        float he, float* f) {
  floatx4_t gk[2], gv[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    gk[rt] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
    gv[rt] = (floatx4_t){vm2f, vm2f, vm2f, vm2f};  // <v,v'> + v_max^2
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const uint4 bk = reinterpret_cast<const uint4*>(st + v * 1024)[lane];
    const uint4 bv = reinterpret_cast<const uint4*>(st + (NV + v) * 1024)[lane];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      gk[rt] = mma_word<T>(Ak[rt][v], bk, gk[rt]);
      gv[rt] = mma_word<T>(Av[rt][v], bv, gv[rt]);
    }
  }
  score_kappa(gk, gv, c2, he, f);
}
// E(i, p) = F(i, y_p) - F(i, y'_p) of the four pairs i = 4g + k: the even lane
// of a pair of lanes takes the pair p of the first 16-row column tile (f0),
// the odd lane that of the second (f1); each gets the partner's F of its p.
__device__ __forceinline__ float4 score_e(const float* f0, const float* f1, bool odd) {
  float e[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float mine = odd ? f1[k] : f0[k];
    const float other = from_partner(odd ? f0[k] : f1[k]);
    e[k] = odd ? other - mine : mine - other;
  }
  return make_float4(e[0], e[1], e[2], e[3]);
}

// LOCAL: the whole round for buckets of at most GT*16 rows in one launch:
// one workgroup per bucket computes the bucket's scores into LDS (its own
// chunk is the whole bucket), then takes the decisions from LDS with the same
// arithmetic as halve_pass_kernel (the scores never leave the CU).  Its rows are
// in order within a half-block (frag_row's order serves stores to the score
// array), so that a 16-row column tile past the bucket has nothing to do.
// STAGED: of those, every row tile in LDS at once (local_staged) instead of a
// ring: no barrier per tile, and a bucket of at most half the blocks spreads a
// half-block's tiles over several waves.  (An instantiation each: together they
// take 88 registers at d = 32, two workgroups per CU; apart 80, three.)  Local
// launches of float rows, d = 128, against rows in frag_row's order and both
// forms in one kernel: 16 buckets of 66 rows 25.5 -> 23.1 us, 600 of 16 rows 28.5
// -> 20.3; d = 32, 600 of 64 rows 19.2 -> 15.6.
// OWN_ONLY: a launch of own chunks only (an instantiation without the
// streamed code, which needs fewer registers).
template <typename T, int D, bool LOCAL, bool OWN_ONLY, int W, bool STAGED = false>
__global__ __launch_bounds__(64 * W)
__attribute__((amdgpu_waves_per_eu(LOCAL && Frag<T, D>::NV <= 2 ? 6 : W == 8 ? 4 : 2)))
void pair_scores_kernel(HalveArgs a) {
  using SS = ScoreShape<T, D, W>;
  constexpr int NV = SS::NV, NBW = SS::BLOCKS, GT = SS::GT, CH = SS::CHUNKS;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m16 = lane & 15;
  const int g = lane >> 4;

  const int N = a.N;
  const int P = N >> 1;
  const int NT = (N + 15) >> 4;
  const int NC = (N + 31) >> 5;  // 32-row column tiles
  const int nb = (N + 63) >> 6;
  // Workgroup -> (bucket, item).  Workgroups are dealt to the eight XCDs in
  // turn (linear id mod 8); XCD x takes buckets x, x+8, ... in sets of il
  // buckets whose workgroups are interleaved, set after set, so the
  // workgroups that share a bucket's rows share one L2 and run close
  // together.  A bucket's items go column chunk by column chunk, the last
  // first: the streamed chunks of every group before its last tile, which
  // read the same column rows one after the other, and beside them the own
  // chunks of the groups that start in it (their float64 pair terms keep the
  // vector ALU busy, the streamed chunks the matrix cores).
  int64_t bl;
  int grp = 0, kc = -1;  // kc < 0: the group's own chunk
  if constexpr (LOCAL) {
    bl = blockIdx.x;
  } else {
    constexpr int GC = GT / 2;
    const int64_t id = blockIdx.x;
    const int64_t k = id >> 3;
    const int64_t per = (int64_t)a.ipb * a.il;
    const int r_ = (int)(k % per);
    bl = (id & 7) + 8 * ((k / per) * a.il + r_ % a.il);
    if (bl >= a.nbk) return;
    int item = r_ / a.il;
    if (OWN_ONLY) {
      grp = item;
    } else {
      for (int c = (NC - 1) / a.ch; c >= 0; --c) {
        const int end = min((c + 1) * a.ch, NC);
        const int cnt = (end - 1) / GC;  // groups 0 .. cnt - 1 end before the chunk's last tile
        // groups g0 .. cnt start in the chunk
        const int g0 = a.own ? (c * a.ch + GC - 1) / GC : cnt + 1;
        const int n = cnt + max(0, cnt + 1 - g0);
        if (item < n) {
          const int j = item - g0;
          grp = j < 0 ? item : g0 + (j >> 1);
          if (j < 0 || (j & 1)) kc = c;
          break;
        }
        item -= n;
      }
    }
  }
  const int64_t bucket = a.b0 + bl;
  const int64_t s = bucket / a.G;
  const int64_t t = bucket % a.G;
  const int jg = grp * (GT / 2);  // the group's first column tile
  if (jg >= NC) return;
  const bool own = OWN_ONLY || kc < 0;
  const int jc0 = own ? jg : max(kc * a.ch, jg + GT / 2);
  const int ntile = min(own ? jg + GT / 2 : (kc + 1) * a.ch, NC) - jc0;

  const T* K = reinterpret_cast<const T*>(a.K) + s * a.ld * D;
  const T* V = reinterpret_cast<const T*>(a.V) + s * a.ld * D;
  const int32_t* rows_in = a.idx_in ? a.idx_in + s * in_stride(a) + t * (int64_t)N : nullptr;
  const int64_t row_base = t * (int64_t)N;
  // (LOCAL: possibly the largest entry of the bucket's own rows, formed below)
  const bool vmax_own = LOCAL && a.vmax_own;
  float vmax = vmax_own ? 0.0f : __uint_as_float(a.vmax_bits[a.vmax_per_bucket ? bucket : s]);
  const double inv_sqrt_d = 1.0 / sqrt((double)D);
  const float c2 = (float)(kLog2e * inv_sqrt_d);

  extern __shared__ __align__(16) unsigned char smem[];
  // own chunks: ring (STAGED: every row tile) | (LOCAL) every score tile of the
  // bucket | pair scales of the group's rows [GT * 16] | half-blocks' largest row
  // scales | (LOCAL) pair terms and the decisions' state
  static_assert(LOCAL || !STAGED, "only local launches stage every tile");
  float* s_e = reinterpret_cast<float*>(smem + (STAGED ? NT * CH * 1024 : SS::OWN_RING));
  float* s_h2 = s_e + (LOCAL ? (int)panel_tiles(nb, NT, 4) : 0) * kETileLds;
  float* s_mh = own ? s_h2 + GT * 16
                    : reinterpret_cast<float*>(smem + SS::STAGES * SS::STAGE) +
                          32 * a.ch * (NBW + 1);  // [2 * NBW]
  float* s_lbt = s_mh + 2 * NBW;  // LOCAL: pair terms [P] and [P]
  float* s_h2p = s_lbt + P;
  // LOCAL decisions: per block and lane the threshold and the bulk alpha of
  // the earlier blocks but the last ([NBW][64] each), and each block's mask
  double* s_thr = reinterpret_cast<double*>((reinterpret_cast<uintptr_t>(s_h2p + P) + 7) & ~(uintptr_t)7);
  double* s_alpha = s_thr + 64 * NBW;
  uint32_t* s_mask = reinterpret_cast<uint32_t*>(s_alpha + 64 * NBW);
  uint32_t* s_vm = s_mask + NBW;  // [W]: the waves' largest |V| entries
  // streamed chunks: ring | scale exponents of the column rows for each of
  // the group's blocks [NBW][32 ch] | column row indices
  float* s_he = reinterpret_cast<float*>(smem + SS::STAGES * SS::STAGE);
  int32_t* s_row = reinterpret_cast<int32_t*>(s_he + 32 * a.ch * NBW);

  // ---- this wave's half-block: rows, fragments and, in chunk 0, pair terms ----
  // STAGED with at most half the blocks: parts waves share a half-block (no more
  // than it has column tiles: a further wave would only read its rows again) and
  // take every parts-th tile; the later parts go through the half-blocks in
  // reverse, so that a SIMD (waves w and w + 4) gets a long and a short one.
  const int nhb = 2 * nb;
  const int parts = STAGED && 2 * nhb <= W ? min(W / nhb, NC) : 1;
  const int part = parts > 1 ? wave / nhb : 0;
  const int hbw = part & 1 ? nhb - 1 - wave % nhb : part ? wave % nhb : wave;  // local half-block
  const int lblk = hbw >> 1, half = hbw & 1;
  const int blk = grp * NBW + lblk;
  // (LOCAL: a half-block without rows takes no part either)
  const bool hb_ok = blk < nb && part < parts && (!LOCAL || hbw < NC);
  const bool odd = (m16 & 1) != 0;
  // Row of the half-block that lane m16 of 16-row tile rt holds.  LOCAL keeps its
  // scores in LDS and the rows in order: a 16-row column tile past the bucket
  // then has nothing to do.
  auto row_of = [&](int rt) { return LOCAL ? 16 * rt + m16 : frag_row(rt, m16); };
  // Streamed chunk: column row o of the chunk in fragment order (tile o / 32,
  // 16-row half o / 16 & 1, lane o % 16); this thread's are o = threadIdx.x +
  // 64 W k.  Their indices are requested first, then their scale exponents
  // from the per-row table, then the fragments, so that each wait covers only
  // what it needs.
  constexpr int RPT = (kScoreRowsStaged + 64 * W - 1) / (64 * W);
  int32_t ridx[RPT];
  float rh[RPT];
  if (!own) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int o = (int)threadIdx.x + k * 64 * W;
      const int j = min((jc0 + (o >> 5)) * 32 + frag_row((o >> 4) & 1, o & 15), N - 1);
      ridx[k] = o < 32 * ntile ? (rows_in ? rows_in[j] : (int32_t)(row_base + j)) : 0;
    }
  }
  int64_t ar[2];
  float arh[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    const int j = blk * 64 + half * 32 + row_of(rt);
    const bool valid = hb_ok && j < N;
    ar[rt] = valid ? (rows_in ? (int64_t)rows_in[j] : row_base + j) : -1;
    arh[rt] = (!own && valid) ? a.rowh2[s * a.n + ar[rt]] : 0.0f;
  }
  if (!own) {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int o = (int)threadIdx.x + k * 64 * W;
      rh[k] = o < 32 * ntile ? a.rowh2[s * a.n + ridx[k]] : 0.0f;
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  uint4 Ak[2][NV], Av[2][NV];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    const bool valid = ar[rt] >= 0;
    const int64_t r = valid ? ar[rt] : 0;
    load_frag<T, D>(K, r, g, valid, Ak[rt]);
    load_frag<T, D>(V, r, g, valid, Av[rt]);
  }
  if (own) {
    // Wait for the fragments here (vmcnt(0)).  Otherwise the first use sits
    // in the tile loop, whose wait then also covers the score stores of
    // earlier tiles on every iteration (stores count in vmcnt on this
    // architecture).
    __builtin_amdgcn_s_waitcnt(0x0F70);
    if constexpr (LOCAL) {
      if (vmax_own) {
        const uint32_t mv = wave_max_u(frag_absmax<T>(Av));
        if (lane == 0) s_vm[wave] = mv;
        __syncthreads();
        uint32_t m = 0u;
#pragma unroll
        for (int w = 0; w < W; ++w) m = max(m, s_vm[w]);
        vmax = __uint_as_float(m);
      }
    }
  }
  const float vm2f = vmax * vmax;
  const double vm2d = (double)vmax * (double)vmax;
  if (own) {
    const int64_t pb = s * (a.n_r >> 1) + t * (int64_t)P;
    if (hb_ok && part == 0) {
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) {
        float rh2, h2f, lbt;
        frag_pair_terms<T, D>(Ak[rt], Av[rt], vm2d, inv_sqrt_d, rh2, h2f, lbt);
        arh[rt] = ar[rt] >= 0 ? rh2 : 0.0f;
        const int j = blk * 64 + half * 32 + row_of(rt);
        if (g == 0) s_h2[(2 * hbw + rt) * 16 + m16] = j < N ? h2f : 0.0f;
        if (g == 0 && j < N && (j & 1) == 0) {
          if (LOCAL) {
            s_h2p[j >> 1] = h2f;
            s_lbt[j >> 1] = lbt;
          } else {
            a.h2[pb + (j >> 1)] = h2f;
            a.lbt[pb + (j >> 1)] = lbt;
          }
        }
        if (a.rowh2_write && g == 0 && j < N) a.rowh2[s * a.n + ar[rt]] = rh2;
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int o = (int)threadIdx.x + k * 64 * W;
      if (o < 32 * ntile) s_row[o] = ridx[k];
    }
  }
  // the largest row scale of each half-block (rows past the bucket: 0, and
  // every row scale is >= 0), published in LDS before the tile loop's first
  // barrier
  const float mh = wave_max_f(fmaxf(arh[0], arh[1]));
  if (lane == 0) s_mh[wave] = part == 0 ? mh : 0.0f;  // (later parts: half-blocks without rows)
  // This wave's scores against 16 pairs (one column tile jc) of its block's
  // panel: pair q of the tile (of this lane), then pairs i = 4g .. 4g+3 of
  // the half-block.  The panel ends after 8 pairs of the last tile when NT is
  // odd.
  const int q = LOCAL ? (odd ? 8 : 0) + (m16 >> 1)
                      : 4 * (m16 >> 2) + 2 * (odd ? 1 : 0) + ((m16 >> 1) & 1);
  float* ew = nullptr;
  if constexpr (!LOCAL)
    ew = a.E + (bl * a.e_tiles + panel_tiles(blk, NT, 4) - 4 * blk) * 256 + q * 16 + 4 * g;
  auto e_tile = [&](int jc) {
    return reinterpret_cast<float4*>(ew + (int64_t)jc * 512 + half * half_run(jc, NT));
  };
  auto in_panel = [&](int jc) { return 2 * jc + (q >> 3) < NT; };

  // LOCAL: the decisions of the bucket's P <= 32 NBW pairs from the scores
  // in LDS, with the arithmetic of halve_pass_kernel: block m's thresholds,
  // then alpha = the float32 signed sums of every earlier block added in
  // block order in float64, then decide_block.  Every wave of the workgroup
  // takes part.  First wave m < nblk forms block m's thresholds (the carry
  // of the earlier blocks is the largest of their pairs' values, which the
  // sequential scan carries forward).  Then block by block, one barrier
  // each: wave 0 adds the previous block's sums to the alpha the helpers
  // have built and decides the block; meanwhile waves 1.. add that previous
  // block's sums to the alpha of the blocks after this one, in block order,
  // so every alpha is the same float64 sum as one wave's.
  auto local_decisions = [&]() {
    const int nblk = (P + 31) / 32;
    const float* Ub = a.U + s * a.u_slice + bucket_u(a, t, P);
    uint8_t* trace = a.trace ? a.trace + s * a.u_slice + bucket_u(a, t, P) : nullptr;
    int32_t* out = a.idx_out + s * out_stride(a) + t * (int64_t)P;
    const int pl = lane & 31;
    auto pair_of = [&](int m) { return 32 * m + min(pl, min(32, P - 32 * m) - 1); };
    // block b's signed sums at pair gp's scale (gp in a later block)
    auto bulk = [&](int b, uint32_t mask, int gp) {
      const float* col = s_e + (panel_tiles(b, NT, 4) + (gp >> 3) - 4 * b) * kETileLds + (gp & 7) * kETileStride;
      float sum = 0.0f;
#pragma unroll
      for (int i = 0; i < 32; ++i) sum += ((mask >> i) & 1u) ? -col[i] : col[i];
      return ldexp((double)sum, (int)scale_shift(fmaxf(s_mh[2 * b], s_mh[2 * b + 1]), s_h2p[gp]));
    };
    if (wave < nblk) {
      const int m = wave;
      const int npb = min(32, P - 32 * m);
      const int gp = pair_of(m);
      double carry = -INFINITY;
      for (int b = 0; b < m; ++b) {  // earlier blocks are whole
        const int q = 32 * b + pl;
        carry = fmax(carry, (double)s_lbt[q] + (double)s_h2p[q] * (0.5 * kLn2));
      }
      carry = wave_max_d(carry);
      s_thr[64 * m + lane] = block_threshold(s_lbt[gp], s_h2p[gp], Ub[gp], npb, lane, a.log_c, carry);
    }
    for (int k = threadIdx.x; k < 64 * NBW; k += 64 * W) s_alpha[k] = 0.0;
    __syncthreads();
    uint32_t prev = 0u;  // wave 0: the last block's mask
    for (int m = 0; m < nblk; ++m) {
      if (wave == 0) {
        const int npb = min(32, P - 32 * m);
        const int gp = pair_of(m);
        double alpha = s_alpha[64 * m + lane];
        if (m > 0) alpha += bulk(m - 1, prev, gp);
        float ef[32];
        const float* oc = s_e + (panel_tiles(m, NT, 4) + (gp >> 3) - 4 * m) * kETileLds + (gp & 7) * kETileStride;
#pragma unroll
        for (int i = 0; i < 32; ++i) ef[i] = oc[i];
        float unused = 0.0f;
        // the block's own scores are at its shifted scale: decide there
        const int sh = (int)scale_shift(fmaxf(s_mh[2 * m], s_mh[2 * m + 1]), s_h2p[gp]);
        prev = decide_block<false>(ldexp(alpha, -sh), ldexp(s_thr[64 * m + lane], -sh), ef, ef, npb,
                                   unused);
        if (lane == 0) s_mask[m] = prev;
        const uint32_t bit = (prev >> pl) & 1u;
        if (lane < npb) {
          const int32_t r0 = rows_in ? rows_in[2 * gp] : (int32_t)(row_base + 2 * gp);
          const int32_t r1 = rows_in ? rows_in[2 * gp + 1] : (int32_t)(row_base + 2 * gp + 1);
          out[gp] = bit ? r1 : r0;
          if (trace) trace[gp] = (uint8_t)bit;
        }
      } else if (m > 0 && m + wave < nblk) {
        const int j = m + wave;  // a later block: block m - 1's sums join its alpha
        s_alpha[64 * j + lane] += bulk(m - 1, s_mask[m - 1], pair_of(j));
      }
      __syncthreads();
    }
  };

  __syncthreads();
  if (own) {
    const float mB = fmaxf(s_mh[2 * lblk], s_mh[2 * lblk + 1]);
    // the decision pass reads each block's largest row scale from here
    if (!LOCAL && (int)threadIdx.x < NBW && grp * NBW + (int)threadIdx.x < nb)
      a.mB[bucket * nb + grp * NBW + threadIdx.x] =
          fmaxf(s_mh[2 * threadIdx.x], s_mh[2 * threadIdx.x + 1]);
    // E of column tile jc (group-local tt) from its two halves' F
    auto put = [&](int tt, const float* fa, const float* fb) {
      const float4 e = score_e(fa, fb, odd);
      if constexpr (LOCAL) {
        if (in_panel(jc0 + tt)) {
          // (pairs 2 g, 2 g + 1 of either 16-row tile)
          float* col = s_e + (panel_tiles(blk, NT, 4) + 2 * (jc0 + tt) + (q >> 3) - 4 * blk) * kETileLds +
                       (q & 7) * kETileStride + 16 * half + 2 * g;
          *reinterpret_cast<float2*>(col) = make_float2(e.x, e.y);
          *reinterpret_cast<float2*>(col + 8) = make_float2(e.z, e.w);
        }
      } else if (in_panel(jc0 + tt)) {
        *e_tile(jc0 + tt) = e;
      }
    };
    // F against 16-row tile i, staged at st
    auto form = [&](int i, const unsigned char* st, float* f) {
      const float h2 = s_h2[i * 16 + m16];
      score_f<T, NV>(Ak, Av, st, lane, vm2f, c2, h2 + scale_shift(mB, h2), f);
    };
    // 16-row tile i (of the fragments of the wave holding half-block i / 2)
    // into a stage
    auto commit = [&](int i, int stage) {
      if (hbw == (i >> 1) && part == 0) {
        unsigned char* st = smem + stage * CH * 1024;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          reinterpret_cast<uint4*>(st + v * 1024)[lane] = (i & 1) ? Ak[1][v] : Ak[0][v];
          reinterpret_cast<uint4*>(st + (NV + v) * 1024)[lane] = (i & 1) ? Av[1][v] : Av[0][v];
        }
      }
    };
    // a half-block takes part from its block's diagonal on
    const int first = hb_ok ? 2 * lblk : GT;
    if constexpr (STAGED) {
      if (hb_ok) {
        commit(2 * hbw, 2 * hbw);
        if (2 * hbw + 1 < NT) commit(2 * hbw + 1, 2 * hbw + 1);
      }
      __syncthreads();
      for (int tt = first + part; tt < ntile; tt += parts) {
        float fa[4], fb[4];
        form(2 * tt, smem + 2 * tt * CH * 1024, fa);
        if (2 * tt + 1 < NT) {
          form(2 * tt + 1, smem + (2 * tt + 1) * CH * 1024, fb);
          put(tt, fa, fb);
        } else {
          put(tt, fa, fa);
        }
      }
      __syncthreads();
    } else {
      commit(0, 0);
      commit(1, 1);
      __syncthreads();
      float f0[4];
      // step i = 2 t + u (16-row tile u of column tile jc0 + t, stage st); tile
      // i + 2 is staged meanwhile
      auto step = [&](int tt, int u, int st) {
        const int i = 2 * tt + u;
        if (i + 2 < 2 * ntile) commit(i + 2, (st + 2) % 3);
        if (tt >= first) {
          float f[4];
          if (LOCAL && i >= NT) {  // a 16-row tile past the bucket
#pragma unroll
            for (int k = 0; k < 4; ++k) f[k] = 0.0f;
          } else {
            form(i, smem + st * CH * 1024, f);
          }
          if (u == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) f0[k] = f[k];
          } else {
            put(tt, f0, f);
          }
        }
        __syncthreads();
      };
      for (int t3 = 0; t3 < ntile; t3 += 3) {  // six steps: stages 0 1 2 0 1 2
        step(t3, 0, 0);
        step(t3, 1, 1);
        if (t3 + 1 < ntile) {  // uniform over the workgroup
          step(t3 + 1, 0, 2);
          step(t3 + 1, 1, 0);
        }
        if (t3 + 2 < ntile) {
          step(t3 + 2, 0, 1);
          step(t3 + 2, 1, 2);
        }
      }
    }
    if constexpr (LOCAL) local_decisions();
  } else if constexpr (!LOCAL && !OWN_ONLY) {
    // Copies of column tile tt into stage st: chunk c = (16-row half, K words
    // then V words), c = wave, wave + W, ...; lane l of word v brings the
    // row's 16-byte word 4 v + l / 16.
    constexpr int L = SS::LPT, NS = SS::STAGES;
    // The waits below count operations: a wave's copies of a tile must be L (or
    // none, in waves that copy nothing), its stores of a tile one.
    static_assert(2 * CH % W == 0 || 2 * CH < W, "as many copies in every wave that copies");
    const uint32_t ring = lds_offset(smem);
    auto issue = [&](int tt, int st) {
#pragma unroll
      for (int k = 0; k < L; ++k) {
        const int c = wave + k * W;
        if (2 * CH % W == 0 || c < 2 * CH) {
          const int w = c % CH;
          const int64_t row = s_row[tt * 32 + (c / CH) * 16 + m16];
          const T* src = (w < NV ? K : V) + row * D;
          copy16_to_lds(reinterpret_cast<const uint4*>(src) + 4 * (w % NV) + g,
                        ring + (uint32_t)(st * SS::STAGE + c * 1024));
        }
      }
    };
    issue(0, 0);
    if (ntile > 1) issue(1, 1);
    // scale exponent of every column row for every block of the group
    float mB[NBW];
#pragma unroll
    for (int b = 0; b < NBW; ++b) mB[b] = fmaxf(s_mh[2 * b], s_mh[2 * b + 1]);
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int o = (int)threadIdx.x + k * 64 * W;
      // 0 for rows past the bucket (whole pairs: N is even)
      const int j = (jc0 + (o >> 5)) * 32 + frag_row((o >> 4) & 1, o & 15);
      const float h2 = j < N ? pair_h2f(rh[k]) : 0.0f;
      if (o < 32 * ntile) {
#pragma unroll
        for (int b = 0; b < NBW; ++b) s_he[b * 32 * a.ch + o] = h2 + scale_shift(mB[b], h2);
      }
    }
    // fragments and the first two tiles (and what the compiler has in flight)
    __builtin_amdgcn_s_waitcnt(0x0F70);
    const float* he = s_he + lblk * 32 * a.ch + m16;
    int st = 0;
    for (int tt = 0; tt < ntile; ++tt) {
      // This wave's copies of tile tt are done once at most its newer
      // operations are outstanding: the stores of tiles tt - 2 and tt - 1 and
      // the copies of tile tt + 1 (none for the last tile).
      if (tt + 1 < ntile) wait_vmcnt<L + 2>(); else wait_vmcnt<2>();
      __syncthreads();
      if (NS == 3 && tt + 2 < ntile) issue(tt + 2, st == 0 ? 2 : st - 1);
      const unsigned char* sp = smem + st * SS::STAGE;
      float f0[4], f1[4];
      score_f<T, NV>(Ak, Av, sp, lane, vm2f, c2, he[tt * 32], f0);
      score_f<T, NV>(Ak, Av, sp + CH * 1024, lane, vm2f, c2, he[tt * 32 + 16], f1);
      if (NS == 2) {
        __syncthreads();  // every wave has read the stage
        if (tt + 2 < ntile) issue(tt + 2, st);
      }
      const float4 e = score_e(f0, f1, odd);
      if (in_panel(jc0 + tt)) *e_tile(jc0 + tt) = e;
      st = st == NS - 1 ? 0 : st + 1;
    }
  }
}

// Scores of a round of few buckets, one wave per unit of 32 rows x 32 columns:
// half-block hb of the bucket against column tile jc >= 2 (hb / 2).  A
// workgroup of the kernel above holds 256 rows and takes its tiles one after
// the other, so a launch of few buckets runs on few CUs and a workgroup's chain
// is its time; here every unit is a wave of its own with its rows read straight
// into registers (no LDS, no barrier), which reads a row N / 32 times but puts
// the launch on every CU.  Same products in the same order, same scales, same
// score layout.  The diagonal units write the pair terms (and row scales), the
// first unit of a block its largest row scale.  In the first round (no table of
// row scales yet) a unit forms the scales it needs itself.
constexpr int kUnitWaves = 4;
__host__ __device__ inline int64_t score_units(int64_t N) {
  const int64_t NC = (N + 31) / 32, nb = (N + 63) / 64;
  return 2 * (nb * NC - nb * (nb - 1));  // two half-blocks of every block, tiles 2 blk .. NC - 1
}

template <typename T, int D>
__global__ __launch_bounds__(64 * kUnitWaves) void score_units_kernel(HalveArgs a) {
  constexpr int NV = Frag<T, D>::NV;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m16 = lane & 15, g = lane >> 4;
  const bool odd = (m16 & 1) != 0;
  const int N = a.N, P = N >> 1;
  const int NT = (N + 15) >> 4, NC = (N + 31) >> 5, nb = (N + 63) >> 6;
  const int64_t id = (int64_t)blockIdx.x * kUnitWaves + wave;
  const int64_t bl = id / a.ipb;
  if (bl >= a.nbk) return;  // whole waves; no barrier below
  // unit -> block (its units: two half-blocks x tiles 2 blk .. NC - 1), half, tile
  int u = (int)(id - bl * a.ipb), blk = 0;
  while (u >= 2 * (NC - 2 * blk)) u -= 2 * (NC - 2 * blk++);
  const int half = u & 1, jc = 2 * blk + (u >> 1);
  const int64_t bucket = a.b0 + bl;
  const int64_t s = bucket / a.G, t = bucket % a.G;
  const T* K = reinterpret_cast<const T*>(a.K) + s * a.ld * D;
  const T* V = reinterpret_cast<const T*>(a.V) + s * a.ld * D;
  const int32_t* rows_in = a.idx_in ? a.idx_in + s * in_stride(a) + t * (int64_t)N : nullptr;
  const int64_t row_base = t * (int64_t)N;
  const bool table = !a.rowh2_write;
  const double inv_sqrt_d = 1.0 / sqrt((double)D);
  const float c2 = (float)(kLog2e * inv_sqrt_d);
  const bool diag = jc == 2 * blk + half;
  auto row_of = [&](int j) { return j < N ? (rows_in ? (int64_t)rows_in[j] : row_base + j) : -1; };

  // rows of the half-block, of the column tile and (for the block's largest
  // scale, without a table) of the block's other half
  int64_t ar[2], br[2], cr[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    ar[rt] = row_of(blk * 64 + half * 32 + frag_row(rt, m16));
    br[rt] = row_of(jc * 32 + frag_row(rt, m16));
    cr[rt] = table ? -1 : row_of(blk * 64 + (half ^ 1) * 32 + frag_row(rt, m16));
  }
  const int64_t tr = table ? row_of(blk * 64 + lane) : -1;
  const float vmax = __uint_as_float(a.vmax_bits[a.vmax_per_bucket ? bucket : s]);
  const float th = tr >= 0 ? a.rowh2[s * a.n + tr] : 0.0f;
  float bh[2];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) bh[rt] = table && br[rt] >= 0 ? a.rowh2[s * a.n + br[rt]] : 0.0f;
  uint4 Ak[2][NV], Av[2][NV], Bk[2][NV], Ck[2][NV];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt) {
    load_frag<T, D>(K, ar[rt] >= 0 ? ar[rt] : 0, g, ar[rt] >= 0, Ak[rt]);
    load_frag<T, D>(K, br[rt] >= 0 ? br[rt] : 0, g, br[rt] >= 0, Bk[rt]);
    load_frag<T, D>(V, ar[rt] >= 0 ? ar[rt] : 0, g, ar[rt] >= 0, Av[rt]);
    if (!table) load_frag<T, D>(K, cr[rt] >= 0 ? cr[rt] : 0, g, cr[rt] >= 0, Ck[rt]);
  }
  const float vm2f = vmax * vmax;
  const double vm2d = (double)vmax * (double)vmax;
  auto scale_of = [&](const uint4* f) {  // a row's scale exponent (0 for a row of zeros)
    return row_h2f(sum_quarters(quarter_self_dot<T, D>(f)), inv_sqrt_d);
  };
  // the block's largest row scale and the columns' pair scales
  float mB;
  if (table) {
    mB = wave_max_f(th);
  } else {
    float m = 0.0f;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) m = fmaxf(m, fmaxf(scale_of(Ak[rt]), scale_of(Ck[rt])));
    mB = wave_max_f(m);
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) bh[rt] = scale_of(Bk[rt]);
  }
  if (diag) {
    const int64_t pb = s * (a.n_r >> 1) + t * (int64_t)P;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      float rh2, h2f, lbt;
      frag_pair_terms<T, D>(Ak[rt], Av[rt], vm2d, inv_sqrt_d, rh2, h2f, lbt);
      const int j = jc * 32 + frag_row(rt, m16);
      if (g == 0 && j < N) {
        if ((j & 1) == 0) {
          a.h2[pb + (j >> 1)] = h2f;
          a.lbt[pb + (j >> 1)] = lbt;
        }
        if (a.rowh2_write) a.rowh2[s * a.n + ar[rt]] = rh2;
      }
    }
  }
  if (half == 0 && jc == 2 * blk && lane == 0) a.mB[bucket * nb + blk] = mB;

  floatx4_t gk[2][2], gv[2][2];  // [column half][row half]
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      gk[ct][rt] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
      gv[ct][rt] = (floatx4_t){vm2f, vm2f, vm2f, vm2f};  // <v,v'> + v_max^2
    }
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) gk[ct][rt] = mma_word<T>(Ak[rt][v], Bk[ct][v], gk[ct][rt]);
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
    load_frag<T, D>(V, br[ct] >= 0 ? br[ct] : 0, g, br[ct] >= 0, Bk[ct]);
#pragma unroll
  for (int ct = 0; ct < 2; ++ct)
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int rt = 0; rt < 2; ++rt) gv[ct][rt] = mma_word<T>(Av[rt][v], Bk[ct][v], gv[ct][rt]);
  float f[2][4];
#pragma unroll
  for (int ct = 0; ct < 2; ++ct) {
    const float h2 = pair_h2f(bh[ct]);
    score_kappa(gk[ct], gv[ct], c2, h2 + scale_shift(mB, h2), f[ct]);
  }
  const float4 e = score_e(f[0], f[1], odd);
  const int q = 4 * (m16 >> 2) + 2 * (odd ? 1 : 0) + ((m16 >> 1) & 1);
  if (2 * jc + (q >> 3) < NT)
    *reinterpret_cast<float4*>(a.E + (bl * a.e_tiles + panel_tiles(blk, NT, 4) - 4 * blk) * 256 +
                               (int64_t)jc * 512 + half * half_run(jc, NT) + q * 16 + 4 * g) = e;
}

// Buckets of at most 64 rows (one decision block of P <= 32 pairs): one
// wavefront per bucket, eight buckets per workgroup, the whole round in
// registers and a 4 KiB score tile in LDS.  The arithmetic is the local
// kernel's, step for step (the same Gram words in the same order, the same
// epilogue, scales, thresholds and decision loop), so both take the same
// decisions; what changes is the size of the work unit: the local kernel
// gives a whole workgroup of eight waves to a bucket, which at 16-64 rows
// leaves most of them idle (the prefill's Compress2 calls are 16-row buckets,
// 98304 of them in one launch).  RT = 16-row tiles per bucket (N <= 16 RT).
constexpr int kTinyWaves = 8;
constexpr int64_t kTinyMinBuckets = 1024;  // launches with fewer take the local kernel
constexpr int kTinyStride = 33;  // floats per score row in LDS (rows i, columns p)

template <typename T, int D, int RT>
__global__ __launch_bounds__(64 * kTinyWaves) void tiny_halve_kernel(HalveArgs a) {
  constexpr int NV = Frag<T, D>::NV;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int m16 = lane & 15, g = lane >> 4;
  const bool odd = (m16 & 1) != 0;
  const int64_t bl = (int64_t)blockIdx.x * kTinyWaves + wave;
  if (bl >= a.nbk) return;  // no barrier below: a wave without a bucket just ends
  const int N = a.N, P = N >> 1;
  const int64_t bucket = a.b0 + bl;
  const int64_t s = bucket / a.G, t = bucket % a.G;
  const T* K = reinterpret_cast<const T*>(a.K) + s * a.ld * D;
  const T* V = reinterpret_cast<const T*>(a.V) + s * a.ld * D;
  const int32_t* rows_in = a.idx_in ? a.idx_in + s * in_stride(a) + t * (int64_t)N : nullptr;
  const int64_t row_base = t * (int64_t)N;
  const double inv_sqrt_d = 1.0 / sqrt((double)D);
  const float c2 = (float)(kLog2e * inv_sqrt_d);

  __shared__ float s_e[kTinyWaves][32 * kTinyStride];  // E(i, p) at [i * stride + p]
  __shared__ float s_h2p[kTinyWaves][32], s_lbt[kTinyWaves][32];
  float* e = s_e[wave];

  // v_max of the slice (requested before the rows, whose wait then covers it:
  // 8192 buckets of 16 bf16 rows, d = 128, 18.4 -> 16.4 us) or, below, of the bucket's
  // own rows
  float vmax = a.vmax_own ? 0.0f : __uint_as_float(a.vmax_bits[a.vmax_per_bucket ? bucket : s]);
  // rows and their fragments
  int64_t ar[RT];
  uint4 Ak[RT][NV], Av[RT][NV];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int j = rt * 16 + m16;
    ar[rt] = j < N ? (rows_in ? (int64_t)rows_in[j] : row_base + j) : -1;
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const bool valid = ar[rt] >= 0;
    load_frag<T, D>(K, valid ? ar[rt] : 0, g, valid, Ak[rt]);
    load_frag<T, D>(V, valid ? ar[rt] : 0, g, valid, Av[rt]);
  }
  if (a.vmax_own) vmax = __uint_as_float(wave_max_u(frag_absmax<T>(Av)));
  const float vm2f = vmax * vmax;
  const double vm2d = (double)vmax * (double)vmax;
  // pair terms; the block's largest row scale (rows past the bucket: 0)
  float h2c[RT];
  float mB = 0.0f;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float rh2, h2f, lbt;
    frag_pair_terms<T, D>(Ak[rt], Av[rt], vm2d, inv_sqrt_d, rh2, h2f, lbt);
    const int j = rt * 16 + m16;
    h2c[rt] = j < N ? h2f : 0.0f;
    mB = fmaxf(mB, ar[rt] >= 0 ? rh2 : 0.0f);
    if (g == 0 && j < N && (j & 1) == 0) {
      s_h2p[wave][j >> 1] = h2f;
      s_lbt[wave][j >> 1] = lbt;
    }
    if (a.rowh2_write && g == 0 && j < N) a.rowh2[s * a.n + ar[rt]] = rh2;
  }
  mB = wave_max_f(mB);
  // scores of every row tile against every column tile from its diagonal on
#pragma unroll
  for (int ct = 0; ct < RT; ++ct) {
    const float he = h2c[ct] + scale_shift(mB, h2c[ct]);
#pragma unroll
    for (int rt = 0; rt <= ct; ++rt) {
      floatx4_t gk = {0.f, 0.f, 0.f, 0.f};
      floatx4_t gv = {vm2f, vm2f, vm2f, vm2f};  // <v,v'> + v_max^2
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        gk = mma_word<T>(Ak[rt][v], Ak[ct][v], gk);
        gv = mma_word<T>(Av[rt][v], Av[ct][v], gv);
      }
      float kap[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) kap[q] = __builtin_amdgcn_exp2f(gk[q] * c2 - he) * gv[q];
      const float F0 = kap[1] - kap[0];
      const float F1 = kap[3] - kap[2];
      const float mine = odd ? F1 : F0;
      const float other = from_partner(odd ? F0 : F1);
      // lane (g, m16): pair i = 8 rt + 2 g + odd of the row tile against pair
      // p = 8 ct + m16 / 2 of the column tile
      e[(8 * rt + 2 * g + (odd ? 1 : 0)) * kTinyStride + 8 * ct + (m16 >> 1)] =
          odd ? other - mine : mine - other;
    }
  }
  // the wave's score writes are complete before any lane reads another's
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  // the block's decisions (no earlier block: alpha starts at zero)
  const int pl = lane & 31;
  const int gp = min(pl, P - 1);
  const float* Ub = a.U + s * a.u_slice + bucket_u(a, t, P);
  double carry = -INFINITY;
  const double thr = block_threshold(s_lbt[wave][gp], s_h2p[wave][gp], Ub[gp], P, lane, a.log_c,
                                     carry);
  const int sh = (int)scale_shift(mB, s_h2p[wave][gp]);
  float ef[32];
#pragma unroll
  for (int i = 0; i < 32; ++i) ef[i] = e[i * kTinyStride + gp];
  float unused = 0.0f;
  const uint32_t smask = decide_block<false>(ldexp(0.0, -sh), ldexp(thr, -sh), ef, ef, P, unused);
  if (lane < P) {
    const uint32_t bit = (smask >> pl) & 1u;
    const int32_t r0 = rows_in ? rows_in[2 * gp] : (int32_t)(row_base + 2 * gp);
    const int32_t r1 = rows_in ? rows_in[2 * gp + 1] : (int32_t)(row_base + 2 * gp + 1);
    a.idx_out[s * out_stride(a) + t * (int64_t)P + gp] = bit ? r1 : r0;
    if (a.trace) a.trace[s * a.u_slice + bucket_u(a, t, P) + gp] = (uint8_t)bit;
  }
}

// Decision pass of one bucket per workgroup, in three roles that run ahead
// of or behind each other, synchronised by progress counters in LDS:
//  - wave 1 (fetcher) stages each block's inputs in a ring of FD + 1 LDS
//    slots, up to FD blocks ahead of the decider (FD blocks' loads in flight):
//    the block's own scores, the scores
//    against the next block's pairs, the row indices, and the thresholds
//    a(1 - 2u), which depend on no decision (the running maximum of b over
//    the bucket is carried from block to block);
//  - wave 0 (decider) takes the decisions of a block one after the other
//    (decide_block), with the block's signed scores against the next block's
//    pairs summed beside them, and publishes them;
//  - waves 2.. (bulk) add each decided block's scores to all pairs two or
//    more blocks later.  Each pair belongs to one bulk wave (64-pair chunks,
//    dealt round robin), which adds the blocks in order; the column chunks
//    are fetched ahead in one stream per wave, across blocks.
// alpha of a pair in block m = (contributions of blocks <= m-2, summed by the
// bulk waves in block order) + (contribution of block m-1, from the decider).
// The decider never waits on global memory.  Every wait is bounded.
constexpr int kSpinLimit = 1 << 16;

// Returns the last value read (>= target unless the spin limit ran out).  A
// wait that runs out sets the call's status word (status nullable): the
// kernel still ends normally, and the caller learns that this call's
// decisions cannot be trusted.
__device__ __forceinline__ int wait_at_least(const int* flag, int target, int32_t* status) {
  int v = 0;
  for (int it = 0; it < kSpinLimit; ++it) {
    v = __hip_atomic_load(flag, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (v >= target) return v;
    __builtin_amdgcn_s_sleep(1);
  }
  if (status) __hip_atomic_store(status, kStatusWaitExhausted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return v;
}
__device__ __forceinline__ void publish(int* flag, int value) {
  __hip_atomic_store(flag, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Decision helpers: rows 0 .. hand_row(c) of chunk c are added by helper
// workgroups, the last kPassHand rows before the chunk's first block by the
// bucket's own bulk waves (the hand-over then has kPassHand + 1 blocks of
// decisions to arrive before the decider needs the chunk).
constexpr int kPassHand = 10;
__device__ __forceinline__ int hand_row(int c) { return 2 * c - 2 - kPassHand; }
// Every access to the words the helpers share with the bucket's workgroup
// (decisions, flags, partials) is a read-modify-write atomic at agent scope:
// all of them are then performed at one place, the L2 of the XCD that runs
// the bucket's workgroup and its helpers (pass_helpers keeps them on one),
// so a flag seen there covers the partials written before it.
// The word reads and the flag updates are made once per wave (lane 0, the
// result broadcast): lanes that each update one flag would each see another
// old value.
__device__ __forceinline__ uint64_t shared_read(uint64_t* p) {
  uint64_t v = 0;
  if ((threadIdx.x & 63) == 0) v = __hip_atomic_fetch_add(p, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __shfl(v, 0);
}
__device__ __forceinline__ uint32_t shared_read(uint32_t* p) {
  uint32_t v = 0;
  if ((threadIdx.x & 63) == 0) v = __hip_atomic_fetch_add(p, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __shfl(v, 0);
}
// flag = max(flag, v); returns the old value (wave-uniform)
__device__ __forceinline__ uint32_t shared_max(uint32_t* p, uint32_t v) {
  uint32_t old = 0;
  if ((threadIdx.x & 63) == 0) old = __hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return __shfl(old, 0);
}
// per lane (each lane its own word)
__device__ __forceinline__ uint64_t shared_read_lane(uint64_t* p) {
  return __hip_atomic_fetch_add(p, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void shared_write(uint64_t* p, uint64_t v) {
  (void)__hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Tag of block m's decisions in a round: nonzero, distinct per round and block.
__device__ __forceinline__ uint32_t helper_tag(int32_t round_tag, int m) {
  return ((uint32_t)round_tag << 16) | (uint32_t)(m + 1);
}
// The decisions in a tagged word once its tag is `tag` (`w` read ahead;
// bounded wait at agent scope, like wait_at_least).
__device__ __forceinline__ uint32_t decided_mask(uint64_t* p, uint64_t w, uint32_t tag,
                                                 int32_t* status) {
  for (int it = 0; (uint32_t)(w >> 32) != tag; ++it) {
    if (it == kSpinLimit) {
      if (status) __hip_atomic_store(status, kStatusWaitExhausted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      break;
    }
    __builtin_amdgcn_s_sleep(2);
    w = shared_read(p);
  }
  return (uint32_t)w;
}
__device__ __forceinline__ void wait_flag(uint32_t* p, uint32_t value, int32_t* status) {
  uint32_t v = shared_read(p);
  for (int it = 0; v < value; ++it) {
    if (it == kSpinLimit) {
      if (status) __hip_atomic_store(status, kStatusWaitExhausted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      break;
    }
    __builtin_amdgcn_s_sleep(2);
    v = shared_read(p);
  }
}

template <int BW, int NCB, int FD>
struct PassLds {
  static constexpr int BP = 32, QW = 8, NSLOT = FD + 1;
  // alpha [P] f64 | decisions of every block [nblk] u32 | counters [16]:
  // last decided block, last staged block, rows completed by each bulk wave |
  // NSLOT input slots, each: thresholds [BP] f64, rows [2][BP] i32, own
  // scores [BP][CW] and next-block scores [BP][CW] 16-byte words | with
  // COAL, per bulk wave a column buffer [2][64][QW / 2] of 16-byte words, the
  // four words of a column's half permuted (PASS_TURN).  A slot's column of BP
  // scores is QW words plus one of padding (CW): reads of whole columns by
  // consecutive lanes then fall in different banks.  COAL: the bulk waves
  // load their chunks coalesced and transpose them in LDS (with six bulk
  // waves, on the largest buckets, the loads limit the bulk); else each lane
  // loads its own column: less LDS, and the decider's LDS accesses do not
  // queue behind the transposes.
  static constexpr int CW = QW + 1;
  static constexpr bool COAL = BW >= 6;
  static constexpr size_t kSlot = BP * 8 + 2 * BP * 4 + 2 * BP * CW * 16;
  static constexpr size_t kColBuf = COAL ? 64 * QW * 16 : 0;
  static_assert(2 + BW <= 16, "counter block");
  __host__ __device__ static constexpr size_t mask_off(int P) { return ((size_t)P * 8 + 15) & ~(size_t)15; }
  __host__ __device__ static constexpr size_t flag_off(int P) {
    return mask_off(P) + (((size_t)(P + BP - 1) / BP * 4 + 15) & ~(size_t)15);
  }
  __host__ __device__ static constexpr size_t slot_off(int P) { return flag_off(P) + 64; }
  __host__ __device__ static constexpr size_t colbuf_off(int P) { return slot_off(P) + NSLOT * kSlot; }
  // pair scale exponents [P] f32 | largest row scale of every block [nblk] f32
  __host__ __device__ static constexpr size_t h2_off(int P) { return colbuf_off(P) + BW * kColBuf; }
  __host__ __device__ static constexpr size_t mb_off(int P) { return h2_off(P) + (((size_t)P * 4 + 15) & ~(size_t)15); }
  // rows of bulk sums completed per 64-pair chunk [nch] i32
  __host__ __device__ static constexpr size_t chunk_off(int P) {
    return mb_off(P) + (((size_t)(P + BP - 1) / BP * 4 + 15) & ~(size_t)15);
  }
  __host__ __device__ static constexpr size_t bytes(int P) {
    return chunk_off(P) + (((size_t)(P + 63) / 64 * 4 + 15) & ~(size_t)15);
  }
};

template <int BW, int NCB, int FD, bool HELP>
__global__ __launch_bounds__(64 * (BW + 2)) void halve_pass_kernel(HalveArgs a) {
  using L = PassLds<BW, NCB, FD>;
  constexpr int RT = 4;
  constexpr int BR = 16 * RT;
  constexpr int BP = BR / 2;
  constexpr int TILE = 8 * BP;
  constexpr int QW = BP / 4;  // 16-byte words per score column
  static_assert(BP == L::BP && QW == L::QW, "layout");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // with helpers: workgroups [0, nbk) take their bucket's decisions, then
  // come helper 1 of every bucket, helper 2, ...
  const int HLP = HELP ? a.pass_h : 0;  // launches without helpers compile none of their code
  const int role = HLP ? (int)(blockIdx.x / a.nbk) : 0;
  const int64_t bl = HLP ? (int64_t)(blockIdx.x % a.nbk) : (int64_t)blockIdx.x;
  const int64_t bucket = a.b0 + bl;
  const int64_t s = bucket / a.G;
  const int64_t t = bucket % a.G;
  const int N = a.N;
  const int P = N >> 1;
  const int NT = (N + 15) >> 4;
  const int nblk = (P + BP - 1) / BP;
  const int nch = (P + 63) >> 6;
  const int32_t* rows_in = a.idx_in ? a.idx_in + s * in_stride(a) + t * (int64_t)N : nullptr;
  const int64_t row_base = t * (int64_t)N;
  const float* Ub = a.U + s * a.u_slice + bucket_u(a, t, P);
  uint8_t* trace = a.trace ? a.trace + s * a.u_slice + bucket_u(a, t, P) : nullptr;
  int32_t* out = a.idx_out + s * out_stride(a) + t * (int64_t)P;
  const int64_t pb = s * (a.n_r >> 1) + t * (int64_t)P;
  const float* Eb = a.E + bl * a.e_tiles * (int64_t)TILE;
  // a valid address for the row loads of round 0 (their values are replaced)
  const int32_t* rsrc = rows_in ? rows_in : reinterpret_cast<const int32_t*>(Ub);

  extern __shared__ __align__(16) unsigned char smem[];
  double* s_alpha = reinterpret_cast<double*>(smem);
  uint32_t* s_mask = reinterpret_cast<uint32_t*>(smem + L::mask_off(P));
  int* s_cnt = reinterpret_cast<int*>(smem + L::flag_off(P));  // decided, staged, rows[BW]
  auto slot = [&](int m) { return smem + L::slot_off(P) + (size_t)(m % L::NSLOT) * L::kSlot; };
  // slot fields
  auto sl_thr = [&](unsigned char* b) { return reinterpret_cast<double*>(b); };
  auto sl_rows = [&](unsigned char* b) { return reinterpret_cast<int32_t*>(b + BP * 8); };
  auto sl_own = [&](unsigned char* b) { return reinterpret_cast<u32x4*>(b + BP * 8 + 2 * BP * 4); };
  auto sl_next = [&](unsigned char* b) { return reinterpret_cast<u32x4*>(b + BP * 8 + 2 * BP * 4 + BP * L::CW * 16); };

  float* s_h2 = reinterpret_cast<float*>(smem + L::h2_off(P));
  float* s_mB = reinterpret_cast<float*>(smem + L::mb_off(P));
  for (int p = threadIdx.x; p < P; p += 64 * (BW + 2)) {
    s_alpha[p] = 0.0;
    s_h2[p] = a.h2[pb + p];
  }
  for (int b = threadIdx.x; b < nblk; b += 64 * (BW + 2)) s_mB[b] = a.mB[bucket * nblk + b];
  int* s_chunk = reinterpret_cast<int*>(smem + L::chunk_off(P));
  for (int c = threadIdx.x; c < (P + 63) / 64; c += 64 * (BW + 2)) s_chunk[c] = 0;
  if (threadIdx.x < 16) s_cnt[threadIdx.x] = threadIdx.x < 2 ? -1 : 0;
  __syncthreads();

  // Signed sum of a column's BP scores (decision bits in SMASK).
#define PASS_SUM(SRC, SMASK, SUM)                                                       \
  do {                                                                                 \
    SUM = 0.0f;                                                                        \
    _Pragma("unroll") for (int q_ = 0; q_ < QW; ++q_) {                                \
      const float e_[4] = {__uint_as_float(SRC[q_].x), __uint_as_float(SRC[q_].y),     \
                           __uint_as_float(SRC[q_].z), __uint_as_float(SRC[q_].w)};    \
      _Pragma("unroll") for (int c_ = 0; c_ < 4; ++c_)                                 \
        SUM += (((SMASK) >> (4 * q_ + c_)) & 1u) ? -e_[c_] : e_[c_];                   \
    }                                                                                  \
  } while (0)
  // 16-byte word Q_ (0..7: pairs i = 4 Q_ .. 4 Q_ + 3 of the block) of the
  // column of pair P_ in block B's score panel (P_ at or after block B).
#define PASS_WORD(B, P_, Q_)                                                            \
  reinterpret_cast<const u32x4*>(Eb + (panel_tiles(B, NT, RT) - (B) * RT) * TILE +     \
                                 (int64_t)((P_) >> 4) * 512 +                          \
                                 ((Q_) >> 2) * half_run((P_) >> 4, NT) + ((P_) & 15) * 16)[(Q_) & 3]
  // A chunk's 64 columns of one block with COAL: word lane % 4 of half k >> 2
  // of column 16 (k & 3) + lane / 4 per load (1 KiB in a row), turned through
  // the wave's column buffer.  Column c's word w of a half sits at slot
  // w ^ (c / 2 % 4) of the column's four: both the writes (two columns per
  // eight lanes) and the reads (one word of eight columns) hit every bank once.
#define PASS_LOAD(B, C0, K) \
  PASS_WORD(B, min((C0) + 16 * ((K) & 3) + lane / 4, P - 1), 4 * ((K) >> 2) + lane % 4)
#define PASS_TURN(BUF, SRC, COL)                                                        \
  do {                                                                                 \
    _Pragma("unroll") for (int k_ = 0; k_ < 8; ++k_) {                                 \
      const int c_ = 16 * (k_ & 3) + lane / 4;                                         \
      BUF[256 * (k_ >> 2) + 4 * c_ + (lane % 4 ^ ((c_ >> 1) & 3))] = SRC[k_];          \
    }                                                                                  \
    _Pragma("unroll") for (int q_ = 0; q_ < QW; ++q_)                                  \
      COL[q_] = BUF[256 * (q_ >> 2) + 4 * lane + ((q_ & 3) ^ ((lane >> 1) & 3))];      \
  } while (0)

  if (role > 0) {
    // ---- helper (waves 2..): the early rows of chunks ----
    // Helper wave hw of T = HLP BW takes chunks c = hw, hw + T, ... whose
    // hand_row(c) >= 0 and that it claims first (the bucket's workgroup
    // claims a chunk it reaches unclaimed and adds all its rows itself, so a
    // helper that is not resident delays nothing), rows 0 .. hand_row(c) in
    // order (a row's decisions from gmask, read with the row's scores and
    // checked by their tag), into a float64 alpha per pair in a register:
    // the same additions in the same order as the bucket's own bulk waves.
    // Then the chunk's partials go to galpha and, once written (vmcnt(0)),
    // its flag to "done".  All at agent scope: the bucket's workgroup runs on
    // another compute unit.
    if (wave < 2) return;
    const int T = HLP * BW;
    const int hw = (role - 1) * BW + (wave - 2);
    uint64_t* gm = a.gmask + bl * nblk;
    uint32_t* gf = a.gflag + bl * nch;
    const uint32_t claimed = 2u * (uint32_t)a.pass_tag, done = claimed + 1u;
    // next item to load: row fb of chunk fc
    int fc = hw, fb = 0;
    auto h_enter = [&]() {  // from fc on, the first chunk with rows that this wave claims
      while (fc < nch && (hand_row(fc) < 0 || shared_max(gf + fc, claimed) >= claimed)) fc += T;
      fb = 0;
    };
    h_enter();
    u32x4* colbuf = reinterpret_cast<u32x4*>(smem + L::colbuf_off(P) + (size_t)(wave - 2) * L::kColBuf);
    auto h_fetch = [&](u32x4* dst, uint64_t& word, int& ib, int& ic) {
      const bool live = fc < nch;
      ib = fb;
      ic = live ? fc : nch;
      if constexpr (L::COAL) {
#pragma unroll
        for (int k = 0; k < 8; ++k) dst[k] = PASS_LOAD(live ? fb : 0, live ? 64 * fc : 0, k);
      } else {
#pragma unroll
        for (int k = 0; k < 8; ++k)
          dst[k] = PASS_WORD(live ? fb : 0, live ? min(64 * fc + lane, P - 1) : 0, k);
      }
      // lane 0's read, broadcast only when the item is used: the wave does
      // not wait for it here
      word = 0;
      if (lane == 0)
        word = __hip_atomic_fetch_add(gm + (live ? fb : 0), (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (live && ++fb > hand_row(fc)) {
        fc += T;
        h_enter();
      }
    };
    u32x4 cb[NCB][8];
    uint64_t mw[NCB];
    int ib[NCB], ic[NCB];
#pragma unroll
    for (int r = 0; r < NCB; ++r) h_fetch(cb[r], mw[r], ib[r], ic[r]);
    bool more = ic[0] < nch;
    double acc = 0.0;
    while (more) {
#pragma unroll
      for (int r = 0; r < NCB; ++r) {
        const int b = ib[r], c = ic[r];
        const bool live = c < nch;
        const uint64_t w0 = __shfl(mw[r], 0);
        const uint32_t smask = live ? decided_mask(gm + b, w0, helper_tag(a.pass_tag, b), a.status) : 0u;
        u32x4 col[QW];
        if constexpr (L::COAL) {
          PASS_TURN(colbuf, cb[r], col);
        } else {
#pragma unroll
          for (int q = 0; q < QW; ++q) col[q] = cb[r][q];
        }
        float sum;
        PASS_SUM(col, smask, sum);
        const int p = 64 * c + lane;
        if (live && b == 0) acc = 0.0;
        if (live && p < P) acc += ldexp((double)sum, (int)scale_shift(s_mB[b], s_h2[p]));
        h_fetch(cb[r], mw[r], ib[r], ic[r]);
        if (live && b == hand_row(c)) {
          if (p < P) shared_write(a.galpha + bl * P + p, __double_as_longlong(acc));
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the partials are written
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          (void)shared_max(gf + c, done);
        }
        more = ic[(r + 1) % NCB] < nch;
      }
    }
  } else if (wave == 0) {
    // ---- decider ----
    __builtin_amdgcn_s_setprio(3);  // ahead of the bulk waves sharing its SIMD
    double anear = 0.0;             // this lane's pair: the previous block's contribution
    for (int m = 0; m < nblk; ++m) {
      const int npb = min(BP, P - m * BP);
      wait_at_least(&s_cnt[1], m, a.status);
      // the bulk sums of blocks 0 .. m-2 are in this block's pairs (64-pair
      // chunk m / 2)
      if (m >= 2) wait_at_least(&s_chunk[m >> 1], m - 1, a.status);
      unsigned char* sb = slot(m);
      const int p = lane;
      const int pl = lane & (BP - 1);
      const bool active = p < npb;
      const int gp = m * BP + p;
      const double alpha_in = s_alpha[min(gp, P - 1)] + anear;
      // the block's own scores are at its shifted scale: decide there
      const float mBm = s_mB[m];
      const int sh = (int)scale_shift(mBm, s_h2[min(gp, P - 1)]);
      const double thr = ldexp(sl_thr(sb)[pl], -sh);
      const int32_t r0 = sl_rows(sb)[pl], r1 = sl_rows(sb)[BP + pl];
      double alpha = ldexp(alpha_in, -sh);
      // this pair's scores against the block's pairs, held in registers
      // before the loop (the loop is the decider's critical path and must
      // not wait on LDS); widened to float64 inside the loop, off the chain.
      // No masking: lane p's alpha is read only at its own decision (step
      // p), before any score of a pair i >= p has been added to it, and the
      // decisions of lanes past the block's last pair are dropped below.
      // The same for this block's scores against the next block's pair pl:
      // their signed sum (the next block's contribution from this block) is
      // accumulated inside the loop, in the order of the bulk sums.
      float ef[BP], en[BP];
      const u32x4* oc = sl_own(sb) + pl * L::CW;
      const u32x4* nc = sl_next(sb) + pl * L::CW;
      u32x4 xs[QW], xn[QW];
#pragma unroll
      for (int q = 0; q < QW; ++q) {
        xs[q] = oc[q];
        xn[q] = nc[q];
      }
#pragma unroll
      for (int q = 0; q < QW; ++q)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          ef[4 * q + c] = __uint_as_float(xs[q][c]);
          en[4 * q + c] = __uint_as_float(xn[q][c]);
          asm volatile("" : "+v"(ef[4 * q + c]), "+v"(en[4 * q + c]));
        }
      __builtin_amdgcn_sched_barrier(0);
      float near = 0.0f;
      const uint32_t smask = decide_block<true>(alpha, thr, ef, en, npb, near);
      if (lane == 0) s_mask[m] = smask;
      publish(&s_cnt[0], m);
      if (HLP && lane == 0)
        shared_write(a.gmask + bl * nblk + m, ((uint64_t)helper_tag(a.pass_tag, m) << 32) | smask);
      const uint32_t bit = (smask >> (p & 31)) & 1u;
      if (active) {
        out[gp] = bit ? r1 : r0;
        if (trace) trace[gp] = (uint8_t)bit;
      }
      // the next block's pairs take this block's signed scores
      anear = ldexp((double)near, (int)scale_shift(mBm, s_h2[min((m + 1) * BP + pl, P - 1)]));
    }
  } else if (wave == 1) {
    // ---- fetcher: block m's inputs into slot m % NSLOT ----
    // Lane l fetches word l%QW of the columns of pairs l/QW + 8r (r < 4) of
    // the block's own scores and of its scores against the next block; lanes
    // < BP also the pair terms, uniform and rows of pair l.  Lanes past a
    // block's last pair read that pair's inputs.  The loads of FD blocks are in
    // flight.
    __builtin_amdgcn_s_setprio(2);
    u32x4 fo[FD][4], fn[FD][4];
    float flbt[FD], fh2[FD], fu[FD];
    int32_t fr0[FD], fr1[FD];
#define PASS_FETCH(B, K)                                                                \
  do {                                                                                 \
    const int b_ = min(B, nblk - 1);                                                   \
    const int npb_ = min(BP, P - b_ * BP);                                             \
    _Pragma("unroll") for (int r_ = 0; r_ < 4; ++r_) {                                 \
      const int pc_ = min(lane / QW + 8 * r_, npb_ - 1);                               \
      fo[K][r_] = PASS_WORD(b_, b_ * BP + pc_, lane % QW);                             \
      /* next block's pairs (the last block reads its own last column) */           \
      const int pn_ = min((b_ + 1) * BP + lane / QW + 8 * r_, P - 1);                  \
      fn[K][r_] = PASS_WORD(b_, pn_, lane % QW);                                       \
    }                                                                                  \
    const int gp_ = b_ * BP + min(lane & (BP - 1), npb_ - 1);                          \
    flbt[K] = a.lbt[pb + gp_];                                                         \
    fh2[K] = a.h2[pb + gp_];                                                           \
    fu[K] = Ub[gp_];                                                                   \
    fr0[K] = rsrc[rows_in ? 2 * gp_ : 0];                                              \
    fr1[K] = rsrc[rows_in ? 2 * gp_ + 1 : 0];                                          \
  } while (0)
    double carry = -INFINITY;  // log b_max over the pairs of earlier blocks
#define PASS_STAGE(B, K)                                                                \
  do {                                                                                 \
    const int npb_ = min(BP, P - (B) * BP);                                            \
    const double thr_ = block_threshold(flbt[K], fh2[K], fu[K], npb_, lane, a.log_c, carry); \
    /* slot B % NSLOT held block B - NSLOT, left once B - NSLOT + 1 is decided */    \
    if ((B) >= L::NSLOT) wait_at_least(&s_cnt[0], (B) - (L::NSLOT - 1), a.status);    \
    unsigned char* sb_ = slot(B);                                                      \
    _Pragma("unroll") for (int r_ = 0; r_ < 4; ++r_) {                                 \
      sl_own(sb_)[(lane / QW + 8 * r_) * L::CW + lane % QW] = fo[K][r_];               \
      sl_next(sb_)[(lane / QW + 8 * r_) * L::CW + lane % QW] = fn[K][r_];              \
    }                                                                                  \
    if (lane < BP) {                                                                   \
      sl_thr(sb_)[lane] = thr_;                                                        \
      sl_rows(sb_)[lane] = rows_in ? fr0[K] : (int32_t)(row_base + 2 * ((B) * BP + lane)); \
      sl_rows(sb_)[BP + lane] = rows_in ? fr1[K] : (int32_t)(row_base + 2 * ((B) * BP + lane) + 1); \
    }                                                                                  \
    publish(&s_cnt[1], B);                                                             \
  } while (0)
    // FD blocks' loads in flight: block m is staged from register set m % FD,
    // which then takes the loads of block m + FD
#pragma unroll
    for (int k = 0; k < FD; ++k) PASS_FETCH(k, k);
    for (int m = 0; m < nblk; m += FD) {
#pragma unroll
      for (int k = 0; k < FD; ++k) {
        if (m + k < nblk) PASS_STAGE(m + k, k);
        PASS_FETCH(m + k + FD, k);
      }
    }
#undef PASS_FETCH
#undef PASS_STAGE
  } else {
    // ---- bulk updates, blocks 0 .. nblk-3 ----
    // Bulk wave w = wave-2 owns the 64-pair chunks c = w, w + BW, ... of the
    // bucket (blocks 2c, 2c+1).  Row b (block b's signed scores) adds to the
    // pairs of block b+2 on, so chunk c takes rows 0 .. 2c-1 (row 2c-1 only
    // in its second block).  A wave's items are (row, chunk) chunk by chunk
    // in increasing c, rows in order within a chunk: items are taken in the
    // order the decider needs them (chunk c before block 2c), and a chunk's
    // progress does not wait for the wave's later chunks.  The items form one
    // stream held in an NCB-slot register ring (with each slot's row and
    // chunk): each consumed slot is refilled at once with the item NCB later,
    // so the loads run ahead whatever the decisions.  Lane l sums column l of
    // the chunk in ascending order (the order of the decider's sums); with
    // COAL the chunk is loaded 16 pairs x 16 scores (1 KiB in a row) per
    // instruction, 4 lanes to a pair, and turned through the wave's LDS column
    // buffer (PASS_LOAD, PASS_TURN).  After row b of chunk c the wave publishes b + 1 in
    // s_chunk[c] (rows completed).  With helpers, a chunk a helper has
    // claimed starts from the helper's partial alpha over rows
    // 0 .. hand_row(c) (taken from galpha once the chunk's flag is "done")
    // and continues with rows hand_row(c) + 1 on; a chunk the wave reaches
    // unclaimed it claims and takes whole.
    const int w = wave - 2;
    const int nrow = nblk - 2;
    auto last_row = [&](int c) { return min(2 * c - 1, nrow - 1); };  // < 0: no item
    uint32_t* gf = HLP ? a.gflag + bl * nch : nullptr;
    const uint32_t claimed = 2u * (uint32_t)a.pass_tag, done = claimed + 1u;
    // next item to load: row fb of chunk fc; fh: fb is the first row after
    // a helper's partial
    int fc = w, fb = 0;
    bool fh = false;
    auto enter = [&]() {  // from fc on, the first chunk with items
      while (fc < nch && last_row(fc) < 0) fc += BW;
      fb = 0;
      fh = false;
      if (fc < nch && HLP && hand_row(fc) >= 0 && shared_max(gf + fc, claimed) >= claimed) {
        fb = hand_row(fc) + 1;
        fh = true;
      }
    };
    enter();
    u32x4* colbuf = reinterpret_cast<u32x4*>(smem + L::colbuf_off(P) + (size_t)w * L::kColBuf);
    auto fetch_next = [&](u32x4* dst, int& ib, int& ic, bool& ih) {
      const bool live = fc < nch;
      ib = fb;
      ic = live ? fc : nch;
      ih = live && fh;
      fh = false;
      // COAL: as PASS_LOAD says; else word k of column lane (past the stream's
      // end: valid columns, never used)
      if constexpr (L::COAL) {
#pragma unroll
        for (int k = 0; k < 8; ++k) dst[k] = PASS_LOAD(live ? fb : 0, live ? 64 * fc : 0, k);
      } else {
        // One address for each half of the column: with the choice of block and
        // pair in every word's address, the last word's load became a branch
        // whose end waits for all loads in flight (8 and 24 buckets of 512 rows
        // 13.3 -> 15.7 us).
        const int b = live ? fb : 0, p = live ? min(64 * fc + lane, P - 1) : 0;
        const u32x4* lo = &PASS_WORD(b, p, 0);
        const u32x4* hi = lo + half_run(p >> 4, NT) / 4;
#pragma unroll
        for (int k = 0; k < 8; ++k) dst[k] = k < 4 ? lo[k] : hi[k - 4];
      }
      if (live && ++fb > last_row(fc)) {
        fc += BW;
        enter();
      }
    };
    u32x4 cb[NCB][8];
    int ib[NCB], ic[NCB];
    bool ih[NCB];
#pragma unroll
    for (int r = 0; r < NCB; ++r) fetch_next(cb[r], ib[r], ic[r], ih[r]);
    int decided = -1;  // last decided block seen
    bool more = ic[0] < nch;
    // Every slot of a turn is used and refilled whether or not the stream
    // has ended (loads past the end are of valid columns, nothing is added):
    // all paths then issue the same loads, and the wait before a slot's use
    // is for that slot's loads only.
    while (more) {
#pragma unroll
      for (int r = 0; r < NCB; ++r) {
        const int b = ib[r], c = ic[r];
        const bool live = c < nch;
        if (live && ih[r]) {
          // the helper's partial alpha of the chunk's pairs (rows 0 .. hand_row(c))
          wait_flag(gf + c, done, a.status);
          __atomic_signal_fence(__ATOMIC_SEQ_CST);
          const int pc = 64 * c + lane;
          if (pc < P)
            s_alpha[pc] = __longlong_as_double((long long)shared_read_lane(a.galpha + bl * P + pc));
          publish(&s_chunk[c], hand_row(c) + 1);
        }
        if (live && decided < b) decided = wait_at_least(&s_cnt[0], b, a.status);
        const uint32_t smask = s_mask[live ? b : 0];
        u32x4 col[QW];
        if constexpr (L::COAL) {
          PASS_TURN(colbuf, cb[r], col);
        } else {
#pragma unroll
          for (int q = 0; q < QW; ++q) col[q] = cb[r][q];
        }
        float sum;
        PASS_SUM(col, smask, sum);
        const int p = 64 * c + lane;
        if (live && p >= (b + 2) * BP && p < P)
          s_alpha[p] += ldexp((double)sum, (int)scale_shift(s_mB[b], s_h2[p]));
        fetch_next(cb[r], ib[r], ic[r], ih[r]);
        if (live) publish(&s_chunk[c], b + 1);
        more = ic[(r + 1) % NCB] < nch;
      }
    }
  }
#undef PASS_SUM
#undef PASS_WORD
#undef PASS_LOAD
#undef PASS_TURN
}

// Gram of rows [0,16) against rows [16,32) through the fragment path used by
// the score kernel (lane-layout self-check).
template <typename T, int D>
__global__ __launch_bounds__(64) void gram16_kernel(const T* rows, float* out) {
  constexpr int NV = Frag<T, D>::NV;
  const int lane = threadIdx.x, m16 = lane & 15, g = lane >> 4;
  uint4 a[NV], b[NV];
  load_frag<T, D>(rows, m16, g, true, a);
  load_frag<T, D>(rows, 16 + m16, g, true, b);
  floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
  acc = mma_rows<T, D>(a, b, acc);
#pragma unroll
  for (int i = 0; i < 4; ++i) out[(4 * g + i) * 16 + m16] = acc[i];
}

// Buckets interleaved per XCD in a score launch (at most the XCD's share):
// enough to stagger the workgroups' ends, few enough that their rows stay in
// the XCD's L2.
template <typename T, int D>
hipError_t launch_scores_td(const HalveArgs& a0, int64_t nbk, hipStream_t st) {
  if constexpr (Elem<T>::bytes == 4) {
    if (score_units(a0.N) * nbk <= unit_launch_max(D, a0.N, nbk, a0.rowh2_write != 0)) {
      HalveArgs u = a0;
      u.nbk = nbk;
      u.ipb = (int32_t)score_units(a0.N);
      const unsigned wgs = (unsigned)((u.ipb * nbk + kUnitWaves - 1) / kUnitWaves);
      hipLaunchKernelGGL((score_units_kernel<T, D>), dim3(wgs), dim3(64 * kUnitWaves), 0, st, u);
      return hipGetLastError();
    }
  }
  constexpr int WO = score_waves<T, D>();
  using SS = ScoreShape<T, D, WO>;  // own and streamed chunks share the groups
  auto kern_mixed = pair_scores_kernel<T, D, false, false, WO>;
  auto kern_own = pair_scores_kernel<T, D, false, true, WO>;
  const int64_t NC = (a0.N + 31) / 32;  // 32-row column tiles
  constexpr int64_t GC = SS::GT / 2;    // per group
  const int64_t groups = (NC + GC - 1) / GC;
  // streamed items of a bucket: for every column chunk, the groups before its
  // last tile
  auto streamed = [&](int64_t c) {
    int64_t w = 0;
    for (int64_t k = 0; k * c < NC; ++k) w += (std::min((k + 1) * c, NC) - 1) / GC;
    return w;
  };
  // Column tiles per streamed chunk (one workgroup's tiles, taken one after
  // the other): long chunks load a group's fragments once for more tiles, so
  // kScoreChunkMax in launches that keep four workgroups per CU, else
  // kScoreChunk, or fewer when the launch would leave the device short of
  // workgroups (a few large buckets: each chunk's tiles are then the launch's
  // critical path).  32 against 16 tiles: 2048 buckets of 1024 rows 875 -> 818
  // us, 128 of 4096 rows 724 -> 673 us; with 2.5 workgroups per CU (64 buckets
  // of 2048 rows) 98 -> 99 us, with 1.75 (64 of 1024 rows) 34 -> 40 us.
  HalveArgs a = a0;
  auto workgroups = [&](int64_t c) { return (groups + streamed(c)) * nbk; };
  if (workgroups(kScoreChunkMax) >= kScoreLongWorkgroups) a.ch = kScoreChunkMax;
  for (const int c : {8, 5, 3})
    if (workgroups(a.ch) <= kScoreMinWorkgroups && c < a.ch) a.ch = c;
  const int lds = std::max(SS::lds_stream(a.ch), (int)SS::LDS_OWN), lds_own = SS::LDS_OWN;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern_mixed),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  if (lds_own > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern_own),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_own);
    if (e != hipSuccess) return e;
  }
  // one workgroup per (bucket, item), buckets padded to a multiple of the
  // eight XCDs (the padding workgroups return at once)
  auto launch = [&](HalveArgs x, bool own, bool stream) {
    x.own = own;
    x.nbk = nbk;
    x.ipb = (int32_t)((own ? groups : 0) + (stream ? streamed(a.ch) : 0));
    x.il = (int32_t)std::min<int64_t>(kScoreSets, (nbk + 7) / 8);
    const int64_t per_xcd = ((nbk + 7) / 8 + x.il - 1) / x.il * x.il;
    const int64_t wgs = 8 * per_xcd * x.ipb;
    // a launch of own chunks only takes the own-only instantiation
    if (!stream)
      hipLaunchKernelGGL(kern_own, dim3((unsigned)wgs), dim3(64 * WO), lds_own, st, x);
    else
      hipLaunchKernelGGL(kern_mixed, dim3((unsigned)wgs), dim3(64 * WO), lds, st, x);
  };
  if (a.rowh2_write && NC > GC) {
    // the streamed chunks read the row scales the own chunks write: two launches
    launch(a, true, false);
    HalveArgs rest_a = a;
    rest_a.rowh2_write = 0;
    launch(rest_a, false, true);
    return hipGetLastError();
  }
  launch(a, true, NC > GC);
  return hipGetLastError();
}

// One wave per bucket for buckets of up to 16 RT rows whose fragments fit
// (RT NV <= 16 words per lane and operand).
template <typename T, int D>
constexpr int tiny_tiles() {
  return Frag<T, D>::NV <= 4 ? 4 : 16 / Frag<T, D>::NV;
}

template <typename T, int D, int RT>
hipError_t launch_tiny_td(const HalveArgs& a0, int64_t nbk, hipStream_t st) {
  HalveArgs a = a0;
  a.nbk = nbk;
  const unsigned wgs = (unsigned)((nbk + kTinyWaves - 1) / kTinyWaves);
  hipLaunchKernelGGL((tiny_halve_kernel<T, D, RT>), dim3(wgs), dim3(64 * kTinyWaves), 0, st, a);
  return hipGetLastError();
}

template <typename T, int D>
hipError_t launch_local_td(const HalveArgs& a0, int64_t nbk, hipStream_t st) {
  // with few buckets one wave per bucket leaves the GPU idle and a bucket's
  // latency (its tiles one after another) sets the time: the local kernel's
  // eight waves per bucket are faster there
  if (nbk >= kTinyMinBuckets) {
    if (a0.N <= 16) return launch_tiny_td<T, D, 1>(a0, nbk, st);
    if constexpr (tiny_tiles<T, D>() >= 2)
      if (a0.N <= 32) return launch_tiny_td<T, D, 2>(a0, nbk, st);
    if constexpr (tiny_tiles<T, D>() >= 4)
      if (a0.N <= 64) return launch_tiny_td<T, D, 4>(a0, nbk, st);
  }
  constexpr int WO = score_waves<T, D>();
  using SS = ScoreShape<T, D, WO>;
  const int64_t NT = (a0.N + 15) / 16, nb = (a0.N + 63) / 64, P = a0.N / 2;
  // ring, score tiles, pair scale exponents of the rows, half-block row scale
  // maxima, pair terms [2][P], then (8-byte aligned) the decisions' thresholds
  // and alphas [2][BLOCKS][64], masks and the waves' |V| maxima
  const size_t rest = (size_t)panel_tiles(nb, NT, 4) * kETileLds * 4 + SS::GT * 16 * 4 +
                      2 * SS::BLOCKS * 4 + 2 * P * 4 + 8 + 2 * 64 * SS::BLOCKS * 8 +
                      SS::BLOCKS * 4 + WO * 4;
  const size_t all = (size_t)NT * SS::CHUNKS * 1024 + rest;
  const bool staged = local_staged(nbk, (int64_t)all, SS::NV <= 2 ? 3 : 2);
  const size_t lds = staged ? all : SS::OWN_RING + rest;
  auto kern = staged ? pair_scores_kernel<T, D, true, true, WO, true>
                     : pair_scores_kernel<T, D, true, true, WO, false>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  HalveArgs a = a0;
  a.ch = kScoreChunk;
  a.e_tiles = 0;
  hipLaunchKernelGGL(kern, dim3((unsigned)nbk), dim3(64 * WO), lds, st, a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_local_t(int64_t d, const HalveArgs& a, int64_t nbk, hipStream_t st) {
  switch (d) {
    case 32: return launch_local_td<T, 32>(a, nbk, st);
    case 64: return launch_local_td<T, 64>(a, nbk, st);
    case 128: return launch_local_td<T, 128>(a, nbk, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
int64_t local_rows_t(int64_t d) {
  switch (d) {
    case 32: return ScoreShape<T, 32, score_waves<T, 32>()>::GT * 16;
    case 64: return ScoreShape<T, 64, score_waves<T, 64>()>::GT * 16;
    case 128: return ScoreShape<T, 128, score_waves<T, 128>()>::GT * 16;
    default: return 0;
  }
}

template <typename T>
hipError_t launch_scores_t(int64_t d, const HalveArgs& a, int64_t nbk, hipStream_t st) {
  switch (d) {
    case 32: return launch_scores_td<T, 32>(a, nbk, st);
    case 64: return launch_scores_td<T, 64>(a, nbk, st);
    case 128: return launch_scores_td<T, 128>(a, nbk, st);
    default: return hipErrorInvalidValue;
  }
}

// Helper workgroups per bucket for a decision launch: rounds of at most
// kHelperMaxBuckets buckets of at least kHelperMinPairs pairs (one launch
// per round: the tags of gmask and gflag are per round), as many as the
// device's compute units hold beside the buckets' own, at most kMaxHelpers.
int pass_helpers(const HalveArgs& a, int64_t nbk) {
  const int64_t P = a.N / 2;
  if (!a.gmask || !a.gflag || !a.galpha || a.pass_tag <= 0 || a.b0 != 0) return 0;
  // helper k of bucket b is workgroup k nbk + b: on the bucket's XCD (the
  // dispatcher deals workgroups to the 8 XCDs in turn) when 8 divides nbk
  if (P < kHelperMinPairs || P % 64 != 0 || nbk < 1 || nbk > kHelperMaxBuckets || nbk % 8 != 0) return 0;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return 0;
  const int64_t h = cus / nbk - 1;
  return (int)(h < 0 ? 0 : (h > kMaxHelpers ? kMaxHelpers : h));
}

template <int BW, int NCB, int FD, bool HELP>
hipError_t launch_pass_k(const HalveArgs& a, int64_t grid, hipStream_t st) {
  const size_t lds = PassLds<BW, NCB, FD>::bytes((int)(a.N / 2));
  auto kern = halve_pass_kernel<BW, NCB, FD, HELP>;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * (BW + 2)), lds, st, a);
  return hipGetLastError();
}

// HELPERS: the shape may take decision helpers (the large shapes).  Helpers
// follow the buckets' own workgroups in the grid; a helper waits only for
// decisions, and a bucket's workgroup never waits for a helper that has not
// claimed a chunk, so any residency order completes.
template <int BW, int NCB, int FD, bool HELPERS = false>
hipError_t launch_pass_w(const HalveArgs& a0, int64_t nbk, hipStream_t st) {
  HalveArgs a = a0;
  a.nbk = nbk;
  a.pass_h = 0;
  if constexpr (HELPERS) {
    a.pass_h = pass_helpers(a, nbk);
    if (a.pass_h > 0) return launch_pass_k<BW, NCB, FD, true>(a, nbk * (1 + a.pass_h), st);
  }
  return launch_pass_k<BW, NCB, FD, false>(a, nbk, st);
}

}  // namespace

int64_t halve_score_tiles(int64_t N) {
  const int64_t NT = (N + 15) / 16;
  const int64_t nb = (N + 63) / 64;
  return panel_tiles(nb, NT, 4);
}

size_t halve_score_bytes(int64_t N) {
  return (size_t)halve_score_tiles(N) * 8 * 32 * 4;  // tiles of 8 columns x 32 rows, float32
}

static HalveArgs with_layout(const HalveArgs& a0) {
  HalveArgs a = a0;
  a.ch = kScoreChunk;
  a.e_tiles = halve_score_tiles(a.N);
  return a;
}

hipError_t launch_scores(int dtype, int64_t d, const HalveArgs& a0, int64_t nbk, hipStream_t st) {
  const HalveArgs a = with_layout(a0);
  return dtype == 0 ? launch_scores_t<float>(d, a, nbk, st) : launch_scores_t<bf16_t>(d, a, nbk, st);
}

int64_t halve_local_rows(int dtype, int64_t d) {
  return dtype == 0 ? local_rows_t<float>(d) : local_rows_t<bf16_t>(d);
}

// Float buckets of 129 to 256 rows: one CU's float matrix rate sets the local
// launch's time (1 to 32 buckets of 256 rows, d = 64: 40 us), against 11.5 us
// for the units and 10 us for the decisions of 1 to 16 buckets.  From about 32
// buckets on the units' own work shows, and at 128 rows both take 20 us.
bool halve_spread(int dtype, int64_t N, int64_t nbk) {
  return dtype == 0 && N > 128 && nbk <= kSpreadMaxBuckets;
}

hipError_t launch_local(int dtype, int64_t d, const HalveArgs& a, int64_t nbk, hipStream_t st) {
  if (a.N > halve_local_rows(dtype, d)) return hipErrorInvalidValue;
  return dtype == 0 ? launch_local_t<float>(d, a, nbk, st) : launch_local_t<bf16_t>(d, a, nbk, st);
}

// Decision pass shapes <bulk waves, chunks in flight per bulk wave, blocks in
// flight in the fetcher> for small (<= 256 pairs after the first two
// blocks), medium (<= 512) and large buckets.  Large buckets run one per CU
// (64 buckets of 2048 rows on the long workload), where ten bulk waves keep
// the decider fed (round 3 there: 69.7 -> 58.7 us against six); a deeper
// fetcher gained nothing.
hipError_t launch_decide(const HalveArgs& a0, int64_t nbk, hipStream_t st) {
  const HalveArgs a = with_layout(a0);
  // bulk waves x prefetched chunks x 64 pairs should cover the pairs after
  // the first two blocks
  const int64_t later = a.N / 2 - 64;
  if (later <= 64) return launch_pass_w<1, 1, 2>(a, nbk, st);
  if (later <= 256) return launch_pass_w<2, 2, 2>(a, nbk, st);
  if (later <= 512) return launch_pass_w<6, 3, 2>(a, nbk, st);
  using Large = PassLds<10, 3, 2>;
  static_assert(Large::bytes(kMaxBucket / 2) <= kCuLds, "the large shape takes every bucket");
  return launch_pass_w<10, 3, 2, true>(a, nbk, st);
}

hipError_t launch_vmax(int dtype, const void* V, int64_t S, int64_t n, int64_t ld, int64_t d,
                       uint32_t* vmax_bits, hipStream_t st, int32_t* status, int64_t zero_words,
                       bool cleared) {
  const int64_t bytes = dtype == 0 ? 4 : 2;
  const int64_t words = n * d * bytes / 16, slice_words = ld * d * bytes / 16;
  if (!cleared) {
    const int64_t zw = zero_words > S ? zero_words : S;
    hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)((zw + 255) / 256)), dim3(256), 0, st,
                       vmax_bits, zw, status);
  }
  // 256 KiB of V per workgroup, less for small inputs so that the scan has
  // about 1024 workgroups (one workgroup reads ~40 GB/s; 64 of them made the
  // ViT-like workload's scan take 13 us), in whole turns of the 8-load loop
  constexpr int64_t kVmaxTurn = 8 * 256;
  int64_t per_block = 16384;
  const int64_t want = (words * S + 1023) / 1024;
  if (want < per_block) per_block = std::max<int64_t>(kVmaxTurn, (want + kVmaxTurn - 1) / kVmaxTurn * kVmaxTurn);
  const int64_t chunks = (words + per_block - 1) / per_block;
  dim3 grid((unsigned)chunks, (unsigned)S);
  if (dtype == 0)
    hipLaunchKernelGGL(vmax_kernel<float>, grid, dim3(256), 0, st, (const float*)V, words,
                       slice_words, per_block, vmax_bits);
  else
    hipLaunchKernelGGL(vmax_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)V, words,
                       slice_words, per_block, vmax_bits);
  return hipGetLastError();
}

hipError_t launch_subsample(int64_t S, int64_t n, int64_t n_kept, const float* U,
                            int64_t u_slice, int32_t* idx0, hipStream_t st, uint32_t* zero,
                            int64_t zero_words, int32_t* also) {
  dim3 grid((unsigned)((n_kept + 255) / 256), (unsigned)S);
  hipLaunchKernelGGL(subsample_kernel, grid, dim3(256), 0, st, n, n_kept, U, u_slice, idx0, zero,
                     zero_words, also);
  return hipGetLastError();
}

hipError_t launch_fill_rows(int64_t S, int64_t n_out, const int32_t* src, int64_t src_stride,
                            int32_t* dst, hipStream_t st) {
  dim3 grid((unsigned)((n_out + 255) / 256), (unsigned)S);
  hipLaunchKernelGGL(fill_rows_kernel, grid, dim3(256), 0, st, n_out, src, src_stride, dst);
  return hipGetLastError();
}

hipError_t launch_assemble(int64_t S, int64_t n, int64_t ns, int64_t n_out, int64_t nw,
                           const int32_t* src, int64_t src_stride, int32_t* dst, float* logw,
                           float lw_core, hipStream_t st) {
  const int64_t m = ns + n_out + nw;
  dim3 grid((unsigned)((m + 255) / 256), (unsigned)S);
  hipLaunchKernelGGL(assemble_kernel, grid, dim3(256), 0, st, n, ns, n_out, nw, src, src_stride,
                     dst, logw, lw_core);
  return hipGetLastError();
}

// Uniform halving: pair p of slice s keeps idx_in[2p+1] iff u < 1/2, else
// idx_in[2p] (idx_in null = the identity).  The pairs of a round are
// consecutive in the slice's current order, bucket after bucket, as are
// their draws, so the buckets need no separate treatment.
// With u_bucket, bucket t (N rows, N/2 pairs) draws from u_bucket[t] on; the
// lists are in_stride / out_stride apart per slice (0: packed).
__global__ void uniform_halve_kernel(int64_t n_r, const int32_t* idx_in, const float* U,
                                     int64_t u_slice, int64_t u_off, int32_t* idx_out,
                                     uint8_t* trace, int64_t N, const int64_t* u_bucket,
                                     int64_t in_stride, int64_t out_stride) {
  const int64_t s = blockIdx.y;
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t P = n_r >> 1;
  if (p >= P) return;
  const int64_t ui =
      s * u_slice + (u_bucket ? u_bucket[p / (N >> 1)] + p % (N >> 1) : u_off + p);
  const int swap = U[ui] < 0.5f;
  const int64_t j = 2 * p + swap;
  idx_out[s * (out_stride ? out_stride : P) + p] =
      idx_in ? idx_in[s * (in_stride ? in_stride : n_r) + j] : (int32_t)j;
  if (trace) trace[ui] = (uint8_t)swap;
}

hipError_t launch_uniform_halve(int64_t S, int64_t n_r, const int32_t* idx_in, const float* U,
                                int64_t u_slice, int64_t u_off, int32_t* idx_out,
                                uint8_t* trace, hipStream_t st, int64_t N,
                                const int64_t* u_bucket, int64_t in_stride, int64_t out_stride) {
  const int64_t P = n_r / 2;
  dim3 grid((unsigned)((P + 255) / 256), (unsigned)S);
  hipLaunchKernelGGL(uniform_halve_kernel, grid, dim3(256), 0, st, n_r, idx_in, U, u_slice,
                     u_off, idx_out, trace, N > 0 ? N : n_r, u_bucket, in_stride, out_stride);
  return hipGetLastError();
}

// Every round of uniform halving of one slice per workgroup, the slice's
// indices held in LDS (n_kept <= kUniformFusedRows): in round r each thread
// reads its pairs' kept indices, the workgroup synchronises, and the halved
// list is written back in place.
constexpr int kUniformThreads = 1024;
constexpr int64_t kUniformFusedRows = 32768;
__global__ __launch_bounds__(kUniformThreads) void uniform_compress_kernel(
    int64_t n_kept, int32_t L, const int32_t* idx0, const float* U, int64_t u_slice,
    int64_t u_off0, int32_t* idx_out, int64_t n_out, uint8_t* trace) {
  extern __shared__ int32_t s_idx[];
  constexpr int PPT = (int)(kUniformFusedRows / 2 / kUniformThreads);  // pairs per thread, round 0
  const int64_t s = blockIdx.x;
  const int tid = threadIdx.x;
  for (int64_t i = tid; i < n_kept; i += kUniformThreads)
    s_idx[i] = idx0 ? idx0[s * n_kept + i] : (int32_t)i;
  __syncthreads();
  int64_t n_r = n_kept, u_off = u_off0;
  for (int32_t r = 0; r < L; ++r) {
    const int64_t P = n_r >> 1;
    int32_t keep[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      const int64_t p = tid + (int64_t)k * kUniformThreads;
      if (p < P) {
        const int64_t ui = s * u_slice + u_off + p;
        const int swap = U[ui] < 0.5f;
        keep[k] = s_idx[2 * p + swap];
        if (trace) trace[ui] = (uint8_t)swap;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
      const int64_t p = tid + (int64_t)k * kUniformThreads;
      if (p < P) s_idx[p] = keep[k];
    }
    __syncthreads();
    n_r = P;
    u_off += P;
  }
  for (int64_t i = tid; i < n_out; i += kUniformThreads) idx_out[s * n_out + i] = s_idx[i];
}

bool uniform_fused_ok(int64_t n_kept) { return n_kept <= kUniformFusedRows; }

hipError_t launch_uniform_compress(int64_t S, int64_t n_kept, int32_t L, const int32_t* idx0,
                                   const float* U, int64_t u_slice, int64_t u_off0,
                                   int32_t* idx_out, int64_t n_out, uint8_t* trace,
                                   hipStream_t st) {
  if (!uniform_fused_ok(n_kept)) return hipErrorInvalidValue;
  const size_t lds = (size_t)n_kept * 4;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(uniform_compress_kernel),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(uniform_compress_kernel, dim3((unsigned)S), dim3(kUniformThreads), lds, st,
                     n_kept, L, idx0, U, u_slice, u_off0, idx_out, n_out, trace);
  return hipGetLastError();
}

hipError_t launch_zero_status(int32_t* status, hipStream_t st) {
  hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(64), 0, st, nullptr, 0, status);
  return hipGetLastError();
}

hipError_t launch_zero_u8(uint8_t* p, int64_t count, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_u8_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, p,
                     count);
  return hipGetLastError();
}

hipError_t launch_gram16(int dtype, int64_t d, const void* rows, float* out, hipStream_t st) {
  dim3 grid(1), block(64);
#define THIN_G16(T, DD) \
  hipLaunchKernelGGL((gram16_kernel<T, DD>), grid, block, 0, st, (const T*)rows, out)
  if (dtype == 0) {
    if (d == 32) THIN_G16(float, 32);
    else if (d == 64) THIN_G16(float, 64);
    else if (d == 128) THIN_G16(float, 128);
    else return hipErrorInvalidValue;
  } else {
    if (d == 32) THIN_G16(bf16_t, 32);
    else if (d == 64) THIN_G16(bf16_t, 64);
    else if (d == 128) THIN_G16(bf16_t, 128);
    else return hipErrorInvalidValue;
  }
#undef THIN_G16
  return hipGetLastError();
}

}  // namespace thin
