// Coreset attention on gfx950: every query of a slice attends over the n_out
// rows idx[s, :] of that slice's K/V (Sec. 2.1 eq. unmaskedatt on the
// coreset; eq. def:att_approx with equal weights, which cancel).  The
// weighted variant (W) gives key j the weight exp(logw[s, j]): its raw score
// <q, k_j> gets the bias sqrt(d) * logw[s, j], staged in LDS beside the keys
// (a key past n_out or of weight 0 has bias -inf, which also masks it).
//
// One workgroup = 4 waves = 64 or 128 queries of one slice.  The coreset is walked
// in chunks of 64 keys staged in LDS (gathered through idx); scores S^T =
// K_I Q^T come from 16x16 MFMA tiles (keys x queries), the softmax is online
// in float32, and O^T += V_I^T P^T reuses the score tile's register layout as
// the B operand.  For bf16 inputs the weights P (float32) enter the bf16 P.V
// MFMA as two terms, P = hi + lo with hi = bf16(P), lo = bf16(P - hi), so the
// product keeps about 16 significant bits of P instead of 8.
#include <math.h>

#include <algorithm>

#include "attn_plan.hpp"
#include "common.hpp"
#include "launch.hpp"

namespace thin {

namespace {

constexpr int KC = 64;   // keys per chunk
constexpr int WAVES = 4;
constexpr int QPB = 128;  // points per prefill tile
// The prefill kernel takes 128 queries per workgroup as 8 waves of
// one 16-query tile: half the registers per wave (128, four waves per SIMD,
// two workgroups per CU), so a chunk's gathers, barriers and arithmetic of
// one workgroup overlap the other's (65536 points x 32 slices: 8.19 -> 5.76
// ms against 4 waves of two tiles).
constexpr int PF_QT = 1;
constexpr int PF_WAVES = 8;
static_assert(16 * PF_QT * PF_WAVES == QPB, "prefill tiles of QPB points");
constexpr double kLog2e = 1.44269504088896340736;

template <typename T, int D>
struct AttnLds {
  // K chunk, row-major, padded by 16 bytes per row.
  static constexpr int k_stride = D * Elem<T>::bytes + 16;
  // V chunk: bf16 is stored transposed [D][KC] (+8 elements pad), fp32 row-major.
  static constexpr int v_stride = Elem<T>::bytes == 2 ? (KC + 8) * 2 : D * 4 + 16;
  static constexpr int v_rows = Elem<T>::bytes == 2 ? D : KC;
  static constexpr int bytes = KC * k_stride + v_rows * v_stride + KC * 4;
};

template <typename TO>
__device__ __forceinline__ void store4(TO* p, float a, float b, float c, float d);

template <>
__device__ __forceinline__ void store4<float>(float* p, float a, float b, float c, float d) {
  *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}
template <>
__device__ __forceinline__ void store4<bf16_t>(bf16_t* p, float a, float b, float c, float d) {
  typedef __bf16 b2 __attribute__((ext_vector_type(2)));
  const b2 lo = {(__bf16)a, (__bf16)b}, hi = {(__bf16)c, (__bf16)d};
  *reinterpret_cast<uint2*>(p) = make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
}

template <typename T, int D, typename TO, bool W, int QT, bool ONE>
__global__ __launch_bounds__(64 * WAVES) void coreset_attn_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
    const int32_t* __restrict__ idx, const float* __restrict__ logw, int64_t n, int64_t n_q,
    int n_out, int extra, TO* __restrict__ O) {
  constexpr int NV = Frag<T, D>::NV;
  constexpr bool BF = Elem<T>::bytes == 2;
  using L = AttnLds<T, D>;
  __shared__ __align__(16) unsigned char lds[L::bytes];
  unsigned char* sK = lds;
  unsigned char* sV = lds + KC * L::k_stride;
  float* sB = reinterpret_cast<float*>(sV + L::v_rows * L::v_stride);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m16 = lane & 15, g = lane >> 4;
  // the slice, and which of its workgroups this is; ONE with `extra` workgroups
  // per slice that have a block more than the others: dealt so that those come first
  int64_t s = blockIdx.y;
  int64_t first = blockIdx.x + (int64_t)gridDim.x * blockIdx.z;
  if (ONE && extra) {
    const Share sh = share_of(blockIdx.x + gridDim.x * blockIdx.y, gridDim.y, gridDim.x, extra);
    s = sh.slice;
    first = sh.part;
  }
  const float* Ws = W ? logw + s * (int64_t)n_out : nullptr;
  const float sqrt_d = (float)sqrt((double)D);
  const T* Ks = K + s * n * D;
  const T* Vs = V + s * n * D;
  const int32_t* Is = idx + s * (int64_t)n_out;
  const float c2 = (float)(kLog2e / sqrt((double)D));

  constexpr int WPR = D * Elem<T>::bytes / 16;  // 16-byte words per row
  // ONE: a coreset of one chunk, staged for the first of the workgroup's blocks
  // of queries (as many apart as there are workgroups) and kept; else one block.
  const int64_t nqb = (n_q + 16 * QT * WAVES - 1) / (16 * QT * WAVES);
  for (int64_t qb = first; qb < nqb; qb += (int64_t)gridDim.x * gridDim.z) {
    const int64_t q0 = qb * (16 * QT * WAVES) + wave * 16 * QT;
    uint4 Bq[QT][NV];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      const int64_t q = q0 + qt * 16 + m16;
      load_frag<T, D>(Q + s * n_q * D, q, g, q < n_q, Bq[qt]);
    }

    float mrun[QT], lrun[QT];
    floatx4_t acc[QT][D / 16];
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      mrun[qt] = -INFINITY;
      lrun[qt] = 0.0f;
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) acc[qt][dt] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
    }

    for (int c0 = 0; c0 < n_out; c0 += KC) {
      const int kc = min(KC, n_out - c0);
      if (!ONE || qb == first) {
        __syncthreads();
        if (W && threadIdx.x < KC)
          sB[threadIdx.x] = (int)threadIdx.x < kc ? Ws[c0 + threadIdx.x] * sqrt_d : -INFINITY;
        for (int w = threadIdx.x; w < KC * WPR; w += 64 * WAVES) {
          const int key = w / WPR, wi = w % WPR;
          uint4 kw = make_uint4(0, 0, 0, 0), vw = make_uint4(0, 0, 0, 0);
          if (key < kc) {
            int64_t r = Is[c0 + key];
            r = r < 0 ? 0 : (r >= n ? n - 1 : r);
            kw = reinterpret_cast<const uint4*>(Ks + r * D)[wi];
            vw = reinterpret_cast<const uint4*>(Vs + r * D)[wi];
          }
          *reinterpret_cast<uint4*>(sK + key * L::k_stride + wi * 16) = kw;
          if (BF) {
            const uint16_t* e = reinterpret_cast<const uint16_t*>(&vw);
#pragma unroll
            for (int j = 0; j < 8; ++j)
              *reinterpret_cast<uint16_t*>(sV + (wi * 8 + j) * L::v_stride + key * 2) = e[j];
          } else {
            *reinterpret_cast<uint4*>(sV + key * L::v_stride + wi * 16) = vw;
          }
        }
        __syncthreads();
      }
      if (q0 >= n_q) continue;  // (whole waves; no barrier below)

      uint4 Ak[4][NV];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        const uint4* p = reinterpret_cast<const uint4*>(sK + (kt * 16 + m16) * L::k_stride);
#pragma unroll
        for (int v = 0; v < NV; ++v) Ak[kt][v] = p[4 * v + g];
      }

#pragma unroll
      for (int qt = 0; qt < QT; ++qt) {
        float sc[4][4];
        float mx = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
          floatx4_t z = {0.f, 0.f, 0.f, 0.f};
          z = mma_rows<T, D>(Ak[kt], Bq[qt], z);
          if (W) {
            const float4 b = *reinterpret_cast<const float4*>(sB + kt * 16 + 4 * g);
            z[0] += b.x; z[1] += b.y; z[2] += b.z; z[3] += b.w;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int key = kt * 16 + 4 * g + i;
            sc[kt][i] = W || key < kc ? z[i] : -INFINITY;
            mx = fmaxf(mx, sc[kt][i]);
          }
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mnew = fmaxf(mrun[qt], mx);
        const float scale = mrun[qt] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((mrun[qt] - mnew) * c2);
        mrun[qt] = mnew;
        float psum = 0.0f;
        float pr[4][4];
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float pv = sc[kt][i] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((sc[kt][i] - mnew) * c2);
            pr[kt][i] = pv;
            psum += pv;
          }
        lrun[qt] = lrun[qt] * scale + psum;
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) acc[qt][dt] *= scale;

        if (BF) {
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            float pv[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) pv[j] = pr[2 * c + (j >> 2)][j & 3];
            bf16x8_t bhi, blo;
            split_bf16x8(pv, bhi, blo);
#pragma unroll
            for (int dt = 0; dt < D / 16; ++dt) {
              const unsigned char* row = sV + (dt * 16 + m16) * L::v_stride;
              uint2 lo = *reinterpret_cast<const uint2*>(row + (32 * c + 4 * g) * 2);
              uint2 hi = *reinterpret_cast<const uint2*>(row + (32 * c + 16 + 4 * g) * 2);
              const bf16x8_t av = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
              acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bhi, acc[qt][dt], 0, 0, 0);
              acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, blo, acc[qt][dt], 0, 0, 0);
            }
          }
        } else {
#pragma unroll
          for (int kt = 0; kt < 4; ++kt)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int key = kt * 16 + 4 * g + i;
#pragma unroll
              for (int dt = 0; dt < D / 16; ++dt) {
                const float av = *reinterpret_cast<const float*>(sV + key * L::v_stride + (dt * 16 + m16) * 4);
                acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, pr[kt][i], acc[qt][dt], 0, 0, 0);
              }
            }
        }
      }
    }

#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      float l = lrun[qt];
      l += __shfl_xor(l, 16);
      l += __shfl_xor(l, 32);
      const float inv = 1.0f / l;
      const int64_t q = q0 + qt * 16 + m16;
      if (q < n_q) {
        TO* orow = O + (s * n_q + q) * D;
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt)
          store4<TO>(orow + dt * 16 + 4 * g, acc[qt][dt][0] * inv, acc[qt][dt][1] * inv,
                     acc[qt][dt][2] * inv, acc[qt][dt][3] * inv);
      }
    }
    if constexpr (!ONE) break;
  }
}

// ---------------------------------------------------------------------------
// bf16, coreset resident in LDS (n_out <= 16*NKT, NKT even).  One workgroup (WR waves)
// stays on one slice and walks a contiguous range of queries, 16*QTR per wave
// per step, with the next step's query fragments loaded during the current
// one; the coreset is staged once: K row-major, V transposed (each thread
// transposes an 8-key x 8-column block in registers).  Softmax is one pass
// over all keys.
// ---------------------------------------------------------------------------
// Row paddings of the staged coreset.  K fragments are read 16 bytes per lane
// from 16 rows at once: a stride of 68 words puts the rows on disjoint banks.
// V^T fragments are read 8 bytes per lane from 16 rows: a stride of 2 (mod 32)
// words keeps those disjoint too (a 16-byte pad gave two-way conflicts).
template <int D, int NKT>
struct ResLds {
  static constexpr int NK = 16 * NKT;          // padded key count
  static constexpr int k_stride = D * 2 + 16;  // bytes per K row
  static constexpr int v_stride = NK * 2 + 8;  // bytes per V^T row (8-byte aligned)
  static constexpr int bytes = NK * k_stride + D * v_stride + NK * 4;
  // P.V multiplies 32 keys at a time
  static_assert(NKT % 2 == 0, "resident coreset needs an even number of 16-key tiles");
};

__device__ __forceinline__ uint32_t pack_lo(uint32_t x, uint32_t y) { return (x & 0xffffu) | (y << 16); }
__device__ __forceinline__ uint32_t pack_hi(uint32_t x, uint32_t y) { return (x >> 16) | (y & 0xffff0000u); }

//   The keys are taken in H passes of NKT / H tiles.  One pass (up to 128
// keys) needs no running maximum and is bound by HBM.  Above 128 keys the
// coreset takes over 100 KB of LDS, one workgroup per CU, and a wave's reads of
// it (512 bytes per key, K and V, for every query tile) keep the CU's LDS as
// busy as the matrix cores: a wave with two query tiles (QTR = 2), each
// fragment serving both, only fits the registers with the scores of half of
// the keys at a time (H = 2, online softmax).  Launches that would leave the
// device short of such workgroups keep one tile and one pass (attn_tile_plan).
// 256 keys, d = 128, 32 x 65536 queries, bf16 output: 521 us with one tile, one
// pass and 512 workgroups, 463 us with two, 440 us with the biases and masks as
// the score MFMAs' initial value instead of two vector instructions per score;
// 192 weighted keys, 64 x 16384 queries: 203 -> 180 us.  What bounds it now is the vector ALU (softmax and
// the split of P, 10 instructions per score) beside the matrix cores.
template <int D, int NKT, int QTR, int WR, int H, typename TO, bool W>
__global__ __launch_bounds__(64 * WR) void coreset_attn_res_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    const int32_t* __restrict__ idx, const float* __restrict__ logw, int64_t n, int64_t n_q,
    int n_out, int64_t q_per_wg, TO* __restrict__ O) {
  using L = ResLds<D, NKT>;
  constexpr int NK = L::NK;
  constexpr int NV = Frag<bf16_t, D>::NV;
  extern __shared__ __align__(16) unsigned char lds[];
  unsigned char* sK = lds;
  unsigned char* sV = lds + NK * L::k_stride;
  float* sB = reinterpret_cast<float*>(sV + D * L::v_stride);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m16 = lane & 15, g = lane >> 4;
  const int64_t s = blockIdx.y;
  // what a key's raw score starts from: its bias, or -inf past n_out
  {
    const float sqrt_d = (float)sqrt((double)D);
    for (int k = threadIdx.x; k < NK; k += 64 * WR)
      sB[k] = k < n_out ? (W ? logw[s * (int64_t)n_out + k] * sqrt_d : 0.0f) : -INFINITY;
  }
  const bf16_t* Ks = K + s * n * D;
  const bf16_t* Vs = V + s * n * D;
  const int32_t* Is = idx + s * (int64_t)n_out;
  const float c2 = (float)(kLog2e / sqrt((double)D));

  // ---- stage the coreset ----
  constexpr int WPR = D / 8;  // 16-byte words per row
  for (int w = threadIdx.x; w < NK * WPR; w += 64 * WR) {
    const int key = w / WPR, wi = w % WPR;
    uint4 kw = make_uint4(0, 0, 0, 0);
    if (key < n_out) {
      int64_t r = Is[key];
      r = r < 0 ? 0 : (r >= n ? n - 1 : r);
      kw = reinterpret_cast<const uint4*>(Ks + r * D)[wi];
    }
    *reinterpret_cast<uint4*>(sK + key * L::k_stride + wi * 16) = kw;
  }
  for (int b = threadIdx.x; b < (NK / 8) * WPR; b += 64 * WR) {
    const int kb = b / WPR, db = b % WPR;  // keys 8kb..8kb+7, columns 8db..8db+7
    uint32_t w[8][4];
#pragma unroll
    for (int r8 = 0; r8 < 8; ++r8) {
      const int key = kb * 8 + r8;
      uint4 vw = make_uint4(0, 0, 0, 0);
      if (key < n_out) {
        int64_t r = Is[key];
        r = r < 0 ? 0 : (r >= n ? n - 1 : r);
        vw = reinterpret_cast<const uint4*>(Vs + r * D)[db];
      }
      w[r8][0] = vw.x; w[r8][1] = vw.y; w[r8][2] = vw.z; w[r8][3] = vw.w;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {  // column 8db + e: the 8 keys' values
      const int k = e >> 1;
      uint4 o;
      if ((e & 1) == 0) {
        o.x = pack_lo(w[0][k], w[1][k]); o.y = pack_lo(w[2][k], w[3][k]);
        o.z = pack_lo(w[4][k], w[5][k]); o.w = pack_lo(w[6][k], w[7][k]);
      } else {
        o.x = pack_hi(w[0][k], w[1][k]); o.y = pack_hi(w[2][k], w[3][k]);
        o.z = pack_hi(w[4][k], w[5][k]); o.w = pack_hi(w[6][k], w[7][k]);
      }
      unsigned char* dst = sV + (db * 8 + e) * L::v_stride + kb * 16;
      if constexpr (L::v_stride % 16 == 0) {
        *reinterpret_cast<uint4*>(dst) = o;
      } else {
        reinterpret_cast<uint2*>(dst)[0] = make_uint2(o.x, o.y);
        reinterpret_cast<uint2*>(dst)[1] = make_uint2(o.z, o.w);
      }
    }
  }
  __syncthreads();

  const int64_t q_begin = (int64_t)blockIdx.x * q_per_wg;
  const int64_t q_end = min(q_begin + q_per_wg, n_q);
  const bf16_t* Qs = Q + s * n_q * D;
  constexpr int QSTEP = 16 * QTR * WR;  // queries per workgroup step

  uint4 Bq[QTR][NV];
#pragma unroll
  for (int qt = 0; qt < QTR; ++qt) {
    const int64_t q = q_begin + wave * 16 * QTR + qt * 16 + m16;
    load_frag<bf16_t, D>(Qs, min(q, n_q - 1), g, true, Bq[qt]);
  }
  // The first queries are consumed here (the compiler waits for them before
  // the loop): the loop is then entered with nothing in flight, so its waits
  // (stores count in vmcnt) are for the next queries' loads only.
#pragma unroll
  for (int qt = 0; qt < QTR; ++qt)
#pragma unroll
    for (int v = 0; v < NV; ++v)
      asm volatile("" : "+v"(Bq[qt][v].x), "+v"(Bq[qt][v].y), "+v"(Bq[qt][v].z), "+v"(Bq[qt][v].w));
  constexpr int KT = NKT / H;  // key tiles per pass
  // keys that every n_out of the tier has (tiers of 32 keys up to 128, then 64)
  constexpr int FULL = 16 * NKT <= 128 ? 16 * NKT - 32 : 16 * NKT - 64;
  static_assert(NKT % H == 0 && KT % 2 == 0, "whole pairs of key tiles per pass");
  for (int64_t q0 = q_begin; q0 < q_end; q0 += QSTEP) {
    const int64_t qw = q0 + wave * 16 * QTR;
    if (sizeof(TO) == 4 && qw >= q_end) break;  // (whole waves; no barrier below)
    // the next queries, requested early (one pass) or once this step's are no
    // longer needed (more passes, where registers are short)
    uint4 Nq[QTR][NV];
    auto next_queries = [&]() {
#pragma unroll
      for (int qt = 0; qt < QTR; ++qt) {
        const int64_t q = qw + QSTEP + qt * 16 + m16;
        load_frag<bf16_t, D>(Qs, min(q, n_q - 1), g, true, Nq[qt]);
      }
    };
    if constexpr (H == 1) next_queries();
    float mrun[QTR], l[QTR], inv_l[QTR];
    floatx4_t acc[QTR][D / 16];
#pragma unroll
    for (int qt = 0; qt < QTR; ++qt) {
      mrun[qt] = -INFINITY;
      l[qt] = 0.f;
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) acc[qt][dt] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int k0 = h * KT;  // the pass's first key tile
      // scores S^T[key][query]; the next key tile's fragment is read while the
      // current one multiplies, and no further (the scheduling barrier keeps
      // the compiler from hoisting every tile's LDS reads at once)
      floatx4_t sc[QTR][KT];
      uint4 a[2][NV];
#pragma unroll
      for (int v = 0; v < NV; ++v)
        a[0][v] = reinterpret_cast<const uint4*>(sK + (k0 * 16 + m16) * L::k_stride)[4 * v + g];
#pragma unroll
      for (int kt = 0; kt < KT; ++kt) {
        if (kt + 1 < KT) {
          const uint4* pk = reinterpret_cast<const uint4*>(sK + ((k0 + kt + 1) * 16 + m16) * L::k_stride);
#pragma unroll
          for (int v = 0; v < NV; ++v) a[(kt + 1) & 1][v] = pk[4 * v + g];
        }
        // unweighted, the tiles every size of the tier fills start from zero
        floatx4_t z = {0.f, 0.f, 0.f, 0.f};
        if (W || 16 * (k0 + kt + 1) > FULL) z = *reinterpret_cast<const floatx4_t*>(sB + (k0 + kt) * 16 + 4 * g);
#pragma unroll
        for (int qt = 0; qt < QTR; ++qt) sc[qt][kt] = mma_rows<bf16_t, D>(a[kt & 1], Bq[qt], z);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (H > 1)
        if (h == H - 1) next_queries();
#pragma unroll
      for (int qt = 0; qt < QTR; ++qt) {
        float mx = mrun[qt];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) mx = fmaxf(mx, sc[qt][kt][i]);
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        if (h > 0) {
          // (no finite score so far: nothing to rescale)
          const float scale = mrun[qt] == -INFINITY
                                  ? 0.f : __builtin_amdgcn_exp2f((mrun[qt] - mx) * c2);
          l[qt] *= scale;
#pragma unroll
          for (int dt = 0; dt < D / 16; ++dt) acc[qt][dt] *= scale;
        }
        mrun[qt] = mx;
        // a pass whose scores are all -inf (keys of weight zero, or products
        // past float32's range) leaves zeros, not NaN
        const float mref = H > 1 && mx == -INFINITY ? 0.f : mx;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float pv = __builtin_amdgcn_exp2f((sc[qt][kt][i] - mref) * c2);
            sc[qt][kt][i] = pv;
            l[qt] += pv;
          }
        if (h == H - 1) {
          l[qt] += __shfl_xor(l[qt], 16);
          l[qt] += __shfl_xor(l[qt], 32);
          inv_l[qt] = 1.0f / l[qt];
        }
      }
      // O^T += V^T P^T, 32 keys per MFMA; P = hi + lo in bf16
#pragma unroll
      for (int c = 0; c < KT / 2; ++c) {
        bf16x8_t bhi[QTR], blo[QTR];
#pragma unroll
        for (int qt = 0; qt < QTR; ++qt) {
          float pv[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) pv[e] = sc[qt][2 * c + (e >> 2)][e & 3];
          split_bf16x8(pv, bhi[qt], blo[qt]);
        }
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) {
          const unsigned char* row = sV + (dt * 16 + m16) * L::v_stride + k0 * 32;
          const uint2 lo = *reinterpret_cast<const uint2*>(row + (32 * c + 4 * g) * 2);
          const uint2 hi = *reinterpret_cast<const uint2*>(row + (32 * c + 16 + 4 * g) * 2);
          const bf16x8_t av = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
          for (int qt = 0; qt < QTR; ++qt) {
            acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bhi[qt], acc[qt][dt], 0, 0, 0);
            acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, blo[qt], acc[qt][dt], 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int qt = 0; qt < QTR; ++qt) {
      if constexpr (sizeof(TO) == 4) {
        // Whole 128-byte lines: for columns 32j..32j+31, lanes m16 < 8 hold
        // the first 16 (O^T tile 2j) and lanes m16 >= 8 the last 16 (tile
        // 2j+1) of rows m16 & 7 (store A) and (m16 & 7) + 8 (store B); the
        // missing halves come from lane l ^ 8 (DPP row rotation by 8).
        const bool upper = m16 >= 8;
        const int64_t qa = qw + qt * 16 + (m16 & 7);
        float* ra = reinterpret_cast<float*>(O) + (s * n_q + min(qa, q_end - 1)) * D;
        float* rb = reinterpret_cast<float*>(O) + (s * n_q + min(qa + 8, q_end - 1)) * D;
#pragma unroll
        for (int j = 0; j < D / 32; ++j) {
          float va[4], vb[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float a = acc[qt][2 * j][i] * inv_l[qt], b = acc[qt][2 * j + 1][i] * inv_l[qt];
            const float y = __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp(
                (int)__float_as_uint(upper ? a : b), 0x128, 0xF, 0xF, false));
            va[i] = upper ? y : a;
            vb[i] = upper ? b : y;
          }
          const int col = 32 * j + (upper ? 16 : 0) + 4 * g;
          // Rows past the range store the last row again, which they computed
          // (their query is the last one): the stores stay unconditional, so the
          // wait for the next queries' loads never covers them.  (One place for
          // such rows of all workgroups is written by one after the other: 40 x
          // 2049 queries, 32 keys, d = 64, 20 us, 8 so; 20 x 4097 11.6, 8.4.)  The
          // output is written once and not read here: non-temporal stores keep
          // it out of the caches, which the next kernels' reads would otherwise
          // first have to write back.
          float* da = ra + col;
          float* db = rb + col;
          typedef float f4_t __attribute__((ext_vector_type(4)));
          __builtin_nontemporal_store((f4_t){va[0], va[1], va[2], va[3]}, reinterpret_cast<f4_t*>(da));
          __builtin_nontemporal_store((f4_t){vb[0], vb[1], vb[2], vb[3]}, reinterpret_cast<f4_t*>(db));
        }
      } else {
        // bf16: lane (g, m16) holds columns 16 dt + 4g .. +3 of query m16.
        // Lanes g = 2h and 2h + 1 (16 apart) exchange one of two adjacent
        // tiles (one row swap per packed word), so that each stores 16
        // contiguous bytes: the even lane columns 16 dt_e + 8h .. +7, the odd
        // lane 16 dt_o + 8h .. +7; the four lanes of a query then write 64
        // contiguous bytes per tile pair, not 8-byte pieces.
        const int64_t q = qw + qt * 16 + m16;
        const bool oddrow = (g & 1) != 0;
        const int h = g >> 1;
        TO* orow = O + (s * n_q + min(q, q_end - 1)) * D;
#pragma unroll
        for (int k = 0; k < D / 32; ++k) {
          typedef __bf16 b2 __attribute__((ext_vector_type(2)));
          uint32_t ev[2], od[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const b2 e2 = {(__bf16)(acc[qt][2 * k][2 * j] * inv_l[qt]),
                           (__bf16)(acc[qt][2 * k][2 * j + 1] * inv_l[qt])};
            const b2 o2 = {(__bf16)(acc[qt][2 * k + 1][2 * j] * inv_l[qt]),
                           (__bf16)(acc[qt][2 * k + 1][2 * j + 1] * inv_l[qt])};
            ev[j] = __builtin_bit_cast(uint32_t, e2);
            od[j] = __builtin_bit_cast(uint32_t, o2);
          }
          // even row lanes receive the partner's even tile, odd row lanes the
          // partner's odd tile
          uint32_t got[2];
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const auto r = __builtin_amdgcn_permlane16_swap(ev[j], od[j], false, false);
            got[j] = oddrow ? r[0] : r[1];
          }
          const uint4 w = oddrow ? make_uint4(got[0], got[1], od[0], od[1])
                                 : make_uint4(ev[0], ev[1], got[0], got[1]);
          if (q < q_end)
            *reinterpret_cast<uint4*>(orow + 16 * (2 * k + (oddrow ? 1 : 0)) + 8 * h) = w;
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v) Bq[qt][v] = Nq[qt][v];
    }
  }
}

constexpr int64_t kDeviceCus = 256;
// waves per workgroup of the resident kernel, up to 128 keys and above
constexpr int kResWaves = 4;
constexpr int kResWavesBig = 8;

template <int D, int NKT, int QTR, int WR, int H, typename TO, bool W>
hipError_t launch_attn_res_w(const void* Q, const void* K, const void* V, const int32_t* idx,
                             const float* logw, int64_t S, int64_t n, int64_t n_q,
                             int64_t n_out, void* O, int64_t run, hipStream_t st) {
  using L = ResLds<D, NKT>;
  auto kern = coreset_attn_res_kernel<D, NKT, QTR, WR, H, TO, W>;
  const size_t lds = L::bytes;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  constexpr int64_t QSTEP = 16 * QTR * WR;
  // whole steps of queries per workgroup: the caller's run of them, or else
  // (run 0) as many as leave about two workgroups per CU, which hold two
  const int64_t steps = (n_q + QSTEP - 1) / QSTEP;
  if (run < 1) {
    const int64_t per_slice = std::min((512 + S - 1) / S, steps);
    run = (steps + per_slice - 1) / per_slice;
  }
  const int64_t q_per_wg = run * QSTEP;
  const int64_t wgs = (n_q + q_per_wg - 1) / q_per_wg;
  dim3 grid((unsigned)wgs, (unsigned)S), block(64 * WR);
  hipLaunchKernelGGL(kern, grid, block, lds, st, (const bf16_t*)Q, (const bf16_t*)K,
                     (const bf16_t*)V, idx, logw, n, n_q, (int)n_out, q_per_wg, (TO*)O);
  return hipGetLastError();
}

template <int D, int NKT, int QTR, int WR, int H, typename TO>
hipError_t launch_attn_res(const void* Q, const void* K, const void* V, const int32_t* idx,
                           const float* logw, int64_t S, int64_t n, int64_t n_q, int64_t n_out,
                           void* O, hipStream_t st, int64_t run = 0) {
  if (logw)
    return launch_attn_res_w<D, NKT, QTR, WR, H, TO, true>(Q, K, V, idx, logw, S, n, n_q, n_out, O, run, st);
  return launch_attn_res_w<D, NKT, QTR, WR, H, TO, false>(Q, K, V, idx, logw, S, n, n_q, n_out, O, run, st);
}

// Above 128 keys: the coreset of d = 128 fills a CU's LDS, and the launch takes
// one or two query tiles per wave (attn_tile_plan); d = 64 leaves room for two
// workgroups of one tile.
template <int D, int NKT, typename TO>
hipError_t launch_attn_res_big(const void* Q, const void* K, const void* V, const int32_t* idx,
                               const float* logw, int64_t S, int64_t n, int64_t n_q, int64_t n_out,
                               void* O, hipStream_t st) {
  if constexpr (D == 128) {
    static_assert(ResLds<D, NKT>::bytes > 80 * 1024, "one workgroup per CU");
    const TilePlan plan = attn_tile_plan(S, n_q, kDeviceCus);
    if (plan.tiles == 2)
      return launch_attn_res<D, NKT, 2, kResWavesBig, 2, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st, plan.split.run);
    return launch_attn_res<D, NKT, 1, kResWavesBig, 1, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st, plan.split.run);
  } else {
    return launch_attn_res<D, NKT, 1, kResWavesBig, 1, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
  }
}

template <int D, typename TO>
hipError_t launch_attn_res_d(int64_t n_out, const void* Q, const void* K, const void* V,
                             const int32_t* idx, const float* logw, int64_t S, int64_t n,
                             int64_t n_q, void* O, hipStream_t st, bool* used) {
  *used = true;
  if (n_out <= 32) return launch_attn_res<D, 2, 1, kResWaves, 1, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
  if (n_out <= 64) return launch_attn_res<D, 4, 1, kResWaves, 1, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
  if (n_out <= 96) return launch_attn_res<D, 6, 1, kResWaves, 1, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
  if (n_out <= 128) return launch_attn_res<D, 8, 1, kResWaves, 1, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
  // (192 = n_out 128 plus 32 sinks and a 32-row window)
  if (n_out <= 192) return launch_attn_res_big<D, 12, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
  if (n_out <= 256) return launch_attn_res_big<D, 16, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
  *used = false;
  return hipSuccess;
}

// ---------------------------------------------------------------------------
// Masked (causal) prefill over the Express cache (Alg. 4 for every point at
// once).  One workgroup = the up to 128 points [q0, q1) of a tile of one
// slice.  Its keys are the tile's cache pieces (rows of the cache, each with
// one log-weight, piece k seen by the points vlo..vhi-1), then the causal
// candidates causal_lo .. q1-1: candidate r is seen by point p iff r == p
// (the point itself) or r was kept and c0[p] <= r < p (p's C_0), with p's
// log-weight w0[p].  C_0 starts never move back (c0 is non-decreasing in p),
// so the points of the tile that see a candidate are an interval too:
// [r, max(r + 1, first tile point whose C_0 starts after r)) if r was kept,
// else [r, r + 1).  Every key then carries one interval of the tile's points
// (offsets from q0 in [0, 128], start in bits 0-15, end in bits 16-30); a
// causal key is flagged by bit 31 and takes the point's bias.  Same
// arithmetic as coreset_attn_kernel, with per-key biases sqrt(d) * logw.
// This kernel takes float rows.
// ---------------------------------------------------------------------------
template <typename T, int D, typename TO>
__global__ __launch_bounds__(64 * PF_WAVES) __attribute__((amdgpu_waves_per_eu(4))) void prefill_attn_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, int64_t n,
    const PrefillTile* __restrict__ tiles, const PrefillSeg* __restrict__ segs,
    const int32_t* __restrict__ c0s, const float* __restrict__ w0s,
    const uint8_t* __restrict__ kept, TO* __restrict__ O) {
  constexpr int NV = Frag<T, D>::NV;
  static_assert(Elem<T>::bytes == 4, "bf16 rows have a kernel of their own, below");
  using L = AttnLds<T, D>;
  __shared__ __align__(16) unsigned char lds[L::bytes];
  // a key's interval of the tile's points that see it (packed as above)
  __shared__ __align__(16) uint32_t s_vis[KC];
  __shared__ int32_t s_row[KC];
  __shared__ int64_t s_seg_end[kPrefillMaxSegs];
  __shared__ PrefillSeg s_seg[kPrefillMaxSegs];
  __shared__ int32_t s_c0[QPB];
  __shared__ float s_w0[QPB];
  unsigned char* sK = lds;
  unsigned char* sV = lds + KC * L::k_stride;
  float* sB = reinterpret_cast<float*>(sV + L::v_rows * L::v_stride);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int m16 = lane & 15, g = lane >> 4;
  const int64_t s = blockIdx.y;
  const PrefillTile tile = tiles[blockIdx.x];
  const int64_t q0 = tile.q0, q1 = tile.q1;
  const int nseg = min(tile.nseg, kPrefillMaxSegs);
  if ((int)threadIdx.x < nseg) s_seg[threadIdx.x] = segs[tile.seg0 + threadIdx.x];
  if ((int)threadIdx.x < QPB && q0 + threadIdx.x < q1) {
    s_c0[threadIdx.x] = c0s[q0 + threadIdx.x];
    s_w0[threadIdx.x] = w0s[q0 + threadIdx.x];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t e = 0;
    for (int k = 0; k < nseg; ++k) s_seg_end[k] = (e += s_seg[k].g.len);
  }
  __syncthreads();
  const int64_t F = nseg ? s_seg_end[nseg - 1] : 0;
  const int64_t M = F + (q1 - tile.causal_lo);
  const T* Ks = K + s * n * D;
  const T* Vs = V + s * n * D;
  const float sqrt_d = (float)sqrt((double)D);
  const float c2 = (float)(kLog2e / sqrt((double)D));
  const int64_t qw = q0 + wave * 16 * PF_QT;

  uint4 Bq[PF_QT][NV];
#pragma unroll
  for (int qt = 0; qt < PF_QT; ++qt) {
    const int64_t q = qw + qt * 16 + m16;
    load_frag<T, D>(Q + s * n * D, q, g, q < q1, Bq[qt]);
  }
  float mrun[PF_QT], lrun[PF_QT];
  floatx4_t acc[PF_QT][D / 16];
#pragma unroll
  for (int qt = 0; qt < PF_QT; ++qt) {
    mrun[qt] = -INFINITY;
    lrun[qt] = 0.0f;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) acc[qt][dt] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
  }

  constexpr int WPR = D * Elem<T>::bytes / 16;
  // A chunk's keys (row, bias, visibility; one thread per key) are gathered
  // into registers one chunk ahead, so their list reads overlap the previous
  // chunk's arithmetic; they reach LDS at the top of the chunk.
  // (registers hold the raw loaded values; anything computed from them is
  // left to the commit, so that no wait for the loads precedes the compute)
  // m_vis / m_vis_nk: the key's packed visibility (a causal candidate's if
  // kept / if not kept; the list read of kept[] is only waited for at commit)
  uint32_t m_vis = 0, m_vis_nk = 0;
  int32_t m_raw = 0, m_cpos = -1;
  uint8_t m_kept = 1;
  float m_bias = -INFINITY;
  bool m_piece = false;
  auto gather_meta = [&](int64_t ck_) {
    if (threadIdx.x >= KC) return;
    const int kc_ = (int)min((int64_t)KC, M - ck_);
    const int64_t kk = ck_ + threadIdx.x;
    // points [lo, hi) as offsets in the tile, clipped to it
    auto vis = [&](int64_t lo, int64_t hi) {
      const uint32_t a = (uint32_t)min(max(lo - q0, (int64_t)0), (int64_t)QPB);
      const uint32_t b = (uint32_t)min(max(hi - q0, (int64_t)0), (int64_t)QPB);
      return a | (b << 16);
    };
    m_vis = 0;
    m_vis_nk = 0;
    m_bias = -INFINITY;
    m_piece = false;
    m_cpos = -1;
    m_raw = 0;
    m_kept = 1;
    if ((int)threadIdx.x < kc_) {
      if (kk < F) {
        // the piece holding key kk: the first k with kk < s_seg_end[k]
        // (binary search: a tile has up to kPrefillMaxSegs pieces)
        int k = 0, hi = nseg - 1;
        while (k < hi) {
          const int mid = (k + hi) >> 1;
          if (kk < s_seg_end[mid]) hi = mid; else k = mid + 1;
        }
        const ExpressSeg& sg = s_seg[k].g;
        const int64_t j = kk - (k ? s_seg_end[k - 1] : 0);
        m_raw = sg.src ? sg.src[s * sg.stride + j] : (int32_t)(sg.start + j);
        m_bias = sg.logw * sqrt_d;
        m_vis = m_vis_nk = vis(s_seg[k].vlo, s_seg[k].vhi);
        m_piece = true;
      } else {
        m_cpos = (int32_t)(tile.causal_lo + (kk - F));
        m_kept = kept[m_cpos];
        // the tile's points whose C_0 starts at or before the candidate: a prefix
        int lo = 0, hi = (int)(q1 - q0);
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if (s_c0[mid] <= m_cpos) lo = mid + 1; else hi = mid;
        }
        m_vis = vis(m_cpos, max((int64_t)m_cpos + 1, q0 + lo)) | 0x80000000u;
        m_vis_nk = vis(m_cpos, (int64_t)m_cpos + 1) | 0x80000000u;
      }
    }
  };
  gather_meta(0);
  for (int64_t ck = 0; ck < M; ck += KC) {
    const int kc = (int)min((int64_t)KC, M - ck);
    __syncthreads();
    if (threadIdx.x < KC) {
      int64_t r = m_piece ? (int64_t)m_raw : (m_cpos >= 0 ? (int64_t)m_cpos : 0);
      r = r < 0 ? 0 : (r >= n ? n - 1 : r);
      s_vis[threadIdx.x] = m_kept ? m_vis : m_vis_nk;
      s_row[threadIdx.x] = (int32_t)r;
      sB[threadIdx.x] = m_bias;
    }
    __syncthreads();
    for (int w = threadIdx.x; w < KC * WPR; w += 64 * PF_WAVES) {
      const int key = w / WPR, wi = w % WPR;
      uint4 kw = make_uint4(0, 0, 0, 0), vw = make_uint4(0, 0, 0, 0);
      if (key < kc) {
        const int64_t r = s_row[key];
        kw = reinterpret_cast<const uint4*>(Ks + r * D)[wi];
        vw = reinterpret_cast<const uint4*>(Vs + r * D)[wi];
      }
      *reinterpret_cast<uint4*>(sK + key * L::k_stride + wi * 16) = kw;
      *reinterpret_cast<uint4*>(sV + key * L::v_stride + wi * 16) = vw;
    }
    __syncthreads();
    if (ck + KC < M) gather_meta(ck + KC);

#pragma unroll
    for (int qt = 0; qt < PF_QT; ++qt) {
      const int64_t p = qw + qt * 16 + m16;  // this lane's point
      const uint32_t pl = (uint32_t)(p - q0);  // its offset in the tile
      const int li = (int)min(p - q0, (int64_t)QPB - 1);
      const float pw0 = p < q1 ? s_w0[li] * sqrt_d : 0.f;
      // the lane's 16 keys: bias where the point sees the key, else -inf
      float sc[4][4];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        const uint4 w4 = *reinterpret_cast<const uint4*>(&s_vis[kt * 16 + 4 * g]);
        const float4 b4 = *reinterpret_cast<const float4*>(&sB[kt * 16 + 4 * g]);
        const uint32_t wv[4] = {w4.x, w4.y, w4.z, w4.w};
        const float kb[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool seen = pl >= (wv[i] & 0xffffu) && pl < ((wv[i] >> 16) & 0x7fffu);
          sc[kt][i] = seen ? ((int32_t)wv[i] < 0 ? pw0 : kb[i]) : -INFINITY;
        }
      }
      // (keeps the masks' LDS reads from being scheduled among the MFMAs
      // below, where their registers would push values out to scratch)
      __builtin_amdgcn_sched_barrier(0);
      float mx = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        // the key tile's fragments from LDS for each query tile (re-read
        // rather than held: the registers keep two workgroups per CU)
        uint4 ak[NV];
        const uint4* pk = reinterpret_cast<const uint4*>(sK + (kt * 16 + m16) * L::k_stride);
#pragma unroll
        for (int v = 0; v < NV; ++v) ak[v] = pk[4 * v + g];
        floatx4_t z = {0.f, 0.f, 0.f, 0.f};
        z = mma_rows<T, D>(ak, Bq[qt], z);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          sc[kt][i] += z[i];  // -inf stays -inf
          mx = fmaxf(mx, sc[kt][i]);
        }
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float mnew = fmaxf(mrun[qt], mx);
      const float scale = (mrun[qt] == -INFINITY || mnew == -INFINITY)
                              ? 0.0f : __builtin_amdgcn_exp2f((mrun[qt] - mnew) * c2);
      mrun[qt] = mnew;
      // exp2(-inf) = 0 for the keys the point does not see; a row that sees
      // none yet subtracts 0 instead of -inf
      const float mref = mnew == -INFINITY ? 0.0f : mnew;
      float psum = 0.0f;
      float pr[4][4];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float pv = __builtin_amdgcn_exp2f((sc[kt][i] - mref) * c2);
          pr[kt][i] = pv;
          psum += pv;
        }
      lrun[qt] = lrun[qt] * scale + psum;
      // (the running maxima of most chunks stay put: no rescale then)
      if (__any(scale != 1.0f)) {
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) acc[qt][dt] *= scale;
      }
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int key = kt * 16 + 4 * g + i;
#pragma unroll
          for (int dt = 0; dt < D / 16; ++dt) {
            const float av = *reinterpret_cast<const float*>(sV + key * L::v_stride + (dt * 16 + m16) * 4);
            acc[qt][dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, pr[kt][i], acc[qt][dt], 0, 0, 0);
          }
        }
    }
  }

#pragma unroll
  for (int qt = 0; qt < PF_QT; ++qt) {
    float l = lrun[qt];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    const float inv = 1.0f / l;
    const int64_t q = qw + qt * 16 + m16;
    if (q < q1) {
      TO* orow = O + (s * n + q) * D;
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt)
        store4<TO>(orow + dt * 16 + 4 * g, acc[qt][dt][0] * inv, acc[qt][dt][1] * inv,
                   acc[qt][dt][2] * inv, acc[qt][dt][3] * inv);
    }
  }
}

// ---------------------------------------------------------------------------
// The same for bf16 rows.  One workgroup = 8 waves of 16 points; the keys go
// in chunks of KC, double-buffered in LDS and copied there straight from
// global memory while the previous chunk is used:
//  - K in MFMA fragment order (16-key tile, 16-byte word, lane): every
//    fragment read is 1 KiB in a row;
//  - V rows as they are, the 32-byte column blocks of row r permuted by
//    XOR with rot(r), so that the transposing reads of four rows by 16 lanes
//    hit different banks.  ds_read_b64_tr_b16 gives lane i of 16 column i of
//    the 4 rows the 16 lanes point at: the A operand of O^T += V^T P^T.
// A key's row, bias and visibility (from the tile's pieces and candidates) are
// gathered by one wave two chunks ahead: its list reads overlap a chunk's
// arithmetic, and one barrier per chunk covers both the copies and them.
// Chunks whose keys are seen by all the tile's points skip the visibility
// tests.  Same arithmetic as above in the same order.
//   What bounds it: per chunk and wave 48 MFMAs (768 cycles), about 170 vector
// instructions and 17 exponentials (900 cycles and more) and 32 KiB of LDS
// reads (2048 cycles of the CU's LDS per workgroup and chunk, about what the
// matrix cores and the vector ALU each need).  Against the kernel above with
// V turned in registers and nothing in flight during a chunk: 65536 points x
// 32 slices, d = 128: 3660 -> 2270 us (2050 to 2180 with the order of tiles below).
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 read_tr16(uint32_t lds) {
  const s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(uintptr_t)lds);
  return __builtin_bit_cast(uint2, r);
}

template <int D>
struct PfLds {
  static constexpr int NV = D / 32;             // 16-byte words per lane of a row fragment
  static constexpr int KB = KC * D * 2;         // bytes of a chunk's keys (and of its values)
  static constexpr int COPIES = KB / 1024;      // wave copies of either
  static constexpr int WPR = D / 8;             // 16-byte words per row
  static constexpr int STAGE = 2 * KB;
  static constexpr int bytes = 2 * STAGE;
  // permutation of row r's 32-byte blocks (D / 16 of them): rows 4 i .. 4 i + 3
  // get blocks in different banks
  __device__ static int rot(int r) { return D == 32 ? (r >> 1) & 1 : r & (D / 16 - 1); }
};

template <int D, typename TO>
__global__ __launch_bounds__(64 * PF_WAVES) __attribute__((amdgpu_waves_per_eu(4))) void prefill_attn_bf16_kernel(
    const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
    int64_t n, int32_t ntiles, int64_t work, const PrefillTile* __restrict__ tiles,
    const PrefillSeg* __restrict__ segs, const int32_t* __restrict__ c0s,
    const float* __restrict__ w0s, const uint8_t* __restrict__ kept, TO* __restrict__ O) {
  using L = PfLds<D>;
  constexpr int NV = L::NV;
  // [2][K chunk, V chunk], aligned so that address bits can be permuted by XOR
  extern __shared__ __align__(1024) unsigned char stages[];
  // a piece: its row list of this slice (null: rows from start on), bias,
  // interval.  (Lists are read through global-memory pointers: a generic load
  // counts in lgkmcnt too, and every wave's wait for LDS would then cover it
  // and, with it, the copies in flight.)
  typedef const __attribute__((address_space(1))) int32_t* list_t;
  struct Piece {
    list_t src;
    int32_t start;
    uint32_t vis;
    float bias;
  };
  __shared__ Piece s_piece[kPrefillMaxSegs];
  __shared__ int32_t s_end[kPrefillMaxSegs];
  __shared__ int32_t s_c0[QPB];
  __shared__ float s_w0[QPB];
  // per key of a chunk (three chunks in turn): row, bias, visibility; and how
  // the chunk is tested: 2, every point sees every key; 1, by interval; 0, by
  // interval and with causal keys that take the point's own bias
  __shared__ int32_t s_row[3][KC];
  __shared__ __align__(16) float s_bias[3][KC];
  __shared__ __align__(16) uint32_t s_vis[3][KC];
  __shared__ int32_t s_test[3];
  __shared__ int32_t s_w0_differs;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m16 = lane & 15, g = lane >> 4;
  // Workgroups are dealt to the eight XCDs in turn; each XCD takes a contiguous
  // eighth of the tiles, slice after slice, so that the cache pieces a slice's
  // tiles share stay in one L2 (65536 points x 32 slices 2318 -> 2054 us at best,
  // 2165 on average over several runs).
  const int64_t per = (work + 7) >> 3;
  const int64_t at = (int64_t)(blockIdx.x & 7) * per + (blockIdx.x >> 3) +
                     (int64_t)(gridDim.x >> 3) * blockIdx.y;
  if (at >= min(work, ((int64_t)(blockIdx.x & 7) + 1) * per)) return;
  const int64_t s = at / ntiles;
  const PrefillTile tile = tiles[at - s * ntiles];
  const int32_t q0 = tile.q0, q1 = tile.q1;
  const int nseg = min(tile.nseg, kPrefillMaxSegs);
  const bf16_t* Ks = K + s * n * D;
  const bf16_t* Vs = V + s * n * D;
  const float sqrt_d = (float)sqrt((double)D);
  const float c2 = (float)(kLog2e / sqrt((double)D));
  // points [lo, hi) as offsets in the tile, clipped to it: start in bits 0-15,
  // length in bits 16-30
  auto vis = [&](int32_t lo, int32_t hi) {
    const uint32_t a = (uint32_t)min(max(lo - q0, 0), QPB);
    const uint32_t b = (uint32_t)min(max(hi - q0, 0), QPB);
    return a | (b > a ? b - a : 0u) << 16;
  };
  if (threadIdx.x == 0) s_w0_differs = 0;
  if ((int)threadIdx.x < nseg) {
    const PrefillSeg sg = segs[tile.seg0 + threadIdx.x];
    s_piece[threadIdx.x] = {(list_t)(sg.g.src ? sg.g.src + s * sg.g.stride : nullptr), (int32_t)sg.g.start,
                            vis(sg.vlo, sg.vhi), sg.g.logw * sqrt_d};
    s_end[threadIdx.x] = (int32_t)sg.g.len;
  }
  if ((int)threadIdx.x < QPB && q0 + (int)threadIdx.x < q1) {
    s_c0[threadIdx.x] = c0s[q0 + threadIdx.x];
    s_w0[threadIdx.x] = w0s[q0 + threadIdx.x];
  }
  const int64_t p = (int64_t)q0 + wave * 16 + m16;  // this lane's point
  uint4 Bq[NV];
  load_frag<bf16_t, D>(Q + s * n * D, p, g, p < q1, Bq);
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t e = 0;
    for (int k = 0; k < nseg; ++k) s_end[k] = (e += s_end[k]);
  }
  // a tile whose points share their C_0 weight (all but those where the level
  // changes) has one bias for its causal keys
  if ((int)threadIdx.x < QPB && q0 + (int)threadIdx.x < q1 && s_w0[threadIdx.x] != s_w0[0]) s_w0_differs = 1;
  __syncthreads();
  const int32_t F = nseg ? s_end[nseg - 1] : 0;
  const int32_t M = F + (q1 - tile.causal_lo);
  const int nch = (M + KC - 1) / KC;
  const uint32_t causal = s_w0_differs ? 0x80000000u : 0u;  // flag of a causal key
  const float w0 = s_w0[0] * sqrt_d;

  // ---- metadata of a chunk's keys (one wave, lane = key of the chunk) ----
  int piece = 0;  // the piece of this lane's last key (keys only grow)
  uint32_t m_vis = 0, m_vis_nk = 0;
  int32_t m_row = 0;
  float m_bias = -INFINITY;
  uint8_t m_kept = 1;
  auto gather = [&](int ck) {
    const int32_t kk = ck * KC + lane;
    m_vis = m_vis_nk = 0;
    m_bias = -INFINITY;
    m_kept = 1;
    m_row = q1 - 1;  // past the last key: a row the tile attends to anyway, seen by none
    if (kk < F) {
      while (kk >= s_end[piece]) ++piece;
      const Piece& pc = s_piece[piece];
      const int32_t j = kk - (piece ? s_end[piece - 1] : 0);
      m_row = pc.src ? pc.src[j] : pc.start + j;
      m_bias = pc.bias;
      m_vis = m_vis_nk = pc.vis;
    } else if (kk < M) {
      m_row = tile.causal_lo + (kk - F);
      m_kept = kept[m_row];
      // the tile's points whose C_0 starts at or before the candidate: a prefix
      int lo = 0, hi = q1 - q0;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (s_c0[mid] <= m_row) lo = mid + 1; else hi = mid;
      }
      m_vis = vis(m_row, max(m_row + 1, q0 + lo)) | causal;
      m_vis_nk = vis(m_row, m_row + 1) | causal;
      m_bias = w0;
    }
  };
  auto commit = [&](int slot) {
    const uint32_t v = m_kept ? m_vis : m_vis_nk;
    s_row[slot][lane] = m_row < 0 ? 0 : (m_row >= n ? (int32_t)(n - 1) : m_row);
    s_bias[slot][lane] = m_bias;
    s_vis[slot][lane] = v;
    const bool all = (int32_t)v >= 0 && (v & 0xffffu) == 0 && (int32_t)(v >> 16) >= q1 - q0;
    const bool every = __ballot(all) == ~(uint64_t)0, own = __ballot((int32_t)v < 0) != 0;
    if (lane == 0) s_test[slot] = every ? 2 : own ? 0 : 1;
  };
  // ---- copies of a chunk's rows into stage b ----
  const uint32_t lds0 = lds_offset(stages);
  auto copies = [&](int slot, int b) {
#pragma unroll
    for (int k = 0; k < (L::COPIES + PF_WAVES - 1) / PF_WAVES; ++k) {
      const int c = wave + k * PF_WAVES;
      if (L::COPIES % PF_WAVES == 0 || c < L::COPIES) {
        // keys: fragment word v of 16-key tile kt
        const int kt = c / NV, v = c % NV;
        const int64_t rk = s_row[slot][kt * 16 + m16];
        copy16_to_lds(reinterpret_cast<const uint4*>(Ks + rk * D) + 4 * v + g,
                      lds0 + (uint32_t)(b * L::STAGE + c * 1024));
        // values: 1024 / (2 D) rows, blocks permuted
        const int r = c * (64 / L::WPR) + lane / L::WPR, w = lane % L::WPR;
        const int64_t rv = s_row[slot][r];
        copy16_to_lds(reinterpret_cast<const uint4*>(Vs + rv * D) + (((w >> 1) ^ L::rot(r)) << 1 | (w & 1)),
                      lds0 + (uint32_t)(b * L::STAGE + L::KB + c * 1024));
      }
    }
  };
  if (wave == 0) {
    gather(0);
    commit(0);
    gather(1);
    commit(1);
  }
  __syncthreads();
  copies(0, 0);

  float mrun = -INFINITY, lrun = 0.0f;
  floatx4_t acc[D / 16];
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) acc[dt] = (floatx4_t){0.f, 0.f, 0.f, 0.f};
  const uint32_t pl = (uint32_t)(p - q0);  // this point's offset in the tile
  const float pw0 = p < q1 ? s_w0[pl] * sqrt_d : 0.f;
  // this lane's address of the transposing reads, but for the stage and block
  const int vr = 4 * g + (m16 >> 2);
  const uint32_t v_lane = (uint32_t)(L::KB + vr * D * 2 + L::rot(vr) * 32 + (m16 & 3) * 8);

  // The queries are waited for here, where the compiler sees it: their first
  // use is in the loop, whose every turn would else wait for the copies too.
  __builtin_amdgcn_s_waitcnt(0x0F70);
#pragma unroll
  for (int v = 0; v < NV; ++v)
    asm volatile("" : "+v"(Bq[v].x), "+v"(Bq[v].y), "+v"(Bq[v].z), "+v"(Bq[v].w));
  int slot = 0;
  for (int ck = 0; ck < nch; ++ck) {
    const int b = ck & 1;
    const int nslot = slot == 2 ? 0 : slot + 1;
    wait_vmcnt<0>();  // this wave's copies of chunk ck
    __syncthreads();
    if (ck + 1 < nch) copies(nslot, b ^ 1);
    if (wave == 0 && ck + 2 < nch) gather(ck + 2);

    // the lane's 16 keys: bias where the point sees the key, else -inf
    floatx4_t sc[4];
    const int test = s_test[slot];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      sc[kt] = *reinterpret_cast<const floatx4_t*>(&s_bias[slot][kt * 16 + 4 * g]);
    }
    if (test < 2) {
      uint32_t wv[4][4];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        const uint4 w4 = *reinterpret_cast<const uint4*>(&s_vis[slot][kt * 16 + 4 * g]);
        wv[kt][0] = w4.x; wv[kt][1] = w4.y; wv[kt][2] = w4.z; wv[kt][3] = w4.w;
      }
      if (test == 0) {
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if ((int32_t)wv[kt][i] < 0) sc[kt][i] = pw0;
            wv[kt][i] &= 0x7fffffffu;
          }
      }
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          sc[kt][i] = pl - (wv[kt][i] & 0xffffu) < (wv[kt][i] >> 16) ? sc[kt][i] : -INFINITY;
    }
    __builtin_amdgcn_sched_barrier(0);
    const uint4* sk = reinterpret_cast<const uint4*>(stages + b * L::STAGE);
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
      uint4 ak[NV];
#pragma unroll
      for (int v = 0; v < NV; ++v) ak[v] = sk[(kt * NV + v) * 64 + lane];
      floatx4_t z = {0.f, 0.f, 0.f, 0.f};
      z = mma_rows<bf16_t, D>(ak, Bq, z);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sc[kt][i] += z[i];  // -inf stays -inf
        mx = fmaxf(mx, sc[kt][i]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float mnew = fmaxf(mrun, mx);
    const float scale = (mrun == -INFINITY || mnew == -INFINITY)
                            ? 0.0f : __builtin_amdgcn_exp2f((mrun - mnew) * c2);
    mrun = mnew;
    // exp2(-inf) = 0 for the keys the point does not see; a row that sees
    // none yet subtracts 0 instead of -inf
    const float mref = mnew == -INFINITY ? 0.0f : mnew;
    float psum = 0.0f;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sc[kt][i] = __builtin_amdgcn_exp2f((sc[kt][i] - mref) * c2);
        psum += sc[kt][i];
      }
    lrun = lrun * scale + psum;
    // (the running maxima of most chunks stay put: no rescale then)
    if (__any(scale != 1.0f)) {
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) acc[dt] *= scale;
    }
    const uint32_t va = lds0 + (uint32_t)(b * L::STAGE) + v_lane;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      float pv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) pv[j] = sc[2 * c + (j >> 2)][j & 3];
      bf16x8_t bhi, blo;
      split_bf16x8(pv, bhi, blo);
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) {
        const uint32_t at = (va ^ (uint32_t)(dt * 32)) + (uint32_t)(32 * c * D * 2);
        const uint2 lo = read_tr16(at), hi = read_tr16(at + 16 * D * 2);
        const bf16x8_t av = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bhi, acc[dt], 0, 0, 0);
        acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, blo, acc[dt], 0, 0, 0);
      }
    }
    if (wave == 0 && ck + 2 < nch) commit(nslot == 2 ? 0 : nslot + 1);
    slot = nslot;
  }

  float l = lrun;
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  const float inv = 1.0f / l;
  if (p < q1) {
    TO* orow = O + (s * n + p) * D;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
      store4<TO>(orow + dt * 16 + 4 * g, acc[dt][0] * inv, acc[dt][1] * inv, acc[dt][2] * inv,
                 acc[dt][3] * inv);
  }
}

template <typename T, int D, typename TO>
hipError_t launch_prefill_t(const void* Q, const void* K, const void* V, int64_t S, int64_t n,
                            const PrefillTile* tiles, int64_t ntiles, const PrefillSeg* segs,
                            const int32_t* c0, const float* w0, const uint8_t* kept, void* O,
                            hipStream_t st) {
  dim3 grid((unsigned)ntiles, (unsigned)S), block(64 * PF_WAVES);
  if constexpr (Elem<T>::bytes == 2) {
    auto kern = prefill_attn_bf16_kernel<D, TO>;
    const size_t lds = PfLds<D>::bytes;
    if (lds > 48 * 1024) {  // beside the kernel's 12 KiB of static LDS
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    const int64_t work = ntiles * S;
    const GridRows g = grid_rows((work + 7) / 8 * 8, 64 * PF_WAVES, 8);
    hipLaunchKernelGGL(kern, dim3((unsigned)g.x, (unsigned)g.rows), block, lds, st,
                       (const bf16_t*)Q, (const bf16_t*)K, (const bf16_t*)V, n, (int32_t)ntiles,
                       work, tiles, segs, c0, w0, kept, (TO*)O);
  } else {
    hipLaunchKernelGGL((prefill_attn_kernel<T, D, TO>), grid, block, 0, st, (const T*)Q,
                       (const T*)K, (const T*)V, n, tiles, segs, c0, w0, kept, (TO*)O);
  }
  return hipGetLastError();
}

template <typename T, typename TO>
hipError_t launch_prefill_d(int64_t d, const void* Q, const void* K, const void* V, int64_t S,
                            int64_t n, const PrefillTile* tiles, int64_t ntiles,
                            const PrefillSeg* segs, const int32_t* c0, const float* w0,
                            const uint8_t* kept, void* O, hipStream_t st) {
  switch (d) {
    case 32: return launch_prefill_t<T, 32, TO>(Q, K, V, S, n, tiles, ntiles, segs, c0, w0, kept, O, st);
    case 64: return launch_prefill_t<T, 64, TO>(Q, K, V, S, n, tiles, ntiles, segs, c0, w0, kept, O, st);
    case 128: return launch_prefill_t<T, 128, TO>(Q, K, V, S, n, tiles, ntiles, segs, c0, w0, kept, O, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T, int D, typename TO>
hipError_t launch_attn_t(const void* Q, const void* K, const void* V, const int32_t* idx,
                         const float* logw, int64_t S, int64_t n, int64_t n_q, int64_t n_out,
                         void* O, hipStream_t st) {
  // Float rows: one 16-query tile per wave, whose registers let more workgroups
  // share a CU, though every 64 queries then stage the coreset (us with two tiles
  // | one: d = 64, 8 x 1024 queries over 128 keys 16.4 | 10.4, 32 x 16384 over 256
  // 349 | 326; d = 128, 8 x 1024 over 48 16.6 | 10.9, 100 x 4096 over 256 828 | 693;
  // d = 32 within 3 % where the queries fill the device: 32 x 16384 over 256 176 |
  // 181).  bf16 rows: two, so that a chunk's staging, which turns V, serves twice
  // the queries (8 x 3000 x 400 keys, d = 128: 38 us, 45 with one).
  constexpr int QT = Elem<T>::bytes == 4 ? 1 : 2;
  constexpr int64_t per = 16 * QT * WAVES;
  const int64_t blocks = (n_q + per - 1) / per;
  auto launch = [&](auto kern, int64_t wgs) {
    const GridRows g = grid_rows(wgs, 64 * WAVES);
    const int extra = g.rows == 1 ? (int)(blocks % wgs) : 0;
    hipLaunchKernelGGL(kern, dim3((unsigned)g.x, (unsigned)S, (unsigned)g.rows), dim3(64 * WAVES),
                       0, st, (const T*)Q, (const T*)K, (const T*)V, idx, logw, n, n_q, (int)n_out,
                       extra, (TO*)O);
  };
  // One chunk of float keys: several blocks of queries per workgroup.  (bf16
  // rows come here with d = 32 or more than 256 keys only; over one chunk of
  // d = 32 a block's arithmetic is so short that the blocks' loads are better
  // overlapped by workgroups of their own: 200 x 4097 queries over 16 keys 38
  // us, 45 with 768 workgroups.)
  if constexpr (Elem<T>::bytes == 4) {
    if (n_out <= KC) {
      constexpr int per_cu = D == 32 ? 5 : D == 64 ? 4 : 2;  // as the registers allow
      const int64_t wgs = split_blocks(S, blocks, per_cu * kDeviceCus);
      if (logw)
        launch(coreset_attn_kernel<T, D, TO, true, QT, true>, wgs);
      else
        launch(coreset_attn_kernel<T, D, TO, false, QT, true>, wgs);
      return hipGetLastError();
    }
  }
  if (logw)
    launch(coreset_attn_kernel<T, D, TO, true, QT, false>, blocks);
  else
    launch(coreset_attn_kernel<T, D, TO, false, QT, false>, blocks);
  return hipGetLastError();
}

template <typename T, typename TO>
hipError_t launch_attn_d(int64_t d, const void* Q, const void* K, const void* V,
                         const int32_t* idx, const float* logw, int64_t S, int64_t n,
                         int64_t n_q, int64_t n_out, void* O, hipStream_t st) {
  switch (d) {
    case 32: return launch_attn_t<T, 32, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
    case 64: return launch_attn_t<T, 64, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
    case 128: return launch_attn_t<T, 128, TO>(Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_prefill_attention(int dtype, int64_t d, int out_dtype, const void* Q,
                                    const void* K, const void* V, int64_t S, int64_t n,
                                    const PrefillTile* tiles, int64_t ntiles,
                                    const PrefillSeg* segs, const int32_t* c0, const float* w0,
                                    const uint8_t* kept, void* O, hipStream_t st) {
  if (ntiles < 1) return hipSuccess;
  if (dtype == 0)
    return out_dtype == 0
               ? launch_prefill_d<float, float>(d, Q, K, V, S, n, tiles, ntiles, segs, c0, w0, kept, O, st)
               : launch_prefill_d<float, bf16_t>(d, Q, K, V, S, n, tiles, ntiles, segs, c0, w0, kept, O, st);
  return out_dtype == 0
             ? launch_prefill_d<bf16_t, float>(d, Q, K, V, S, n, tiles, ntiles, segs, c0, w0, kept, O, st)
             : launch_prefill_d<bf16_t, bf16_t>(d, Q, K, V, S, n, tiles, ntiles, segs, c0, w0, kept, O, st);
}

hipError_t launch_attention(int dtype, int64_t d, int out_dtype, const void* Q, const void* K,
                            const void* V, const int32_t* idx, const float* logw, int64_t S,
                            int64_t n, int64_t n_q, int64_t n_out, void* O, hipStream_t st) {
  if (dtype == 0) {
    if (out_dtype == 0)
      return launch_attn_d<float, float>(d, Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
    return launch_attn_d<float, bf16_t>(d, Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
  }
  bool used = false;
  hipError_t e = hipSuccess;
  if (d == 64)
    e = out_dtype == 0
            ? launch_attn_res_d<64, float>(n_out, Q, K, V, idx, logw, S, n, n_q, O, st, &used)
            : launch_attn_res_d<64, bf16_t>(n_out, Q, K, V, idx, logw, S, n, n_q, O, st, &used);
  else if (d == 128)
    e = out_dtype == 0
            ? launch_attn_res_d<128, float>(n_out, Q, K, V, idx, logw, S, n, n_q, O, st, &used)
            : launch_attn_res_d<128, bf16_t>(n_out, Q, K, V, idx, logw, S, n, n_q, O, st, &used);
  if (used) return e;
  if (out_dtype == 0)
    return launch_attn_d<bf16_t, float>(d, Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
  return launch_attn_d<bf16_t, bf16_t>(d, Q, K, V, idx, logw, S, n, n_q, n_out, O, st);
}

}  // namespace thin
