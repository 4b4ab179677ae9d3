// Device helpers of the Express cache (Sec. 3, Alg. 1 and 2): index-list
// moves, the per-call v_max of a Halve call and the layout of the weighted
// key list a point attends over (Alg. 5).  The Halve calls themselves are
// the KH rounds of compress.hip, one bucket per slice.
#include "attn_plan.hpp"
#include "common.hpp"
#include "launch.hpp"

namespace thin {

namespace {

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

// dst[s * dst_stride + j] = src[s * src_stride + j]  (j < len)
__global__ void rows_copy_kernel(const int32_t* src, int64_t src_stride, int32_t* dst,
                                 int64_t dst_stride, int64_t len) {
  const int64_t s = blockIdx.y;
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < len) dst[s * dst_stride + j] = src[s * src_stride + j];
}

// v_max of a Halve call (eq. katt over the rows it thins): the largest
// |V[s, row, c]| over its N rows idx[s * in_stride + t * N + j], as the
// float's bit pattern at vmax_bits[s * G + t].  One workgroup per call (G
// calls per slice); a row is d * bytes / 16 16-byte words.  What bounds it is the
// bytes that one CU has in flight: 16 waves of 8 words per lane, 128 KiB (32 calls
// of 1024 float rows, d = 128: 15.6 us, 29.3 with four waves).
constexpr int kVmaxWaves = 16;
template <typename T>
__global__ __launch_bounds__(64 * kVmaxWaves) void vmax_rows_kernel(
    const T* V, int64_t ld, int64_t d, const int32_t* idx, int64_t in_stride, int64_t N, int64_t G,
    int64_t calls, uint32_t* vmax_bits) {
  constexpr int kU = 8;
  const int64_t c = blockIdx.x + (int64_t)gridDim.x * blockIdx.y;
  if (c >= calls) return;
  const int64_t s = c / G, t = c % G;
  const int64_t wpr = d * Elem<T>::bytes / 16;
  const u32x4* base = reinterpret_cast<const u32x4*>(V + s * ld * d);
  const int32_t* rows = idx + s * in_stride + t * N;
  uint32_t m = 0u;
  // kU words per thread per pass: every row index of a pass is requested,
  // then every word, so a pass waits for two memory latencies, not 2 kU
  // (wpr is a power of two for every supported d and element size)
  const int sh = __builtin_ctzll((unsigned long long)wpr);
  const int32_t total = (int32_t)(N * wpr);
  for (int32_t w0 = threadIdx.x; w0 < total; w0 += kU * (int32_t)blockDim.x) {
    int64_t row[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int32_t w = w0 + u * (int32_t)blockDim.x;
      row[u] = w < total ? (int64_t)rows[w >> sh] : -1;
    }
    u32x4 x[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int32_t w = w0 + u * (int32_t)blockDim.x;
      x[u] = row[u] >= 0 ? base[row[u] * wpr + (w & (int32_t)(wpr - 1))] : (u32x4){0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (Elem<T>::bytes == 4) {
          m = max(m, x[u][c] & 0x7fffffffu);
        } else {
          m = max(m, (x[u][c] << 16) & 0x7fffffffu);
          m = max(m, x[u][c] & 0x7fff0000u);
        }
      }
  }
  const float mf = wave_max(__uint_as_float(m));
  __shared__ float part[kVmaxWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) part[wave] = mf;
  __syncthreads();
  if (wave == 0) {
    const float call = wave_max(lane < kVmaxWaves ? part[lane] : 0.0f);
    if (lane == 0) vmax_bits[c] = __float_as_uint(call);
  }
}

// Key j of slice s: the segment k with off_k <= j < off_k + len_k gives
// src_k[s * stride_k + j - off_k] (src_k null: start_k + j - off_k) and logw_k;
// slice s's keys start at s * out_stride.
__global__ void express_keys_kernel(ExpressSegs segs, int64_t m, int64_t out_stride, int32_t* idx,
                                    float* logw) {
  const int64_t s = blockIdx.y;
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= m) return;
  int k = 0;
  int64_t off = 0;
  while (k + 1 < segs.n && j >= off + segs.seg[k].len) off += segs.seg[k++].len;
  const ExpressSeg& g = segs.seg[k];
  const int64_t r = j - off;
  idx[s * out_stride + j] = g.src ? g.src[s * g.stride + r] : (int32_t)(g.start + r);
  logw[s * out_stride + j] = g.logw;
}

// ---------------------------------------------------------------------------
// Weighted attention of one query per slice (a decoding step, Alg. 5) over
// the m keys of the cache segments (read in place: no key list is written),
// each key with its segment's log-weight.  The keys of a slice are split
// over `split` workgroups of 16 waves; a wave takes a contiguous run of keys
// and reads them with 16-byte loads, a key row spread over LPK lanes, so one
// load instruction brings 64 / LPK keys (4 bf16 rows of d = 128) and a wave
// keeps kDecUnroll such loads of K and of V in flight.  Each lane group of a
// key keeps an online softmax (log2 domain) of its keys; the groups merge by
// lane shuffles, the waves in LDS.  split == 1: the workgroup normalises and
// writes the output row itself (one launch per step); else it writes its
// unnormalised partial (max, sum, acc[D]) and a second kernel merges them.
// ---------------------------------------------------------------------------
constexpr int kDecWaves = 16;
constexpr int kDecUnroll = 8;
constexpr int64_t kDecMaxWorkgroups = 256;  // one per CU

// The EPW elements of a 16-byte word as floats.
template <typename T>
__device__ __forceinline__ void word_to_floats(const u32x4& w, float* out);
template <>
__device__ __forceinline__ void word_to_floats<float>(const u32x4& w, float* out) {
#pragma unroll
  for (int c = 0; c < 4; ++c) out[c] = __uint_as_float(w[c]);
}
template <>
__device__ __forceinline__ void word_to_floats<bf16_t>(const u32x4& w, float* out) {
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    out[2 * c] = __uint_as_float(w[c] << 16);
    out[2 * c + 1] = __uint_as_float(w[c] & 0xffff0000u);
  }
}

template <typename TO>
__device__ __forceinline__ void store_out(TO* p, float v);
template <>
__device__ __forceinline__ void store_out<float>(float* p, float v) { *p = v; }
template <>
__device__ __forceinline__ void store_out<bf16_t>(bf16_t* p, float v) {
  *reinterpret_cast<__bf16*>(p) = (__bf16)v;
}

// Sum over the LPK lanes of a key row (LPK consecutive lanes, aligned); every
// lane gets it.  Within 16 lanes by DPP adds (no LDS): rotations within the
// row of 16, or, for rows of 4 or 8 lanes, quad permutes and the half mirror.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(x), CTRL, 0xF, 0xF, false));
}
template <int LPK>
__device__ __forceinline__ float row_sum(float x) {
  static_assert(LPK == 4 || LPK == 8 || LPK == 16 || LPK == 32, "key rows of 64..512 bytes");
  if constexpr (LPK == 32) x += __shfl_xor(x, 16);
  if constexpr (LPK >= 16) {
    x = dpp_add<0x128>(x);
    x = dpp_add<0x124>(x);
    x = dpp_add<0x122>(x);
    x = dpp_add<0x121>(x);
  } else {
    x = dpp_add<0xB1>(x);
    x = dpp_add<0x4E>(x);
    if constexpr (LPK == 8) x = dpp_add<0x141>(x);
  }
  return x;
}

// The values of the lower and the upper of a pair of lane groups OFF apart
// (OFF = 16, 32: one swap instruction; else LDS), the same pair in both.
template <int OFF>
__device__ __forceinline__ void both(float x, float& lower, float& upper) {
  if constexpr (OFF == 32 || OFF == 16) {
    const uint32_t u = __float_as_uint(x);
    const auto r = OFF == 32 ? __builtin_amdgcn_permlane32_swap(u, u, false, false)
                             : __builtin_amdgcn_permlane16_swap(u, u, false, false);
    lower = __uint_as_float(r[0]);
    upper = __uint_as_float(r[1]);
  } else {
    const float y = __shfl_xor(x, OFF);
    const bool up = (threadIdx.x & OFF) != 0;
    lower = up ? y : x;
    upper = up ? x : y;
  }
}

// Merge of two online-softmax states (m, l, acc) in the log2 domain; an empty
// state has m = -inf.
template <int EPW>
__device__ __forceinline__ void softmax_merge(float& m, float& l, float* acc, float m2, float l2,
                                              const float* acc2) {
  const float M = fmaxf(m, m2);
  const float a = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
  const float b = m2 == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m2 - M);
  l = l * a + l2 * b;
#pragma unroll
  for (int e = 0; e < EPW; ++e) acc[e] = acc[e] * a + acc2[e] * b;
  m = M;
}
template <int OFF, int EPW>
__device__ __forceinline__ void merge_groups(float& m, float& l, float* acc) {
  float m0, m1, l0, l1, a0[EPW], a1[EPW];
  both<OFF>(m, m0, m1);
  both<OFF>(l, l0, l1);
#pragma unroll
  for (int e = 0; e < EPW; ++e) both<OFF>(acc[e], a0[e], a1[e]);
  softmax_merge<EPW>(m0, l0, a0, m1, l1, a1);
  m = m0;
  l = l0;
#pragma unroll
  for (int e = 0; e < EPW; ++e) acc[e] = a0[e];
}

// The segments as the kernel reads them: keys [end of the previous segment,
// end) are the rows src[s * stride + at + j] (src null: at + j), j the key's
// position in the whole list.  Caches of at most kDecFewSegs segments (every
// mbar up to 9) launch with an argument of that size: a third of the bytes to
// write and to read per step.
struct DecSeg {
  const int32_t* src;
  int64_t stride;
  int32_t at;
  int32_t end;
  float logw;
};
constexpr int kDecFewSegs = 12;
template <int NS>
struct DecSegs {
  DecSeg seg[NS];
  int n;
};

// Dot product of a 16-byte word of q (as loaded, and as floats) with one of a
// key: bf16 pairs by the dot instruction (exact products, float32 sums).
template <typename T>
__device__ __forceinline__ float word_dot(const u32x4& qw, const float* q, const u32x4& k);
template <>
__device__ __forceinline__ float word_dot<float>(const u32x4&, const float* q, const u32x4& k) {
  float d = 0.f;
#pragma unroll
  for (int c = 0; c < 4; ++c) d = __builtin_fmaf(q[c], __uint_as_float(k[c]), d);
  return d;
}
template <>
__device__ __forceinline__ float word_dot<bf16_t>(const u32x4& qw, const float*, const u32x4& k) {
  float d = 0.f;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint32_t a = qw[c], b = k[c];  // (a bit cast of a vector's element itself reads element 0)
    d = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a),
                                        __builtin_bit_cast(bf16x2_t, b), d, false);
  }
  return d;
}

// C workgroups share a slice's run of keys (blockIdx.z = c): each forms every
// key's weight and adds its D / C columns of V, so nothing is merged between
// them.  What bounds a step is one CU's vector ALU and the chain of latencies
// (kernel argument, query, list, rows, the merge in LDS): with 32 slices, 410
// keys of 128 bf16 and one workgroup per slice, the arithmetic after the rows
// arrived took 2.3 us of 7.6 (most of it unpacking and adding V) and the
// look-ups 2 us.
template <typename T, int D, typename TO, int C, int NS>
__global__ __launch_bounds__(64 * kDecWaves) void decode_attn_kernel(
    const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, int64_t ld,
    int32_t m, int split, float* __restrict__ part, TO* __restrict__ O, int32_t* app,
    int64_t app_stride, int32_t app_val, DecSegs<NS> segs) {
  constexpr int LPK = D * Elem<T>::bytes / 16;  // lanes per key row (16 bytes each)
  constexpr int KPI = 64 / LPK;                 // keys per load instruction
  constexpr int EPW = 16 / Elem<T>::bytes;      // elements per 16-byte word
  constexpr int EPV = EPW / C;                  // V elements per lane (of this workgroup's columns)
  constexpr int VB = 16 / C;                    // their bytes
  constexpr int DV = D / C;
  static_assert(LPK >= 1 && LPK <= 64 && 64 % LPK == 0, "row of 16..1024 bytes");
  static_assert(VB >= 4, "a V word of 4, 8 or 16 bytes");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane / LPK, pos = lane % LPK;
  const int64_t s = blockIdx.y;
  const int cz = blockIdx.z;
  // the segment table: lane k holds segment k (one parallel read of the kernel
  // argument); no LDS, no barrier
  const int nseg = segs.n;
  DecSeg seg{};
  if (lane < NS) seg = segs.seg[lane];
  const u32x4 qw = reinterpret_cast<const u32x4*>(Q + s * D)[pos];
  const int32_t k0 = (int32_t)((int64_t)m * blockIdx.x / split);
  const int32_t k1 = (int32_t)((int64_t)m * (blockIdx.x + 1) / split);
  // this wave's contiguous run of keys
  const int32_t per = (k1 - k0 + kDecWaves - 1) / kDecWaves;
  const int32_t w0 = min(k1, k0 + per * wave), w1 = min(k1, w0 + per);
  const float c2 = (float)(1.4426950408889634 / sqrt((double)D));
  const float l2e = 1.4426950408889634f;
  const u32x4* Ks = reinterpret_cast<const u32x4*>(K + s * ld * D);
  const unsigned char* Vs = reinterpret_cast<const unsigned char*>(V + s * ld * D) + cz * DV * Elem<T>::bytes + pos * VB;
  const uint64_t g_src = (uint64_t)(uintptr_t)(seg.src ? seg.src + s * seg.stride : nullptr);
  float q[EPW];
  word_to_floats<T>(qw, q);
  float mrun = -INFINITY, lrun = 0.f, acc[EPV];
#pragma unroll
  for (int e = 0; e < EPV; ++e) acc[e] = 0.f;
  constexpr int BK = KPI * kDecUnroll;  // keys per batch
  constexpr int NL = (BK + 63) / 64;    // a lane looks up this many of them
  for (int32_t j0 = w0; j0 < w1; j0 += BK) {
    // Key j0 + 64 h + lane of the batch: its segment (the number of segments
    // that end at or before it), row index and log-weight.  Every key is
    // looked up by one lane and handed to the lanes that read its row, so the
    // batch waits for one list read and then for its rows.
    int32_t row[NL];
    float lw[NL];
#pragma unroll
    for (int h = 0; h < NL; ++h) {
      const int32_t j = min(j0 + 64 * h + lane, w1 - 1);
      int k = 0;
      for (int i = 0; i + 1 < nseg; ++i) k += j >= __builtin_amdgcn_readlane(seg.end, i) ? 1 : 0;
      const uint64_t src = (uint64_t)(uint32_t)__shfl((int)(uint32_t)g_src, k) |
                           (uint64_t)(uint32_t)__shfl((int)(uint32_t)(g_src >> 32), k) << 32;
      row[h] = __shfl(seg.at, k) + j;
      lw[h] = __shfl(seg.logw, k) * l2e;
      if (src) row[h] = reinterpret_cast<const __attribute__((address_space(1))) int32_t*>(src)[row[h]];
    }
    u32x4 kw[kDecUnroll];
    uint32_t vw[kDecUnroll][VB / 4];
    float sc[kDecUnroll];
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
      const int k = u * KPI;  // key k + sub of the batch (past the run: its last key again, dropped)
      const int64_t r = __shfl(row[k / 64], k % 64 + sub);
      const float w = __shfl(lw[k / 64], k % 64 + sub);
      sc[u] = j0 + k + sub < w1 ? w : -INFINITY;
      kw[u] = Ks[r * LPK + pos];
      const unsigned char* v = Vs + r * (D * Elem<T>::bytes);
      if constexpr (VB == 16) {
        const u32x4 x = *reinterpret_cast<const u32x4*>(v);
#pragma unroll
        for (int c = 0; c < 4; ++c) vw[u][c] = x[c];
      } else if constexpr (VB == 8) {
        const uint2 x = *reinterpret_cast<const uint2*>(v);
        vw[u][0] = x.x;
        vw[u][1] = x.y;
      } else {
        vw[u][0] = *reinterpret_cast<const uint32_t*>(v);
      }
    }
    float mx = mrun;
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
      const float d = row_sum<LPK>(word_dot<T>(qw, q, kw[u]));
      sc[u] = sc[u] == -INFINITY ? -INFINITY : __builtin_fmaf(d, c2, sc[u]);
      mx = fmaxf(mx, sc[u]);
    }
    if (mx == -INFINITY) continue;  // nothing of positive weight yet
    const float scale = mrun == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mrun - mx);
    lrun *= scale;
#pragma unroll
    for (int e = 0; e < EPV; ++e) acc[e] *= scale;
#pragma unroll
    for (int u = 0; u < kDecUnroll; ++u) {
      const float p = __builtin_amdgcn_exp2f(sc[u] - mx);  // 0 for a dropped key
      lrun += p;
#pragma unroll
      for (int e = 0; e < VB / 4; ++e) {
        const uint32_t x = sc[u] == -INFINITY ? 0u : vw[u][e];  // (an infinite entry of a dropped key)
        if constexpr (Elem<T>::bytes == 4) {
          acc[e] = __builtin_fmaf(p, __uint_as_float(x), acc[e]);
        } else {
          acc[2 * e] = __builtin_fmaf(p, __uint_as_float(x << 16), acc[2 * e]);
          acc[2 * e + 1] = __builtin_fmaf(p, __uint_as_float(x & 0xffff0000u), acc[2 * e + 1]);
        }
      }
    }
    mrun = mx;
  }
  // the wave's KPI key groups merge into lanes 0..LPK-1
  if constexpr (LPK <= 4) merge_groups<4, EPV>(mrun, lrun, acc);
  if constexpr (LPK <= 8) merge_groups<8, EPV>(mrun, lrun, acc);
  if constexpr (LPK <= 16) merge_groups<16, EPV>(mrun, lrun, acc);
  merge_groups<32, EPV>(mrun, lrun, acc);
  __shared__ float s_m[kDecWaves], s_l[kDecWaves], s_acc[kDecWaves][DV];
  if (lane == 0) {
    s_m[wave] = mrun;
    s_l[wave] = lrun;
  }
  if (lane < LPK) {
#pragma unroll
    for (int e = 0; e < EPV; ++e) s_acc[wave][pos * EPV + e] = acc[e];
  }
  __syncthreads();
  const int c = threadIdx.x;
  if (c < DV) {
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) M = fmaxf(M, s_m[w]);
    float a = 0.f, L = 0.f;
#pragma unroll
    for (int w = 0; w < kDecWaves; ++w) {
      const float f = s_m[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s_m[w] - M);
      a = __builtin_fmaf(s_acc[w][c], f, a);
      L = __builtin_fmaf(s_l[w], f, L);
    }
    if (split == 1) {
      store_out<TO>(O + s * D + cz * DV + c, a / L);
    } else {
      float* out = part + (s * split + blockIdx.x) * (int64_t)(D + 2);
      out[2 + cz * DV + c] = a;
      if (c == 0 && cz == 0) {
        out[0] = M;
        out[1] = L;
      }
    }
  }
  if (split == 1 && app && cz == 0 && threadIdx.x == 0) app[s * app_stride] = app_val;
}

// One workgroup per slice: the partials' maxima and sums are staged in LDS
// (one load each), then thread c merges column c of every partial.  With
// app non-null, thread 0 also writes the point's position app_val to
// app[s * app_stride] (the point entering its cache list).
template <int D, typename TO>
__global__ __launch_bounds__(128) void decode_attn_merge_kernel(const float* __restrict__ part,
                                                                int split, TO* __restrict__ O,
                                                                int32_t* app, int64_t app_stride,
                                                                int32_t app_val) {
  const int64_t s = blockIdx.x;
  if (app && threadIdx.x == 0) app[s * app_stride] = app_val;
  const float* p = part + s * split * (int64_t)(D + 2);
  __shared__ float s_w[kDecodeMaxSplit], s_l[kDecodeMaxSplit];
  __shared__ float s_M;
  if (threadIdx.x < split) {
    s_w[threadIdx.x] = p[threadIdx.x * (D + 2)];
    s_l[threadIdx.x] = p[threadIdx.x * (D + 2) + 1];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float M = -INFINITY;
    for (int k = 0; k < split; ++k) M = fmaxf(M, s_w[k]);
    s_M = M;
  }
  __syncthreads();
  if (threadIdx.x < split)  // each partial's scale exp2(m_k - M), 0 for an empty one
    s_w[threadIdx.x] = s_w[threadIdx.x] == -INFINITY ? 0.f
                                                     : __builtin_amdgcn_exp2f(s_w[threadIdx.x] - s_M);
  __syncthreads();
  float L = 0.f;
  for (int k = 0; k < split; ++k) L = __builtin_fmaf(s_l[k], s_w[k], L);
  for (int c = threadIdx.x; c < D; c += blockDim.x) {
    float v[kDecodeMaxSplit];
#pragma unroll
    for (int k = 0; k < kDecodeMaxSplit; ++k) v[k] = k < split ? p[k * (D + 2) + 2 + c] : 0.f;
    float a = 0.f;
#pragma unroll
    for (int k = 0; k < kDecodeMaxSplit; ++k) a = __builtin_fmaf(v[k], k < split ? s_w[k] : 0.f, a);
    store_out<TO>(O + s * D + c, a / L);
  }
}

struct Append {
  int32_t* dst;
  int64_t stride;
  int32_t val;
};

template <typename T, int D, typename TO, int C, int NS>
void launch_decode_c(const void* Q, const void* K, const void* V, const ExpressSegs& g, int64_t S,
                     int64_t ld, int64_t m, int split, float* part, void* O, const Append& ap,
                     hipStream_t st) {
  DecSegs<NS> segs;
  segs.n = g.n;
  int64_t off = 0;
  for (int k = 0; k < NS; ++k) {
    const ExpressSeg& x = g.seg[k < g.n ? k : 0];
    segs.seg[k] = {x.src, x.stride, (int32_t)((x.src ? 0 : x.start) - off), (int32_t)(off + x.len),
                   x.logw};
    if (k < g.n) off += x.len;
  }
  hipLaunchKernelGGL((decode_attn_kernel<T, D, TO, C, NS>), dim3((unsigned)split, (unsigned)S, C),
                     dim3(64 * kDecWaves), 0, st, (const T*)Q, (const T*)K, (const T*)V, ld,
                     (int32_t)m, split, part, (TO*)O, ap.dst, ap.stride, ap.val, segs);
}

template <typename T, int D, typename TO, int NS>
void launch_decode_n(const void* Q, const void* K, const void* V, const ExpressSegs& g, int64_t S,
                     int64_t ld, int64_t m, int split, float* part, void* O, const Append& ap,
                     hipStream_t st) {
  // Four workgroups per slice (else two, one) while the launch has at most one
  // per CU: each then has a CU to itself, with a quarter of V's work.  32
  // slices, ~410 keys, bf16, d = 128: 6.3 us (6.4 to 6.7 on average over 16384
  // points) with four, 6.8 with two, 7.6 with
  // one (9.4 with one look-up after the other and one workgroup per slice).
  const int64_t wgs = S * split;
  if (wgs * 4 <= kDecMaxWorkgroups)
    launch_decode_c<T, D, TO, 4, NS>(Q, K, V, g, S, ld, m, split, part, O, ap, st);
  else if (wgs * 2 <= kDecMaxWorkgroups)
    launch_decode_c<T, D, TO, 2, NS>(Q, K, V, g, S, ld, m, split, part, O, ap, st);
  else
    launch_decode_c<T, D, TO, 1, NS>(Q, K, V, g, S, ld, m, split, part, O, ap, st);
}

template <typename T, int D, typename TO>
hipError_t launch_decode_t(const void* Q, const void* K, const void* V, const ExpressSegs& g,
                           int64_t S, int64_t ld, int64_t m, int split, float* part, void* O,
                           const Append& ap, hipStream_t st) {
  if (g.n <= kDecFewSegs)
    launch_decode_n<T, D, TO, kDecFewSegs>(Q, K, V, g, S, ld, m, split, part, O, ap, st);
  else
    launch_decode_n<T, D, TO, kExpressMaxSegs>(Q, K, V, g, S, ld, m, split, part, O, ap, st);
  if (split > 1)
    hipLaunchKernelGGL((decode_attn_merge_kernel<D, TO>), dim3((unsigned)S), dim3(128), 0, st,
                       (const float*)part, split, (TO*)O, ap.dst, ap.stride, ap.val);
  return hipGetLastError();
}

template <typename T, typename TO>
hipError_t launch_decode_d(int64_t d, const void* Q, const void* K, const void* V,
                           const ExpressSegs& g, int64_t S, int64_t ld, int64_t m, int split,
                           float* part, void* O, const Append& ap, hipStream_t st) {
  switch (d) {
    case 32: return launch_decode_t<T, 32, TO>(Q, K, V, g, S, ld, m, split, part, O, ap, st);
    case 64: return launch_decode_t<T, 64, TO>(Q, K, V, g, S, ld, m, split, part, O, ap, st);
    case 128: return launch_decode_t<T, 128, TO>(Q, K, V, g, S, ld, m, split, part, O, ap, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

int decode_attention_split(int64_t m) {
  const int64_t sp = (m + kDecodeKeysPerGroup - 1) / kDecodeKeysPerGroup;
  return (int)(sp < 1 ? 1 : (sp > kDecodeMaxSplit ? kDecodeMaxSplit : sp));
}

hipError_t launch_decode_attention(int dtype, int64_t d, int out_dtype, const void* Q,
                                   const void* K, const void* V, const ExpressSegs& g, int64_t S,
                                   int64_t ld, int64_t m, float* part, void* O, int32_t* app,
                                   int64_t app_stride, int32_t app_val, hipStream_t st) {
  if (m < 1 || g.n < 1) return hipErrorInvalidValue;
  const int split = decode_attention_split(m);
  const Append ap{app, app_stride, app_val};
  if (dtype == 0)
    return out_dtype == 0
               ? launch_decode_d<float, float>(d, Q, K, V, g, S, ld, m, split, part, O, ap, st)
               : launch_decode_d<float, bf16_t>(d, Q, K, V, g, S, ld, m, split, part, O, ap, st);
  return out_dtype == 0
             ? launch_decode_d<bf16_t, float>(d, Q, K, V, g, S, ld, m, split, part, O, ap, st)
             : launch_decode_d<bf16_t, bf16_t>(d, Q, K, V, g, S, ld, m, split, part, O, ap, st);
}

hipError_t launch_rows_copy(const int32_t* src, int64_t src_stride, int32_t* dst,
                            int64_t dst_stride, int64_t len, int64_t S, hipStream_t st) {
  if (len <= 0) return hipSuccess;
  dim3 grid((unsigned)((len + 255) / 256), (unsigned)S);
  hipLaunchKernelGGL(rows_copy_kernel, grid, dim3(256), 0, st, src, src_stride, dst, dst_stride,
                     len);
  return hipGetLastError();
}

hipError_t launch_vmax_rows(int dtype, const void* V, int64_t ld, int64_t d, const int32_t* idx,
                            int64_t in_stride, int64_t N, int64_t G, int64_t S,
                            uint32_t* vmax_bits, hipStream_t st) {
  // a call's words are counted in 32 bits
  const int64_t words = N * d * (dtype == 0 ? 4 : 2) / 16;
  if (words >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  const GridRows g = grid_rows(S * G, 64 * kVmaxWaves);
  const dim3 grid((unsigned)g.x, (unsigned)g.rows), block(64 * kVmaxWaves);
  if (dtype == 0)
    hipLaunchKernelGGL((vmax_rows_kernel<float>), grid, block, 0, st, (const float*)V, ld, d, idx,
                       in_stride, N, G, S * G, vmax_bits);
  else
    hipLaunchKernelGGL((vmax_rows_kernel<bf16_t>), grid, block, 0, st, (const bf16_t*)V, ld, d, idx,
                       in_stride, N, G, S * G, vmax_bits);
  return hipGetLastError();
}

hipError_t launch_express_keys(const ExpressSegs& segs, int64_t S, int64_t m, int64_t out_stride,
                               int32_t* idx, float* logw, hipStream_t st) {
  if (m <= 0 || segs.n < 1 || out_stride < m) return hipErrorInvalidValue;
  dim3 grid((unsigned)((m + 255) / 256), (unsigned)S);
  hipLaunchKernelGGL(express_keys_kernel, grid, dim3(256), 0, st, segs, m, out_stride, idx, logw);
  return hipGetLastError();
}

}  // namespace thin
