// Scoring kernels for fp32 inputs and for every shape the bf16 kernels do not cover (any head_dim <= 256, any window,
// any stride): the contraction runs on the fp32 matrix instruction v_mfma_f32_32x32x2_f32 (fp32 products and sums;
// bf16 inputs are widened, which is exact).  Same two passes and the same partial results as the bf16 kernels:
//   pass 1: per (row, key chunk) the running (M, Z, E) in the log2 domain   (paper Eq. 1, Eq. 4)
//   pass 2: p = 2^(x - lse2), column sums over a workgroup's rows           (paper Eq. 2)
//
// A wave owns 32 query rows as matrix operands in registers for the whole kernel and takes tiles of 32 keys, whose
// operands it reads from global memory straight into registers: lane l holds row l%32 and, of every eight
// components, the four of its half l/32, so a lane reads 16 contiguous bytes and a pair of lanes 32, and all bytes
// of a line are used within a tile (A and B see the same order of components, so the sums do not care).  A tile is
// d/2 matrix instructions of 64 cycles against 16 logits of softmax per lane: the matrix pipe binds, no LDS staging
// would help.  Four waves make a workgroup: NW of them hold different row-chunks of the KV group and take the same
// keys (their second to fourth read of a tile hits L1; their column sums are added before they leave the
// workgroup), and the 4/NW waves of a row-chunk take every (4/NW)-th tile, so that a short sequence with few rows
// still spreads over the chip.
//
// Measured, one layer's two passes, fp32, 8 heads x 32 rows, 1024 keys, d = 64: 107 us as dot products in vector
// instructions with both operands in LDS (16 x 16 threads, two LDS reads per fma, one key lane's dot products one
// after the other) -> 13.5 us here, most of it launch, load latency and the 32 matrix instructions of the one tile
// that each wave has; the whole layer 132 -> 39.6 us with the kernels of that time around them.  (Ordinary calls of that
// length now go through score_short.hip; these take longer ones and other head sizes, strides and alignments.)
#include "common.h"

#include <type_traits>

namespace skv {
namespace {

typedef __attribute__((ext_vector_type(16))) float floatx16;

constexpr float kNegBig = -1.0e30f;

__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

// components c .. c+3 of a row (zero from d on); VEC: the four are in bounds together and aligned
template <typename T, bool VEC>
__device__ __forceinline__ void load4(const T* __restrict__ row, int c, int d, float (&o)[4]) {
  if constexpr (VEC) {
    if (c < d) {
      if constexpr (sizeof(T) == 4) {
        const float4 v = *reinterpret_cast<const float4*>(row + c);
        o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
      } else {
        const ushort4 v = *reinterpret_cast<const ushort4*>(row + c);
        o[0] = widen(v.x); o[1] = widen(v.y); o[2] = widen(v.z); o[3] = widen(v.w);
      }
    } else {
      o[0] = o[1] = o[2] = o[3] = 0.f;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = c + i < d ? widen(row[c + i]) : 0.f;
  }
}

// DP: head_dim rounded up to 64, 128 or 256
template <class TAB, typename T, int DP, bool VEC, int PASS>
__global__ __launch_bounds__(256, DP == 256 ? 1 : 2) void score_f32_kernel(
    const T* __restrict__ q, const T* __restrict__ k, int64_t ksh, int64_t kst, int kshare, TAB seq, int Hq,
    int G, int d, int w, uint32_t w_recip, int causal, float c2, int R, int RC, int NW, int KC, int64_t n_chunks,
    float* __restrict__ stats, const float* __restrict__ lse2, float* __restrict__ colsum, int64_t total,
    float* __restrict__ probs) {
  constexpr int NC = DP / 8;   // groups of eight components; each lane holds four of every group
  __shared__ float sh[PASS == 1 ? 4 * 3 * 32 : 4 * kF32KeyCap];

  const int lane = threadIdx.x & 63, l32 = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wr = wave % NW, wk = wave / NW, nwk = 4 / NW;   // row-chunk inside the workgroup; first tile and tile step
  const int rcg = (RC + NW - 1) / NW;
  const int gp = blockIdx.x % G;
  const int g = kshare == 1 ? gp : (gp % (G / kshare)) * kshare + gp / (G / kshare);
  const int64_t t = blockIdx.x / G;
  const int rc_raw = (int)(t % rcg) * NW + wr;
  const bool live = rc_raw < RC;                 // a wave beyond the last row-chunk computes on it and writes nothing
  const int rc = live ? rc_raw : RC - 1;
  const int64_t chunk = t / rcg;
  int b = 0;
  while (b + 1 < seq.batch && chunk >= seq.chunk_start[b + 1]) ++b;
  const int64_t tok0 = seq.cu[b];
  const int64_t n = seq.cu[b + 1] - tok0;
  const int ni = (int)n;
  const int key0 = (int)((chunk - seq.chunk_start[b]) * (int64_t)KC);
  const int key_end = min(ni, key0 + KC);
  const int nsub = (key_end - key0 + 31) / 32;
  const int n_full = causal ? ni - w : ni;       // keys below n_full are visible to every row

  const int row = rc * 32 + l32;                 // as a matrix operand: row inside the KV group (h_local * w + i)
  const T* qr = q + ((int64_t)b * Hq * w + (int64_t)g * R + min(row, R - 1)) * d;
  float qf[NC][4];
#pragma unroll
  for (int c = 0; c < NC; ++c) load4<T, VEC>(qr, 8 * c + 4 * lh, d, qf[c]);

  const T* kg = k + (int64_t)(g / kshare) * ksh + tok0 * kst;

  float M = kNegBig, Z = 0.f, E = 0.f;           // pass 1: statistics of this lane's row
  const int lim1 = causal ? ni - w + row - w * (int)__umulhi((uint32_t)row, w_recip) + 1 : ni;
  float nl[16];                                  // pass 2: -lse2 of the 16 rows this lane sees (-inf: a padded row)
  if constexpr (PASS == 2) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = rc * 32 + 8 * (i / 4) + 4 * lh + (i % 4);
      nl[i] = r < R ? -lse2[(int64_t)b * G * R + (int64_t)g * R + r] : -INFINITY;
    }
  }

  for (int s = wk; s < nsub; s += nwk) {
    const int jbase = key0 + 32 * s;
    const T* kr = kg + (int64_t)min(jbase + l32, ni - 1) * kst;
    float kf[NC][4];
#pragma unroll
    for (int c = 0; c < NC; ++c) load4<T, VEC>(kr, 8 * c + 4 * lh, d, kf[c]);
    floatx16 acc = {};
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (PASS == 1) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[c][e], qf[c][e], acc, 0, 0, 0);
        else                     acc = __builtin_amdgcn_mfma_f32_32x32x2f32(qf[c][e], kf[c][e], acc, 0, 0, 0);
      }
    const bool masked = jbase + 32 > n_full;
    if constexpr (PASS == 1) {
      if (masked) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (jbase + 8 * (i / 4) + 4 * lh + (i % 4) >= lim1) acc[i] = -INFINITY;
      }
      float tm = acc[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) tm = fmaxf(tm, acc[i]);
      const float Mn = fmaxf(M, tm * c2);        // (finite: kNegBig at least)
      const float dl = M - Mn;
      const float f = __builtin_amdgcn_exp2f(dl);
      float z = Z * f, e = (E + dl * Z) * f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float x = clamp_exponent(fmaf(acc[i], c2, -Mn));
        const float p = __builtin_amdgcn_exp2f(x);
        z += p;
        e = fmaf(p, x, e);
      }
      M = Mn; Z = z; E = e;
    } else {
      const int j = jbase + l32;                 // this lane's key
      float pr[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) pr[i] = __builtin_amdgcn_exp2f(fmaf(acc[i], c2, nl[i]));
      if (masked && causal) {   // a row's window index is the row modulo the window (exact for rows below 65536)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int r = rc * 32 + 8 * (i / 4) + 4 * lh + (i % 4);
          if (j > ni - w + r - w * (int)__umulhi((uint32_t)r, w_recip)) pr[i] = 0.f;
        }
      }
      if (probs != nullptr && live && j < ni) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int r = rc * 32 + 8 * (i / 4) + 4 * lh + (i % 4);
          if (r < R) probs[((int64_t)g * R + r) * n + j] = pr[i];
        }
      }
      float cs0 = 0.f, cs1 = 0.f;
#pragma unroll
      for (int i = 0; i < 16; i += 2) { cs0 += pr[i]; cs1 += pr[i + 1]; }
      float cs = cs0 + cs1;
      cs += __shfl_xor(cs, 32);
      if (lh == 0) sh[wr * kF32KeyCap + 32 * s + l32] = live ? cs : 0.f;
    }
  }

  if constexpr (PASS == 1) {
    // lane halves hold disjoint keys of a row, the waves of a row-chunk disjoint tiles: halves first, then wave order
    const float M2 = __shfl_xor(M, 32), Z2 = __shfl_xor(Z, 32), E2 = __shfl_xor(E, 32);
    merge_stats(M, Z, E, M2, Z2, E2);
    if (wk > 0 && lh == 0) {
      sh[(wave * 3 + 0) * 32 + l32] = M;
      sh[(wave * 3 + 1) * 32 + l32] = Z;
      sh[(wave * 3 + 2) * 32 + l32] = E;
    }
    __syncthreads();
    if (wk == 0 && live && lh == 0) {
      for (int o = wave + NW; o < 4; o += NW)
        merge_stats(M, Z, E, sh[(o * 3 + 0) * 32 + l32], sh[(o * 3 + 1) * 32 + l32], sh[(o * 3 + 2) * 32 + l32]);
      float* sp = stats + (((int64_t)(g * RC + rc) * n_chunks + chunk) * 3) * 32 + l32;
      sp[0] = M;
      sp[32] = Z;
      sp[64] = E;
    }
  } else {
    __syncthreads();
    float* out = colsum + ((int64_t)g * rcg + t % rcg) * total + tok0 + key0;
    for (int i = threadIdx.x; i < key_end - key0; i += 256) {
      float s = sh[i];
      for (int o = 1; o < NW; ++o) s += sh[o * kF32KeyCap + i];
      out[i] = s;
    }
  }
}

template <typename T, int DP, bool VEC>
hipError_t launch_cfg(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq, const void* q, const void* k,
                      int64_t ksh, int64_t kst, float c2, float* stats, const float* lse2, float* colsum, int64_t total,
                      float* probs, int pass, hipStream_t st) {
  // the row modulo the window, for causal masks: floor(2^32 / w) + 1; a window of one row sees every key
  const int causal = s.causal && s.window > 1;
  const uint32_t w_recip = s.window > 1 ? (uint32_t)(((uint64_t)1 << 32) / (uint64_t)s.window) + 1u : 0u;
  const dim3 g((unsigned)(s.n_kv_heads * p.CP * p.grid_chunks)), blk(256);
#define SKV_ARGS                                                                                                    \
  g, blk, 0, st, (const T*)q, (const T*)k, ksh, kst, p.kshare, tab, s.n_q_heads, s.n_kv_heads, s.head_dim, s.window, \
      w_recip, causal, c2, p.R, p.RC, p.NW, p.KC, p.n_chunks, stats, lse2, colsum, total, probs
  with_table(seq, [&](const auto& tab) {
    using TAB = std::decay_t<decltype(tab)>;
    if (pass == 1) hipLaunchKernelGGL((score_f32_kernel<TAB, T, DP, VEC, 1>), SKV_ARGS);
    else hipLaunchKernelGGL((score_f32_kernel<TAB, T, DP, VEC, 2>), SKV_ARGS);
  });
#undef SKV_ARGS
  return hipGetLastError();
}

}  // namespace

hipError_t launch_score_f32(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq, const void* q,
                            const void* k, int64_t ksh, int64_t kst, float c2, float* stats, const float* lse2,
                            float* colsum, int64_t total, float* probs, int pass, hipStream_t st) {
  if (p.grid_chunks == 0) return hipSuccess;
  const size_t e = s.dtype == STRUCTKV_DTYPE_F32 ? 4 : 2;
  // four components per load: whole groups of eight, rows and pointers aligned to the load
  const bool vec = s.head_dim % 8 == 0 && kst % 4 == 0 && ksh % 4 == 0 && (((uintptr_t)q | (uintptr_t)k) & (4 * e - 1)) == 0;
#define SKV_F32(T, DP)                                                                                               \
  return vec ? launch_cfg<T, DP, true>(s, p, seq, q, k, ksh, kst, c2, stats, lse2, colsum, total, probs, pass, st)   \
             : launch_cfg<T, DP, false>(s, p, seq, q, k, ksh, kst, c2, stats, lse2, colsum, total, probs, pass, st)
  if (s.dtype == STRUCTKV_DTYPE_F32) {
    if (s.head_dim <= 64) { SKV_F32(float, 64); }
    if (s.head_dim <= 128) { SKV_F32(float, 128); }
    SKV_F32(float, 256);
  }
  if (s.head_dim <= 64) { SKV_F32(uint16_t, 64); }
  if (s.head_dim <= 128) { SKV_F32(uint16_t, 128); }
  SKV_F32(uint16_t, 256);
#undef SKV_F32
}

}  // namespace skv
