// Scoring of short sequences in ONE launch: row statistics, entropies and column sums (paper Eq. 1, 2, 4) with the logits
// kept in registers between the maximum, the sums and the probabilities, instead of two passes over the keys with a merge
// of the partial statistics between them.
//
// Below a few thousand keys the two passes and the merge are three launches, each a few microseconds of ramp, load latency
// and drain around one to eight tiles per wave; nothing on the chip is busy.  Here a workgroup of sixteen waves holds ALL keys
// of one sequence against 16 NRB rows of one KV group: wave v takes the 16-key tiles v, v + 16, ... (TW of them, four logits
// per lane and row block each), the rows' maxima and sums cross the waves through LDS, and p = 2^(x-M) / Z needs neither a
// second exponential nor lse.  S^T = K Q^T on the 16 x 16 instructions: a lane owns one query row and four keys of a tile, so
// the statistics are per lane and the sum over the 16 rows is four DPP moves inside a row of lanes.
//   bf16: v_mfma_f32_16x16x32_bf16, two row blocks per workgroup (the keys' way from L2 into the CU is what a workgroup
//         costs: more rows per key, and half the column-sum planes)
//   fp32: v_mfma_f32_16x16x4_f32, one row block (n d / 8 cycles of matrix pipe per workgroup bind: more, lighter workgroups)
// Where the line lies (short_plan in api.cpp) and what it measured stands there.
#include "common.h"

namespace skv {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;

constexpr int kWaves = 16;
constexpr float kLn2 = 0.6931471805599453f;

// sum over the 16 lanes of a DPP row, in every lane of it: exchanges inside quads, then mirrored halves and rows
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float row_sum(float v) {
  return dpp_add<0x140>(dpp_add<0x141>(dpp_add<0x4E>(dpp_add<0xB1>(v))));
}

// matrix operands of one row or key: lane l holds row l%16.  bf16: of every 32 components the eight of its quarter l/16;
// fp32: of every 16 components the four of its quarter (the four steps of a group take them in the same order on both sides):
// either way its piece c is the 16-byte piece 4 c + l/16 of the row.
template <typename T, int D> struct Frag {
  static constexpr int PIECES = D * (int)sizeof(T) / 64;
  floatx4 v[PIECES];
  __device__ __forceinline__ static void mul(floatx4& acc, const Frag& a, const Frag& b) {
#pragma unroll
    for (int c = 0; c < PIECES; ++c) {
      if constexpr (sizeof(T) == 2) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.v[c]), __builtin_bit_cast(bf16x8, b.v[c]), acc, 0, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v[c][e], b.v[c][e], acc, 0, 0, 0);
      }
    }
  }
};

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* gbl_ptr_t;

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// grid: (sequence, row-chunk of 16 NRB rows, KV head), KV heads fastest; every sequence has at most 256 TW keys
template <class TAB, typename T, int D, int NRB, int TW>
__global__ __launch_bounds__(64 * kWaves) void score_short_kernel(
    const T* __restrict__ q, const T* __restrict__ k, int64_t ksh, int64_t kst, TAB seq, int Hq, int G, int w,
    uint32_t w_recip, int causal, float c2, int R, int RC, float* __restrict__ row_ent, float* __restrict__ colsum,
    int64_t total) {
  short_kernel_priority();
  __shared__ float sM[kWaves][16 * NRB], sZ[kWaves][16 * NRB], sE[kWaves][16 * NRB];
  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int g = blockIdx.x % G;
  const int t = blockIdx.x / G;
  const int rc = t % RC, b = t / RC;
  const int64_t tok0 = seq.cu[b];
  const int n = (int)(seq.cu[b + 1] - tok0);
  float* ent_out = row_ent + (int64_t)b * Hq * w + (int64_t)g * R;
  if (n == 0) {   // an empty sequence: entropies of zero
    const int row = rc * 16 * NRB + (int)threadIdx.x;
    if (threadIdx.x < 16 * NRB && row < R) ent_out[row] = 0.f;
    return;
  }
  const T* qg = q + ((int64_t)b * Hq * w + (int64_t)g * R) * D;
  const T* kg = k + (int64_t)g * ksh + tok0 * kst;
  // A wave's key tiles come through LDS of its own, by direct-to-LDS loads of whole 1 KB pieces: read straight into
  // operands, neighbouring lanes are different rows, every load instruction takes 64 line look-ups instead of 16, and a tile
  // per wave took 2.5 us.  16-byte piece (key, seg) sits at unit key * SEGS + (seg ^ swz(key)), which keeps the operand reads
  // (16 keys at one seg) free of bank conflicts.  No other wave touches the slots: no barrier, only waits.
  typedef Frag<T, D> F;
  constexpr int ROWB = D * (int)sizeof(T), SEGS = ROWB / 16, TILEB = 16 * ROWB, INST = TILEB / 1024;
  constexpr int SLOTS = TILEB <= 4096 ? 2 : 1;
  __shared__ __attribute__((aligned(1024))) uint8_t ring[kWaves * SLOTS * TILEB];
  uint8_t* slots = ring + wave * SLOTS * TILEB;
  auto tile0 = [&](int i) __attribute__((always_inline)) { return (i * kWaves + wave) * 16; };   // first key of the wave's tile i
  auto swz = [](int key) __attribute__((always_inline)) { return SEGS >= 16 ? key : key >> 1; };   // (keys 0 .. 15)
  auto issue = [&](int i) __attribute__((always_inline)) {   // (rows past the end re-read the last key)
#pragma unroll
    for (int ii = 0; ii < INST; ++ii) {
      const int unit = ii * 64 + lane, key = unit / SEGS, seg = (unit % SEGS) ^ swz(key);
      const T* src = kg + (int64_t)min(tile0(i) + key, n - 1) * kst + seg * (16 / (int)sizeof(T));
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)src, (lds_ptr_t)(slots + (i % SLOTS) * TILEB + ii * 1024), 16, 0, 0);
    }
  };
  F qf[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    const T* row = qg + (int64_t)min((rc * NRB + rb) * 16 + l16, R - 1) * D;
#pragma unroll
    for (int c = 0; c < F::PIECES; ++c) qf[rb].v[c] = *reinterpret_cast<const floatx4*>(row + (4 * c + lg) * (16 / (int)sizeof(T)));
  }
  // Eight tiles: those past the sequence's end are left out (uniform in the wave), so that a length of just over 1024 keys
  // costs five of them (a layer step of 1280 keys, 32 heads on 8, window 8, in a graph: 20.4 -> 18.5 us).  With two or four
  // the tests cost more than they save (1024 fp32 keys, 8 heads, window 32: 20.2 -> 20.8 us).
  auto has = [&](int i) __attribute__((always_inline)) { return TW < 8 || tile0(i) < n; };
  if (has(0)) issue(0);
  if (SLOTS > 1 && TW > 1 && has(1)) issue(1);
  // (never fewer than two: an array of exactly 32 floats becomes ONE 32-register value, and 400 registers spill)
  floatx4 acc[NRB < 2 ? 2 : NRB][TW];
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    if (!has(i)) break;
    if (i + 1 < TW && SLOTS > 1 && has(i + 1)) wait_vmcnt<INST>(); else wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    F kf;
    const uint8_t* slot = slots + (i % SLOTS) * TILEB;
#pragma unroll
    for (int c = 0; c < F::PIECES; ++c)
      kf.v[c] = *reinterpret_cast<const floatx4*>(slot + (l16 * SEGS + ((4 * c + lg) ^ swz(l16))) * 16);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the operands are in registers: the slot may be overwritten
    __builtin_amdgcn_sched_barrier(0);
    if (i + SLOTS < TW && has(i + SLOTS)) issue(i + SLOTS);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) acc[rb][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (tile0(i) < n) {   // (uniform in the wave)
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) F::mul(acc[rb][i], kf, qf[rb]);
    }
  }

  // tiles that some row does not see whole (uniform in the wave): the masks and their clamp cost a fifth of the vector work
  auto masked = [&](int i) __attribute__((always_inline)) { return tile0(i) + 16 > (causal ? n - w : n); };
  // keys a row sees: all, or up to its own place in the window (the row modulo the window; rows stay below 65536)
  auto seen = [&](int row) __attribute__((always_inline)) {
    return causal ? n - w + row - w * (int)__umulhi((uint32_t)row, w_recip) + 1 : n;
  };
  float M[NRB], Z[NRB], E[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    const int lim = seen((rc * NRB + rb) * 16 + l16);
    float m = -INFINITY;
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      if (!has(i)) break;
      if (masked(i)) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (tile0(i) + 4 * lg + j >= lim) acc[rb][i][j] = -INFINITY;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) m = fmaxf(m, acc[rb][i][j]);
    }
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    if (lg == 0) sM[wave][rb * 16 + l16] = m;
  }
  __syncthreads();
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    float m = sM[0][rb * 16 + l16];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) m = fmaxf(m, sM[v][rb * 16 + l16]);
    M[rb] = m * c2;
    float z = 0.f, e = 0.f;
#pragma unroll
    for (int i = 0; i < TW; ++i) {
      if (!has(i)) break;
      floatx4 xs;
#pragma unroll
      for (int j = 0; j < 4; ++j) xs[j] = fmaf(acc[rb][i][j], c2, -M[rb]);
      if (masked(i)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) xs[j] = clamp_exponent(xs[j]);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x = xs[j];
        const float p = __builtin_amdgcn_exp2f(x);
        acc[rb][i][j] = p;
        z += p;
        e = fmaf(p, x, e);
      }
    }
    z += __shfl_xor(z, 16); e += __shfl_xor(e, 16);
    z += __shfl_xor(z, 32); e += __shfl_xor(e, 32);
    if (lg == 0) { sZ[wave][rb * 16 + l16] = z; sE[wave][rb * 16 + l16] = e; }
  }
  __syncthreads();
  float inv[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    const int row = (rc * NRB + rb) * 16 + l16;
    Z[rb] = sZ[0][rb * 16 + l16]; E[rb] = sE[0][rb * 16 + l16];
#pragma unroll
    for (int v = 1; v < kWaves; ++v) { Z[rb] += sZ[v][rb * 16 + l16]; E[rb] += sE[v][rb * 16 + l16]; }
    inv[rb] = row < R ? 1.0f / Z[rb] : 0.f;                                 // a padded row adds nothing
    if (wave == 0 && lg == 0 && row < R) ent_out[row] = kLn2 * (__log2f(Z[rb]) - E[rb] / Z[rb]);
  }
  float* out = colsum + ((int64_t)g * RC + rc) * total + tok0;
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int key = tile0(i) + 4 * lg + l16;   // (of the lanes that write: l16 < 4)
    if (tile0(i) >= n) continue;
    float mine = 0.f;
    if (masked(i)) {   // (a row that is not a number stays off the keys that it does not see)
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (tile0(i) + 4 * lg + j >= seen((rc * NRB + rb) * 16 + l16)) acc[rb][i][j] = -INFINITY;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float s = 0.f;
      if (masked(i)) {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) s = acc[rb][i][j] == -INFINITY ? s : fmaf(acc[rb][i][j], inv[rb], s);
      } else {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) s = fmaf(acc[rb][i][j], inv[rb], s);
      }
      s = row_sum(s);
      if (l16 == j) mine = s;
    }
    if (l16 < 4 && key < n) out[key] = mine;
  }
}

template <typename T, int D, int NRB>
hipError_t launch_cfg(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq, const void* q, const void* k, int64_t ksh,
                      int64_t kst, float c2, float* row_ent, float* colsum, int64_t total, hipStream_t st) {
  // the row modulo the window, for causal masks: floor(2^32 / w) + 1; a window of one row sees every key
  const int causal = s.causal && s.window > 1;
  const uint32_t w_recip = s.window > 1 ? (uint32_t)(((uint64_t)1 << 32) / (uint64_t)s.window) + 1u : 0u;
  constexpr int kMostTiles = sizeof(T) == 2 ? 8 : 4;   // (fp32 operands leave no registers for more)
  int64_t longest = 0;
  for (int b = 0; b < seq.batch; ++b) longest = seq.cu[b + 1] - seq.cu[b] > longest ? seq.cu[b + 1] - seq.cu[b] : longest;
  if (p.RPC != 16 * NRB || longest > 16 * kWaves * kMostTiles) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((int64_t)seq.batch * s.n_kv_heads * p.RC)), blk(64 * kWaves);
#define SKV_SHORT(TW)                                                                                                   \
  hipLaunchKernelGGL((score_short_kernel<TAB, T, D, NRB, TW>), grid, blk, 0, st, (const T*)q, (const T*)k, ksh, kst, tab, \
                     s.n_q_heads, s.n_kv_heads, s.window, w_recip, causal, c2, p.R, p.RC, row_ent, colsum, total)
  with_table(seq, [&](const auto& tab) {
    using TAB = std::decay_t<decltype(tab)>;
    if (longest <= 16 * kWaves * 2) SKV_SHORT(2);
    else if (longest <= 16 * kWaves * 4) SKV_SHORT(4);
    else if constexpr (kMostTiles == 8) SKV_SHORT(8);
  });
#undef SKV_SHORT
  return hipGetLastError();
}

}  // namespace

hipError_t launch_score_short(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq, const void* q, const void* k,
                              int64_t ksh, int64_t kst, float c2, float* row_ent, float* colsum, int64_t total, hipStream_t st) {
#define SKV_CFG(T, d, nrb) \
  if (s.head_dim == d && p.RPC == 16 * nrb) return launch_cfg<T, d, nrb>(s, p, seq, q, k, ksh, kst, c2, row_ent, colsum, total, st)
  if (s.dtype == STRUCTKV_DTYPE_BF16) {
    SKV_CFG(uint16_t, 64, 1);
    SKV_CFG(uint16_t, 64, 2);
    SKV_CFG(uint16_t, 128, 1);
    SKV_CFG(uint16_t, 128, 2);
  } else {
    SKV_CFG(float, 64, 1);
    SKV_CFG(float, 128, 1);
  }
#undef SKV_CFG
  return hipErrorInvalidValue;
}

}  // namespace skv
