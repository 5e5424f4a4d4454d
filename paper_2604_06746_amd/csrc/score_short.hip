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
//   fp32: one row block (the products bind: more, lighter workgroups), v_mfma_f32_16x16x4_f32 or, of 64 components, bf16 thirds (ThirdsOfRows)
// Where the line lies (short_plan in api.cpp) and what it measured stands there.
// What a workgroup takes, by cycle counters: the keys' way into the CU (1500 keys of 256 bytes: 6 of 16 k cycles, 56 bytes a cycle;
// fp32: the products, 13 of 22 k), then maxima, sums and column sums, 8 k
// cycles.  Of the latter a third was LDS reads of every wave's maxima and sums by every lane (now a quarter each, exchanged between the
// rows of lanes) and sums over 16 lanes one at a time (now four together), and before the first tile 4 k cycles of line look-ups for the
// query operands (now by quads of lanes): a layer step of 1K tokens in fp32 18.0 -> 17.0 us, four short prompts 18.8 -> 16.6 us.
// Other workgroups that pull the keys into the XCD's L2 meanwhile: 0.1 us, not kept.
#include "common.h"

namespace skv {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;

constexpr int kWaves = 16;
constexpr float kLn2 = 0.6931471805599453f;

template <int CTRL>
__device__ __forceinline__ float dpp(float v) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true)); }
// The sums of s[0..3] over the 16 lanes of a DPP row, that of s[j] in the lanes j, j + 4, ... of it: two halvings inside the quads, then
// the quads added up (eleven instructions where four sums of sixteen lanes each take twenty).
__device__ __forceinline__ float row_sums(const float (&s)[4], bool odd, bool upper) {
  const float a = (odd ? s[1] : s[0]) + dpp<0xB1>(odd ? s[0] : s[1]);   // quad_perm 1,0,3,2
  const float b = (odd ? s[3] : s[2]) + dpp<0xB1>(odd ? s[2] : s[3]);
  float c = (upper ? b : a) + dpp<0x4E>(upper ? a : b);                 // quad_perm 2,3,0,1
  c += dpp<0x124>(c);                                                   // row_ror 4, 8
  return c + dpp<0x128>(c);
}
// a value of each of the four rows of lanes, combined, in all of them
template <class F>
__device__ __forceinline__ float over_groups(float v, F f) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = f(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// matrix operands of one row or key: lane l holds row l%16.  bf16: of every 32 components the eight of its quarter l/16;
// fp32: of every 16 components the four of its quarter (the four steps of a group take them in the same order on both sides):
// either way its piece c is the 16-byte piece PIECES (l/16) + c of the row (any order will do that both sides share).
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

// One side's eight components of a 16 x 16 x 32 product, by their upper, middle and lower eight bits: x = h + m + l (cut off,
// not rounded: a finite x stays finite, and what is left after two cuts has eight bits).  Exactly so from 2^-110 on; below, the lower third
// loses the bits under 2^-133, where bf16 numbers end.
struct Thirds {
  bf16x8 h, m, l;
  __device__ __forceinline__ static Thirds of(floatx4 a, floatx4 b) {
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    u32x4 h, m, l;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x = i < 2 ? a[2 * i] : b[2 * i - 4], y = i < 2 ? a[2 * i + 1] : b[2 * i - 3];
      const float x1 = x - upper(x), y1 = y - upper(y), x2 = x1 - upper(x1), y2 = y1 - upper(y1);
      h[i] = pair(x, y);
      m[i] = pair(x1, y1);
      l[i] = pair(x2, y2);
    }
    return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
  }
  __device__ __forceinline__ static float upper(float x) { return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); }
  // the bits of x that the lower third has no place for
  __device__ __forceinline__ static uint32_t lost(float x) {
    const float x1 = x - upper(x);
    return __float_as_uint(x1 - upper(x1)) & 0xFFFFu;
  }
  __device__ __forceinline__ static uint32_t pair(float x, float y) {
    return __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);
  }
};

// Query rows of 64 fp32 components as the products' second operand: eight of the nine products of thirds (the ninth is at most 2^-30 of
// the whole), the largest and the others summed apart.  The fp32 instruction runs on the vector ALU's multipliers, keeps all waves of the
// SIMD from them and took 60 cycles for four components; eight of these take 128 for 32, beside the 90 vector instructions that cut up
// the keys.  A layer step of 1K tokens 16.7 -> 15.9 us; its error against 64 bits (2-norm, N(0, 1) inputs with heavy hitters)
// 1.3e-7 -> 0.8e-7, eight times larger logits 1.6e-6 -> 0.6e-6: 32 products a rounding, not one.  (128 components: the thirds of the queries
// and the keys' registers do not fit, 24.5 -> 28.2 us.)
// The fp32 instruction takes a tile again whose logits are not finite (infinities have no thirds and end as NaN), and all tiles where what
// the lower third loses of numbers below 2^-110 may matter.  Of a key that is less than 2^-133 a component, and with queries (times the
// scale) below 2^90 less than 2^-37 of 64 products together: nothing to an exponent in fp32.  So the queries alone decide: larger ones,
// or such as lose something themselves.  One wave looks at them, and the others hear of it behind the barrier of the rows' maxima (0.1 us
// a layer step; every wave asking its queries 0.27, its keys 0.4).
struct ThirdsOfRows {
  typedef Frag<float, 64> F;
  static constexpr int STEPS = F::PIECES / 2;
  Thirds q[STEPS];
  __device__ __forceinline__ explicit ThirdsOfRows(const F& f) {
#pragma unroll
    for (int i = 0; i < STEPS; ++i) q[i] = Thirds::of(f.v[2 * i], f.v[2 * i + 1]);
  }
  // whether products of these rows (all of the wave's) and tiny numbers need the fp32 instruction
  __device__ __forceinline__ static bool inexact(const F& f, float c2) {
    uint32_t lost = 0u;
    float most = 0.f;
#pragma unroll
    for (int c = 0; c < F::PIECES; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lost |= Thirds::lost(f.v[c][e]);
        most = fmaxf(most, fabsf(f.v[c][e]));
      }
    return __ballot(lost != 0u || most * fmaxf(c2, 1.f) >= 0x1p90f) != 0ull;
  }
  __device__ __forceinline__ static F operand(const float* row) {
    F f;
#pragma unroll
    for (int c = 0; c < F::PIECES; ++c) f.v[c] = *reinterpret_cast<const floatx4*>(row + 4 * c);
    return f;
  }
  __device__ __forceinline__ void mul(floatx4& acc, const F& k, const float* row) const {   // row: where the lane's components stand
    floatx4 large = acc, small = {0.f, 0.f, 0.f, 0.f};
#define SKV_MUL(sum, x, y) sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(t.x, q[i].y, sum, 0, 0, 0)
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
      const Thirds t = Thirds::of(k.v[2 * i], k.v[2 * i + 1]);
      SKV_MUL(small, l, m); SKV_MUL(large, h, h);
      SKV_MUL(small, m, l); SKV_MUL(small, m, m);
      SKV_MUL(small, l, h); SKV_MUL(small, h, l);
      SKV_MUL(small, m, h); SKV_MUL(small, h, m);
    }
#undef SKV_MUL
    large += small;
    const float none = (large[0] - large[0]) + (large[1] - large[1]) + ((large[2] - large[2]) + (large[3] - large[3]));
    if (__builtin_expect(__ballot(none != 0.f) != 0ull, 0)) {   // (uniform)
      F::mul(acc, k, operand(row));
    } else {
      acc = large;
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
    constexpr int E = 16 / (int)sizeof(T);   // elements of a piece
    if constexpr (F::PIECES % 4 == 0) {      // by quads of lanes, see quad_transpose
#pragma unroll
      for (int c = 0; c < F::PIECES; ++c)
        qf[rb].v[c] = *reinterpret_cast<const floatx4*>(qg + (int64_t)min((rc * NRB + rb) * 16 + (l16 & 12) + c % 4, R - 1) * D +
                                                        (F::PIECES * lg + c / 4 * 4 + (lane & 3)) * E);
    } else {
      const T* row = qg + (int64_t)min((rc * NRB + rb) * 16 + l16, R - 1) * D;
#pragma unroll
      for (int c = 0; c < F::PIECES; ++c) qf[rb].v[c] = *reinterpret_cast<const floatx4*>(row + (F::PIECES * lg + c) * E);
    }
  }
  // Eight tiles: those past the sequence's end are left out (uniform in the wave), so that a length of just over 1024 keys
  // costs five of them (a layer step of 1280 keys, 32 heads on 8, window 8, in a graph: 20.4 -> 18.5 us).  With two or four
  // the tests cost more than they save (1024 fp32 keys, 8 heads, window 32: 20.2 -> 20.8 us).
  auto has = [&](int i) __attribute__((always_inline)) { return TW < 8 || tile0(i) < n; };
  if (has(0)) issue(0);
  if (SLOTS > 1 && TW > 1 && has(1)) issue(1);
  if constexpr (F::PIECES % 4 == 0) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int c = 0; c < F::PIECES; c += 4) {
        quad_transpose(qf[rb].v[c], qf[rb].v[c + 1], qf[rb].v[c + 2], qf[rb].v[c + 3]);
#pragma unroll
        for (int x = 0; x < 4; ++x) asm volatile("" : "+v"(qf[rb].v[c + x]));
      }
  }
  constexpr bool CUT = sizeof(T) == 4 && D == 64 && TW > 2;   // (300 keys, two tiles a wave: 12.1 us in a graph without, 12.3 with)
  const auto thirds = [&]() __attribute__((always_inline)) { if constexpr (CUT) return ThirdsOfRows(qf[0]); else return 0; }();
  static_assert(!CUT || NRB == 1, "one row block");
  __shared__ int again;   // all tiles with the fp32 instruction
  if constexpr (CUT)
    if (wave == 1) {
      const bool inexact = ThirdsOfRows::inexact(qf[0], c2);
      if (lane == 0) again = inexact;
    }
  auto q_row = [&]() __attribute__((always_inline)) { return qg + (int64_t)min(rc * 16 + l16, R - 1) * D + F::PIECES * lg * (16 / (int)sizeof(T)); };
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
      kf.v[c] = *reinterpret_cast<const floatx4*>(slot + (l16 * SEGS + ((F::PIECES * lg + c) ^ swz(l16))) * 16);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the operands are in registers: the slot may be overwritten
    __builtin_amdgcn_sched_barrier(0);
    if (i + SLOTS < TW && has(i + SLOTS)) issue(i + SLOTS);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) acc[rb][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (tile0(i) < n) {   // (uniform in the wave)
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        if constexpr (CUT) thirds.mul(acc[rb][i], kf, q_row());
        else F::mul(acc[rb][i], kf, qf[rb]);
      }
    }
  }

  // tiles that some row does not see whole (uniform in the wave): the masks and their clamp cost a fifth of the vector work
  auto masked = [&](int i) __attribute__((always_inline)) { return tile0(i) + 16 > (causal ? n - w : n); };
  // keys a row sees: all, or up to its own place in the window (the row modulo the window; rows stay below 65536)
  auto seen = [&](int row) __attribute__((always_inline)) {
    return causal ? n - w + row - w * (int)__umulhi((uint32_t)row, w_recip) + 1 : n;
  };
  float M[NRB], Z[NRB], E[NRB];
  auto row_maximum = [&](int rb) __attribute__((always_inline)) {
    float m = sM[lg][rb * 16 + l16];   // (each row of lanes reads a quarter of the waves': the reads were what the phase took)
#pragma unroll
    for (int v = 4; v < kWaves; v += 4) m = fmaxf(m, sM[v + lg][rb * 16 + l16]);
    return over_groups(m, [](float x, float y) { return fmaxf(x, y); }) * c2;
  };
#pragma unroll
  for (int round = 0; round < (CUT ? 2 : 1); ++round) {
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
      m = over_groups(m, [](float x, float y) { return fmaxf(x, y); });
      if (lg == 0) sM[wave][rb * 16 + l16] = m;
    }
    __syncthreads();
    if constexpr (CUT) {
      M[0] = row_maximum(0);
      if (round > 0 || __builtin_expect(__builtin_amdgcn_readfirstlane(again) == 0, 1)) break;   // (the same for all waves)
      const F qr = ThirdsOfRows::operand(q_row());
#pragma unroll
      for (int i = 0; i < TW; ++i) {
        acc[0][i] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (tile0(i) < n)
          F::mul(acc[0][i], ThirdsOfRows::operand(kg + (int64_t)min(tile0(i) + l16, n - 1) * kst + F::PIECES * lg * 4), qr);
      }
      __syncthreads();   // (the maxima have been read)
    }
  }
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    if constexpr (!CUT) M[rb] = row_maximum(rb);
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
    auto add = [](float x, float y) { return x + y; };
    z = over_groups(z, add);
    e = over_groups(e, add);
    if (lg == 0) { sZ[wave][rb * 16 + l16] = z; sE[wave][rb * 16 + l16] = e; }
  }
  __syncthreads();
  float inv[NRB];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    const int row = (rc * NRB + rb) * 16 + l16;
    Z[rb] = sZ[lg][rb * 16 + l16];
#pragma unroll
    for (int v = 4; v < kWaves; v += 4) Z[rb] += sZ[v + lg][rb * 16 + l16];
    Z[rb] = over_groups(Z[rb], [](float x, float y) { return x + y; });
    inv[rb] = row < R ? 1.0f / Z[rb] : 0.f;                                 // a padded row adds nothing
    if (wave == 0) {
      E[rb] = sE[lg][rb * 16 + l16];
#pragma unroll
      for (int v = 4; v < kWaves; v += 4) E[rb] += sE[v + lg][rb * 16 + l16];
      E[rb] = over_groups(E[rb], [](float x, float y) { return x + y; });
      if (lg == 0 && row < R) ent_out[row] = kLn2 * (__log2f(Z[rb]) - E[rb] / Z[rb]);
    }
  }
  float* out = colsum + ((int64_t)g * RC + rc) * total + tok0;
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int key = tile0(i) + 4 * lg + l16;   // (of the lanes that write: l16 < 4)
    if (tile0(i) >= n) continue;
    if (masked(i)) {   // (a row that is not a number stays off the keys that it does not see)
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (tile0(i) + 4 * lg + j >= seen((rc * NRB + rb) * 16 + l16)) acc[rb][i][j] = -INFINITY;
    }
    float s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s[j] = 0.f;
      if (masked(i)) {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) s[j] = acc[rb][i][j] == -INFINITY ? s[j] : fmaf(acc[rb][i][j], inv[rb], s[j]);
      } else {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) s[j] = fmaf(acc[rb][i][j], inv[rb], s[j]);
      }
    }
    const float mine = row_sums(s, lane & 1, lane & 2);
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
