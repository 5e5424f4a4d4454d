// bf16 MFMA scoring kernels for more than 128 query rows per KV head and head_dim 128 (GQA 4 x window 64: the headline
// shape) in long key chunks (the plan says from where on; shorter ones stay with score_mfma_ring.hip), paper Eq. 1, Eq. 2,
// Eq. 4.  The work of a workgroup -- four waves of 64 rows that share 32-key tiles in an LDS ring, a key chunk, its partial
// statistics or column sums -- is that of score_mfma_ring.hip, whose plan, partial results and column-sum planes these kernels
// share; what differs is the loop.  (Loader, swizzle, rerun vote, planes and final write are that file's with other lane numbers: a
// fault found in one is to be looked for in the other.)  The order of requests, waits and tiles is score_schedule.h's.
//
// What bounds these shapes is the issue port at the clock that the power limit leaves.  A loop of nothing but this
// softmax and these MFMAs on N(0,1) data runs at 1.7 GHz with v_mfma_f32_32x32x16_bf16 and at 2.05 GHz with
// v_mfma_f32_16x16x32_bf16 (2.4 GHz on zeros), because the accumulators of the smaller product are moved half as often per
// multiplication; with HBM traffic and all else whole launches run at 1.9 GHz (128K tokens) and 1.65 (1M).  Per 32-key tile and 64-row
// wave (cycles a SIMD): 32 logits a lane x 20 (fma, add, fma of 4 cycles and an exponential of 8) and 32 MFMAs x 8.5, against 16 x 7.75
// of the larger ones.  By the counters that is 99 % of pass 1's and 92 % of pass 2's cycles at 1M tokens, 81 % and 75 % at
// 128K; what is left to lose is what a wave waits for: LDS, the tile barrier, branches.  Hence:
//   * 16 x 16 x 32 products, two by two of them a unit of 32 keys x 32 rows;
//   * the MFMAs of a unit are issued between the softmax instructions of the unit before, across tiles; a tile's operands are
//     requested from LDS piece by piece as soon as the registers of the tile before are free;
//   * a tile is one straight run of instructions: masked and ragged tiles, the chunk's very last ones, and a rerun with the
//     running maximum go through a plain loop of their own (which also keeps their registers out of this one).
// Two tiles a run: one has more address arithmetic a tile, four more code than is fetched in time by chunks of 16 tiles.
// 32 heads on 8, window 64, back to back, against 32 x 32 x 16 with the masks in the loop and only the MFMAs of a tile's
// second row block under the softmax of its first: 128K tokens pass 1 83.8 -> 82.6 us, pass 2 80.2 -> 79.0 us (one round of
// workgroups, of which start and end are a sixth); 1M tokens 625 -> 605 and 590 -> 560 us.
#include "score_schedule.h"

#include <utility>

namespace skv {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float floatx4;

constexpr float kNegBig = -1.0e30f;

// f(IntC<0>{}), f(IntC<1>{}), ... f(IntC<N - 1>{})
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F f, std::integer_sequence<int, I...>) { (f(IntC<I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void static_for(F f) { static_for_seq(f, std::make_integer_sequence<int, N>{}); }

// Sums over groups of lanes without a trip through the LDS crossbar: one vector instruction that swaps parts of two
// registers, and one addition.  add_halves: lanes 0..31 get a of lane l + a of lane l + 32, lanes 32..63 the same of b.
// add_rows: groups 0 and 2 of 16 lanes get a of their own and of the next group, groups 1 and 3 the same of b.
__device__ __forceinline__ float add_halves(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_rows(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* gbl_ptr_t;

// wait until at most N vector-memory operations and no LDS operation are outstanding (gfx9 encoding of s_waitcnt: vmcnt in
// bits 3:0 and 15:14, lgkmcnt in bits 11:8)
template <int N>
__device__ __forceinline__ void wait_loads_lds() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

constexpr int D = 128, NRB = 2, NW = 4, NBUF = 4;
constexpr int RPC = 32 * NRB;                 // query rows per wave
constexpr int SEGS = D / 8;                   // 16-byte pieces per key row
constexpr int TILE_BYTES = 32 * D * 2;
constexpr int IPW = 32 * SEGS / 64 / NW;      // wave-wide 1 KB load instructions per tile and wave
constexpr int PD = NBUF - 1;                  // tiles requested ahead of the one being consumed
constexpr int KP = 8;                         // pieces of 16 bytes that a lane holds of a tile's keys, and of a block of 32 rows
constexpr int NST = 2 * NRB;                  // query rows of a lane in pass 1
constexpr int kParked = 8;                    // tiles whose column sums can be parked

// PPW > 0 (pass 2): planes per head, SPLIT heads in 32 rows, as in score_mfma_ring.hip; NT: the non-temporal cache policy
template <class TAB, int PASS, bool DUMP, int PPW, bool NT, int SPLIT>
__global__ __launch_bounds__(64 * NW, 3) void score_mfma_wide_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, int64_t ksh, int64_t kst, int kshare,
    TAB seq, int Hq, int G, int w, uint32_t w_recip, int causal, float c2, int R, int RC, int KC, int64_t n_chunks,
    float* __restrict__ stats, const float* __restrict__ lse2, float* __restrict__ colsum,
    int64_t total, float* __restrict__ probs) {
  __shared__ __attribute__((aligned(1024))) uint8_t ring[NBUF * TILE_BYTES];
  // pass 2: the workgroup's column sums of its whole key chunk collect in LDS and are written out once at the
  // end, so that the key loop holds no global store (a store between the tile loads would make the
  // waits below wait for younger loads than they have to).  Each wave parks its sums of a tile (64 floats, two per key) in
  // csbuf[tile % 8] and one wave adds them up, in wave order, after a barrier in front of which every wave has waited for its
  // LDS operations.  Both buffers live in DYNAMIC LDS behind the ring (csout [KCAP] floats, then csbuf [8][NW][64] floats)
  // and are addressed by number, through asm: the ring stays the kernel's only LDS object, whose reads the compiler then never
  // orders behind the tile loads in flight.
  constexpr bool PLANES = PPW > 0;
  constexpr int NP = PLANES ? PPW * SPLIT : 1;   // planes per wave
  constexpr int KCAP = PASS == 2 ? (PLANES ? planes_lds_keys(NW, NP) : ring_key_cap(NW)) : 1;
  static_assert(!PLANES || (PASS == 2 && !DUMP && PPW <= NRB), "per-head planes are a pass-2 output");
  static_assert(SPLIT == 1 || PPW == NRB, "several heads per 32 rows: all of a wave's rows have planes of their own");

  const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
  // workgroup -> (KV head g, group of row-chunks, key chunk); wave -> row-chunk inside the group
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // a scalar: addresses built from it stay in SGPRs
  const int rcg = (RC + NW - 1) / NW;
  // groups that share a K head (kshare > 1) get workgroup numbers a multiple of G/kshare apart: with the
  // usual eight KV heads they run on the same XCD at about the same time, and its L2 serves the re-reads
  const int gp = blockIdx.x % G;
  const int g = kshare == 1 ? gp : (gp % (G / kshare)) * kshare + gp / (G / kshare);
  const int64_t t = blockIdx.x / G;
  // a wave beyond the last row-chunk still helps loading tiles and keeps the barriers matched; it
  // computes on a valid chunk (the last one) and simply does not write results
  const int rc_raw = (int)(t % rcg) * NW + wave;
  const bool live = rc_raw < RC;
  const int rc = live ? rc_raw : RC - 1;
  const int64_t chunk = t / rcg;
  const int grc = g * RC + rc;
  const int plane = g * rcg + (int)(t % rcg);   // pass 2: the workgroup's column-sum plane
  const int gheads = PLANES ? R / w : 1;        // ... or the planes, one per query head of the group
  int b = 0;
  while (b + 1 < seq.batch && chunk >= seq.chunk_start[b + 1]) ++b;
  const int64_t tok0 = seq.cu[b];
  const int ni = (int)(seq.cu[b + 1] - tok0);
  const int key0 = (int)((chunk - seq.chunk_start[b]) * (int64_t)KC);
  const int key_end = min(ni, key0 + KC);
  const int n_full = causal ? ni - w : ni;   // keys below n_full are visible to every row
  const int nsub = (key_end - key0 + 31) / 32;
  const TileChunk<PASS> chunk_tiles{key0, nsub, ni, n_full, causal};

  // ---- the row-chunk's queries as MFMA operands (registers, whole kernel) ----
  // piece p of block rb: row 16 (p / 4) + l16 of it, components 32 (p % 4) + 8 lg on (keys the same way)
  const uint16_t* qg = q + ((int64_t)b * Hq * w + (int64_t)g * R) * D;
  bf16x8 qf[NRB][KP];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int p = 0; p < KP; ++p)
      qf[rb][p] = *reinterpret_cast<const bf16x8*>(qg + (int64_t)min(rc * RPC + rb * 32 + p / 4 * 16 + l16, R - 1) * D + p % 4 * 32 + 8 * lg);
  // pass 2: lse2 of the rows whose logits a lane sees, requested with the queries; padded rows get +inf, so that their p is 0
  float row_lse[PASS == 2 ? 8 * NRB : 1] = {};
  if constexpr (PASS == 2) {
#pragma unroll
    for (int i = 0; i < 8 * NRB; ++i) {
      const int row = rc * RPC + i / 4 * 16 + 4 * lg + i % 4;
      const float v = lse2[(int64_t)b * G * R + (int64_t)g * R + min(row, R - 1)];
      row_lse[i] = row < R ? -v : -INFINITY;
    }
  }

  const uint16_t* kg = k + (int64_t)(g / kshare) * ksh + tok0 * kst;
  auto tile_key = [&](int s) __attribute__((always_inline)) { return chunk_tiles.key(s); };
  // Tile layout in LDS: 16-byte piece (key, seg) sits at unit key*SEGS + (seg ^ (key % 16)); any 16
  // consecutive keys at a fixed seg then hit 16 different groups of 4 banks (conflict-free operand reads).
  // Loader: instruction I, lane L writes unit I*64 + L, so it must fetch that unit's (key, seg).
  // Byte offset of the unit that this lane fetches first, relative to the tile's first key row; the second lies 16 rows on.
  static_assert(IPW == 2 && NW * 64 == 16 * SEGS, "two requests a wave, 16 rows apart");
  uint32_t voff = (uint32_t)((wave * 4 + lane / SEGS) * kst + ((lane % SEGS) ^ ((wave * 4 + lane / SEGS) & 15)) * 8) * 2u;
  const int64_t half_tile = 16 * kst * 2;
  // Tiles are requested in order; `next` is the first key row of the next one, of the chunk's last tile once that has been
  // requested (it never leaves the chunk).
  const int64_t tile_stride = (PASS == 2 ? -32 : 32) * kst * 2;
  const uint8_t* next = nullptr;   // wave-uniform
  auto issue_full = [&](int s) __attribute__((always_inline)) {   // all 32 rows lie before the sequence's end
    uint8_t* slot = ring + (s % NBUF) * TILE_BYTES + wave * 1024;
    asm volatile("" : "+v"(voff));   // opaque: 32 bits beside a scalar base, not a 64-bit pair kept across the loop
    __builtin_amdgcn_global_load_lds((gbl_ptr_t)(next + voff), (lds_ptr_t)slot, 16, 0, NT ? 2 : 0);
    __builtin_amdgcn_global_load_lds((gbl_ptr_t)(next + half_tile + voff), (lds_ptr_t)(slot + NW * 1024), 16, 0, NT ? 2 : 0);
    if (chunk_tiles.more(s)) next += tile_stride;
  };
  // (the lane number is opaque where the rarer code forms something from it: nothing of that stays in registers across the loop)
  auto opaque_lane = [&]() __attribute__((always_inline)) { int l = lane; asm volatile("" : "+v"(l)); return l; };
  auto issue_tile = [&](int s) __attribute__((always_inline)) {
    const int jbase = tile_key(s);
    if (chunk_tiles.whole(s)) { issue_full(s); return; }
    // ragged tail: rows past the end re-read the last valid row (their logits are masked)
    uint8_t* slot = ring + (s % NBUF) * TILE_BYTES + wave * 1024;
    const int l = opaque_lane();
#pragma unroll
    for (int ii = 0; ii < IPW; ++ii) {
      const int unit = (ii * NW + wave) * 64 + l, key = unit / SEGS;
      const int seg = (unit % SEGS) ^ (key & 15);
      __builtin_amdgcn_global_load_lds((gbl_ptr_t)(next + (uint32_t)(min(key, ni - 1 - jbase) * kst + seg * 8) * 2u),
                                       (lds_ptr_t)(slot + ii * NW * 1024), 16, 0, NT ? 2 : 0);
    }
    if (chunk_tiles.more(s)) next += tile_stride;
  };
  // the first tiles are requested under the query operands' latency
  auto issue_first = [&]() __attribute__((always_inline)) {
    next = reinterpret_cast<const uint8_t*>(kg + (int64_t)tile_key(0) * kst);
    for (int s = 0; s < PD && s < nsub; ++s) issue_tile(s);
  };
  issue_first();

  // opaque to the compiler from here on, so that it keeps the operands in registers instead of re-loading
  // them inside the key loop (pinned only after ALL loads are in flight: one latency, not one per load)
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int p = 0; p < KP; ++p) asm volatile("" : "+v"(qf[rb][p]));

  // Operands of a tile, piece p: key 16 (p / 4) + l16, components as in qf.  Plain loads: an asm ds_read whose result is
  // waited for by a later asm statement is NOT safe -- the compiler may copy the "loaded" register in between, before the
  // data has arrived.
  bf16x8 kf[KP];
  uint32_t piece0 = (uint32_t)(l16 * SEGS + (lg ^ l16)) * 16u;   // where piece 0 lies in a tile; the others differ by an XOR
  auto read_piece = [&](int slot, auto p_tag) __attribute__((always_inline)) {
    constexpr int p = decltype(p_tag)::value;
    static_assert(SEGS == 16, "a key's 16 pieces fill 256 bytes");
    kf[p] = *reinterpret_cast<const bf16x8*>(ring + slot * TILE_BYTES + (piece0 ^ (p % 4 * 64)) + p / 4 * 16 * SEGS * 16);
  };
  auto read_tile = [&](int s) __attribute__((always_inline)) {
    static_for<KP>([&](auto p_tag) __attribute__((always_inline)) { read_piece(s % NBUF, p_tag); });
  };

  // Logit i of a unit (32 keys x 32 rows) belongs, in a lane, to 16-key half i / 8 and 16-row half i / 4 % 2 of it.
  // pass 1: row 16 (i / 4 % 2) + l16 of the block, key 16 (i / 8) + 4 lg + i % 4; pass 2: key 16 (i / 8) + l16, row
  // 16 (i / 4 % 2) + 4 lg + i % 4.
  auto stat_of = [](int rb, int i) { return 2 * rb + i / 4 % 2; };
  float M[NST], Z[NST], E[NST];   // pass 1: statistics of the lane's four query rows
#pragma unroll
  for (int i = 0; i < NST; ++i) { M[i] = kNegBig; Z[i] = 0.f; E[i] = 0.f; }
  // pass 2: column sums of the lane's two keys over the rows that it sees, kept apart where they are of different heads: which
  // sum logit i of block rb goes into, and whether it is the first there.  (SPLIT 4: of 16 rows 8 are of lane groups 0 and 1,
  // 8 of groups 2 and 3.)
  constexpr int NSUM = SPLIT > 1 ? 2 * NRB : PPW == 2 ? 2 : 1;
  float cs[NSUM][2] = {};
  auto sum_of = [](int rb, int i) { return SPLIT > 1 ? 2 * rb + i / 4 % 2 : PPW == 2 ? rb : 0; };
  auto starts_sum = [](int rb, int i) { return SPLIT > 1 ? i % 4 == 0 : i % 8 == 0 && (PPW == 2 || rb == 0); };

  constexpr int NM = 16;   // MFMAs of a unit: four k-steps of four products (keys, then rows)
  auto unit_mfma = [&](floatx4 (&acc)[4], auto rb_tag, auto m_tag) __attribute__((always_inline)) {
    constexpr int rb = decltype(rb_tag)::value, m = decltype(m_tag)::value, ks = m / 4, kb = m / 2 % 2, qb = m % 2, x = 2 * kb + qb;
    const floatx4 c = ks == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : acc[x];
    if constexpr (PASS == 1) acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[4 * kb + ks], qf[rb][4 * qb + ks], c, 0, 0, 0);
    else                     acc[x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[rb][4 * qb + ks], kf[4 * kb + ks], c, 0, 0, 0);
  };
  auto unit_mfmas = [&](floatx4 (&acc)[4], auto rb_tag) __attribute__((always_inline)) {
    static_for<NM>([&](auto m_tag) __attribute__((always_inline)) { unit_mfma(acc, rb_tag, m_tag); });
  };
  // The softmax arithmetic of a unit with everything it can need: masks, and in pass 1 the running maximum as the rows'
  // reference.  jb: the tile's first key.
  auto softmax_any = [&](floatx4 (&acc)[4], auto rb_tag, int jb) __attribute__((always_inline)) {
    constexpr int rb = decltype(rb_tag)::value;
    const int l = opaque_lane();
    if constexpr (PASS == 1) {
      if (jb + 32 > n_full) {   // the ragged tail and the causal triangle
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int row = rc * RPC + rb * 32 + i / 4 % 2 * 16 + (l & 15);   // (its place in the window: the row modulo the window)
          const int lim = causal ? ni - w + row - w * (int)__umulhi((uint32_t)row, w_recip) + 1 : ni;
          if (jb + i / 8 * 16 + 4 * (l >> 4) + i % 4 >= lim) acc[i / 4][i % 4] = -INFINITY;
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int t = 2 * rb + h;
        float mx = acc[h][0];
#pragma unroll
        for (int i = 1; i < 8; ++i) mx = fmaxf(mx, acc[h + i / 4 * 2][i % 4]);
        const float Mn = fmaxf(M[t], mx * c2);
        const float dl = M[t] - Mn;
        const float f = __builtin_amdgcn_exp2f(dl);
        E[t] = (E[t] + dl * Z[t]) * f;
        Z[t] *= f;
        M[t] = Mn;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int t = stat_of(rb, i);
        const float x = clamp_exponent(fmaf(acc[i / 4][i % 4], c2, -M[t]));
        const float p = __builtin_amdgcn_exp2f(x);
        Z[t] += p;
        E[t] = fmaf(p, x, E[t]);
      }
    } else {
      float p[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) p[i] = __builtin_amdgcn_exp2f(fmaf(acc[i / 4][i % 4], c2, row_lse[8 * rb + i % 8]));
      if (DUMP || (causal && jb + 32 > n_full)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int j = jb + i / 8 * 16 + (l & 15);
          const int r = rc * RPC + rb * 32 + i / 4 % 2 * 16 + 4 * (l >> 4) + i % 4;
          // causal only (keys past the end of the sequence are simply never written): a row's window index is the
          // row modulo the window (any window: heads may straddle row blocks), by multiplication with its
          // reciprocal -- exact for rows below 65536
          if (causal && j - (ni - w) > r - w * (int)__umulhi((uint32_t)r, w_recip)) p[i] = 0.f;
          if (DUMP && j < ni && r < R) probs[((int64_t)g * R + r) * ni + j] = p[i];
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        float& sum = cs[sum_of(rb, i)][i / 8];
        sum = starts_sum(rb, i) ? p[i] : sum + p[i];
      }
    }
  };
  // The MFMAs of one unit (rows rbn, result an) under the softmax of the one before (logits ap, rows rbp), in this order: a
  // logit's exponential, the next one's exponent, the sums of the one before, so that no instruction waits for the one in
  // front of it, and the MFMAs between them.  (Left to itself the scheduler puts the MFMAs first and the softmax behind
  // them.)  after(m) follows MFMA m: an operand of the next tile, requested from LDS as soon as its register is free.  The
  // MFMAs sit under the first two thirds of the logits: beside tile loads in flight the compiler waits for ALL LDS reads
  // before it uses one, and the last of them needs its time too.
  // FIXED reference in pass 1: M stays what the chunk's first keys set it to -- no maximum, no rescaling of the running sums
  // (a sixth of the vector instructions).  Any reference gives the same statistics as long as nothing overflows; whether
  // something came near that is checked after the loop.
  auto unit_step = [&](floatx4 (&an)[4], auto rbn, floatx4 (&ap)[4], auto rbp, auto after) __attribute__((always_inline)) {
    constexpr int rb = decltype(rbp)::value;
    float x[16], p[16];
    auto exponent = [&](auto L) __attribute__((always_inline)) {
      constexpr int i = decltype(L)::value;
      x[i] = fmaf(ap[i / 4][i % 4], c2, PASS == 1 ? -M[stat_of(rb, i)] : row_lse[PASS == 2 ? 8 * rb + i % 8 : 0]);
    };
    auto sums = [&](auto L) __attribute__((always_inline)) {
      constexpr int i = decltype(L)::value;
      if constexpr (PASS == 1) {
        Z[stat_of(rb, i)] += p[i];
        E[stat_of(rb, i)] = fmaf(p[i], x[i], E[stat_of(rb, i)]);
      } else {
        float& sum = cs[sum_of(rb, i)][i / 8];
        sum = starts_sum(rb, i) ? p[i] : sum + p[i];
      }
    };
    exponent(IntC<0>{});
    static_for<16>([&](auto L) __attribute__((always_inline)) {
      constexpr int i = decltype(L)::value;
      static_for<NM>([&](auto m_tag) __attribute__((always_inline)) {
        if constexpr (decltype(m_tag)::value * 11 / NM == i) { unit_mfma(an, rbn, m_tag); after(m_tag); }
      });
      p[i] = __builtin_amdgcn_exp2f(x[i]);
      if constexpr (i + 1 < 16) exponent(IntC<i + 1>{});
      if constexpr (i > 0) sums(IntC<i - 1>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    sums(IntC<15>{});
  };

  // pass 2: add up the waves' sums of tile s (see csbuf above for when this is safe).
  // The LDS accesses to csbuf and csout inside the key loop are written as asm: for compiler-generated ones the
  // compiler cannot always rule out that the tile loads in flight (which write LDS too) alias them, and then
  // waits for ALL of those loads (vmcnt 0) in front of the access, which empties the ring every tile.
  // The column-sum buffers never overlap the ring, so no such wait is needed.
  const uint32_t csout_lds = __builtin_amdgcn_groupstaticsize();   // dynamic LDS starts where the static part ends
  const uint32_t csbuf_lds = csout_lds + (uint32_t)KCAP * 4u;
  auto flush_colsum = [&](int s) __attribute__((always_inline)) {   // (both lane halves do the same)
    if constexpr (PASS == 2 && !PLANES) {
      const int l = opaque_lane();
      // key 16 h + c of a tile: lanes 32 h + c and 32 h + 16 + c
      const uint32_t a = csbuf_lds + (uint32_t)((s % kParked) * NW * 256) + (uint32_t)((l & 16) * 2 + (l & 15)) * 4u;
      // all reads AND their wait in ONE asm statement (nothing can get between a read and its wait; one LDS
      // round trip for the lot)
      float lo[4], hi[4];
      static_assert(NW == 4, "written out for four waves");
      asm volatile("ds_read_b32 %0, %8\n\tds_read_b32 %1, %8 offset:64\n\t"
                   "ds_read_b32 %2, %8 offset:256\n\tds_read_b32 %3, %8 offset:320\n\t"
                   "ds_read_b32 %4, %8 offset:512\n\tds_read_b32 %5, %8 offset:576\n\t"
                   "ds_read_b32 %6, %8 offset:768\n\tds_read_b32 %7, %8 offset:832\n\t"
                   "s_waitcnt lgkmcnt(0)"
                   : "=&v"(lo[0]), "=&v"(hi[0]), "=&v"(lo[1]), "=&v"(hi[1]), "=&v"(lo[2]), "=&v"(hi[2]),
                     "=&v"(lo[3]), "=&v"(hi[3])
                   : "v"(a));
      // a wave's sum of a key = its two lanes'; then the waves in order
      float sum = lo[0] + hi[0];
#pragma unroll
      for (int wv = 1; wv < 4; ++wv) sum += lo[wv] + hi[wv];
      const uint32_t o = csout_lds + (uint32_t)(128 * (nsub - 1 - s)) + (uint32_t)(l & 31) * 4u;
      asm volatile("ds_write_b32 %0, %1" : : "v"(o), "v"(sum) : "memory");
    }
  };
  // pass 2: park the column sums of tile s
  auto park_colsum = [&](int s) __attribute__((always_inline)) {
    const int l = opaque_lane();
    if constexpr (PASS == 2 && PLANES) {
      // every wave keeps its own sums, one list per head: groups of lanes added here, no exchange between waves.  Of a pair of
      // planes some lanes store one, the others the other.
      constexpr int PAIR = NP > 1 ? 2 : 1;
      const int key = SPLIT == 4 ? l & 31 : (l >> 5) * 16 + (l & 15);   // the lane's key, and its plane of the pair
      const int second = SPLIT == 4 ? l >> 5 : (l >> 4) & 1;
      const bool mine = PAIR == 2 || !second;
      const int half = PAIR == 2 ? second : 0, jbase = tile_key(s);
      const uint32_t a0 = csout_lds + (uint32_t)(((wave * NP + half) * KCAP + (jbase - key0 - 32 * kPlanesDirectTiles + key)) * 4);
      const bool last = jbase < key0 + 32 * kPlanesDirectTiles;   // the last tiles of the loop: straight to their planes
#pragma unroll
      for (int sp = 0; sp < NP; sp += PAIR) {
        float val;
        if constexpr (SPLIT == 4) {
          val = add_rows(cs[sp / 2][0], cs[sp / 2][1]);
        } else {
          const float a = add_halves(cs[sp][0], cs[sp][1]);
          val = add_rows(a, PAIR == 2 ? add_halves(cs[sp + PAIR - 1][0], cs[sp + PAIR - 1][1]) : a);
        }
        if (last) {
          const int head = rc * NP + sp + half;
          if (mine && live && head < gheads && jbase + key < key_end)
            colsum[((int64_t)g * gheads + head) * total + tok0 + jbase + key] = val;
        } else if (mine) {
          asm volatile("ds_write_b32 %0, %1" : : "v"(a0 + (uint32_t)(sp * KCAP * 4)), "v"(val) : "memory");
        }
      }
    } else if constexpr (PASS == 2) {   // no more exchange between lanes in the key loop than brings two sums a key into 64 lanes
      const float v = add_halves(cs[0][0], cs[0][1]);
      const uint32_t a = csbuf_lds + (uint32_t)(((s % kParked) * NW + wave) * 256) + (uint32_t)l * 4u;
      asm volatile("ds_write_b32 %0, %1" : : "v"(a), "v"(live ? v : 0.f) : "memory");
    }
  };

  int unflushed = 0;   // pass 2: the first tile whose parked sums have not been added up
  floatx4 acc[2][4];
  auto wait = [&](auto later) __attribute__((always_inline)) { wait_loads_lds<decltype(later)::value * IPW>(); };
  // a plain s_barrier, not __syncthreads(), whose fence waits for ALL outstanding loads and would drain the ring
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // The loop's step: one tile that every row sees whole, software-pipelined over its units: the MFMAs of a unit run under the
  // softmax of the unit before, and the first unit of the tile was computed in the step before, or by this:
  auto begin = [&](int s) __attribute__((always_inline)) {
    read_tile(s);
    unit_mfmas(acc[0], IntC<0>{});
    if (PASS == 1 && s == 0) {   // the first keys set the reference
      unit_mfmas(acc[1], IntC<1>{});
#pragma unroll
      for (int t = 0; t < NST; ++t) {
        float mx = acc[t / 2][t % 2][0];
#pragma unroll
        for (int i = 1; i < 8; ++i) mx = fmaxf(mx, acc[t / 2][t % 2 + i / 4 * 2][i % 4]);
        M[t] = mx * c2;
      }
    }
  };
  auto step = [&](int s) __attribute__((always_inline)) {
    const int in = (s + 1) % NBUF;
    asm volatile("" : "+v"(piece0));   // opaque: one register across the loop, not four
    auto read = [&](auto m_tag) __attribute__((always_inline)) {   // (behind the second of the two MFMAs that use a piece)
      constexpr int m = decltype(m_tag)::value;
      if constexpr (m % 2 == 1) read_piece(in, IntC<4 * (m / 2 % 2) + m / 4>{});
    };
    unit_step(acc[1], IntC<1>{}, acc[0], IntC<0>{}, read);
    unit_step(acc[0], IntC<0>{}, acc[1], IntC<1>{}, [](auto) __attribute__((always_inline)) {});
    if constexpr (PASS == 1) {   // (computed here and not, all of it, behind the loop, where it is next needed)
#pragma unroll
      for (int i = 0; i < NST; ++i) asm volatile("" : "+v"(Z[i]), "+v"(E[i]));
    }
  };
  // one tile with everything it can need, by itself
  auto any = [&](int s) __attribute__((always_inline)) {
    read_tile(s);
    static_for<NRB>([&](auto rb) __attribute__((always_inline)) { unit_mfmas(acc[0], rb); softmax_any(acc[0], rb, tile_key(s)); });
  };
  auto add_one = [&](int s) __attribute__((always_inline)) { if (wave == s % NW) flush_colsum(s); };
  auto add_each = [&](int s) __attribute__((always_inline)) { flush_colsum(s + wave); };
  auto ops = chunk_ops(wait, barrier, issue_tile, issue_full, begin, step, any, park_colsum, add_one, add_each);
  // the whole key chunk, its first PD tiles already requested (the attention rows themselves only come out of the plain tiles)
  auto run_chunk = [&](bool fast) __attribute__((always_inline)) {
    go_through_chunk<PD, NW, PASS == 2 && !PLANES>(chunk_tiles, fast && !DUMP, unflushed, ops);
  };
  if constexpr (PASS == 1) {
    // Fast run with the fixed reference; then a workgroup-wide vote (every wave has to take part in a rerun:
    // they load the tiles together).  A sum whose exponent shows that some logit lay 2^60 above its row's
    // reference (or that is inf / NaN) sends the workgroup through the chunk again with the running maximum.
    const uint32_t flag_lds = __builtin_amdgcn_groupstaticsize();   // one word of dynamic LDS
    if (threadIdx.x == 0) asm volatile("ds_write_b32 %0, %1" : : "v"(flag_lds), "v"(0) : "memory");
    run_chunk(true);
    bool suspect = false;
#pragma unroll
    for (int i = 0; i < NST; ++i) {
      const uint32_t ez = (__float_as_uint(Z[i]) >> 23) & 0xFFu, ee = (__float_as_uint(E[i]) >> 23) & 0xFFu;
      suspect = suspect || ez >= 127u + 60u || ee >= 127u + 66u;
    }
    if (nsub > 0) {   // (with no tile there was no barrier either: nothing ran, nothing to vote on)
      if (__builtin_amdgcn_ballot_w64(suspect) != 0 && lane == 0)
        asm volatile("ds_write_b32 %0, %1" : : "v"(flag_lds), "v"(1) : "memory");
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __syncthreads();
      int flag;
      asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(flag) : "v"(flag_lds) : "memory");
      if (__builtin_amdgcn_readfirstlane(flag) != 0) {
#pragma unroll
        for (int i = 0; i < NST; ++i) { M[i] = kNegBig; Z[i] = 0.f; E[i] = 0.f; }
        issue_first();
        run_chunk(false);
      }
    }
#pragma unroll
    for (int i = 0; i < NST; ++i) {
      // the four groups of lanes hold disjoint key subsets of the same query row
#pragma unroll
      for (int x = 16; x <= 32; x <<= 1) {
        const float M2 = __shfl_xor(M[i], x), Z2 = __shfl_xor(Z[i], x), E2 = __shfl_xor(E[i], x);
        merge_stats(M[i], Z[i], E[i], M2, Z2, E2);
      }
      if (live && lg == 0) {
        float* sp = stats + (((int64_t)grc * n_chunks + chunk) * 3) * RPC + i * 16 + l16;
        sp[0] = M[i];
        sp[RPC] = Z[i];
        sp[2 * RPC] = E[i];
      }
    }
  } else {
    run_chunk(true);
    // the asm LDS writes are unknown to the compiler, so the barriers' own fences do not wait for them
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if constexpr (PLANES) {
      const int head0 = (int)(t % rcg) * NW * NP;   // the workgroup's first head (heads beyond the group's do not exist)
      for (int pl = 0; pl < NW * NP && head0 + pl < gheads; ++pl) {
        float* out = colsum + ((int64_t)g * gheads + head0 + pl) * total + tok0 + key0 + 32 * kPlanesDirectTiles;
        for (int i = threadIdx.x; i < key_end - key0 - 32 * kPlanesDirectTiles; i += 64 * NW) {   // (the other tiles' sums are there already)
          float v;
          const uint32_t a = csout_lds + (uint32_t)(pl * KCAP + i) * 4u;
          asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(a));
          out[i] = v;
        }
      }
    } else {
      for (int s = unflushed + wave; s < nsub; s += NW) flush_colsum(s);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __syncthreads();
      float* out = colsum + (int64_t)plane * total + tok0 + key0;
      for (int i = threadIdx.x; i < key_end - key0; i += 64 * NW) {
        float v;
        asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(csout_lds + (uint32_t)i * 4u));
        out[i] = v;
      }
    }
  }
}

}  // namespace

hipError_t launch_score_mfma_wide(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq, const void* q, const void* k,
                                  int64_t ksh, int64_t kst, float c2, float* stats, const float* lse2, float* colsum,
                                  int64_t total, float* probs, int pass, hipStream_t st) {
  if (!p.wide || s.head_dim != D || p.RB != NRB || p.NW != NW) return hipErrorInvalidValue;
  const dim3 g((unsigned)((int64_t)s.n_kv_heads * ceil_div(p.RC, NW) * p.grid_chunks)), blk(64 * NW);
  // dynamic LDS: pass 1 the word of the rerun vote; pass 2 the column sums of the key chunk and the waves' parked sums
  const int ppw = pass == 2 && probs == nullptr ? p.planes : 0, np = ppw * p.split;
  const unsigned dyn = pass == 1 ? 16u : np ? (unsigned)(NW * np * planes_lds_keys(NW, np) * 4)
                                            : (unsigned)(ring_key_cap(NW) * 4 + kParked * NW * 64 * 4);
  // causal masks: floor(2^32 / w) + 1 (the row modulo the window); a window of one row sees every key
  const int causal = s.causal && s.window > 1;
  const uint32_t w_recip = s.window > 1 ? (uint32_t)(((uint64_t)1 << 32) / (uint64_t)s.window) + 1u : 0u;
  if (p.split > 1 && ppw != NRB && ppw != 0) return hipErrorInvalidValue;
  with_table(seq, [&](const auto& tab) {
    using T = std::decay_t<decltype(tab)>;
#define SKV_WIDE(PASS, DUMP, PPW, NT, SPLIT)                                                                          \
  hipLaunchKernelGGL((score_mfma_wide_kernel<T, PASS, DUMP, PPW, NT, SPLIT>), g, blk, dyn, st, (const uint16_t*)q,      \
                     (const uint16_t*)k, ksh, kst, p.kshare, tab, s.n_q_heads, s.n_kv_heads, s.window, w_recip, causal, c2, \
                     p.R, p.RC, p.KC, p.n_chunks, stats, lse2, colsum, total, probs)
    if (pass == 1 && p.stream_k) SKV_WIDE(1, false, 0, true, 1);
    else if (pass == 1) SKV_WIDE(1, false, 0, false, 1);
    else if (ppw && p.split == 2) SKV_WIDE(2, false, NRB, false, 2);
    else if (ppw && p.split == 4) SKV_WIDE(2, false, NRB, false, 4);
    else if (ppw == 1) SKV_WIDE(2, false, 1, false, 1);
    else if (ppw == 2) SKV_WIDE(2, false, 2, false, 1);
    else if (probs == nullptr && p.stream_k) SKV_WIDE(2, false, 0, true, 1);
    else if (probs == nullptr) SKV_WIDE(2, false, 0, false, 1);
    else SKV_WIDE(2, true, 0, false, 1);
#undef SKV_WIDE
  });
  return hipGetLastError();
}

}  // namespace skv
