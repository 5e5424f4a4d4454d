// Internal declarations shared by the libstructkv translation units (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <type_traits>

#include "../../include/structkv.h"

namespace skv {

// Record a thread-local error message and return the status.
structkv_status fail(structkv_status st, const char* fmt, ...);
void clear_error();

#define SKV_HIP_CHECK(expr)                                                              \
  do {                                                                                   \
    hipError_t _e = (expr);                                                              \
    if (_e != hipSuccess)                                                                \
      return skv::fail(STRUCTKV_ERR_HIP, "%s: %s", #expr, hipGetErrorString(_e));        \
  } while (0)

constexpr int kMaxBatch = STRUCTKV_MAX_BATCH;

// Per-sequence table passed by value in kernel arguments (host arrays never touch the device heap).
template <int N>
struct SeqTab {
  int64_t cu[N + 1];          // token offsets
  int64_t out_off[N + 1];     // output-row offsets (top-k / gather)
  int32_t k[N];               // top-k budget
  int32_t chunk_start[N + 1]; // cumulative key-chunk counts (scoring) / block counts (top-k)
  int32_t batch;
};
using SeqTable = SeqTab<kMaxBatch>;

// Kernels take the table in one of two sizes: the 1.6 KB of a full one are copied into the launch's argument buffer
// on every launch, which costs the host 4.3 us per launch against 2.75 us with a few words (back-to-back launches of a
// trivial kernel), and short layers are bound by the host's launches.
using SmallTable = SeqTab<8>;
template <class F>
void with_table(const SeqTable& s, F f) {
  if (s.batch > 8) { f(s); return; }
  SmallTable t;
  for (int i = 0; i <= 8; ++i) { t.cu[i] = s.cu[i]; t.out_off[i] = s.out_off[i]; t.chunk_start[i] = s.chunk_start[i]; }
  for (int i = 0; i < 8; ++i) t.k[i] = s.k[i];
  t.batch = s.batch;
  f(t);
}

// The short, latency-bound kernels of a layer (combine, reduce, accumulate, top-k, gather) call this first.  When
// layers run as chains on several streams such a kernel shares a SIMD with waves of another layer's scoring
// kernel -- those of score_mfma_ring.hip run at priority 1 while they have MFMAs to issue (those of score_mfma_wide.hip stay at
// the default) -- and would queue behind them, and it is the short kernels that sit on a chain's critical path.
#ifdef __HIPCC__
__device__ __forceinline__ void short_kernel_priority() { __builtin_amdgcn_s_setprio(2); }

// the exponent of a masked logit (-infinity) made one whose terms vanish: 2^-200 = 0, and 0 * -200 = 0.  The maximum is the
// one that passes NaN on: fmaxf would take a logit that is not a number for a masked one (and the builtin becomes fmaxf
// where a file is compiled without regard to NaN).
__device__ __forceinline__ float clamp_exponent(float x) {
  float r;
  asm("v_maximum3_f32 %0, %1, %2, %2" : "=v"(r) : "v"(x), "s"(-200.f));
  return r;
}

// merge partial softmax statistics (M, Z, E) of two disjoint key sets, log2 domain:
//   Z = sum 2^(x-M),  E = sum 2^(x-M) (x-M)
__device__ inline void merge_stats(float& M, float& Z, float& E, float M2, float Z2, float E2) {
  const float Mn = fmaxf(M, M2);
  const float d1 = M - Mn, d2 = M2 - Mn;
  const float f1 = __builtin_amdgcn_exp2f(d1), f2 = __builtin_amdgcn_exp2f(d2);
  E = (E + d1 * Z) * f1 + (E2 + d2 * Z2) * f2;
  Z = Z * f1 + Z2 * f2;
  M = Mn;
}
#endif

#ifdef __HIPCC__
// Eq. 4's means over window rows and heads for sequence b, by the first 256 threads of the calling workgroup (all of its
// threads call): eight lanes share a head, each sums every eighth window row, then a fixed shuffle tree
__device__ inline void finish_entropy(const float* __restrict__ row_ent, float* __restrict__ ent_head, float* __restrict__ entropy,
                                      int b, int Hq, int w, float (&hsum)[256]) {
  float part = 0.f;
  for (int h0i = 0; h0i < Hq && threadIdx.x < 256; h0i += 32) {   // (whole waves)
    const int h = h0i + (threadIdx.x >> 3);
    float s = 0.f;
    if (h < Hq) {
      const float* re = row_ent + ((int64_t)b * Hq + h) * w;
      for (int i = threadIdx.x & 7; i < w; i += 8) s += re[i];
    }
    s += __shfl_xor(s, 1);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 4);
    if (h < Hq && (threadIdx.x & 7) == 0) {
      s /= (float)w;
      ent_head[(int64_t)b * Hq + h] = s;
      part += s;
    }
  }
  if (threadIdx.x < 256) hsum[threadIdx.x] = part;
  __syncthreads();
  if (threadIdx.x == 0) {
    float s = 0.f;
    for (int t = 0; t < 256; t += 8) s += hsum[t];
    entropy[b] = s / (float)Hq;
  }
  __syncthreads();
}
#endif

#ifdef __HIPCC__
// Rows of 16-byte pieces as matrix operands: a lane holds pieces of ONE row, so neighbouring lanes of a load straight into that
// layout read different rows and every load instruction takes 64 line look-ups.  Loaded instead by quads of lanes that read 64
// contiguous bytes, register r the quad's row r, and exchanged inside the quad: 16 look-ups and, for four registers, 64 vector instructions.
typedef __attribute__((ext_vector_type(4))) float quad_piece_t;
template <int CTRL>
__device__ __forceinline__ void quad_exchange(quad_piece_t& a, quad_piece_t& b, bool second) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x = a[e], y = b[e];
    const float ox = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, true));
    const float oy = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(y), CTRL, 0xF, 0xF, true));
    a[e] = second ? oy : x;
    b[e] = second ? y : ox;
  }
}
// piece r of lane c of a quad <-> piece c of lane r
__device__ __forceinline__ void quad_transpose(quad_piece_t& v0, quad_piece_t& v1, quad_piece_t& v2, quad_piece_t& v3) {
  const bool odd = threadIdx.x & 1, upper = threadIdx.x & 2;
  quad_exchange<0xB1>(v0, v1, odd);     // quad_perm 1,0,3,2
  quad_exchange<0xB1>(v2, v3, odd);
  quad_exchange<0x4E>(v0, v2, upper);   // quad_perm 2,3,0,1
  quad_exchange<0x4E>(v1, v3, upper);
}
#endif

// ---- selection (radix select on order-preserving keys) ---------------------------------------
constexpr int kTopkBins = 2048;      // digits 0 and 1: 11 bits each; digit 2: the last 10 bits

#ifdef __HIPCC__
// order-preserving 32-bit key of a score: larger float <=> larger key; -0.0 orders as +0.0
__device__ inline uint32_t score_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
#endif

// How one selection call runs, by its longest searched prefix (n_b - keep_tail):
//   short  up to kShortSeq scores: one workgroup per sequence does everything in one launch (in a layer step several, which
//          select for themselves and copy a share of the kept rows each).  At 8192 scores 7.9 us against 12.5 us for the mid
//          form's three launches (in a layer step two of those fall away); at 16384 one workgroup needs 13.2 us.
//   mid    up to kMidSeq: a histogram whose fine bins lie around the scores that matter, so that the k-th largest's bin
//          holds few scores (the candidates) or, where the scores crowd together, few different ones; one launch lists
//          or counts them, one resolves them and places the indices (one does both for shorter sequences, see kDirectSeq).
//          131072 scores: 14.9 us spread over octaves, 18.7 all equal (the long form 23.1 and 23.9); in a layer step two
//          launches after the reduce kernel.
//   long   beyond: three radix digits (11/11/10 bits), one launch each, then the placement.  Every workgroup of the mid
//          form reads all candidates of its sequence and all counts before it, a thread each: 256 workgroups at most.
//          At the limit 16.4 us (mid; all equal 21.5) and 26.5 us (long; 28.6).
enum { kSelShort = 0, kSelMid = 1, kSelLong = 2 };
constexpr int kShortSeq = 8192;
constexpr int kMidSeq = 262144;
constexpr int kDirectSeq = 16384;   // ... of which up to here one launch behind the histogram (topk_direct_kernel), where ...
constexpr int kDirectBlocks = 256;  // ... no more workgroups than this read a whole sequence each

// Bins of the mid form, ascending with the keys, in four tiers of 1024: half octaves over all keys; around a centre 16 octaves
// in bins of 1/64 instead, four octaves in bins of 1/256, and an eighth of an octave in bins of 1/8192.  Even bins of 1/128
// octave held more scores than can be listed once the scores differ by a few per cent, as the in-degrees of diffuse attention
// do (N(0,1) queries and keys, a window of 64: 3 %), and for ties no width is small enough: a crowded bin is counted in
// kSubBins instead (compact), which for the innermost bins are single keys.  Why not three tiers: with end bins that took all
// keys beyond 32 octaves a crowd in one of them took 196 us at 131072 scores; with quarter octaves over all keys in their
// place a 32K-token layer whose threshold lies among heavy hitters, four octaves above the mean, took 0.9 us longer.  Why no
// finer third tier: every bin that is hit is an addition into the merged histogram (scores spread over two octaves, bins of
// 1/512: 0.6 us).
constexpr int kTiers = 4, kTierBins = 1024;
constexpr int kTierShift[kTiers + 1] = {22, 17, 15, 10, 10};   // (the last entry stands for what is not there)
static_assert((uint64_t)kTierBins << kTierShift[0] == (uint64_t)1 << 32, "the outermost tier covers all keys");
// bins of a tier that the next one takes the place of, and how many bins more its place then has, its own splits included
constexpr uint32_t kTierSplit[kTiers] = {kTierBins >> 5, kTierBins >> 2, kTierBins >> 5, 0};
constexpr uint32_t kTierExtra[kTiers] = {3 * kTierBins - 32 - 256 - 32, 2 * kTierBins - 256 - 32, kTierBins - 32, 0};
static_assert(kTierSplit[0] == 32 && kTierSplit[1] == 256 && kTierSplit[2] == 32, "the differences of the shifts");
constexpr int kUsedBins = kTierBins + (int)kTierExtra[0];
constexpr int kFineBins = 4096;                    // words of the histogram (the rest stays zero)
static_assert(kUsedBins <= kFineBins, "the bins fit the histogram");
constexpr int kSubBits = 10, kSubBins = 1 << kSubBits;   // bins of a crowded bin
static_assert(kTierShift[kTiers - 1] == kSubBits, "an innermost bin's sub-bins are single keys");
constexpr int kKeyEnds = kFineBins + kSubBins + 512;      // smallest and largest key of a crowded bin, by workgroup
static_assert(kKeyEnds + 2 * (kMidSeq / 1024) <= 3 * kTopkBins, "histograms, candidate counter and key ends share one sequence's words");
constexpr int kCandCap = 2048;                            // most candidates of a sequence that are listed (list_cap)

// where the tiers lie: a tier's first bin, in keys >> its shift, and that bin's number
struct BinTiers {
  uint32_t start[kTiers + 1], first[kTiers + 1];
};
__host__ __device__ inline BinTiers bins_around(uint32_t centre) {
  BinTiers t{};
#pragma unroll
  for (int i = 1; i < kTiers; ++i) {   // (in bins of the tier outside, which it must not leave)
    const uint32_t half = kTierSplit[i - 1] / 2, least = t.start[i - 1], most = least + kTierBins - 2 * half;
    const uint32_t c = centre >> kTierShift[i - 1];
    uint32_t at = c < least + half ? least : c - half;
    at = at < most ? at : most;
    t.start[i] = at << (kTierShift[i - 1] - kTierShift[i]);
    t.first[i] = t.first[i - 1] + (at - least);
  }
  return t;
}
// bin of a key
__host__ __device__ inline uint32_t fine_bin(uint32_t key, const BinTiers& t) {
  uint32_t bin = 0;
#pragma unroll
  for (int i = 0; i < kTiers; ++i) {   // (the innermost tier that has the key)
    const uint32_t k = (key >> kTierShift[i]) - t.start[i];
    const uint32_t extra = key >= (t.start[i + 1] << kTierShift[i + 1]) ? kTierExtra[i] : 0u;
    if (k < (uint32_t)kTierBins) bin = t.first[i] + k + extra;
  }
  return bin;
}
// first key of a bin, and the bits that tell its keys apart
__host__ __device__ inline void fine_range(uint32_t bin, const BinTiers& t, uint32_t* lo, uint32_t* width) {
#pragma unroll
  for (int i = 0; i < kTiers; ++i) {   // (the innermost tier in whose place the bin is)
    const uint32_t u = bin - t.first[i];
    const uint32_t extra = bin >= t.first[i + 1] ? kTierExtra[i] : 0u;
    if (u < kTierBins + kTierExtra[i]) {
      *lo = (t.start[i] + u - extra) << kTierShift[i];
      *width = (uint32_t)kTierShift[i];
    }
  }
}

#ifdef __HIPCC__
// Add a workgroup's LDS histogram of `nb` bins (even) into the merged one, two bins an addition: their counts stay below 2^32,
// so none carries into its neighbour.  What this costs is the number of additions (1024 bins of a near tier hit by each of 128
// workgroups: a 128K layer's reduce kernel 7.55 us one by one, 6.96 in pairs).
__device__ inline void merge_bins(const uint32_t* h /*LDS, 8-byte aligned*/, int nb, uint32_t* __restrict__ gh, int threads) {
  for (int i = threadIdx.x; i < nb / 2; i += threads) {
    const unsigned long long two = reinterpret_cast<const unsigned long long*>(h)[i];
    if (two) atomicAdd(reinterpret_cast<unsigned long long*>(gh) + i, two);
  }
}
// the bins for the in-degrees of a sequence, which add up to `mass` over n keys
__device__ inline BinTiers bins_around_mean(float mass, int64_t n) { return bins_around(score_key(mass / (float)(n > 0 ? n : 1))); }
#endif

// Bins of the pivot detector's rows (the in-degrees of one query head: non-negative, mean w/n), ascending with the keys: quarter
// octaves, and in the place of the 64 around the mean 16 octaves in bins of 1/64.  The k-th largest's bin holds about 1 % of a
// row then, where one of a quarter octave holds 10 to 25 %; finer ones mean more additions into the merged histograms (bins of
// 1/256 are hit by a thousand of a workgroup's 4096 scores).  No bin leaves its octave.
constexpr uint32_t kRowOuterShift = 21, kRowInnerShift = 17, kRowSplit = 64, kRowExtra = 1024 - kRowSplit;
static_assert((kRowSplit << (kRowOuterShift - kRowInnerShift)) - kRowSplit == kRowExtra && 1024 + kRowExtra <= (uint32_t)kTopkBins,
              "the inner bins take the place of kRowSplit outer ones and all fit the histogram");
// the first of the outer bins that are split, in keys >> kRowOuterShift (keys of non-negative scores: 1024 and up)
__host__ __device__ inline uint32_t row_bins_at(uint32_t centre) {
  const uint32_t c = centre >> kRowOuterShift, least = 1024u, most = 2048u - kRowSplit;
  const uint32_t at = c < least + kRowSplit / 2 ? least : c - kRowSplit / 2;
  return at < most ? at : most;
}
__host__ __device__ inline uint32_t row_bin(uint32_t key, uint32_t at) {
  const uint32_t o = key >> kRowOuterShift, shift = kRowOuterShift - kRowInnerShift;
  if (o < at) return o - 1024u;
  return o - at < kRowSplit ? (key >> kRowInnerShift) - (at << shift) + (at - 1024u) : o - 1024u + kRowExtra;
}
// the same for the rows of a call: in-degrees that add up to w over n keys.  Computed once, on the host, and handed to the three
// kernels that have to agree on the bins.
inline uint32_t row_bins_of(int w, int64_t n) {
  const float mean = (float)w / (float)n;
  uint32_t bits;
  __builtin_memcpy(&bits, &mean, sizeof(bits));
  return row_bins_at(bits | 0x80000000u);   // (score_key of a positive number)
}
// first key of a bin, and the bits that tell its keys apart
__host__ __device__ inline void row_bin_range(uint32_t bin, uint32_t at, uint32_t* lo, uint32_t* width) {
  const uint32_t in = bin - (at - 1024u);
  const bool inner = in < kRowSplit + kRowExtra;
  *width = inner ? kRowInnerShift : kRowOuterShift;
  *lo = inner ? ((at << (kRowOuterShift - kRowInnerShift)) + in) << kRowInnerShift
              : (bin + 1024u - (bin >= at - 1024u ? kRowExtra : 0u)) << kRowOuterShift;
}
constexpr int kRowWords = kTopkBins + 64;   // of a row: its histogram, the candidate counter and (first row) the finished rows

struct TopkWs {
  uint32_t* hist;    // [B][3][kTopkBins]; mid: the histogram in the first kFineBins words, that of a crowded bin in the next
                     //         kSubBins, then the candidate counter; from kKeyEnds on the key ends
  uint32_t* state;   // [B][8]; long: digit 0, k left after it, 22-bit prefix, k left after it
                     //         mid: first key of the k-th largest's bin, its width in bits, k left inside it, keys in it,
                     //              the centre of the bins
  uint32_t* suf;     // long: [blocks][1024] suffix sums of the workgroup's last-digit histogram
                     // mid: [blocks] x kSubBins 16-bit words: suffix sums of the workgroup's counts in a crowded bin, or, in
                     //      the words of a sequence's workgroups, its candidates (key, workgroup)
  uint32_t* meta;    // long: [blocks][2] keys above the 22-bit prefix, keys equal to it; mid: [blocks] keys above the bin
  int mode;          // kSelShort / kSelMid / kSelLong
  int direct;        // mid: one launch behind the histogram (at most kDirectSeq scores a sequence, kDirectBlocks workgroups), not two
  int beside;        // mid: other layers' scoring is expected to run at the same time (the second half of a layer step)
  float mass;        // > 0: the scores are in-degrees with this sum per sequence (fused layer step)
  const struct ReduceWork* red;   // (host) short: the kernel forms the scores itself (a layer step of short sequences)
  const struct CopyWork* copy;    // (host) or NULL: the last launch copies the kept rows as well (a layer step) ...
  int copy_parts;                 //        ... with this many workgroups per sequence
};

// What the reduce kernel does after pass 2; in a layer step of short sequences the selection's only launch does it.
struct ReduceWork {
  const float* colsum;   // [planes][total]
  int planes;
  int64_t total;
  float* indeg;
  const float* row_ent;  // [B][Hq][w]
  float* ent_head;
  float* entropy;
  int Hq, w;
  float* cen;            // or NULL; C <- lambda C + inv_w D
  float lambda, inv_w;
};
// ... up to this many tokens a sequence and planes: a workgroup sums its sequence's planes alone, eight or sixteen in flight
constexpr int kReduceShortSeq = 2048, kReduceShortPlanes = 64;

// What the scoring call's small kernels do for the selection that follows it in a fused layer step: the
// combine kernel zeroes the digit histograms, the reduce kernel histograms the first digit of the scores
// it has just formed and writes the kept window's indices.
struct SelectFusion {
  uint32_t* hist;        // [B][3][kTopkBins]; NULL = no fusion
  int32_t* idx_out;
  int keep_tail;
  int mode;              // kSelMid: fine bins; kSelLong: the top 11 bits
};

// Most keys of a workgroup: what the scoring kernels have LDS for to collect column sums in.  bf16 kernels by waves per
// workgroup; with NP column-sum planes per wave all tiles but the loop's last three are collected there (score_mfma_ring.hip).
constexpr int ring_key_cap(int nw) { return nw == 4 ? 2048 : 896; }
constexpr int kPlanesDirectTiles = 3;
constexpr int planes_lds_keys(int nw, int np) { return nw == 4 ? 1280 / np : (np <= 4 ? 1024 / np : 256) - 32 * kPlanesDirectTiles; }
constexpr int planes_key_cap(int nw, int np) { return planes_lds_keys(nw, np) + 32 * kPlanesDirectTiles; }
constexpr int kF32KeyCap = 1024;   // fp32 kernels: of up to four row-chunks

// the form of a selection whose longest searched prefix has `longest` scores
static inline int selection_mode(int64_t longest) { return longest <= kShortSeq ? kSelShort : longest <= kMidSeq ? kSelMid : kSelLong; }

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ---- rows copied by the launch that selects them ----------------------------------------------
// The cache store of a layer step whose rows the selection's last launch moves itself: 16-byte units, a power of two a row.
struct CopyWork {
  const uint8_t* src[2];   // K and V (one of them alone: twice the same)
  uint8_t* dst[2];
  int64_t ssh, sst, dsh, dst_tok;   // strides in bytes: head and token, source and destination
  uint32_t G, planes;      // KV heads; (tensor, head) pairs: G or 2 G
  uint32_t recip;          // floor(2^32 / planes) + 1: divides what stays below 2^32 / planes exactly (0: one plane)
  uint32_t upr_shift;      // log2 of the 16-byte units of a row
};
constexpr int kCopyRows = 512;   // most rows of a workgroup
// strides in bytes; false: other units or widths, which the gather kernel takes
inline bool make_copy_work(const void* k_src, const void* v_src, int64_t ssh, int64_t sst, void* k_dst, void* v_dst, int64_t dsh,
                    int64_t dst_tok, int G, int row_bytes, CopyWork* c) {
  *c = CopyWork{};
  c->src[0] = (const uint8_t*)k_src; c->src[1] = (const uint8_t*)v_src;
  c->dst[0] = (uint8_t*)k_dst; c->dst[1] = (uint8_t*)v_dst;
  if (!c->src[0]) { c->src[0] = c->src[1]; c->dst[0] = c->dst[1]; c->src[1] = nullptr; }
  if (!c->src[0]) return false;
  const int tensors = c->src[1] ? 2 : 1;
  if (tensors == 1) { c->src[1] = c->src[0]; c->dst[1] = c->dst[0]; }
  const uintptr_t bits = (uintptr_t)c->src[0] | (uintptr_t)c->src[1] | (uintptr_t)c->dst[0] | (uintptr_t)c->dst[1] |
                         (uintptr_t)ssh | (uintptr_t)sst | (uintptr_t)dsh | (uintptr_t)dst_tok | (uintptr_t)row_bytes;
  const uint32_t upr = (uint32_t)row_bytes / 16;
  if ((bits & 15) != 0 || (upr & (upr - 1)) != 0 || tensors * G > 2048) return false;   // (rows x planes^2 < 2^32: recip)
  c->ssh = ssh; c->sst = sst; c->dsh = dsh; c->dst_tok = dst_tok;
  c->G = (uint32_t)G;
  c->planes = (uint32_t)(tensors * G);
  c->recip = c->planes > 1 ? (uint32_t)(((uint64_t)1 << 32) / c->planes) + 1u : 0u;
  while ((1u << c->upr_shift) < upr) ++c->upr_shift;
  return true;
}

#ifdef __HIPCC__
// Every row is read once and written once and neither is touched again by this kernel: the 16-byte units move with
// the non-temporal policy, which keeps them from displacing what the next layer's scoring will read (measured on
// back-to-back launches: 16.0 -> 14.2 us at 34 MB, 52.6 -> 47.2 us at 221 MB; non-temporal stores alone were slower
// at 34 MB).  The builtins take clang's own vector types, not HIP's structs.
typedef unsigned __attribute__((ext_vector_type(4))) u32x4;
template <typename V> __device__ inline V load_once(const uint8_t* p) {
  if constexpr (sizeof(V) == 16) {
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    V r; r.x = t[0]; r.y = t[1]; r.z = t[2]; r.w = t[3];
    return r;
  } else {
    return *reinterpret_cast<const V*>(p);
  }
}
template <typename V> __device__ inline void store_once(uint8_t* p, V v) {
  if constexpr (sizeof(V) == 16) {
    const u32x4 t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<u32x4*>(p));
  } else {
    *reinterpret_cast<V*>(p) = v;
  }
}

// Copy rows [0, rows) of a list, `out_row` the first one's place in the destination and token0 + at(row) the source token, by all
// THREADS threads of the workgroup.  A row's (tensor, head) pairs lie next to each other in the order of the units: few rows still
// spread over all threads.  DEPTH units a thread are in flight.
template <int THREADS, int DEPTH, class At>
__device__ __forceinline__ void copy_rows(const CopyWork& c, uint32_t rows, int64_t out_row, int64_t token0, At at) {
  const uint32_t units = (rows * c.planes) << c.upr_shift;
  for (uint32_t u0 = threadIdx.x; u0 < units; u0 += DEPTH * THREADS) {
    uint4 v[DEPTH];
    uint8_t* to[DEPTH];
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) {
      const uint32_t u = u0 + i * THREADS;
      to[i] = nullptr;
      if (u < units) {
        const uint32_t part = (u & ((1u << c.upr_shift) - 1u)) << 4, q = u >> c.upr_shift;
        const uint32_t row = c.recip ? __umulhi(q, c.recip) : q, plane = q - row * c.planes;
        const bool second = plane >= c.G;
        const int64_t g = second ? plane - c.G : plane;
        v[i] = load_once<uint4>((second ? c.src[1] : c.src[0]) + g * c.ssh + (token0 + at(row)) * c.sst + part);
        to[i] = (second ? c.dst[1] : c.dst[0]) + g * c.dsh + (out_row + row) * c.dst_tok + part;
      }
    }
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
      if (to[i]) store_once<uint4>(to[i], v[i]);
  }
}
#endif

// ---- scoring plan: how one structkv_score_layer call is cut into workgroups ----------------
struct ScorePlan {
  int path;          // 0 = bf16 kernels, 1 = fp32 kernels (inputs widened), 2 = both passes at once (score_short.hip)
  int R;             // query rows per KV head: (H_q/G) * w
  int RPC;           // rows per row-chunk (a workgroup's share of R)
  int RC;            // row-chunks per KV head
  int KC;            // keys per key-chunk (one workgroup)
  int WK;            // partial statistics written per (row-chunk, key-chunk)
  int RB;            // 32-row blocks per wave (1 or 2)
  int NW;            // waves (row-chunks) per workgroup sharing the key tiles (bf16: 1 or 4; fp32: 1, 2 or 4)
  int CP;            // pass-2 column-sum planes per KV head (the waves of a workgroup add theirs up first)
  int planes;        // MFMA path, pass 2: 0, or column-sum planes per WAVE (1: a wave's rows are one query head's
                     // window; 2: each of its two 32-row blocks is) instead of one per workgroup: CP = query heads per
                     // KV head, and the planes are the per-head in-degrees
  int split;         // ... times the heads of every 32-row block (windows of 16 and 8: 2 and 4; planes = RB then), else 1
  int wide;          // 1 = the kernels of score_mfma_wide.hip (more than 128 rows of 128 components, long key chunks)
  int kshare;        // consecutive groups that read the same K head (1 in ordinary scoring; the per-head
                     // scoring of the pivot metrics runs every query head as its own group: H_q/G)
  int64_t n_chunks;  // sum over sequences of ceil(n_b / KC): the stride of the per-chunk statistics
  int64_t grid_chunks;  // key chunks covered by ONE launch (= n_chunks unless the batch is scored in groups)
  int stream_k;      // MFMA path: 1 = fetch K with the non-temporal policy (K is larger than the memory-side cache)
  // workspace carve (byte offsets)
  size_t off_stats, off_lse, off_rowent, off_colsum, off_enthead, total_bytes;
};

// Launchers (each enqueues on `stream`, returns hipGetLastError()).
hipError_t launch_score_mfma_ring(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq,
                                  const void* q, const void* k, int64_t ksh, int64_t kst, float c2,
                                  float* stats, const float* lse2, float* colsum, int64_t total,
                                  float* probs, int pass, hipStream_t st);
// the kernels of a plan with `wide` set (RB 2, NW 4, head_dim 128)
hipError_t launch_score_mfma_wide(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq,
                                  const void* q, const void* k, int64_t ksh, int64_t kst, float c2,
                                  float* stats, const float* lse2, float* colsum, int64_t total,
                                  float* probs, int pass, hipStream_t st);
hipError_t launch_score_f32(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq,
                            const void* q, const void* k, int64_t ksh, int64_t kst, float c2,
                            float* stats, const float* lse2, float* colsum, int64_t total,
                            float* probs, int pass, hipStream_t st);
// a plan of path 2: both passes in one launch
hipError_t launch_score_short(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq, const void* q, const void* k,
                              int64_t ksh, int64_t kst, float c2, float* row_ent, float* colsum, int64_t total, hipStream_t st);
// zero_words > 0: the kernel also clears that many 32-bit words at zero_ptr (the selection's histograms)
hipError_t launch_score_combine(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq,
                                const float* stats, float* lse2, float* row_ent, uint32_t* zero_ptr,
                                int64_t zero_words, hipStream_t st);
// fuse != NULL: seq.k / seq.out_off must hold the selection's budgets and output offsets
hipError_t launch_score_reduce(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq,
                               const float* colsum, int64_t total, float* indeg, const float* row_ent,
                               float* ent_head, float* entropy, float* centrality, float lambda, float inv_w,
                               const SelectFusion* fuse, hipStream_t st);
hipError_t launch_group_sums(const structkv_shape& s, const ScorePlan& p, const float* colsum, int64_t total,
                             float* groups, hipStream_t st);
hipError_t launch_accumulate(float* c, const float* d, int64_t n, float lambda, float inv_w, hipStream_t st);
hipError_t launch_topk(const float* scores, const SeqTable& seq, int keep_tail, int32_t* idx_out,
                       void* ws, hipStream_t st);
// The same selection split for a fused layer step.  topk_plan: workgroups per sequence (into plan->chunk_start)
// and the workspace carve.  launch_topk_rest: digits 1 and 2 and the ordered write, for a call whose histograms
// were zeroed, whose first digit was histogrammed and whose window indices were written by the scoring kernels
// (SelectFusion).
void topk_plan(const SeqTable& seq_in, int keep_tail, void* wsp, SeqTable* plan, TopkWs* ws, unsigned* blocks);
hipError_t launch_topk_rest(const float* scores, const SeqTable& plan, int keep_tail, const TopkWs& ws,
                            unsigned blocks, int32_t* idx_out, hipStream_t st);
size_t topk_workspace_bytes(int batch, int64_t total_tokens);
// the library's own top-k scratch on the current device (structkv_select_topk_static); no allocation.  It takes the calls
// that topk_static_fits names (whatever forms the selection takes, and whatever words those need)
bool topk_static_fits(int batch, int64_t total_tokens);
hipError_t topk_static_scratch(void** ptr, size_t* bytes);
// pivot metrics: partial sums part [H][kPivotMaxSlices][2] of every head, then the means over the heads
constexpr int kPivotMaxSlices = 64;
hipError_t launch_pivot_heads(const float* heads, int H, int64_t n, const int32_t* idx, int64_t k, float inv_w,
                              float* part, hipStream_t st);
hipError_t launch_zero_floats(float* p, int n, hipStream_t st);   // a fill kernel (safe inside a captured graph)
hipError_t launch_pivot_finish(const float* part, int H, int64_t n, float inv_w, int valid, float* sparsity,
                               float* variance, hipStream_t st);
// pivot metrics from the hot path's own scoring, whose pass 2 leaves the per-head in-degrees [H][n] in its column-sum planes
// (red.colsum): the reduce kernel's work for the layer, histograms hist [H][kRowWords] (cleared before) and variance partials
// var_part [H][pivot_shares(n)]; then the mass of each row's kk largest and the means over the heads.  at: row_bins_of(w, n), the same
// for both; cand: H x n floats, part_above: H x pivot_shares(n), state: [H][4], sums: [H][2]
constexpr int kPivotShare = 4096;
inline int pivot_shares(int64_t n) { return (int)((n + kPivotShare - 1) / kPivotShare); }
hipError_t launch_pivot_planes(const ReduceWork& red, uint32_t at, uint32_t* hist, float* var_part, hipStream_t st);
hipError_t launch_pivot_mass(const ReduceWork& red, uint32_t kk, uint32_t at, uint32_t* hist, uint32_t* state, float* cand,
                             float* part_above, const float* var_part, float* sums, float* sparsity, float* variance, hipStream_t st);
hipError_t launch_block_scores(const float* scores, const SeqTable& seq, int block, float* out, hipStream_t st);
hipError_t launch_positions(const int64_t* pos_src, const SeqTable& seq, const int32_t* idx, int64_t* pos_dst,
                            hipStream_t st);
hipError_t launch_gather(const void* k_src, const void* v_src, int64_t ssh, int64_t sst, void* k_dst,
                         void* v_dst, int64_t dsh, int64_t dst_, int G, int row_bytes,
                         const SeqTable& seq, const int32_t* idx, hipStream_t st);

}  // namespace skv
