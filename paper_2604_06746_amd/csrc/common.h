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
// kernel, which run at priority 1 while they have MFMAs to issue: at the default priority the short kernel would
// queue behind them, and it is the short kernels that sit on a chain's critical path.
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
//   short  up to kShortSeq scores: one workgroup per sequence does everything in one launch.  At 8192 scores 7.8 us
//          against 15.3 us for the mid form's four launches (in a layer step, where two of those fall away, about
//          even); at 16384 one workgroup needs 13.2 us.
//   mid    up to kMidSeq: a histogram whose fine bins lie around the scores that matter, so that the k-th largest's bin
//          holds few scores (the candidates); one launch lists them, one resolves them and places the indices.
//          131072 scores: 18.0 us, long form 22.6; in a layer step 12.5 us after the reduce kernel, long form 20.6.
//   long   beyond: three radix digits (11/11/10 bits), one launch each, then the placement.  Every workgroup of the mid
//          form reads all candidates of its sequence and all counts before it, a thread each: 256 workgroups at most.
//          At the limit 21.8 us (mid) and 24.4 us (long).
enum { kSelShort = 0, kSelMid = 1, kSelLong = 2 };
constexpr int kShortSeq = 8192;
constexpr int kMidSeq = 262144;
constexpr int kFineBins = 4096, kFineShift = 16;   // fine bins: 1/128 of an octave wide, 32 octaves of them
constexpr int kCandCap = 16384;                    // most candidates of a sequence that are listed (beyond: the scores are
constexpr int kCandTotal = 262144;                 // read again), and of a call

#ifdef __HIPCC__
// first key of the fine bins for the in-degrees of a sequence: they add up to `mass` over n keys, so no more than n/64 of
// them lie above 64 times their mean; 26 octaves below it and 6 above
__device__ inline uint32_t fine_base(float mass, int64_t n) {
  return score_key(mass / (float)(n > 0 ? n : 1)) - (26u << 23);
}
// bin of a key; the first and the last bin also take what lies beyond them
__device__ inline uint32_t fine_bin(uint32_t key, uint32_t base) {
  return key < base ? 0u : min((key - base) >> kFineShift, (uint32_t)(kFineBins - 1));
}
#endif

struct TopkWs {
  uint32_t* hist;    // [B][3][kTopkBins]; mid: the fine histogram in the first kFineBins words, then the candidate counter
  uint32_t* state;   // [B][8]; long: digit 0, k left after it, 22-bit prefix, k left after it
                     //         mid: first and last key of the k-th largest's bin, its width in bits, k left inside it,
                     //              keys in it, first key of the fine bins
  uint32_t* suf;     // long: [blocks][1024] suffix sums of the workgroup's last-digit histogram
  uint2* cand;       // mid: candidates (key, workgroup) of sequence b from min(cu[b], b*cand_cap) on
  uint32_t* meta;    // long: [blocks][2] keys above the 22-bit prefix, keys equal to it; mid: [blocks] keys above the bin
  int cand_cap;      // mid: most candidates listed per sequence
  int mode;          // kSelShort / kSelMid / kSelLong
  float mass;        // > 0: the scores are in-degrees with this sum per sequence (fused layer step)
  const struct ReduceWork* red;   // (host) short: the kernel forms the scores itself (a layer step of short sequences)
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

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

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
// pass 3 (a plan of path 2): both passes in one launch (launch_score_short); `stats` takes the row entropies
hipError_t launch_score_simt(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq,
                             const void* q, const void* k, int64_t ksh, int64_t kst, float c2,
                             float* stats, const float* lse2, float* colsum, int64_t total,
                             float* probs, int pass, hipStream_t st);
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
// pivot metrics from the hot path's own scoring, whose pass 2 leaves the per-head in-degrees [H][n] in its
// column-sum planes: first radix digit + variance partials, the top-k mass by radix select, the means over the heads
int pivot_plane_shares(int64_t n);
hipError_t launch_pivot_planes(const float* heads, int H, int64_t n, float inv_w, uint32_t* hist, float* part,
                               hipStream_t st);
hipError_t launch_topk_mass(const float* rows, int H, int64_t n, uint32_t kk, const TopkWs& ws, float* cand,
                            float* part_above, float* mass, float* tail, hipStream_t st);
hipError_t launch_pivot_finish_planes(const float* var_part, int Pv, const float* mass_part, int Pm, const float* tail,
                                      int H, int64_t n, float inv_w, float* sparsity, float* variance, hipStream_t st);
hipError_t launch_block_scores(const float* scores, const SeqTable& seq, int block, float* out, hipStream_t st);
hipError_t launch_positions(const int64_t* pos_src, const SeqTable& seq, const int32_t* idx, int64_t* pos_dst,
                            hipStream_t st);
hipError_t launch_gather(const void* k_src, const void* v_src, int64_t ssh, int64_t sst, void* k_dst,
                         void* v_dst, int64_t dsh, int64_t dst_, int G, int row_bytes,
                         const SeqTable& seq, const int32_t* idx, hipStream_t st);

}  // namespace skv
