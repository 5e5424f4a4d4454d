// Exact, deterministic top-k selection (paper Eq. 10 / Eq. 13) on order-preserving 32-bit keys, then an index-ordered
// compaction.  Ties at the threshold go to the lowest indices; no floating-point atomics anywhere; stream order is the
// only synchronisation between launches (no workgroup ever waits for another one).
//
// These kernels move a few bytes per score; launches, dependent memory round trips and barriers are what they cost.
// So there are three forms, by the longest sequence (topk_plan):
//   short (one launch): a workgroup of 1024 threads per sequence (several where they also copy the kept rows), keys in registers; the range between the smallest and
//     the largest key is cut into 2048 bins, then the k-th largest's bin again, until it is one key.
//   mid (fused into the scoring kernels: two launches or one; alone: four or three):
//     [init]    zero the histogram, write the kept window, find from a sample where the k-th largest lies (alone only)
//     [hist]    histogram over bins that are finest around it (in a layer step the reduce kernel does this)
//     compact   find the k-th largest's bin; every workgroup counts its scores above the bin and lists those in it -- the
//               candidates -- or, where these are many, counts them in 1024 sub-bins, for all workgroups and for its own
//     place     every workgroup resolves the candidates (in registers, bins as in the short form) or the sub-bins down to
//               the k-th key, counts what the workgroups before it have selected, and writes its own indices
//     or, up to 16384 scores, direct: the work of both, every workgroup on all scores of its sequence
//   long: radix select in three digit passes (11/11/10 bits from the top):
//     init, hist0 (top digit; a layer step's scoring kernels do both), hist1, hist2 (which also publishes the suffix
//     sums of each workgroup's last-digit histogram), write.
#include "common.h"

#include <algorithm>
#include <mutex>

namespace skv {
namespace {

// Scratch of structkv_select_topk_static, the entry point for callers that cannot allocate: the histograms,
// search state and per-workgroup suffix sums that structkv_select_topk takes from the caller's workspace live
// here instead.  Every GPU the library runs on holds its own copy until the process ends.  In host code the
// array's name is only a handle for hipGetSymbolAddress; kernels get the address that call returns.
// It takes the calls whose histograms and suffix sums fill 4 MiB at most; the mid form's words come on top.
constexpr size_t kStaticScratchLists = (size_t)4 << 20;
constexpr size_t kStaticScratchBytes = kStaticScratchLists + kMaxBatch * 256;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kThreads = 256;
constexpr int kBins = kTopkBins;          // digits 0 and 1: 11 bits
constexpr int kLowBins = 1024;            // digit 2: 10 bits
constexpr int kTargetPerBlock = 2048;     // long form: most scores a workgroup holds in registers (eight per thread)
constexpr int kSmallTarget = 1024;        // share of a workgroup when the whole call is short: more, lighter
constexpr int64_t kSmallTotal = 262144;   // workgroups shorten each kernel's serial part
constexpr int kMaxBlocksPerSeq = 1024;    // beyond that a workgroup's share grows instead

// the calling workgroup's sequence and its contiguous share [lo, hi) of the prefix that is searched
struct Share {
  int b;
  uint32_t nblk, blk, first;   // workgroups of the sequence, rank of this one, global id of rank 0
  int64_t lo, hi;
  const float* sc;
};

template <class TAB>
__device__ inline Share my_share(const float* scores, const TAB& seq, int keep_tail) {
  Share s;
  int b = 0;
  while (b + 1 < seq.batch && (int)blockIdx.x >= seq.chunk_start[b + 1]) ++b;
  s.b = b;
  s.first = (uint32_t)seq.chunk_start[b];
  s.nblk = (uint32_t)(seq.chunk_start[b + 1] - seq.chunk_start[b]);
  s.blk = blockIdx.x - s.first;
  const int64_t m = seq.cu[b + 1] - seq.cu[b] - keep_tail;
  const int64_t per = (m + s.nblk - 1) / s.nblk;
  s.lo = min(m, (int64_t)s.blk * per);
  s.hi = min(m, s.lo + per);
  s.sc = scores + seq.cu[b];
  return s;
}

template <class TAB>
__global__ __launch_bounds__(kThreads) void topk_init_kernel(TAB seq, int keep_tail, TopkWs ws,
                                                             int32_t* __restrict__ idx_out) {
  short_kernel_priority();
  const int b = blockIdx.y;
  const int tid = blockIdx.x * kThreads + threadIdx.x;
  const int stride = gridDim.x * kThreads;
  for (int i = tid; i < 3 * kBins; i += stride) ws.hist[(size_t)b * 3 * kBins + i] = 0u;
  const int64_t m = seq.cu[b + 1] - seq.cu[b] - keep_tail;
  for (int i = tid; i < keep_tail; i += stride)
    idx_out[seq.out_off[b] + seq.k[b] + i] = (int32_t)(m + i);
}

// Inclusive scan over the 64 lanes: shifts inside the rows of 16, then the row totals handed on (DPP moves: six vector
// instructions; the same scan by shuffles is six dependent trips through the LDS crossbar).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += dpp_or_zero<0x111, 0xF>(v);   // row_shr 1, 2, 4, 8
  v += dpp_or_zero<0x112, 0xF>(v);
  v += dpp_or_zero<0x114, 0xF>(v);
  v += dpp_or_zero<0x118, 0xF>(v);
  v += dpp_or_zero<0x142, 0xA>(v);   // lane 15 of a row to the next row; then lane 31 to the upper half
  v += dpp_or_zero<0x143, 0xC>(v);
  return v;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(v), 63); }
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {   // same moves; lanes without a source see 0
  v = max(v, dpp_or_zero<0x111, 0xF>(v));
  v = max(v, dpp_or_zero<0x112, 0xF>(v));
  v = max(v, dpp_or_zero<0x114, 0xF>(v));
  v = max(v, dpp_or_zero<0x118, 0xF>(v));
  v = max(v, dpp_or_zero<0x142, 0xA>(v));
  v = max(v, dpp_or_zero<0x143, 0xC>(v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Inclusive scan over the first NWV lanes: one value per wave of the workgroup, read from LDS by a lane each and not all of them by
// every lane (16 waves x 16 reads are a thousand cycles of the LDS; an 8192-score selection does that four times).
template <int NWV>
__device__ __forceinline__ uint32_t waves_scan(uint32_t v) {
  static_assert(NWV == 4 || NWV == 8 || NWV == 16, "lanes of one DPP row");
  v += dpp_or_zero<0x111, 0xF>(v);
  v += dpp_or_zero<0x112, 0xF>(v);
  if (NWV > 4) v += dpp_or_zero<0x114, 0xF>(v);
  if (NWV > 8) v += dpp_or_zero<0x118, 0xF>(v);
  return v;
}
// ... of which the waves before the calling one
__device__ __forceinline__ uint32_t waves_before(uint32_t scan) {
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  return wv ? (uint32_t)__builtin_amdgcn_readlane((int)scan, wv - 1) : 0u;
}

// exclusive scan of one value per thread over the workgroup (THREADS / 64 waves); returns the total.
// One barrier; `sh` must not be written again before another one (TRAIL: here).
template <int THREADS = kThreads, bool TRAIL = true>
__device__ inline uint32_t block_excl_scan(uint32_t v, uint32_t* sh /*[>= THREADS / 64]*/, uint32_t* excl) {
  constexpr int NWV = THREADS / 64;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const uint32_t x = wave_scan(v);
  if (lane == 63) sh[wv] = x;
  __syncthreads();
  const uint32_t s = waves_scan<NWV>(sh[lane & (NWV - 1)]);
  *excl = waves_before(s) + x - v;
  if (TRAIL) __syncthreads();
  return (uint32_t)__builtin_amdgcn_readlane((int)s, NWV - 1);
}

// What select_bin reads, sixteen bytes at a time where a thread has four bins or more: a histogram in LDS, whose type carries the
// alignment (a plain array of words is promised four bytes), or a merged one in the workspace, whose carve keeps it.
template <int NB>
struct alignas(16) LdsBins {
  uint32_t n[NB];
  __device__ __forceinline__ uint32_t& operator[](uint32_t i) { return n[i]; }
};
struct MergedBins {
  const uint32_t* n;   // 16-byte aligned
};
static_assert(3 * kBins % 4 == 0 && kRowWords % 4 == 0, "every sequence's and every row's histogram keeps the workspace's alignment");

// Scan the NB bins of a histogram from the top until `krem` (1 .. their sum) keys are covered.
// Returns the bin (all threads), how many keys lie above it and how many in it.
// Two barriers; `scan` and `res` must not be written again before another one.
template <int THREADS, int NB, class Bins>
__device__ inline void select_bin(const Bins& bins, uint32_t krem, uint32_t* scan /*[>= THREADS / 64]*/,
                                  uint32_t* res /*[3]*/, uint32_t* bin_out, uint32_t* above_out, uint32_t* in_bin_out = nullptr) {
  static_assert(std::is_same_v<Bins, LdsBins<NB>> || std::is_same_v<Bins, MergedBins>, "bins that are 16-byte aligned");
  constexpr int PER = NB / THREADS;
  const uint32_t* __restrict__ gh = bins.n;
  static_assert(NB % THREADS == 0, "bins split evenly over the threads");
  const int t = threadIdx.x;
  uint32_t mine[PER];   // bins NB-1-PER*t downwards
  uint32_t sum = 0;
  if constexpr (PER % 4 == 0) {
#pragma unroll
    for (int q = 0; q < PER / 4; ++q) {
      const uint4 v = *reinterpret_cast<const uint4*>(gh + NB - PER * t - 4 * (q + 1));
      mine[4 * q] = v.w; mine[4 * q + 1] = v.z; mine[4 * q + 2] = v.y; mine[4 * q + 3] = v.x;
    }
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) mine[i] = gh[NB - 1 - (PER * t + i)];
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) sum += mine[i];
  uint32_t run;
  block_excl_scan<THREADS, false>(sum, scan, &run);
  if (run < krem && run + sum >= krem) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (run < krem && run + mine[i] >= krem) {
        res[0] = (uint32_t)(NB - 1 - (PER * t + i));
        res[1] = run;
        res[2] = mine[i];
      }
      run += mine[i];
    }
  }
  __syncthreads();
  *bin_out = res[0];
  *above_out = res[1];
  if (in_bin_out) *in_bin_out = res[2];
}

// add a workgroup's LDS histogram into the merged one
__device__ inline void merge_hist(const uint32_t* h, int nb, uint32_t* __restrict__ gh) {
  for (int i = threadIdx.x; i < nb; i += kThreads)
    if (h[i]) atomicAdd(&gh[i], h[i]);
}

// A workgroup's share normally fits eight scores per thread; those are loaded into registers before the
// histogram scan so that the two latencies overlap.  Longer shares (capped workgroup count) loop instead.
constexpr int kPerThread = kTargetPerBlock / kThreads;

// thread t takes scores lo + t, lo + t + 256, ...
__device__ inline bool preload_strided(const Share& s, float (&v)[kPerThread]) {
  const bool fast = s.hi - s.lo <= kTargetPerBlock;
  if (fast) {
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const int64_t j = s.lo + threadIdx.x + i * kThreads;
      v[i] = j < s.hi ? s.sc[j] : 0.f;
    }
  }
  return fast;
}

template <class F>
__device__ inline void for_each_strided(const Share& s, const float (&v)[kPerThread], bool fast, F f) {
  if (fast) {
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
      if (s.lo + threadIdx.x + i * kThreads < s.hi) f(score_key(v[i]));
  } else {
    for (int64_t j = s.lo + threadIdx.x; j < s.hi; j += kThreads) f(score_key(s.sc[j]));
  }
}

template <class TAB>
__global__ __launch_bounds__(kThreads) void topk_hist0_kernel(const float* __restrict__ scores, TAB seq,
                                                              int keep_tail, TopkWs ws) {
  short_kernel_priority();
  __shared__ uint32_t h[kBins];
  const Share s = my_share(scores, seq, keep_tail);
  const int t = threadIdx.x;
  float v[kPerThread];
  const bool fast = preload_strided(s, v);
  for (int i = t; i < kBins; i += kThreads) h[i] = 0u;
  __syncthreads();
  for_each_strided(s, v, fast, [&](uint32_t key) { atomicAdd(&h[key >> 21], 1u); });
  __syncthreads();
  merge_hist(h, kBins, ws.hist + (size_t)s.b * 3 * kBins);
}

template <class TAB>
__global__ __launch_bounds__(kThreads) void topk_hist1_kernel(const float* __restrict__ scores, TAB seq,
                                                              int keep_tail, TopkWs ws) {
  short_kernel_priority();
  __shared__ uint32_t h[kBins];
  __shared__ uint32_t scan[4];
  __shared__ uint32_t res[3];
  const Share s = my_share(scores, seq, keep_tail);
  const int t = threadIdx.x;
  uint32_t* gh = ws.hist + (size_t)s.b * 3 * kBins;
  float v[kPerThread];
  const bool fast = preload_strided(s, v);
  for (int i = t; i < kBins; i += kThreads) h[i] = 0u;
  uint32_t bin0, above0;
  select_bin<kThreads, kBins>(MergedBins{gh}, (uint32_t)seq.k[s.b], scan, res, &bin0, &above0);   // its barriers cover h[] = 0
  if (s.blk == 0 && t == 0) {
    ws.state[s.b * 8 + 0] = bin0;
    ws.state[s.b * 8 + 1] = (uint32_t)seq.k[s.b] - above0;
  }
  for_each_strided(s, v, fast, [&](uint32_t key) {
    if ((key >> 21) == bin0) atomicAdd(&h[(key >> 10) & (kBins - 1)], 1u);
  });
  __syncthreads();
  merge_hist(h, kBins, gh + kBins);
}

template <class TAB>
__global__ __launch_bounds__(kThreads) void topk_hist2_kernel(const float* __restrict__ scores, TAB seq,
                                                              int keep_tail, TopkWs ws) {
  short_kernel_priority();
  __shared__ uint32_t h[kLowBins];
  __shared__ uint32_t scan[4];
  __shared__ uint32_t res[3];
  __shared__ uint32_t above_cnt;
  const Share s = my_share(scores, seq, keep_tail);
  const int t = threadIdx.x;
  uint32_t* gh = ws.hist + (size_t)s.b * 3 * kBins;
  float v[kPerThread];
  const bool fast = preload_strided(s, v);
  for (int i = t; i < kLowBins; i += kThreads) h[i] = 0u;
  if (t == 0) above_cnt = 0u;
  const uint32_t bin0 = ws.state[s.b * 8 + 0], krem0 = ws.state[s.b * 8 + 1];
  uint32_t bin1, above1;
  select_bin<kThreads, kBins>(MergedBins{gh + kBins}, krem0, scan, res, &bin1, &above1);   // its barriers cover h[], above_cnt = 0
  const uint32_t prefix = (bin0 << 11) | bin1;     // the top 22 bits of the k-th largest key
  if (s.blk == 0 && t == 0) {
    ws.state[s.b * 8 + 2] = prefix;
    ws.state[s.b * 8 + 3] = krem0 - above1;
  }
  uint32_t above = 0;
  for_each_strided(s, v, fast, [&](uint32_t key) {
    const uint32_t hi = key >> 10;
    above += hi > prefix;
    if (hi == prefix) atomicAdd(&h[key & (kLowBins - 1)], 1u);
  });
  if (above) atomicAdd(&above_cnt, above);
  __syncthreads();
  merge_hist(h, kLowBins, gh + 2 * kBins);
  // suffix sums of h: thread t owns the four bins 1023-4t .. 1020-4t (descending), scanned from the top
  uint32_t own[4];
  uint32_t sum = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) { own[i] = h[kLowBins - 1 - (4 * t + i)]; sum += own[i]; }
  uint32_t run;
  const uint32_t ncand = block_excl_scan(sum, scan, &run);
  if (ncand) {
    uint32_t* suf = ws.suf + (size_t)blockIdx.x * kLowBins;
#pragma unroll
    for (int i = 0; i < 4; ++i) { run += own[i]; suf[kLowBins - 1 - (4 * t + i)] = run; }
  }
  if (t == 0) {
    ws.meta[2 * (size_t)blockIdx.x] = above_cnt;
    ws.meta[2 * (size_t)blockIdx.x + 1] = ncand;
  }
}

template <class TAB>
__global__ __launch_bounds__(kThreads) void topk_write_kernel(const float* __restrict__ scores, TAB seq,
                                                              int keep_tail, TopkWs ws,
                                                              int32_t* __restrict__ idx_out) {
  short_kernel_priority();
  __shared__ uint32_t scan[4];
  __shared__ uint32_t res[3];
  __shared__ uint32_t cnt[2];
  const Share s = my_share(scores, seq, keep_tail);
  const int t = threadIdx.x;
  const uint32_t* gh = ws.hist + (size_t)s.b * 3 * kBins;
  if (t == 0) { cnt[0] = 0u; cnt[1] = 0u; }
  // this workgroup's share; thread t owns a contiguous slice of it (loaded before the histogram scan)
  const int64_t sub = (s.hi - s.lo + kThreads - 1) / kThreads;
  const int64_t tlo = min(s.hi, s.lo + t * sub), thi = min(s.hi, tlo + sub);
  const bool fast = sub <= kPerThread;
  float v[kPerThread];
  if (fast) {
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) v[i] = tlo + i < thi ? s.sc[tlo + i] : 0.f;
  }
  // counts of the first workgroup this thread will add up, also requested before the scan
  const bool has0 = (uint32_t)t < s.blk;
  const uint2 m0 = has0 ? *reinterpret_cast<const uint2*>(ws.meta + 2 * ((size_t)s.first + t)) : make_uint2(0u, 0u);
  const uint32_t prefix = ws.state[s.b * 8 + 2], krem1 = ws.state[s.b * 8 + 3];
  uint32_t t10, above2;
  select_bin<kThreads, kLowBins>(MergedBins{gh + 2 * kBins}, krem1, scan, res, &t10, &above2);   // its barriers cover cnt[] = 0
  const uint32_t T = (prefix << 10) | t10;   // the k-th largest key
  const uint32_t need = krem1 - above2;      // how many keys equal to T are taken (lowest indices first)

  // selected keys in the workgroups before this one
  uint32_t g0 = 0, e0 = 0;
  auto add_block = [&](size_t w, uint32_t above, uint32_t ncand) {
    g0 += above;
    if (ncand) {
      const uint32_t* suf = ws.suf + w * kLowBins;
      const uint32_t ge = suf[t10];
      const uint32_t gt = t10 + 1 < (uint32_t)kLowBins ? suf[t10 + 1] : 0u;
      g0 += gt;
      e0 += ge - gt;
    }
  };
  if (has0) add_block((size_t)s.first + t, m0.x, m0.y);
  for (uint32_t i = t + kThreads; i < s.blk; i += kThreads) {
    const size_t w = (size_t)s.first + i;
    add_block(w, ws.meta[2 * w], ws.meta[2 * w + 1]);
  }
  if (g0) atomicAdd(&cnt[0], g0);
  if (e0) atomicAdd(&cnt[1], e0);

  uint32_t gt = 0, eq = 0;
  if (fast) {
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const uint32_t key = score_key(v[i]);
      gt += tlo + i < thi && key > T;
      eq += tlo + i < thi && key == T;
    }
  } else {
    for (int64_t j = tlo; j < thi; ++j) {
      const uint32_t key = score_key(s.sc[j]);
      gt += key > T;
      eq += key == T;
    }
  }
  uint32_t gt_before, eq_before;
  block_excl_scan(gt, scan, &gt_before);
  block_excl_scan(eq, scan, &eq_before);   // the barriers inside also order the cnt[] atomics above
  gt_before += cnt[0];
  eq_before += cnt[1];
  int32_t* out = idx_out + seq.out_off[s.b];
  auto place = [&](uint32_t key, int64_t j) {
    if (key > T) {
      out[gt_before + min(eq_before, need)] = (int32_t)j;
      ++gt_before;
    } else if (key == T) {
      if (eq_before < need) out[gt_before + eq_before] = (int32_t)j;
      ++eq_before;
    }
  };
  if (fast) {
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
      if (tlo + i < thi) place(score_key(v[i]), tlo + i);
  } else {
    for (int64_t j = tlo; j < thi; ++j) place(score_key(s.sc[j]), j);
  }
}


// ---- short and mid forms ----------------------------------------------------------------------------------------

constexpr int kWide = 1024;        // threads of a short-form workgroup
static_assert(kReduceShortSeq <= 2 * kWide, "a workgroup that forms the scores holds two per thread");
constexpr int kMidShare = 1024;    // scores of a mid-form workgroup

constexpr int kListed = 64;        // keys that one wave ranks directly

// LDS of resolve_key
struct ResolveLds {
  LdsBins<kBins> hist;
  uint32_t list[kListed];
  uint32_t scan[16], res[3], n;
};

// One more in h[bin] for every calling lane; lanes that share one of two values add up first (an LDS atomic of 64 lanes on one
// word takes 64 turns: 131072 equal scores, 100 us a sweep).
__device__ __forceinline__ void count_ties(uint32_t* h, uint32_t bin) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool mine = bin == (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
    const unsigned long long same = __ballot(mine);
    if (mine) {
      if ((int)(threadIdx.x & 63) == __ffsll((long long)same) - 1) atomicAdd(&h[bin], (uint32_t)__popcll(same));
      return;
    }
  }
  atomicAdd(&h[bin], 1u);
}

// The krem-th largest of the keys that `each` visits, all of them in [lo, lo + 2^width): the range in 2048 bins,
// histogrammed in LDS; the k-th largest's bin again in 2048 bins, and so on, until the bin holds at most 64 keys (mostly
// after one round), which every wave ranks for itself, a key per lane.  T: that key; need: how many keys equal to it are
// among the krem.  l.hist must be zero and l.n zero, a barrier in between.  TIES: many of the keys are expected to be equal.
template <int THREADS, bool TIES = false, class Each>
__device__ inline void resolve_key(Each each, uint32_t lo, int width, uint32_t krem, ResolveLds& l, uint32_t* T, uint32_t* need) {
  uint32_t prefix = 0u;
  int rem = width;
  while (rem > 0) {
    const int bits = min(11, rem), sh = rem - bits;
    each([&](uint32_t key) {
      const uint32_t off = key - lo;
      if (rem == width || (off >> rem) == prefix) {
        const uint32_t at = (off >> sh) & ((1u << bits) - 1u);
        if constexpr (TIES) count_ties(l.hist.n, at); else atomicAdd(&l.hist[at], 1u);
      }
    });
    __syncthreads();
    uint32_t bin, above, in_bin;
    select_bin<THREADS, kBins>(l.hist, krem, l.scan, l.res, &bin, &above, &in_bin);
    prefix = (prefix << bits) | bin;
    krem -= above;
    rem = sh;
    if (rem == 0) break;
    if (in_bin <= (uint32_t)kListed) {
      each([&](uint32_t key) {
        if (((key - lo) >> rem) == prefix) l.list[atomicAdd(&l.n, 1u)] = key;
      });
      __syncthreads();
      const uint32_t lane = threadIdx.x & 63;
      const uint32_t mine = lane < in_bin ? l.list[lane] : 0u;
      uint32_t gt = 0u, ge = 0u;
      for (uint32_t i = 0; i < in_bin; ++i) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)mine, (int)i);
        gt += o > mine;
        ge += o >= mine;
      }
      const unsigned long long hit = __ballot(lane < in_bin && gt < krem && ge >= krem);
      const int at = __ffsll((long long)hit) - 1;
      *T = (uint32_t)__builtin_amdgcn_readlane((int)mine, at);
      *need = krem - (uint32_t)__builtin_amdgcn_readlane((int)gt, at);
      return;
    }
    for (int i = threadIdx.x; i < kBins; i += THREADS) l.hist[i] = 0u;
    __syncthreads();
  }
  *T = lo + prefix;
  *need = krem;
}

// Place the selected ones of a workgroup's PER x THREADS keys in ascending order: those above T and, of those equal to T, the first
// `need` of the sequence; g0 / e0: keys above / equal to T before the workgroup.  A wave's keys are consecutive (key i of a lane stands at
// j0 + 64 i + lane), so that what counts between its rounds is scalar and only the waves' totals go through LDS; with rounds over the
// whole workgroup 128 counts were scanned by every wave (8192 scores 5.5 k cycles of 18 k).  put(place, index): an ascending place each.
template <int THREADS, int PER, class Put>
__device__ inline void place_ordered(const uint32_t (&key)[PER], int j0, int m, uint32_t T, uint32_t need, uint32_t g0,
                                     uint32_t e0, uint32_t* tot /*[THREADS / 64]*/, Put put) {
  constexpr int NWV = THREADS / 64;
  static_assert(PER * THREADS < 65536, "both counts of a word stay below 2^16");
  const int lane = threadIdx.x & 63;
  auto before = [](unsigned long long mask) __attribute__((always_inline)) {
    return (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
  };
  unsigned long long mg[PER], me[PER];
  uint32_t cg = 0u, ce = 0u;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const bool in = j0 + 64 * i + lane < m;
    mg[i] = __ballot(in && key[i] > T);
    me[i] = __ballot(in && key[i] == T);
    cg += (uint32_t)__popcll(mg[i]);
    ce += (uint32_t)__popcll(me[i]);
  }
  if (lane == 0) tot[threadIdx.x >> 6] = cg | (ce << 16);
  __syncthreads();
  const uint32_t p = waves_before(waves_scan<NWV>(tot[lane & (NWV - 1)]));
  uint32_t g = g0 + (p & 0xFFFFu), e = e0 + (p >> 16);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (me[i] == 0ull || e >= need) {   // (uniform) no key of the round is equal to T, or none of those is taken
      if ((mg[i] >> lane) & 1ull) put(g + before(mg[i]) + min(e, need), j0 + 64 * i + lane);
    } else {
      const uint32_t gb = g + before(mg[i]), eb = e + before(me[i]);
      if ((mg[i] >> lane) & 1ull) put(gb + min(eb, need), j0 + 64 * i + lane);
      else if (((me[i] >> lane) & 1ull) && eb < need) put(gb + eb, j0 + 64 * i + lane);
    }
    g += (uint32_t)__popcll(mg[i]);
    e += (uint32_t)__popcll(me[i]);
  }
}

// short form: a workgroup has all of a sequence of at most PER x 1024 scores; also writes the kept window.
// SUM (a layer step): it first does what the reduce kernel does -- the column-sum planes of its sequence's tokens (at most
// PER x 1024 with the window) added up in ascending order, the centrality update, the entropies' means -- and selects on the
// scores it holds: one launch fewer (a layer step of 1K tokens is a handful of 3 us kernels: see short_plan in api.cpp).
// COPY (a layer step): `parts` workgroups per sequence, which all select for themselves and then copy a share each of the kept
// rows, instead of a gather launch that reads the indices again (one
// launch fewer for the host as well).  A layer step, 32 heads on 8, head_dim 128, window 8, a fifth kept, us a call eager (in a graph) with
// the gather launch -> here: 512 tokens 17.0 -> 14.1 (11.9 -> 11.2), 2048 19.7 -> 18.6 (18.7 -> 18.0), 8192 29.0 -> 28.5 (26.8 -> 25.9);
// thirteen layers on four streams, a layer in a graph: 1000 tokens 21.7 -> 18.2, 8192 29.0 -> 25.4.
template <int PER, class TAB, bool SUM, bool COPY>
__global__ __launch_bounds__(kWide) void topk_short_kernel(const float* __restrict__ scores, TAB seq, int keep_tail,
                                                           int32_t* __restrict__ idx_out, ReduceWork red, CopyWork copy, int parts) {
  short_kernel_priority();
  constexpr int NWV = kWide / 64;
  __shared__ ResolveLds l;
  __shared__ uint32_t ends[2][NWV], tot[NWV];
  __shared__ int32_t mine[COPY ? kCopyRows : 1];   // the source tokens of the rows that this workgroup copies
  if constexpr (SUM) {   // the second half of the launch: the entropies' means beside the selections (ahead of them in the same
                         // workgroups: four short prompts 20.8 us a layer step, beside 20.1; 1K tokens in fp32 19.9 and 19.4)
    __shared__ float hsum[256];
    const int selecting = COPY ? seq.batch * parts : seq.batch;
    if ((int)blockIdx.x >= selecting) {
      finish_entropy(red.row_ent, red.ent_head, red.entropy, (int)blockIdx.x - selecting, red.Hq, red.w, hsum);
      return;
    }
  }
  const int t = threadIdx.x, b = COPY ? (int)blockIdx.x % seq.batch : (int)blockIdx.x, part = COPY ? (int)blockIdx.x / seq.batch : 0;
  const bool writes = part == 0;   // the others' results are the same
  const int j0 = (t >> 6) * (64 * PER), lane = t & 63;   // key i of a lane: place_ordered
  const int m = (int)(seq.cu[b + 1] - seq.cu[b]) - keep_tail;
  const uint32_t k = (uint32_t)seq.k[b];
  const float* sc = scores + seq.cu[b];
  int32_t* out = idx_out + seq.out_off[b];
  float v[PER];
  if constexpr (SUM) {
    constexpr int U = 16 / PER;   // planes in flight
    const int n = m + keep_tail;
    int64_t at[PER];
    float c[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      at[i] = seq.cu[b] + max(0, min(j0 + 64 * i + lane, n - 1));   // (an empty sequence reads nothing below)
      v[i] = 0.f;
      c[i] = writes && red.cen && n > 0 ? red.cen[at[i]] : 0.f;
    }
    for (int p = 0; n > 0 && p < red.planes; p += U) {
      float x[U][PER];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < PER; ++i) x[u][i] = p + u < red.planes ? red.colsum[(int64_t)(p + u) * red.total + at[i]] : 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < PER; ++i) v[i] += x[u][i];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (writes && j0 + 64 * i + lane < n) {
        red.indeg[at[i]] = v[i];
        if (red.cen) red.cen[at[i]] = fmaf(red.lambda, c[i], red.inv_w * v[i]);
      }
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) v[i] = k > 0u && j0 + 64 * i + lane < m ? sc[j0 + 64 * i + lane] : 0.f;
  }
  for (int i = t; writes && i < keep_tail; i += kWide) out[k + i] = m + i;
  // rows [r0, r1) of the sequence's k + keep_tail are this workgroup's to copy
  const uint32_t rows = k + (uint32_t)keep_tail, share = COPY ? (rows + (uint32_t)parts - 1u) / (uint32_t)parts : 0u;
  const uint32_t r0 = min(rows, (uint32_t)part * share), r1 = min(rows, r0 + share);
  auto copy_share = [&]() __attribute__((always_inline)) {
    copy_rows<kWide, 4>(copy, r1 - r0, seq.out_off[b] + r0, seq.cu[b], [&](uint32_t r) {
      return r0 + r < k ? mine[r] : m + (int)(r0 + r - k);
    });
  };
  if (k == 0u) {
    if constexpr (COPY) copy_share();
    return;
  }
  if (COPY && !writes && r0 >= k) {   // (nothing but the kept window)
    copy_share();
    return;
  }
  for (int i = t; i < kBins; i += kWide) l.hist[i] = 0u;
  if (t == 0) l.n = 0u;
  uint32_t key[PER], inv = 0u, mx = 0u;   // largest ~key and largest key
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    key[i] = score_key(v[i]);
    if (j0 + 64 * i + lane < m) { inv = max(inv, ~key[i]); mx = max(mx, key[i]); }
  }
  inv = wave_max(inv);
  mx = wave_max(mx);
  if (lane == 0) { ends[0][t >> 6] = inv; ends[1][t >> 6] = mx; }
  __syncthreads();
  inv = wave_max(ends[0][lane & (NWV - 1)]);
  mx = wave_max(ends[1][lane & (NWV - 1)]);
  const uint32_t mn = ~inv;
  uint32_t T, need;
  resolve_key<kWide>([&](auto f) {
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (j0 + 64 * i + lane < m) f(key[i]);
  }, mn, 32 - __clz((int)(mx - mn)), k, l, &T, &need);
  place_ordered<kWide, PER>(key, j0, m, T, need, 0u, 0u, tot, [&](uint32_t at, int j) {
    if (writes) out[at] = j;
    if constexpr (COPY)
      if (at - r0 < r1 - r0) mine[at - r0] = j;
  });
  if constexpr (COPY) {
    __syncthreads();
    copy_share();
  }
}

// mid form, alone: zero the histograms and the candidate counter, write the kept window, and centre the bins on the k-th
// largest of a sample (1024 scores; it only places the bins, the result does not depend on it)
template <class TAB>
__global__ __launch_bounds__(kWide) void topk_mid_init_kernel(const float* __restrict__ scores, TAB seq, int keep_tail,
                                                              TopkWs ws, int32_t* __restrict__ idx_out) {
  short_kernel_priority();
  constexpr int NWV = kWide / 64;
  __shared__ LdsBins<kBins> h;
  __shared__ uint32_t scan[NWV], res[3], ends[2][NWV];
  const int b = blockIdx.x, t = threadIdx.x;
  const int64_t m = seq.cu[b + 1] - seq.cu[b] - keep_tail;
  const uint32_t k = (uint32_t)seq.k[b];
  const float v = m > 0 ? scores[seq.cu[b] + (m * t) / kWide] : 0.f;
  for (int i = t; i < kFineBins + kSubBins + 1; i += kWide) ws.hist[(size_t)b * 3 * kBins + i] = 0u;
  for (int i = t; i < keep_tail; i += kWide) idx_out[seq.out_off[b] + k + i] = (int32_t)(m + i);
  if (k == 0u) return;
  for (int i = t; i < kBins; i += kWide) h[i] = 0u;
  __syncthreads();
  const uint32_t key = score_key(v);
  atomicAdd(&h[key >> 21], 1u);
  __syncthreads();
  uint32_t digit, above, in_digit;
  const uint32_t rank = (uint32_t)max((int64_t)1, ((int64_t)k * kWide) / m);
  select_bin<kWide, kBins>(h, rank, scan, res, &digit, &above, &in_digit);
  // where the rank lies among the sample's keys with that digit, as if they filled it evenly; where they crowd together,
  // between the smallest and the largest of them
  uint32_t least = digit << 21, span = (1u << 21) - 1u;
  if (in_digit > (uint32_t)kWide / 6) {   // (scores spread over two octaves: 140; a quarter microsecond saved)
    const bool in = (key >> 21) == digit;
    const uint32_t wmx = wave_max(in ? key : 0u), winv = wave_max(in ? ~key : 0u);
    if ((t & 63) == 0) { ends[0][t >> 6] = wmx; ends[1][t >> 6] = winv; }
    __syncthreads();
    uint32_t mx = 0u, inv = 0u;
    for (int i = 0; i < NWV; ++i) { mx = max(mx, ends[0][i]); inv = max(inv, ends[1][i]); }
    least = ~inv;
    span = mx - least;
  }
  if (t == 0) ws.state[b * 8 + 4] = least + span - span / in_digit * (rank - above);   // (rank - above: 1 .. in_digit)
}

// the calling workgroup's sequence b, its number inside it and its first score
template <class TAB>
__device__ inline void mid_share(const TAB& seq, int* b_out, uint32_t* blk, int* j0) {
  int b = 0;
  while (b + 1 < seq.batch && (int)blockIdx.x >= seq.chunk_start[b + 1]) ++b;
  *b_out = b;
  *blk = blockIdx.x - (uint32_t)seq.chunk_start[b];
  *j0 = (int)*blk * kMidShare;
}

// Workgroups of 512 threads on two shares: what this costs is clearing and merging a histogram per workgroup, and where there are many,
// finding its sequence (one after the other, 64 x 17000 scores took 47.3 us in a graph, a sequence per lane 32.6).  Selections alone, us
// in a graph, 256 threads on one share / 512 on one / 512 on two / 1024 on two: 131072 scores 16.5 / 15.8 / 14.8 / 14.9, 8 x 32768
// 16.3 / 15.8 / 15.3 / 15.5, 64 x 17000 34.5 / 34.7 / 32.6 / 33.8, 8 x 262144 38.2 / 39.2 / 30.7 / 32.2.
constexpr int kHistThreads = 512, kHistShares = 2;
template <class TAB>
__global__ __launch_bounds__(kHistThreads) void topk_mid_hist_kernel(const float* __restrict__ scores, TAB seq, int keep_tail,
                                                                     TopkWs ws) {
  short_kernel_priority();
  constexpr int NT = kHistThreads, PER = kHistShares * kMidShare / NT;
  __shared__ alignas(8) uint32_t h[kFineBins];
  // the sequence and the number inside it, a sequence per lane
  static_assert(kMaxBatch <= 64, "a wave holds all sequences");
  const int lane = threadIdx.x & 63;
  const int wgs = lane < seq.batch ? (seq.chunk_start[lane + 1] - seq.chunk_start[lane] + kHistShares - 1) / kHistShares : 0;
  const uint32_t ends = wave_scan((uint32_t)wgs);
  const int b = __popcll(__ballot(lane < seq.batch && ends <= blockIdx.x));
  const int at = (int)blockIdx.x - (b ? __builtin_amdgcn_readlane((int)ends, b - 1) : 0);
  const int t = threadIdx.x, j0 = at * (kHistShares * kMidShare);
  const int m = (int)(seq.cu[b + 1] - seq.cu[b]) - keep_tail;
  const float* sc = scores + seq.cu[b];
  float v[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) v[i] = j0 + i * NT + t < m ? sc[j0 + i * NT + t] : 0.f;
  const BinTiers tiers = bins_around(ws.state[b * 8 + 4]);
  for (int i = t; i < kFineBins; i += NT) h[i] = 0u;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (j0 + i * NT + t < m) atomicAdd(&h[fine_bin(score_key(v[i]), tiers)], 1u);
  __syncthreads();
  merge_bins(h, kFineBins, ws.hist + (size_t)b * 3 * kBins, NT);
}

// Most candidates of a sequence of `nblk` workgroups that are listed; the list lies in the words of their suffix sums.  In an
// innermost bin the sub-bins are the better of the two as soon as a list takes more than one entry a thread (131072 scores within
// 0.3 / 0.1 / 0.05 %, 870 / 2400 / 4400 candidates: 19.6 / 22.0 / 27.0 us as lists, 18.7 / 18.9 / 18.6 as sub-bins); in a wider
// one the sub-bin's keys have to be picked out of the scores (a layer step of 131072 tokens, window 8, 700 candidates in a
// bin of 1/256 octave: 43.0 us with the list, 48.3 with sub-bins), which is worth it where the list's words or its time run out.
__device__ __forceinline__ uint32_t list_cap(uint32_t nblk, uint32_t width) {
  return width <= (uint32_t)kSubBits ? 256u
                                     : min((uint32_t)kCandCap, nblk * (uint32_t)(kSubBins * sizeof(uint16_t) / sizeof(uint2)));
}
__device__ __forceinline__ uint16_t* sub_sums(const TopkWs& ws, uint32_t workgroup) {
  return reinterpret_cast<uint16_t*>(ws.suf) + (size_t)workgroup * kSubBins;
}

// NT threads a workgroup of compact and place: a thread's share of the histogram, the candidates and the scores is a chain of its own, so
// 512 threads end sooner than 256 (layer steps of 32K tokens 48.3 -> 47.2 us, a truncation at 128K 96.2 -> 95.0; 1024 are no better).  Not
// where there are more than 256 workgroups (554K tokens in eight sequences 478 -> 483 us), nor in the second half of a layer step by itself,
// which runs beside other layers' scoring and gets on the chip the sooner the smaller its workgroups are (32 layers of
// 128K tokens on four streams 5.20 ms with 256, 5.22 with 512, 5.29 with 1024).  What else runs beside other work -- a selection on a side
// stream, whole steps on streams of their own -- does not say so: with 512 threads place has 84 registers (136 with the scores of four shares in flight a wave, as with
// 256, not of one), so that its two waves per SIMD fit where ONE workgroup of scoring has left, as the one of 256 threads does
// (four streams of 64K-token steps, window 64, us a step in a graph: 256 threads 88.5, 512 of 136 registers 90.0, of 84 88.1; alone 72.9, 72.1,
// 71.9 at a window of 8).
template <int NT, class TAB>
__global__ __launch_bounds__(NT) void topk_compact_kernel(const float* __restrict__ scores, TAB seq, int keep_tail,
                                                                TopkWs ws) {
  short_kernel_priority();
  constexpr int NWV = NT / 64, kMidPer = kMidShare / NT, N = kMidPer * NWV;
  __shared__ uint32_t scan[NWV], res[3], wtot[N], gbase, ends[2][NWV];
  __shared__ alignas(8) uint32_t h[kSubBins];
  int b;
  uint32_t blk;
  int j0;
  mid_share(seq, &b, &blk, &j0);
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int n = (int)(seq.cu[b + 1] - seq.cu[b]), m = n - keep_tail;
  const uint32_t first = (uint32_t)seq.chunk_start[b], nblk = (uint32_t)seq.chunk_start[b + 1] - first;
  const float* sc = scores + seq.cu[b];
  float v[kMidPer];
#pragma unroll
  for (int i = 0; i < kMidPer; ++i) v[i] = j0 + i * NT + t < m ? sc[j0 + i * NT + t] : 0.f;
  uint32_t* gh = ws.hist + (size_t)b * 3 * kBins;
  const BinTiers tiers = ws.mass > 0.f ? bins_around_mean(ws.mass, n) : bins_around(ws.state[b * 8 + 4]);
  const uint32_t k = (uint32_t)seq.k[b];
  uint32_t bin, above, in_bin, lo, width;
  select_bin<NT, kFineBins>(MergedBins{gh}, k, scan, res, &bin, &above, &in_bin);
  fine_range(bin, tiers, &lo, &width);
  const uint32_t hi = lo + ((1u << width) - 1u);
  const bool listed = in_bin <= list_cap(nblk, width);
  if (blk == 0 && t == 0) {
    uint32_t* st = ws.state + (size_t)b * 8;
    st[0] = lo;
    st[1] = width;
    st[2] = k - above;
    st[3] = in_bin;
  }
  uint32_t key[kMidPer];
  unsigned long long mc[kMidPer];
#pragma unroll
  for (int i = 0; i < kMidPer; ++i) {
    const bool in = j0 + i * NT + t < m;
    key[i] = score_key(v[i]);
    mc[i] = __ballot(in && key[i] >= lo && key[i] <= hi);
    const unsigned long long ma = __ballot(in && key[i] > hi);
    if (lane == 0) wtot[i * NWV + wv] = (uint32_t)__popcll(mc[i]) | ((uint32_t)__popcll(ma) << 16);
  }
  if (!listed)
    for (int i = t; i < kSubBins; i += NT) h[i] = 0u;
  __syncthreads();
  const uint32_t own = lane < N ? wtot[lane] : 0u;   // every wave scans the counts for itself
  const uint32_t x = wave_scan(own);
  if (t == N - 1) {
    ws.meta[blockIdx.x] = x >> 16;
    const uint32_t c = x & 0xFFFFu;
    gbase = c && listed ? atomicAdd(&gh[kFineBins + kSubBins], c) : 0u;
  }
  if (!listed) {
    // a crowded bin: counts of its sub-bins, and for the placement the workgroup's own from the top down
    const uint32_t sh = width - kSubBits;
    uint32_t inv = 0u, mx = 0u;   // largest ~key and largest key
#pragma unroll
    for (int i = 0; i < kMidPer; ++i)
      if ((mc[i] >> lane) & 1ull) {
        atomicAdd(&h[(key[i] - lo) >> sh], 1u);
        inv = max(inv, ~key[i]);
        mx = max(mx, key[i]);
      }
    inv = wave_max(inv);
    mx = wave_max(mx);
    if (lane == 0) { ends[0][wv] = inv; ends[1][wv] = mx; }
    __syncthreads();
    if (t == 0) {
      for (int i = 0; i < NWV; ++i) { inv = max(inv, ends[0][i]); mx = max(mx, ends[1][i]); }
      *reinterpret_cast<uint2*>(gh + kKeyEnds + 2 * blk) = make_uint2(~inv, mx);
    }
    merge_bins(h, kSubBins, gh + kFineBins, NT);
    constexpr int SB = kSubBins / NT;
    uint32_t cs[SB], sum = 0u;
#pragma unroll
    for (int i = 0; i < SB; ++i) { cs[i] = h[kSubBins - 1 - (SB * t + i)]; sum += cs[i]; }
    uint32_t run;
    block_excl_scan<NT, false>(sum, scan, &run);
    uint16_t* out = sub_sums(ws, blockIdx.x) + kSubBins - 1 - SB * t;
#pragma unroll
    for (int i = 0; i < SB; ++i) { run += cs[i]; out[-i] = (uint16_t)run; }   // (at most the workgroup's 1024 scores)
    return;
  }
  __syncthreads();
  uint2* cand = reinterpret_cast<uint2*>(sub_sums(ws, first)) + gbase;
#pragma unroll
  for (int i = 0; i < kMidPer; ++i) {
    const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(x - own), i * NWV + wv) & 0xFFFFu;
    if ((mc[i] >> lane) & 1ull) cand[before + (uint32_t)__popcll(mc[i] & ((1ull << lane) - 1ull))] = make_uint2(key[i], blk);
  }
}

template <int NT, class TAB>
__global__ __launch_bounds__(NT) void topk_place_kernel(const float* __restrict__ scores, TAB seq, int keep_tail, TopkWs ws,
                                                              int32_t* __restrict__ idx_out) {
  short_kernel_priority();
  // candidates a thread keeps in registers; the first is requested before their number is known
  constexpr int kMidPer = kMidShare / NT, CPT = 1024 / NT;
  constexpr int kPicked = CPT * NT;   // most keys of a sub-bin that are copied together
  __shared__ ResolveLds l;
  __shared__ uint32_t tot[NT / 64], cnt[2], npick, nhold, ends[2][NT / 64];
  __shared__ uint8_t holders[256];
  __shared__ uint2 picked[kPicked];
  int b;
  uint32_t blk;
  int j0;
  mid_share(seq, &b, &blk, &j0);
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  j0 += wv * (64 * kMidPer);   // the wave's first score: place_ordered
  const int m = (int)(seq.cu[b + 1] - seq.cu[b]) - keep_tail;
  const uint32_t first = (uint32_t)seq.chunk_start[b], nblk = (uint32_t)seq.chunk_start[b + 1] - first;   // (at most 256)
  const float* sc = scores + seq.cu[b];
  const uint32_t* st = ws.state + (size_t)b * 8;
  const uint32_t lo = st[0], krem = st[2], c = st[3];
  const int width = (int)st[1];
  const uint2* cand = reinterpret_cast<const uint2*>(sub_sums(ws, first));
  uint2 x[CPT];
  x[0] = t < 256 ? cand[t] : make_uint2(0u, 0u);   // (every sequence here has at least one workgroup, whose words hold 256)
  float v[kMidPer];
#pragma unroll
  for (int i = 0; i < kMidPer; ++i) v[i] = j0 + 64 * i + lane < m ? sc[j0 + 64 * i + lane] : 0.f;
  uint32_t g0 = (uint32_t)t < blk ? ws.meta[first + t] : 0u;
  for (int i = t; i < kBins; i += NT) l.hist[i] = 0u;
  if (t == 0) { cnt[0] = 0u; cnt[1] = 0u; l.n = 0u; npick = 0u; nhold = 0u; }
  __syncthreads();
  uint32_t T, need, e0 = 0u;
  // the krem_-th largest of the `count` entries (key, workgroup) that `more` reads beyond those in x; all in [from, from + 2^bits)
  auto resolve_entries = [&](const uint2* more, uint32_t count, uint32_t from, int bits, uint32_t krem_) {
    auto each = [&](auto f) {
#pragma unroll
      for (int r = 0; r < CPT; ++r)
        if ((uint32_t)(r * NT + t) < count) f(x[r]);
      for (uint32_t i = CPT * NT + t; i < count; i += NT) f(more[i]);
    };
    resolve_key<NT>([&](auto f) { each([&](uint2 e) { f(e.x); }); }, from, bits, krem_, l, &T, &need);
    each([&](uint2 e) {
      g0 += e.y < blk && e.x > T;
      e0 += e.y < blk && e.x == T;
    });
  };
  if (c <= list_cap(nblk, (uint32_t)width)) {
#pragma unroll
    for (int r = 0; r < CPT; ++r)
      if (r > 0 || t >= 256) x[r] = (uint32_t)(r * NT + t) < c ? cand[r * NT + t] : make_uint2(0u, 0u);
    resolve_entries(cand, c, lo, width, krem);
  } else {
    const uint32_t* sub = ws.hist + (size_t)b * 3 * kBins + kFineBins;
    const int sh = width - kSubBits;
    uint32_t s, above, in_sub;
    select_bin<NT, kSubBins>(MergedBins{sub}, krem, l.scan, l.res, &s, &above, &in_sub);
    const uint32_t ksub = krem - above, from = lo + (s << sh);
    uint32_t mine = 0u;   // keys of the sub-bin in workgroup t's scores
    if ((uint32_t)t < nblk) {
      const uint16_t* sums = sub_sums(ws, first + t);
      const uint32_t ge = sums[s], gt = s + 1 < (uint32_t)kSubBins ? sums[s + 1] : 0u;
      mine = ge - gt;
      if ((uint32_t)t < blk) g0 += gt;
    }
    if (sh == 0) {   // an innermost bin: the sub-bin is one key
      T = from;
      need = ksub;
      if ((uint32_t)t < blk) e0 = mine;
    } else {
      // the keys of the sub-bin are in the scores themselves, in the workgroups that have counted some
      if (mine) holders[atomicAdd(&nhold, 1u)] = (uint8_t)t;   // (in any order: nothing below depends on it)
      uint32_t inv = 0u, mx = 0u;
      if (mine) {
        const uint2 ends_of = *reinterpret_cast<const uint2*>(sub + (kKeyEnds - kFineBins) + 2 * t);
        inv = ~ends_of.x;
        mx = ends_of.y;
      }
      inv = wave_max(inv);
      mx = wave_max(mx);
      if (lane == 0) { ends[0][wv] = inv; ends[1][wv] = mx; }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < NT / 64; ++i) { inv = max(inv, ends[0][i]); mx = max(mx, ends[1][i]); }
      const uint32_t nh = nhold;
      // f(key, workgroup), a wave to the scores of kAtOnce workgroups
      auto visit = [&](auto f) {
        constexpr uint32_t kAtOnce = NT == 256 ? 4 : 1;
        constexpr int PER = kMidShare / 64;
        for (uint32_t i0 = wv * kAtOnce; i0 < nh; i0 += kAtOnce * (NT / 64)) {
          float y[kAtOnce][PER];
          int u[kAtOnce];
#pragma unroll
          for (uint32_t a = 0; a < kAtOnce; ++a) {
            u[a] = __builtin_amdgcn_readfirstlane((int)holders[min(i0 + a, nh - 1)]);
            const float* p = sc + u[a] * kMidShare;
            const int left = m - u[a] * kMidShare;
            if (left >= kMidShare) {
#pragma unroll
              for (int i = 0; i < PER; ++i) y[a][i] = p[lane + 64 * i];
            } else {
#pragma unroll
              for (int i = 0; i < PER; ++i) y[a][i] = p[min(lane + 64 * i, left - 1)];
            }
          }
#pragma unroll
          for (uint32_t a = 0; a < kAtOnce; ++a) {
            const int left = i0 + a < nh ? m - u[a] * kMidShare : 0;
#pragma unroll
            for (int i = 0; i < PER; ++i) {
              const uint32_t q = score_key(y[a][i]);
              if (q - from < (1u << sh) && lane + 64 * i < left) f(q, (uint32_t)u[a]);
            }
          }
        }
      };
      if (~inv == mx) {   // ties
        T = mx;
        need = ksub;
        if ((uint32_t)t < blk) e0 = mine;
      } else if (in_sub <= (uint32_t)kPicked) {
        visit([&](uint32_t q, uint32_t u) { picked[atomicAdd(&npick, 1u)] = make_uint2(q, u); });
        __syncthreads();
#pragma unroll
        for (int r = 0; r < CPT; ++r) x[r] = picked[r * NT + t];
        resolve_entries(picked, in_sub, from, sh, ksub);
      } else {
        resolve_key<NT, true>([&](auto f) { visit([&](uint32_t q, uint32_t) { f(q); }); }, from, sh, ksub, l, &T, &need);
        visit([&](uint32_t q, uint32_t u) {
          g0 += u < blk && q > T;
          e0 += u < blk && q == T;
        });
      }
    }
  }
  g0 = wave_sum(g0);
  e0 = wave_sum(e0);
  if (lane == 0) { atomicAdd(&cnt[0], g0); atomicAdd(&cnt[1], e0); }
  uint32_t key[kMidPer];
#pragma unroll
  for (int i = 0; i < kMidPer; ++i) key[i] = score_key(v[i]);
  __syncthreads();
  int32_t* out = idx_out + seq.out_off[b];
  place_ordered<NT, kMidPer>(key, j0, m, T, need, cnt[0], cnt[1], tot, [&](uint32_t at, int j) { out[at] = j; });
}

// Mid form, up to kDirectSeq scores a sequence: compact and place in one launch.  Every workgroup reads ALL scores of its sequence, a
// thread sixteen of them in registers: lists the candidates in LDS (or, where they are too many, resolves them where they are), counts what
// stands before its own share of 1024, and places that.  The launch that it saves is worth 4.5 us, a thread's sixteen scores cost 2.5,
// 32 of them more than the launch (layer steps of 32 heads on 8, window 8, us in a graph, compact + place / here: 9000 tokens 29.8 / 27.9, 16392
// 37.1 / 34.7; with 32 scores a thread 24000 tokens 43.5 / 43.4, 32768 48.8 / 49.7).  Also beside other layers: 13 layers of 9000 to 16384
// tokens on four streams 24 / 22 us a layer.  A workgroup's own share of the work is a sixteenth, which costs nothing while each has a CU
// to itself and more than the launch beyond kDirectBlocks of them (selections alone, us in a graph: 8 x 16000 scores 14.9 / 13.9, 17 x 9000
// 16.6 / 15.0, 17 x 16000 -- 272 workgroups -- 17.3 / 17.2, 32 x 12000 20.1 / 20.7, 64 x 9000 25.3 / 30.1, 64 x 16000 30.7 / 40.0).
constexpr int kDirectList = 4096;   // candidates that are listed; more are resolved where they are ...
constexpr int kDirectFew = 512;     // ... and above this many they are expected to be equal (16000 scores, 3200 of them equal, 16.2 -> 14.2 us)
template <class TAB>
__global__ __launch_bounds__(kWide) void topk_direct_kernel(const float* __restrict__ scores, TAB seq, int keep_tail, TopkWs ws,
                                                            int32_t* __restrict__ idx_out) {
  short_kernel_priority();
  constexpr int NWV = kWide / 64, PER = kDirectSeq / kWide;
  static_assert(kMidShare == kWide, "a key of the share per thread");
  __shared__ ResolveLds l;
  __shared__ uint32_t list[kDirectList], tot[NWV], cnt[2], listed;
  int b;
  uint32_t blk;
  int j0;
  mid_share(seq, &b, &blk, &j0);
  const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n = (int)(seq.cu[b + 1] - seq.cu[b]), m = n - keep_tail;
  const float* sc = scores + seq.cu[b];
  const int w0 = wv * (64 * PER);   // the wave's first score: its round i is scores w0 + 64 i to w0 + 64 i + 63
  uint32_t key[PER];
  const bool whole = w0 + 64 * PER <= m;   // (uniform) the wave's scores all exist
  if (whole) {
    const float* mine = sc + w0 + lane;
#pragma unroll
    for (int i = 0; i < PER; ++i) key[i] = __float_as_uint(mine[64 * i]);
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) key[i] = __float_as_uint(sc[min(w0 + 64 * i + lane, m - 1)]);
  }
  const uint32_t own[1] = {score_key(sc[min(j0 + t, m - 1)])};
  for (int i = t; i < kBins; i += kWide) l.hist[i] = 0u;
  if (t == 0) { l.n = 0u; listed = 0u; cnt[0] = 0u; cnt[1] = 0u; }
  const BinTiers tiers = ws.mass > 0.f ? bins_around_mean(ws.mass, n) : bins_around(ws.state[b * 8 + 4]);
  uint32_t bin, above, in_bin, lo, width;
  select_bin<kWide, kFineBins>(MergedBins{ws.hist + (size_t)b * 3 * kBins}, (uint32_t)seq.k[b], l.scan, l.res, &bin, &above, &in_bin);
  fine_range(bin, tiers, &lo, &width);
  const uint32_t krem = (uint32_t)seq.k[b] - above, span = (1u << width) - 1u;
  // keys (score_key; where no score of the wave has its sign bit set, one instruction instead of five)
  uint32_t any = 0u;
#pragma unroll
  for (int i = 0; i < PER; ++i) any |= key[i];
  if (__ballot((int)any < 0) == 0ull) {
#pragma unroll
    for (int i = 0; i < PER; ++i) key[i] |= 0x80000000u;
  } else {
#pragma unroll
    for (int i = 0; i < PER; ++i) key[i] = score_key(__uint_as_float(key[i]));
  }
  if (!whole) {   // what does not exist lies below the bin, and below T
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (w0 + 64 * i + lane >= m) key[i] = lo - 1u;   // (a bin from 0 on: the largest key, which no finite score has)
  }
  if (in_bin <= (uint32_t)kDirectList) {
    uint32_t found = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) found += (uint32_t)__popcll(__ballot(key[i] - lo <= span));
    uint32_t at = 0u;
    if (found) {   // (uniform)
      if (lane == 0) at = atomicAdd(&listed, found);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const bool c = key[i] - lo <= span;
        const unsigned long long mc = __ballot(c);
        if (mc) {
          if (c) list[at + (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(mc >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mc, 0u))] = key[i];
          at += (uint32_t)__popcll(mc);
        }
      }
    }
  }
  __syncthreads();
  uint32_t T, need;
  if (in_bin <= (uint32_t)kDirectFew) {
    resolve_key<kWide>([&](auto f) {
      for (uint32_t i = t; i < in_bin; i += kWide) f(list[i]);
    }, lo, (int)width, krem, l, &T, &need);
  } else {   // a crowd: mostly ties
    resolve_key<kWide, true>([&](auto f) {
      if (in_bin <= (uint32_t)kDirectList) {
        for (uint32_t i = t; i < in_bin; i += kWide) f(list[i]);
      } else {
#pragma unroll
        for (int i = 0; i < PER; ++i)
          if (key[i] - lo <= span) f(key[i]);
      }
    }, lo, (int)width, krem, l, &T, &need);
  }
  // keys above and equal to T in the shares before this one, whole rounds of 64
  uint32_t g = 0u, e = 0u;
#pragma unroll
  for (int i = 0; i < PER; ++i)
    if (w0 + 64 * i < j0) {   // (uniform; all of them lie before the prefix's end)
      g += (uint32_t)__popcll(__ballot(key[i] > T));
      e += (uint32_t)__popcll(__ballot(key[i] == T));
    }
  if (lane == 0 && g) atomicAdd(&cnt[0], g);
  if (lane == 0 && e) atomicAdd(&cnt[1], e);
  __syncthreads();
  int32_t* out = idx_out + seq.out_off[b];
  place_ordered<kWide, 1>(own, j0 + wv * 64, m, T, need, cnt[0], cnt[1], tot, [&](uint32_t at, int j) { out[at] = j; });
}

// The pivot detector's metrics from rows of in-degrees (one per query head) whose histograms over the bins of row_bin have been
// built by whoever read the rows first.  The sum of a row's kk largest scores takes no placement and no ordered list.  Two kernels:
//   compact : every workgroup finds the k-th largest key's bin from the row's histogram, adds up its scores ABOVE it (a
//             partial sum per workgroup, fixed order) and appends its scores IN it -- the candidates -- to the row's
//             list (one integer atomic per workgroup reserves the place; the order of the list differs from run to
//             run, and nothing below depends on it);
//   select  : one workgroup per row takes the candidates (the first 32768 in registers), finds the remaining
//             bits 11 at a time with histograms in LDS, and adds the candidates above the k-th key T as integers (they share
//             their exponent: exact, whatever the order), `krem` copies of T's own value for the ties, and the
//             partial sums; also the row's variance.  The workgroup that ends last forms the means over the rows.
// Scores must be non-negative (in-degrees), rows at most 2^24 long.  Both kernels are a few dependent reads and barriers long:
// what they cost grows with the candidates, which is why the bins are fine around the mean, and the
// means take no launch of their own (32 heads, compact + select + means: 128K tokens 28.2 -> 17.8 us, 32K 16.3 -> 11.5 us).
__device__ inline float key_score(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7FFFFFFFu) : ~key);
}

constexpr int kCompThreads = 512;             // the compact kernel
constexpr int kSelThreads = 1024;             // the select kernel: sixteen waves per row ...
constexpr int kSelFew = 512;                  // ... of which eight end at once where they are enough for the candidates
constexpr int kCandPerThread = 32;            // candidates one of its threads keeps in registers
constexpr int kFewPerThread = 2;              // ... where no thread has more

__global__ __launch_bounds__(kCompThreads) void mass_compact_kernel(const float* __restrict__ rows, int64_t n, uint32_t kk,
                                                                    uint32_t at, uint32_t* __restrict__ hist,
                                                                    uint32_t* __restrict__ state, float* __restrict__ cand,
                                                                    float* __restrict__ part_above) {
  short_kernel_priority();
  constexpr int NT = kCompThreads, PER = kPivotShare / NT;
  __shared__ uint32_t scan[NT / 64];
  __shared__ uint32_t res[3];
  __shared__ float red[NT / 64];
  __shared__ float stage[kPivotShare];
  __shared__ uint32_t cnt, gbase;
  const int p = blockIdx.x, h = blockIdx.y, P = gridDim.x, t = threadIdx.x, lane = t & 63;
  const float* d = rows + (int64_t)h * n;
  const int64_t lo = (int64_t)p * kPivotShare;
  float x[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {   // loads first, the histogram scan under them
    const int64_t j = lo + t + i * NT;
    x[i] = j < n ? d[j] : 0.f;
  }
  if (t == 0) cnt = 0u;
  uint32_t* gh = hist + (size_t)h * kRowWords;
  uint32_t t0, above0;
  select_bin<NT, kBins>(MergedBins{gh}, kk, scan, res, &t0, &above0);   // its barriers cover cnt = 0
  float sum = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const bool in = lo + t + i * NT < n;
    const uint32_t bin = row_bin(score_key(fabsf(x[i])), at);
    if (in && bin > t0) sum += x[i];
    const bool c = in && bin == t0;
    const unsigned long long m = __ballot(c);
    if (m) {   // one LDS atomic per wave and step reserves the wave's places
      const int first = __ffsll((long long)m) - 1;
      uint32_t base = 0u;
      if (lane == first) base = atomicAdd(&cnt, (uint32_t)__popcll(m));
      base = __shfl(base, first);
      if (c) stage[base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = x[i];
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) red[t >> 6] = sum;
  __syncthreads();
  if (t == 0) {
    gbase = cnt ? atomicAdd(&gh[kBins], cnt) : 0u;   // the row's candidate counter, behind its histogram
    float s = 0.f;
    for (int i = 0; i < NT / 64; ++i) s += red[i];
    part_above[(int64_t)h * P + p] = s;
    if (p == 0) {
      state[h * 4 + 0] = t0;
      state[h * 4 + 1] = kk - above0;
    }
  }
  __syncthreads();
  float* out = cand + (int64_t)h * n + gbase;
  for (uint32_t i = t; i < cnt; i += NT) out[i] = stage[i];
}

// The `krem`-th largest of c0 candidates, all of whose keys are T plus `bits` open ones: T and krem become that key and how
// many copies of it count; returns the calling thread's share of the significands above it.  PER candidates a thread are kept
// in registers, any others read again on each pass.
template <int NT, int PER>
__device__ inline unsigned long long resolve_row(const float* __restrict__ c, uint32_t c0, uint32_t bits, LdsBins<kBins>& hh,
                                                 uint32_t* scan, uint32_t* res, uint32_t& T, uint32_t& krem) {
  const int t = threadIdx.x;
  float v[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const uint32_t i = (uint32_t)(r * NT + t);
    v[r] = i < c0 ? c[i] : 0.f;
  }
  auto each = [&](auto f) {
#pragma unroll
    for (int r = 0; r < PER; ++r)
      if ((uint32_t)(r * NT + t) < c0) f(score_key(fabsf(v[r])));
    for (uint32_t i = (uint32_t)(PER * NT + t); i < c0; i += NT) f(score_key(fabsf(c[i])));
  };
  while (bits > 0) {   // 17 open bits: 11 and 6; 21: 11 and 10
    const uint32_t take = min(bits, 11u), shift = bits - take;
    for (int i = t; i < kBins; i += NT) hh[i] = 0u;
    __syncthreads();
    each([&](uint32_t key) {
      if (((key ^ T) >> bits) == 0u) atomicAdd(&hh[(key >> shift) & ((1u << take) - 1u)], 1u);
    });
    __syncthreads();
    uint32_t digit, above;
    select_bin<NT, kBins>(hh, krem, scan, res, &digit, &above);
    T |= digit << shift;
    krem -= above;
    bits = shift;
  }
  // every candidate lies in one quarter of an octave or less: they share one exponent and their 24-bit significands
  // add up exactly as integers, in any order
  unsigned long long acc = 0ull;
  const uint32_t hidden = ((T >> 23) & 0xFFu) ? 0x00800000u : 0u;   // (subnormals have no hidden one)
  each([&](uint32_t key) {
    if (key > T) acc += (unsigned long long)((key & 0x007FFFFFu) | hidden);
  });
  return acc;
}

// Few candidates: no long row of steps that find nothing (32K tokens, window 8: 10.2 us without, 6.9 with; 128K, window 64: 12.5
// and 8.5), and up to a thousand of them eight waves, which meet at a barrier sooner than sixteen (a barrier waits for the waves
// that have not ended).  How many there are the row decides and not its length: of a flat row all keys are candidates, of others a
// hundredth (32 heads, window 8, us a call in a graph with sixteen waves / eight up to 32768 keys / here: 2048 keys 26.7 / 25.8 / 25.5,
// 32K 45.4 / 44.7 / 44.2; flat rows 32.0 / 32.3 / 31.4 and 113.4 / 117.9 / 112.7).
__global__ __launch_bounds__(kSelThreads) void mass_select_kernel(const float* __restrict__ cand, int64_t n, int w, uint32_t at,
                                                                  uint32_t* __restrict__ hist,
                                                                  const uint32_t* __restrict__ state,
                                                                  const float* __restrict__ part_above,
                                                                  const float* __restrict__ var_part, int P,
                                                                  float* __restrict__ sums, float* __restrict__ sparsity,
                                                                  float* __restrict__ variance) {
  short_kernel_priority();
  constexpr int NT = kSelThreads;
  __shared__ LdsBins<kBins> hh;
  __shared__ uint32_t scan[NT / 64];
  __shared__ uint32_t res[3];
  __shared__ unsigned long long red64[NT / 64];
  __shared__ float redf[NT / 64], redv[NT / 64];
  __shared__ uint32_t done;
  const int h = blockIdx.x, H = gridDim.x, t = threadIdx.x, lane = t & 63;
  const uint32_t bin = state[h * 4 + 0];
  uint32_t krem = state[h * 4 + 1];
  const uint32_t c0 = hist[(size_t)h * kRowWords + kBins];   // candidates = keys in that bin
  const float* c = cand + (int64_t)h * n;
  const float* pas = part_above + (int64_t)h * P;
  const float* pvs = var_part + (int64_t)h * P;
  float pa = t < P ? pas[t] : 0.f, pv = t < P ? pvs[t] : 0.f;
  const bool few = c0 <= (uint32_t)(kFewPerThread * kSelFew);   // (uniform)
  const int threads = few ? kSelFew : NT, waves = threads / 64;
  if (t >= threads) return;
  for (int p = t + threads; p < P; p += threads) { pa += pas[p]; pv += pvs[p]; }
  uint32_t T, bits;
  row_bin_range(bin, at, &T, &bits);
  unsigned long long acc;
  if (few) acc = resolve_row<kSelFew, kFewPerThread>(c, c0, bits, hh, scan, res, T, krem);
  else if (c0 <= (uint32_t)(kFewPerThread * NT)) acc = resolve_row<NT, kFewPerThread>(c, c0, bits, hh, scan, res, T, krem);
  else acc = resolve_row<NT, kCandPerThread>(c, c0, bits, hh, scan, res, T, krem);
  const uint32_t expo = (T >> 23) & 0xFFu;            // biased exponent (scores are non-negative)
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    acc += __shfl_xor(acc, off);
    pa += __shfl_xor(pa, off);
    pv += __shfl_xor(pv, off);
  }
  if (lane == 0) { red64[t >> 6] = acc; redf[t >> 6] = pa; redv[t >> 6] = pv; }
  __syncthreads();
  if (t == 0) {
    unsigned long long a = 0ull;
    float sa = 0.f, sv = 0.f;
    for (int i = 0; i < waves; ++i) { a += red64[i]; sa += redf[i]; sv += redv[i]; }
    const double m = ldexp((double)a, (int)(expo ? expo : 1u) - 150) + (double)krem * (double)key_score(T) + (double)sa;
    __hip_atomic_store(&sums[2 * h], sv / (float)n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&sums[2 * h + 1], (float)m * (1.0f / (float)w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // release this row's sums, acquire those of the rows that ended before
    done = __hip_atomic_fetch_add(&hist[kBins + 1], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (done != (uint32_t)(H - 1)) return;   // (uniform) the last one adds the rows up, in row order
  float* row = reinterpret_cast<float*>(hh.n);
  static_assert(2 * kMaxBatch <= kBins, "the sums of all rows fit");
  for (int i = t; i < 2 * H; i += threads) row[i] = __hip_atomic_load(&sums[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (t == 0) {
    float vt = 0.f, rt = 0.f;
    for (int i = 0; i < H; ++i) { vt += row[2 * i]; rt += row[2 * i + 1]; }
    *sparsity = rt / (float)H;
    *variance = vt / (float)H;
  }
}

// scores per workgroup of the long form: lighter, more workgroups shorten each kernel's serial part while there are few
inline int share_target(int64_t total_tokens) {
  return total_tokens <= kSmallTotal ? kSmallTarget : kTargetPerBlock;
}

// upper bound of the workgroups one call of the long form launches (the mid form: at most twice as many)
size_t max_blocks(int batch, int64_t total_tokens) {
  const size_t B = (size_t)(batch > 0 ? batch : 1);
  // monotone in total_tokens, so a workspace sized for a long call also serves every shorter one
  const int64_t small = total_tokens < kSmallTotal ? total_tokens : kSmallTotal;
  const int64_t by_small = small / kSmallTarget, by_large = total_tokens / kTargetPerBlock;
  size_t nb = (size_t)(by_small > by_large ? by_small : by_large) + B;
  if (nb > B * kMaxBlocksPerSeq) nb = B * kMaxBlocksPerSeq;
  return nb;
}

// the suffix sums of the long form, or of the mid form (16-bit words, at most twice as many workgroups)
size_t lists_bytes(size_t nb) { return align_up(sizeof(uint32_t) * kLowBins * nb, 256); }
static_assert(2 * sizeof(uint16_t) * kSubBins == sizeof(uint32_t) * kLowBins, "the mid form's words fit the long form's");

}  // namespace

size_t topk_workspace_bytes(int batch, int64_t total_tokens) {
  const size_t B = (size_t)(batch > 0 ? batch : 1);
  const size_t nb = max_blocks(batch, total_tokens);
  return align_up(sizeof(uint32_t) * 3 * B * kBins, 256) + align_up(sizeof(uint32_t) * 8 * B, 256) +
         lists_bytes(nb) + align_up(sizeof(uint32_t) * 2 * nb, 256);
}

// digit histograms, search state of the long form, suffix sums and counts: what the static scratch's limit is stated in
bool topk_static_fits(int batch, int64_t total_tokens) {
  const size_t B = (size_t)(batch > 0 ? batch : 1);
  const size_t nb = max_blocks(batch, total_tokens);
  return align_up(sizeof(uint32_t) * 3 * B * kBins, 256) + align_up(sizeof(uint32_t) * 4 * B, 256) +
         align_up(sizeof(uint32_t) * kLowBins * nb, 256) + align_up(sizeof(uint32_t) * 2 * nb, 256) <= kStaticScratchLists;
}

// Device address and size of the static scratch on the CURRENT device (looked up once per device).
hipError_t topk_static_scratch(void** ptr, size_t* bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* dev_ptr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (dev_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr || ((uintptr_t)p & 255)) return hipErrorInvalidSymbol;
    dev_ptr[dev] = p;
  }
  *ptr = dev_ptr[dev];
  *bytes = kStaticScratchBytes;
  return hipSuccess;
}

// the form a call takes, workgroups per sequence (none where nothing is selected) and the workspace carve
void topk_plan(const SeqTable& seq_in, int keep_tail, void* wsp, SeqTable* plan, TopkWs* ws, unsigned* blocks) {
  *plan = seq_in;
  const int B = plan->batch;
  int64_t longest = 0;
  for (int b = 0; b < B; ++b) {
    const int64_t m = plan->cu[b + 1] - plan->cu[b] - keep_tail;
    if (plan->k[b] > 0 && m > longest) longest = m;
  }
  ws->mode = selection_mode(longest);
  ws->mass = 0.f;
  ws->red = nullptr;
  ws->copy = nullptr;
  ws->beside = 0;
  const int target = ws->mode == kSelMid ? kMidShare : share_target(plan->cu[B]);
  plan->chunk_start[0] = 0;
  for (int b = 0; b < B; ++b) {
    const int64_t m = plan->cu[b + 1] - plan->cu[b] - keep_tail;
    int64_t nblk = plan->k[b] > 0 ? ceil_div(m, target) : 0;
    if (nblk > kMaxBlocksPerSeq) nblk = kMaxBlocksPerSeq;   // (long form: shares grow; the mid form has 256 at most)
    plan->chunk_start[b + 1] = plan->chunk_start[b] + (int)nblk;
  }
  *blocks = (unsigned)plan->chunk_start[B];
  ws->direct = longest <= kDirectSeq && *blocks <= (unsigned)kDirectBlocks;
  const size_t nb = max_blocks(B, plan->cu[B]);   // sum of ceil(m_b / target) <= total / target + B: blocks <= nb (long), 2 nb (mid)
  const size_t Bz = (size_t)(B > 0 ? B : 1);
  uint8_t* p = (uint8_t*)wsp;
  ws->hist = (uint32_t*)p;    p += align_up(sizeof(uint32_t) * 3 * Bz * kBins, 256);
  ws->state = (uint32_t*)p;   p += align_up(sizeof(uint32_t) * 8 * Bz, 256);
  ws->suf = (uint32_t*)p;     p += lists_bytes(nb);
  ws->meta = (uint32_t*)p;
}

// What a fused layer step leaves of the selection: everything in the short form (window indices included), the last two
// launches in the mid form, the last three in the long one.
hipError_t launch_topk_rest(const float* scores, const SeqTable& plan, int keep_tail, const TopkWs& ws,
                            unsigned blocks, int32_t* idx_out, hipStream_t st) {
  with_table(plan, [&](const auto& tab) {
    using T = std::decay_t<decltype(tab)>;
    if (ws.mode == kSelShort) {
      int64_t longest = 0;
      for (int b = 0; b < plan.batch; ++b)
        if (ws.red || plan.k[b] > 0) longest = std::max(longest, plan.cu[b + 1] - plan.cu[b] - (ws.red ? 0 : keep_tail));
      const ReduceWork red = ws.red ? *ws.red : ReduceWork{};
      const CopyWork copy = ws.copy ? *ws.copy : CopyWork{};
      const int parts = ws.copy ? ws.copy_parts : 1;
#define SKV_SHORT_(PER, SUM, COPY)                                                                                      \
  hipLaunchKernelGGL((topk_short_kernel<PER, T, SUM, COPY>), dim3((unsigned)(plan.batch * (SUM ? parts + 1 : parts))), dim3(kWide), 0, st, \
                     scores, tab, keep_tail, idx_out, red, copy, parts)
#define SKV_SHORT(PER, SUM)                                                  \
  if (ws.copy) SKV_SHORT_(PER, SUM, true); else SKV_SHORT_(PER, SUM, false)
      if (ws.red) { if (longest <= kWide) { SKV_SHORT(1, true); } else { SKV_SHORT(2, true); } }
      else if (longest <= 2 * kWide) { SKV_SHORT(2, false); }
      else if (longest <= 4 * kWide) { SKV_SHORT(4, false); }
      else { SKV_SHORT(8, false); }
#undef SKV_SHORT_
#undef SKV_SHORT
    } else if (blocks == 0) {
      return;
    } else if (ws.mode == kSelMid && ws.direct) {
      hipLaunchKernelGGL((topk_direct_kernel<T>), dim3(blocks), dim3(kWide), 0, st, scores, tab, keep_tail, ws, idx_out);
    } else if (ws.mode == kSelMid) {
#define SKV_MID(NT)                                                                                                          \
  hipLaunchKernelGGL((topk_compact_kernel<NT, T>), dim3(blocks), dim3(NT), 0, st, scores, tab, keep_tail, ws);                \
  hipLaunchKernelGGL((topk_place_kernel<NT, T>), dim3(blocks), dim3(NT), 0, st, scores, tab, keep_tail, ws, idx_out)
      if (ws.beside || blocks > 256) { SKV_MID(256); } else { SKV_MID(512); }
#undef SKV_MID
    } else {
      hipLaunchKernelGGL((topk_hist1_kernel<T>), dim3(blocks), dim3(kThreads), 0, st, scores, tab, keep_tail, ws);
      hipLaunchKernelGGL((topk_hist2_kernel<T>), dim3(blocks), dim3(kThreads), 0, st, scores, tab, keep_tail, ws);
      hipLaunchKernelGGL((topk_write_kernel<T>), dim3(blocks), dim3(kThreads), 0, st, scores, tab, keep_tail, ws, idx_out);
    }
  });
  return hipGetLastError();
}

hipError_t launch_pivot_mass(const ReduceWork& red, uint32_t kk, uint32_t at, uint32_t* hist, uint32_t* state, float* cand,
                             float* part_above, const float* var_part, float* sums, float* sparsity, float* variance, hipStream_t st) {
  const int P = pivot_shares(red.total);
  hipLaunchKernelGGL(mass_compact_kernel, dim3((unsigned)P, (unsigned)red.Hq), dim3(kCompThreads), 0, st, red.colsum, red.total, kk,
                     at, hist, state, cand, part_above);
  hipLaunchKernelGGL(mass_select_kernel, dim3((unsigned)red.Hq), dim3(kSelThreads), 0, st, cand, red.total, red.w, at, hist, state,
                     part_above, var_part, P, sums, sparsity, variance);
  return hipGetLastError();
}

// seq.out_off must hold the output offsets, seq.k the budgets.
hipError_t launch_topk(const float* scores, const SeqTable& seq_in, int keep_tail, int32_t* idx_out,
                       void* wsp, hipStream_t st) {
  if (seq_in.batch == 0) return hipSuccess;
  SeqTable seq;
  TopkWs ws;
  unsigned blocks = 0;
  topk_plan(seq_in, keep_tail, wsp, &seq, &ws, &blocks);
  with_table(seq, [&](const auto& tab) {
    using T = std::decay_t<decltype(tab)>;
    if (ws.mode == kSelMid) {
      hipLaunchKernelGGL((topk_mid_init_kernel<T>), dim3((unsigned)seq.batch), dim3(kWide), 0, st, scores, tab, keep_tail, ws, idx_out);
      unsigned hist_wgs = 0;
      for (int b = 0; b < seq.batch; ++b) hist_wgs += (unsigned)ceil_div(seq.chunk_start[b + 1] - seq.chunk_start[b], kHistShares);
      if (hist_wgs > 0)
        hipLaunchKernelGGL((topk_mid_hist_kernel<T>), dim3(hist_wgs), dim3(kHistThreads), 0, st, scores, tab, keep_tail, ws);
    } else if (ws.mode == kSelLong) {
      hipLaunchKernelGGL((topk_init_kernel<T>), dim3(4, seq.batch), dim3(kThreads), 0, st, tab, keep_tail, ws, idx_out);
      if (blocks > 0) hipLaunchKernelGGL((topk_hist0_kernel<T>), dim3(blocks), dim3(kThreads), 0, st, scores, tab, keep_tail, ws);
    }
  });
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_topk_rest(scores, seq, keep_tail, ws, blocks, idx_out, st);
}

}  // namespace skv
