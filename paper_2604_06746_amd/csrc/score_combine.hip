// Small kernels around the two scoring passes:
//   combine : merge the per-key-chunk softmax statistics of every query row into
//             lse2 = M + log2 Z (what pass 2 normalises with) and the row entropies of Eq. 4.
//   reduce  : D_j = sum over KV heads / row-chunks of the pass-2 column sums (Eq. 2 without 1/w),
//             plus the means over window rows and heads that finish Eq. 4; optionally also the
//             centrality update below on the value it has just formed.
//   accumulate : C <- lambda C + inv_w D   (Alg. 1 line 6 / Eq. 3).
//   group sums : the same column sums per KV head only (Eq. 2's inner sum over h in H_g), on request.
#include "common.h"

namespace skv {
namespace {

constexpr float kLn2 = 0.6931471805599453f;

// one workgroup of 1024 threads per (sequence b, KV head g, block of 32 query rows): thread = (row,
// slot); the 32 slots of a row split its partial statistics (consecutive threads read consecutive rows,
// the contiguous direction of the partials), then merge in a fixed order: lane pairs, then the sixteen waves as a tree over
// sixteen lanes per row (one thread that merged them one after the other spent fifteen LDS reads and thirty exponentials in a
// chain: a 32K-token layer 49.6 -> 49.3 us at a window of 8, 55.1 -> 54.75 at 32).
constexpr int kCombRows = 32, kCombSlots = 32;

// the value of another lane of the sixteen: across pairs, quads, eights, sixteens (the lanes of a group hold the same merge)
template <int CTRL>
__device__ __forceinline__ float lane_of_other(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int CTRL>
__device__ __forceinline__ void merge_lanes(float& M, float& Z, float& E) {
  const float M2 = lane_of_other<CTRL>(M), Z2 = lane_of_other<CTRL>(Z), E2 = lane_of_other<CTRL>(E);
  merge_stats(M, Z, E, M2, Z2, E2);
}

template <class TAB>
__global__ __launch_bounds__(kCombRows* kCombSlots) void score_combine_kernel(
    TAB seq, int G, int R, int RPC, int RC, int WK, int64_t n_chunks, int row_blocks,
    const float* __restrict__ stats, float* __restrict__ lse2, float* __restrict__ row_ent,
    uint32_t* __restrict__ zero_ptr, int64_t zero_words) {
  short_kernel_priority();
  constexpr int WV = kCombSlots / 2;
  static_assert(WV == 16, "a row's waves are merged by the sixteen lanes of a DPP row");
  __shared__ float sM[WV][kCombRows + 1], sZ[WV][kCombRows + 1], sE[WV][kCombRows + 1];
  // fused layer step: clear the digit histograms of the selection that follows the scoring
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < zero_words; i += (int64_t)gridDim.x * blockDim.x)
    zero_ptr[i] = 0u;
  const int rblk = blockIdx.x % row_blocks;
  const int bg = blockIdx.x / row_blocks;
  const int b = bg / G, g = bg % G;
  const int rl = threadIdx.x & (kCombRows - 1);
  const int slot = threadIdx.x / kCombRows;
  const int row = rblk * kCombRows + rl;
  const int64_t c0 = seq.chunk_start[b], c1 = seq.chunk_start[b + 1];
  const int rowc = min(row, R - 1);
  const int rc = rowc / RPC, rr = rowc % RPC;
  const int grc = g * RC + rc;
  float M = -1.0e30f, Z = 0.f, E = 0.f;
  const int64_t np = (c1 - c0) * WK;
  const float* base = stats + (((int64_t)grc * n_chunks + c0) * WK * 3) * RPC + rr;
  int64_t p = slot;
  for (; p + 3 * kCombSlots < np; p += 4 * kCombSlots) {   // four partials in flight
    float m[4], z[4], e[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float* sp = base + (p + u * kCombSlots) * 3 * RPC;
      m[u] = sp[0]; z[u] = sp[RPC]; e[u] = sp[2 * RPC];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) merge_stats(M, Z, E, m[u], z[u], e[u]);
  }
  for (; p < np; p += kCombSlots) {
    const float* sp = base + p * 3 * RPC;
    merge_stats(M, Z, E, sp[0], sp[RPC], sp[2 * RPC]);
  }
  {  // the two slots of a wave
    const float M2 = __shfl_xor(M, 32), Z2 = __shfl_xor(Z, 32), E2 = __shfl_xor(E, 32);
    merge_stats(M, Z, E, M2, Z2, E2);
  }
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) < kCombRows) { sM[wv][rl] = M; sZ[wv][rl] = Z; sE[wv][rl] = E; }
  __syncthreads();
  if (threadIdx.x >= kCombRows * WV) return;   // (whole waves)
  const int rr2 = threadIdx.x / WV, out_row = rblk * kCombRows + rr2, wave = threadIdx.x % WV;
  M = sM[wave][rr2]; Z = sZ[wave][rr2]; E = sE[wave][rr2];
  merge_lanes<0xB1>(M, Z, E);    // quad_perm 1,0,3,2
  merge_lanes<0x4E>(M, Z, E);    // quad_perm 2,3,0,1
  merge_lanes<0x141>(M, Z, E);   // row_half_mirror
  merge_lanes<0x140>(M, Z, E);   // row_mirror
  if (wave == 0 && out_row < R) {
    float ent = 0.f, l2 = 0.f;
    if (c1 > c0) {
      const float lz = __log2f(Z);
      l2 = M + lz;
      ent = kLn2 * (lz - E / Z);   // -sum a ln a  with a = 2^(x-M)/Z
    }
    const int64_t o = (int64_t)b * G * R + (int64_t)g * R + out_row;
    lse2[o] = l2;
    row_ent[o] = ent;
  }
}

// grid covers the tokens, V floats per thread (V = 4 for long inputs, else 1 so that enough workgroups
// exist to use every CU); planes are added in ascending order, eight loads in flight.
// B workgroups behind those of the tokens (token_wgs) finish Eq. 4, one a sequence: a chain of loads, shuffles and barriers that
// made the first workgroups the launch's last ones when they did it at their end (the kernel
// at 32K tokens 4.6 -> 4.1 us, the layer 49.3 -> 48.6 at a window of 8, 54.75 -> 53.7 at 32).  With `cen` != NULL the kernel also applies
// C <- lambda C + inv_w D with the arithmetic of accumulate_kernel (one fma on the rounded product).
// FUSE > 0 (a fused layer step, Eq. 13 follows Eq. 2 directly): the kernel also starts the selection on the scores it has
// just formed -- their histogram (kSelMid: bins that are finest around their mean, kSelLong: the top 11 bits of their keys) and the
// kept window's indices; workgroups of 1024 threads then, so that there are fewer histograms to merge.
template <class TAB, int V, int FUSE>
__global__ __launch_bounds__(FUSE ? 1024 : 256) void score_reduce_kernel(
    const float* __restrict__ colsum, int GRC, int64_t total, float* __restrict__ indeg,
    const float* __restrict__ row_ent, float* __restrict__ ent_head, float* __restrict__ entropy, int B,
    int Hq, int w, float* __restrict__ cen, float lambda, float inv_w, TAB seq, SelectFusion fs, uint32_t token_wgs) {
  short_kernel_priority();
  __shared__ float hsum[256];
  if (blockIdx.x >= token_wgs) {
    finish_entropy(row_ent, ent_head, entropy, (int)(blockIdx.x - token_wgs), Hq, w, hsum);
    return;
  }
  constexpr bool FUSED = FUSE != 0;
  constexpr int NT = FUSED ? 1024 : 256;
  constexpr int BINS = FUSE == kSelMid ? kFineBins : kTopkBins;
  __shared__ alignas(8) uint32_t h0[FUSED ? BINS : 2];
  const float mass = (float)w * (float)Hq;
  const int64_t i0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * V;
  int b_wg = 0;   // FUSED: the sequence of the workgroup's first token; its digits are counted in LDS
  BinTiers tiers{};   // kSelMid: that sequence's bins
  if constexpr (FUSED) {
    for (int i = threadIdx.x; i < BINS; i += NT) h0[i] = 0u;
    const int64_t first = min((int64_t)blockIdx.x * blockDim.x * V, total > 0 ? total - 1 : 0);
    while (b_wg + 1 < B && first >= seq.cu[b_wg + 1]) ++b_wg;
    if constexpr (FUSE == kSelMid) tiers = bins_around_mean(mass, seq.cu[b_wg + 1] - seq.cu[b_wg]);
    __syncthreads();
  }
  if (i0 < total) {   // V == 4 only when total % 4 == 0
    float a[V], c[V];
#pragma unroll
    for (int j = 0; j < V; ++j) a[j] = 0.f;
    if (cen) {
      if constexpr (V == 4) {
        const float4 t = *reinterpret_cast<const float4*>(cen + i0);
        c[0] = t.x; c[1] = t.y; c[2] = t.z; c[3] = t.w;
      } else {
        c[0] = cen[i0];
      }
    }
    const float* cp = colsum + i0;
    int p = 0;
    for (; p + 8 <= GRC; p += 8) {
      float v[8][V];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if constexpr (V == 4) {
          const float4 t = *reinterpret_cast<const float4*>(cp + (int64_t)(p + u) * total);
          v[u][0] = t.x; v[u][1] = t.y; v[u][2] = t.z; v[u][3] = t.w;
        } else {
          v[u][0] = cp[(int64_t)(p + u) * total];
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int j = 0; j < V; ++j) a[j] += v[u][j];
    }
    for (; p < GRC; ++p)
#pragma unroll
      for (int j = 0; j < V; ++j) a[j] += cp[(int64_t)p * total + j];
    if constexpr (V == 4) *reinterpret_cast<float4*>(indeg + i0) = make_float4(a[0], a[1], a[2], a[3]);
    else indeg[i0] = a[0];
    if (cen) {
#pragma unroll
      for (int j = 0; j < V; ++j) c[j] = fmaf(lambda, c[j], inv_w * a[j]);
      if constexpr (V == 4) *reinterpret_cast<float4*>(cen + i0) = make_float4(c[0], c[1], c[2], c[3]);
      else cen[i0] = c[0];
    }
    if constexpr (FUSED) {
      int b = b_wg;
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const int64_t i = i0 + j;
        while (b + 1 < B && i >= seq.cu[b + 1]) ++b;
        // only the prefix [0, n_b - keep_tail) of a sequence with a budget is searched
        if (seq.k[b] > 0 && i - seq.cu[b] < seq.cu[b + 1] - seq.cu[b] - fs.keep_tail) {
          const uint32_t key = score_key(a[j]);
          uint32_t digit = key >> 21;
          if constexpr (FUSE == kSelMid)
            digit = fine_bin(key, b == b_wg ? tiers : bins_around_mean(mass, seq.cu[b + 1] - seq.cu[b]));
          if (b == b_wg) atomicAdd(&h0[digit], 1u);
          else atomicAdd(&fs.hist[(size_t)b * 3 * kTopkBins + digit], 1u);
        }
      }
    }
  }
  if constexpr (FUSED) {
    __syncthreads();
    uint32_t* gh = fs.hist + (size_t)b_wg * 3 * kTopkBins;
    merge_bins(h0, BINS, gh, NT);
    // the kept window: indices n_b - keep_tail .. n_b - 1 behind the k_b selected ones
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, gsz = (int64_t)token_wgs * blockDim.x;
    const int64_t tail = fs.keep_tail;
    for (int64_t u = gtid; u < (int64_t)B * tail; u += gsz) {
      const int b = (int)(u / tail);
      const int64_t i = u - (int64_t)b * tail;
      fs.idx_out[seq.out_off[b] + seq.k[b] + i] = (int32_t)(seq.cu[b + 1] - seq.cu[b] - tail + i);
    }
  }
}

// per-KV-head in-degree: the column-sum planes of head g added up in plane order
__global__ __launch_bounds__(256) void group_sums_kernel(const float* __restrict__ colsum, int CP, int64_t total,
                                                         float* __restrict__ groups) {
  short_kernel_priority();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int g = blockIdx.y;
  if (i >= total) return;
  float a = 0.f;
  for (int c = 0; c < CP; ++c) a += colsum[((int64_t)g * CP + c) * total + i];
  groups[(int64_t)g * total + i] = a;
}

__global__ __launch_bounds__(256) void accumulate_kernel(float* __restrict__ c, const float* __restrict__ d,
                                                         int64_t n, float lambda, float inv_w, int vec) {
  short_kernel_priority();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (vec) {
    const int64_t i4 = i * 4;
    if (i4 + 3 < n) {
      float4 cv = *reinterpret_cast<float4*>(c + i4);
      const float4 dv = *reinterpret_cast<const float4*>(d + i4);
      cv.x = fmaf(lambda, cv.x, inv_w * dv.x);
      cv.y = fmaf(lambda, cv.y, inv_w * dv.y);
      cv.z = fmaf(lambda, cv.z, inv_w * dv.z);
      cv.w = fmaf(lambda, cv.w, inv_w * dv.w);
      *reinterpret_cast<float4*>(c + i4) = cv;
    } else {
      for (int64_t j = i4; j < n; ++j) c[j] = fmaf(lambda, c[j], inv_w * d[j]);
    }
  } else if (i < n) {
    c[i] = fmaf(lambda, c[i], inv_w * d[i]);
  }
}

}  // namespace

hipError_t launch_score_combine(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq,
                                const float* stats, float* lse2, float* row_ent, uint32_t* zero_ptr,
                                int64_t zero_words, hipStream_t st) {
  const int row_blocks = (int)ceil_div(p.R, kCombRows);
  const int64_t blocks = (int64_t)seq.batch * s.n_kv_heads * row_blocks;
  if (blocks == 0) return hipSuccess;
  with_table(seq, [&](const auto& tab) {
    hipLaunchKernelGGL((score_combine_kernel<std::decay_t<decltype(tab)>>), dim3((unsigned)blocks), dim3(kCombRows * kCombSlots), 0, st,
                       tab, s.n_kv_heads, p.R, p.RPC, p.RC, p.WK, p.n_chunks, row_blocks, stats, lse2, row_ent, zero_ptr, zero_words);
  });
  return hipGetLastError();
}

hipError_t launch_score_reduce(const structkv_shape& s, const ScorePlan& p, const SeqTable& seq,
                               const float* colsum, int64_t total, float* indeg, const float* row_ent,
                               float* ent_head, float* entropy, float* centrality, float lambda, float inv_w,
                               const SelectFusion* fuse, hipStream_t st) {
  const bool vec = (total % 4 == 0) && (((uintptr_t)indeg | (uintptr_t)colsum | (uintptr_t)centrality) & 15) == 0 &&
                   total >= (int64_t)4 * 256 * 1024;
  const bool fused = fuse != nullptr && fuse->hist != nullptr;
  const int threads = fused ? 1024 : 256;
  int64_t blocks = ceil_div(ceil_div(total, vec ? 4 : 1), threads);
  if (blocks == 0) blocks = 1;
  const SelectFusion fs = fused ? *fuse : SelectFusion{};
#define SKV_REDUCE(V, F)                                                                                       \
  hipLaunchKernelGGL((score_reduce_kernel<T, V, F>), dim3((unsigned)(blocks + seq.batch)), dim3(threads), 0, st, colsum, \
                     s.n_kv_heads * p.CP, total, indeg, row_ent, ent_head, entropy, seq.batch, s.n_q_heads,    \
                     s.window, centrality, lambda, inv_w, tab, fs, (uint32_t)blocks)
  with_table(seq, [&](const auto& tab) {
    using T = std::decay_t<decltype(tab)>;
    if (vec) { if (!fused) SKV_REDUCE(4, 0); else if (fs.mode == kSelMid) SKV_REDUCE(4, kSelMid); else SKV_REDUCE(4, kSelLong); }
    else     { if (!fused) SKV_REDUCE(1, 0); else if (fs.mode == kSelMid) SKV_REDUCE(1, kSelMid); else SKV_REDUCE(1, kSelLong); }
  });
#undef SKV_REDUCE
  return hipGetLastError();
}

hipError_t launch_group_sums(const structkv_shape& s, const ScorePlan& p, const float* colsum, int64_t total,
                             float* groups, hipStream_t st) {
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(group_sums_kernel, dim3((unsigned)ceil_div(total, 256), (unsigned)s.n_kv_heads), dim3(256), 0,
                     st, colsum, p.CP, total, groups);
  return hipGetLastError();
}

hipError_t launch_accumulate(float* c, const float* d, int64_t n, float lambda, float inv_w, hipStream_t st) {
  if (n == 0) return hipSuccess;
  // four floats per thread only when that still leaves enough workgroups to use every CU
  const int vec = (((uintptr_t)c | (uintptr_t)d) & 15) == 0 && n >= (int64_t)4 * 256 * 1024;
  const int64_t work = vec ? ceil_div(n, 4) : n;
  hipLaunchKernelGGL(accumulate_kernel, dim3((unsigned)ceil_div(work, 256)), dim3(256), 0, st, c, d, n,
                     lambda, inv_w, vec);
  return hipGetLastError();
}

}  // namespace skv
