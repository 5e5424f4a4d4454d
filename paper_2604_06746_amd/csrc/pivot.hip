// Sparsity and variance of the attention for Dynamic Pivot Layer Detection (paper Eq. 5-6), from the
// per-head in-degree vectors D_h (what structkv_score_layer_groups returns when every query head is its own
// group).  Reading of the paper's free row index: a head's attention is pooled over the window rows,
// a_h[j] = D_h[j] / w, a probability vector over the keys.
//   variance_h = (1/n) sum_j (a_h[j] - 1/n)^2          (the mean of a probability vector is 1/n)
//   sparsity_h = sum of a_h over the k keys selected by structkv_select_topk
// A head's keys are cut into up to kPivotMaxSlices slices, one workgroup each; all sums follow a fixed order,
// so results are bit-reproducible.
#include "common.h"

namespace skv {
namespace {

// sum over the workgroup in a fixed order (256 threads); result valid in thread 0
__device__ inline float block_sum(float v, float* sh /*[256]*/) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  return sh[0];
}

// grid (H, P): workgroup (h, p) takes the p-th slice of head h's keys and of its selected indices and writes
// two partial sums; heads [H][n], idx [H][k] (head-local key indices), part [H][P][2]
__global__ __launch_bounds__(256) void pivot_head_kernel(const float* __restrict__ heads, int64_t n,
                                                         const int32_t* __restrict__ idx, int64_t k, float inv_w,
                                                         float* __restrict__ part) {
  __shared__ float sh[256];
  const int h = blockIdx.x, p = blockIdx.y, P = gridDim.y;
  const float* d = heads + (int64_t)h * n;
  const float mean = 1.0f / (float)n;
  const int64_t per = (n + P - 1) / P, lo = (int64_t)p * per, hi = lo + per < n ? lo + per : n;
  float v = 0.f;
  for (int64_t j = lo + threadIdx.x; j < hi; j += 256) {
    const float a = d[j] * inv_w - mean;
    v = fmaf(a, a, v);
  }
  const float vs = block_sum(v, sh);
  __syncthreads();
  const int64_t kper = (k + P - 1) / P, klo = (int64_t)p * kper, khi = klo + kper < k ? klo + kper : k;
  float r = 0.f;
  const int32_t* ix = idx + (int64_t)h * k;
  for (int64_t i = klo + threadIdx.x; i < khi; i += 256) {
    int64_t j = ix[i];
    if (j < 0 || j >= n) j = 0;
    r += d[j];
  }
  const float rs = block_sum(r, sh);
  if (threadIdx.x == 0) {
    part[((int64_t)h * P + p) * 2 + 0] = vs;
    part[((int64_t)h * P + p) * 2 + 1] = rs;
  }
}

// Everything that reads all of the per-head in-degrees which a scoring call leaves in its column-sum planes (pass 2 with one
// plane per query head), in one launch of 1-D workgroups:
//   workgroup 0               the means of the row entropies (Eq. 4),
//   then ceil(n / 512)        the layer's in-degrees, the planes added up in ascending order as the reduce kernel does,
//   then H x pivot_shares(n)  hist[h][row_bin of heads[h][j]] += 1;   part[h][p] = sum over the share's keys of (heads/w - 1/n)^2
// Short launches that wait on memory run side by side here instead of one after the other.  In bins of a quarter octave most
// of a workgroup's LDS additions met in a few words.  With the finer ones and one launch, 32 heads: 128K tokens
// 18.4 -> 9.6 us (the 16.8 MB of planes read twice, the second time from the caches), 32K 8.0 -> 4.3 us.
constexpr int kPlaneThreads = 512;

__global__ __launch_bounds__(kPlaneThreads) void pivot_planes_kernel(ReduceWork rw, int reduce_wgs, int shares, uint32_t at,
                                                                     uint32_t* __restrict__ hist, float* __restrict__ part) {
  short_kernel_priority();
  constexpr int NT = kPlaneThreads, PER = kPivotShare / NT;
  __shared__ alignas(8) uint32_t h0[kTopkBins];
  __shared__ float sh[256];
  const int64_t n = rw.total;
  int wg = (int)blockIdx.x;
  if (wg == 0) {
    finish_entropy(rw.row_ent, rw.ent_head, rw.entropy, 0, rw.Hq, rw.w, sh);
    return;
  }
  if (--wg < reduce_wgs) {
    const int64_t i = (int64_t)wg * NT + threadIdx.x;
    if (i >= n) return;
    const float* cp = rw.colsum + i;
    float a = 0.f;
    int p = 0;
    for (; p + 16 <= rw.planes; p += 16) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = cp[(int64_t)(p + u) * n];
#pragma unroll
      for (int u = 0; u < 16; ++u) a += v[u];
    }
    for (; p < rw.planes; ++p) a += cp[(int64_t)p * n];
    rw.indeg[i] = a;
    return;
  }
  wg -= reduce_wgs;
  const int h = wg / shares, p = wg % shares;
  const float* d = rw.colsum + (int64_t)h * n;
  const int64_t lo = (int64_t)p * kPivotShare;
  float x[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {   // loads first, the histogram's clearing under them
    const int64_t j = lo + threadIdx.x + i * NT;
    x[i] = j < n ? d[j] : 0.f;
  }
  for (int i = threadIdx.x; i < kTopkBins; i += NT) h0[i] = 0u;
  __syncthreads();
  const float mean = 1.0f / (float)n, inv_w = 1.0f / (float)rw.w;
  float v = 0.f;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    if (lo + threadIdx.x + i * NT < n) {
      atomicAdd(&h0[row_bin(score_key(fabsf(x[i])), at)], 1u);   // (the absolute value: a NaN's sign)
      const float a = x[i] * inv_w - mean;
      v = fmaf(a, a, v);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();   // completes the LDS histogram too
  merge_bins(h0, kTopkBins, hist + (size_t)h * kRowWords, NT);
  if (threadIdx.x == 0) {
    float vs = 0.f;
    for (int i = 0; i < NT / 64; ++i) vs += sh[i];
    part[(int64_t)h * shares + p] = vs;
  }
}

// per head: the partial sums in slice order; then the means over the heads, in head order (valid == 0: zeros)
__global__ __launch_bounds__(256) void pivot_finish_kernel(const float* __restrict__ part, int H, int P, int64_t n,
                                                           float inv_w, int valid, float* __restrict__ sparsity,
                                                           float* __restrict__ variance) {
  __shared__ float sv[256], sr[256];
  float rt = 0.f, vt = 0.f;
  if (valid) {
    for (int h0 = 0; h0 < H; h0 += 256) {   // heads in rounds of 256, each round summed in head order
      const int h = h0 + (int)threadIdx.x;
      float vs = 0.f, rs = 0.f;
      if (h < H)
        for (int p = 0; p < P; ++p) { vs += part[((int64_t)h * P + p) * 2]; rs += part[((int64_t)h * P + p) * 2 + 1]; }
      sv[threadIdx.x] = vs / (float)n;
      sr[threadIdx.x] = rs * inv_w;
      __syncthreads();
      if (threadIdx.x == 0)
        for (int i = 0; i < 256 && h0 + i < H; ++i) { vt += sv[i]; rt += sr[i]; }
      __syncthreads();
    }
  }
  if (threadIdx.x == 0) {
    *sparsity = rt / (float)H;
    *variance = vt / (float)H;
  }
}

__global__ void zero_floats_kernel(float* __restrict__ p, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

}  // namespace

hipError_t launch_zero_floats(float* p, int n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_floats_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

int pivot_slices(int64_t n) {
  const int64_t p = (n + 8191) / 8192;
  return (int)(p < 1 ? 1 : (p > kPivotMaxSlices ? kPivotMaxSlices : p));
}

hipError_t launch_pivot_heads(const float* heads, int H, int64_t n, const int32_t* idx, int64_t k, float inv_w,
                              float* part, hipStream_t st) {
  if (H == 0 || n == 0) return hipSuccess;
  hipLaunchKernelGGL(pivot_head_kernel, dim3((unsigned)H, (unsigned)pivot_slices(n)), dim3(256), 0, st, heads, n,
                     idx, k, inv_w, part);
  return hipGetLastError();
}

hipError_t launch_pivot_finish(const float* part, int H, int64_t n, float inv_w, int valid, float* sparsity,
                               float* variance, hipStream_t st) {
  hipLaunchKernelGGL(pivot_finish_kernel, dim3(1), dim3(256), 0, st, part, H, pivot_slices(n), n, inv_w, valid,
                     sparsity, variance);
  return hipGetLastError();
}

hipError_t launch_pivot_planes(const ReduceWork& red, uint32_t at, uint32_t* hist, float* var_part, hipStream_t st) {
  const int64_t reduce_wgs = ceil_div(red.total, kPlaneThreads);
  const int shares = pivot_shares(red.total);
  hipLaunchKernelGGL(pivot_planes_kernel, dim3((unsigned)(1 + reduce_wgs + (int64_t)red.Hq * shares)), dim3(kPlaneThreads), 0, st,
                     red, (int)reduce_wgs, shares, at, hist, var_part);
  return hipGetLastError();
}

}  // namespace skv
