// Turnstile updates of resident sketches (the streaming setting of the
// cyclic method: Algorithm 1 keeps the sketch x_k of every tensor, and an
// update X_k(i) += delta changes one bucket of it per sample, in O(q_k)).
//
// A resident plan (TN_FLAG_RESIDENT) keeps the time-domain sketches of all S
// samples, [sample][slot][m] (FP64 for FP64 data, FP32 otherwise), and the
// packed hash tables of all samples.  An update adds s(i) delta to bucket
// (sum_u h_u(i_u)) mod m of the tensor's first slot (the combine adds a
// tensor's slots), with the complement bucket on the second mode of each
// contraction (Def. 14), exactly as the scatter would for that entry.
#include <algorithm>

#include "tn_internal.h"

namespace tn {
namespace {

constexpr int kUpdates = 4;  // per thread and round, their index loads in flight together

// The words of kUpdates updates u0, u0 + step, ... below n: bucket, sign of the
// update in bit 31, and the update x; in[k] false outside the range or the
// tensor.  A digit takes one multiplication and a correction, by inv =
// floor((2^32 - 1) / n): for i < 2^32 (tensors have at most 2^31 entries), i
// inv / 2^32 is less than one below i / n.
__device__ __forceinline__ void update_words(const ModeDesc *__restrict__ modes, int mode0, int q, int64_t size,
                                             const int32_t *__restrict__ tab, uint32_t m, int64_t u0, int64_t step,
                                             int64_t n, const int64_t *__restrict__ idx,
                                             const double *__restrict__ delta, bool *in, uint32_t *b, double *x) {
  const uint32_t mask = m - 1;
  uint32_t i[kUpdates];
#pragma unroll
  for (int k = 0; k < kUpdates; ++k) {
    const int64_t u = min(u0 + k * step, n - 1), e = idx[u];
    in[k] = u0 + k * step < n && e >= 0 && e < size;  // outside the tensor: ignored
    i[k] = in[k] ? (uint32_t)e : 0u;
    x[k] = delta[u];
    b[k] = 0;
  }
  for (int j = q - 1; j >= 0; --j) {  // row-major: the last mode varies fastest
    const ModeDesc md = modes[mode0 + j];
    const uint32_t dn = (uint32_t)md.n, inv = 0xffffffffu / dn;
#pragma unroll
    for (int k = 0; k < kUpdates; ++k) {
      uint32_t quo = __umulhi(i[k], inv), d = i[k] - quo * dn;
      if (d >= dn) {
        d -= dn;
        ++quo;
      }
      i[k] = quo;
      const uint32_t v = (uint32_t)tab[md.table_off + d];
      uint32_t h = v & ~kSignBit;
      if (md.comp) h = (m - h) & mask;
      b[k] = (((b[k] & ~kSignBit) + h) & mask) | ((b[k] ^ v) & kSignBit);
    }
  }
#pragma unroll
  for (int k = 0; k < kUpdates; ++k)
    if (b[k] & kSignBit) x[k] = -x[k];
}

// Few updates: straight into the sketch.  A block's 256 threads are 2^lg
// updates x (256 >> lg) samples, lg as large as the call's updates fill.
template <typename A>
__global__ __launch_bounds__(256) void stream_update_kernel(
    const ModeDesc *__restrict__ modes, int mode0, int q, int64_t size, const int32_t *__restrict__ tables,
    int64_t W, int64_t S, int log2m, int64_t sample_stride, int64_t slot_off, A *__restrict__ ybuf, int64_t n,
    const int64_t *__restrict__ idx, const double *__restrict__ delta, int lg) {
  const uint32_t m = 1u << log2m;
  const int tid = threadIdx.x, lanes = 1 << lg;
  const int64_t u0 = (int64_t)blockIdx.x * (lanes * kUpdates) + (tid & (lanes - 1));
  for (int64_t s = (int64_t)blockIdx.y * (256 >> lg) + (tid >> lg); s < S; s += (int64_t)gridDim.y * (256 >> lg)) {
    bool in[kUpdates];
    uint32_t b[kUpdates];
    double x[kUpdates];
    update_words(modes, mode0, q, size, tables + s * W, m, u0, lanes, n, idx, delta, in, b, x);
    A *y = ybuf + s * sample_stride + slot_off;
#pragma unroll
    for (int k = 0; k < kUpdates; ++k)
      if (in[k]) atomicAdd(y + (b[k] & (m - 1)), (A)x[k]);
  }
}

// Many updates: a block adds its share of them to one sample's sketch in
// LDS, in FP64, and the sums to the sketch in one coalesced pass.  Adds to
// random words of memory run at 22 per ns whatever their type and wherever
// their blocks are, adds of whole lines at 226, FP64 adds in LDS at 1670
// (FP32 ones, a compare-and-swap loop there, at 200).
constexpr int kShareThreads = 512;
template <typename A>
__global__ __launch_bounds__(kShareThreads) void stream_share_kernel(
    const ModeDesc *__restrict__ modes, int mode0, int q, int64_t size, const int32_t *__restrict__ tables,
    int64_t W, int64_t S, int log2m, int64_t sample_stride, int64_t slot_off, A *__restrict__ ybuf, int64_t n,
    const int64_t *__restrict__ idx, const double *__restrict__ delta, int64_t share) {
  extern __shared__ __align__(16) double acc[];
  const uint32_t m = 1u << log2m;
  const int tid = threadIdx.x;
  const int64_t first = (int64_t)blockIdx.x * share, last = min(first + share, n);
  for (int64_t s = blockIdx.y; s < S; s += gridDim.y) {
    for (uint32_t i = tid; i < m; i += kShareThreads) acc[i] = 0.0;
    __syncthreads();
    for (int64_t u0 = first; u0 < last; u0 += kUpdates * kShareThreads) {
      bool in[kUpdates];
      uint32_t b[kUpdates];
      double x[kUpdates];
      update_words(modes, mode0, q, size, tables + s * W, m, u0 + tid, kShareThreads, last, idx, delta, in, b, x);
#pragma unroll
      for (int k = 0; k < kUpdates; ++k)
        if (in[k])
          __hip_atomic_fetch_add(&acc[b[k] & (m - 1)], x[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    A *y = ybuf + s * sample_stride + slot_off;
    for (uint32_t i = tid; i < m; i += kShareThreads) {
      const double v = acc[i];
      if (v != 0.0) atomicAdd(y + i, (A)v);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(uint4 *__restrict__ p, int64_t quads, int tail) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t i = t; i < quads; i += (int64_t)gridDim.x * blockDim.x) p[i] = make_uint4(0u, 0u, 0u, 0u);
  if (t < tail) reinterpret_cast<uint32_t *>(p + quads)[t] = 0u;
}

// LDS of 128 KB at most; blocks that keep every CU at work.
constexpr int kMaxLog2Share = 14;
constexpr int64_t kShareBlocks = 1024;
// A share's pass over its m words takes as long as 16 m adds to random words of
// memory (direct / shares, FP32: m = 16384, 16384 updates, one sample 4.6 / 15.9
// us, 16 samples 16.2 / 16.2, 64 samples 53 / 17; m = 4096, 16384 updates, one
// sample 4.6 / 5.7, four 5.9 / 5.8, 16 16.0 / 5.9).
constexpr int64_t kShareAdds = 16;

}  // namespace

int launch_stream_update(const ModeDesc *modes, int mode0, int q, int64_t size, const int32_t *tables, int64_t W,
                         int64_t S, int log2m, int64_t n_slots, int32_t slot0, int dtype, void *ybuf, int64_t n,
                         const int64_t *idx, const double *delta, hipStream_t st) {
  if (n == 0) return TN_OK;
  const int64_t m = 1ll << log2m;
  auto run = [&](auto kern, dim3 grid, int threads, size_t lds, auto *y, auto split) -> int {
    if (lds > 65536)
      TN_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, grid, dim3(threads), lds, st, modes, mode0, q, size, tables, W, S, log2m, n_slots * m,
                       (int64_t)slot0 * m, y, n, idx, delta, split);
    TN_HIP_CHECK(hipGetLastError());
    return TN_OK;
  };
  if (n >= m && n * S >= kShareAdds * m && log2m <= kMaxLog2Share) {
    // shares of at least m updates, so that the pass over the sketch does not
    // outweigh them, and blocks for the chip
    const int64_t shares = std::max<int64_t>(1, std::min(n / m, (kShareBlocks + S - 1) / S));
    const int64_t share = (n + shares - 1) / shares;
    const dim3 grid((unsigned)shares, (unsigned)std::min<int64_t>(S, 65535));
    const size_t lds = (size_t)m * 8;
    if (dtype == TN_F64)
      return run(stream_share_kernel<double>, grid, kShareThreads, lds, reinterpret_cast<double *>(ybuf), share);
    return run(stream_share_kernel<float>, grid, kShareThreads, lds, reinterpret_cast<float *>(ybuf), share);
  }
  int lg = 0;  // lanes along the updates: the call's updates, kUpdates to a lane
  while (lg < 8 && ((int64_t)kUpdates << lg) < n) ++lg;
  const int64_t per = (int64_t)kUpdates << lg, rows = 256 >> lg;
  const dim3 grid((unsigned)((n + per - 1) / per), (unsigned)std::min<int64_t>((S + rows - 1) / rows, 65535));
  if (dtype == TN_F64)
    return run(stream_update_kernel<double>, grid, 256, 0, reinterpret_cast<double *>(ybuf), lg);
  return run(stream_update_kernel<float>, grid, 256, 0, reinterpret_cast<float *>(ybuf), lg);
}

// Zero a 16-byte-aligned buffer with a kernel (graph-safe, unlike a memset
// node).  bytes must be a multiple of 4.
int launch_fill_zero(void *buf, size_t bytes, hipStream_t st) {
  const int64_t quads = (int64_t)(bytes / 16);
  const int tail = (int)(bytes % 16 / 4);
  if (bytes == 0) return TN_OK;
  const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>((quads + 255) / 256, 2048));
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, st, reinterpret_cast<uint4 *>(buf), quads, tail);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

}  // namespace tn
