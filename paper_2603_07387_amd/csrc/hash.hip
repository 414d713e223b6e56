// Count-sketch hash tables on the device (the hash family of tn_sketch.h), one
// packed int32 entry per (sample, stream, index).
#include <algorithm>

#include "hash_device.h"
#include "tn_internal.h"

namespace tn {
namespace {

// 2^lg lanes per (stream, sample) derive its coefficients, each for itself, and
// take its indices in turn.  One lane does the least work in all, more take
// less time each.  WAVE: 64 lanes, so that the pair is the wave's and its
// coefficients are derived in scalar registers.
template <bool WAVE>
__global__ __launch_bounds__(256) void hashgen_kernel(const StreamDesc *__restrict__ streams, int64_t n_streams,
                                                      int64_t W, int64_t sample0, int64_t samples, int lg,
                                                      uint32_t mask, int32_t *__restrict__ out) {
  const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x, gid = block * 256 + threadIdx.x;
  const int64_t pairs = n_streams * samples;
  const int64_t pair = WAVE ? block * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : gid >> lg;
  if (pair >= pairs) return;
  const int64_t r = pairs <= 0xffffffffll ? (int64_t)((uint32_t)pair / (uint32_t)n_streams) : pair / n_streams;
  const StreamDesc sd = streams[pair - r * n_streams];
  const HashCoeffs c = hash_coeffs(sd.seed, (uint64_t)(sample0 + r), sd.stream);
  int32_t *dst = out + r * W + sd.offset;
  const int step = WAVE ? 64 : 1 << lg;
  for (int i = (int)gid & (step - 1); i < sd.n; i += step) dst[i] = (int32_t)hash_packed(c, (uint32_t)i, mask);
}

__global__ void copy_i32_kernel(const int32_t *__restrict__ src, int32_t *__restrict__ dst,
                                int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

}  // namespace

int launch_hashgen(const StreamDesc *streams, int64_t n_streams, int64_t W, int64_t sample0,
                   int64_t samples, int64_t m, int64_t max_n, int32_t *out, hipStream_t st) {
  if (n_streams == 0 || samples == 0) return TN_OK;
  if (!streams || !out) return set_error(TN_ERR_ARG, "hashgen: null stream table or output");
  if (samples > 65535 || n_streams > 0x7fffffff)
    return set_error(TN_ERR_UNSUPPORTED, "hashgen: %lld samples x %lld streams per launch",
                     (long long)samples, (long long)n_streams);
  // Lanes until there are 65536 threads (48 pairs of 64 indices: 9.9 us with one
  // lane each, 3.0 with 64; 6016 pairs of 64: 11.0, 5.0), and up to four while
  // there are not a million (557056 pairs of 2 to 32: 48 us with one, 31 with
  // two, 50 with eight; 262144 of 16: 24 with one, 15 with four, 33 with 16).
  // Streams of more than 64 indices: enough lanes for 64 each (16384 pairs of
  // 512: 17.8 us with 64 lanes, 18.8 with four, 17.0 with eight), above 512 all
  // 64, whose stores are whole lines (16500 pairs of 1024: 16.2 us with 64 lanes,
  // 25.6 with four, 17.4 with 16).
  constexpr int64_t kLaneIndices = 64, kLongStream = 512;
  const int64_t pairs = n_streams * samples;
  int lg = 0;
  while (lg < 6 && ((int64_t)1 << lg) < max_n &&
         (pairs << lg < (lg < 2 ? (int64_t)1 << 20 : (int64_t)1 << 16) ||
          max_n >> lg > kLaneIndices || max_n > kLongStream))
    ++lg;
  // (the runtime refuses 2^32 threads in x)
  const int64_t blocks = ((pairs << lg) + 255) / 256, gx = std::min<int64_t>(blocks, 1 << 22), gy = (blocks + gx - 1) / gx;
  if (gy > 65535)
    return set_error(TN_ERR_UNSUPPORTED, "hashgen: %lld samples x %lld streams per launch", (long long)samples,
                     (long long)n_streams);
  hipLaunchKernelGGL(lg == 6 ? hashgen_kernel<true> : hashgen_kernel<false>, dim3((unsigned)gx, (unsigned)gy), dim3(256),
                     0, st, streams, n_streams, W, sample0, samples, lg, (uint32_t)(m - 1), out);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

int launch_copy_i32(const int32_t *src, int32_t *dst, int64_t n, hipStream_t st) {
  if (n == 0) return TN_OK;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(copy_i32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, src, dst, n);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

}  // namespace tn
