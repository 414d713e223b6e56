// Regressor of the learned sketch-size selector (tn_mlp.h): a 3-layer tanh
// perceptron in FP32 with hand-written forward, backward and Adam kernels.
//
//   mlp_fwd_bwd_kernel : a block takes 16 rows (of very large batches four
//                        times 16 in turn); the parameters and the rows'
//                        activations live in LDS; it writes predictions and/or
//                        the block's partial gradient (sums over its rows) and
//                        partial loss, FP64.
//   mlp_rows_kernel    : predictions of narrow networks for many rows, a lane
//                        to a row.
//   mlp_reduce_kernel  : sums the blocks' partials in a fixed order
//                        (deterministic), 64 parameters per block, and either
//                        exports the gradient or applies a bias-corrected Adam
//                        step.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/tn_mlp.h"
#include "tn_internal.h"

struct tn_mlp {
  int device = 0;
  int D = 0, H = 0;
  int64_t P = 0;
  float *d_params = nullptr;
  float *d_m = nullptr, *d_v = nullptr;
  double *d_partial = nullptr;  // [blocks][P + 1]
  int64_t partial_blocks = 0;
  double *d_scalar = nullptr;   // [0] loss of the last reduction, [1] running epoch loss
  int64_t t = 0;                // Adam steps taken
  size_t lds = 0;
};

namespace tn {
namespace {

constexpr int kRows = 64;  // rows of activations that the size limit of tn_mlp_create counts
constexpr int kTile = 16;  // rows a block takes at a time
constexpr int kRS = 20;    // floats between units in LDS: 16 rows and 4 spare (16-byte accesses, bank spread)
// Batches of more tiles than this give each block four: the partials of a
// block are as long as the parameters.
constexpr int64_t kManyTiles = 1024;

// LDS floats: the weights with one spare column, biases, output layer; the
// inputs and four activation arrays unit by unit, kRS floats each, units padded
// to a multiple of four; the rows' output derivatives.
__host__ __device__ constexpr int mlp_up4(int x) { return (x + 3) & ~3; }
size_t mlp_lds_bytes(int D, int H) {
  const size_t w = (size_t)H * (D + 1) + (size_t)H * (H + 1) + 3 * (size_t)H + 1;
  return 4 * (((w + 3) & ~(size_t)3) + (size_t)kRS * ((size_t)mlp_up4(D) + 4 * (size_t)mlp_up4(H)) + kTile);
}

// Eight waves, two rows each; a lane takes one unit (H > 64: two) of its wave's
// rows, so that a weight is read once for two rows, from a padded row (no bank
// conflicts), and the rows' values by 8-byte broadcast.  Every dot product
// runs in the order of its index, in FP32 as before.  The gradients of the
// weight matrices are taken as 4 x 4 tiles per thread, over the rows in order,
// in FP64.
// What bounds it: the latency of its phases (16 rows are 0.3 M multiply-adds);
// 4096 rows fill the 256 CUs with one block each.  One step of 4096 rows, 32
// inputs, 64 hidden units: 239 us with 64 rows per block, unpadded weights (64
// lanes of one bank) and one gradient entry per thread; 23 us now.
__global__ __launch_bounds__(512) void mlp_fwd_bwd_kernel(
    const float *__restrict__ params, int D, int H, const float *__restrict__ X,
    const float *__restrict__ y, int64_t row0, int64_t n, float scale, float *__restrict__ pred,
    double *__restrict__ partial, int64_t P, int tiles) {
  extern __shared__ __align__(16) float sm[];
  const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
  if (row0 + block * tiles * kTile >= n) return;  // padding of the grid
  const int D1 = D + 1, H1 = H + 1, H4 = mlp_up4(H);
  float *W1 = sm;                 // [H][D + 1]
  float *W2 = W1 + H * D1;        // [H][H + 1]
  float *b1 = W2 + H * H1;        // [H]
  float *b2 = b1 + H;             // [H]
  float *W3 = b2 + H;             // [H]
  float *b3 = W3 + H;             // [1]
  float *xs = sm + (((H * D1 + H * H1 + 3 * H + 1) + 3) & ~3);  // [D][kRS]
  float *h1 = xs + kRS * mlp_up4(D);  // [H][kRS]
  float *h2 = h1 + kRS * H4;
  float *d2 = h2 + kRS * H4;      // dL/da2
  float *d1 = d2 + kRS * H4;      // dL/da1
  float *dy = d1 + kRS * H4;      // [16]
  __shared__ double lpart[kTile];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float *pW2 = params + (int64_t)H * D + H, *pb2 = pW2 + (int64_t)H * H;
  for (int j = wave; j < H; j += 8) {
    for (int d = lane; d < D; d += 64) W1[j * D1 + d] = params[j * D + d];
    for (int k = lane; k < H; k += 64) W2[j * H1 + k] = pW2[j * H + k];
  }
  for (int j = tid; j < H; j += 512) {
    b1[j] = params[H * D + j];
    b2[j] = pb2[j];
    W3[j] = pb2[H + j];
  }
  if (tid == 0) b3[0] = pb2[2 * H];
  double *out = partial ? partial + block * (P + 1) : nullptr;
  for (int tile = 0; tile < tiles; ++tile) {
    const int64_t base = row0 + (block * tiles + tile) * kTile;
    if (tile > 0) {
      if (base >= n) break;  // uniform over the block
      __syncthreads();       // the last tile's readers are done
    }
    for (int s = wave; s < kTile; s += 8)
      for (int d = lane; d < D; d += 64) xs[d * kRS + s] = (base + s < n) ? X[(base + s) * D + d] : 0.f;
    __syncthreads();
    const int r0 = 2 * wave;
    // a_j = bias_j + sum_i w[j][i] in[i] for the wave's two rows, then tanh
    auto layer = [&](const float *w, int ws, int ni, const float *bias, const float *in, float *to) {
      for (int j = lane; j < H; j += 64) {
        const float *wj = w + j * ws;
        float a0 = bias[j], a1 = a0;
#pragma unroll 8
        for (int i = 0; i < ni; ++i) {
          const float v = wj[i];
          const float2 x2 = *reinterpret_cast<const float2 *>(in + i * kRS + r0);
          a0 = fmaf(v, x2.x, a0);
          a1 = fmaf(v, x2.y, a1);
        }
        *reinterpret_cast<float2 *>(to + j * kRS + r0) = make_float2(tanhf(a0), tanhf(a1));
      }
    };
    // a wave reads only the rows it wrote itself, but for the output layer
    layer(W1, D1, D, b1, xs, h1);
    __syncthreads();
    layer(W2, H1, H, b2, h1, h2);
    __syncthreads();
    if (tid < kTile) {
      const int s = tid;
      float o = b3[0];
#pragma unroll 8
      for (int j = 0; j < H; ++j) o = fmaf(W3[j], h2[j * kRS + s], o);
      const bool valid = base + s < n;
      if (pred && valid) pred[base + s] = o;
      if (partial) {
        const float r = valid ? o - y[base + s] : 0.f;
        dy[s] = r * scale;
        lpart[s] = 0.5 * (double)r * (double)r;
      }
    }
    if (!partial) continue;
    __syncthreads();
    for (int j = lane; j < H; j += 64) {
      const float2 t2 = *reinterpret_cast<const float2 *>(h2 + j * kRS + r0);
      const float2 y2 = *reinterpret_cast<const float2 *>(dy + r0);
      const float w = W3[j];
      *reinterpret_cast<float2 *>(d2 + j * kRS + r0) =
          make_float2(y2.x * w * (1.f - t2.x * t2.x), y2.y * w * (1.f - t2.y * t2.y));
    }
    __syncthreads();
    for (int k = lane; k < H; k += 64) {
      float a0 = 0.f, a1 = 0.f;
#pragma unroll 8
      for (int j = 0; j < H; ++j) {
        const float v = W2[j * H1 + k];
        const float2 g2 = *reinterpret_cast<const float2 *>(d2 + j * kRS + r0);
        a0 = fmaf(v, g2.x, a0);
        a1 = fmaf(v, g2.y, a1);
      }
      const float2 t2 = *reinterpret_cast<const float2 *>(h1 + k * kRS + r0);
      *reinterpret_cast<float2 *>(d1 + k * kRS + r0) =
          make_float2(a0 * (1.f - t2.x * t2.x), a1 * (1.f - t2.y * t2.y));
    }
    __syncthreads();
    auto emit = [&](int64_t p, double g) { out[p] = tile > 0 ? out[p] + g : g; };
    // 4 x 4 tiles of the two weight matrices' gradients: sum_s u[j][s] v[i][s]
    const int tj = H4 / 4, t1 = tj * (mlp_up4(D) / 4), t2 = tj * tj;
    for (int t = tid; t < t1 + t2; t += 512) {
      const bool first = t < t1;
      const int q = first ? t : t - t1, ni = first ? D : H, ti = mlp_up4(ni) / 4;
      const int j0 = 4 * (q / ti), i0 = 4 * (q - (q / ti) * ti);
      const float *u = (first ? d1 : d2) + j0 * kRS, *v = (first ? xs : h1) + i0 * kRS;
      double g[4][4] = {};
#pragma unroll
      for (int s0 = 0; s0 < kTile; s0 += 4) {
        float4 a[4], b[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[e] = *reinterpret_cast<const float4 *>(u + e * kRS + s0);
          b[e] = *reinterpret_cast<const float4 *>(v + e * kRS + s0);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int f = 0; f < 4; ++f)
              g[e][f] += (double)reinterpret_cast<const float *>(&a[e])[s] *
                         (double)reinterpret_cast<const float *>(&b[f])[s];
      }
      const int64_t off = first ? 0 : (int64_t)H * D + H;
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int f = 0; f < 4; ++f)
          if (j0 + e < H && i0 + f < ni) emit(off + (int64_t)(j0 + e) * ni + i0 + f, g[e][f]);
    }
    // biases and output layer
    for (int j = tid; j < H; j += 512) {
      double g1 = 0.0, g2 = 0.0, g3 = 0.0;
#pragma unroll 4
      for (int s = 0; s < kTile; ++s) {
        g1 += d1[j * kRS + s];
        g2 += d2[j * kRS + s];
        g3 += (double)dy[s] * h2[j * kRS + s];
      }
      emit((int64_t)H * D + j, g1);
      emit((int64_t)H * D + H + (int64_t)H * H + j, g2);
      emit((int64_t)H * D + 2 * H + (int64_t)H * H + j, g3);
    }
    if (tid == 511) {
      double g = 0.0, l = 0.0;
      for (int s = 0; s < kTile; ++s) {
        g += dy[s];
        l += lpart[s];
      }
      emit(P - 1, g);
      emit(P, l);
    }
  }
}

// Predictions of narrow networks (H <= kRowUnits) for many rows: a block's lanes
// are 64 rows, its waves (mlp_row_waves) take four units each in turn.  The rows'
// inputs, kRowInputs at a time, and both layers live in LDS unit by unit,
// kRowStride floats each; weights come through the scalar cache, four units' at
// a time.  Every dot product runs in the order of its index, as in
// mlp_fwd_bwd_kernel, whose lanes are units and are left idle by a narrow layer.
// Bound by vector instructions, most of them tanh's, and by the inputs' loads.
constexpr int kRowUnits = 32, kRowStride = 65, kRowInputs = 32;
// Waves with units of their own, or four where the inputs take several loads
// (262144 rows of 256 inputs and 4 units: 101 us with one wave, 69 with four;
// 1048576 rows of 8 inputs and one unit: 19, 32).
int mlp_row_waves(int D, int H) { return D > kRowInputs ? 4 : std::min(4, (H + 3) / 4); }
__global__ __launch_bounds__(256) void mlp_rows_kernel(const float *__restrict__ params, int D, int H,
                                                      const float *__restrict__ X, int64_t n,
                                                      float *__restrict__ pred) {
  extern __shared__ __align__(16) float sm[];
  float *h1 = sm, *h2 = h1 + H * kRowStride;  // [H][kRowStride]
  float *xs = h2 + H * kRowStride;            // [min(D, kRowInputs)][kRowStride]
  const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), step = nth / 16;  // four units per wave
  const int64_t base = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * 64;
  if (base >= n) return;  // padding of the grid
  const int rows = (int)min((int64_t)64, n - base);
  const float *Xb = X + base * D;
  // Units' sums over ni inputs, four units at a time: from(unit) to put(unit, sum).
  auto layer = [&](const float *__restrict__ w, int ws, int ni, const float *in, auto from, auto put) {
    for (int j = 4 * wave; j < H; j += step) {
      float a[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = from(min(j + q, H - 1));
      const float *w0 = w + j * ws;
      const int s1 = j + 1 < H ? ws : 0, s2 = j + 2 < H ? 2 * ws : 0, s3 = j + 3 < H ? 3 * ws : 0;
#pragma unroll 4
      for (int i = 0; i < ni; ++i) {
        const float x = in[i * kRowStride + lane];
        a[0] = fmaf(w0[i], x, a[0]);
        a[1] = fmaf(w0[i + s1], x, a[1]);
        a[2] = fmaf(w0[i + s2], x, a[2]);
        a[3] = fmaf(w0[i + s3], x, a[3]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (j + q < H) put(j + q, a[q]);
    }
  };
  const float *pb1 = params + H * D, *pW2 = pb1 + H, *pb2 = pW2 + H * H, *pW3 = pb2 + H;
  for (int d0 = 0; d0 < D; d0 += kRowInputs) {
    const int nd = min(kRowInputs, D - d0);
    __syncthreads();  // the last inputs' readers are done
    if (nd == kRowInputs) {
      constexpr int G = 8;  // loads in flight
      for (int i0 = tid; i0 < 64 * kRowInputs; i0 += nth * G) {
        float v[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const int i = i0 + nth * g;
          v[g] = Xb[(int64_t)min(i / kRowInputs, rows - 1) * D + d0 + i % kRowInputs];
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const int i = i0 + nth * g;
          xs[i % kRowInputs * kRowStride + i / kRowInputs] = v[g];
        }
      }
    } else {
      for (int i = tid; i < rows * nd; i += nth) {
        const int s = i / nd, d = i - s * nd;
        xs[d * kRowStride + s] = Xb[s * D + d0 + d];
      }
    }
    __syncthreads();
    const bool last = d0 + nd == D;
    layer(params + d0, D, nd, xs, [&](int j) { return d0 == 0 ? pb1[j] : h1[j * kRowStride + lane]; },
          [&](int j, float a) { h1[j * kRowStride + lane] = last ? tanhf(a) : a; });
  }
  __syncthreads();
  layer(pW2, H, H, h1, [&](int j) { return pb2[j]; }, [&](int j, float a) { h2[j * kRowStride + lane] = tanhf(a); });
  __syncthreads();
  if (tid >= rows) return;
  float o = pW3[H];
#pragma unroll 8
  for (int j = 0; j < H; ++j) o = fmaf(pW3[j], h2[j * kRowStride + tid], o);
  pred[base + tid] = o;
}
static_assert(4 * kRowStride * (2 * kRowUnits + kRowInputs) <= 65536, "LDS without an attribute");

// mode 0: grad[p] = sum; mode 1: Adam.  scalar[0] = summed loss * loss_scale and
// scalar[1] += summed loss * epoch_scale (the epoch's mean loss, batch by batch).
// A block takes 64 parameters; its eight waves each sum a run of the partials,
// and the runs' sums are added in order.  (One thread per parameter over 64
// partials: 17 us per step, latency; 5 us now, over 256.)
__global__ __launch_bounds__(512) void mlp_reduce_kernel(const double *__restrict__ partial, int64_t blocks,
                                                         int64_t P, int mode, float *__restrict__ grad,
                                                         float *__restrict__ params, float *__restrict__ m,
                                                         float *__restrict__ v, float lr, float c1, float c2,
                                                         double loss_scale, double epoch_scale,
                                                         double *__restrict__ scalar) {
  __shared__ double run[8][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t p = (int64_t)blockIdx.x * 64 + lane;
  const int64_t per = (blocks + 7) / 8, q0 = min(blocks, wave * per), q1 = min(blocks, q0 + per);
  double t = 0.0;
  if (p <= P) {
#pragma unroll 16
    for (int64_t b = q0; b < q1; ++b) t += partial[b * (P + 1) + p];
  }
  run[wave][lane] = t;
  __syncthreads();
  if (wave != 0 || p > P) return;
  double g = 0.0;
#pragma unroll
  for (int w = 0; w < 8; ++w) g += run[w][lane];
  if (p == P) {
    scalar[0] = g * loss_scale;
    scalar[1] += g * epoch_scale;
    return;
  }
  if (mode == 0) {
    grad[p] = (float)g;
    return;
  }
  const float gf = (float)g;
  const float mm = 0.9f * m[p] + 0.1f * gf;
  const float vv = 0.999f * v[p] + 0.001f * gf * gf;
  m[p] = mm;
  v[p] = vv;
  params[p] -= lr * (mm * c1) / (sqrtf(vv * c2) + 1e-8f);
}

uint64_t splitmix(uint64_t &state) {
  uint64_t z = (state += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

int ensure_partial(tn_mlp *net, int64_t blocks) {
  if (blocks <= net->partial_blocks) return TN_OK;
  if (net->d_partial) (void)hipFree(net->d_partial);
  net->d_partial = nullptr;
  net->partial_blocks = 0;
  hipError_t e = hipMalloc((void **)&net->d_partial, (size_t)blocks * (size_t)(net->P + 1) * 8);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return set_error(TN_ERR_OOM, "mlp: hipMalloc of the gradient partials");
  }
  net->partial_blocks = blocks;
  return TN_OK;
}

// Blocks in x and y: the runtime refuses 2^32 threads in x (2^29 rows).
constexpr int64_t kGridX = (int64_t)1 << 21;
static_assert(kGridX * 512 <= 0xffffffffll, "threads in x");
dim3 mlp_grid(int64_t blocks) {
  const int64_t gx = std::min(blocks, kGridX);
  return dim3((unsigned)gx, (unsigned)((blocks + gx - 1) / gx));
}
size_t mlp_rows_lds(int D, int H) { return 4 * (size_t)kRowStride * (size_t)(std::min(D, kRowInputs) + 2 * H); }
// Whether predictions take a lane per row: with two tiles of 16 rows or more to
// a CU.  By tiles / by rows: 1048576 rows of 8 inputs and 16 units 659 / 56 us,
// of 8 and 32 816 / 108; 16384 rows of 100 and 4 23.6 / 9.6; 8192 rows of 256
// and 16 22.0 / 18.3, 4096 of them 11.7 / 18.3.
bool mlp_by_rows(int H, int64_t rows) { return H <= kRowUnits && rows >= 8192; }

// Tiles of 16 rows per block, and blocks, for a batch of `rows` rows.
int mlp_tiles(int64_t rows) { return rows > kManyTiles * kTile ? 4 : 1; }
int64_t mlp_blocks(int64_t rows) {
  const int64_t per = (int64_t)kTile * mlp_tiles(rows);
  return (rows + per - 1) / per;
}

int fwd_bwd(tn_mlp *net, const float *X, const float *y, int64_t row0, int64_t rows, int64_t n,
            hipStream_t st, float *pred, bool grad) {
  const int64_t blocks = mlp_blocks(rows);
  if (blocks == 0) return TN_OK;
  if (blocks > 0x7fffffff) return set_error(TN_ERR_UNSUPPORTED, "mlp: too many rows");
  if (grad) {
    int rc = ensure_partial(net, blocks);
    if (rc != TN_OK) return rc;
  }
  if (!grad && mlp_by_rows(net->H, rows)) {
    hipLaunchKernelGGL(mlp_rows_kernel, mlp_grid((rows + 63) / 64), dim3(64 * mlp_row_waves(net->D, net->H)),
                       mlp_rows_lds(net->D, net->H), st, net->d_params, net->D, net->H, X + row0 * net->D, rows,
                       pred + row0);
    TN_HIP_CHECK(hipGetLastError());
    return TN_OK;
  }
  hipLaunchKernelGGL(mlp_fwd_bwd_kernel, mlp_grid(blocks), dim3(512), net->lds, st,
                     net->d_params, net->D, net->H, X, y, row0, row0 + rows < n ? row0 + rows : n,
                     (float)(1.0 / (double)rows), pred, grad ? net->d_partial : nullptr, net->P, mlp_tiles(rows));
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

int reduce(tn_mlp *net, int64_t rows, int mode, float *grad, float lr, hipStream_t st,
           double epoch_scale = 0.0) {
  const int64_t blocks = mlp_blocks(rows);
  float c1 = 1.f, c2 = 1.f;
  if (mode == 1) {
    net->t += 1;
    c1 = (float)(1.0 / (1.0 - std::pow(0.9, (double)net->t)));
    c2 = (float)(1.0 / (1.0 - std::pow(0.999, (double)net->t)));
  }
  const unsigned g = (unsigned)((net->P + 1 + 63) / 64);
  hipLaunchKernelGGL(mlp_reduce_kernel, dim3(g), dim3(512), 0, st, net->d_partial, blocks, net->P,
                     mode, grad, net->d_params, net->d_m, net->d_v, lr, c1, c2,
                     1.0 / (double)rows, epoch_scale, net->d_scalar);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

}  // namespace
}  // namespace tn

using namespace tn;

extern "C" {

int tn_mlp_create(int32_t d_in, int32_t hidden, uint64_t seed, tn_mlp **out) {
  clear_error();
  if (!out) return set_error(TN_ERR_ARG, "out is null");
  *out = nullptr;
  if (d_in < 1 || d_in > 256 || hidden < 1 || hidden > 128)
    return set_error(TN_ERR_ARG, "mlp: d_in %d or hidden %d out of range", d_in, hidden);
  tn_mlp *net = new (std::nothrow) tn_mlp();
  if (!net) return set_error(TN_ERR_OOM, "host allocation");
  net->D = d_in;
  net->H = hidden;
  net->P = (int64_t)hidden * d_in + hidden + (int64_t)hidden * hidden + hidden + hidden + 1;
  // The documented limit on d_in and hidden: parameters and 64 rows of
  // activations in LDS (more than the kernel takes).
  const int64_t floats = net->P + 2 + (int64_t)kRows * d_in + 4 * (int64_t)kRows * hidden + kRows;
  net->lds = mlp_lds_bytes(d_in, hidden);
  int dev = 0, maxlds = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&maxlds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) {
    delete net;
    return set_error(TN_ERR_HIP, "mlp: no device");
  }
  net->device = dev;
  if ((size_t)floats * 4 + 1024 > (size_t)maxlds) {
    delete net;
    return set_error(TN_ERR_UNSUPPORTED, "mlp: %zu bytes of LDS needed", (size_t)floats * 4);
  }
  if (net->lds > 65536 &&
      hipFuncSetAttribute((const void *)mlp_fwd_bwd_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)net->lds) != hipSuccess) {
    delete net;
    return set_error(TN_ERR_HIP, "mlp: LDS attribute");
  }
  std::vector<float> h((size_t)net->P, 0.f);
  uint64_t state = seed;
  auto fill = [&](int64_t off, int fan_out, int fan_in) {
    const double a = std::sqrt(6.0 / (double)(fan_in + fan_out));
    for (int64_t i = 0; i < (int64_t)fan_out * fan_in; ++i) {
      const double u = (double)(splitmix(state) >> 11) * (1.0 / 9007199254740992.0);
      h[(size_t)(off + i)] = (float)((2.0 * u - 1.0) * a);
    }
  };
  const int64_t o1 = 0, o2 = (int64_t)hidden * d_in + hidden, o3 = o2 + (int64_t)hidden * hidden + hidden;
  fill(o1, hidden, d_in);
  fill(o2, hidden, hidden);
  fill(o3, 1, hidden);
  bool ok = hipMalloc((void **)&net->d_params, (size_t)net->P * 4) == hipSuccess &&
            hipMalloc((void **)&net->d_m, (size_t)net->P * 4) == hipSuccess &&
            hipMalloc((void **)&net->d_v, (size_t)net->P * 4) == hipSuccess &&
            hipMalloc((void **)&net->d_scalar, 16) == hipSuccess;
  if (!ok) {
    (void)hipGetLastError();
    tn_mlp_destroy(net);
    return set_error(TN_ERR_OOM, "mlp: hipMalloc");
  }
  if (hipMemcpy(net->d_params, h.data(), (size_t)net->P * 4, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemset(net->d_m, 0, (size_t)net->P * 4) != hipSuccess ||
      hipMemset(net->d_v, 0, (size_t)net->P * 4) != hipSuccess ||
      hipMemset(net->d_scalar, 0, 16) != hipSuccess) {
    tn_mlp_destroy(net);
    return set_error(TN_ERR_HIP, "mlp: initial upload");
  }
  *out = net;
  return TN_OK;
}

int64_t tn_mlp_num_params(const tn_mlp *net) {
  if (!net) return set_error(TN_ERR_ARG, "null net");
  return net->P;
}

int tn_mlp_shape(const tn_mlp *net, int32_t *d_in, int32_t *hidden) {
  clear_error();
  if (!net || !d_in || !hidden) return set_error(TN_ERR_ARG, "null argument");
  *d_in = net->D;
  *hidden = net->H;
  return TN_OK;
}

int tn_mlp_get_params(const tn_mlp *net, float *host_out) {
  clear_error();
  if (!net || !host_out) return set_error(TN_ERR_ARG, "null argument");
  TN_HIP_CHECK(hipDeviceSynchronize());
  TN_HIP_CHECK(hipMemcpy(host_out, net->d_params, (size_t)net->P * 4, hipMemcpyDeviceToHost));
  return TN_OK;
}

int tn_mlp_set_params(tn_mlp *net, const float *host_in) {
  clear_error();
  if (!net || !host_in) return set_error(TN_ERR_ARG, "null argument");
  TN_HIP_CHECK(hipDeviceSynchronize());
  TN_HIP_CHECK(hipMemcpy(net->d_params, host_in, (size_t)net->P * 4, hipMemcpyHostToDevice));
  TN_HIP_CHECK(hipMemset(net->d_m, 0, (size_t)net->P * 4));
  TN_HIP_CHECK(hipMemset(net->d_v, 0, (size_t)net->P * 4));
  TN_HIP_CHECK(hipDeviceSynchronize());
  net->t = 0;
  return TN_OK;
}

int tn_mlp_predict(tn_mlp *net, const float *X, int64_t n, void *stream, float *out) {
  clear_error();
  if (!net || n < 0) return set_error(TN_ERR_ARG, "bad argument");
  if (n == 0) return TN_OK;
  if (!X || !out) return set_error(TN_ERR_ARG, "null X or out");
  return fwd_bwd(net, X, nullptr, 0, n, n, (hipStream_t)stream, out, false);
}

int tn_mlp_grad(tn_mlp *net, const float *X, const float *y, int64_t n, void *stream, float *grad,
                double *loss) {
  clear_error();
  if (!net || !X || !y || !grad || n < 1) return set_error(TN_ERR_ARG, "bad argument");
  hipStream_t st = (hipStream_t)stream;
  int rc = fwd_bwd(net, X, y, 0, n, n, st, nullptr, true);
  if (rc == TN_OK) rc = reduce(net, n, 0, grad, 0.f, st);
  if (rc == TN_OK && loss) {
    TN_HIP_CHECK(hipMemcpyAsync(loss, net->d_scalar, 8, hipMemcpyDeviceToHost, st));
    TN_HIP_CHECK(hipStreamSynchronize(st));
  }
  return rc;
}

int tn_mlp_step(tn_mlp *net, const float *X, const float *y, int64_t n, float lr, void *stream) {
  clear_error();
  if (!net || !X || !y || n < 1) return set_error(TN_ERR_ARG, "bad argument");
  hipStream_t st = (hipStream_t)stream;
  int rc = fwd_bwd(net, X, y, 0, n, n, st, nullptr, true);
  if (rc == TN_OK) rc = reduce(net, n, 1, nullptr, lr, st);
  return rc;
}

int tn_mlp_train(tn_mlp *net, const float *X, const float *y, int64_t n, int32_t batch,
                 int32_t epochs, float lr, void *stream, double *losses) {
  clear_error();
  if (!net || !X || !y || n < 1 || batch < 1 || epochs < 0) return set_error(TN_ERR_ARG, "bad argument");
  hipStream_t st = (hipStream_t)stream;
  for (int ep = 0; ep < epochs; ++ep) {
    if (losses) TN_HIP_CHECK(hipMemsetAsync(net->d_scalar + 1, 0, 8, st));
    for (int64_t r0 = 0; r0 < n; r0 += batch) {
      const int64_t rows = std::min<int64_t>(batch, n - r0);
      int rc = fwd_bwd(net, X, y, r0, rows, n, st, nullptr, true);
      if (rc == TN_OK) rc = reduce(net, rows, 1, nullptr, lr, st, 1.0 / (double)n);
      if (rc != TN_OK) return rc;
    }
    if (losses) {
      TN_HIP_CHECK(hipMemcpyAsync(&losses[ep], net->d_scalar + 1, 8, hipMemcpyDeviceToHost, st));
      TN_HIP_CHECK(hipStreamSynchronize(st));
    }
  }
  return TN_OK;
}

void tn_mlp_destroy(tn_mlp *net) {
  if (!net) return;
  (void)hipDeviceSynchronize();
  if (net->d_params) (void)hipFree(net->d_params);
  if (net->d_m) (void)hipFree(net->d_m);
  if (net->d_v) (void)hipFree(net->d_v);
  if (net->d_partial) (void)hipFree(net->d_partial);
  if (net->d_scalar) (void)hipFree(net->d_scalar);
  delete net;
}

}  // extern "C"
