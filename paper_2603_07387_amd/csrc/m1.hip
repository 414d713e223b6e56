// Cyclic-network estimator (Eq. (1), Algorithm 1) on gfx950.
//
// Per sample r and tensor k the time-domain tensor sketch is
//     y_{k,r}[(sum_u h_u(i_u)) mod m] += (prod_u s_u(i_u)) X_k(i)
// (Def. 12 in the column form of Algorithm 3; the second mode of every
// contraction uses the complement bucket (m - h) mod m, Def. 14).  The
// estimate is e_1^T F^{-1}(F y_1 o ... o F y_p) = (1/m) sum_j prod_k Y_k[j].
//
// Kernels:
//   m1_scatter  : one block takes one slot (a run of rows of one tensor), whose
//                 entries it reads once for the largest and once per batch of
//                 samples, and accumulates the sketches of SB samples at a time in
//                 LDS in 64-bit fixed point; a wave per sample for small slots.
//   m1_big_scatter: m >= 2^15, FP32 sketches: scatter and the combine's first
//                 transforms in one, a pair of tensors' sketches by ranges.
//   m1_combine  : one block per (network, sample): two real sketches share one
//                 complex FFT in LDS (z = y_a + i y_b), the pair's product
//                 spectrum Y_a Y_b = (Z[j]^2 - conj(Z[-j])^2) / 4i is folded into
//                 per-thread FP64 accumulators over the half spectrum, and the
//                 Hermitian sum (1/m)(P_0 + P_{m/2} + 2 Re sum_{0<j<m/2} P_j)
//                 gives the estimate.
//   sample_stats: FP64 mean and unbiased variance over samples per network.
#include <algorithm>

#include "block_map.h"
#include "m1_device.h"

#include <hip/hip_bf16.h>

namespace tn {
namespace {

using namespace m1dev;


// Four consecutive entries of a row, loaded with one or two vector loads from
// any element-aligned address.
typedef float f32x4e __attribute__((ext_vector_type(4), aligned(4)));
typedef double f64x4e __attribute__((ext_vector_type(4), aligned(8)));
typedef unsigned short u16x4e __attribute__((ext_vector_type(4), aligned(2)));
template <typename T>
struct Quad;
template <>
struct Quad<float> {
  using type = f32x4e;
};
template <>
struct Quad<double> {
  using type = f64x4e;
};
template <>
struct Quad<uint16_t> {
  using type = u16x4e;
};

// x with its sign flipped when bit (kSignBit or 0) is set.
__device__ __forceinline__ float flip_sign(float x, uint32_t bit) { return __uint_as_float(__float_as_uint(x) ^ bit); }
__device__ __forceinline__ double flip_sign(double x, uint32_t bit) {
  return __hiloint2double((int)((uint32_t)__double2hiint(x) ^ bit), __double2loint(x));
}

// The packed row words of SB samples (one 16-byte LDS read per four).
template <int SB>
__device__ __forceinline__ void load_row(const uint32_t *p, uint32_t *out) {
  if constexpr (SB == 1)
    out[0] = p[0];
  else
    load_cols<SB>(p, out);
}

// One block streams one slot and accumulates the sketches of SB samples at a
// time in LDS in 64-bit fixed point, then writes them out as floating point,
// for the sample batches [grp gs, grp gs + gs) of the launch.
//
// Columns stay with their threads: thread t takes the four columns 4 (t mod V)
// .. + 3 (V = ceil(L / 4) vectors per row; the last vector of a row of other
// length starts at L - 4 and its columns already covered are scaled by 0) of
// the rows t / V + k (NT / V).  Its SB x 4 column words are held in registers
// for a batch, no term divides or tests a row end, and a vector reads only its
// row's SB words from LDS (rowt, one 16-byte broadcast read for four samples),
// row_chunk(SB) rows at a time.
// A term is then one add, one and-or and the LDS atomic with BANKS = 2:
// sketches are pairs of banks of m words, +1 terms in the positive bank, -1
// terms in the negative one, the sketch their difference.  Sample s's positive
// bank is at byte 8 m s, its negative bank signbit further (a power of two of
// at least 16 m); the words hold bucket * 8 plus signbit for sign -1, so the
// sum of a row and a column word carries the product of the signs in the
// signbit position (the bucket sum stays below 16 m).  With BANKS = 1 (half the
// LDS) the signs are in bit 31 and the product flips the sign of the entry
// before its conversion.
// What bounds it: random 64-bit LDS atomics.  16 lanes at a time fall into the
// 32 pairs of LDS banks, 2.35 deep on average: 9.4 cycles per wave instruction,
// 5.5 of them conflicts (LDS counters), against three vector instructions
// at four samples and two banks.
//
// The hash words of a batch (all modes of the slot's tensor, complement
// applied, [word][sample]) are staged in LDS for tensors of at most four modes
// of together at most kStageWords indices; the next batch's are loaded during
// the current one.  Other tensors read the global tables.  Everything else a
// block needs is set up once for all of its batches: measured on the batch of
// 4096 networks, a block's start (its chain of dependent loads) takes 8 to 9
// us, as long as the scatter itself when each block takes one batch.
//
// The fixed-point scale is 62 - lgN - e for |x| < 2^e and N <= 2^lgN terms, so
// sums cannot overflow and do not depend on the order of the atomics.  bound_in:
// per slot the power of two 2^(e - 1) (0 for an all-zero slot) recorded before;
// without it the block first takes the maximum over its slot (read again by
// the scatter, from the caches); the first group's blocks record it in
// bound_out.
//
// RANGED (m above 2^kMaxLog2Acc buckets, one bank, one sample): the block takes
// the ranges of 2^kMaxLog2Acc buckets one after the other and drops the terms
// outside the current one; `rsplit` blocks share a group's ranges where the
// groups are few.
//
// slots: in decreasing order of size (id: the slot's number), so that the last
// blocks to start are short; their blocks as slot_block gives them.
// Registers: six waves per SIMD (three blocks per CU) for 512-thread blocks with
// one bank, whose LDS leaves room for them at m = 1024 (batch of 4096 networks:
// 2.64 against 2.75 ms per call with four, and with four row vectors in flight
// instead of two), four otherwise.
template <typename T, typename A, int SB, int BANKS, int NT, bool RANGED = false>
__global__ __launch_bounds__(NT, BANKS == 1 && NT == 512 && SB * sizeof(A) <= 16 ? 6 : 4) void m1_scatter_kernel(
    const ScatterSlot *__restrict__ slots, int32_t n, const ModeDesc *__restrict__ modes,
    const void *const *__restrict__ data, const int32_t *__restrict__ tables, int64_t W, int64_t samples,
    int log2m, int64_t n_slots, A *__restrict__ ybuf, const double *__restrict__ bound_in,
    double *__restrict__ bound_out, int32_t gs, int32_t groups, int32_t gx, int32_t rsplit) {
  constexpr int kRows = row_chunk(SB);  // rows whose words are in the LDS at a time
  static_assert(!RANGED || (BANKS == 1 && SB == 1), "bucket ranges use one bank and one sample");
  using Q = typename Quad<T>::type;
  constexpr int U = BANKS == 1 || SB * sizeof(T) >= 32 ? 2 : 4;  // row vectors in flight per thread
  static_assert(kStageWords <= NT, "one staged word per thread");
  // No static LDS: the accumulators start at LDS address 0.
  extern __shared__ __align__(16) unsigned char smem[];
  const SlotBlock sb = slot_block(blockIdx.x, (uint32_t)n, (uint32_t)gx);
  const int32_t pos = (int32_t)sb.slot, run = (int32_t)sb.group + (int32_t)blockIdx.y * gx;
  const int32_t grp = RANGED ? run / rsplit : run;
  if (pos >= n || grp >= groups) return;  // padding of the grid
  const ScatterSlot sl = slots[pos];
  const int32_t sid = sl.id;
  const int tid = threadIdx.x;
  const uint32_t m = 1u << log2m, mask = m - 1;
  constexpr int log2acc = kMaxLog2Acc;
  const uint32_t ma = RANGED ? 1u << log2acc : m;  // accumulator words per sample
  const uint32_t signbit = BANKS == 2 ? sign_bank_offset(SB, m) : kSignBit;
  const uint32_t acc_bytes = BANKS == 2 ? (uint32_t)sign_bank_bytes(SB, m) : (uint32_t)SB * 8u * ma;
  const uint32_t acc_end = (acc_bytes + 15u) & ~15u;
  unsigned long long *acc = reinterpret_cast<unsigned long long *>(smem);
  uint32_t *rowt = reinterpret_cast<uint32_t *>(smem + acc_end);  // [kRows][SB]
  uint32_t *stage = rowt + kRows * SB;                        // [kStageWords][SB]
  unsigned long long *s_max = reinterpret_cast<unsigned long long *>(stage + kStageWords * SB);
  const int L = sl.L, rows = sl.rows;
  const T __attribute__((address_space(1))) *X =
      (const T __attribute__((address_space(1))) *)(reinterpret_cast<const T *>(data[sl.tensor]) +
                                                    sl.row0 * (int64_t)L);

  // The thread's columns and first row; threads past the last whole row of
  // vectors have no work in the loop.
  const int V = (L + 3) >> 2, RP = NT / V;  // L <= 1024 <= 4 NT
  const int rt = tid / V, v = tid - rt * V;
  const bool active = rt < RP;
  const int c0 = max(0, min(4 * v, L - 4));
  auto load = [&](int r) {
    const int off = min(r, rows - 1) * L + c0;
    if (L >= 4) return *(const Q __attribute__((address_space(1))) *)(X + off);
    Q q = {};
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (i < L) q[i] = X[off + i];
    return q;
  };
  Q nxt[U];
#pragma unroll
  for (int u = 0; u < U; ++u) nxt[u] = load(rt + u * RP);

  // The tensor's modes, first ones first; the staged words of mode j start at
  // word mo[j] (mode sizes past the last are 0).
  const int q = sl.q, split = sl.split, mode0 = sl.mode0;
  int mn[4], mo[4], tot = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    mn[j] = j < q ? modes[mode0 + j].n : 0;
    mo[j] = tot;
    tot += mn[j];
  }
  const bool staged = q <= 4 && tot <= kStageWords;  // uniform
  // This thread's staged word: its table offset and complement flag.
  int64_t w_off = 0;
  bool w_comp = false;
  if (staged && tid < tot) {
    const int j = tid >= mo[3] && mn[3] > 0 ? 3 : tid >= mo[2] && mn[2] > 0 ? 2 : tid >= mo[1] && mn[1] > 0 ? 1 : 0;
    const ModeDesc md = modes[mode0 + j];
    const int base = j == 0 ? 0 : j == 1 ? mo[1] : j == 2 ? mo[2] : mo[3];
    w_off = md.table_off + (tid - base);
    w_comp = md.comp != 0;
  }
  const int32_t batch_end = min((grp + 1) * gs, (int32_t)((samples + SB - 1) / SB));
  uint32_t pre[SB];  // the next batch's staged words
  auto fetch = [&](int32_t b) {
    if (staged && tid < tot && b < batch_end) {
#pragma unroll
      for (int s = 0; s < SB; ++s)
        pre[s] = (uint32_t)tables[min((int64_t)b * SB + s, samples - 1) * W + w_off];
    }
  };
  auto put = [&](int32_t b) {
    if (staged && tid < tot && b < batch_end) {
#pragma unroll
      for (int s = 0; s < SB; ++s) {
        uint32_t h = pre[s] & ~kSignBit;
        if (w_comp) h = (m - h) & mask;
        stage[tid * SB + s] = (h << 3) | (pre[s] & kSignBit);
      }
    }
  };
  fetch(grp * gs);

  // Largest |x| of the slot, when it was not recorded before.
  double bound;
  if (bound_in != nullptr) {
    bound = bound_in[sid];
  } else {
    const uint32_t N = (uint32_t)rows * (uint32_t)L;
    double lmax = 0.0;
    if (tid == 0) s_max[0] = 0ull;
    if (RP * U >= rows) {  // all of it is in nxt
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) lmax = fmax(lmax, fabs((double)to_acc_any((T)nxt[u][i])));
    } else {
      const Q __attribute__((address_space(1))) *Xq = (const Q __attribute__((address_space(1))) *)X;
      const uint32_t NQ = N / 4;
      for (uint32_t i0 = tid; i0 < NQ; i0 += NT * U) {
        Q t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) t[u] = Xq[min(i0 + (uint32_t)u * NT, NQ - 1)];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) lmax = fmax(lmax, fabs((double)to_acc_any((T)t[u][i])));
      }
      if (4 * NQ + tid < N) lmax = fmax(lmax, fabs((double)to_acc_any((T)X[4 * NQ + tid])));
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) lmax = fmax(lmax, __shfl_xor(lmax, off, 64));
    __syncthreads();
    if ((tid & 63) == 0) atomicMax(s_max, (unsigned long long)__double_as_longlong(lmax));
    __syncthreads();
    const double bm = __longlong_as_double((long long)s_max[0]);
    int e = 0;
    (void)frexp(bm, &e);  // 2^(e - 1) <= bm < 2^e
    bound = bm > 0.0 ? ldexp(1.0, e - 1) : 0.0;
    if (bound_out != nullptr && tid == 0 && grp == 0) bound_out[sid] = bound;
  }
  int scale = 0;
  if (bound > 0.0) {
    const uint32_t N = (uint32_t)rows * (uint32_t)L;
    int e;
    (void)frexp(bound, &e);  // bound = 2^(e - 1)
    scale = 62 - max(N > 1 ? 32 - __clz(N - 1) : 0, 11) - e;
  }
  const double sc = ldexp(1.0, scale);
  double scq[4];  // 0 for columns past the row or covered by the vector before
#pragma unroll
  for (int i = 0; i < 4; ++i) scq[i] = (c0 + i >= 4 * v && i < L) ? sc : 0.0;

  // Byte address of a term: ((row word + column word) & amask) | soff[s], one
  // and-or instruction.  The values pass through empty asm statements so that
  // the mask is held in a vector register (the instruction takes one scalar
  // operand) and the LDS base, 0 here (the block has no static LDS), is not
  // added again for every term.
  uint32_t amask = (mask << 3) | (BANKS == 2 ? signbit : 0u);
  asm("" : "+v"(amask));
  uint32_t soff[SB];
#pragma unroll
  for (int s = 0; s < SB; ++s) {
    soff[s] = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char *)smem) +
              (uint32_t)s * 8u * ma;
    asm("" : "+s"(soff[s]));
  }
  auto add = [](uint32_t byte, long long t) {
    __hip_atomic_fetch_add((__attribute__((address_space(3))) unsigned long long *)byte, (unsigned long long)t,
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // A sum of words (bucket * 8, sign in bit 31) as the address part of a term.
  auto to_offset = [&](uint32_t w) {
    return (w & (mask << 3)) | ((uint32_t)((int32_t)w >> 31) & signbit);
  };
  constexpr double kMagic = 6755399441055744.0;  // 1.5 2^52: x sc + kMagic holds round(x sc) in its low bits
  const long long kMagicBits = __double_as_longlong(kMagic);
  // idx / n for idx < 2^21: (idx + 1/2) / n is at least 1 / 2n from an integer
  auto divide = [](uint32_t idx, float rn) { return (uint32_t)(((float)idx + 0.5f) * rn); };
  const float rn[4] = {1.0f / (float)max(mn[0], 1), 1.0f / (float)max(mn[1], 1), 1.0f / (float)max(mn[2], 1),
                       1.0f / (float)max(mn[3], 1)};
  // Sum over the modes [j0, j1) of the words of index idx, for the SB samples
  // of the batch starting at s0.
  auto words = [&](uint32_t idx, int j0, int j1, int64_t s0, uint32_t *w) {
#pragma unroll
    for (int s = 0; s < SB; ++s) w[s] = 0;
    if (staged) {
#pragma unroll
      for (int j = 3; j >= 0; --j) {
        if (j < j0 || j >= j1) continue;
        const uint32_t qt = j > j0 ? divide(idx, rn[j]) : 0u;
        uint32_t t[SB];
        load_row<SB>(stage + (mo[j] + (int)(idx - qt * (uint32_t)mn[j])) * SB, t);
        idx = qt;
#pragma unroll
        for (int s = 0; s < SB; ++s) w[s] += t[s];
      }
    } else {
      for (int j = j1 - 1; j >= j0; --j) {
        const ModeDesc md = modes[mode0 + j];
        const uint32_t qt = j > j0 ? idx / (uint32_t)md.n : 0u;
        const uint32_t d = idx - qt * (uint32_t)md.n;
        idx = qt;
#pragma unroll
        for (int s = 0; s < SB; ++s) {
          const uint32_t t = (uint32_t)tables[min(s0 + s, samples - 1) * W + md.table_off + d];
          uint32_t h = t & ~kSignBit;
          if (md.comp) h = (m - h) & mask;
          // (the sum is reduced each time: the bucket part stays clear of bit 31 for any order)
          w[s] = ((w[s] + (h << 3)) & (mask << 3)) | ((w[s] ^ t) & kSignBit);
        }
      }
    }
  };

  // Few rows and columns: the column words too are formed once per block, after
  // the row words, instead of by every thread for its own columns (64 triangles
  // of 64 x 64, 256 samples, m = 256, FP64: 205 -> 188 us per call).
  const bool few = rows + L <= kFewWords;
  lds_zero(acc, acc_bytes, tid, NT);
  put(grp * gs);
  for (int32_t batch = grp * gs; batch < batch_end; ++batch) {
    const int64_t s0 = (int64_t)batch * SB;
    __syncthreads();  // the staged words are there, the accumulators cleared
    uint32_t lv[SB][4];
    if (!few) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t w[SB];
        words((uint32_t)min(c0 + i, L - 1), split, q, s0, w);
#pragma unroll
        for (int s = 0; s < SB; ++s) lv[s][i] = to_offset(w[s]);
      }
    }
    fetch(batch + 1);
    const int nranges = RANGED ? 1 << (log2m - log2acc) : 1, rstep = RANGED ? rsplit : 1;
    const int range0 = RANGED ? run - grp * rsplit : 0;
    for (int range = range0; range < nranges; range += rstep) {
      const uint32_t rlo = (uint32_t)range << (3 + log2acc), rlen = 8u << log2acc;
      for (int rb = 0; rb < rows; rb += kRows) {
        const int re = min(rows, rb + kRows);
        if (rb > 0) __syncthreads();  // the last chunk's readers are done
        if (range == range0 || rows > kRows) {
          // rows, then (few) columns
          for (int r = rb + tid; r < re + (few ? L : 0); r += NT) {
            uint32_t w[SB];
            const bool row = r < re;
            words(row ? (uint32_t)(sl.row0 + r) : (uint32_t)(r - re), row ? 0 : split, row ? split : q, s0, w);
#pragma unroll
            for (int s = 0; s < SB; ++s) rowt[(r - rb) * SB + s] = to_offset(w[s]);
          }
        }
        __syncthreads();
        if (few && range == range0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            uint32_t w[SB];
            load_row<SB>(rowt + (rows + min(c0 + i, L - 1)) * SB, w);
#pragma unroll
            for (int s = 0; s < SB; ++s) lv[s][i] = w[s];
          }
        }
        if (!active) continue;
        // The thread's rows of this chunk (rt + k RP across chunks, so that nxt
        // runs on).
        for (int r = rb + ((rt - rb) % RP + RP) % RP; r < re; r += U * RP) {
          Q cur[U];
#pragma unroll
          for (int u = 0; u < U; ++u) cur[u] = nxt[u];
          // the next round's rows, or the first ones of the next chunk, or of
          // the next range or batch
          int rn_ = r + U * RP;
          if (rn_ >= re) {
            if (re < rows) rn_ = re + ((rt - re) % RP + RP) % RP;
            if (rn_ >= rows) rn_ = rt;
          }
#pragma unroll
          for (int u = 0; u < U; ++u) nxt[u] = load(rn_ + u * RP);
          uint32_t hv[2][SB];
          load_row<SB>(rowt + (r - rb) * SB, hv[0]);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int ru = r + u * RP;
            if (u + 1 < U) load_row<SB>(rowt + (min(ru + RP, re - 1) - rb) * SB, hv[(u + 1) & 1]);
            if (ru < re) {
              const uint32_t *h = hv[u & 1];
              if constexpr (BANKS == 2) {
                long long t[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                  t[i] = __double_as_longlong(fma((double)to_acc_any((T)cur[u][i]), scq[i], kMagic)) - kMagicBits;
#pragma unroll
                for (int s = 0; s < SB; ++s)
#pragma unroll
                  for (int i = 0; i < 4; ++i) add(((h[s] + lv[s][i]) & amask) | soff[s], t[i]);
              } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                  for (int s = 0; s < SB; ++s) {
                    const uint32_t a = h[s] + lv[s][i];
                    const double x = (double)flip_sign(to_acc_any((T)cur[u][i]), a & kSignBit);
                    const long long t = __double_as_longlong(fma(x, scq[i], kMagic)) - kMagicBits;
                    if constexpr (RANGED) {
                      const uint32_t o = (a & amask) ^ rlo;
                      if (o < rlen) add(o + soff[0], t);
                    } else {
                      add((a & amask) | soff[s], t);
                    }
                  }
                }
              }
            }
          }
        }
      }
      __syncthreads();
      if (range + rstep >= nranges) put(batch + 1);
      // Sketches out, accumulators cleared: (positive bank minus negative bank)
      // 2^-scale, four buckets per thread and 16-byte accesses when a sketch
      // has at least four.
      const int lga = RANGED ? log2acc : log2m;
      const uint32_t r0 = (uint32_t)range << log2acc;  // first bucket of the range
      const int nsb = (int)min((int64_t)SB, samples - s0);
      auto value = [&](unsigned long long p, unsigned long long neg) {
        return (A)ldexp((double)(long long)(p - neg), -scale);
      };
      if (lga >= 2) {
        for (int i4 = tid; i4 < (SB << (lga - 2)); i4 += NT) {
          const int i = 4 * i4, s = i >> lga, b = i & ((1 << lga) - 1);
          ulonglong2 *ap = reinterpret_cast<ulonglong2 *>(acc + i);
          const ulonglong2 p0 = ap[0], p1 = ap[1];
          ap[0] = ap[1] = make_ulonglong2(0ull, 0ull);
          ulonglong2 n0 = make_ulonglong2(0ull, 0ull), n1 = n0;
          if constexpr (BANKS == 2) {
            ulonglong2 *an = reinterpret_cast<ulonglong2 *>(acc + i + signbit / 8);
            n0 = an[0];
            n1 = an[1];
            an[0] = an[1] = make_ulonglong2(0ull, 0ull);
          }
          if (s < nsb) {
            const A v0 = value(p0.x, n0.x), v1 = value(p0.y, n0.y), v2 = value(p1.x, n1.x), v3 = value(p1.y, n1.y);
            A *dst = ybuf + ((s0 + s) * n_slots + sid) * (int64_t)m + r0 + b;
            if constexpr (sizeof(A) == 4) {
              *reinterpret_cast<float4 *>(dst) = make_float4(v0, v1, v2, v3);
            } else {
              reinterpret_cast<double2 *>(dst)[0] = make_double2(v0, v1);
              reinterpret_cast<double2 *>(dst)[1] = make_double2(v2, v3);
            }
          }
        }
      } else {
        for (int i = tid; i < (SB << lga); i += NT) {
          const unsigned long long p = acc[i], neg = BANKS == 2 ? acc[i + signbit / 8] : 0ull;
          acc[i] = 0ull;
          if constexpr (BANKS == 2) acc[i + signbit / 8] = 0ull;
          if ((i >> lga) < nsb)
            ybuf[((s0 + (i >> lga)) * n_slots + sid) * (int64_t)m + (i & ((1 << lga) - 1))] = value(p, neg);
        }
      }
    }
  }
}

// Slots of at most kSmallSlot entries (and at most four modes of together at
// most kStageWords indices): a wave takes one sample at a time on its own, so
// nothing waits at a block barrier.  Its lanes hold the slot's entries and,
// packed, the positions of their modes' hash words, for all of the wave's
// samples; per sample they stage the words, add the entries to the wave's m
// accumulators and write the sketch out, clearing the accumulators for the
// next sample.  The same fixed point, bit for bit, as m1_scatter_kernel.
// What bounds it: writing the m-word sketches of tensors of far fewer entries.
template <typename T, typename A>
__global__ __launch_bounds__(256) void m1_scatter_small_kernel(
    const ScatterSlot *__restrict__ slots, int32_t n, const ModeDesc *__restrict__ modes,
    const void *const *__restrict__ data, const int32_t *__restrict__ tables, int64_t W, int64_t samples,
    int log2m, int64_t n_slots, A *__restrict__ ybuf, double *__restrict__ bound_out, int32_t gs, int32_t groups,
    int32_t gx) {
  constexpr int K = kSmallSlot / 64, KW = kStageWords / 64;
  static_assert(kStageWords <= 255 && kStageWords % 64 == 0, "word positions are packed in bytes");
  extern __shared__ __align__(16) unsigned char smem[];
  const SlotBlock sb = slot_block(blockIdx.x, (uint32_t)n, (uint32_t)gx);
  const int32_t pos = (int32_t)sb.slot, grp = (int32_t)sb.group + (int32_t)blockIdx.y * gx;
  if (pos >= n || grp >= groups) return;  // padding of the grid
  const ScatterSlot sl = slots[pos];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t m = 1u << log2m, mask = m - 1, abytes = max(8u * m, 16u);
  unsigned char *mine = smem + (size_t)wave * (abytes + kStageWords * 4);
  unsigned long long *acc = reinterpret_cast<unsigned long long *>(mine);
  uint32_t *stage = reinterpret_cast<uint32_t *>(mine + abytes);
  const int N = sl.rows * sl.L, q = sl.q;
  const T *X = reinterpret_cast<const T *>(data[sl.tensor]) + sl.row0 * (int64_t)sl.L;
  const int64_t s_end = min(samples, (int64_t)(grp + 1) * gs * 4);
  int64_t s = (int64_t)grp * gs * 4 + wave;

  using XA = decltype(to_acc_any(T{}));
  XA x[K];
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (64 * k < N) x[k] = lane + 64 * k < N ? to_acc_any(X[lane + 64 * k]) : (XA)0;
  int mn[4], mo[4], tot = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    mn[j] = j < q ? modes[sl.mode0 + j].n : 1;
    mo[j] = tot;
    tot += j < q ? mn[j] : 0;
  }
  // the lane's staged words: table offset and complement flag
  int64_t w_off[KW];
  bool w_comp[KW];
#pragma unroll
  for (int i = 0; i < KW; ++i) {
    const int w = lane + 64 * i;
    w_off[i] = 0;
    w_comp[i] = false;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < q && w >= mo[j] && w < tot) {
        const ModeDesc md = modes[sl.mode0 + j];
        w_off[i] = md.table_off + (w - mo[j]);
        w_comp[i] = md.comp != 0;
      }
  }
  uint32_t pre[KW];
  auto fetch = [&](int64_t t) {
#pragma unroll
    for (int i = 0; i < KW; ++i)
      if (64 * i < tot) pre[i] = lane + 64 * i < tot ? (uint32_t)tables[t * W + w_off[i]] : 0u;
  };
  if (s < s_end) fetch(s);
  // word positions of the lane's entries, 8 bits per mode
  uint32_t at[K];
  {
    const float rn[4] = {1.0f / (float)mn[0], 1.0f / (float)mn[1], 1.0f / (float)mn[2], 1.0f / (float)mn[3]};
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (64 * k < N) {
        uint32_t idx = (uint32_t)(sl.row0 * sl.L) + (uint32_t)min(lane + 64 * k, N - 1);
        at[k] = 0;
#pragma unroll
        for (int j = 3; j >= 0; --j)
          if (j < q) {
            const uint32_t qt = j > 0 ? (uint32_t)(((float)idx + 0.5f) * rn[j]) : 0u;  // idx < 2^21
            at[k] |= (uint32_t)(mo[j] + (int)(idx - qt * (uint32_t)mn[j])) << (8 * j);
            idx = qt;
          }
      }
  }
  double lmax = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (64 * k < N) lmax = fmax(lmax, fabs((double)x[k]));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) lmax = fmax(lmax, __shfl_xor(lmax, off, 64));
  int scale = 0;
  if (lmax > 0.0) {
    int e;
    (void)frexp(lmax, &e);  // max|x| < 2^e
    scale = 62 - 11 - e;    // N <= 2^11 (see m1_scatter_kernel)
  }
  if (bound_out != nullptr && grp == 0 && threadIdx.x == 0)
    bound_out[sl.id] = lmax > 0.0 ? ldexp(1.0, 50 - scale) : 0.0;  // 2^(e - 1)
  const double sc = ldexp(1.0, scale);
  constexpr double kMagic = 6755399441055744.0;
  const long long kMagicBits = __double_as_longlong(kMagic);
  for (uint32_t i = lane; i < abytes / 16; i += 64) reinterpret_cast<uint4 *>(acc)[i] = make_uint4(0u, 0u, 0u, 0u);
  // The wave's own LDS operations complete in order; the fences keep the
  // compiler from moving them across each other.
  auto fence = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  for (; s < s_end; s += 4) {
#pragma unroll
    for (int i = 0; i < KW; ++i)
      if (64 * i < tot) {
        uint32_t h = pre[i] & ~kSignBit;
        if (w_comp[i]) h = (m - h) & mask;
        stage[lane + 64 * i] = (h << 3) | (pre[i] & kSignBit);
      }
    if (s + 4 < s_end) fetch(s + 4);
    fence();
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (64 * k < N) {
        uint32_t a = stage[at[k] & 255u];
        if (q > 1) a += stage[(at[k] >> 8) & 255u];
        if (q > 2) a += stage[(at[k] >> 16) & 255u];
        if (q > 3) a += stage[at[k] >> 24];
        const long long t = __double_as_longlong(fma((double)flip_sign(x[k], a & kSignBit), sc, kMagic)) - kMagicBits;
        if (lane + 64 * k < N)
          __hip_atomic_fetch_add(reinterpret_cast<unsigned long long *>(mine + (a & (mask << 3))),
                                 (unsigned long long)t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
    fence();
    A *dst = ybuf + (s * n_slots + sl.id) * (int64_t)m;
    auto value = [&](unsigned long long t) { return (A)ldexp((double)(long long)t, -scale); };
    if (log2m >= 2) {
      for (uint32_t i4 = lane; i4 < m / 4; i4 += 64) {
        ulonglong2 *ap = reinterpret_cast<ulonglong2 *>(acc + 4 * i4);
        const ulonglong2 p0 = ap[0], p1 = ap[1];
        ap[0] = ap[1] = make_ulonglong2(0ull, 0ull);
        if constexpr (sizeof(A) == 4) {
          reinterpret_cast<float4 *>(dst)[i4] = make_float4(value(p0.x), value(p0.y), value(p1.x), value(p1.y));
        } else {
          reinterpret_cast<double2 *>(dst)[2 * i4] = make_double2(value(p0.x), value(p0.y));
          reinterpret_cast<double2 *>(dst)[2 * i4 + 1] = make_double2(value(p1.x), value(p1.y));
        }
      }
    } else if ((uint32_t)lane < m) {
      dst[lane] = value(acc[lane]);
      acc[lane] = 0ull;
    }
    fence();
  }
}

// (pr, pi) *= (qr, qi), its roundings written out: an estimate is the same
// whichever kernel takes the product.
__device__ __forceinline__ void times(double &pr, double &pi, double qr, double qi) {
  const double nr = fma(pr, qr, -(pi * qi));
  pi = fma(pi, qr, pr * qi);
  pr = nr;
}

// The first 256 threads add the terms j0 + t of all NTH threads t, those below
// H, in the order in which 256 threads would take them: the result does not
// depend on the block's size.
template <int NTH>
__device__ __forceinline__ void sum_as_256(double term, int64_t j0, int64_t H, double *terms, double &sum) {
  __syncthreads();  // earlier readers are done
  terms[threadIdx.x] = term;
  __syncthreads();
  if (threadIdx.x < 256) {
    for (int t = threadIdx.x; t < NTH; t += 256)
      if (j0 + t < H) sum += terms[t];
  }
}

// NTH threads: 256, or 1024 for m >= 8192 (a block then fills most of a
// CU's LDS, and the per-thread share of the half spectrum stays small) and
// where there are not more blocks than CUs.
// The transform is held padded in LDS (pad32).  TWL: the half table of
// twiddles is staged beside it (padded too); otherwise (no room for it) the
// two-level table (Tw2) is.
// Network j's tensors are the entries [nets[j].t0, nets[j].t1) of the slot
// ranges: entry k's sketch is the sum of the slots [tbeg[k], tend[k]) (a
// plan's tensors in order: tbeg = first slot of each tensor, tend = tbeg + 1;
// a partial plan lists each entry's, or each group entry's, sub-tensors).
// SCALED (group entries): every tensor is scaled by the power of two up to its
// largest entry (bound), pexp their exponents' sum, so that the product of a group's
// tensors, which are not neighbours in the network, neither overflows nor
// vanishes where the whole product does not.  Exact: the spectra's bits are those
// of the plain product, their exponents apart.
template <typename A, int LOG2M, bool TWL, int NTH, bool SCALED>
__global__ __launch_bounds__(NTH) void m1_combine_kernel(
    const NetDesc *__restrict__ nets, const int32_t *__restrict__ tbeg, const int32_t *__restrict__ tend,
    const A *__restrict__ ybuf, int64_t n_slots, int64_t sample0, int64_t S,
    const typename Cplx<A>::type *__restrict__ tw, double *__restrict__ est, double2 *__restrict__ part,
    const double *__restrict__ bound, int32_t *__restrict__ pexp) {
  using A2 = typename Cplx<A>::type;
  constexpr int M = 1 << LOG2M;
  constexpr int H = M / 2 + 1;
  constexpr int NC = (H + NTH - 1) / NTH;
  // sketch points per thread and load round: all of a round's loads are in
  // flight together
  constexpr int G = M >= 8 * NTH ? 8 : (M >= NTH ? M / NTH : 1);
  extern __shared__ __align__(16) unsigned char smem[];
  A2 *z = reinterpret_cast<A2 *>(smem);
  __shared__ double red[NTH / 64];

  const NetDesc nd = nets[blockIdx.x];
  const int64_t s = blockIdx.y;
  const A *y = ybuf + s * n_slots * (int64_t)M;
  const int tid = threadIdx.x;
  // Tensors [kb, ke): the network's, or with part (gridDim.z blocks per
  // network and sample) share blockIdx.z of its pairs, pairs taken from t0 on
  // (an empty share leaves the product at 1).
  int kb = nd.t0, ke = nd.t1;
  if (part != nullptr) {
    const int np = (nd.t1 - nd.t0 + 1) / 2, per = (np + (int)gridDim.z - 1) / (int)gridDim.z;
    kb = min(nd.t1, nd.t0 + 2 * per * (int)blockIdx.z);
    ke = min(nd.t1, kb + 2 * per);
  }
  // Twiddles: staged in LDS after z (every butterfly pass reads them; from the
  // global table each pass would wait on a cache round trip).  The first
  // barrier below publishes them.
  A2 *t = z + pad32(M);
  if constexpr (TWL) {
    for (int j = tid; j < M / 2; j += NTH) t[pad32(j)] = tw[j];
  } else {
    static_assert(M >= 128, "two-level twiddles");
    for (int j = tid; j < M / 128 + 64; j += NTH) t[j] = tw[j < M / 128 ? 64 * j : j - M / 128];
  }

  double pr[NC], pi[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) { pr[c] = 1.0; pi[c] = 0.0; }
  int esum = 0;
  // Largest power of two up to any entry of the slots [from, to).  (The first
  // load is not waited for where there is one slot.)
  auto largest = [&](int from, int to) {
    double b = bound[from];
    for (int sl = from + 1; sl < to; ++sl) b = fmax(b, bound[sl]);
    return b;
  };

  // With one load round per pair (M <= NTH G), the first slot of each tensor
  // of the next pair is loaded before this pair's transform: the loads stay
  // in flight through the transform's LDS passes and barriers.
  constexpr bool ONE_ROUND = M <= NTH * G;
  A f1[G], f2[G];
  auto first_slots = [&](int k) {
    const bool pk = (k + 1) < ke;
    const int s1 = tbeg[k], s2 = pk ? tbeg[k + 1] : s1;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int b = g * NTH + tid;
      f1[g] = y[(int64_t)s1 * M + (b < M ? b : 0)];
      f2[g] = pk ? y[(int64_t)s2 * M + (b < M ? b : 0)] : (A)0;
    }
  };
  // Adds the slots [from, to) to a round's points, in slot order, the loads of
  // U slots in flight together.  (b < M only fails when M < NTH: those threads
  // read point 0 and store nothing.)
  constexpr int U = G >= 8 ? 2 : 4;
  auto add_slots = [&](A *v, int from, int to, int p0) {
    auto load = [&](A *w, int sl) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int b = p0 + g * NTH + tid;
        w[g] = y[(int64_t)sl * M + (b < M ? b : 0)];
      }
    };
    int sl = from;
    for (; sl + U <= to; sl += U) {
      A w[U][G];
#pragma unroll
      for (int i = 0; i < U; ++i) load(w[i], sl + i);
#pragma unroll
      for (int i = 0; i < U; ++i)
#pragma unroll
        for (int g = 0; g < G; ++g) v[g] += w[i][g];
    }
    for (; sl < to; ++sl) {
      A w[G];
      load(w, sl);
#pragma unroll
      for (int g = 0; g < G; ++g) v[g] += w[g];
    }
  };
  if constexpr (ONE_ROUND)
    if (kb < ke) first_slots(kb);

  for (int k = kb; k < ke; k += 2) {
    const bool pair = (k + 1) < ke;
    // slots [a0, a1) of the first tensor of the pair, [b0, b1) of the second
    const int a0 = tbeg[k], a1 = tend[k];
    const int b0 = pair ? tbeg[k + 1] : 0, b1 = pair ? tend[k + 1] : 0;
    double ba = 1.0, bb = 1.0;
    if constexpr (SCALED) {
      ba = largest(a0, a1);
      if (pair) bb = largest(b0, b1);
    }
    if constexpr (ONE_ROUND) {
      A v1[G], v2[G];
#pragma unroll
      for (int g = 0; g < G; ++g) { v1[g] = f1[g]; v2[g] = f2[g]; }
      add_slots(v1, a0 + 1, a1, 0);
      add_slots(v2, b0 + 1, b1, 0);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int b = g * NTH + tid;
        if (b < M) z[pad32(bitrev<LOG2M>(b))] = A2{v1[g], v2[g]};
      }
    }
    for (int p0 = 0; !ONE_ROUND && p0 < M; p0 += NTH * G) {
      A v1[G], v2[G];
#pragma unroll
      for (int g = 0; g < G; ++g) v1[g] = v2[g] = 0;
      add_slots(v1, a0, a1, p0);
      add_slots(v2, b0, b1, p0);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int b = p0 + g * NTH + tid;
        if (b < M) z[pad32(bitrev<LOG2M>(b))] = A2{v1[g], v2[g]};
      }
    }
    __syncthreads();
    if constexpr (ONE_ROUND)
      if (k + 2 < ke) first_slots(k + 2);
    if constexpr (TWL)
      fft_lds<A, LOG2M, true, NTH>(z, t);
    else
      fft_lds_tw<A, LOG2M, true, NTH>(z, Tw2<A>{t, t + M / 128});
    double half = 0.5, quarter = 0.25;
    if constexpr (SCALED) {
      const int ek = min(max((ba > 0.0 ? ilogb(ba) : 0) + (bb > 0.0 ? ilogb(bb) : 0), -1000), 1000);
      esum += ek;
      half = ldexp(0.5, -ek);
      quarter = ldexp(0.25, -ek);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = tid + NTH * c;
      if (j < H) {
        const A2 za = z[pad32(j)], zb = z[pad32((M - j) & (M - 1))];
        const double ar = za.x, ai = za.y, br = zb.x, bi = -(double)zb.y;  // B = conj(Z[-j])
        double qr, qi;
        if (pair) {
          const double dr = (ar * ar - ai * ai) - (br * br - bi * bi);
          const double di = 2.0 * (ar * ai - br * bi);
          qr = quarter * di;     // -i (A^2 - B^2) / 4
          qi = -quarter * dr;
        } else {
          qr = half * (ar + br);  // (A + B) / 2
          qi = half * (ai + bi);
        }
        times(pr[c], pi[c], qr, qi);
      }
    }
    __syncthreads();
  }

  if (part != nullptr) {  // this share's product spectrum, for m1_combine_join_kernel or m1_outer_kernel
    double2 *o = part + (((int64_t)blockIdx.x * gridDim.y + s) * gridDim.z + blockIdx.z) * H;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = tid + NTH * c;
      if (j < H) o[j] = make_double2(pr[c], pi[c]);
    }
    if (SCALED && s == 0 && tid == 0) pexp[blockIdx.x] = esum;
    return;
  }
  double sum = 0.0;
  if constexpr (NTH > 256 && LOG2M < 13) {
    double *terms = reinterpret_cast<double *>(smem);
#pragma unroll
    for (int c = 0; c < NC; ++c)
      sum_as_256<NTH>((tid + NTH * c == 0 || 2 * (tid + NTH * c) == M ? 1.0 : 2.0) * pr[c], NTH * c, H, terms, sum);
  } else {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int j = tid + NTH * c;
      if (j < H) sum += ((j == 0 || 2 * j == M) ? 1.0 : 2.0) * pr[c];
    }
  }
  const double tot = block_sum<NTH>(sum, red);
  if (tid == 0) est[(int64_t)blockIdx.x * S + sample0 + s] = tot / (double)M;
}

// The split combine's join: per (network, sample) the product over its
// gsplit shares' spectra, in share order, then the Hermitian sum as in
// m1_combine_kernel.  Its blocks are few, so each is wide and keeps
// kJoinLoads loads per thread in flight (64 samples of 16 shares, m = 4096:
// 39 us with 256 threads and one load at a time, 9.2 so).
constexpr int kJoinThreads = 1024, kJoinLoads = 8;
__global__ __launch_bounds__(kJoinThreads) void m1_combine_join_kernel(const double2 *__restrict__ part, int gsplit,
                                                                       int64_t m, int64_t sample0, int64_t S,
                                                                       double *__restrict__ est) {
  __shared__ double red[kJoinThreads / 64];
  const int64_t H = m / 2 + 1;
  const double2 *q = part + ((int64_t)blockIdx.x * gridDim.y + blockIdx.y) * gsplit * H;
  __shared__ double terms[kJoinThreads];
  double sum = 0.0;
  for (int64_t j0 = 0; j0 < H; j0 += kJoinThreads) {
    const int64_t j = min(j0 + threadIdx.x, H - 1);
    double pr = 1.0, pi = 0.0;
    for (int g0 = 0; g0 < gsplit; g0 += kJoinLoads) {
      double2 v[kJoinLoads];
#pragma unroll
      for (int g = 0; g < kJoinLoads; ++g) v[g] = q[(int64_t)min(g0 + g, gsplit - 1) * H + j];
#pragma unroll
      for (int g = 0; g < kJoinLoads; ++g)
        if (g0 + g < gsplit)
          times(pr, pi, v[g].x, v[g].y);
    }
    sum_as_256<kJoinThreads>(((j == 0 || 2 * j == m) ? 1.0 : 2.0) * pr, j0, H, terms, sum);
  }
  const double tot = block_sum<kJoinThreads>(sum, red);
  if (threadIdx.x == 0) est[(int64_t)blockIdx.x * S + sample0 + blockIdx.y] = tot / (double)m;
}

// All entries of a partial contraction from the product spectra of two groups
// of its tensor pairs: entry loff[a] + roff[b] of sample s is
// (with pexp: 2^(pexp[a] + pexp[nl + b]) times) (1/m) sum_j w_j Re(L_a[j] R_b[j]), L_a = spec[a][s], R_b = spec[nl + b][s],
// w_j = 1 at j = 0 and m/2, else 2: a real product of depth m + 2, taken on
// v_mfma_f64_16x16x4f64 (A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k,
// D[i][j] element i / 4 of lane j + 16 (i % 4)).  A block owns a 16 x 16 tile
// of one sample; its waves take the frequencies in turn, four of a row per
// load instruction (64 bytes), and add their sums in wave order.  Bound by the
// latency of these loads, which come out of the L2: kOuterLoads of each
// operand are in flight per lane.
constexpr int kOuterLoads = 8;
__global__ __launch_bounds__(256) void m1_outer_kernel(const double2 *__restrict__ spec, int32_t nl, int32_t nr,
                                                       const int32_t *__restrict__ loff,
                                                       const int32_t *__restrict__ roff,
                                                       const int32_t *__restrict__ pexp, int64_t m, int64_t sample0, int64_t S, double *__restrict__ est) {
  typedef double f64x4 __attribute__((ext_vector_type(4)));
  __shared__ double sums[3][64][4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int a0 = 16 * (int)blockIdx.x, b0 = 16 * (int)blockIdx.y;
  const int64_t s = blockIdx.z, n = gridDim.z, H = m / 2 + 1;
  const double2 *pa = spec + ((int64_t)min(a0 + (lane & 15), nl - 1) * n + s) * H;
  const double2 *pb = spec + ((int64_t)(nl + min(b0 + (lane & 15), nr - 1)) * n + s) * H;
  const int b = b0 + (lane & 15);
  int ex[4] = {0, 0, 0, 0};
  if (pexp != nullptr) {
#pragma unroll
    for (int i = 0; i < 4; ++i) ex[i] = pexp[min(a0 + 4 * i + (lane >> 4), nl - 1)] + pexp[nl + min(b, nr - 1)];
  }
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int64_t j0 = 4 * wave; j0 < H; j0 += 16 * kOuterLoads) {
    double2 va[kOuterLoads], vb[kOuterLoads];
#pragma unroll
    for (int u = 0; u < kOuterLoads; ++u) {
      const int64_t j = min(j0 + 16 * u + (lane >> 4), H - 1);
      va[u] = pa[j];
      vb[u] = pb[j];
    }
#pragma unroll
    for (int u = 0; u < kOuterLoads; ++u) {
      const int64_t j = j0 + 16 * u + (lane >> 4);
      const double w = (j == 0 || 2 * j == m) ? 1.0 : 2.0;
      const bool in = j < H;  // beyond: terms of 0
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? va[u].x : 0.0, in ? w * vb[u].x : 0.0, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? va[u].y : 0.0, in ? -w * vb[u].y : 0.0, acc, 0, 0, 0);
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) sums[wave - 1][lane][i] = acc[i];
  }
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int a = a0 + 4 * i + (lane >> 4);
    const double v = ((acc[i] + sums[0][lane][i]) + sums[1][lane][i]) + sums[2][lane][i];
    if (a < nl && b < nr)
      est[(int64_t)(loff[a] + roff[b]) * S + sample0 + s] = ldexp(v / (double)m, ex[i]);
  }
}

// ---------------------------------------------------------------------------
// Combine when the m-point FFT does not fit in LDS (m = 2^14 with FP64 data,
// m >= 2^15):
// the same estimate (1/m) Re sum_j prod_k Y_k[j], with the spectra taken in two
// passes through HBM.  As in the in-LDS combine, the tensors of a network go
// in pairs, z = y_a + i y_b (an odd one out with y_b = 0), and the pair's
// product spectrum is Y_a Y_b = (Z[j]^2 - conj(Z[-j])^2) / 4i.  With
// m = n1 n2 (n2 = 256), b = b1 + n1 b2 and j = j2 + n2 j1,
//   Z[j2 + n2 j1] = sum_b1 w_n1^(b1 j1) w_m^(b1 j2) sum_b2 z[b1 + n1 b2] w_n2^(b2 j2),
// w_n = exp(-2 pi i / n).
// Pass 1 (per pair, sample and run of columns b1): the n2-point DFTs over b2
// of the columns, all in one batched LDS transform, times w_m^(b1 j2), stored
// transposed as C[j2][b1].
// Pass 2 (per network, sample and mirror pair of rows): -(j2 + n2 j1) mod m is
// (n2 - j2) + n2 (n1 - 1 - j1) for j2 > 0, so row j2 holds the negated
// frequencies of row n2 - j2.  A block takes rows j2 and n2 - j2 (j2 in
// 1..127), or the self-mirrored rows 0 and 128, of every pair of the network,
// takes their n1-point DFTs in one batched LDS transform, and sums
// prod_pairs (Y_a Y_b)[j] over its frequencies in FP64: 2 Re over row j2 (row
// n2 - j2 holds the conjugates), Re over both self-mirrored rows.  Every
// frequency is visited once and the blocks' sums are added in a fixed order,
// so the result matches the in-LDS combine up to FFT rounding.
constexpr int kBigN2 = 256, kBigRowPairs = kBigN2 / 2;
static_assert(kBigRowPairs == kBigPartials, "one partial sum per row block");
// LDS stride between the transforms of a batch: pad32(256) and one more
// element, so that reading the same point of consecutive transforms (the
// transposed store) falls into distinct banks.
constexpr int kBigStr = kBigN2 + kBigN2 / 32 + 1;

// w_m^e from the half table tw[j] = w_m^j, j < m/2.
template <typename A2>
__device__ __forceinline__ A2 twiddle_at(const A2 *__restrict__ tw, uint32_t e, uint32_t m) {
  e &= m - 1;
  if (e < m / 2) return tw[e];
  const A2 t = tw[e - m / 2];
  return A2{-t.x, -t.y};
}

// Two radix-2 stages on four points, as in fft_lds_batch, with the roundings of
// their complex products written out: the two kernels that take pass 1 give
// the same bits.
template <bool SWAP, typename A2>
__device__ __forceinline__ void big_butterfly(A2 &za, A2 &zb, const A2 w) {
  const auto tr = fma(w.x, zb.x, -(w.y * zb.y));
  const auto ti = SWAP ? fma(w.x, zb.y, w.y * zb.x) : fma(w.y, zb.x, w.x * zb.y);
  zb = A2{za.x - tr, za.y - ti};
  za = A2{za.x + tr, za.y + ti};
}
template <typename A2>
__device__ __forceinline__ void big_radix4(A2 &z0, A2 &z1, A2 &z2, A2 &z3, const A2 w1, const A2 w2, const A2 w3) {
  big_butterfly<false>(z0, z1, w1);
  big_butterfly<false>(z2, z3, w1);
  big_butterfly<false>(z0, z2, w2);
  big_butterfly<true>(z1, z3, w3);
}
// v w_m^e from the two-level table (likewise).
template <typename A2>
__device__ __forceinline__ A2 big_twiddled(const A2 v, const A2 *thi, const A2 *tlo, uint32_t e) {
  const A2 wh = thi[e / kBigN2], wl = tlo[e % kBigN2];
  const A2 w = A2{fma(wh.x, wl.x, -(wh.y * wl.y)), fma(wh.y, wl.x, wh.x * wl.y)};
  return A2{fma(v.x, w.x, -(v.y * w.y)), fma(v.x, w.y, v.y * w.x)};
}

// Columns per pass-1 block: one 128-byte line of each input row per block
// for FP32 sketches, 256 bytes for FP64 (the transforms then fill 68 KB of LDS).
template <typename A>
constexpr int big_cols() { return sizeof(A) == 4 ? 32 : 16; }
// LDS: the batch of transforms, the padded 256-point half table, and the
// two-level table of the transposed store's twiddles w_m^e = hi[e / 256]
// lo[e % 256] (m / 256 <= 256 and 256 entries).
template <typename A>
constexpr size_t big_cols_lds() {
  return sizeof(typename Cplx<A>::type) * (size_t)(big_cols<A>() * kBigStr + kBigN2 / 2 + kBigN2 / 64 + 2 * kBigN2);
}

template <typename A>
__global__ __launch_bounds__(256) void m1_big_cols_kernel(const int32_t *__restrict__ tslot,
                                                          const int32_t *__restrict__ pairs, int64_t n_pairs,
                                                          const A *__restrict__ ybuf, int64_t n_slots, int log2m,
                                                          const typename Cplx<A>::type *__restrict__ tw,
                                                          typename Cplx<A>::type *__restrict__ cbuf) {
  using A2 = typename Cplx<A>::type;
  constexpr int CB = big_cols<A>();    // columns b1 of this block
  constexpr int RS = 256 / CB;         // b2 = r0 + RS i: the thread's points of its column
  constexpr int RPT = kBigN2 / RS;     // points per thread
  constexpr int G = 8;                 // loads in flight per tensor and round
  static_assert(RPT % G == 0, "load rounds");
  extern __shared__ __align__(16) unsigned char smem[];
  A2 *z = reinterpret_cast<A2 *>(smem);
  A2 *tw2 = z + CB * kBigStr;
  A2 *thi = tw2 + kBigN2 / 2 + kBigN2 / 64, *tlo = thi + kBigN2;
  const uint32_t m = 1u << log2m, n1 = m / kBigN2;
  const int64_t pr = blockIdx.x, s = blockIdx.y;
  const uint32_t b1_0 = blockIdx.z * CB;
  const int tid = threadIdx.x, c = tid % CB, r0 = tid / CB;
  if (tid < kBigN2 / 2) tw2[pad32(tid)] = tw[(uint32_t)tid * n1];  // w_n2^t = w_m^(t n1)
  if ((uint32_t)tid < n1) thi[tid] = twiddle_at(tw, (uint32_t)tid * kBigN2, m);  // (published by the
  tlo[tid] = twiddle_at(tw, (uint32_t)tid, m);                                  //  barrier below)
  const int ta = pairs[2 * pr], tb = pairs[2 * pr + 1];
  const int a0 = tslot[ta], a1 = tslot[ta + 1];
  const int bb0 = tb >= 0 ? tslot[tb] : 0, bb1 = tb >= 0 ? tslot[tb + 1] : 0;
  const A *y = ybuf + s * n_slots * (int64_t)m + b1_0 + c;
  // z[b1 + n1 b2] = y_a + i y_b (each summed over its tensor's slots), stored
  // bit-reversed for the transform of column c
  for (int i0 = 0; i0 < RPT; i0 += G) {
    A va[G], vb[G];
#pragma unroll
    for (int g = 0; g < G; ++g) va[g] = vb[g] = 0;
    for (int sl = a0; sl < a1; ++sl) {
#pragma unroll
      for (int g = 0; g < G; ++g) va[g] += y[(int64_t)sl * m + (int64_t)n1 * (r0 + RS * (i0 + g))];
    }
    for (int sl = bb0; sl < bb1; ++sl) {
#pragma unroll
      for (int g = 0; g < G; ++g) vb[g] += y[(int64_t)sl * m + (int64_t)n1 * (r0 + RS * (i0 + g))];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) z[c * kBigStr + pad32(bitrev<8>(r0 + RS * (i0 + g)))] = A2{va[g], vb[g]};
  }
  __syncthreads();
#pragma unroll 1
  for (int lg = 1; lg < 8; lg += 2) {
    const int h = 1 << (lg - 1);
    for (int q = tid; q < CB * (kBigN2 / 4); q += 256) {
      A2 *zt = z + (q >> 6) * kBigStr;
      const int qq = q & 63, k = qq & (h - 1), base = ((qq >> (lg - 1)) << (lg + 1)) + k;
      // (copies: through references into LDS each stage would store and load its points)
      A2 z0 = zt[pad32(base)], z1 = zt[pad32(base + h)], z2 = zt[pad32(base + 2 * h)], z3 = zt[pad32(base + 3 * h)];
      big_radix4(z0, z1, z2, z3, tw2[pad32(k << (8 - lg))], tw2[pad32(k << (7 - lg))], tw2[pad32((k + h) << (7 - lg))]);
      zt[pad32(base)] = z0;
      zt[pad32(base + h)] = z1;
      zt[pad32(base + 2 * h)] = z2;
      zt[pad32(base + 3 * h)] = z3;
    }
    __syncthreads();
  }
  // C[j2][b1] = Z_b1[j2] w_m^(b1 j2): lanes of consecutive b1 write one
  // contiguous run per j2
  A2 *out = cbuf + (s * n_pairs + pr) * (int64_t)m + b1_0 + c;
  const uint32_t b1 = b1_0 + c;
#pragma unroll 4
  for (int i = 0; i < RPT; ++i) {
    const int j2 = r0 + RS * i;
    const uint32_t e = (b1 * (uint32_t)j2) & (m - 1);
    out[(int64_t)j2 * n1] = big_twiddled(z[c * kBigStr + pad32(j2)], thi, tlo, e);
  }
}

// Scatter and pass 1 in one kernel, for FP32 sketches of tensors of one slot
// each: the sketches themselves (m words of each tensor and sample) are neither
// written nor read.  Block: one tensor pair of one sample; its 32-column
// ranges of b1 one after the other (`split` blocks share them where the pairs
// and samples are few).  Per range the 32 x 256 buckets of each tensor are
// accumulated in LDS in 64-bit fixed point, as in m1_scatter_kernel, and turned
// into FP32 in registers, 16 points of a column (b2 = q + 16 i) per thread: in
// bit-reversed order they are one run of 16, so the first four stages of the
// column's transform stay in the registers.  The points change hands once, in
// the accumulators' place, and the last four stages leave a thread the results
// that it stores.
// The range of a term depends on the low bits of its bucket, row word plus
// column word: with the tensor's columns sorted by these bits (once per block),
// a row's terms of one range are consecutive columns, from pos[] of the range's
// first bits minus the row's, around the end of the (doubled) list.  So a range
// takes its own terms only, a group of lanes per row.  A column's word holds
// bucket * 8, sign in bit 31 and, in bits 20 to 29 that the sum of two words'
// buckets does not reach, the column.
// 48 lattices of 16 tensors of bond 16 (65536 entries each), 6 samples,
// m = 65536, FP32: 0.86 ms, against 0.78 for the scatter of the sketches and
// 0.70 for pass 1 alone.  Bound by vector instructions (974 per thread and
// range outside the scatter, most of them the transform's) and, in the scatter,
// by the entries' gather: a load instruction takes a clock per line, and 16
// lanes of a row fall into 7 of its lines of 1 KB.  Ranges of 64 columns (one
// block of 1024 threads per CU, half the reads of the entries) take the same
// time; five terms in flight and 8 lanes to a row 0.92 ms.
constexpr int kBigCols = 32, kBigThreads = 512;
constexpr int kBigPos = kBigN2 + kBigCols + 4;  // positions of the n1 low bits, and of the first ones again
constexpr int kBigTerms = 3;  // loads in flight per lane
constexpr int64_t kBigSplitBlocks = 256;  // one to a CU
constexpr int kBigZ = kBigCols * kBigN2;  // buckets of a range: accumulators [b2][column], then points [position][column]
static_assert(kBigCols * kBigN2 == 16 * kBigThreads, "16 points per thread and range");
// LDS: transforms, twiddles, and per tensor of the pair the doubled column
// list, the row words and the columns' positions.
constexpr size_t big_scatter_lds(int max_cols, int max_rows) {
  return (size_t)8 * (kBigZ + kBigN2 / 2 + kBigN2 / 64 + 2 * kBigN2) +
         2 * ((size_t)8 * max_cols + (size_t)4 * max_rows + 4 * kBigPos) + 16;
}
// lanes per row (log2) so that kBigTerms rounds take nearly every row's terms
// of a range: `mean` of them, plus two standard deviations
__device__ __forceinline__ int big_row_lanes(int mean) {
  int lg = 2;
  while (lg < 6 && (kBigTerms << lg) < mean + 2 * (int)sqrtf((float)mean) + 1) ++lg;
  return lg;
}

template <typename T>
__global__ __launch_bounds__(kBigThreads, 4) void m1_big_scatter_kernel(
    const ScatterSlot *__restrict__ slots, const ModeDesc *__restrict__ modes, const void *const *__restrict__ data,
    const int32_t *__restrict__ tables, int64_t W, const int32_t *__restrict__ pairs, int32_t n_pairs,
    int32_t samples, int32_t split, int log2m, int max_cols, int max_rows, const float2 *__restrict__ tw,
    float2 *__restrict__ cbuf, const double *__restrict__ bound_in, double *__restrict__ bound_out) {
  extern __shared__ __align__(16) unsigned char smem[];
  // (slot_block: the samples of a pair are neighbours on one XCD; its entries,
  // read once per range, come out of that L2)
  const SlotBlock sb = slot_block(blockIdx.x, (uint32_t)n_pairs, (uint32_t)(samples * split));
  const int32_t pr = (int32_t)sb.slot, s = (int32_t)sb.group / split, part = (int32_t)sb.group % split;
  if (pr >= n_pairs) return;  // padding of the grid
  const int tid = threadIdx.x, lane = tid & 63;
  const uint32_t m = 1u << log2m, mask = m - 1, n1 = m / kBigN2, lmask = n1 - 1;
  const int lg1 = log2m - 8;
  unsigned long long *acc = reinterpret_cast<unsigned long long *>(smem);  // [b2][column of the range]
  float2 *z = reinterpret_cast<float2 *>(smem);
  float2 *tw2 = z + kBigZ, *thi = tw2 + kBigN2 / 2 + kBigN2 / 64, *tlo = thi + kBigN2;
  unsigned long long *s_max = reinterpret_cast<unsigned long long *>(tlo + kBigN2);  // [2]
  uint32_t *list0 = reinterpret_cast<uint32_t *>(s_max + 2), *rowt0 = list0 + 4 * max_cols;
  int32_t *pos0 = reinterpret_cast<int32_t *>(rowt0 + 2 * max_rows);

  const int nt = pairs[2 * pr + 1] >= 0 ? 2 : 1;
  ScatterSlot sl[2];
  const T __attribute__((address_space(1))) *X[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    sl[t] = slots[pairs[2 * pr + (t < nt ? t : 0)]];
    X[t] = (const T __attribute__((address_space(1))) *)(reinterpret_cast<const T *>(data[sl[t].tensor]));
  }

  // Once per block: twiddles, row words, sorted columns, the largest |x|.
  if (tid < kBigN2 / 2) tw2[pad32(tid)] = tw[(uint32_t)tid * n1];  // w_n2^t = w_m^(t n1)
  if ((uint32_t)tid < n1) thi[tid] = twiddle_at(tw, (uint32_t)tid * kBigN2, m);
  if (tid < kBigN2) tlo[tid] = twiddle_at(tw, (uint32_t)tid, m);
  if (tid < 2) s_max[tid] = 0ull;
  const int32_t *tab = tables + s * W;
  // Sum over the modes [u0, u1) of the words of index idx.
  auto word = [&](int u0, int u1, uint32_t idx) {
    uint32_t w = 0;
    for (int u = u1 - 1; u >= u0; --u) {
      const ModeDesc md = modes[u];
      const uint32_t qt = u > u0 ? idx / (uint32_t)md.n : 0u, d = idx - qt * (uint32_t)md.n;
      idx = qt;
      const uint32_t v = (uint32_t)tab[md.table_off + d];
      uint32_t h = v & ~kSignBit;
      if (md.comp) h = (m - h) & mask;
      w = ((w + (h << 3)) & (mask << 3)) | ((w ^ v) & kSignBit);
    }
    return w;
  };
  constexpr int CT = kMaxCols / kBigThreads;  // columns per thread
  uint32_t cw[2][CT];
  int32_t *cursor = reinterpret_cast<int32_t *>(smem);  // [2][kBigN2], before the accumulators are cleared
  for (int t = 0; t < nt; ++t)
    if ((uint32_t)tid < n1) pos0[t * kBigPos + tid] = 0;
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    if (t >= nt) break;
    const int mode0 = sl[t].mode0, sp = mode0 + sl[t].split;
    for (int r = tid; r < sl[t].rows; r += kBigThreads) rowt0[t * max_rows + r] = word(mode0, sp, (uint32_t)r);
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      const int col = tid + i * kBigThreads;
      if (col >= sl[t].L) continue;
      cw[t][i] = word(sp, mode0 + sl[t].q, (uint32_t)col);
      atomicAdd(&pos0[t * kBigPos + ((cw[t][i] >> 3) & lmask)], 1);
    }
  }
  // Largest |x| of each tensor, when it was not recorded before.
  if (bound_in == nullptr) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (t >= nt) break;
      using Q = typename Quad<T>::type;
      const Q __attribute__((address_space(1))) *Xq = (const Q __attribute__((address_space(1))) *)X[t];
      const uint32_t N = (uint32_t)sl[t].rows * (uint32_t)sl[t].L, NQ = N / 4;
      float lmax = 0.0f;
      for (uint32_t i0 = tid; i0 < NQ; i0 += kBigThreads * 8) {
        Q v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = Xq[min(i0 + (uint32_t)u * kBigThreads, NQ - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) lmax = fmaxf(lmax, fabsf(to_acc_any((T)v[u][i])));
      }
      if (4 * NQ + tid < N) lmax = fmaxf(lmax, fabsf(to_acc_any((T)X[t][4 * NQ + tid])));
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) lmax = fmaxf(lmax, __shfl_xor(lmax, off, 64));
      if (lane == 0) atomicMax(&s_max[t], (unsigned long long)__double_as_longlong((double)lmax));
    }
  }
  __syncthreads();
  // exclusive sums of the counts, one wave per tensor, four counts to a lane
  if (tid < 64 * nt) {
    int32_t *p = pos0 + (tid >> 6) * kBigPos, *c = cursor + (tid >> 6) * kBigN2;
    const bool in = 4u * (uint32_t)lane < n1;
    int n[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      n[i] = in ? p[4 * lane + i] : 0;
      sum += n[i];
    }
    int upto = sum;
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(upto, off, 64);
      if (lane >= off) upto += o;
    }
    int at = upto - sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (in) p[4 * lane + i] = c[4 * lane + i] = at;
      at += n[i];
    }
    if (lane == 63) p[n1] = upto;
    // the next turn's first ones
    const int total = __shfl(upto, 63, 64);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * lane + i <= kBigCols) p[n1 + 4 * lane + i] = total + (upto - sum) + (i > 0 ? n[0] : 0) +
                                                            (i > 1 ? n[1] : 0) + (i > 2 ? n[2] : 0);
  }
  __syncthreads();
  double sc[2];
  int scale[2], lgl[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    uint32_t *list = list0 + t * 2 * max_cols;
#pragma unroll
    for (int i = 0; i < CT; ++i) {
      const int col = tid + i * kBigThreads;
      if (t >= nt || col >= sl[t].L) continue;
      const int at = atomicAdd(&cursor[t * kBigN2 + ((cw[t][i] >> 3) & lmask)], 1);
      list[at] = list[at + sl[t].L] = cw[t][i] | ((uint32_t)col << 20);
    }
    double bound;
    if (bound_in != nullptr) {
      bound = bound_in[sl[t].id];
    } else {
      const double bm = __longlong_as_double((long long)s_max[t < nt ? t : 0]);
      int e = 0;
      (void)frexp(bm, &e);  // 2^(e - 1) <= bm < 2^e
      bound = bm > 0.0 ? ldexp(1.0, e - 1) : 0.0;
      if (t < nt && s == 0 && part == 0 && tid == 0) bound_out[sl[t].id] = bound;
    }
    scale[t] = 0;
    if (bound > 0.0) {
      const uint32_t N = (uint32_t)sl[t].rows * (uint32_t)sl[t].L;
      int e;
      (void)frexp(bound, &e);  // bound = 2^(e - 1)
      scale[t] = 62 - max(N > 1 ? 32 - __clz(N - 1) : 0, 11) - e;
    }
    sc[t] = ldexp(1.0, scale[t]);
    lgl[t] = big_row_lanes(max(1, sl[t].L * kBigCols / (int)n1));
  }
  __syncthreads();  // the lists are there, the cursors no longer used
  lds_zero(smem, 8 * kBigCols * kBigN2, tid, kBigThreads);

  constexpr double kMagic = 6755399441055744.0;  // 1.5 2^52: x sc + kMagic holds round(x sc) in its low bits
  const long long kMagicBits = __double_as_longlong(kMagic);
  constexpr int kRowBit = 3 + __builtin_ctz(kBigCols);
  const int sh = lg1 + 3 - kRowBit;  // a word's b2, to its byte offset [b2][kBigCols]
  const uint32_t lds0 =
      (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char *)smem);
  const int c = tid % kBigCols, q0 = tid / kBigCols;
  const int ranges = (int)n1 / kBigCols;
  for (int range = part; range < ranges; range += split) {
    float2 p[16];  // points of column c; at first in the order of their buckets
    auto sketch = [&](int t, auto put) {
      const int L = sl[t].L, rows = sl[t].rows, lanes = 1 << lgl[t], sub = tid & (lanes - 1);
      const uint32_t *list = list0 + t * 2 * max_cols, *rowt = rowt0 + t * max_rows;
      const int32_t *pos = pos0 + t * kBigPos;
      for (int r = tid >> lgl[t]; r < rows; r += kBigThreads >> lgl[t]) {
        const uint32_t h = rowt[r];
        const uint32_t first = ((uint32_t)(kBigCols * range) - (h >> 3)) & lmask, end = first + kBigCols;
        const int j0 = pos[first], j1 = pos[end], base = r * L;
        for (int j = j0 + sub; j < j1; j += kBigTerms * lanes) {
          uint32_t w[kBigTerms];
          float x[kBigTerms];
#pragma unroll
          for (int k = 0; k < kBigTerms; ++k) w[k] = list[min(j + k * lanes, j1 - 1)];
#pragma unroll
          for (int k = 0; k < kBigTerms; ++k) x[k] = to_acc_any(X[t][(uint32_t)base + ((w[k] >> 20) & 1023u)]);
          // (all loads before the first use: they would sink into the branches)
#pragma unroll
          for (int k = 0; k < kBigTerms; ++k) asm volatile("" : "+v"(x[k]));
#pragma unroll
          for (int k = 0; k < kBigTerms; ++k) {
            if (j + k * lanes >= j1) break;
            const uint32_t a = h + w[k];
            const double xd = (double)flip_sign(x[k], a & kSignBit);
            const long long v64 = __double_as_longlong(fma(xd, sc[t], kMagic)) - kMagicBits;
            const uint32_t at = ((a >> sh) & ((kBigN2 - 1) << kRowBit)) | (a & ((kBigCols - 1) << 3));
            __hip_atomic_fetch_add((__attribute__((address_space(3))) unsigned long long *)(lds0 + at),
                                   (unsigned long long)v64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        unsigned long long *a = acc + (q0 + 16 * i) * kBigCols + c;
        put(i, (float)ldexp((double)(long long)*a, -scale[t]));
        *a = 0ull;
      }
      __syncthreads();
    };
    __syncthreads();  // the accumulators are cleared
    // (bit-reversed: b2 = q0 + 16 i is at 16 bitrev(q0) + bitrev(i))
    sketch(0, [&](int i, float v) { p[bitrev<4>(i)] = float2{v, 0.0f}; });
    if (nt == 2) sketch(1, [&](int i, float v) { p[bitrev<4>(i)].y = v; });
#pragma unroll
    for (int g = 0; g < 16; g += 4) big_radix4(p[g], p[g + 1], p[g + 2], p[g + 3], tw2[0], tw2[0], tw2[pad32(64)]);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      big_radix4(p[k], p[k + 4], p[k + 8], p[k + 12], tw2[pad32(32 * k)], tw2[pad32(16 * k)], tw2[pad32(16 * k + 64)]);
#pragma unroll
    for (int i = 0; i < 16; ++i) z[(16 * bitrev<4>(q0) + i) * kBigCols + c] = p[i];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      p[j] = z[(q0 + 16 * j) * kBigCols + c];
      acc[(q0 + 16 * j) * kBigCols + c] = 0ull;  // nobody else's
    }
#pragma unroll
    for (int g = 0; g < 16; g += 4)
      big_radix4(p[g], p[g + 1], p[g + 2], p[g + 3], tw2[pad32(8 * q0)], tw2[pad32(4 * q0)], tw2[pad32(4 * q0 + 64)]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int kk = q0 + 16 * k;
      big_radix4(p[k], p[k + 4], p[k + 8], p[k + 12], tw2[pad32(2 * kk)], tw2[pad32(kk)], tw2[pad32(kk + 64)]);
    }
    // C[j2][b1] = Z_b1[j2] w_m^(b1 j2), as in m1_big_cols_kernel
    const uint32_t b1 = (uint32_t)(range * kBigCols + c);
    float2 *out = cbuf + ((int64_t)s * n_pairs + pr) * (int64_t)m + b1;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int j2 = q0 + 16 * j;
      out[(int64_t)j2 * n1] = big_twiddled(p[j], thi, tlo, (b1 * (uint32_t)j2) & mask);
    }
  }
}

// Pairs per pass-2 round: 2 rows each, KP * 2 transforms in LDS (34 KB).
template <typename A>
constexpr int big_rows_pairs() { return sizeof(A) == 4 ? 8 : 4; }

template <typename A, int LOG2N1>
__global__ __launch_bounds__(256) void m1_big_rows_kernel(const int32_t *__restrict__ pair0,
                                                          const int32_t *__restrict__ pairs, int64_t n_pairs,
                                                          const typename Cplx<A>::type *__restrict__ cbuf,
                                                          const typename Cplx<A>::type *__restrict__ tw,
                                                          double *__restrict__ partial) {
  using A2 = typename Cplx<A>::type;
  constexpr int N1 = 1 << LOG2N1;
  constexpr uint32_t M = (uint32_t)N1 * kBigN2;
  constexpr int KP = big_rows_pairs<A>();
  constexpr int STR = N1 + N1 / 32 + 1;
  constexpr int NL = 2 * KP * N1 / 256;  // loads per thread and round
  static_assert(NL >= 1 && (2 * KP * N1) % 256 == 0, "load rounds");
  __shared__ A2 z[2 * KP * STR];
  __shared__ A2 tw1[N1 / 2 + N1 / 64];
  __shared__ double red[4];
  const int net = blockIdx.x;
  const int64_t s = blockIdx.y;
  const int rp = blockIdx.z, tid = threadIdx.x;
  const int rowA = rp == 0 ? 0 : rp, rowB = rp == 0 ? kBigN2 / 2 : kBigN2 - rp;
  if (tid < N1 / 2) tw1[pad32(tid)] = tw[(uint32_t)tid * kBigN2];  // w_n1^t = w_m^(t n2)
  const int p0 = pair0[net], p1 = pair0[net + 1];
  double pr1 = 1.0, pi1 = 0.0, pr2 = 1.0, pi2 = 0.0;  // rows A and (rp = 0) B
  // pair product at frequency (row t, point j1), mirror at (row u, point j1m)
  auto pair_q = [&](int t, int j1, int u, int j1m, bool pair, double &qr, double &qi) {
    const A2 za = z[t * STR + pad32(j1)], zb = z[u * STR + pad32(j1m)];
    const double ar = za.x, ai = za.y, br = zb.x, bi = -(double)zb.y;  // B = conj(Z[-j])
    if (pair) {
      const double dr = (ar * ar - ai * ai) - (br * br - bi * bi);
      const double di = 2.0 * (ar * ai - br * bi);
      qr = 0.25 * di;  // -i (A^2 - B^2) / 4
      qi = -0.25 * dr;
    } else {
      qr = 0.5 * (ar + br);  // (A + B) / 2
      qi = 0.5 * (ai + bi);
    }
  };
  for (int q0 = p0; q0 < p1; q0 += KP) {
    const int nk = min(KP, p1 - q0);
    __syncthreads();  // the previous round's readers are done (and tw1 is written)
    A2 v[NL];
#pragma unroll
    for (int g = 0; g < NL; ++g) {
      const int i = min(tid + 256 * g, 2 * nk * N1 - 1);
      const int t = i / N1, e = i % N1;  // transform t: pair q0 + t/2, row A or B
      v[g] = cbuf[(s * n_pairs + q0 + t / 2) * (int64_t)M + (int64_t)((t & 1) ? rowB : rowA) * N1 + e];
    }
#pragma unroll
    for (int g = 0; g < NL; ++g) {
      const int i = tid + 256 * g;
      if (i < 2 * nk * N1) z[(i / N1) * STR + pad32(bitrev<LOG2N1>(i % N1))] = v[g];
    }
    __syncthreads();
    fft_lds_batch<A, LOG2N1, STR, 256>(z, tw1, 2 * nk);  // ends with a barrier
    if (tid < N1) {
      for (int k = 0; k < nk; ++k) {
        const bool pair = pairs[2 * (q0 + k) + 1] >= 0;
        double qr, qi, nr;
        if (rp == 0) {
          pair_q(2 * k, tid, 2 * k, (N1 - tid) & (N1 - 1), pair, qr, qi);  // row 0
          nr = pr1 * qr - pi1 * qi;
          pi1 = pr1 * qi + pi1 * qr;
          pr1 = nr;
          pair_q(2 * k + 1, tid, 2 * k + 1, N1 - 1 - tid, pair, qr, qi);  // row n2 / 2
          nr = pr2 * qr - pi2 * qi;
          pi2 = pr2 * qi + pi2 * qr;
          pr2 = nr;
        } else {
          pair_q(2 * k, tid, 2 * k + 1, N1 - 1 - tid, pair, qr, qi);  // row j2, mirror in row n2 - j2
          nr = pr1 * qr - pi1 * qi;
          pi1 = pr1 * qi + pi1 * qr;
          pr1 = nr;
        }
      }
    }
  }
  const double part = tid < N1 ? (rp == 0 ? pr1 + pr2 : 2.0 * pr1) : 0.0;
  const double tot = block_sum_256(part, red);
  if (tid == 0) partial[((int64_t)net * gridDim.y + s) * kBigRowPairs + rp] = tot;
}

__global__ __launch_bounds__(256) void m1_big_sum_kernel(const double *__restrict__ partial, int64_t n_nets,
                                                         int64_t samples, int parts, int64_t sample0, int64_t S,
                                                         double inv_m, double *__restrict__ est) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;  // (network, sample)
  if (i >= n_nets * samples) return;
  const int64_t net = i / samples, s = i - net * samples;
  double v = 0.0;
  for (int q = 0; q < parts; ++q) v += partial[i * parts + q];
  est[net * S + sample0 + s] = v * inv_m;
}

__global__ __launch_bounds__(256) void sample_stats_kernel(const double *__restrict__ est,
                                                           int64_t S, double *__restrict__ stats) {
  __shared__ double red[4];
  __shared__ double mean_sh;
  const double *x = est + (int64_t)blockIdx.x * S;
  double sum = 0.0;
  for (int64_t i = threadIdx.x; i < S; i += 256) sum += x[i];
  const double tot = block_sum_256(sum, red);
  if (threadIdx.x == 0) mean_sh = tot / (double)S;
  __syncthreads();
  const double mu = mean_sh;
  double sq = 0.0;
  for (int64_t i = threadIdx.x; i < S; i += 256) {
    const double d = x[i] - mu;
    sq += d * d;
  }
  const double ss = block_sum_256(sq, red);
  if (threadIdx.x == 0) {
    stats[2 * blockIdx.x] = mu;
    stats[2 * blockIdx.x + 1] = S > 1 ? ss / (double)(S - 1) : 0.0;
  }
}

template <typename A>
__global__ void slots_to_tensors_kernel(const int32_t *__restrict__ tslot, int64_t n_tensors,
                                        const A *__restrict__ ybuf, int64_t n_slots, int log2m,
                                        double *__restrict__ out) {
  const int64_t m = 1ll << log2m;
  const int64_t k = blockIdx.x, s = blockIdx.y;
  for (int64_t b = threadIdx.x; b < m; b += blockDim.x) {
    double v = 0.0;
    for (int sl = tslot[k]; sl < tslot[k + 1]; ++sl) v += (double)ybuf[(s * n_slots + sl) * m + b];
    out[(s * n_tensors + k) * m + b] = v;
  }
}

template <typename A>
__global__ void twiddle_kernel(int64_t m, typename Cplx<A>::type *out) {
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < m / 2;
       j += (int64_t)gridDim.x * blockDim.x) {
    double sv, cv;
    sincospi(-2.0 * (double)j / (double)m, &sv, &cv);
    out[j] = typename Cplx<A>::type{(A)cv, (A)sv};
  }
}

constexpr size_t kWideLds = 81920;

// One launch over the slots that are not small and all batches of SB samples.
// A block takes `gs` batches: 16 samples where that leaves 2048 blocks (the
// block's start is shared by all of them), fewer otherwise.  More than 16 leave
// too few blocks of one slot side by side on an XCD to share its entries in
// the L2 (256 lattices of bond 16, 32 samples: 2.83 ms per call with 16 samples
// per block, 2.96 with 32).
constexpr int64_t kSlotBlocks = 2048, kBlockSamples = 16;
constexpr int64_t kNarrowSlot = 16384;  // entries
// One to a CU.  A FP64 lattice of 16 tensors, bond 16, m = 65536, 4 samples: 109
// us per call with a slot's ranges in one block, 85 so; up to 512 blocks (a
// second round, half as long) cost a lattice of 9 of bond 9, 8 samples, 96
// against 90.
constexpr int64_t kRangeBlocks = 256;
template <typename T, typename A, int SB, int BANKS, int NT, bool RANGED = false>
int scatter_launch(const M1Launch &L, hipStream_t st) {
  const int64_t n = L.n_big;
  if (n == 0) return TN_OK;
  auto kern = m1_scatter_kernel<T, A, SB, BANKS, NT, RANGED>;
  const size_t lds = m1_scatter_lds(SB, BANKS, L.log2m);
  if (lds > 65536)
    TN_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  const int64_t batches = (L.samples + SB - 1) / SB;
  const int64_t gs = std::max<int64_t>(1, std::min({batches, kBlockSamples / SB, n * batches / kSlotBlocks}));
  const int64_t groups = (batches + gs - 1) / gs;
  // The ranges of a group on blocks of their own while there is a CU for each
  // (a block fills one).
  int64_t rsplit = 1;
  if (RANGED)
    while (rsplit < (int64_t)1 << (L.log2m - kMaxLog2Acc) && 2 * rsplit * n * groups <= kRangeBlocks) rsplit *= 2;
  // groups per grid row: the grid's x extent stays within 2^31 threads
  const int64_t slots8 = (n + 7) / 8 * 8, runs = groups * rsplit;
  const int64_t gx = std::max<int64_t>(1, std::min<int64_t>(runs, ((int64_t)1 << 21) / slots8));
  const dim3 grid(slot_blocks((uint32_t)n, (uint32_t)gx), (unsigned)((runs + gx - 1) / gx));
  hipLaunchKernelGGL(kern, grid, dim3(NT), lds, st, L.slots, (int32_t)n, L.modes, L.data, L.tables, L.W,
                     L.samples, L.log2m, L.n_slots, reinterpret_cast<A *>(L.ybuf),
                     L.record_bound ? nullptr : L.slot_bound, L.slot_bound, (int32_t)gs, (int32_t)groups,
                     (int32_t)gx, (int32_t)rsplit);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

template <typename T, typename A, int SB>
int scatter_sb(const M1Launch &all, hipStream_t st) {
  // Fewer blocks than give a block several batches: one launch for slots of both
  // kinds (the sums are the same; 6 tensors of 29 to 6496 entries, one sample,
  // m = 64: 23.0 us per call with two launches, 17.3 with one; 250 samples, m =
  // 1024: 63.7, 48.0; 60 networks of the batch, 16 samples, m = 1024: 94, 81).
  M1Launch L = all;
  if (L.n_big > 0 && L.n_slots * ((L.samples + SB - 1) / SB) < kSlotBlocks) L.n_big = L.n_slots;
  const bool ranged = L.log2m > kMaxLog2Acc;
  if (ranged && (SB != 1 || L.banks != 1))
    return set_error(TN_ERR_ARG, "scatter: m = 2^%d takes one bank and one sample per pass", L.log2m);
  if constexpr (SB == 1)
    if (ranged) return scatter_launch<T, A, 1, 1, 1024, true>(L, st);
  // 1024 threads when a block's LDS leaves no room for a second one on its
  // CU, so that the CU still runs 16 waves; else 512.
  const bool wide = m1_scatter_lds(SB, L.banks, L.log2m) > kWideLds;
  int rc;
  // 256 threads where every slot is small and there are blocks enough: less of
  // a batch goes into the words and barriers of a block (64 triangles of 64 x
  // 64, 256 samples, m = 256: 159 against 188 us per call in FP64, 145 against
  // 160 in FP32; 96 x 96: 244, 277).  For large slots 512 (256 lattices of
  // 65536 entries a tensor: 2.81 against 2.89 ms; the ladder 540, 636 us).
  const int64_t batches = (L.samples + SB - 1) / SB;
  const bool narrow = L.max_entries <= kNarrowSlot && L.n_big * batches >= kSlotBlocks;
  if (!wide && narrow)
    rc = L.banks == 2 ? scatter_launch<T, A, SB, 2, 256>(L, st) : scatter_launch<T, A, SB, 1, 256>(L, st);
  else if (wide)
    rc = L.banks == 2 ? scatter_launch<T, A, SB, 2, 1024>(L, st) : scatter_launch<T, A, SB, 1, 1024>(L, st);
  else
    rc = L.banks == 2 ? scatter_launch<T, A, SB, 2, 512>(L, st) : scatter_launch<T, A, SB, 1, 512>(L, st);
  if (rc != TN_OK || L.n_big == L.n_slots) return rc;
  // small slots: four samples at a time per block, one per wave
  const int64_t n = L.n_slots - L.n_big, steps = (L.samples + 3) / 4;
  const int64_t gs = std::max<int64_t>(1, std::min({steps, kBlockSamples / 4, n * steps / kSlotBlocks}));
  const int64_t groups = (steps + gs - 1) / gs, slots8 = (n + 7) / 8 * 8;
  const int64_t gx = std::max<int64_t>(1, std::min<int64_t>(groups, ((int64_t)1 << 21) / slots8));
  const size_t lds = 4 * (std::max<size_t>((size_t)8 << L.log2m, 16) + kStageWords * 4);
  auto kern = m1_scatter_small_kernel<T, A>;
  if (lds > 65536)
    TN_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  const dim3 grid(slot_blocks((uint32_t)n, (uint32_t)gx), (unsigned)((groups + gx - 1) / gx));
  hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, L.slots + L.n_big, (int32_t)n, L.modes, L.data, L.tables, L.W,
                     L.samples, L.log2m, L.n_slots, reinterpret_cast<A *>(L.ybuf),
                     L.record_bound ? L.slot_bound : nullptr, (int32_t)gs, (int32_t)groups, (int32_t)gx);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

template <typename T, typename A>
int scatter_t(const M1Launch &L, hipStream_t st) {
  switch (L.sb) {
    case 1: return scatter_sb<T, A, 1>(L, st);
    case 2: return scatter_sb<T, A, 2>(L, st);
    case 4: return scatter_sb<T, A, 4>(L, st);
    case 8: return scatter_sb<T, A, 8>(L, st);
    default: return set_error(TN_ERR_ARG, "scatter: unsupported sample batch %d", L.sb);
  }
}

constexpr int64_t kFewCombineBlocks = 256;
template <typename A, int LOG2M, int NTH = LOG2M >= 13 ? 1024 : 256>
int combine_m(const NetDesc *nets, int64_t n_nets, const int32_t *tbeg, const int32_t *tend, const void *ybuf,
              int64_t n_slots, int64_t samples, int64_t sample0, int64_t S, const void *tw,
              double *est, int32_t csplit, double *cpart, const double *bound, int32_t *pexp, hipStream_t st) {
  using A2 = typename Cplx<A>::type;
  // z (m points, one spare element per 32: bank spread) and, when the total
  // stays within 64 KB, the m/2 twiddles (padded), else the two-level table
  constexpr int M = 1 << LOG2M;
  constexpr size_t zt = sizeof(A2) * (size_t)(M + M / 32 + M / 2 + M / 64 + 2);
  constexpr bool TWL = zt <= 65536 || M < 128;
  constexpr size_t lds = TWL ? zt : sizeof(A2) * (size_t)(M + M / 32 + M / 128 + 64);
  if constexpr (lds > kMaxLdsBytes) {
    return set_error(TN_ERR_UNSUPPORTED, "combine: the %d-point transform does not fit in LDS", M);
  } else {
    // 1024 threads also where a CU has one block at most (m = 2048, 4096): 32
    // samples of three tensors of 16 slots each, m = 4096, FP32: 47 us with
    // 256 threads, 22 so
    const int64_t blocks = n_nets * samples * csplit;
    if constexpr (LOG2M >= 11 && NTH == 256)
      if (blocks <= kFewCombineBlocks)
        return combine_m<A, LOG2M, 1024>(nets, n_nets, tbeg, tend, ybuf, n_slots, samples, sample0, S, tw, est, csplit,
                                         cpart, bound, pexp, st);
    auto kern = bound ? m1_combine_kernel<A, LOG2M, TWL, NTH, true> : m1_combine_kernel<A, LOG2M, TWL, NTH, false>;
    if (lds > 65536)
      TN_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)lds));
    const bool split = cpart != nullptr;
    dim3 grid((unsigned)n_nets, (unsigned)samples, split ? (unsigned)csplit : 1u);
    double2 *part = reinterpret_cast<double2 *>(cpart);
    hipLaunchKernelGGL(kern, grid, dim3(NTH), lds, st, nets, tbeg, tend,
                       reinterpret_cast<const A *>(ybuf), n_slots, sample0, S,
                       reinterpret_cast<const A2 *>(tw), est, part, bound, pexp);
    TN_HIP_CHECK(hipGetLastError());
    if (split && est != nullptr) {
      hipLaunchKernelGGL(m1_combine_join_kernel, dim3((unsigned)n_nets, (unsigned)samples),
                         dim3(kJoinThreads), 0, st, part, (int)csplit, (int64_t)M, sample0, S, est);
      TN_HIP_CHECK(hipGetLastError());
    }
    return TN_OK;
  }
}

template <typename A>
int combine_big(int64_t n_nets, const int32_t *tslot, const int32_t *pairs, const int32_t *pair0,
                int64_t n_pairs, const void *ybuf, int64_t n_slots, int64_t samples, int64_t sample0, int64_t S,
                int log2m, const void *tw, void *cbuf, double *partial, double *est, hipStream_t st) {
  using A2 = typename Cplx<A>::type;
  const uint32_t m = 1u << log2m, n1 = m / kBigN2;
  if (ybuf != nullptr) {
    constexpr size_t lds = big_cols_lds<A>();
    TN_HIP_CHECK(hipFuncSetAttribute((const void *)m1_big_cols_kernel<A>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(m1_big_cols_kernel<A>, dim3((unsigned)n_pairs, (unsigned)samples, n1 / big_cols<A>()),
                       dim3(256), lds, st, tslot, pairs, n_pairs, reinterpret_cast<const A *>(ybuf), n_slots, log2m,
                       reinterpret_cast<const A2 *>(tw), reinterpret_cast<A2 *>(cbuf));
    TN_HIP_CHECK(hipGetLastError());
  }
  dim3 g2((unsigned)n_nets, (unsigned)samples, kBigRowPairs);
  const A2 *cb = reinterpret_cast<const A2 *>(cbuf), *t2 = reinterpret_cast<const A2 *>(tw);
  if (log2m == 14)
    hipLaunchKernelGGL((m1_big_rows_kernel<A, 6>), g2, dim3(256), 0, st, pair0, pairs, n_pairs, cb, t2, partial);
  else if (log2m == 15)
    hipLaunchKernelGGL((m1_big_rows_kernel<A, 7>), g2, dim3(256), 0, st, pair0, pairs, n_pairs, cb, t2, partial);
  else
    hipLaunchKernelGGL((m1_big_rows_kernel<A, 8>), g2, dim3(256), 0, st, pair0, pairs, n_pairs, cb, t2, partial);
  TN_HIP_CHECK(hipGetLastError());
  const int64_t np = n_nets * samples;
  hipLaunchKernelGGL(m1_big_sum_kernel, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, st, partial, n_nets,
                     samples, kBigRowPairs, sample0, S, 1.0 / (double)m, est);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

template <typename A>
int combine_t(const NetDesc *nets, int64_t n_nets, const int32_t *tbeg, const int32_t *tend, const void *ybuf,
              int64_t n_slots, int64_t samples, int64_t sample0, int64_t S, int log2m,
              const void *tw, double *est, int32_t csplit, double *cpart, const double *bound, int32_t *pexp,
              hipStream_t st) {
#define TN_COMBINE_CASE(LG)                                                                            \
  case LG:                                                                                             \
    return combine_m<A, LG>(nets, n_nets, tbeg, tend, ybuf, n_slots, samples, sample0, S, tw, est, csplit, \
                            cpart, bound, pexp, st);
  switch (log2m) {
    TN_COMBINE_CASE(0) TN_COMBINE_CASE(1) TN_COMBINE_CASE(2) TN_COMBINE_CASE(3)
    TN_COMBINE_CASE(4) TN_COMBINE_CASE(5) TN_COMBINE_CASE(6) TN_COMBINE_CASE(7)
    TN_COMBINE_CASE(8) TN_COMBINE_CASE(9) TN_COMBINE_CASE(10) TN_COMBINE_CASE(11)
    TN_COMBINE_CASE(12) TN_COMBINE_CASE(13) TN_COMBINE_CASE(14)
    default: return set_error(TN_ERR_UNSUPPORTED, "combine: log2(m) = %d", log2m);
  }
#undef TN_COMBINE_CASE
}

}  // namespace

size_t m1_scatter_lds(int sb, int banks, int log2m) {
  const size_t ma = (size_t)1 << std::min(log2m, kMaxLog2Acc);  // bucket ranges above
  const size_t acc = banks == 2 ? sign_bank_bytes(sb, (uint32_t)ma) : (size_t)sb * 8 * ma;
  return ((acc + 15) & ~(size_t)15) + (size_t)sb * 4 * (row_chunk(sb) + kStageWords) + 16;
}

int launch_m1_scatter(const M1Launch &L, hipStream_t st) {
  if (L.n_slots == 0 || L.samples == 0) return TN_OK;
  if ((L.samples + L.sb - 1) / L.sb > 65535)
    return set_error(TN_ERR_UNSUPPORTED, "scatter: too many sample batches in one launch");
  switch (L.dtype) {
    case TN_F64: return scatter_t<double, double>(L, st);
    case TN_F32: return scatter_t<float, float>(L, st);
    case TN_BF16: return scatter_t<uint16_t, float>(L, st);
    default: return set_error(TN_ERR_ARG, "scatter: dtype %d", L.dtype);
  }
}

size_t m1_big_scatter_lds(int max_cols, int max_rows) { return big_scatter_lds(max_cols, max_rows); }

int launch_m1_big_scatter(const M1Launch &L, const int32_t *pairs, int64_t n_pairs, int max_cols, int max_rows,
                          const void *tw, void *cbuf, hipStream_t st) {
  if (n_pairs == 0 || L.samples == 0) return TN_OK;
  // a block per range where whole pairs leave CUs without a block
  const int64_t ranges = (int64_t)(1 << L.log2m) / kBigN2 / kBigCols, blocks = n_pairs * L.samples;
  const int64_t split = std::max<int64_t>(1, std::min<int64_t>(ranges, (kBigSplitBlocks + blocks - 1) / blocks));
  const int64_t grid = (n_pairs * L.samples * split + kXcds - 1) / kXcds * kXcds;
  if (grid > (int64_t)1 << 21 || (L.log2m != 15 && L.log2m != 16))
    return set_error(TN_ERR_UNSUPPORTED, "scatter with the first transforms: %lld blocks, m = 2^%d", (long long)grid,
                     L.log2m);
  const size_t lds = big_scatter_lds(max_cols, max_rows);
  auto run = [&](auto kern) -> int {
    TN_HIP_CHECK(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kBigThreads), lds, st, L.slots, L.modes, L.data, L.tables,
                       L.W, pairs, (int32_t)n_pairs, (int32_t)L.samples, (int32_t)split, L.log2m, max_cols, max_rows,
                       reinterpret_cast<const float2 *>(tw), reinterpret_cast<float2 *>(cbuf),
                       L.record_bound ? nullptr : L.slot_bound, L.slot_bound);
    TN_HIP_CHECK(hipGetLastError());
    return TN_OK;
  };
  if (L.dtype == TN_F32) return run(m1_big_scatter_kernel<float>);
  if (L.dtype == TN_BF16) return run(m1_big_scatter_kernel<uint16_t>);
  return set_error(TN_ERR_ARG, "scatter with the first transforms: dtype %d", L.dtype);
}

int launch_m1_combine(const NetDesc *nets, int64_t n_nets, const int32_t *tbeg, const int32_t *tend, int dtype,
                      const void *ybuf, int64_t n_slots, int64_t samples, int64_t sample0,
                      int64_t S, int log2m, const void *tw, double *est, int32_t csplit, double *cpart,
                      hipStream_t st, const double *bound, int32_t *pexp) {
  if (n_nets == 0 || samples == 0) return TN_OK;
  if (samples > 65535) return set_error(TN_ERR_UNSUPPORTED, "combine: samples per launch");
  if (dtype == TN_F64)
    return combine_t<double>(nets, n_nets, tbeg, tend, ybuf, n_slots, samples, sample0, S, log2m, tw, est, csplit,
                             cpart, bound, pexp, st);
  return combine_t<float>(nets, n_nets, tbeg, tend, ybuf, n_slots, samples, sample0, S, log2m, tw, est, csplit,
                          cpart, bound, pexp, st);
}

int launch_m1_outer(const double *spec, int64_t nl, int64_t nr, const int32_t *loff, const int32_t *roff,
                    const int32_t *pexp, int64_t samples, int64_t sample0, int64_t S, int64_t m, double *est, hipStream_t st) {
  if (samples > 65535 || nr > 16 * 65535) return set_error(TN_ERR_UNSUPPORTED, "outer product: grid");
  const dim3 grid((unsigned)((nl + 15) / 16), (unsigned)((nr + 15) / 16), (unsigned)samples);
  hipLaunchKernelGGL(m1_outer_kernel, grid, dim3(256), 0, st, reinterpret_cast<const double2 *>(spec), (int32_t)nl,
                     (int32_t)nr, loff, roff, pexp, m, sample0, S, est);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

int launch_m1_combine_big(int64_t n_nets, const int32_t *tslot, const int32_t *pairs, const int32_t *pair0,
                          int64_t n_pairs, int dtype, const void *ybuf, int64_t n_slots, int64_t samples,
                          int64_t sample0, int64_t S, int log2m, const void *tw, void *cbuf, double *partial,
                          double *est, hipStream_t st) {
  if (n_nets == 0 || samples == 0) return TN_OK;
  if (samples > 65535) return set_error(TN_ERR_UNSUPPORTED, "combine: samples per launch");
  if (log2m < kMaxLog2Acc || log2m > kMaxLog2M1)
    return set_error(TN_ERR_ARG, "two-pass combine: m = 2^%d", log2m);
  if (n_pairs > 0x7fffffff) return set_error(TN_ERR_UNSUPPORTED, "two-pass combine: %lld tensor pairs",
                                             (long long)n_pairs);
  if (dtype == TN_F64)
    return combine_big<double>(n_nets, tslot, pairs, pair0, n_pairs, ybuf, n_slots, samples, sample0, S, log2m,
                               tw, cbuf, partial, est, st);
  return combine_big<float>(n_nets, tslot, pairs, pair0, n_pairs, ybuf, n_slots, samples, sample0, S, log2m, tw,
                            cbuf, partial, est, st);
}

int launch_m1_slots_to_tensors(const int32_t *tslot, int64_t n_tensors, int dtype,
                               const void *ybuf, int64_t n_slots, int64_t samples, int log2m,
                               double *out, hipStream_t st) {
  if (n_tensors == 0 || samples == 0) return TN_OK;
  dim3 grid((unsigned)n_tensors, (unsigned)samples);
  if (dtype == TN_F64)
    hipLaunchKernelGGL(slots_to_tensors_kernel<double>, grid, dim3(256), 0, st, tslot, n_tensors,
                       reinterpret_cast<const double *>(ybuf), n_slots, log2m, out);
  else
    hipLaunchKernelGGL(slots_to_tensors_kernel<float>, grid, dim3(256), 0, st, tslot, n_tensors,
                       reinterpret_cast<const float *>(ybuf), n_slots, log2m, out);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

int launch_twiddles(int64_t m, int dtype, void *out, hipStream_t st) {
  if (m < 2) return TN_OK;
  const unsigned blocks = (unsigned)((m / 2 + 255) / 256);
  if (dtype == TN_F64)
    hipLaunchKernelGGL(twiddle_kernel<double>, dim3(blocks), dim3(256), 0, st, m,
                       reinterpret_cast<double2 *>(out));
  else
    hipLaunchKernelGGL(twiddle_kernel<float>, dim3(blocks), dim3(256), 0, st, m,
                       reinterpret_cast<float2 *>(out));
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

int launch_sample_stats(const double *est, int64_t n_nets, int64_t S, double *stats,
                        hipStream_t st) {
  if (n_nets == 0) return TN_OK;
  hipLaunchKernelGGL(sample_stats_kernel, dim3((unsigned)n_nets), dim3(256), 0, st, est, S, stats);
  TN_HIP_CHECK(hipGetLastError());
  return TN_OK;
}

}  // namespace tn
