// Combine: direct reading of expert outputs from the windows and local weighted reduction in token
// order (paper, Section 5.2 "Prefill Combine", Section 5.3 "Decode Combine"; second loop of
// Algorithms 1 and 2):  Y[t,:] = sum_j W[t,j] * Yexp[row_map[t,j], :].
//
// Work unit = (token, 16-byte output column); workgroups of one to three waves or of a whole row or an equal part of one, or, for large launches, a
// persistent grid whose threads hold their results back until a round's loads are done.  A thread fetches its column from up to 8 window rows
// at once (8 independent 16-byte loads in flight per lane), folds them into fp32 accumulators in
// ascending j with one fused multiply-add per branch, rounds once and stores 16 bytes.  Every window
// row is read exactly once and Y is written exactly once, in token order: no un-permute buffer.
// Row ids and weights are uniform per workgroup and live in scalar registers.
#include <atomic>
#include <type_traits>
#include <utility>

#include "device_utils.h"
#include "launch.h"
#include "moe_rbf.h"

namespace moe_rbf {

constexpr int kGather = 8;  // rows fetched together
constexpr int kRowMost = 640;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// two bf16 packed in a dword -> two floats (exact)
__device__ __forceinline__ float bf16_lo(unsigned u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(unsigned u) { return __uint_as_float(u & 0xffff0000u); }
// two floats -> two bf16, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
  f32x2 f;
  f.x = lo;
  f.y = hi;
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}

template <int DT>
struct Acc;

template <>
struct Acc<MOE_DTYPE_BF16> {
  float a[8];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < 8; ++i) a[i] = 0.0f;
  }
  __device__ __forceinline__ void fma(float w, u32x4 y) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[2 * i] = __builtin_fmaf(w, bf16_lo(y[i]), a[2 * i]);
      a[2 * i + 1] = __builtin_fmaf(w, bf16_hi(y[i]), a[2 * i + 1]);
    }
  }
  __device__ __forceinline__ u32x4 result() const {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = pack_bf16(a[2 * i], a[2 * i + 1]);
    return r;
  }
};

template <>
struct Acc<MOE_DTYPE_F32> {
  float a[4];
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = 0.0f;
  }
  __device__ __forceinline__ void fma(float w, u32x4 y) {
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = __builtin_fmaf(w, __uint_as_float(y[i]), a[i]);
  }
  __device__ __forceinline__ u32x4 result() const {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __float_as_uint(a[i]);
    return r;
  }
};

// BLOCK: threads of a workgroup; kRowMost: as many as the launch says, up to that (whole rows, see launch_combine).
// KFIX > 0: the routing degree is the compile-time constant KFIX (straight-line code, no bounds tests, all rows at once; us per
// combine, rows taken 8 at a time / this: T = 300, H = 4096: k = 5 4.4 / 4.25, k = 10 6.9 / 6.3);
// KFIX == 0: any k, rows taken kGather at a time.
template <int BLOCK, int DT, int KFIX>
__global__ __launch_bounds__(BLOCK) void combine_rows_kernel(const u32x4 *__restrict__ Yexp,
                                                             const float *__restrict__ W,
                                                             const int32_t *__restrict__ row_map,
                                                             u32x4 *__restrict__ Y, int k_arg, int H16, int chunks) {
  const int k = KFIX > 0 ? KFIX : k_arg;
  const int t = blockIdx.x / chunks;
  const int c = blockIdx.x - t * chunks;
  const int col = c * (BLOCK == kRowMost ? (int)blockDim.x : BLOCK) + threadIdx.x;
  if (col >= H16) return;
  // both arrays are 16-byte aligned (checked at the boundary): lets the scalar loads be wide
  const int32_t *rows = (const int32_t *)__builtin_assume_aligned(row_map, 16) + (size_t)t * k;
  const float *w = (const float *)__builtin_assume_aligned(W, 16) + (size_t)t * k;
  const u32x4 *base = Yexp + col;
  Acc<DT> acc;
  acc.zero();
  constexpr int G = KFIX > 0 ? KFIX : kGather;
  for (int j0 = 0; j0 < k; j0 += G) {
    int row[G];
    float wj[G];
    u32x4 y[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const bool in = (KFIX > 0 && KFIX % G == 0) || j0 + u < k;
      row[u] = in ? uniform(rows[j0 + u]) : -1;
      wj[u] = in ? __uint_as_float(uniform(__float_as_uint(w[j0 + u]))) : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < G; ++u)
      y[u] = row[u] >= 0 ? load_stream(base + (size_t)row[u] * (size_t)H16) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < G; ++u)
      if (row[u] >= 0) acc.fma(wj[u], y[u]);
  }
  store_stream(Y + (size_t)t * (size_t)H16 + col, acc.result());
}

// Large launches: a persistent grid, one workgroup of 8 waves per compute unit, whose threads hold the results of up to
// 56 units and store them only after the last row load of the launch.  All waves run the same
// amount of work, so chip-wide the reads come first and the 11 % of writes follow in a burst instead of being
// mixed into the read stream (measured inside plan -> dispatch -> combine layers, H = 7168, k = 8, 28 units held:
// T = 4096 179.3-180.0 against 184.4-185.3 us per layer, T = 8192 351.6 / 360.4, Zipf T = 16384 676.6 / 681.3).
// Every change from reading to writing costs about 6 us (the CUs do not finish together, and the write burst has to start),
// so a thread holds as many results as the CU has room for: 36 in registers (144 of the 256 VGPRs that 8 waves may take)
// and 20 in the 160 KB of LDS, which are otherwise idle.  us per layer, X not cached, 28 units and two rounds per launch /
// up to 56 units and one: H = 7168: T = 5000 209.4 / 204.5, 6200 281 / 273, Zipf 16384 722 / 707; H = 4096: T = 11000
// 268 / 260.5, group-limited 32768 845 / 837.
// K: the routing degree; G: its rows that are in flight together.  Degrees of 10 and 5 take this form too, the former 5 rows at a time:
// us per combine, combine_rows_kernel / this with 2, 5, 8, 10 rows in flight: k = 10: H = 3456, T = 25255 341 / 381, 290, 304, 298; H = 2048,
// T = 12000 92 / 113, 87, -, -.  us per layer: k = 10: H = 7168, T = 8000 414 / 389; k = 5: H = 7168, T = 8000 230 / 226;
// H = 5120, T = 16000 358 / 351; not where many of the padded columns are idle (see launch_combine).  k = 8 with 4 rows in flight: H = 4096, T = 16000 388 / 384, but Zipf H = 7168, T = 16384 710 / 721;
// k = 6 with 3: 6 % slower.
// Same arithmetic as combine_rows_kernel
// (ascending j, one fma per placed branch, one rounding).  Units (token, column) are numbered token-major over
// columns padded to a multiple of 64, so that a wave stays inside one token: without the padding (H = 4104: 115
// against 95 us per combine) the row numbers are no longer scalar and every unit waits for them.
constexpr int kDeferBlock = 512;
constexpr int kDeferRegs = 36;     // results per thread held in registers ...
constexpr int kDeferLds = 20;      // ... and in LDS (all 160 KB)

// Straight-line repetition while f returns true (the loop is longer than what the compiler unrolls fully when asked).
// It is left at once where a wave has no unit left: to test and skip each of the remaining copies means as many jumps
// into code that is not cached, about 0.2 us each.
template <int... I, typename F>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F &&f) {
  (void)(f(std::integral_constant<int, I>{}) && ...);
}

template <int DT, int K, int G>
__device__ __forceinline__ u32x4 combine_unit(const u32x4 *__restrict__ Yexp, const float *__restrict__ wt,
                                              const int32_t *__restrict__ rm, int t, int col, int H16) {
  static_assert(K % G == 0, "whole rounds of rows");
  const int ts = uniform(t);
  const int32_t *rows = rm + (size_t)ts * K;
  const float *w = wt + (size_t)ts * K;
  Acc<DT> acc;
  acc.zero();
#pragma unroll
  for (int j0 = 0; j0 < K; j0 += G) {
    int row[G];
    float wj[G];
    u32x4 y[G];
#pragma unroll
    for (int u = 0; u < G; ++u) {
      row[u] = uniform(rows[j0 + u]);
      wj[u] = __uint_as_float(uniform(__float_as_uint(w[j0 + u])));
    }
#pragma unroll
    for (int u = 0; u < G; ++u)
      y[u] = row[u] >= 0 ? load_stream(Yexp + (size_t)row[u] * (size_t)H16 + col) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int u = 0; u < G; ++u)
      if (row[u] >= 0) acc.fma(wj[u], y[u]);
  }
  return acc.result();
}

template <int DT, int K, int G>
__global__ __launch_bounds__(kDeferBlock) void combine_deferred_kernel(const u32x4 *__restrict__ Yexp,
                                                                       const float *__restrict__ W,
                                                                       const int32_t *__restrict__ row_map,
                                                                       u32x4 *__restrict__ Y, int H16,
                                                                       int cols_pad, int units, int dq, int dr,
                                                                       int first, int in_lds) {
  // this launch covers units [first, units), at most in_lds + kDeferRegs a thread
  extern __shared__ u32x4 held[];
  const int nthreads = (int)gridDim.x * kDeferBlock;
  const int g = (int)blockIdx.x * kDeferBlock + (int)threadIdx.x;
  const int32_t *rm = (const int32_t *)__builtin_assume_aligned(row_map, 16);
  const float *wt = (const float *)__builtin_assume_aligned(W, 16);
  const long long u0 = (long long)first + g;
  const long long wave0 = (long long)first + (int)blockIdx.x * kDeferBlock + uniform((int)threadIdx.x & ~(kWave - 1));
  const int t0 = (int)(u0 / cols_pad), col0 = (int)(u0 - (long long)t0 * cols_pad);
  u32x4 res[kDeferRegs];
  long long u = wave0;                 // the wave's first unit: scalar
  int t = t0, col = col0;
  auto step = [&] {
    u += nthreads;
    col += dr;
    t += dq;
    if (col >= cols_pad) col -= cols_pad, ++t;
  };
#pragma unroll 1
  for (int r = 0; r < in_lds && u < units; ++r) {
    if (col < H16) held[r * kDeferBlock + threadIdx.x] = combine_unit<DT, K, G>(Yexp, wt, rm, t, col, H16);
    step();
  }
  unrolled(std::make_integer_sequence<int, kDeferRegs>{}, [&](auto r) {
    if (u >= units) return false;
    if (col < H16) res[r] = combine_unit<DT, K, G>(Yexp, wt, rm, t, col, H16);
    step();
    return true;
  });
  u = wave0, t = t0, col = col0;
#pragma unroll 1
  for (int r = 0; r < in_lds && u < units; ++r) {
    if (col < H16) store_stream(Y + (size_t)t * (size_t)H16 + col, held[r * kDeferBlock + threadIdx.x]);
    step();
  }
  unrolled(std::make_integer_sequence<int, kDeferRegs>{}, [&](auto r) {
    if (u >= units) return false;
    if (col < H16) store_stream(Y + (size_t)t * (size_t)H16 + col, res[r]);
    step();
    return true;
  });
}

// The form for at most 28 units a thread (one launch, no LDS): the loop that the compiler unrolls by itself, with the tests as
// lane masks.  us per layer, the form above / this one: k = 6: H = 7168, T = 3000 105.9 / 102.3, T = 4096 139.1 / 134.6;
// k = 8: H = 7168: T = 2400 107.1 / 106.4, 3584 155.1 / 154.3, 4096 175.8 / 175.8; H = 1024, T = 28000 178.9 /
// 178.1; H = 4104, T = 6300 176.0 / 174.2; fp32: H = 2056, T = 5000 138.8 / 138.2.  Not for more units: with 36 results the
// compiler keeps part of them in scratch memory (H = 7168: T = 4096 211, T = 4600 244 against 193).  The unit's code is written
// out and the loop over `base`, which runs once, stays: as a call of combine_unit the compiler schedules it otherwise, which costs
// fp32 rows up to 1.7 % (H = 3584, T = 4000, k = 6 132.7 / 134.8; H = 896, T = 9984, k = 8 111.1 / 112.4) and gains 0.5 % on
// bf16 rows of 14 KB; without the loop H = 896, T = 9984 takes 111.7 and bf16 rows move by 0.8 % either way.
constexpr int kRoundUnits = 28;

template <int DT, int K>
__global__ __launch_bounds__(kDeferBlock) void combine_round_kernel(const u32x4 *__restrict__ Yexp,
                                                                       const float *__restrict__ W,
                                                                       const int32_t *__restrict__ row_map,
                                                                       u32x4 *__restrict__ Y, int H16,
                                                                       int cols_pad, int units, int dq, int dr,
                                                                       int first) {
  // this launch covers units [first, units)
  constexpr int R = kRoundUnits, G = K;
  const int nthreads = (int)gridDim.x * kDeferBlock;
  const int g = (int)blockIdx.x * kDeferBlock + (int)threadIdx.x;
  const int32_t *rm = (const int32_t *)__builtin_assume_aligned(row_map, 16);
  const float *wt = (const float *)__builtin_assume_aligned(W, 16);
  for (long long base = first; base < units; base += (long long)nthreads * R) {
    const long long u0 = base + g;
    const int t0 = (int)(u0 / cols_pad), col0 = (int)(u0 - (long long)t0 * cols_pad);
    u32x4 res[R];
    int t = t0, col = col0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (u0 + (long long)r * nthreads < units && col < H16) {     // the first test is uniform per wave
        const int ts = uniform(t);
        const int32_t *rows = rm + (size_t)ts * K;
        const float *w = wt + (size_t)ts * K;
        Acc<DT> acc;
        acc.zero();
        for (int j0 = 0; j0 < K; j0 += G) {
          int row[G];
          float wj[G];
          u32x4 y[G];
#pragma unroll
          for (int u = 0; u < G; ++u) {
            row[u] = uniform(rows[j0 + u]);
            wj[u] = __uint_as_float(uniform(__float_as_uint(w[j0 + u])));
          }
#pragma unroll
          for (int u = 0; u < G; ++u)
            y[u] = row[u] >= 0 ? load_stream(Yexp + (size_t)row[u] * (size_t)H16 + col) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
          for (int u = 0; u < G; ++u)
            if (row[u] >= 0) acc.fma(wj[u], y[u]);
        }
        res[r] = acc.result();
      }
      col += dr;
      t += dq;
      if (col >= cols_pad) col -= cols_pad, ++t;
    }
    t = t0, col = col0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (u0 + (long long)r * nthreads < units && col < H16) store_stream(Y + (size_t)t * (size_t)H16 + col, res[r]);
      col += dr;
      t += dq;
      if (col >= cols_pad) col -= cols_pad, ++t;
    }
  }
}

// Compute units of the current device (asked once per device; no allocation).  Calls may come from several host
// threads: the cache holds the same value whoever fills it.
static int device_cus() {
  static std::atomic<int> cus[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cus[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) n = 256;
    cus[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

template <int DT>
static hipError_t launch_combine_deferred(const Dims &d, const void *expert_out, const float *W, const PlanView &p,
                                          void *y, int cols_pad, int units, hipStream_t s) {
  const int grid = device_cus();
  const int nthreads = grid * kDeferBlock;
  const long long per_thread = ((long long)units + nthreads - 1) / nthreads;
  if (per_thread <= kRoundUnits && (d.k == 8 || d.k == 6)) {
    auto once = [&](auto kernel) {
      return launch(kernel, dim3(grid), dim3(kDeferBlock), 0, s, (const u32x4 *)expert_out, W, (const int32_t *)p.row_map,
                    (u32x4 *)y, d.H16, cols_pad, units, nthreads / cols_pad, nthreads % cols_pad, 0);
    };
    return d.k == 8 ? once(combine_round_kernel<DT, 8>) : once(combine_round_kernel<DT, 6>);
  }
  // As few launches as can hold all results, of equal length.
  const long long launches = (per_thread + kDeferRegs + kDeferLds - 1) / (kDeferRegs + kDeferLds);
  const int each = (int)((per_thread + launches - 1) / launches);
  const int in_lds = each > kDeferRegs ? each - kDeferRegs : 0;
  const size_t lds = (size_t)in_lds * kDeferBlock * sizeof(u32x4);
  auto go = [&](auto kernel, RaisedOn &raised) {
    if (lds > 64 * 1024) {
      const hipError_t e = raise_lds_limit((const void *)kernel, kDeferLds * kDeferBlock * (int)sizeof(u32x4), raised);
      if (e != hipSuccess) return e;
    }
    const long long per = (long long)nthreads * each;
    for (long long first = 0; first < units; first += per) {
      const long long end = first + per < units ? first + per : units;
      const hipError_t e = launch(kernel, dim3(grid), dim3(kDeferBlock), lds, s, (const u32x4 *)expert_out, W,
                                  (const int32_t *)p.row_map, (u32x4 *)y, d.H16, cols_pad, (int)end,
                                  nthreads / cols_pad, nthreads % cols_pad, (int)first, in_lds);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  };
  static RaisedOn raised10, raised8, raised6, raised5;
  switch (d.k) {
    case 10: return go(combine_deferred_kernel<DT, 10, 5>, raised10);
    case 8: return go(combine_deferred_kernel<DT, 8, 8>, raised8);
    case 6: return go(combine_deferred_kernel<DT, 6, 6>, raised6);
    case 5: return go(combine_deferred_kernel<DT, 5, 5>, raised5);
    default: return hipErrorInvalidValue;      // other routing degrees keep combine_rows_kernel (see launch_combine)
  }
}

// Waves of a workgroup that takes a whole row, or an equal part of one of more than 10 waves (of 3 waves or more, where that leaves none
// idle).
static int row_waves(int waves) {
  const int most = kRowMost / kWave;
  for (int w = most; w >= 3; --w)
    if (waves % w == 0) return w;
  const int parts = (waves + most - 1) / most;
  return (waves + parts - 1) / parts;
}

// B: threads of a workgroup, or kRowMost: row_waves
template <int DT, int B>
static hipError_t launch_combine_dt(const Dims &d, const void *expert_out, const float *W, const PlanView &p, void *y,
                                    hipStream_t s) {
  const int block = B == kRowMost ? row_waves((d.H16 + kWave - 1) / kWave) * kWave : B;
  const int chunks = (d.H16 + block - 1) / block;
  const dim3 grid((unsigned)d.T * (unsigned)chunks);
  if (B == kRowMost && (uint64_t)grid.x * (unsigned)block > kMostThreads)
    return launch_combine_dt<DT, 128>(d, expert_out, W, p, y, s);
  auto go = [&](auto kernel) {
    return launch(kernel, grid, dim3((unsigned)block), 0, s, (const u32x4 *)expert_out, W, (const int32_t *)p.row_map, (u32x4 *)y,
                  d.k, d.H16, chunks);
  };
  switch (d.k) {
    case 10: return go(combine_rows_kernel<B, DT, 10>);
    case 8: return go(combine_rows_kernel<B, DT, 8>);
    case 6: return go(combine_rows_kernel<B, DT, 6>);
    case 5: return go(combine_rows_kernel<B, DT, 5>);
    case 4: return go(combine_rows_kernel<B, DT, 4>);
    case 3: return go(combine_rows_kernel<B, DT, 3>);
    case 2: return go(combine_rows_kernel<B, DT, 2>);
    case 1: return go(combine_rows_kernel<B, DT, 1>);
    default: return go(combine_rows_kernel<B, DT, 0>);
  }
}

// Does a launch that does not hold its results back take workgroups of whole rows?  Rows that are no multiple of a line: a wave's 1 KB
// shares its first and last line with its neighbours, which a workgroup of the whole row finds in the compute unit's cache.  Rows with idle
// columns: fewer workgroups.  Against it: the launch lasts as long as the compute unit with the most rows, and 262 rows on 256 units are
// uneven where 262 times 9 one-wave workgroups are not.  So rows of 5 waves and more take it from 2.4 M window vectors and 2.5 workgroups a
// compute unit on, from 1.7 M where the last workgroups nearly fill the units, or where a row is little work.
// us per layer, one wave (T * H16 <= 1.5 M) or two / the row; the second pair, if any, with expert_out rotating through 600 MB instead of
// the same in each layer:
//   not taken: H = 4104, k = 8: T = 262 12.3 / 13.1, 12.2 / 12.9, 372 15.3 / 15.6, 15.4 / 15.4; H = 5000: k = 8, T = 304 15.1 / 16.0, 15.1 / 15.8, k = 4,
//     T = 655 17.3 / 17.8, 17.5 / 17.2, k = 2, T = 960 15.7 / 16.0, 15.4 / 15.6; H = 8200, k = 10, T = 142 14.5 / 15.7; H = 10800, k = 8, T = 96 11.2 / 12.1;
//   taken: H = 2664, k = 8, T = 700 (2.7 a unit) 21.1 / 20.4; H = 4104: k = 8, T = 455 (1.8) 18.1 / 17.6, T = 797 31.1 / 30.8, 1170 42.4 / 40.9, k = 6, T = 3001 73.8 / 70.5, k = 4, T = 1717 35.6 / 34.0; H = 10800, k = 8, T = 1156 85.8 / 83.5;
//     little work: k = 2: H = 4104, T = 543 10.9 / 10.5, H = 5000, T = 172 8.7 / 8.5; k = 1, H = 4104, T = 543 13.1 / 12.3;
//     up to 4 waves: H = 1032, k = 8, T = 2159 27.2 / 26.3; H = 1544, k = 8, T = 3109 45.3 / 43.1; H = 520, k = 8, T = 13549 71.8 / 65.2;
//   rows of whole lines with idle columns: taken: H = 576, k = 8, T = 2636 20.5 / 19.2; H = 1664, k = 4, T = 9122 61.9 / 60.7; k = 1: H = 1152, T = 1318
//     8.9 / 8.4, H = 2112, T = 719 8.7 / 8.1; not (3 or 5 waves): H = 1152: k = 8, T = 898 14.2 / 14.5, k = 2, T = 4167 19.8 / 20.1; H = 2112: k = 2, T = 2273
//     15.8 / 16.5, k = 1, T = 3800 17.1 / 17.5.
// Known losses, up to 2.5 %: 1 shape in 80, most of them rows of 11 waves as 2 times 6 with expert_out written just in front of combine (H = 5128, k = 8, T = 700 54.5 / 55.4 with that copy; else 32.2 / 32.0).
// Rows of whole lines and waves: no gain (H = 2048, T = 5000, k = 6 27.7 / 28.4 a combine).
static bool whole_rows(const Dims &d, int waves, bool ragged, bool idle) {
  const int64_t vecs = (int64_t)d.T * d.H16, window = vecs * d.k;
  if (!(ragged || idle) || vecs < 100000) return false;
  if (waves <= 2 || (d.k <= 2 && window < 600000) || (ragged && waves <= 4) || (d.k == 1 && (ragged || waves == 4))) return true;
  if (!ragged && waves != 4) return false;
  const int w = row_waves(waves);
  const int64_t cus = device_cus(), groups = (int64_t)d.T * ((waves + w - 1) / w), even = (groups + cus - 1) / cus * cus;   // workgroups, and as many to each unit
  return (window >= 2400000 && groups * 2 >= cus * 5) ||
         (d.k > 2 && window >= 1700000 && groups * 4 >= cus * 7 && groups * 20 >= even * 17);
}

hipError_t launch_combine(const Dims &d, const void *expert_out, const float *W, const PlanView &p, void *y,
                          hipStream_t s) {
  // One-wave workgroups while the launch is small (latency-bound: every wave starts as early as possible),
  // two-wave workgroups once it streams.  Measured, H = 7168, k = 8, 64 / 128 threads: T = 128: 4.61 / 4.74 us,
  // T = 1024: 22.5 / 22.7, T = 2048: 43.1 / 43.0, T = 4096: 88.1 / 86.9.
  const bool small = (int64_t)d.T * d.H16 <= (int64_t)1536 * 1024;
  // Streaming launches with a routing degree of 5, 6, 8 or 10 take the deferred-store form.  Measured inside layers,
  // us per layer deferred / not: H = 7168: T = 2048 91.5 / 92.2, 3072 136.2 / 138.3, 4096 180.4 / 185.2,
  // 6144 264.9 / 267.7, 8192 348.1 / 355.2, 16384 702.9 / 713.1, Zipf 16384 673.5 / 681.8; H = 4096: T = 4096
  // 103.4 / 104.3, 16384 380.2 / 387.5, group-limited 32768 846.6 / 848.5; degrees of 5 and 10: see there; k = 4: T = 4096
  // 104.1 / 103.4, H = 2176, T = 24000 96 / 86 (a combine), k = 3: H = 7168, T = 8000 83 / 74 (smaller degrees, and degrees without a
  // compile-time form, whose results array the compiler would spill, stay).
  // The others: rows of an odd number of waves that is a multiple of 3 take workgroups of 3 waves, so that no workgroup is half
  // idle.  us per layer, 2 waves / 3: T = 20000: H = 1152: k = 1 50.8 / 48.2, k = 3 73.2 / 68.4, k = 5 104.9 / 98.5; H = 1536, k = 4 109.3 / 105.9.
  // (Of 5 or 7 where a row of whole lines has as many: no gain.  The columns past the last whole wave of several tokens packed into one wave:
  // H = 4104, k = 6 33.3 / 34.3 a combine.)
  const int cols_pad = (d.H16 + 63) / 64 * 64, waves = cols_pad / kWave;
  const bool threes = waves % 2 == 1 && waves % 3 == 0;
  // Results are held back only where few padded columns are idle, judged inside layers: alone in a loop the held form reads better than it is,
  // since the rest of the layer is slower behind it.  us per layer, held / rows of whole workgroups (see whole_rows):
  //   k = 10 (a third of the row idle at most): H = 704, T = 29545 174.5 / 166.2, 1032, T = 20155 200.3 / 194.2, but 800, T = 55000 371.0 / 376.3, 1280, T = 16250
  //     157.6 / 160.5, 2056, T = 10116 171.5 / 174.9, 4104, T = 5068 168.6 / 173.4, 5128, T = 4056 161.3 / 177.0;
  //   k = 5 (a seventh): H = 1664, T = 12500 95.3 / 91.4, 2056, T = 10116 103.5 / 98.6, 4104, T = 5068 101.7 / 97.5 (this line was drawn for rows of 1 to 3 waves a
  //     workgroup; ragged rows would still gain: H = 1800, T = 11555 103.9 / 100.1, 5000, T = 4160 97.8 / 95.6, but 5128, T = 4056 97.3 / 98.9);
  //   k = 8 (three eighths): H = 320, T = 80000 170.0 / 167.8, 352 189.5 / 195.8; 520, T = 60000 270.9 / 259.7, 576, T = 40000 158.2 / 149.9, 640 162.1 / 159.8, 672 171.7 /
  //     172.5, 1032, T = 20000 159.1 / 160.4;
  //   k = 6 (a fifth, of one wave a quarter): H = 384, T = 60000 119.2 / 116.6, but 400, T = 52000 136.7 / 140.1, 432, T = 48148 133.7 / 138.4; 520, T = 60000 223.5 / 198.2,
  //     576, T = 40000 134.3 / 119.3, 768, T = 60000 235.0 / 227.9, 1152, T = 18055 107.9 / 105.8, 1216, T = 17105 105.7 / 105.0, but 832, T = 25000 105.2 / 106.5, 1280, T = 16250
  //     104.4 / 105.3, 2176: T = 9558 103.1 / 105.0, T = 20000 208.5 / 212.6; rows of 2 waves and more that are no multiple of a line from a tenth on:
  //     2056, T = 30000 343.3 / 332.8, 4104: T = 5068 113.0 / 112.5, T = 18600 403.6 / 396.2, 2664: T = 7807 112.3 / 112.8, T = 15600 220.6 / 216.7 (of one wave, which share
  //     no line inside the row: 456, T = 45614 140.2 / 144.3).
  const bool ragged = d.H16 % 8 != 0 || ((uintptr_t)expert_out >> 4) % 8 != 0;
  const int pad = cols_pad - d.H16;
  const bool idle = pad * 20 >= cols_pad * 3;
  const bool held = (d.k == 8 && cols_pad * 5 < d.H16 * 8) ||
                    (d.k == 6 && pad * (waves == 1 ? 4 : 5) < cols_pad && !(ragged && waves > 1 && pad * 10 >= cols_pad)) ||
                    (d.k == 10 && cols_pad * 3 <= d.H16 * 4) ||
                    (d.k == 5 && !threes && cols_pad * 7 <= d.H16 * 8 && d.H16 >= 60);
  const long long units = (long long)d.T * cols_pad;
  if (!small && held && units < 0x7fffffffLL)
    return d.dtype == MOE_DTYPE_BF16
               ? launch_combine_deferred<MOE_DTYPE_BF16>(d, expert_out, W, p, y, cols_pad, (int)units, s)
               : launch_combine_deferred<MOE_DTYPE_F32>(d, expert_out, W, p, y, cols_pad, (int)units, s);
  auto rows = [&](auto dtype) {
    constexpr int DT = decltype(dtype)::value;
    if (whole_rows(d, waves, ragged, idle)) return launch_combine_dt<DT, kRowMost>(d, expert_out, W, p, y, s);
    if (small) return launch_combine_dt<DT, 64>(d, expert_out, W, p, y, s);
    return threes ? launch_combine_dt<DT, 192>(d, expert_out, W, p, y, s) : launch_combine_dt<DT, 128>(d, expert_out, W, p, y, s);
  };
  return d.dtype == MOE_DTYPE_BF16 ? rows(std::integral_constant<int, MOE_DTYPE_BF16>{})
                                   : rows(std::integral_constant<int, MOE_DTYPE_F32>{});
}

}  // namespace moe_rbf
