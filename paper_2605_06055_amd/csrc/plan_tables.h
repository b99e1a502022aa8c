// Shared device code of the two schedules: turning per-expert counts into the plan's count / offset
// tables (paper, Section 5.2 "Prefill Notify"; Section 5.1, definition of the large offset o_{e,r}).
//
// Layout of the window: destination rank d owns a region; inside it the blocks of its experts follow
// each other; inside an expert's block the sub-blocks of the source ranks follow each other in rank
// order.  With
//   own[e]    = branches this rank sends to expert e                     (c^exp)
//   pre[e]    = branches the source ranks BELOW this one send to e       (column sum of M over rows < me)
//   post[e]   = branches the source ranks ABOVE this one send to e       (column sum of M over rows > me)
//   g         = exclusive scan over e of own + pre + post
// the block of expert e starts at  B[e] = region_start(d) + g[e] - g[d*E_r]  and this rank's sub-block at
// o_{e,me} = B[e] + pre[e].  With one source rank pre = post = 0.
//
// Row numbers are int32.  With several sources the row total is device data (the sum of M); it is also
// accumulated in 64 bits, and when it reaches 2^31 no branch is placed and status[2] reports it.
#pragma once
#include "device_utils.h"
#include "launch.h"

namespace moe_rbf {

// First window row of expert e's whole block.  g = exclusive scan of the block sizes over ALL experts.
// Tight windows: region r starts where the previous one ends, so B[e] = g[e].
// Fixed stride : region r starts at r*stride and expert blocks are packed from there.
__device__ __forceinline__ int expert_first_row(const int *g, int e, const Dims &d) {
  if (d.stride <= 0) return g[e];
  const int r = e / d.Er;
  return (int)(r * d.stride) + g[e] - g[r * d.Er];
}

// First row past the rank region that holds expert e (no limit for tight windows).
__device__ __forceinline__ int region_row_limit(int e, const Dims &d) {
  return d.stride > 0 ? (int)((e / d.Er + 1) * d.stride) : 0x7fffffff;
}

// a / b for 0 <= a < 2^20, 0 < b <= 1024 and quotients below 1024 or so: the error of the reciprocal stays below the 0.5 / b that is
// between the exact value and the next integer.
__device__ __forceinline__ int small_div(int a, int b) {
  return (int)(((float)a + 0.5f) * __builtin_amdgcn_rcpf((float)b));
}

// Rows of the other source ranks: column sums of M (R x E) below and above this rank's row, added up in LDS by all threads of a
// workgroup of at least 512.  What bounds it is the round trip, and the instructions that every workgroup repeats: a thread takes
// four columns (16-byte loads, all of them in flight for 32 ranks and 256 experts) over a run of consecutive ranks on one side of
// this one, so that it adds to one array only.  (Where rows are not whole pieces of 16 bytes: one column at a time.)
// us per decode dispatch, 32 sources, E = 256, k = 8, H = 7168, with a column per thread, two sums and a 64-bit one for each element and
// reductions over the wave for each slot / now: T = 1 5.3 / 4.7, 64 6.0 / 5.3, 128 7.35 / 6.4, 512 18.2 / 14.0; plan of 5870 branches,
// E = 64 8.15 / 6.8, of 32 768 13.0 / 11.7.
struct SourceSums {
  static constexpr int kRows = 4;        // rows requested together
  static constexpr int kShort = 128;     // rows of a run whose total needs 32 bits only, if its elements are below 2^15
  u32x4 v[kRows];
  int quad, first, end;                  // four columns, and the run of ranks
  bool below;

  __device__ __forceinline__ void load(const int32_t *__restrict__ M, const Dims &d, int r) {
#pragma unroll
    for (int u = 0; u < kRows; ++u)
      v[u] = r + u < end ? ((const u32x4 *)(M + (size_t)(r + u) * (size_t)d.E))[quad] : u32x4{0u, 0u, 0u, 0u};
  }
  __device__ __forceinline__ void request(const int32_t *__restrict__ M, const Dims &d) {
    first = end = 0;
    if (d.E % 4 != 0) return;
    const int quads = d.E >> 2, parts = small_div((int)blockDim.x, quads);     // E <= 1024: at least two parts
    const int part = small_div((int)threadIdx.x, quads);
    quad = (int)threadIdx.x - part * quads;
    const int lower = d.me, upper = d.R - 1 - d.me;            // ranks on the two sides
    const int parts_below = lower == 0 ? 0 : upper == 0 ? parts : min(max(small_div(parts * lower, d.R - 1), 1), parts - 1);
    below = part < parts_below;
    const int n = below ? lower : upper, share = below ? parts_below : parts - parts_below, start = below ? 0 : d.me + 1;
    const int each = n > 0 ? small_div(n + share - 1, share) : 0;
    first = start + (below ? part : part - parts_below) * each;
    end = part < parts ? min(start + n, first + each) : first;
    load(M, d, first);
  }
  // pre[e], post[e] += the sums; they start at zero.  Returns the wave's total plus that of `more`, exact below 2^31 (and at
  // least 2^31 otherwise).
  __device__ __forceinline__ unsigned long long add(const int32_t *__restrict__ M, const Dims &d, int *pre, int *post, int more) {
    u32x4 sum = {0u, 0u, 0u, 0u};
    unsigned any = d.E % 4 != 0 || end - first > kShort ? ~0u : 0u;
    for (int r = first; r < end; r += kRows) {
      if (r > first) load(M, d, r);
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i] += v[0][i] + v[1][i] + v[2][i] + v[3][i];
#pragma unroll
      for (int u = 0; u < kRows; ++u) any |= v[u][0] | v[u][1] | v[u][2] | v[u][3];
    }
    if (first < end) {
      int *to = (below ? pre : post) + 4 * quad;
#pragma unroll
      for (int i = 0; i < 4; ++i) atomicAdd(to + i, (int)sum[i]);
    }
    if (__ballot(any >= 1u << 15) == 0)
      return (unsigned)__builtin_amdgcn_readlane(
          wave_inclusive_scan((int)(sum[0] + sum[1] + sum[2] + sum[3]) + more), kWave - 1);
    return add_wide(M, d, pre, post, more);
  }
  // The total in 64 bits, from memory again; where rows are not whole pieces of 16 bytes, the sums too.
  __device__ __forceinline__ unsigned long long add_wide(const int32_t *__restrict__ M, const Dims &d, int *pre, int *post,
                                                         int more) {
    unsigned wide = (unsigned)more;
    if (d.E % 4 != 0) {
      for (int col = (int)threadIdx.x; col < d.E; col += (int)blockDim.x) {
        int low = 0, high = 0;
#pragma unroll 8
        for (int r = 0; r < d.R; ++r) {
          const int n = r != d.me ? M[(size_t)r * d.E + col] : 0;
          (r < d.me ? low : high) += n;
          wide = __builtin_elementwise_add_sat(wide, (unsigned)n);
        }
        pre[col] = low, post[col] = high;
      }
    } else {
      for (int r = first; r < end; ++r) {
        const u32x4 n = ((const u32x4 *)(M + (size_t)r * (size_t)d.E))[quad];
#pragma unroll
        for (int i = 0; i < 4; ++i) wide = __builtin_elementwise_add_sat(wide, n[i]);
      }
    }
    return wave_sum_u64(wide);
  }
};

// The sums of a requested SourceSums; rows (LDS, zeroed by the caller) += the total in 64 bits.
__device__ __forceinline__ void add_sources(SourceSums &sums, const int32_t *__restrict__ M, const Dims &d, int *pre, int *post,
                                            unsigned long long *rows) {
  const unsigned long long wave_rows = sums.add(M, d, pre, post, 0);
  if (lane_id() == 0 && wave_rows) atomicAdd(rows, wave_rows);
}

// Tile histograms in the plan's workspace.  PACKED: 16-bit counts, rows of round4(E + 1) of them (8-byte pieces; never more bytes than
// E + 1 words): for tiles of fewer than 2^16 branches.  Otherwise words, rows of E + 1.  Slot E counts the invalid ids.
template <bool PACKED>
__device__ __host__ __forceinline__ int hist_pitch(int E) { return PACKED ? (E + 4) / 4 * 2 : E + 1; }     // in words

// Sums the tile histograms over four ranges of tiles, [0, b0), [b0, b1), [b1, b2), [b2, tiles), into sums[range * (E + 1) + e] (LDS, zeroed
// by the caller, who also synchronises) with all threads of the workgroup.  Every workgroup of the plan's second launch reads all
// histograms, so what bounds it is the instructions and round trips per row: a thread takes four columns in one 8-byte piece over a
// run of consecutive tiles, adds them in pairs of 16 bits, and adds to LDS only where a range or its run ends (or before a count can
// pass 16 bits).  us per plan, one column per thread with a select per row and range / now (with the bank conflicts of the wave
// prefix gone, see plan_rank_kernel): 32 768 branches, E = 256 10.7 / 9.2, E = 512 14.2 / 10.7; 82 560, E = 512 20.0 / 12.9; 131 072, E = 128
// 13.5 / 11.7, E = 1024 34.4 / 21.9.
template <bool PACKED>
__device__ __forceinline__ void sum_tile_hists(const int32_t *__restrict__ hist, int tiles, int tile, int E, int b0, int b1, int b2,
                                               int *sums) {
  constexpr int kWords = PACKED ? 2 : 1, kBatch = 8;           // tiles requested together
  const int pitch = hist_pitch<PACKED>(E), cols = pitch / kWords;
  const int nthreads = (int)blockDim.x;
  const int parts = max(1, nthreads / cols);
  const int part = parts > 1 ? small_div((int)threadIdx.x, cols) : 0;
  if (part >= parts) return;
  const int each = (tiles + parts - 1) / parts;
  const int most = PACKED ? 65535 / tile : 0x7fffffff;         // rows whose packed sums fit
  const int first = part * each, end = min(tiles, first + each);
  for (int col = (int)threadIdx.x - part * cols; col < cols; col += nthreads) {
    const unsigned *src = (const unsigned *)hist + (size_t)col * kWords;
    unsigned acc[kWords] = {}, v[kBatch][kWords];
    int held = 0;
    auto flush = [&](int r) {                                  // rows up to r - 1 are in acc
      int *to = sums + (r <= b0 ? 0 : r <= b1 ? 1 : r <= b2 ? 2 : 3) * (E + 1) + col * (PACKED ? 4 : 1);
#pragma unroll
      for (int w = 0; w < kWords; ++w) {
        if (!PACKED) atomicAdd(to, (int)acc[w]);
        else if (acc[w]) {                                     // (the padding past slot E stays zero)
          if (acc[w] & 0xffffu) atomicAdd(to + 2 * w, (int)(acc[w] & 0xffffu));
          if (acc[w] >> 16) atomicAdd(to + 2 * w + 1, (int)(acc[w] >> 16));
        }
        acc[w] = 0;
      }
      held = 0;
    };
    for (int r0 = first; r0 < end; r0 += kBatch) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
#pragma unroll
        for (int w = 0; w < kWords; ++w) v[u][w] = r0 + u < end ? src[(size_t)(r0 + u) * pitch + w] : 0u;
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int r = r0 + u;
        if (r < end) {
          if (held > 0 && (r == b0 || r == b1 || r == b2 || held == most)) flush(r);
#pragma unroll
          for (int w = 0; w < kWords; ++w) acc[w] += v[u][w];  // no carry between the halves
          ++held;
        }
      }
    }
    if (held > 0) flush(end);
  }
}

// Do the rows of all sources together reach 2^31?  others_rows: 64-bit sum of the other sources' counts;
// all_rows_low: the int32 sum (possibly wrapped) of own and others; this rank's own count is below 2^31, so
// it is the difference of the two low words.
__device__ __forceinline__ bool rows_overflow(unsigned long long others_rows, int all_rows_low) {
  const unsigned own = (unsigned)all_rows_low - (unsigned)others_rows;
  return others_rows + own >= (1ull << 31);
}

// One workgroup writes expert_count, rank_count, expert_offset, region_base, recv_count, recv_offset and
// status from LDS copies of own[0..E), pre (nullptr with a single
// source rank) and g[0..E].  Must be called by every thread of the workgroup.
// Branches dropped for capacity: this rank's sub-block of expert e covers rows [o, o + own); the part at
// or past the region's end is dropped.  overflow: the row total does not fit in int32 (the offset tables
// are then meaningless and status[2] says so).
__device__ __forceinline__ void write_plan_tables(const int *own, const int *pre, const int *g,
                                                  const Dims &d, const PlanView &p, int n_invalid, int *lds_counter,
                                                  bool overflow = false) {
  const int nthreads = blockDim.x;
  const bool fixed = d.stride > 0;
  if (threadIdx.x == 0) *lds_counter = 0;
  __syncthreads();
  int dropped = 0;
  for (int e = threadIdx.x; e < d.E; e += nthreads) {
    const int c = own[e];
    const int block = expert_first_row(g, e, d);
    const int o = block + (pre ? pre[e] : 0);
    const int all = g[e + 1] - g[e];                                    // own and the other sources'
    p.expert_count[e] = c;
    p.expert_offset[e] = o;
    if (p.recv_count) p.recv_count[e] = all;
    if (p.recv_offset) p.recv_offset[e] = block;
    if (fixed) dropped += min(c, max(0, o + c - region_row_limit(e, d)));
    if (e == d.E - 1) {
      p.expert_offset[d.E] = block + all;
      if (p.recv_offset) p.recv_offset[d.E] = block + all;
      p.region_base[d.R] = fixed ? (int)(d.R * d.stride) : g[d.E];
    }
  }
  for (int r = threadIdx.x; r < d.R; r += nthreads) {
    p.region_base[r] = fixed ? (int)(r * d.stride) : g[r * d.Er];
    if (!pre) p.rank_count[r] = g[(r + 1) * d.Er] - g[r * d.Er];     // own counts are all there is in g
  }
  // With several sources g also counts the other ranks' rows, so the own counts of a rank's experts are summed here,
  // one wave per rank.  (One thread per rank was a chain of E_r dependent LDS reads that the whole launch waited
  // for: with R = 1 the decode dispatch of 222 tokens of H = 2048 took 13.1 us at E = 256 and the plan of 24 576 branches
  // 28.8 us at E = 512, against 5.5 and 12.5 us now, in replayed graphs.)
  if (pre) {
    for (int r = threadIdx.x / kWave; r < d.R; r += nthreads / kWave) {
      int c = 0;
      for (int e = r * d.Er + lane_id(); e < (r + 1) * d.Er; e += kWave) c += own[e];
      c = __builtin_amdgcn_readlane(wave_inclusive_scan(c), kWave - 1);
      if (lane_id() == 0) p.rank_count[r] = c;
    }
  }
  if (dropped) atomicAdd(lds_counter, dropped);
  __syncthreads();
  if (threadIdx.x == 0) {
    p.status[0] = n_invalid;
    p.status[1] = overflow ? 0 : *lds_counter;
    p.status[2] = overflow ? 1 : 0;
  }
}

// The routing ids of a workgroup, requested in pieces of 16 bytes.  Piece q holds ids 4q..4q+3; past the last id: -1.
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ i32x4 load_ids(const int32_t *__restrict__ K, int q, int N) {
  const int i = 4 * q;
  if (i + 4 <= N) return ((const i32x4 *)K)[q];
  i32x4 v = {-1, -1, -1, -1};
  if (i < N) v[0] = K[i];
  if (i + 1 < N) v[1] = K[i + 1];
  if (i + 2 < N) v[2] = K[i + 2];
  return v;
}

// One workgroup builds the whole histogram from the routing ids themselves (counts only: LDS integer
// atomics) and writes the tables.  Used where no per-tile histograms exist: the fused decode dispatch and
// the single-launch plan.  LDS: 4E + 3 ints.  Must be called by every thread of the workgroup; with several source ranks one of at least
// 512 threads (SourceSums), as the plan and the histogram kernel of the decode dispatch have.
// The launch waits for this workgroup, so the next trip's ids are requested ahead of this one's counting.
__device__ __forceinline__ void tables_from_ids_block(const int32_t *__restrict__ K, const Dims &d, const PlanView &p,
                                                    int *lds) {
  const int E = d.E, tid = threadIdx.x, nthreads = blockDim.x;
  int *total = lds;            // [E]
  int *g = total + E;          // [E+1]
  int *pre = g + E + 1;        // [E]  several source ranks only
  int *post = pre + E;         // [E]
  int *misc = post + E;        // [2]
  __shared__ unsigned long long others_rows;
  const bool multi = p.source_count != nullptr;
  const bool few = d.N <= nthreads;      // one id a thread: shorter code, 0.3 us less for a batch of one token
  const int only = few && tid < d.N ? K[tid] : -1;
  i32x4 next = few ? i32x4{-1, -1, -1, -1} : load_ids(K, tid, d.N);
  SourceSums sums;
  if (multi) sums.request(p.source_count, d);
  for (int e = tid; e < E; e += nthreads) {
    total[e] = 0;
    pre[e] = 0;
    post[e] = 0;
  }
  if (tid == 0) misc[0] = 0, others_rows = 0;
  __syncthreads();
  auto count = [&](int e) {
    if ((unsigned)e < (unsigned)E) atomicAdd(&total[e], 1);
    else if (e != -1) atomicAdd(&misc[0], 1);
  };
  if (few) {
    count(only);
  } else {
#pragma unroll 1
    for (int q = tid; 4 * q < d.N; q += nthreads) {
      const i32x4 ids = next;
      next = load_ids(K, q + nthreads, d.N);
#pragma unroll
      for (int n = 0; n < 4; ++n) count(ids[n]);
    }
  }
  if (multi) add_sources(sums, p.source_count, d, pre, post, &others_rows);
  __syncthreads();
  exclusive_scan_lds([&](int e) { return total[e] + (multi ? pre[e] + post[e] : 0); }, g, E, uniform(tid / kWave), nthreads / kWave);
  __syncthreads();
  write_plan_tables(total, multi ? pre : nullptr, g, d, p, misc[0], misc + 1, multi && rows_overflow(others_rows, g[E]));
}

}  // namespace moe_rbf
