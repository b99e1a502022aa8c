// Prefill Layout + Notify for one source rank (paper, Section 5.2): per-expert and per-rank branch
// counts, large offsets o (exclusive scan of the counts inside each rank region), the stable small
// offset s of every branch and the row map o[K] + s.  No payload is touched.
//
// The small offset must be the number of EARLIER branches (smaller flat index t*k+j) with the same
// expert, so it cannot come from global atomics (arbitrary order).  It is built from counts per tile
// and a prefix over the tiles in front, the scheme the paper names for its Layout kernel:
//   pass 1  plan_tile_hist : one workgroup per tile of branches -> LDS histogram -> tile_hist[tile][E+1]
//                            (slot E counts ids outside [0,E) other than -1)
//   pass 2  plan_rank      : one workgroup (16 waves) per tile.  Column sums of tile_hist over earlier
//                            tiles give the tile's starting count per expert; every workgroup also forms
//                            the totals and their exclusive scan (cheap, E <= 1024), so there is no third
//                            launch.  Each wave owns a contiguous segment of the tile; segment histograms
//                            are prefix-summed over the waves with a DPP row scan, and inside a wave the
//                            rank among lanes holding the same id comes from ballots.  Integer LDS atomics
//                            are used for COUNTS only, which do not depend on order.  One extra workgroup
//                            writes the count/offset tables.
// Both kernels are latency-bound (a few microseconds): loads are requested before LDS is cleared and
// the serial chain is kept to three barriers.  Small batches skip pass 1.
#include "device_utils.h"
#include "launch.h"
#include "plan_tables.h"

namespace moe_rbf {

constexpr int kPlanBlock = 1024;                  // 16 waves
constexpr int kPlanWaves = kPlanBlock / kWave;
constexpr int kPlanMinTile = kPlanBlock;          // one branch per thread
constexpr int kPlanMaxTiles = 512;
constexpr int kCopies = 4;                        // of each count of a single-launch plan
__device__ __forceinline__ int sum4(const int *p) {
  const i32x4 v = *(const i32x4 *)p;
  return (v[0] + v[1]) + (v[2] + v[3]);
}

// Every pass-2 workgroup sums the histograms of all tiles, so many tiles cost more than long ones from about
// 200 000 branches on (from fewer with many experts, from more with few).  Measured, us per plan without the order list with tiles of
// 1024 / 2048 / 4096 branches: E = 256: 32 768 branches 9.0 / 10.0 / 12.5, 131 072 11.5 / 11.0 / 12.9, 196 608 12.5 / 11.7 / 13.4, 262 144 19.9 / 12.9 /
// 13.7, 400 000 28.5 / 14.1 / 14.5, 524 288 42 / 21.2 / 15.9; E = 64: 131 072 8.4 / 9.2 / 11.3, 196 608 8.9 / 9.8 / 11.8, 262 144 12.8 / 9.7 / 11.6;
// E = 1024: 65 536 15.6 / 15.1 / 16.5, 131 072 20.4 / 17.8 / 18.0, 262 144 47 / 22.3 / 20.3.
int plan_tile_size(int64_t N) {
  int64_t tile = N >= 196608 ? 2 * kPlanMinTile : kPlanMinTile;
  while ((N + tile - 1) / tile > kPlanMaxTiles) tile *= 2;
  return (int)tile;
}
int plan_tile_count(int64_t N) {
  const int64_t tile = plan_tile_size(N);
  const int64_t tiles = (N + tile - 1) / tile;
  return tiles < 1 ? 1 : (int)tiles;
}

template <bool PACKED>
__global__ __launch_bounds__(kPlanBlock) void plan_tile_hist_kernel(const int32_t *__restrict__ K, int N, int E,
                                                                     int tile, int32_t *__restrict__ tile_hist) {
  extern __shared__ int hist[];  // [E+1], padded to pairs of words if PACKED
  const long long start = (long long)blockIdx.x * tile;
  const long long end = min(start + (long long)tile, (long long)N);
  const long long i0 = start + threadIdx.x;
  const int first_id = i0 < end ? K[i0] : -1;     // requested before the histogram is cleared
  const int pitch = hist_pitch<PACKED>(E);
  for (int e = threadIdx.x; e < (PACKED ? 2 : 1) * pitch; e += kPlanBlock) hist[e] = 0;
  __syncthreads();
  for (long long i = i0; i < end; i += kPlanBlock) {
    const int e = i == i0 ? first_id : K[i];
    if (e >= 0 && e < E) atomicAdd(&hist[e], 1);
    else if (e != -1) atomicAdd(&hist[E], 1);
  }
  __syncthreads();
  int32_t *out = tile_hist + (size_t)blockIdx.x * pitch;
  for (int w = threadIdx.x; w < pitch; w += kPlanBlock) out[w] = PACKED ? hist[2 * w] | hist[2 * w + 1] << 16 : hist[w];
}

// Inclusive prefix sum inside each row of 16 consecutive lanes (DPP row shifts).
__device__ __forceinline__ int row16_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  return v;
}

// Pass 2.  Workgroups 0..tiles-1 rank one tile each; workgroup `tiles` writes the count/offset tables.
// A tile is split into 16 contiguous wave segments (64 branches each when the tile is 1024 branches).
// FUSED: there was no pass 1.  Every workgroup counts the ids outside its own tile itself (in front of the
// tile, and all others), which costs N LDS atomics per workgroup instead of a launch (see plan_in_one_launch).
// What bounds it is the chain: launch, round trip for the ids, LDS atomics, barrier, scans, barrier, stores.  Rows of the
// segment histograms have odd length: with rows of E words an expert's 16 counts lay in one LDS bank, and their prefix took 16
// cycles an access (plan of 6656 branches, E = 256 8.1 / 6.2 us, of 7040, E = 512 10.1 / 7.3).  Two or four elements of that prefix in flight per
// thread are slower (+0.1, +0.2 us: the code is longer).
// With one copy of each count popular experts serialise the atomics: 12 000 branches of degree 1, Zipf, 16 experts 8.5 us, with four 6.7;
// uniform 6656, E = 256 6.0 / 5.9.
// WARM: the grid carries spare workgroups that read the caller's prefetch range (compiled apart so that the
// usual plan carries none of it).
template <bool FUSED, bool WARM, bool PACKED>
__global__ __launch_bounds__(kPlanBlock) void plan_rank_kernel(const int32_t *__restrict__ K,
                                                                const int32_t *__restrict__ tile_hist, int tiles,
                                                                int tile, Dims d, PlanView p, WarmRange warm) {
  extern __shared__ __align__(16) int lds[];     // sum4 reads 16 bytes at a time
  const int E = d.E;
  // Branches of expert e (slot E: invalid ids) in four ranges of tiles: in front of this tile's sorted stretch (a run of
  // d.order_tiles tiles), in front of the tile inside it, from the tile to the stretch's end, behind it.  FUSED (the whole batch is one
  // stretch): in front of the tile and all others, each in kCopies counts, one for every kCopies-th lane, so that a popular
  // expert's atomics do not all meet in one word.
  int *range = lds;                    // [4][E+1];  FUSED: [2][E][kCopies]
  int *g = range + (FUSED ? 2 * kCopies * E : 4 * (E + 1));        // [E+1]  exclusive scan of the block sizes over all experts
  int *st_excl = g + E + 1;            // [E+1]  exclusive scan of the stretch's counts
  int *pre = st_excl + E + 1;          // [E]    branches of the source ranks below this one (several sources only)
  int *post = pre + E;                 // [E]    ... above this one
  int *misc = post + E;                // [2]    scratch
  int *wcur = misc + 2;                // [waves][E|1] segment histograms, then running s per wave segment.  The odd row length
  const int wrow = E | 1;              // spreads an expert's 16 counts over the LDS banks
  __shared__ unsigned long long others_rows;   // rows of the other source ranks, 64-bit
  const int tid = threadIdx.x, wave = uniform(tid / kWave), lane = tid % kWave;
  const int me = blockIdx.x;
  const bool multi = p.source_count != nullptr;
  if (tid == 0) others_rows = 0;

  if (WARM && me > tiles) {            // spare workgroups: pull the caller's memory (normally X) into the caches
    constexpr int kPer = 8;            // vectors per thread and trip
    const u32x4 *src = (const u32x4 *)warm.ptr;
    const long long wgs = (long long)gridDim.x - tiles - 1, w = me - tiles - 1;
    const long long chunk = (warm.vecs + wgs - 1) / wgs;
    const long long lo = w * chunk, hi = min(lo + chunk, warm.vecs);
    unsigned acc = 0;
    for (long long i = lo + tid; i < hi; i += (long long)kPlanBlock * kPer) {
      u32x4 v[kPer];
#pragma unroll
      for (int u = 0; u < kPer; ++u)
        v[u] = i + (long long)u * kPlanBlock < hi ? src[i + (long long)u * kPlanBlock] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int u = 0; u < kPer; ++u) acc |= v[u][0];
    }
    asm volatile("" ::"v"(acc));       // the loads are kept although nothing uses their values
    return;
  }
  if (me == tiles) {                   // tables workgroup
    if (FUSED) {
      tables_from_ids_block(K, d, p, lds);
      return;
    }
    SourceSums sums;
    if (multi) sums.request(p.source_count, d);
    for (int e = tid; e < 4 * (E + 1); e += kPlanBlock) range[e] = 0;
    for (int e = tid; e < 2 * E; e += kPlanBlock) pre[e] = 0;        // pre and post
    __syncthreads();
    sum_tile_hists<PACKED>(tile_hist, tiles, tile, E, tiles, tiles, tiles, range);          // all in the first range
    if (multi) add_sources(sums, p.source_count, d, pre, post, &others_rows);
    __syncthreads();
    exclusive_scan_lds([&](int e) { return range[e] + (multi ? pre[e] + post[e] : 0); }, g, E, wave, kPlanWaves);
    __syncthreads();
    write_plan_tables(range, multi ? pre : nullptr, g, d, p, range[E], misc, multi && rows_overflow(others_rows, g[E]));
    return;
  }

  // The sorted stretch this tile belongs to (FUSED: the whole batch is one stretch)
  const bool ordered = d.order_tiles > 0;
  const int st0 = !ordered ? me : FUSED ? 0 : (me / d.order_tiles) * d.order_tiles;
  const int st1 = !ordered ? me : FUSED ? tiles : min(tiles, st0 + d.order_tiles);
  const int seg = tile / kPlanWaves;
  const long long seg_start = (long long)me * tile + (long long)wave * seg;
  const int rounds = seg / kWave;
  // the first round's id is requested before anything else and stays in a register
  const long long i_first = seg_start + lane;
  const int id_first = i_first < d.N ? K[i_first] : -1;
  constexpr int kBatch = 8;            // FUSED: ids of other tiles, kBatch per thread and trip
  const int tile_start = me * tile;    // FUSED only runs with N <= tiles * tile well inside 31 bits
  const int tile_end = min(tile_start + tile, d.N);
  int other[kBatch];
  if (FUSED) {
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = u * kPlanBlock + tid;
      other[u] = (i < d.N && (i < tile_start || i >= tile_end)) ? K[i] : -1;
    }
  }

  SourceSums sums;
  if (multi) sums.request(p.source_count, d);
  for (int e = tid; e < (FUSED ? 2 * kCopies * E : 4 * (E + 1)); e += kPlanBlock) range[e] = 0;
  for (int e = tid; e < 2 * E; e += kPlanBlock) pre[e] = 0;          // pre and post
  for (int x = tid; x < kPlanWaves * wrow; x += kPlanBlock) wcur[x] = 0;
  int *rest = range + kCopies * E, *const copy = range + lane % kCopies, *const rest_copy = rest + lane % kCopies;   // FUSED
  __syncthreads();
  if (FUSED) {
    for (int i0 = 0; i0 < d.N; i0 += kBatch * kPlanBlock) {
      int next[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {                 // the next trip's ids are requested first
        const int i = i0 + (kBatch + u) * kPlanBlock + tid;
        next[u] = (i < d.N && (i < tile_start || i >= tile_end)) ? K[i] : -1;
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int e = other[u];
        if (e >= 0 && e < E) atomicAdd((i0 + u * kPlanBlock + tid < tile_start ? copy : rest_copy) + e * kCopies, 1);
        other[u] = next[u];
      }
    }
  } else {
    sum_tile_hists<PACKED>(tile_hist, tiles, tile, E, st0, me, st1, range);
  }
  if (multi) add_sources(sums, p.source_count, d, pre, post, &others_rows);
  // histogram of each wave's segment (counts only: atomics are order-free here)
  for (int rd = 0; rd < rounds; ++rd) {
    const long long i = seg_start + (long long)rd * kWave + lane;
    const int e = rd == 0 ? id_first : (i < d.N ? K[i] : -1);
    if (e >= 0 && e < E) {
      atomicAdd(&wcur[wave * wrow + e], 1);
      if (FUSED) atomicAdd(rest_copy + e * kCopies, 1);  // the tile's own ids complete the counts
    }
  }
  __syncthreads();
  auto in_front = [&](int e) { return FUSED ? sum4(range + e * kCopies) : range[e] + range[E + 1 + e]; };
  auto all = [&](int e) {
    return in_front(e) + (FUSED ? sum4(rest + e * kCopies) : range[2 * (E + 1) + e] + range[3 * (E + 1) + e]);
  };
  auto in_stretch = [&](int e) { return FUSED ? all(e) : range[E + 1 + e] + range[2 * (E + 1) + e]; };
  exclusive_scan_lds([&](int e) { return all(e) + (multi ? pre[e] + post[e] : 0); }, g, E, wave, kPlanWaves);
  if (ordered) exclusive_scan_lds(in_stretch, st_excl, E, kPlanWaves - 1 - wave, kPlanWaves);
  // exclusive prefix of the segment counts over the 16 waves, seeded with the count in earlier tiles:
  // element (e, w) sits in lane w of a 16-lane row, so one DPP row scan does it
  for (int x = tid; x < kPlanWaves * E; x += kPlanBlock) {
    const int e = x / kPlanWaves, w = x % kPlanWaves;
    const int c = wcur[w * wrow + e];
    const int incl = row16_inclusive_scan(c);
    wcur[w * wrow + e] = in_front(e) + incl - c;
  }
  __syncthreads();

  // rows are int32: if the blocks of all sources together do not fit, nothing is placed
  const bool overflow = multi && rows_overflow(others_rows, g[E]);
  // stable ranks inside each wave segment: 64 branches per round, rounds in index order.  Lanes with
  // the same id all read the segment's running count, then the lowest of them advances it.
  const int bits = id_bits(E);
  int *mine = wcur + wave * wrow;
  for (int rd = 0; rd < rounds; ++rd) {
    const long long i = seg_start + (long long)rd * kWave + lane;
    const bool in = i < d.N;
    const int e = rd == 0 ? id_first : (in ? K[i] : -1);
    const bool valid = e >= 0 && e < E;
    const unsigned long long peers = match_any(e, valid, bits);
    int s = -1, row = -1;
    if (valid) {
      const int base = mine[e];
      const int rank = __popcll(peers & ((1ull << lane) - 1ull));
      if (rank == 0 && rounds > 1) mine[e] = base + __popcll(peers);   // LDS ops of a wave execute in order
      s = base + rank;
      row = expert_first_row(g, e, d) + pre[e] + s;                    // o_{e,me} + s
      if (row >= region_row_limit(e, d) || overflow) row = -1;
    }
    if (in) {
      if (p.send_idx) p.send_idx[i] = s;
      p.row_map[i] = row;
    }
    if (ordered) {
      // position of the branch among the counted branches of its stretch, sorted by (expert, flat index), i.e.
      // by window row; branches that are not counted leave the tail of the stretch's list, which is marked unused
      typedef int i32x2 __attribute__((ext_vector_type(2)));
      i32x2 *list = (i32x2 *)p.order;
      const long long st_base = (long long)st0 * tile;
      if (valid) list[st_base + st_excl[e] + (FUSED ? s : s - range[e])] = i32x2{(int)i / d.k, row};
      if (in && (int)(i - st_base) >= st_excl[E]) list[i] = i32x2{-1, -1};
    }
    // the next round of this wave must see this round's counter updates
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// No tokens: the tables still describe the (possibly non-empty) blocks of the other source ranks.
__global__ __launch_bounds__(kPlanBlock) void plan_empty_kernel(Dims d, PlanView p) {
  extern __shared__ int lds[];
  const int E = d.E;
  int *total = lds;                    // [E]   zeros
  int *g = total + E;                  // [E+1]
  int *pre = g + E + 1;                // [E]
  int *post = pre + E;                 // [E]
  int *misc = post + E;                // [2]
  __shared__ unsigned long long others_rows;
  const bool multi = p.source_count != nullptr;
  SourceSums sums;
  if (multi) sums.request(p.source_count, d);
  for (int e = threadIdx.x; e < E; e += kPlanBlock) {
    total[e] = 0;
    pre[e] = 0;
    post[e] = 0;
  }
  if (threadIdx.x == 0) others_rows = 0;
  __syncthreads();
  if (multi) add_sources(sums, p.source_count, d, pre, post, &others_rows);
  __syncthreads();
  exclusive_scan_lds([&](int e) { return total[e] + (multi ? pre[e] + post[e] : 0); }, g, E, uniform((int)threadIdx.x / kWave),
                     kPlanWaves);
  __syncthreads();
  write_plan_tables(total, multi ? pre : nullptr, g, d, p, 0, misc,
                    multi && rows_overflow(others_rows, g[E]));
}

hipError_t launch_plan_empty(const Dims &d, const PlanView &p, hipStream_t s) {
  const size_t lds = (size_t)(4 * d.E + 1 + 2) * sizeof(int);
  return launch(plan_empty_kernel, dim3(1), dim3(kPlanBlock), lds, s, d, p);
}

// Largest batch (in tiles of 1024 branches) that needs no workspace.
#ifndef MOE_PLAN_FUSED_MAX_TILES
#define MOE_PLAN_FUSED_MAX_TILES 12
#endif

bool plan_uses_workspace(int64_t N) { return N > (int64_t)MOE_PLAN_FUSED_MAX_TILES * kPlanMinTile; }

// Batches planned with one launch: all that need no workspace, and further ones whose order list is one stretch (such a plan sorts
// the whole batch) and whose experts are not too few.  us per plan, two launches / one: k = 8: 17 920 branches, E = 256 9.0 / 7.6, Zipf 8.4 / 7.3; k = 6: 18 006, E = 96
// 8.1 / 7.1, 24 576, E = 256 8.7 / 7.6, E = 64 7.3 / 6.9; 28 672, E = 96 7.85 / 7.85, E = 256 8.85 / 8.3; 32 768 9.2 / 9.0; degrees below 4, where
// a popular expert may have a large part of all branches: Zipf, 18 000 of degree 1, E = 16 7.5 / 8.6, of degree 3 7.0 / 7.2.
static bool plan_in_one_launch(const Dims &d, int tiles) {
  if (!plan_uses_workspace(d.N)) return true;
  // Few experts: the atomics of all workgroups meet in few words.  us per plan, two launches / one: E = 8: 16 000 branches 7.45 / 6.35,
  // 20 000 7.45 / 7.3, 24 576 7.5 / 8.0, 28 600 7.45 / 8.9; E = 4: 13 000 7.35 / 7.0, 20 000 7.4 / 9.2; E = 12: 24 576 7.6 / 7.5, 28 600 7.6 / 8.1.
  if (d.N > 2 * kPlanMinTile * d.E) return false;
  return d.k >= 4 && d.N <= 28 * kPlanMinTile && (d.order_tiles == 0 || d.order_tiles >= tiles);
}

// Measured on the same buffers, k = 8 unless noted, us per LAYER (plan + dispatch + combine) with the list / in token
// order, with stretches of about 28 MB of X (3.5 MB per XCD, most of its L2), which did best:
//   H = 7168, balanced: T = 1536 69.3 / 75.4, 2048 94.4 / 97.6, 3072 134.3 / 136.2, 4096 171.3 / 181.1, 5120 221.6 / 220.8,
//             6144 258.5 / 263.7, 7168 309 / 303.6 (a loss), 8192 352.9 / 347.4 (a loss), 16384 702 / 691.5 (a loss);
//             Zipf routing: T = 4096 171.1 / 171.0, T = 16384 665 / 660 (a loss); k = 6, T = 4096: 134.6 / 137.2;
//             k = 4, T = 8192: 194.2 / 190.9 (a loss)
//   H = 6144: T = 4096 150.5 / 159.7, 6144 227.5 / 242.0, 8192 292.3 / 312.8
//   H = 8192: T = 4096 192.7 / 201.5, 6144 285.3 / 301.5;  H = 16384: T = 2048 203.7 / 204.6, 3072 289.8 / 303.0
//   H = 4096, balanced: T = 2048 59.1 / 61.6, 4096 108.4 / 109.4, 8192 204.4 / 208.5, 16384 390.1 / 418.7;
//             group-limited, E = 128: T = 8192 202.4 / 205.8, 16384 379.2 / 405.2, 32768 940 / 830 (a loss)
// A loop of dispatches alone gains more (T = 4096, H = 7168: 76.8 / 85.2 us).  Inside a layer the gain depends on
// X still being in the Infinity Cache when the dispatch starts (the list makes every token row be fetched at
// k scattered moments of its stretch), so the list is used
//   for rows of 12 KB or more while X holds at most 96 MiB and the window at most 770 MiB,
//   for narrower rows with windows of up to 1100 MiB,
// and for larger X with bulk reads (order_streams_x).
// (All layers here were measured with the plan as it was before its tile histograms were packed, on both sides.  The list cost that plan 1.3 us
// at 32 768 branches and 2.8 at 131 072; it costs the present one 0.4 to 0.65 up to 65 536, 1.0 at 131 072, 1.4 at 262 144, so both sides are 1 to 4 us
// shorter now and the list's by 0.7 to 2 us more.  And with slices in one block.  Now, list / token order, E = 256 or 64, X cached; not cached: H = 7168: k = 8: T = 1536 68.0 / 75.6;
// 69.4 / 73.4, 3072 136.7 / 136.2; 136.3 / 136.0, 4096 180.6 / 187.2; 199 / 249, 5800 246 / 251; 277 / 345; k = 6, T = 4096 137.6 / 137.9; 159 / 187; k = 4, T = 4096 103.9 / 98.9; 122 / 129; k = 2,
// T = 4096 67.9 / 63.9; 73.9 / 71.9 (a loss); H = 6144: T = 4096 149.9 / 166.3; 174 / 182; H = 4096: T = 8192 193 / 207; 227 / 226, k = 2, T = 10000 86.6 / 85.6; 102 / 97 (a loss); H = 5120, k = 4,
// T = 5000 91.9 / 87.8; 116 / 104 (a loss); H = 3072, T = 8192 147 / 158; 176 / 169; H = 2560, T = 12288 187 / 199; 231 / 207; H = 1024, T = 32768 193 / 210; 243 / 220.  The lines below have not been drawn
// again: degrees of 2 and 4 would be better off without the list at more widths than those named.)
// Rows of 2 to 4 KB, us per layer with the list / in token order: H = 2048: T = 8192 105.4 / 108.0, 16384 197.0 / 204.3,
// 32768 388.6 / 407.6; H = 1024: T = 16384 110.0 / 113.4, 65536 405.7 / 426.0.  With slices cut at cache lines and units
// packed side by side the same holds for most widths from 1.5 KB on (sum of the kernels' us): H = 2560, T = 11468
// 190.8 / 202.3; H = 3072, T = 9557 183.9 / 194.5; H = 3584, T = 8192 187.1 / 202.2; H = 768, T = 32768 173.6 / 181.5.
// It depends on the degree there, since the plan pays for the list per branch, and in token order one unit stores all 2 or 4
// branches of a token (odd degrees share no loads, larger even ones in part).  us per layer, list / token order:
//   rows under 2 KB: from a degree of 8 on.  H = 896: T = 11702: k = 2 33.4 / 32.6, k = 6 61.1 / 60.8, k = 8 74.3 / 77.2,
//     k = 10 90.3 / 94.9; T = 4681: k = 4 28.0 / 26.5, k = 8 38.0 / 37.7; T = 35108: k = 6 158.7 / 161.6 (a loss), k = 8 193.7 / 200.5;
//   rows of 4 to 8 KB, degrees of 2 and 4: not where a slice has more than 48 vectors (the token-order unit's wave is then
//     nearly full) and not for degree 4 without bulk reads.  H = 3584: T = 8777: k = 2 72.2 / 70.2, k = 3 91.5 / 103.1, k = 5 131.7 /
//     156.9, k = 6 150.9 / 152.1, k = 8 185.8 / 199.6; T = 2925: k = 4 44.6 / 43.7; with bulk reads T = 13897: k = 2 124.7 / 123.4,
//     k = 4 195.3 / 190.0; H = 3200: T = 9830: k = 2 74.5 / 71.9, k = 4 113.7 / 108.3, T = 24576: k = 4 316.9 / 294.3;
//     H = 2560: T = 12288: k = 2 72.0 / 74.4, k = 4 111.5 / 108.2; T = 19456: k = 2 123.3 / 139.2, k = 4 198.4 / 208.9.
// Narrower rows pay more for the list in the plan than dispatch gains (H = 640, T = 10000 59.2 / 57.2), and so do
// batches whose X is in the L2s anyway: H = 2048, T = 1400 26.9 / 26.5; H = 2560, T = 1024 23.5 / 23.1; but H = 3072,
// T = 1400 (8.6 MB) 34.5 / 35.7.  (Plan and dispatch, with the list / without: H = 4096, T = 500 17.1 / 16.2, H = 7168, T = 128
// 11.7 / 11.4; a dispatch alone, on a plan that is kept, is up to 0.6 us slower without: T = 128 4.0 / 4.2, T = 300 8.7 / 9.2.)
// From 80 MiB of X on the list is used at every window size with X read in bulk (order_streams_x), except for degrees that
// re-read X too little: us per layer, X not cached, list with bulk reads / the rule above: k = 2: H = 7168, T = 14000 225.5 /
// 214.6; H = 4096, T = 28000 246 / 266; k = 1: H = 4096, T = 20000 128 / 122; around the line: H = 7168: T = 5000 (72 MB)
// 217 / 209, 6200 (89 MB) 280 / 294; H = 2560, T = 14000 (72 MB) 219 / 216; H = 4096, T = 11000 (90 MB) 267 / 295.
// A single-launch plan has one stretch, the whole batch: that much X, read in bulk first, has left the L2s before it is copied.  Such
// batches (rows of 20 KB and more, degrees of 3 to 8) keep the rule above; us per layer, list with bulk reads / now, fp32: H = 8192:
// k = 3, T = 3200 175.1 / 159.2; k = 4, T = 3000 203.7 / 198.9; H = 12288, k = 6, T = 1800 241 / 232; H = 16384: k = 5, T = 2400
// 396.8 / 393.1; k = 6, T = 2000 367.7 / 381.8 (a loss); k = 8, T = 1500 349.7 / 339.5.
bool order_streams_x(const Dims &d) {
  const int64_t row_bytes = (int64_t)d.H16 * 16;
  return plan_uses_workspace(d.N) && (int64_t)d.T * row_bytes > ((int64_t)80 << 20) && (d.k >= 3 || (d.k == 2 && row_bytes < 12288));
}

int plan_order_tiles(const Dims &d) {
  const int64_t row_bytes = (int64_t)d.H16 * 16, x = (int64_t)d.T * row_bytes, window = (int64_t)d.N * row_bytes;
  constexpr int64_t mib = 1 << 20;
  if (d.H16 < 96 || x <= 5 * mib) return 0;
  const bool bulk = order_streams_x(d);
  if (d.H16 < 128 && d.k < 8 && !bulk) return 0;
  if (d.H16 > 256 && d.H16 < 512 && (d.k == 2 || d.k == 4) && (d.H16 > 384 || (d.k == 4 && !bulk))) return 0;
  if (!bulk && (row_bytes < 12288 ? window > 1100 * mib : (window > 770 * mib || x > 96 * mib))) return 0;
  const int tile = plan_tile_size(d.N), tiles = plan_tile_count(d.N);
  if (!plan_uses_workspace(d.N)) return tiles;                      // single-launch plan: the batch is one stretch
  // stretches of about 28 MB of X (24 MB where it is read in bulk: with 20 or 28 MB the layers above differ by 2 % either
  // way), all of (nearly) the same length
  const int64_t most = (bulk ? 24 : 28) * mib / row_bytes * d.k / tile;
  if (most < 1) return 1;
  const int64_t n = (tiles + most - 1) / most;
  return (int)((tiles + n - 1) / n);
}

template <bool FUSED, bool PACKED>
static hipError_t launch_plan_rank(const Dims &d, const int32_t *K, const PlanView &p, const int32_t *tile_hist,
                                   int tiles, int tile, const WarmRange &warm, hipStream_t s) {
  const size_t lds = (size_t)((FUSED ? 2 * kCopies * d.E : 4 * (d.E + 1)) + 2 * (d.E + 1) + 2 * d.E + 2 + kPlanWaves * (d.E | 1)) *
                     sizeof(int);
  if (lds > 64 * 1024) {   // beyond the default dynamic LDS limit (E > ~580)
    static RaisedOn raised_warm, raised_plain;
    const hipError_t e = warm.ptr
        ? raise_lds_limit((const void *)plan_rank_kernel<FUSED, true, PACKED>, 128 * 1024, raised_warm)
        : raise_lds_limit((const void *)plan_rank_kernel<FUSED, false, PACKED>, 128 * 1024, raised_plain);
    if (e != hipSuccess) return e;
  }
  if (!warm.ptr)
    return launch(plan_rank_kernel<FUSED, false, PACKED>, dim3(tiles + 1), dim3(kPlanBlock), lds, s, K, tile_hist, tiles, tile,
                  d, p, warm);
  // spare workgroups for plan->prefetch: 8192 vectors (128 KB) each
  const unsigned spare = (unsigned)((warm.vecs + 8191) / 8192);
  return launch(plan_rank_kernel<FUSED, true, PACKED>, dim3(tiles + 1 + spare), dim3(kPlanBlock), lds, s, K, tile_hist, tiles,
                tile, d, p, warm);
}

template <bool PACKED>
static hipError_t launch_plan_passes(const Dims &d, const int32_t *K, const PlanView &p, int32_t *tile_hist, int tiles, int tile,
                                     const WarmRange &warm, hipStream_t s) {
  const size_t lds = (size_t)hist_pitch<PACKED>(d.E) * (PACKED ? 2 : 1) * sizeof(int);
  const hipError_t err = launch(plan_tile_hist_kernel<PACKED>, dim3(tiles), dim3(kPlanBlock), lds, s, K, d.N, d.E, tile, tile_hist);
  if (err != hipSuccess) return err;
  return launch_plan_rank<false, PACKED>(d, K, p, tile_hist, tiles, tile, warm, s);
}

hipError_t launch_plan(const Dims &d, const int32_t *K, const PlanView &p, int32_t *tile_hist, const WarmRange &warm,
                       hipStream_t s) {
  const int tile = plan_tile_size(d.N);
  const int tiles = plan_tile_count(d.N);
  if (plan_in_one_launch(d, tiles)) return launch_plan_rank<true, true>(d, K, p, nullptr, tiles, tile, warm, s);
  return tile < 65536 ? launch_plan_passes<true>(d, K, p, tile_hist, tiles, tile, warm, s)
                      : launch_plan_passes<false>(d, K, p, tile_hist, tiles, tile, warm, s);
}

}  // namespace moe_rbf
