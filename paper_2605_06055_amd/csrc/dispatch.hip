// Dispatch: direct placement of token rows into destination expert windows (paper, Section 5.2
// "Prefill Dispatch", Section 5.3 "Decode Dispatch"; first loop of Algorithms 1 and 2).
// No staging copy exists: HBM traffic is T*H bytes read and T*k*H bytes written.
//
// Prefill schedule (row map from moe_plan): XCD-affine column slices, see dispatch_slices_kernel.
// Decode schedule: ONE launch, no grid-wide synchronisation: every workgroup derives the rows of its
//   token from the routing ids themselves (see the decode section below).
#include <algorithm>

#include "device_utils.h"
#include "launch.h"
#include "moe_rbf.h"
#include "plan_tables.h"
#include "quant.h"

namespace moe_rbf {

constexpr int kSlices = 8;   // column slices per row = XCDs per device
constexpr int kLine = 8;     // 16-byte vectors of a 128-byte cache line

// Both prefill kernels split a destination row into 8 column slices, one per XCD, cut at cache lines of the
// DESTINATION: a line that two XCDs write halves of leaves two L2s as partial writes, and that costs far more than
// the bytes.  (With cuts every ceil(H16 / 8) vectors, whatever line they fell into, us per dispatch of 528 MB, before /
// now: H = 2560 98 / 84, 4608 95 / 84, 7680 88 / 81; rows that are no multiple of a line: H = 1032 214 / 116, 2056 181 /
// 97, 4104 119 / 99, 7176 124 / 87; H = 640, 378 MB: 175 / 64.)  A row that starts `a` vectors into its first line
// touches n = ceil((a + H16) / 8) lines; slice c holds the lines [c*n/8, (c+1)*n/8).  Where n is no multiple of 8
// the slices differ by a line, so slice c of token t goes to XCD (c - t) mod 8: every XCD gets its share of the longer
// ones, and a (token, slice) still belongs to one XCD, whose L2 serves its k reads.

// Prefill dispatch in token order, for rows that start at a cache line.  Work unit = (J consecutive branches of one token,
// one column slice); a workgroup holds U units.  Workgroups are handed to the 8 XCDs round-robin, so workgroup b runs on
// XCD b % 8 and the k re-reads of X[t]'s slice by the branches of a token hit in that
// XCD's L2 (X is fetched from HBM once), every wave issues few 16-byte stores per lane, and the 8 XCDs
// together lay down whole destination rows.  Stores are streaming (nontemporal) so that they do not
// evict the X slices from L2; loads are ordinary so that they stay.
// (If the hardware maps workgroups differently the result is unchanged; only the L2 reuse is lost.)
template <int BLOCK, int J, int U>
__global__ __launch_bounds__(BLOCK) void dispatch_slices_kernel(const u32x4 *__restrict__ X,
                                                                const int32_t *__restrict__ row_map,
                                                                u32x4 *__restrict__ window, int k, int H16, int rotate,
                                                                int N) {
  // U units per workgroup, each with BLOCK / U lanes: narrow slices (small H) still fill the workgroup
  constexpr int kLanes = BLOCK / U;
  const int unit = U == 1 ? 0 : (int)threadIdx.x / kLanes;
  const int lane = U == 1 ? (int)threadIdx.x : (int)threadIdx.x % kLanes;
  const int g = (blockIdx.x / kSlices) * U + unit;
  const int n = g * J;                       // J consecutive branches of one token (J divides k)
  if (U > 1 && n >= N) return;
  int row[J];
#pragma unroll
  for (int u = 0; u < J; ++u) row[u] = kLanes % kWave == 0 ? uniform(row_map[n + u]) : row_map[n + u];
  const int t = n / k;
  const int c = (blockIdx.x + (t & rotate)) % kSlices;         // rotate: 7, or 0 where the slices are equal
  const int lines = (H16 + kLine - 1) / kLine;
  const int begin = ((c * lines) >> 3) * kLine, end = min(((c * lines + lines) >> 3) * kLine, H16);
  const u32x4 *src = X + (size_t)t * (size_t)H16;
  for (int col = begin + lane; col < end; col += kLanes) {
    const u32x4 v = src[col];
#pragma unroll
    for (int u = 0; u < J; ++u)
      if (row[u] >= 0) store_stream(window + (size_t)row[u] * (size_t)H16 + col, v);
  }
}

// Vector offset of a row: one 32 x 32 -> 64 bit product (a sign-extended index would take three multiplications a lane).
__device__ __forceinline__ size_t row_offset(int row, int H16) {
  return (size_t)((unsigned long long)(unsigned)row * (unsigned)H16);
}

// Column of vector l of slice c, for slices that are all equal: pieces of `piece` vectors (2^shift, or the whole slice with
// shift = 31) in turn over the slices.
// With pieces of the largest power of two that divides the slice an XCD writes the same few address bits in every row (a row
// being a whole number of 8 pieces), so a DRAM page is written by one XCD.  Slices of another length are not in step with the pages:
// each is written by several XCDs, which do not run in step either.  Plain fills in order, 2 GB, an XCD owning every 8th block: 256
// bytes 6.1 TB/s, 512 7.0, 1024 7.35, 2048 6.7, 4096 7.2, but 768 5.4, 1536 5.0, 1792 5.3, 3584 5.3, whatever the occupancy.
// An XCD then also fetches X less often: H = 6144, T = 12160 in bulk 1.57 times in one block and 1.06 in pieces, Zipf H = 7168, T = 16384 1.19 / 1.05.
// us per dispatch along the list, slices in one block / in pieces, k = 8: X of 58 MB: H = 12288 (1 KB) 77.3 / 73.8, 6144 (512 bytes) 80.5 /
// 75.1, 14336 79.2 / 75.6, 10240 79.1 / 76.7; 256 bytes: 3072 81.7 / 77.3, 5120 80.6 / 79.5, 9216 79.8 / 77.4; 128 bytes: 2560
// 82.4 / 86.0, 4608 80.4 / 85.2, 7680 82.2 / 86.6 (but 3584 84.6 / 80.8).  With bulk reads, X of 100, 150, 235 MB: 12288 142 / 133, 235 / 208, 386 /
// 344; 6144 151 / 139, 252 / 234, 417 / 374; 14336 160 / 142, 251 / 232, 357 / 347; 7168 161 / 156, 254 / 255, 384 / 379; 5120 153 / 144, 253 /
// 254, 401 / 402; 3072 150.5 / 153.7, 255 / 262, 388 / 395 (of the rows under 8 KB with 256-byte pieces these are the only ones; they keep one block there).
// X that is not cached (58 MB, 8 copies in turn), us per layer: 6144 206.1 / 205.9, 3072 209.9 / 208.4 (T = 9898 213.4 / 218.2, cached 178.0 / 178.6), 5120 215.1 / 213.5, 12288 197.6 / 194.4, 9216 209.9 /
// 208.1; but units that are alone in a workgroup (H = 7168, see ALONE below) read such an X better in one block: 197.9 / 204.1 (k = 4 123.8 / 128.5),
// and a cached one better in pieces: 174.5 / 171.8.  They keep the block.  (That is this one width: 104 vectors have no pieces of 256 bytes.  With the block
// as a compile-time case the kernel needs 6 VGPRs instead of 14: cached 174.8 against 176.2 with it, not cached 199.0 / 198.1; not kept.)
// Larger pieces than divide the row, owned by address all the same, are needed by 2 to 8 XCDs for each token: H = 7168 82 / 104, 119, 125
// (with stretches shortened to what L2 then holds 87, 97, 112).  Other kinds of stores, which fills like (ordinary, sc1, sc0 sc1 6.2 to
// 7.3 TB/s along the list's runs, nt 5.0), push X out of L2: 148 us.
__device__ __forceinline__ int slice_col(int c, int l, int piece, int shift) {
  return (int)__umul24(l >> shift, piece * kSlices) + (int)__umul24(c, piece) + (l & (int)((1u << shift) - 1u));
}

// Prefill dispatch, one unit per (branch, column slice).  LIST: along the plan's order list, unit p copies a slice of
// X[token] to window[row] for the p-th (token, row) pair.  The pairs are sorted by row inside stretches of tokens whose X
// slices fit the L2 of an XCD, so consecutive workgroups of an XCD write consecutive rows of one expert block and re-read
// tokens from L2.  Without LIST: in token order, for narrow rows and for rows that do not start at a cache line (ALIGNED =
// false; their cuts differ from branch to branch).  ROTATE: the slices are not all equal (see above; always so without ALIGNED).
// A unit takes `lanes` = the longest slice's vectors, and a workgroup is U units side by side without a gap: 4 waves or so,
// up to 10 where only that is a whole number of waves (72 lanes: 8 units, 9 waves).  Units padded to 64 or 128 lanes leave up to half of a wave idle while workgroups can only be started at
// about 4.7 per ns (H = 4608: 84 us against 95 with 72 of 128 lanes busy).  Unequal short slices leave lanes idle all
// the same; there Q = 2 consecutive branches per unit pay (H = 640 77 -> 64 us, 768 86 -> 72), while equal or longer
// slices lose with them (H = 1536 82 -> 88, 3072 81 -> 88, 8192 74 -> 86: more writes in flight arrive in less order).
// WARM (with LIST, for an X that no longer fits the Infinity Cache beside the window): the grid's y dimension walks the
// stretches, and the first warm_blocks workgroups of each read the stretch's X, every XCD the slices that its units are
// about to copy.  The list asks for a token's row at k scattered moments while the chip is saturated with writes; what is
// not cached then comes in 1 KB pieces, and the write stream waits behind them.  Read in bulk, 24 MB at a time and just
// before it is used, X costs little more than its bytes.  Nothing waits for the reads: they are a hint.  A unit reads one token:
// the readers then fill all wave slots of the chip, and the copies behind them start when X is there.  With 8 tokens a unit they held
// 12 slots of 32, and the copies in the others asked for X in random order in the meantime; the gap in the stores at each stretch was
// 6.4 us for 24 MB.  us per dispatch, X not cached, 8 tokens / 1 (4, 2: in between): group-limited T = 32768, H = 4096 449 / 426;
// T = 24000 288 / 278; H = 6144, T = 12160 263 / 252; H = 2560, T = 45888 427 / 406; H = 7168: T = 16384 395 / 384, k = 4, T = 10463 148 /
// 141; H = 4104, T = 14000 220 / 208; H = 7400, T = 9000 223 / 214.  (X is fetched as often with 8 tokens as with one, only later.  Of slices of more than
// 512 vectors, rows over 64 KB, the readers read the first 512.)  What it costs where X is cached: us per layer, 8 / 1: H = 7168: T = 8192 355.3 / 357.9, k = 4,
// T = 10463 260.5 / 263.9; H = 4096: T = 12000 275.4 / 278.8, k = 3, T = 24000 261.0 / 264.4; H = 7680, T = 5515 252.6 / 254.3; H = 6144, T = 8128, Zipf 279.1 / 283.6.  Where
// the plan has prefetched X it depends: H = 6144, T = 8128, Zipf 289.7 / 293.5; H = 4096, T = 12000 286.4 / 288.8; H = 7168, T = 16384, Zipf 695.8 / 698.9; but H = 2560, T = 34000
// 567.8 / 561.5; H = 12288, T = 6080 445.3 / 434.1; H = 7168, k = 4, T = 10463 296.7 / 285.3; so the readers do not ask whether it has.
// us per layer, token order / list / list with bulk reads, X not cached when the layer starts: H = 7168: T = 8192 485 / 420 /
// 383, 13000 760 / 699 / 602, Zipf 16384 933 / 812 / 725; H = 8192, T = 12000 768 / 656 / 609; H = 4096: T = 24000 633 / 683 /
// 605, 11000 294 (list) / 268; H = 3072, k = 10, T = 32768 1087 / 908 / 799; H = 4096, k = 3, T = 16000 263 / 212 / 188; X
// fully cached: H = 7168: T = 8192 356 / 357 / 371, 16384 709 / 718 / 741; H = 4096, T = 20000 505 / 466 / 479.  So a cached X
// loses 1 to 4 % (k = 4, T = 10000, H = 7168 233 / 246: 6 %), and one that is not wins 8 to 25 %.  (These are with 8 tokens a reader and slices in one block.  Now,
// token order / list with bulk reads: cached H = 7168: T = 6144 266 / 267, 8192 372 / 372, 16384 692 / 719, k = 4, T = 8192 193 / 212; H = 6144, T = 8192 311 / 291; H = 4096, T = 16384
// 421 / 405; not cached 363 / 267, 488 / 381, 949 / 750, 249 / 219, 340 / 298, 435 / 408.)  The latter decides: X of this size
// stays cached only while little else runs, and not even always when the kernel in front of the layer has just written
// it (H = 7168, T = 16384, token order / list with bulk reads: 928 / 757).
// ALONE: one unit per workgroup of 128 threads, its entry in scalar registers.  Slices of 104 and 112 vectors nearly fill two
// waves that way, packed they take 13 and 14 waves for 8 units, and without bulk reads they do better alone.  us per layer, packed /
// alone, T = 700, 1400, 2800, 4096: H = 6400 36.8 / 35.9, 64.3 / 61.7, 115.1 / 111.0, 164.5 / 158.0; H = 6656 37.2 / 36.4, 64.1 /
// 62.1, 115.2 / 113.5, 165.4 / 160.1; H = 6912 38.2 / 37.1, 65.4 / 63.7, 119.2 / 119.3, 170.6 / 165.6; H = 7168 38.7 / 37.9,
// 66.5 / 65.3, 120.9 / 124.4, 174.7 / 172.8 (with X not cached 210 / 197).  Shorter and longer slices do not: H = 5632 33.0 / 33.6,
// 55.2 / 56.7, 98.0 / 101.0, 137.6 / 141.1; H = 7424 (120 vectors) 40.1 / 39.2, 69.3 / 68.1, 126.9 / 127.7, 181.1 / 184.9; H = 7680
// 40.3 / 39.9, 70.2 / 70.7, 129.0 / 134.4, 184.5 / 188.5; H = 8192 42.0 / 42.0, 73.8 / 75.2, 136.0 / 138.3, 189.7 / 190.5.
template <int Q, bool LIST, bool ROTATE, bool ALIGNED, bool WARM, bool ALONE = false>
__global__ __launch_bounds__(640) void dispatch_units_kernel(const u32x4 *__restrict__ X,
                                                             const int32_t *__restrict__ entries,
                                                             u32x4 *__restrict__ window, int k, int H16, int misalign,
                                                             int N, int lanes, unsigned magic, int U, int T,
                                                             int warm_blocks, int stretch, int piece, int shift) {
  typedef int i32x2 __attribute__((ext_vector_type(2)));
  const int unit = ALONE ? 0 : (int)__umulhi(threadIdx.x, magic);          // threadIdx.x / lanes
  const int lane = (int)threadIdx.x - (int)__umul24(unit, lanes);
  int block = (int)blockIdx.x, stretch_start = stretch;        // without WARM: the first branch of the launch
  if (WARM) {
    stretch_start = (int)blockIdx.y * stretch;
    if (block < warm_blocks) {                                 // warm_blocks is a multiple of 8: XCD = block % 8
      const int t = stretch_start / k + (block / kSlices) * U + unit;
      const int last = min((stretch_start + stretch + k - 1) / k, T);
      const int c = (block + (ROTATE ? t : 0)) % kSlices;
      const int n = (H16 + kLine - 1) / kLine, cn = (int)__umul24(c, n);
      const int x = ROTATE ? (cn >> 3) * kLine + lane : slice_col(c, lane, piece, shift);
      if (t < last && (ROTATE ? x < min(((cn + n) >> 3) * kLine, H16) : lane < H16 / kSlices)) {
        const unsigned used = X[row_offset(t, H16) + (unsigned)x][0];
        asm volatile("" ::"v"(used));    // the load is kept although nothing uses its value
      }
      return;
    }
    block -= warm_blocks;
    N = min(N, stretch_start + stretch);
  }
  const int p0 = stretch_start + (block / kSlices) * U * Q + unit * Q;
  int t[Q], row[Q], col[Q], end[Q];
  u32x4 v[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int p = p0 + q;
    t[q] = row[q] = -1;
    if (p < N) {
      if (LIST) {
        const i32x2 pair = ((const i32x2 *)entries)[p];
        t[q] = pair[0], row[q] = pair[1];
      } else {
        t[q] = p / k, row[q] = entries[p];
      }
    }
    if (ALONE) t[q] = uniform(t[q]), row[q] = uniform(row[q]);
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (ROTATE) {
      const int a = ALIGNED ? 0 : (misalign + (int)((unsigned)row[q] * (unsigned)H16)) & (kLine - 1);
      const int c = (blockIdx.x + t[q]) % kSlices;
      const int n = (a + H16 + kLine - 1) / kLine;
      const int cn = (int)__umul24(c, n);
      col[q] = (cn >> 3) * kLine - a + lane;                   // below 0: the line's part in front of the row
      end[q] = min(((cn + n) >> 3) * kLine - a, H16);
      if (!ALIGNED && col[q] < 0) col[q] += lanes;             // (past the slice, unless it is longer than a workgroup)
    } else {
      col[q] = slice_col((int)blockIdx.x % kSlices, lane, piece, shift);
      end[q] = lane < H16 / kSlices ? H16 : 0;
    }
    if ((t[q] | row[q]) < 0) end[q] = 0;                       // nothing to do
    if (col[q] < end[q]) v[q] = X[row_offset(t[q], H16) + (unsigned)col[q]];
  }
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    if (col[q] >= end[q]) continue;
    store_stream(window + (row_offset(row[q], H16) + (unsigned)col[q]), v[q]);
    if (Q == 1 && ROTATE) {                                    // slices longer than a workgroup
      for (int x = col[q] + lanes; x < end[q]; x += lanes)
        store_stream(window + (row_offset(row[q], H16) + (unsigned)x), X[row_offset(t[q], H16) + (unsigned)x]);
    } else if (Q == 1) {
      for (int l = lane + lanes; l < H16 / kSlices; l += lanes) {
        const unsigned x = (unsigned)slice_col((int)blockIdx.x % kSlices, l, piece, shift);
        store_stream(window + (row_offset(row[q], H16) + x), X[row_offset(t[q], H16) + x]);
      }
    }
  }
}

// ---- decode -------------------------------------------------------------------------------------
//
// Row of branch (t,j) with expert e:  region/expert base + #{ids i : lo <= K_i < e} + #{i < t*k+j : K_i = e}
// (lo = 0 and base = 0 for tight windows; lo = first expert of e's rank and base = rank*stride otherwise).
// Both terms are plain counts over the routing ids of the batch (at most 3584 here, see decode_by_hist), so a payload workgroup gets
// them with compares on the ids it holds in registers, wave ballots (the counts land in scalar
// registers) and one LDS exchange between its waves: no histogram, no scan, one barrier.  The two
// counts of a slot travel packed in one word (low 16 bits: ids below e; high 16 bits: equal ids in
// front of the branch).
// One extra workgroup (the first, since it takes longest) builds the histogram and writes the tables for
// combine and the experts.


// QUANT: the workgroup holds a whole row (chunks == 1), quantises it once and fans the codes and the
// row's scale out instead of the bf16 payload.
// SB: slots of a token ranked together (one LDS exchange per SB slots).  The slots of a token may be split
// over `groups` workgroups (each ranks and stores only its own slots of the chunk): more, smaller
// workgroups spread the stores over all compute units and shorten each one's counting.
// GROUPS is a compile-time constant so that the index arithmetic in front of the first loads stays short.
template <int BLOCK, int V, int SB, int GROUPS, bool QUANT>
__global__ __launch_bounds__(BLOCK) void decode_dispatch_kernel(const u32x4 *__restrict__ X,
                                                                const int32_t *__restrict__ K,
                                                                void *__restrict__ window_any,
                                                                float *__restrict__ window_scale, Dims d, PlanView p,
                                                                int chunks, int per_group) {
  constexpr int groups = GROUPS;
  extern __shared__ int lds[];                                  // tables workgroup
  __shared__ int part[(BLOCK / kWave) * SB];            // per-wave packed counts of a slot batch
  constexpr int kWaves = BLOCK / kWave;
  const int per_token = chunks * groups;
  if (blockIdx.x == 0) {                 // the tables workgroup goes first: it is the longest one
    tables_from_ids_block(K, d, p, lds);
    return;
  }
  const int b = (int)blockIdx.x - 1;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  // workgroup -> (token, chunk, slot group).  Workgroups go to the 8 XCDs round-robin: the workgroups of a
  // token are given to one XCD, whose L2 then serves their re-reads of the token row (the ragged tail of
  // tokens past a multiple of 8 is mapped plainly).
  int t, rem;
  {
    const int full = (d.T & ~7) * per_token;
    if (b >= full) {
      t = b / per_token;
      rem = b - t * per_token;
    } else if (chunks == 1) {             // the usual case: compile-time divisor
      const int q = b >> 3;
      t = (q / GROUPS) * 8 + (b & 7);
      rem = q % GROUPS;
    } else {
      const int q = b >> 3, tq = q / per_token;
      t = tq * 8 + (b & 7);
      rem = q - tq * per_token;
    }
  }
  const int c = rem / groups, grp = rem % groups;
  const int first = t * d.k;
  const int jg0 = grp * per_group, jg1 = min(d.k, jg0 + per_group);       // per_group: slots of a group, whole batches

  // everything that comes from memory is requested up front: payload, routing ids, own slots' ids
  const int col0 = c * (BLOCK * V) + tid;
  const u32x4 *src = X + (size_t)t * (size_t)d.H16;
  u32x4 v[V];
#pragma unroll
  for (int x = 0; x < V; ++x) {
    const int col = col0 + x * BLOCK;
    // read once by this workgroup: streaming, unless sibling workgroups of the token read it too
    v[x] = col < d.H16 ? (groups > 1 ? src[col] : load_stream(src + col)) : u32x4{0u, 0u, 0u, 0u};
  }
  constexpr int kIds = 4;        // ids per thread kept in registers (first kIds passes over K)
  int id[kIds];
#pragma unroll
  for (int u = 0; u < kIds; ++u) {
    const int i = u * BLOCK + tid;
    id[u] = i < d.N ? K[i] : -1;
  }
  u32x2 q[V];
  float scale = 0.0f;
  if (QUANT) {
    __shared__ float red[BLOCK / kWave];
    scale = quantise_row<BLOCK, V>(v, q, red);
  }

  const bool fixed = d.stride > 0;
  for (int j0 = jg0; j0 < jg1; j0 += SB) {
    // lane u < SB of every wave owns slot j0+u
    const bool own = lane < SB && j0 + lane < jg1;
    const int my_e = own ? K[first + j0 + lane] : -1;
    const bool my_valid = my_e >= 0 && my_e < d.E;
    const int my_rank = my_valid ? my_e / d.Er : 0;
    const int my_lo = fixed ? my_rank * d.Er : 0;
    int e[SB], lo[SB], below[SB], front[SB];
#pragma unroll
    for (int u = 0; u < SB; ++u) {
      e[u] = __builtin_amdgcn_readlane(my_e, u);
      lo[u] = __builtin_amdgcn_readlane(my_lo, u);
      below[u] = 0;
      front[u] = 0;
    }
    // wave-wide counts by ballot: they land in scalar registers, no lane reduction is needed
    for (int i0 = 0, pass = 0; i0 < d.N; i0 += BLOCK, ++pass) {
      const int i = i0 + tid;
      int x;
      if (pass < kIds) {
        x = id[0];
#pragma unroll
        for (int q = 1; q < kIds; ++q) x = pass == q ? id[q] : x;
      } else {
        x = i < d.N ? K[i] : -1;
      }
      const int ahead = first + j0 - i;               // slot u is behind id i  <=>  u + ahead > 0
      // ids outside [0,E) never satisfy either test: as unsigned values they are huge (or x > e)
      if (fixed) {
#pragma unroll
        for (int u = 0; u < SB; ++u)
          below[u] += __popcll(__ballot((unsigned)(x - lo[u]) < (unsigned)(e[u] - lo[u])));
      } else {
#pragma unroll
        for (int u = 0; u < SB; ++u) below[u] += __popcll(__ballot((unsigned)x < (unsigned)e[u]));
      }
#pragma unroll
      for (int u = 0; u < SB; ++u)
        front[u] += __popcll(__ballot(x == e[u]) & __ballot(ahead + u > 0));   // two masks, and-ed as scalars
    }
    if (j0 > jg0) __syncthreads();                      // the previous batch's exchange has been read
    {
      int mine = 0;                                   // lane u carries this wave's packed counts of slot u
#pragma unroll
      for (int u = 0; u < SB; ++u) mine = lane == u ? below[u] + (front[u] << 16) : mine;
      if (lane < SB) part[wave * SB + lane] = mine;
    }
    __syncthreads();
    int packed = 0;
    if (lane < SB) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) packed += part[w * SB + lane];
    }
    int s = -1, row = -1;
    if (own && my_valid) {
      s = packed >> 16;
      row = (fixed ? (int)(my_rank * d.stride) : 0) + (packed & 0xffff) + s;
      if (fixed && row >= (int)((my_rank + 1) * d.stride)) row = -1;
    }
    if (own && c == 0 && wave == 0) {
      if (p.send_idx) p.send_idx[first + j0 + lane] = s;
      p.row_map[first + j0 + lane] = row;
      if (d.order_tiles > 0) {          // a later prefill-schedule dispatch on this plan walks the order list
        p.order[2 * (first + j0 + lane)] = t;
        p.order[2 * (first + j0 + lane) + 1] = row;
      }
    }
    // fan the chunk out to this batch's destination rows
    const int nb = min(SB, jg1 - j0);
    for (int u = 0; u < nb; ++u) {
      const int r = __builtin_amdgcn_readlane(row, u);
      if (r < 0) continue;
      if (QUANT) {
        u32x2 *dst = (u32x2 *)window_any + (size_t)r * (size_t)d.H16;    // H bytes per row = H16 8-byte units
#pragma unroll
        for (int x = 0; x < V; ++x) {
          const int col = col0 + x * BLOCK;
          if (col < d.H16) __builtin_nontemporal_store(q[x], dst + col);
        }
        if (tid == 0) window_scale[r] = scale;
      } else {
        u32x4 *dst = (u32x4 *)window_any + (size_t)r * (size_t)d.H16;
#pragma unroll
        for (int x = 0; x < V; ++x) {
          const int col = col0 + x * BLOCK;
          if (col < d.H16) store_stream(dst + col, v[x]);
        }
      }
    }
  }
}

// Decode dispatch of larger batches, where every workgroup's counting over all ids is what the launch waits for.  A workgroup
// takes up to 8 consecutive branches: all of TT tokens, or (TT = 1) one of GROUPS parts of a token's slots.  It counts the ids
// once into an LDS histogram (low 16 bits: the expert's branches; high 16 bits: those in front of the workgroup's
// first; at most MOE_DECODE_MAX_BRANCHES = 8192), then each wave takes a slot and sums the counts of the experts below.
// Compares and ballots (decode_dispatch_kernel) cost 8 instructions per id and slot, this one LDS atomic per id, but two barriers
// more; figures of both at decode_by_hist.  What is left at T = 512, H = 7168, k = 8 (13.7 us): 66 MB at the scattered-write rate
// 10.6, launch 1.7, the ids' round trip and the counting.  Short code counts: the trips over the ids are not unrolled, since each
// jump into code that is not cached costs 0.1 to 0.2 us here, and two trips requested ahead are no better than one.
template <int MOST, int V, int TT, int GROUPS, bool QUANT, bool MULTI>
__global__ __launch_bounds__(MOST) void decode_hist_kernel(const u32x4 *__restrict__ X, const int32_t *__restrict__ K,
                                                            void *__restrict__ window_any,
                                                            float *__restrict__ window_scale, Dims d, PlanView p,
                                                            int chunks, int width, int per_group) {
  static_assert(TT == 1 || GROUPS == 1, "a workgroup takes whole tokens or part of one");
  const int block = (int)blockDim.x, waves = block / kWave;      // whole waves, at most MOST threads
  constexpr int kSlots = 8;                                     // slots ranked together
  extern __shared__ int lds[];
  __shared__ int rows[kSlots];
  __shared__ float red[QUANT ? TT * (MOST / kWave) : 1];
  __shared__ unsigned long long all_rows;                       // of all sources
  if (blockIdx.x == 0) {                 // the tables workgroup goes first: it is the longest one
    tables_from_ids_block(K, d, p, lds);
    return;
  }
  const int b = (int)blockIdx.x - 1;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = uniform(tid / kWave);
  // workgroup -> (first token, chunk, slot group); the workgroups of a token share an XCD (see decode_dispatch_kernel)
  const int sets = (d.T + TT - 1) / TT, per_set = chunks * GROUPS;
  int set, rem;
  if (per_set == 1) {
    set = b, rem = 0;
  } else if (b >= (sets & ~7) * per_set) {
    set = b / per_set;
    rem = b - set * per_set;
  } else {
    const int q = b >> 3, sq = q / per_set;
    set = sq * 8 + (b & 7);
    rem = q - sq * per_set;
  }
  const int c = rem / GROUPS, t0 = set * TT;
  const int jlo = GROUPS == 1 ? 0 : (rem % GROUPS) * per_group;
  const int first = t0 * d.k + jlo;                             // the workgroup's branches: [first, first + slots)
  const int slots = TT == 1 ? min(d.k - jlo, per_group) : min(TT, d.T - t0) * d.k;
  if (slots <= 0) return;

  // everything that comes from memory is requested up front
  const int col0 = c * width + tid, end = min(c * width + width, d.H16);
  u32x4 v[TT][V];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt)
#pragma unroll
    for (int x = 0; x < V; ++x) {
      const int col = col0 + x * block;
      const u32x4 *src = X + (size_t)(t0 + tt) * (size_t)d.H16 + col;
      v[tt][x] = (TT == 1 || t0 + tt < d.T) && col < end ? (GROUPS > 1 ? *src : load_stream(src)) : u32x4{0u, 0u, 0u, 0u};
    }
  i32x4 next = load_ids(K, tid, d.N);
  int my_e = lane < min(kSlots, slots) ? K[first + lane] : -1;
  SourceSums sums;
  if (MULTI) sums.request(p.source_count, d);

  int *hist = lds;                       // [E]
  int *pre = hist + d.E;                 // [E]  several source ranks only: branches of the ranks below this one
  int *post = pre + d.E;                 // [E]  ... above this one
  for (int e = tid; e < (MULTI ? 3 : 1) * d.E; e += block) hist[e] = 0;
  if (MULTI && tid == 0) all_rows = 0;
  __syncthreads();
  int valid = 0;
#pragma unroll 1
  for (int q = tid; 4 * q < d.N; q += block) {
    const i32x4 ids = next;
    next = load_ids(K, q + block, d.N);
    const int ahead = first - 4 * q;                            // id n of the piece is in front <=> n < ahead
#pragma unroll
    for (int n = 0; n < 4; ++n)
      if ((unsigned)ids[n] < (unsigned)d.E) {
        atomicAdd(&hist[ids[n]], n < ahead ? 0x10001 : 1);
        if (MULTI) ++valid;
      }
  }
  if (MULTI) {
    const unsigned long long rows_of_wave = sums.add(p.source_count, d, pre, post, valid);
    if (lane == 0) atomicAdd(&all_rows, rows_of_wave);
  }
  if (QUANT) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const float amax = wave_amax(v[tt]);
      if (lane == 0) red[tt * waves + wave] = amax;
    }
  }
  __syncthreads();
  u32x2 q[TT][V];
  float scale[TT];
  if (QUANT) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) scale[tt] = quantise_with(v[tt], red + tt * waves, waves, q[tt]);
  }

  const bool fixed = d.stride > 0;
  const bool overflow = MULTI && all_rows >= (1ull << 31);      // rows are int32: if they do not fit, nothing is placed
  for (int j0 = 0; j0 < slots; j0 += kSlots) {
    const int nb = min(kSlots, slots - j0);
    if (j0 > 0) {                        // the previous slots are now in front too
      __syncthreads();
      if (wave == 0 && (unsigned)my_e < (unsigned)d.E) atomicAdd(&hist[my_e], 0x10000);
      my_e = lane < nb ? K[first + j0 + lane] : -1;
      __syncthreads();
    }
    for (int u = wave; u < nb; u += waves) {
      const int e = __builtin_amdgcn_readlane(my_e, u);
      int s = -1, row = -1;
      if ((unsigned)e < (unsigned)d.E) {
        const int rank = fixed ? e / d.Er : 0, lo = fixed ? rank * d.Er : 0;
        int below = 0;
        for (int x0 = 0; x0 < e; x0 += 4 * kWave) {
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            const int x = x0 + n * kWave + lane;
            if (x >= lo && x < e) below += (hist[x] & 0xffff) + (MULTI ? pre[x] + post[x] : 0);
          }
        }
        below = __builtin_amdgcn_readlane(wave_inclusive_scan(below), kWave - 1);
        s = (hist[e] >> 16) + __popcll(__ballot(my_e == e) & ((1ull << u) - 1ull));
        row = (fixed ? (int)(rank * d.stride) : 0) + below + (MULTI ? pre[e] : 0) + s;
        if ((fixed && row >= (int)((rank + 1) * d.stride)) || overflow) row = -1;
      }
      if (lane == 0) {
        rows[u] = row;
        if (c == 0) {
          const int n = first + j0 + u;
          if (p.send_idx) p.send_idx[n] = s;
          p.row_map[n] = row;
          if (d.order_tiles > 0) {        // a later prefill-schedule dispatch on this plan walks the order list
            p.order[2 * n] = TT == 1 ? t0 : n / d.k;
            p.order[2 * n + 1] = row;
          }
        }
      }
    }
    __syncthreads();
    const int row_of = rows[lane & (kSlots - 1)];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
      const int u0 = TT == 1 ? 0 : tt * d.k, u1 = TT == 1 ? nb : min(u0 + d.k, nb);
      for (int u = u0; u < u1; ++u) {
        const int r = __builtin_amdgcn_readlane(row_of, u);
        if (r < 0) continue;
        if (QUANT) {
          u32x2 *dst = (u32x2 *)window_any + (size_t)r * (size_t)d.H16;  // H bytes per row = H16 8-byte units
#pragma unroll
          for (int x = 0; x < V; ++x) {
            const int col = col0 + x * block;
            if (col < end) __builtin_nontemporal_store(q[tt][x], dst + col);
          }
          if (tid == 0) window_scale[r] = scale[tt];
        } else {
          u32x4 *dst = (u32x4 *)window_any + (size_t)r * (size_t)d.H16;
#pragma unroll
          for (int x = 0; x < V; ++x) {
            const int col = col0 + x * block;
            if (col < end) store_stream(dst + col, v[tt][x]);
          }
        }
      }
    }
  }
}

// Quantised dispatch with the row map from moe_plan: one workgroup per token holds the whole row,
// quantises it once and stores the codes and the scale to the k destination rows.
template <int BLOCK, int V>
__global__ __launch_bounds__(BLOCK) void dispatch_quant_rows_kernel(const u32x4 *__restrict__ X,
                                                                    const int32_t *__restrict__ row_map,
                                                                    u32x2 *__restrict__ window_q,
                                                                    float *__restrict__ window_scale, int k, int H16) {
  __shared__ float red[BLOCK / kWave];
  const int t = blockIdx.x, tid = threadIdx.x;
  const u32x4 *src = X + (size_t)t * (size_t)H16;
  u32x4 v[V];
  bool has[V];
#pragma unroll
  for (int x = 0; x < V; ++x) {
    const int col = tid + x * BLOCK;
    has[x] = col < H16;
    // ordinary loads, as in dispatch_slices_kernel: X may stay in the Infinity Cache from one layer to the next
    // (with streaming loads the headline dispatch takes 61-63 us instead of 47)
    v[x] = has[x] ? src[col] : u32x4{0u, 0u, 0u, 0u};
  }
  u32x2 q[V];
  const float scale = quantise_row<BLOCK, V>(v, q, red);
  const int32_t *rows = row_map + (size_t)t * k;
  for (int j0 = 0; j0 < k; j0 += 8) {
    int row[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) row[u] = j0 + u < k ? uniform(rows[j0 + u]) : -1;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (row[u] < 0) continue;
      u32x2 *dst = window_q + (size_t)row[u] * (size_t)H16;
#pragma unroll
      for (int x = 0; x < V; ++x)
        if (has[x]) __builtin_nontemporal_store(q[x], dst + tid + x * BLOCK);
      if (tid == 0) window_scale[row[u]] = scale;
    }
  }
}

// dispatch_units_kernel cuts its slices with 24-bit products (a 32-bit one per lane costs 0.5 % of a layer: T = 3001, H = 4104
// 74.3 / 74.0 us).  Rows of 2^24 lines (2 GiB) or more are left to the token-order slices, which cut in scalar registers.
static bool cuts_in_24_bits(const Dims &d) { return (d.H16 + 2 * kLine - 2) / kLine < 1 << 24; }

static hipError_t launch_dispatch_units(const Dims &d, const void *x, const PlanView &p, void *window, bool list,
                                        hipStream_t s) {
  constexpr int kMost = 640;                                   // threads of a workgroup
  const int misalign = (int)(((uintptr_t)window >> 4) & (kLine - 1));
  const bool aligned = misalign == 0 && d.H16 % kLine == 0;
  const int lines = (d.H16 + (aligned ? 0 : kLine - 1) + kLine - 1) / kLine;      // lines a row touches at most
  const bool rotate = !aligned || lines % kSlices != 0;
  int lanes = std::min((lines + kSlices - 1) / kSlices * kLine, 512);
  // units per workgroup: about 256 threads, a whole number of waves where that is near
  int U = std::max(1, 256 / lanes);
  for (int u = U; u >= 1 && U * lanes % kWave != 0; --u)
    if (u * lanes % kWave == 0) U = u;
  for (int u = U; u * lanes <= kMost && U * lanes % kWave != 0; ++u)
    if (u * lanes % kWave == 0) U = u;
  const unsigned magic = (unsigned)(((1ull << 32) + lanes - 1) / lanes);
  const int Q = rotate && lanes <= 40 ? 2 : 1;
  bool warm = list && order_streams_x(d);
  int stretch = 0, warm_blocks = 0;
  int64_t warm_grid = 0;
  if (warm) {
    stretch = d.order_tiles * plan_tile_size(d.N);
    const int tokens = stretch / d.k + 2;                      // a stretch may begin and end inside a token
    warm_blocks = (tokens + U - 1) / U * kSlices;
    warm_grid = warm_blocks + ((int64_t)stretch + U * Q - 1) / (U * Q) * kSlices;
    warm = (uint64_t)warm_grid * (uint64_t)(U * lanes) <= kMostThreads;        // (not so from a few thousand branches a token on)
  }
  const bool alone = list && aligned && !warm && lanes > 96 && lanes <= 112;
  if (alone) U = 1, lanes = 128;
  // equal slices as pieces, from 256 bytes on (24-bit products); narrow rows that are read in bulk from 512 bytes on, units that are alone
  // in a workgroup in one block (see slice_col)
  int piece = d.H16 / kSlices, shift = 31;
  if (!rotate && !alone && d.H16 < 1 << 24 && (piece & -piece) >= (warm && d.H16 < 512 ? 32 : 16))
    piece &= -piece, shift = __builtin_ctz((unsigned)piece);
  const int per = U * Q;
  auto go = [&](auto kernel) {
    auto part = [&](dim3 grid, int start) {
      return launch(kernel, grid, dim3((unsigned)(U * lanes)), 0, s, (const u32x4 *)x,
                    (const int32_t *)(list ? p.order : p.row_map), (u32x4 *)window, d.k, d.H16, misalign, d.N, lanes, magic,
                    U, d.T, warm_blocks, start, piece, shift);
    };
    if (warm) return part(dim3((unsigned)warm_grid, (unsigned)((d.N + stretch - 1) / stretch)), stretch);
    // one launch, or as many as the limit on its threads asks for (windows of more than about 2 GiB at 16 bytes a row, 57 GiB
    // at 14 KB): `most` branches each
    const int64_t most = (int64_t)(kMostThreads / (unsigned)(U * lanes * kSlices)) * per;
    for (int64_t first = 0; first < d.N; first += most) {
      const int64_t groups = (std::min(most, d.N - first) + per - 1) / per;
      const hipError_t e = part(dim3((unsigned)(groups * kSlices)), (int)first);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  };
  if (alone) return rotate ? go(dispatch_units_kernel<1, true, true, true, false, true>)
                           : go(dispatch_units_kernel<1, true, false, true, false, true>);
#define GO(LIST_, WARM_)                                                                                     \
  if (list == LIST_ && warm == WARM_) {                                                                      \
    if (!aligned) return Q == 2 ? go(dispatch_units_kernel<2, LIST_, true, false, WARM_>)                    \
                                : go(dispatch_units_kernel<1, LIST_, true, false, WARM_>);                   \
    if (!rotate) return go(dispatch_units_kernel<1, LIST_, false, true, WARM_>);                             \
    return Q == 2 ? go(dispatch_units_kernel<2, LIST_, true, true, WARM_>)                                   \
                  : go(dispatch_units_kernel<1, LIST_, true, true, WARM_>);                                  \
  }
  GO(false, false)
  GO(true, false)
  GO(true, true)
#undef GO
  return hipErrorInvalidValue;
}

template <int J, int U>
static hipError_t launch_dispatch_ju(const Dims &d, const void *x, const PlanView &p, void *window, int rotate,
                                     hipStream_t s) {
  const unsigned units = (unsigned)(d.N / J);
  const dim3 grid((units + U - 1) / U * (unsigned)kSlices);
  if ((uint64_t)grid.x * 128 > kMostThreads && cuts_in_24_bits(d))
    return launch_dispatch_units(d, x, p, window, false, s);
  return launch(dispatch_slices_kernel<128, J, U>, grid, dim3(128), 0, s, (const u32x4 *)x,
                (const int32_t *)p.row_map, (u32x4 *)window, d.k, d.H16, rotate, d.N);
}

hipError_t launch_dispatch(const Dims &d, const void *x, const PlanView &p, void *window, hipStream_t s) {
  if (d.order_tiles > 0 && p.order && cuts_in_24_bits(d)) return launch_dispatch_units(d, x, p, window, true, s);
  // Rows that do not start at a cache line, and narrow rows while X is no larger than the Infinity Cache (us per
  // dispatch, units / token-order slices: H = 512, T = 32768 47 / 53; H = 640, T = 10000 20.6 / 21.1).
  const bool x_cold = (int64_t)d.T * d.H16 * 16 > ((int64_t)256 << 20);
  if (cuts_in_24_bits(d) && (d.H16 % kLine != 0 || ((uintptr_t)window >> 4) % kLine != 0 || (d.H16 < 96 && !x_cold)))
    return launch_dispatch_units(d, x, p, window, false, s);
  // A workgroup should move a few KB, so that the grid stays within what the dispatcher sustains (about 3000
  // workgroups per microsecond), with its lanes busy.
  //   Normally one unit per workgroup; a unit takes J branches of its token until it moves 4 KB (1.75 KB
  //   when the slice fills both waves): one load feeds J stores.
  //   Slices of at most 16 columns (H <= 1024 for bf16), or of at most 32 when the routing degree does not
  //   allow enough branches per unit: a unit is as many lanes as the slice has columns (a power of two, at
  //   least 8) and 128 / lanes units, i.e. branches of neighbouring tokens, share the workgroup; J until it
  //   moves 8 KB.
  // Measured in a plan -> dispatch -> combine sequence, k = 8, us per dispatch, this rule / one unit only:
  //   H = 512, T = 131072: 212 / 544;  H = 1024, T = 131072: 466 / 828;  H = 2048, T = 65536: 436 / 459;
  //   H = 2048, k = 6, T = 8192: 37 / 58 (launches alone).
  const int lines = (d.H16 + kLine - 1) / kLine;
  const int slice = (lines + kSlices - 1) / kSlices * kLine;
  const int rotate = lines % kSlices != 0 ? kSlices - 1 : 0;
  const int slice_bytes = slice * 16;
  int lanes = 8;                                   // lanes of a unit
  while (lanes < 128 && lanes < slice) lanes *= 2;
  int want = slice <= 64 ? 4096 : 1792;
  int U = 1, J = 1;
  while (J < 8 && J * slice_bytes < want && d.k % (2 * J) == 0) J *= 2;
  // An X larger than the Infinity Cache (256 MiB) comes from HBM whatever ran before.  Reads that miss it are
  // slow while the chip is saturated with writes, and the units of a (token, slice) all wait on the same lines,
  // so fewer, larger units do better there: 2 branches per unit, 8 where a slice is a single wave.
  // Measured, k = 8, us per dispatch with this rule / without: H = 7168: T = 20480 501 / 752, 24576 632 / 915,
  // 32768 943 / 1292; H = 4096, T = 65536: 957 / 1064 (J = 4) / 1961 (J = 1).
  if (x_cold) {
    const int most = slice <= 64 ? 8 : 2;
    while (J < most && d.k % (2 * J) == 0) J *= 2;
  }
  if (slice <= 16 || (slice <= 32 && J * slice_bytes < want)) {     // narrow, or the routing degree allows too few branches
    U = 128 / lanes;
    want = 8192;
    J = 1;
    while (J < 8 && U * J * slice_bytes < want && d.k % (2 * J) == 0) J *= 2;
  }
#define GO(J_, U_) if (J == J_ && U == U_) return launch_dispatch_ju<J_, U_>(d, x, p, window, rotate, s)
  GO(1, 1); GO(2, 1); GO(4, 1); GO(8, 1);
  GO(1, 2); GO(2, 2); GO(4, 2); GO(8, 2);
  GO(1, 4); GO(2, 4); GO(4, 4); GO(8, 4);
  GO(1, 8); GO(2, 8); GO(4, 8); GO(8, 8);
  GO(1, 16); GO(2, 16); GO(4, 16); GO(8, 16);
#undef GO
  return hipErrorInvalidValue;
}

// Which kernel a decode batch takes: compares and ballots while the counting is small (fewer barriers), the histogram beyond.
// us per dispatch, ballots / histogram, in replayed graphs on cold buffers, by the number of branches (E = 256, or 64 for degrees beyond 8):
//   k = 8: H = 2048: 1408 4.7 / 4.3, 5000 12.4 / 7.6; H = 4096: 1152 4.75 / 4.6, 1408 4.95 / 4.9, 5000 15.2 / 10.7; H = 5120: 1408 5.2 / 5.4, 1536 5.7 / 5.6,
//     3500 10.8 / 9.7; H = 7168: 1408 6.0 / 6.5, 1536 6.6 / 6.7, 1700 7.2 / 7.2, 2304 9.4 / 8.8; H = 10 240: 1408 7.9 / 8.0, 1700 10.6 / 9.1; H = 14 336: 1536
//     10.4 / 11.0, 1700 12.9 / 12.7.  More experts, H = 7168: E = 512: 1900 7.7 / 7.9, 2304 9.4 / 9.0; E = 1024: 2304 9.4 / 9.3, 3000 11.1 / 11.2
//   k = 6: H = 4096: 1404 5.9 / 5.0; H = 7168: 2304 9.4 / 9.9, 3500 13.0 / 13.0, 4092 15.7 / 14.3; H = 14 336: 1700 12.1 / 12.5, 3500 22.4 / 24.0, 4092 25.9 / 25.0
//   k = 10, H = 7168: 1400 7.2 / 6.6; k = 16: H = 2048: 1152 5.2 / 4.5; H = 7168: 1536 6.1 / 6.6, 1700 8.0 / 7.1
//   k = 5: H = 2048 (five slots for four waves): 600 4.2 / 4.3, 1020 4.35 / 4.6, 1400 5.5 / 4.9; E = 512: 1280 4.85 / 5.0, 1410 5.5 / 5.3; H = 4096: 600
//     4.45 / 4.35, 2300 7.45 / 6.45; H = 7168, E = 1024: 640 5.1 / 5.7, 1280 6.6 / 6.8, 1700 8.4 / 8.1
//   k = 4, 3, 2, 1, H = 4096: 600 4.45 / 4.35, 4.45 / 4.35, 4.85 / 4.45, 5.65 / 4.7; 5000 20 / 11.5, 23 / 15, 31 / 12.4, 54 / 15.4; k = 4, H = 7168, E = 1024: 1024
//     5.6 / 6.1, 1700 8.3 / 8.1
//   quantised: k = 8: H = 2048: 1152 4.45 / 4.6, 1280 4.5 / 4.55, 1536 4.8 / 4.6; H = 7168: 640 4.6 / 4.5, 1152 5.85 / 5.55, E = 1024: 1280 5.9 / 6.3, 1536 6.6 / 6.4;
//     k = 6, H = 2048: 1152 4.5 / 4.55, 1278 4.8 / 4.6; k = 10, H = 2048: 640 4.35 / 4.5, 1020 4.9 / 4.6; k = 5, H = 2048: 320 4.3 / 4.45, 640 4.7 / 4.6, E = 512: 640
//     4.8 / 5.2, 1025 5.65 / 5.3; k = 4, H = 4096: 128 4.4 / 4.15, 4096 14.7 / 7.8; k = 2, H = 2048, E = 512: 128 4.05 / 4.25, 320 4.4 / 4.4, 640 5.1 / 4.65
// (Rows of 1024 to 1280 vectors: where the workgroups of 5 waves fill the compute units unevenly the histogram loses: k = 8, 2600 branches 13.2 / 14.8.)
// With several source ranks always the histogram, to which the other ranks' rows are added.
static bool decode_by_hist(const Dims &d, const PlanView &p, bool quant) {
  if (p.source_count) return true;
  const bool wide = d.H16 > 1024;
  const int more = std::max(0, d.E - 256);            // experts past 256: the counts take longer to clear, scan and sum
  if (quant) {
    if (d.k == 5 && d.H16 <= 256) return d.N > 600 + more;
    if (d.k < 6) return wide || more == 0 || d.N > 256;
    if (d.k > 8 || !(d.H16 <= 256 || (d.E > 512 && !wide))) return d.N > 1024;
    return d.N > (d.k == 6 ? 1152 : 1280);
  }
  if (d.k == 5 && d.H16 <= 256) return d.N > 1152 + more;
  if (d.k < 6) return d.N > 600 + (d.E > 512 && d.k >= 3 && (d.k == 5 || !wide) ? more : 0);
  // rows of which the ballots' workgroups of 1024 vectors leave a large part idle
  const bool narrow = d.H16 <= 512 || (wide && d.H16 <= 1280);
  if (d.k > 8) return d.N > (narrow || d.k < 12 ? 1408 : 1536);
  if (narrow) return d.N > 1408;
  if (d.k == 6 && d.H16 > 832) return d.N > 3584;
  return d.N > 1536 + 2 * more;
}

template <int V, int TT, int G, bool QUANT>
static hipError_t launch_decode_hist_shape(const Dims &d, const void *x, const int32_t *K, const PlanView &p,
                                           void *window, float *window_scale, hipStream_t s) {
  constexpr int kMost = QUANT ? 1024 : 512;
  // chunks of nearly the same length, and as many waves as a chunk needs, but enough to count the ids
  const int chunks = (d.H16 + kMost * V - 1) / (kMost * V);
  const int width = ((d.H16 + chunks - 1) / chunks + kLine - 1) / kLine * kLine;
  // (7 waves: 8, us per dispatch, 7 / 8 waves, k = 8: H = 3584: 2600 branches 6.7 / 6.3, 4096 9.0 / 8.4; H = 6400, 4096 13.1 / 12.6; H = 7168: 2048 8.1 / 7.8, 4096
  // 14.4 / 13.8; H = 14 336, 4096 25.5 / 24.5; k = 2, H = 7168, 4096 17.4 / 16.0; equal elsewhere.  5 and 6 waves stay: k = 8: H = 5120, 3200 9.1 / 10.4, H = 6144,
  // 3200 10.5 / 11.7, H = 10 240, 1600 8.8 / 10.0; but 8 would do better in rows of one vector a lane: H = 2560, 2600 6.0 / 5.3, H = 3072, 4096 8.2 / 7.6)
  int threads = std::max(p.source_count ? 512 : 256, ((width + V - 1) / V + kWave - 1) / kWave * kWave);
  if (threads == 7 * kWave) threads = 8 * kWave;
  const int per_group = (d.k + G - 1) / G;
  const size_t lds = (size_t)(4 * d.E + 1 + 2) * sizeof(int);
  const dim3 grid((unsigned)((d.T + TT - 1) / TT) * (unsigned)(chunks * G) + 1u);
  auto go = [&](auto kernel) {
    return launch(kernel, grid, dim3((unsigned)threads), lds, s, (const u32x4 *)x, K, window, window_scale, d, p, chunks, width,
                  per_group);
  };
  return p.source_count ? go(decode_hist_kernel<kMost, V, TT, G, QUANT, true>)
                        : go(decode_hist_kernel<kMost, V, TT, G, QUANT, false>);
}

// How many branches a workgroup takes.  Degrees of 6 and more: a token's slots, in one workgroup or two.  More workgroups spread
// the stores, fewer repeat the counting less: us per dispatch, two / one, k = 8: H = 4096 (8 waves): T = 256 5.5 / 5.6, 320 6.5 / 6.4, 512
// 9.7 / 9.0; H = 2048 (4 waves): T = 512 6.5 / 6.6; H = 5120 (5 waves, 2 vectors a lane): T = 512 11.1 / 11.6; H = 7168: T = 384
// 12.0 / 11.1, 512 13.7 / 14.3; quantised H = 7168: T = 256 5.8 / 5.9, 384 9.1 / 7.4, 512 10.1 / 9.3.  With several sources every
// workgroup also adds up the count matrix, so one workgroup pays earlier: 32 sources, H = 7168: T = 64 5.3 / 5.65, 128 6.7 / 6.4, 512
// 16.1 / 14.0; k = 10, T = 300 10.7 / 10.8.
// Smaller degrees: whole tokens, up to 8 branches, as long as about 384 workgroups remain (k = 4, H = 4096, T = 800: two tokens 8.0,
// one 10.1; quantised T = 512: 5.5 / 5.1, T = 800 7.2 / 8.9).
template <int V, bool QUANT>
static hipError_t launch_decode_hist(const Dims &d, const void *x, const int32_t *K, const PlanView &p, void *window,
                                     float *window_scale, hipStream_t s) {
  if (d.k >= 6) {
    const bool whole = p.source_count ? d.N >= 1024 && d.k <= 8
                                      : d.H16 > 256 && (QUANT ? d.N > 2560 : d.H16 <= 512 && d.N > 2304);
    return whole ? launch_decode_hist_shape<V, 1, 1, QUANT>(d, x, K, p, window, window_scale, s)
                 : launch_decode_hist_shape<V, 1, 2, QUANT>(d, x, K, p, window, window_scale, s);
  }
  constexpr int kMost = QUANT ? 8 / V : 8;       // tokens whose rows fit in registers (with their codes)
  const int chunks = QUANT ? 1 : (d.H16 + 512 * V - 1) / (512 * V);
  int tt = d.k >= 5 ? 1 : d.k >= 3 ? 2 : d.k == 2 ? 4 : 8;
  while (tt > 1 && (tt > kMost || (int64_t)d.T * chunks < (int64_t)tt * 384)) tt /= 2;
  if (tt == 1) return launch_decode_hist_shape<V, 1, 1, QUANT>(d, x, K, p, window, window_scale, s);
  if (tt == 2) return launch_decode_hist_shape<V, 2, 1, QUANT>(d, x, K, p, window, window_scale, s);
  if (tt == 4) return launch_decode_hist_shape<V, 4 < kMost ? 4 : kMost, 1, QUANT>(d, x, K, p, window, window_scale, s);
  return launch_decode_hist_shape<V, kMost, 1, QUANT>(d, x, K, p, window, window_scale, s);
}

template <int B, int V, int SB, int G>
static hipError_t launch_decode_dispatch_shape(const Dims &d, const void *x, const int32_t *K, const PlanView &p,
                                               void *window, hipStream_t s) {
  const int chunks = (d.H16 + B * V - 1) / (B * V);
  const int per_group = ((d.k + G - 1) / G + SB - 1) / SB * SB;
  const size_t lds = (size_t)(4 * d.E + 1 + 2) * sizeof(int);
  const dim3 grid((unsigned)d.T * (unsigned)(chunks * G) + 1u);
  return launch(decode_dispatch_kernel<B, V, SB, G, false>, grid, dim3(B), lds, s, (const u32x4 *)x, K, window,
                (float *)nullptr, d, p, chunks, per_group);
}

hipError_t launch_decode_dispatch(const Dims &d, const void *x, const int32_t *K, const PlanView &p, void *window,
                                  hipStream_t s) {
  if (decode_by_hist(d, p, false))
    return d.H16 <= 512 ? launch_decode_hist<1, false>(d, x, K, p, window, nullptr, s)
                        : launch_decode_hist<2, false>(d, x, K, p, window, nullptr, s);
  // With a routing degree of at least 6 the slots of a token are split over 4 workgroups of 8 waves (2 slots
  // each), or over 2 (4 slots each) once the batch is so large that the counting, which every workgroup of a
  // token repeats over all ids, outweighs the better spread of the stores (degree 6, and batches of many experts).
  // Measured, k = 8, us per dispatch (one workgroup per token and chunk / two groups / four groups):
  //   H = 7168: T = 16: 3.9 / 3.5 / 3.5, T = 64: 4.2 / 4.0 / 4.1, T = 128: 5.4 / 4.9 / 4.8, T = 144: 6.0 / 5.5 / 5.2,
  //             T = 256: 8.8 / 8.0 / 7.7;  H = 4096: T = 128: 4.7 / 4.2 / 4.2, T = 256: 6.3 / 5.7 / 6.2.
  if (d.k >= 6) {
    if (d.N <= 1536) return launch_decode_dispatch_shape<512, 2, 2, 4>(d, x, K, p, window, s);
    return launch_decode_dispatch_shape<512, 2, 4, 2>(d, x, K, p, window, s);
  }
  // Few slots per token: one workgroup per token and chunk.  Every workgroup of a token repeats the
  // counting, so from about 900 branches on (which come here with more than 512 experts) two vectors per lane, half as many
  // chunks, win.
  if (d.H16 > 512 && d.N >= 896) return launch_decode_dispatch_shape<512, 2, 8, 1>(d, x, K, p, window, s);
  return launch_decode_dispatch_shape<512, 1, 8, 1>(d, x, K, p, window, s);
}

// Whole-row workgroup shapes (threads, vectors per thread) covering H16 <= 4096, for the quantised kernels.
// Prefill: one workgroup per token.  (Smaller workgroups with more vectors per thread, and the slots of a token
// split over 2-4 workgroups as in the decode kernel, change the dispatch by less than 2 % either way.)
#define MOE_QUANT_ROW_SHAPES(GO) \
  if (d.H16 <= 256) GO(256, 1);  \
  else if (d.H16 <= 512) GO(512, 1);  \
  else if (d.H16 <= 1024) GO(1024, 1); \
  else if (d.H16 <= 2048) GO(1024, 2); \
  else GO(1024, 4)
// Decode: 8 waves where they cover the row, as for the unquantised kernel.
#define MOE_QUANT_DECODE_SHAPES(GO) \
  if (d.H16 <= 256) GO(256, 1);  \
  else if (d.H16 <= 512) GO(512, 1);  \
  else if (d.H16 <= 1024) GO(512, 2); \
  else if (d.H16 <= 2048) GO(1024, 2); \
  else GO(1024, 4)

hipError_t launch_dispatch_quant(const Dims &d, const void *x, const PlanView &p, void *window_q, float *window_scale,
                                 hipStream_t s) {
#define GO(B_, V_)                                                                                         \
  return launch(dispatch_quant_rows_kernel<B_, V_>, dim3((unsigned)d.T), dim3(B_), 0, s, (const u32x4 *)x, \
                (const int32_t *)p.row_map, (u32x2 *)window_q, window_scale, d.k, d.H16)
  MOE_QUANT_ROW_SHAPES(GO);
#undef GO
}

template <int B, int V, int SB, int G>
static hipError_t launch_decode_quant_shape(const Dims &d, const void *x, const int32_t *K, const PlanView &p,
                                            void *window_q, float *window_scale, hipStream_t s) {
  const size_t lds = (size_t)(4 * d.E + 1 + 2) * sizeof(int);
  const int per_group = ((d.k + G - 1) / G + SB - 1) / SB * SB;
  const dim3 grid((unsigned)d.T * (unsigned)G + 1u);
  return launch(decode_dispatch_kernel<B, V, SB, G, true>, grid, dim3(B), lds, s, (const u32x4 *)x, K, window_q,
                window_scale, d, p, 1, per_group);
}

// Slot groups as in launch_decode_dispatch; no batch of more than 1280 branches comes here, and of smaller degrees only rows of up to 1024
// vectors (see decode_by_hist).  Measured, k = 8, us per quantised dispatch, one workgroup of 1024 threads per token / this rule: H = 7168:
// T = 32: 5.1 / 3.8, T = 128: 6.0 / 5.1; H = 4096, T = 128: 5.3 / 4.5; H = 2048, T = 128: 5.1 / 4.2.
template <int B, int V>
static hipError_t launch_decode_quant_bv(const Dims &d, const void *x, const int32_t *K, const PlanView &p,
                                         void *window_q, float *window_scale, hipStream_t s) {
  if constexpr (B < 1024)
    if (d.k < 6) return launch_decode_quant_shape<B, V, 8, 1>(d, x, K, p, window_q, window_scale, s);
  return launch_decode_quant_shape<B, V, 2, 4>(d, x, K, p, window_q, window_scale, s);
}

hipError_t launch_decode_dispatch_quant(const Dims &d, const void *x, const int32_t *K, const PlanView &p,
                                        void *window_q, float *window_scale, hipStream_t s) {
  if (decode_by_hist(d, p, true)) {
    if (d.H16 <= 512) return launch_decode_hist<1, true>(d, x, K, p, window_q, window_scale, s);
    if (d.H16 <= 2048) return launch_decode_hist<2, true>(d, x, K, p, window_q, window_scale, s);
    return launch_decode_hist<4, true>(d, x, K, p, window_q, window_scale, s);
  }
#define GO(B_, V_) return launch_decode_quant_bv<B_, V_>(d, x, K, p, window_q, window_scale, s)
  MOE_QUANT_DECODE_SHAPES(GO);
#undef GO
}

}  // namespace moe_rbf
