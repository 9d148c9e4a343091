// Duplicated entries, LSD radix sort of 64-bit (bin | depth) keys, bin ranges and masks.
//
// Background ("Gaussian sorting"): every Gaussian emits one entry per overlapped tile and
// the entries of a tile are ordered by depth with a radix sort.  With cross-tile grouping
// (Grouped Rasterization, Algorithm 1) the entry is per overlapped group of GxG tiles and
// carries a tile-membership bit mask; entries are ordered by (group, depth).
//
// Key = (bin << 32) | bits(float depth): depths are positive, so their IEEE bits order as
// unsigned integers.  An LSD radix sort takes the low (depth) digits first.  Those digits
// are a property of the Gaussian, not of the entry, so their passes run on the visible
// Gaussians before duplication (V elements instead of K entries): the visible list is
// sorted stably by depth bits, entries are emitted in that order (one thread per entry,
// load-balanced over Gaussians of any footprint), and the remaining passes sort the
// entries stably on the bin digits.  The result is exactly the stable sort of the 64-bit
// keys of Gaussian-major emission, i.e. the order (bin, depth bits, Gaussian index).
//
// Each pass is three kernels without inter-workgroup waits: per-tile digit counts, one
// workgroup per digit scanning its row of tile counts (and writing the row total), and a
// stable scatter that derives the digit bases from the row totals and writes each digit's
// run through LDS so that lanes store consecutive addresses.  The depth sort takes the 31
// bits of a positive depth in four passes (8, 8, 8 and 7 bits); its last pass also counts,
// per tile and digit, the entries of the keys' Gaussians, so that its scatter writes each
// Gaussian's first entry in depth order (the offset scan the binning needs) next to the
// sorted keys.  (Three passes of up to 11 bits were measured slower: a 2,048-digit pass
// costs nearly two 256-digit ones.)  These passes are bound by their launches, about 4 us each
// however few the keys: sorts of up to 1,024 tiles leave the scans of the first three passes out
// (DigitRows; preparation of 2M Gaussians 302 -> 295 us, a 4K frame 106 -> 101).
#include "gs_sort.hpp"

namespace gsi {
namespace {

__global__ __launch_bounds__(kBlock) void k_fill_u32(uint32_t *p, uint64_t n, uint32_t v) {
  uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (; i < n; i += stride) p[i] = v;
}

// ---- radix sort --------------------------------------------------------------
// Workgroup tile: 4 waves x R rounds x 64 lanes.  Wave w owns the contiguous sub-tile
// [w*64R, (w+1)*64R) and walks it in rounds of 64 consecutive keys, so (wave, round, lane)
// order is input order and per-digit ranks are stable.  Sorts of up to 2^20 keys use R = 4
// (1,024-key tiles: the ~200K visible Gaussians of a 1M scene still give ~200 workgroups, and
// the per-pass digit scans stay short; 512-key tiles were 1.3 % slower end to end), larger
// ones R = 8 (2,048 keys).
constexpr int kDigits = 256;                   // digits of at most 8 bits
// A sort of more than kSmallSort keys on exactly 9 bits (the bins of 4x4 groups at 1080p, 8x8
// at 2160p) takes them in one pass of 512 digits: one pass over the entries instead of two
// (5 + 4 bits), its per-tile counts still 1 byte per key with 2,048-key tiles.
constexpr int kWideDigits = 512;
constexpr int kWideBits = 9;
constexpr int kDepthBits = 31;                 // a positive float's sign bit is zero
constexpr int kSmallR = 4;                      // sorts up to kSmallSort keys: 1,024-key tiles
constexpr int kLargeR = 8;                      // larger sorts: 2,048-key tiles
constexpr uint64_t kSmallSort = 1ull << 20;
template <int R>
struct SortTile {
  static constexpr int kRounds = R;
  static constexpr int kWaveTile = R * 64;
  static constexpr int kTile = 4 * kWaveTile;
};

// lanes of the wave holding the same digit as this lane (among lanes with valid keys)
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid, int nbits) {
  uint64_t peers = __ballot(valid);
  for (int b = 0; b < nbits; ++b) {
    const bool bit = (d >> b) & 1u;
    const uint64_t m = __ballot(bit);
    peers &= bit ? m : ~m;
  }
  return peers;
}

__device__ __forceinline__ uint32_t block_exclusive_scan_u32(uint32_t v, uint32_t *sh4, uint32_t *total) {
  return block_exclusive_scan_t<uint32_t>(v, sh4, total);
}

// Blocks of 8x8 tiles that a footprint overlaps.
__device__ __forceinline__ uint32_t rect_blocks(ushort4 r) {
  return (uint32_t)(((r.z - 1) / kBlockTiles - r.x / kBlockTiles + 1) *
                    ((r.w - 1) / kBlockTiles - r.y / kBlockTiles + 1));
}

// Entries of Gaussian g (EntryCounts).
__device__ __forceinline__ uint32_t entries_of(const EntryCounts &e, uint32_t g) {
  if (!e.rect) return e.count[g];
  const uint32_t n = rect_blocks(e.rect[g]);
  return e.count ? min(n, e.count[g]) : n;
}

// Weights of the depth sort's last pass: the entries of each key's Gaussian vals[i], gathered by the
// count kernel and left in key order in weights[i] for the scatter (a second gather of 6M
// Gaussians' footprints in depth order took 19 us), summed per tile and digit into
// wcounts[d * tiles + tile], scanned over the tiles of each digit into wprefix (64-bit) with the
// digit totals in wtotals.
struct DigitWeights {
  const uint32_t *vals;
  EntryCounts entries;
  uint32_t *weights;
  uint32_t *wcounts;
  uint64_t *wprefix;
  uint64_t *wtotals;
};

// Per-tile digit counts: counts[d * tiles + tile].  Keys are loaded up front (8 in flight
// per lane) and counted with one LDS atomic each.
template <typename KT, int R, int DIG, bool WEIGHTED>
__global__ __launch_bounds__(kBlock) void k_radix_count(const KT *keys, uint64_t n_host, const uint32_t *n_dev,
                                                        int shift, int nbits, uint32_t tiles_max, uint32_t *counts,
                                                        DigitWeights wt) {
  constexpr int kRounds = SortTile<R>::kRounds, kWaveTile = SortTile<R>::kWaveTile, kSortTile = SortTile<R>::kTile;
  // (weighted: the digits are the depths' exponents, a few of which hold all keys; 8 counters of each, for
  // the lanes in turn, instead of atomics all on the same ones)
  constexpr int C = WEIGHTED ? 8 : 1;
  __shared__ uint32_t h[DIG * C / (WEIGHTED ? 2 : 1)];   // (at most 7 bits)
  __shared__ uint32_t hw[WEIGHTED ? DIG * C / 2 : 1];
  const uint64_t n = count_of(n_host, n_dev);
  const uint32_t tile = xcd_sort_tile(blockIdx.x, (n + kSortTile - 1) / kSortTile);
  if (tile == ~0u) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int ndig = 1 << nbits;
  for (int d = t; d < ndig * C; d += kBlock) {
    h[d] = 0;
    if (WEIGHTED) hw[d] = 0;
  }
  const uint32_t dmask = (1u << nbits) - 1u;
  const uint64_t base = (uint64_t)tile * kSortTile + (uint64_t)w * kWaveTile;
  KT key[kRounds];
  uint32_t c[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    key[r] = i < n ? keys[i] : (KT)0;
    c[r] = WEIGHTED && i < n ? wt.vals[i] : 0u;
  }
  if (WEIGHTED) {
#pragma unroll
    for (int r = 0; r < kRounds; ++r) c[r] = base + (uint64_t)r * 64 + lane < n ? entries_of(wt.entries, c[r]) : 0u;
  }
  block_sync();
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const bool valid = base + (uint64_t)r * 64 + lane < n;
    const uint32_t d = (uint32_t)(key[r] >> shift) & dmask;
    if (valid) {
      if (WEIGHTED) wt.weights[base + (uint64_t)r * 64 + lane] = c[r];
      const uint32_t k = d * C + (lane & (C - 1));
      atomicAdd(&h[k], 1u);   // (cheaper than grouping equal digits per wave first)
      if (WEIGHTED) atomicAdd(&hw[k], c[r]);
    }
  }
  block_sync();
  for (int d = t; d < ndig; d += kBlock) {
    uint32_t s = 0, sw = 0;
#pragma unroll
    for (int k = 0; k < C; ++k) {
      s += h[d * C + k];
      if (WEIGHTED) sw += hw[d * C + k];
    }
    counts[(uint64_t)d * tiles_max + tile] = s;
    if (WEIGHTED) wt.wcounts[(uint64_t)d * tiles_max + tile] = sw;
  }
}

// One workgroup per digit d: counts[d][*] becomes the exclusive prefix over tiles (within the
// digit) and totals[d] the digit's total.
// With weights (wt.wcounts), the digit's row of weights likewise into wt.wprefix and wt.wtotals.
__global__ __launch_bounds__(kBlock) void k_radix_digit_scan(uint32_t *counts, uint32_t tiles_max,
                                                             uint32_t *totals, uint64_t n_host, const uint32_t *n_dev,
                                                             uint32_t tile_size, DigitWeights wt) {
  __shared__ uint32_t sh[4];
  __shared__ uint64_t sh8[4];
  const int d = blockIdx.x, t = threadIdx.x;
  uint32_t *row = counts + (uint64_t)d * tiles_max;
  // tiles holding keys (the count kernel wrote no counts for the others)
  const uint64_t n = count_of(n_host, n_dev);
  const uint32_t tiles = (uint32_t)((n + tile_size - 1) / tile_size);
  const uint32_t per = (tiles + kBlock - 1) / kBlock;
  const uint32_t b0 = t * per;
  uint32_t s = 0;
  for (uint32_t i = 0; i < per; ++i)
    if (b0 + i < tiles) s += row[b0 + i];
  uint32_t tot;
  uint32_t run = block_exclusive_scan_u32(s, sh, &tot);
  if (t == 0) totals[d] = tot;
  for (uint32_t i = 0; i < per; ++i)
    if (b0 + i < tiles) {
      const uint32_t c = row[b0 + i];
      row[b0 + i] = run;
      run += c;
    }
  if (wt.wcounts) {
    const uint32_t *wrow = wt.wcounts + (uint64_t)d * tiles_max;
    uint64_t *prow = wt.wprefix + (uint64_t)d * tiles_max;
    uint64_t ws = 0;
    for (uint32_t i = 0; i < per; ++i)
      if (b0 + i < tiles) ws += wrow[b0 + i];
    uint64_t wtot;
    uint64_t wrun = block_exclusive_scan_t<uint64_t>(ws, sh8, &wtot);
    if (t == 0) wt.wtotals[d] = wtot;
    for (uint32_t i = 0; i < per; ++i)
      if (b0 + i < tiles) {
        prow[b0 + i] = wrun;
        wrun += wrow[b0 + i];
      }
  }
}

// Digit counts of a depth pass as rows, for sorts of few tiles: 16-bit counts of every group of
// 2^gshift tiles (group[g * 256 + d]) and, with gshift > 0, of the group's tiles before each tile
// (before[tile * 256 + d]).  A scatter workgroup adds up all the rows by itself (sum_rows), which needs
// no scan between the count and the scatter: 200 tiles (1M Gaussians, a fifth visible) in 50 groups are
// 25 KB to read from L2 and 2 us, in place of a launch of 4.3.
constexpr int kRowShift = 2;
struct DigitRows {
  uint16_t *group;
  uint16_t *before;
  int gshift;
};

// Rows of 4 tiles by a workgroup of 4 x 256 threads.  (The weighted last pass is left to the scan: its
// gathers want more workgroups than a quarter of the tiles, 9.7 us against 6.1 at 200 tiles.)
template <int R>
__global__ __launch_bounds__(kBlock << kRowShift) void k_count_rows(const uint32_t *keys, const uint32_t *n_dev,
                                                                    int shift, int nbits, DigitRows rows) {
  constexpr int kWaveTile = SortTile<R>::kWaveTile, kSortTile = SortTile<R>::kTile, kTiles = 1 << kRowShift;
  __shared__ uint32_t h[kTiles][kDigits];
  const uint64_t n = *n_dev;
  const uint32_t tiles = (uint32_t)((n + kSortTile - 1) / kSortTile);
  const uint32_t tile0 = blockIdx.x << kRowShift;
  if (tile0 >= tiles) return;
  const int t = threadIdx.x & (kBlock - 1), tl = threadIdx.x / kBlock, lane = t & 63, w = t >> 6;
  h[tl][t] = 0;
  const uint32_t dmask = (1u << nbits) - 1u;
  const uint64_t base = (uint64_t)(tile0 + tl) * kSortTile + (uint64_t)w * kWaveTile;
  uint32_t key[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    key[r] = i < n ? keys[i] : 0u;
  }
  block_sync();
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (base + (uint64_t)r * 64 + lane < n) atomicAdd(&h[tl][(key[r] >> shift) & dmask], 1u);
  block_sync();
  uint32_t pre = 0;
#pragma unroll
  for (int k = 0; k < kTiles; ++k) pre += k < tl ? h[k][t] : 0u;
  if (tile0 + tl < tiles) rows.before[(uint64_t)(tile0 + tl) * kDigits + t] = (uint16_t)pre;
  if (tl == kTiles - 1) rows.group[(uint64_t)blockIdx.x * kDigits + t] = (uint16_t)(pre + h[tl][t]);
}

// Sums over the workgroup of the rows [0, mid) and [0, end), of this thread's digit.  Each half-wave
// takes every eighth row, 8 loads in flight, and the halves meet in part (2 x 8 rows of sums).
__device__ __forceinline__ void sum_rows(const uint16_t *rows, uint32_t mid, uint32_t end, uint32_t *part,
                                         uint32_t *before, uint32_t *all) {
  uint32_t a[8] = {}, b[8] = {};   // all rows, and those before mid
  const uint4 *p = reinterpret_cast<const uint4 *>(rows) + (threadIdx.x & 31);
  const int half = threadIdx.x >> 5, col = (threadIdx.x & 31) * 8;
  for (uint32_t r = half; r < end; r += 64) {
    uint4 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = r + 8u * k < end ? p[(uint64_t)(r + 8u * k) * 32] : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 8; q += 4) {
      uint32_t x[4] = {}, y[4] = {};   // (four rows' 16-bit pairs add up in place: a row's count is at most 2^13)
#pragma unroll
      for (int k = q; k < q + 4; ++k) {
        const uint32_t u[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
        const uint32_t m = r + 8u * k < mid ? ~0u : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          x[j] += u[j];
          y[j] += u[j] & m;
        }
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        a[j] += (j & 1) ? x[j / 2] >> 16 : x[j / 2] & 0xffffu;
        b[j] += (j & 1) ? y[j / 2] >> 16 : y[j / 2] & 0xffffu;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    part[half * kDigits + col + j] = a[j];
    part[(8 + half) * kDigits + col + j] = b[j];
  }
  block_sync();
  uint32_t x = 0, y = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    x += part[k * kDigits + threadIdx.x];
    y += part[(8 + k) * kDigits + threadIdx.x];
  }
  *all = x;
  *before = y;
}

// Stable scatter of one tile: ranks from per-wave digit counters; the tile's start for digit
// d is (keys with a smaller digit) + offsets[d][tile]; keys are placed in LDS in tile-local
// digit order and then stored so that consecutive lanes write consecutive addresses.
// Final placement of the bin sort's last pass (fin != nullptr): the value of each key is the
// rank of its Gaussian in depth order; instead of the rank the pass writes the Gaussian index
// order[rank] to vals and the 64-bit key (bin << 32) | dkeys[rank] to keys (the two V-sized
// arrays stay in cache), next to the sorted bin keys.
struct FinalOut {
  const uint32_t *order;   // visible Gaussians in depth order
  const uint32_t *dkeys;   // their depth bits
  uint32_t *vals;          // Gaussian index of each sorted entry
  uint64_t *keys;          // 64-bit key of each sorted entry
  uint32_t bin_mask;       // the bin bits of a sort key (above them: the member-tile rectangle)
};

// First entries of the depth sort's last pass (WEIGHTED): dpos[p] = the entries of the
// Gaussians before the p-th in depth order, i.e. the exclusive scan of their entry counts
// (dpos[n] = all entries), and first[b] = p for every block b of kFirstsBlock entries whose
// first entry is one of the p-th Gaussian's (b < nfirst).  The key's place among the entries
// is the digit's weight base (the weights of smaller digits, then of this digit in earlier
// tiles) plus the weights of the keys before it in its tile's run of the digit.
struct FirstEntries {
  uint64_t *dpos;
  uint32_t *first;
  uint64_t nfirst;
  uint32_t *total;              // if set: all entries, at most *limit (32 bits, for the kernels that follow)
  const uint32_t *limit;
};

// Chunk table of the two-level binning (start != nullptr; one pass over the block bits): before each
// block, the entries (high word) and chunks of `chunk` entries (low word); start[digits] = all.
struct ChunkTable {
  uint64_t *start;
  uint32_t chunk;
};

// ROWS: the counts are rows (DigitRows; 256 digits), else scanned (k_radix_digit_scan).
template <typename KT, int R, int DIG, bool WEIGHTED, bool ROWS>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(const KT *kin, const uint32_t *vin, KT *kout, uint32_t *vout,
                                                          uint64_t n_host, const uint32_t *n_dev, int shift, int nbits,
                                                          uint32_t tiles_max, const uint32_t *offsets,
                                                          const uint32_t *totals, FinalOut fin, DigitWeights wt,
                                                          FirstEntries fe, ChunkTable ct, DigitRows rows) {
  constexpr int kRounds = SortTile<R>::kRounds, kWaveTile = SortTile<R>::kWaveTile, kSortTile = SortTile<R>::kTile;
  constexpr int M = DIG / kBlock;   // digits per thread in the digit-level scans
  static_assert(DIG % kBlock == 0, "digits in whole multiples of the workgroup");
  __shared__ uint32_t wcnt[4][DIG];
  __shared__ uint32_t bstart[DIG];
  __shared__ uint32_t gbase[DIG];
  __shared__ uint32_t sh4[4];
  __shared__ uint64_t sh8[4];
  __shared__ KT s_key[kSortTile];
  __shared__ uint32_t s_val[kSortTile];
  __shared__ uint64_t gw[WEIGHTED ? DIG : 1];          // weight base of each digit in this tile
  __shared__ uint32_t s_w[WEIGHTED ? kSortTile : 1];   // key weights in tile-local sorted order
  __shared__ uint32_t s_wx[WEIGHTED ? kSortTile : 1];  // their exclusive scan
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint64_t n = count_of(n_host, n_dev);
  if (WEIGHTED && n == 0 && blockIdx.x == 0 && t == 0) {   // no keys: no entries
    fe.dpos[0] = 0;
    if (fe.total) *fe.total = 0u;
  }
  const uint32_t tile = xcd_sort_tile(blockIdx.x, (n + kSortTile - 1) / kSortTile);
  if (tile == ~0u) return;
  const uint64_t tile0 = (uint64_t)tile * kSortTile;
  const int ndig = 1 << nbits;
  const uint32_t dmask = (1u << nbits) - 1u;
  const uint64_t lt = (1ull << lane) - 1ull;
  const uint64_t base = tile0 + (uint64_t)w * kWaveTile;
  KT key[kRounds];
  uint32_t val[kRounds], pos[kRounds], dig[kRounds], kw[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    key[r] = i < n ? kin[i] : (KT)0;
    val[r] = i < n ? vin[i] : 0u;
    kw[r] = WEIGHTED && i < n ? wt.weights[i] : 0u;
  }
  // this thread's digits t*M .. t*M + M - 1: their totals, this tile's offsets within them and,
  // weighted, the same two of the weights
  uint32_t tot_d[M], off_d[M];
  uint64_t wtot_d[WEIGHTED ? M : 1], woff_d[WEIGHTED ? M : 1];
  if constexpr (ROWS) {
    static_assert(M == 1 && DIG == kDigits && !WEIGHTED, "a digit per thread");
    __shared__ uint32_t part[16 * kDigits];
    const uint32_t tiles = (uint32_t)((n + kSortTile - 1) / kSortTile);
    const uint32_t in_group = rows.gshift ? rows.before[(uint64_t)tile * kDigits + t] : 0u;
    sum_rows(rows.group, tile >> rows.gshift, (tiles + (1u << rows.gshift) - 1u) >> rows.gshift, part, &off_d[0],
             &tot_d[0]);
    off_d[0] += in_group;
  } else
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const int d = t * M + j;
    tot_d[j] = d < ndig ? totals[d] : 0u;
    off_d[j] = d < ndig ? offsets[(uint64_t)d * tiles_max + tile] : 0u;
    if (WEIGHTED) {
      wtot_d[j] = d < ndig ? wt.wtotals[d] : 0ull;
      woff_d[j] = d < ndig ? wt.wprefix[(uint64_t)d * tiles_max + tile] : 0ull;
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    for (int d = t; d < ndig; d += kBlock) wcnt[k][d] = 0;
  block_sync();
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const bool valid = base + (uint64_t)r * 64 + lane < n;
    const uint32_t d = (uint32_t)(key[r] >> shift) & dmask;
    dig[r] = d;
    const uint64_t peers = match_digit(d, valid, nbits);
    const uint32_t rank = (uint32_t)__popcll(peers & lt);
    const uint32_t old = wcnt[w][d];
    pos[r] = old + rank;
    // every lane of the wave has read the counter before the group's first lane updates it,
    // and the update is visible to the whole wave before the next round reads (the counters
    // are written and read by lanes of this wave only; the fences order the LDS accesses
    // across the barrier for the compiler as well as the hardware)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (valid && rank == 0) wcnt[w][d] = old + (uint32_t)__popcll(peers);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  block_sync();
  // per digit: tile-local start (scan over digits of the tile's counts) and global start
  // (scan over digits of the totals, plus this tile's offset within the digit)
  uint32_t c[M][4], loc = 0, gsum = 0;
  uint64_t wsum = 0;
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const int d = t * M + j;
#pragma unroll
    for (int k = 0; k < 4; ++k) c[j][k] = d < ndig ? wcnt[k][d] : 0u;
    loc += c[j][0] + c[j][1] + c[j][2] + c[j][3];
    gsum += tot_d[j];
    if (WEIGHTED) wsum += wtot_d[j];
  }
  uint32_t all;
  uint32_t bs = block_exclusive_scan_u32(loc, sh4, &all);
  uint32_t gb = block_exclusive_scan_u32(gsum, sh4, &all);
  uint64_t wall = 0, wb = 0;
  if (WEIGHTED) wb = block_exclusive_scan_t<uint64_t>(wsum, sh8, &wall);
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const int d = t * M + j;
    if (d < ndig) {
      bstart[d] = bs;
      gbase[d] = gb + off_d[j];
      wcnt[0][d] = bs;
      wcnt[1][d] = bs + c[j][0];
      wcnt[2][d] = bs + c[j][0] + c[j][1];
      wcnt[3][d] = bs + c[j][0] + c[j][1] + c[j][2];
      if (WEIGHTED) gw[d] = wb + woff_d[j];
    }
    bs += c[j][0] + c[j][1] + c[j][2] + c[j][3];
    gb += tot_d[j];
    if (WEIGHTED) wb += wtot_d[j];
  }
  if (!WEIGHTED && ct.start && tile == 0) {   // (uniform)
    uint64_t v[M], sum = 0, call;
#pragma unroll
    for (int j = 0; j < M; ++j) {
      v[j] = (uint64_t)tot_d[j] << 32 | (tot_d[j] + ct.chunk - 1u) / ct.chunk;
      sum += v[j];
    }
    uint64_t run = block_exclusive_scan_t<uint64_t>(sum, sh8, &call);
#pragma unroll
    for (int j = 0; j < M; ++j) {
      if (t * M + j <= ndig) ct.start[t * M + j] = run;
      run += v[j];
    }
    if (t == 0) ct.start[ndig] = call;
  }
  if (WEIGHTED && tile == 0 && t == 0) {
    fe.dpos[n] = wall;
    if (fe.total) *fe.total = wall < (uint64_t)*fe.limit ? (uint32_t)wall : *fe.limit;
  }
  block_sync();
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const uint64_t i = base + (uint64_t)r * 64 + lane;
    if (i < n) {
      const uint32_t lp = wcnt[w][dig[r]] + pos[r];
      s_key[lp] = key[r];
      s_val[lp] = val[r];
      if (WEIGHTED) s_w[lp] = kw[r];
    }
  }
  block_sync();
  const uint32_t nvalid = (uint32_t)((n - tile0) < (uint64_t)kSortTile ? (n - tile0) : (uint64_t)kSortTile);
  if (WEIGHTED) {
    // exclusive scan of the weights in tile-local sorted order (R consecutive keys per thread;
    // 32 bits hold a tile's sum unless the frame has 2^32 entries, which the caller rejects)
    uint32_t x[kRounds], ssum = 0;
#pragma unroll
    for (int q = 0; q < kRounds; ++q) {
      const uint32_t i = (uint32_t)t * kRounds + q;
      x[q] = i < nvalid ? s_w[i] : 0u;
      ssum += x[q];
    }
    uint32_t tall;
    uint32_t ex = block_exclusive_scan_u32(ssum, sh4, &tall);
#pragma unroll
    for (int q = 0; q < kRounds; ++q) {
      s_wx[t * kRounds + q] = ex;
      ex += x[q];
    }
    block_sync();
    for (uint32_t i = t; i < nvalid; i += kBlock) {
      const KT k = s_key[i];
      const uint32_t d = (uint32_t)(k >> shift) & dmask;
      const uint32_t p = gbase[d] + (i - bstart[d]);
      kout[p] = k;
      vout[p] = s_val[i];
      const uint64_t o = gw[d] + (s_wx[i] - s_wx[bstart[d]]);
      fe.dpos[p] = o;
      const uint64_t end = o + s_w[i];
      for (uint64_t bk = (o + kFirstsBlock - 1) / kFirstsBlock; bk * kFirstsBlock < end && bk < fe.nfirst; ++bk)
        fe.first[bk] = p;
    }
    return;
  }
  if (fin.vals) {
    // all gathers of the thread first, then the stores (several round trips in flight)
    uint32_t gi[kRounds], dk[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const uint32_t i = (uint32_t)t + (uint32_t)r * kBlock;
      const uint32_t v = i < nvalid ? s_val[i] : 0u;
      gi[r] = i < nvalid ? fin.order[v] : 0u;
      dk[r] = i < nvalid ? fin.dkeys[v] : 0u;
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const uint32_t i = (uint32_t)t + (uint32_t)r * kBlock;
      if (i >= nvalid) break;
      const KT k = s_key[i];
      const uint32_t d = (uint32_t)(k >> shift) & dmask;
      const uint32_t p = gbase[d] + (i - bstart[d]);
      kout[p] = k;
      fin.vals[p] = gi[r];
      fin.keys[p] = ((uint64_t)((uint32_t)k & fin.bin_mask) << 32) | dk[r];
    }
    return;
  }
  for (uint32_t i = t; i < nvalid; i += kBlock) {
    const KT k = s_key[i];
    const uint32_t d = (uint32_t)(k >> shift) & dmask;
    kout[gbase[d] + (i - bstart[d])] = k;
    vout[gbase[d] + (i - bstart[d])] = s_val[i];
  }
}

// Depth keys of the visible Gaussians (key[i] = bits(depth of order[i]), i < *nvis), the entry
// and visible counts, and the first depth pass's per-tile digit counts (one workgroup per sort
// tile of R x 256 keys; counts[d * tiles + tile] for the digit bits [0, nbits0)).
// ROWS: the counts as a 16-bit row per tile (DigitRows with gshift 0).
template <int R, bool ROWS>
__global__ __launch_bounds__(kBlock) void k_depth_keys(const uint32_t *order, const float4 *rgb, const uint32_t *nvis,
                                                       uint32_t *keys, const uint64_t *K, uint64_t *counts,
                                                       uint64_t *host_counts, uint64_t capacity, int nbits0,
                                                       uint32_t *dcounts, uint32_t tiles) {
  constexpr int kSortTile = SortTile<R>::kTile;
  __shared__ uint32_t h[kDigits];
  const uint32_t V = *nvis;
  if (blockIdx.x == 0 && threadIdx.x == 0) {   // the entry and visible counts, side by side
    const uint64_t k = *K;
    counts[0] = k;
    counts[1] = V;
    // the entry count of a bin sort that reads it on the device: 0 (nothing binned) on overflow
    reinterpret_cast<uint32_t *>(counts + 2)[0] = k <= capacity ? (uint32_t)k : 0u;
    if (host_counts) {     // the caller's pinned host memory, polled by the host
      host_counts[0] = k;
      host_counts[1] = V;
    }
  }
  // the tile order of the sort's own passes over the V keys
  const uint32_t tile = xcd_sort_tile(blockIdx.x, ((uint64_t)V + kSortTile - 1) / kSortTile);
  if (tile == ~0u) return;
  const uint64_t tile0 = (uint64_t)tile * kSortTile;
  const int ndig = 1 << nbits0;
  for (int d = threadIdx.x; d < ndig; d += kBlock) h[d] = 0;
  block_sync();
  const uint32_t dmask = (1u << nbits0) - 1u;
  uint32_t g[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint64_t i = tile0 + (uint64_t)r * kBlock + threadIdx.x;
    g[r] = i < V ? order[i] : 0u;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const uint64_t i = tile0 + (uint64_t)r * kBlock + threadIdx.x;
    if (i < V) {
      const uint32_t k = __float_as_uint(rgb[g[r]].w);
      keys[i] = k;
      atomicAdd(&h[k & dmask], 1u);
    }
  }
  block_sync();
  if constexpr (ROWS) {
    static_assert(kDigits == kBlock, "a digit per thread");
    reinterpret_cast<uint16_t *>(dcounts)[(uint64_t)tile * kDigits + threadIdx.x] = (uint16_t)h[threadIdx.x];
    return;
  }
  for (int d = threadIdx.x; d < ndig; d += kBlock) dcounts[(uint64_t)d * tiles + tile] = h[d];
}

// The whole depth sort of a small scene in one workgroup: the keys stay in LDS over the four passes and
// the weights are scanned at the end.  The passes above are eleven launches of about 4 us, whatever
// their size; this is bound by its own serial steps, about 5 us a pass (a frame of 4,096 Gaussians, all
// visible, 81 -> 69 us; of 8,192, 94 -> 89, beyond which the keys outgrow one CU).
// Each pass ranks as k_radix_scatter does, wave by wave over consecutive keys.
constexpr int kOneR = 8;
constexpr int kOneThreads = 1024;
constexpr uint64_t kOneKeys = (uint64_t)kOneR * kOneThreads;

__global__ __launch_bounds__(kOneThreads) void k_depth_sort_one(uint32_t *order, const float4 *rgb,
                                                                const uint32_t *nvis, uint32_t *keys,
                                                                const uint64_t *K, uint64_t *counts,
                                                                uint64_t *host_counts, uint64_t capacity,
                                                                EntryCounts bins, EntryCounts blocks, BlockRule rule,
                                                                FirstEntries fe) {
  constexpr int kWaves = kOneThreads / 64;
  __shared__ uint32_t s_key[kOneKeys];
  __shared__ uint32_t s_val[kOneKeys];
  __shared__ uint16_t wcnt[kWaves][kDigits];
  __shared__ uint32_t sh4[4];
  __shared__ uint64_t sh16[kWaves];
  __shared__ uint32_t s_and, s_or;
  __shared__ bool s_blocks;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint32_t n = *nvis;   // at most kOneKeys: the host's bound
  uint32_t limit = 0;
  if (t == 0) {   // (as k_depth_keys)
    s_and = ~0u;
    s_or = 0u;
    const uint64_t k = *K;
    s_blocks = rule.takes(k, n);
    counts[0] = k;
    counts[1] = n;
    limit = k <= capacity ? (uint32_t)k : 0u;
    reinterpret_cast<uint32_t *>(counts + 2)[0] = limit;
    if (host_counts) {
      host_counts[0] = k;
      host_counts[1] = n;
    }
  }
  const uint32_t rounds = (n + kOneThreads - 1) / kOneThreads;   // of 64 keys per wave
  const uint32_t base = (uint32_t)w * 64 * rounds + lane;
  const uint64_t lt = (1ull << lane) - 1ull;
  uint32_t key[kOneR], val[kOneR], pos[kOneR];
#pragma unroll
  for (int r = 0; r < kOneR; ++r) {
    const uint32_t i = base + 64u * r;
    val[r] = (uint32_t)r < rounds && i < n ? order[i] : 0u;
  }
#pragma unroll
  for (int r = 0; r < kOneR; ++r)
    key[r] = (uint32_t)r < rounds && base + 64u * r < n ? __float_as_uint(rgb[val[r]].w) : 0u;
  // digits that all keys share need no pass (the depths' exponents, often)
  uint32_t ka = ~0u, ko = 0u;
#pragma unroll
  for (int r = 0; r < kOneR; ++r) {
    if ((uint32_t)r < rounds && base + 64u * r < n) {
      ka &= key[r];
      ko |= key[r];
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    ka &= __shfl_xor(ka, off, 64);
    ko |= __shfl_xor(ko, off, 64);
  }
  block_sync();
  if (lane == 0) {
    atomicAnd(&s_and, ka);
    atomicOr(&s_or, ko);
  }
  block_sync();
  const uint32_t differ = s_and ^ s_or;
  for (int shift = 0; shift < kDepthBits; shift += 8) {
    if (((differ >> shift) & 0xffu) == 0u) continue;   // (uniform)
    for (int d = lane; d < kDigits; d += 64) wcnt[w][d] = 0;
    block_sync();   // (and every wave has read its keys of the pass before)
#pragma unroll
    for (int r = 0; r < kOneR; ++r) {
      if ((uint32_t)r >= rounds) break;
      const bool valid = base + 64u * r < n;
      const uint32_t d = (key[r] >> shift) & 0xffu;
      const uint64_t peers = match_digit(d, valid, 8);
      const uint32_t rank = (uint32_t)__popcll(peers & lt);
      const uint32_t old = wcnt[w][d];
      pos[r] = old + rank;
      // (the counters are this wave's own: see k_radix_scatter)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if (valid && rank == 0) wcnt[w][d] = (uint16_t)(old + (uint32_t)__popcll(peers));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    block_sync();
    // the digits' starts, one digit per thread of the first four waves
    uint32_t c[kWaves], all = 0, incl = 0;
    if (t < kDigits) {
#pragma unroll
      for (int k = 0; k < kWaves; ++k) {
        c[k] = wcnt[k][t];
        all += c[k];
      }
      incl = all;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(incl, off, 64);
        if (lane >= off) incl += u;
      }
      if (lane == 63) sh4[w] = incl;
    }
    block_sync();
    if (t < kDigits) {
      uint32_t run = incl - all;
#pragma unroll
      for (int k = 0; k < 4; ++k) run += k < w ? sh4[k] : 0u;
#pragma unroll
      for (int k = 0; k < kWaves; ++k) {
        wcnt[k][t] = (uint16_t)run;
        run += c[k];
      }
    }
    block_sync();
#pragma unroll
    for (int r = 0; r < kOneR; ++r) {
      if ((uint32_t)r < rounds && base + 64u * r < n) {
        const uint32_t p = wcnt[w][(key[r] >> shift) & 0xffu] + pos[r];
        s_key[p] = key[r];
        s_val[p] = val[r];
      }
    }
    block_sync();
#pragma unroll
    for (int r = 0; r < kOneR; ++r) {
      const uint32_t i = base + 64u * r;
      key[r] = (uint32_t)r < rounds && i < n ? s_key[i] : 0u;
      val[r] = (uint32_t)r < rounds && i < n ? s_val[i] : 0u;
    }
  }
  // keys and Gaussians out; the entries before each, over consecutive keys of each lane and round
  const bool by_blocks = s_blocks;
  const EntryCounts entries{by_blocks ? blocks.count : bins.count, by_blocks ? blocks.rect : nullptr};
  uint32_t ew[kOneR];
#pragma unroll
  for (int r = 0; r < kOneR; ++r) {
    const uint32_t i = base + 64u * r;
    const bool in = (uint32_t)r < rounds && i < n;
    if (in) {
      keys[i] = key[r];
      order[i] = val[r];
    }
    ew[r] = in ? entries_of(entries, val[r]) : 0u;
  }
  uint64_t ex[kOneR], wave_sum = 0;   // entries of the wave's keys before each
#pragma unroll
  for (int r = 0; r < kOneR; ++r) {
    uint64_t incl = ew[r];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint64_t u = __shfl_up(incl, off, 64);
      if (lane >= off) incl += u;
    }
    ex[r] = wave_sum + incl - ew[r];
    wave_sum += __shfl(incl, 63, 64);
  }
  if (lane == 0) sh16[w] = wave_sum;
  block_sync();
  uint64_t before = 0, wall = 0;
#pragma unroll
  for (int k = 0; k < kWaves; ++k) {
    const uint64_t x = sh16[k];
    before += k < w ? x : 0ull;
    wall += x;
  }
#pragma unroll
  for (int r = 0; r < kOneR; ++r) {
    const uint32_t i = base + 64u * r;
    if ((uint32_t)r >= rounds || i >= n) continue;
    const uint64_t o = before + ex[r], end = o + ew[r];
    fe.dpos[i] = o;
    for (uint64_t bk = (o + kFirstsBlock - 1) / kFirstsBlock; bk * kFirstsBlock < end && bk < fe.nfirst; ++bk)
      fe.first[bk] = i;
  }
  if (t == 0) {
    fe.dpos[n] = wall;
    if (by_blocks) *fe.total = wall < (uint64_t)limit ? (uint32_t)wall : limit;
  }
}

// ---- binning: one thread per entry -------------------------------------------
// dpos[i] = first entry of the i-th visible Gaussian in depth order (exclusive scan of its
// bin count; dpos[V] = K).  Every visible Gaussian owns at least one entry, so a workgroup's
// ITEMS consecutive entries span at most ITEMS consecutive Gaussians: the offset scan's block
// firsts (or a wave-wide search) give the first, the workgroup stages their offsets in LDS,
// and each entry finds its Gaussian by binary search there.

// Last Gaussian (local index) of the staged offsets s_pos[0..span] whose first entry is <= e
// (span <= ITEMS, s_pos[0] <= e < s_pos[span]), in a fixed number of steps: no data-dependent
// loop, so the searches of a thread's several entries interleave.
template <int ITEMS>
__device__ __forceinline__ uint32_t local_gaussian_fixed(const uint64_t *s_pos, uint32_t span, uint64_t e) {
  uint32_t lo = 0;
#pragma unroll
  for (uint32_t step = ITEMS / 2; step > 0; step >>= 1) {
    const uint32_t c = lo + step;
    const bool take = c <= span && s_pos[c <= span ? c : span] <= e;
    lo = take ? c : lo;
  }
  return lo;
}

// The bin ranges start empty (the ranges kernel writes the non-empty ones after the sort):
// every workgroup of the binning grid clears its grid-stride share (and, for the two-level
// binning, of its sums).
__device__ __forceinline__ void clear_ranges(uint32_t *ranges, uint64_t nranges) {
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < nranges; i += (uint64_t)gridDim.x * kBlock)
    ranges[i] = 0u;
}

// Stages the first-entry offsets of the Gaussians that own entries [e0, e0 + ITEMS) into
// s_pos[0..span] (s_pos[l] = dpos[first + l]) and, with s_g, their indices s_g[l] = order[first + l].
template <int ITEMS>
__device__ __forceinline__ void stage_block_gaussians(const uint64_t *dpos, const uint32_t *block_first, uint32_t nvis,
                                                      uint64_t e0, uint64_t *s_pos, uint32_t *s_first,
                                                      uint32_t *first, uint32_t *span,
                                                      const uint32_t *order = nullptr, uint32_t *s_g = nullptr) {
  const int t = threadIdx.x, lane = t & 63;
  if (block_first) {
    // recorded by the offset scan (e0 is a multiple of its 1,024-entry blocks)
    if (t == 0) *s_first = block_first[e0 / kFirstsBlock];
  } else if (t < 64) {
    // 64-ary search for the last Gaussian i with dpos[i] <= e0, over [lo, hi)
    uint32_t lo = 0, hi = nvis;
    while (hi - lo > 1) {
      const uint32_t step = (hi - lo + 63) / 64;
      const uint32_t probe = lo + (uint32_t)lane * step;
      const bool le = probe < hi && dpos[probe] <= e0;
      const uint64_t m = __ballot(le);
      // dpos increases, so the lanes with le set are 0..j; lane j's probe is the new lower bound
      const int j = 63 - __clzll(m);
      const uint32_t nlo = lo + (uint32_t)j * step;
      hi = (nlo + step < hi) ? nlo + step : hi;
      lo = nlo;
    }
    if (lane == 0) *s_first = lo;
  }
  block_sync();
  *first = *s_first;
  *span = (nvis - *first) < (uint32_t)ITEMS ? (nvis - *first) : (uint32_t)ITEMS;
  for (uint32_t i = t; i <= *span; i += kBlock) {
    s_pos[i] = dpos[*first + i];
    if (s_g && i < *span) s_g[i] = order[*first + i];
  }
  block_sync();
}

// What the binning takes for block entries (two-level binning; all null otherwise): words to
// clear and, under opacity-aware culling, the Gaussians' records.  A Gaussian with fewer entries
// than its footprint has blocks takes the blocks the alpha-cut ellipse meets, any further entry
// an empty member rectangle.
struct BlockBinning {
  uint32_t *zero;
  uint64_t nzero;
  const double2 *xy;
  const float4 *conic;
};
constexpr uint32_t kEmptyDesc = 1u;   // x0 = 1, x1 = 1: no tile

// Entry j of such a Gaussian: its j-th block, or false.  A block row's blocks are those of a group row
// of 8x8 groups, so each row costs its 8 spans, however many blocks it holds (tested block by block, the
// long diagonal splats of a dense scene held their workgroups for longer than all others took).
__device__ __forceinline__ bool culled_block(const BlockBinning &bb, uint32_t g, ushort4 r, uint32_t j, int *gx,
                                             int *gy) {
  const double2 m = bb.xy[g];
  const float4 co = bb.conic[g];
  const TightEllipse el = tight_ellipse(m.x, m.y, co.x, co.y, co.z, co.w, r.x, r.z - 1, r.y);
  for (int by = r.y / kBlockTiles; by <= (r.w - 1) / kBlockTiles; ++by) {
    const TightGroupRow row = tight_group_row(el, kBlockTiles, by, r.w - 1);
    const uint32_t n = tight_group_count(row);
    if (j < n) {
      *gx = tight_group_nth(row, j);
      *gy = by;
      return true;
    }
    j -= n;
  }
  return false;
}

// The first radix pass's per-tile digit counts, taken where the keys are written (the binning
// workgroup covers exactly one sort tile, in the sort's XCD-aware tile order):
// counts[d * tiles + tile] for the digit bits [0, nbits0).
struct FirstCounts {
  uint32_t *counts;   // nullptr: no sort follows
  int nbits0;
  uint32_t tiles;
};

// One workgroup per sort tile of entries.  Each thread first finds the Gaussians of all its
// entries (LDS searches, interleaved), then gathers their rects (one round trip for all of
// them), then writes: the entry's Gaussian comes from the staged block, not from a gather per
// entry.
template <int ITEMS>
__global__ __launch_bounds__(kBlock) void k_binning(const uint32_t *order, const uint64_t *dpos,
                                                    const uint32_t *block_first, uint32_t nvis_host,
                                                    uint64_t K_host, const uint32_t *nvis_dev, const uint32_t *K_dev,
                                                    const ushort4 *rect, int G, int GX, int desc_shift,
                                                    uint32_t *bin_keys, uint32_t *vals, uint32_t *ranges,
                                                    uint64_t nranges, FirstCounts fc, BlockBinning bb) {
  constexpr int NI = ITEMS / kBlock;
  __shared__ uint64_t s_pos[ITEMS + 1];
  __shared__ uint32_t s_g[ITEMS];
  __shared__ uint32_t s_first;
  __shared__ uint32_t h[kWideDigits];
  const uint32_t nvis = (uint32_t)count_of(nvis_host, nvis_dev);
  const uint64_t K = count_of(K_host, K_dev);
  const uint32_t tile = xcd_sort_tile(blockIdx.x, (K + ITEMS - 1) / ITEMS);
  const uint64_t e0 = (uint64_t)tile * ITEMS;
  clear_ranges(ranges, nranges);
  clear_ranges(bb.zero, bb.nzero);
  if (tile == ~0u) return;
  for (int d = threadIdx.x; d < kWideDigits; d += kBlock) h[d] = 0;
  uint32_t first, span;
  stage_block_gaussians<ITEMS>(dpos, block_first, nvis, e0, s_pos, &s_first, &first, &span, order, s_g);
  const uint32_t dmask = (1u << fc.nbits0) - 1u;
  uint32_t l[NI];
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const uint64_t e = e0 + (uint64_t)it * kBlock + threadIdx.x;
    l[it] = e < K ? local_gaussian_fixed<ITEMS>(s_pos, span, e) : 0u;
  }
  ushort4 r[NI];
#pragma unroll
  for (int it = 0; it < NI; ++it) r[it] = rect[s_g[l[it]]];   // (l < span: a staged Gaussian)
#pragma unroll
  for (int it = 0; it < NI; ++it) {
    const uint64_t e = e0 + (uint64_t)it * kBlock + threadIdx.x;
    if (e < K) {
      const uint32_t j = (uint32_t)(e - s_pos[l[it]]);
      const int gx0 = r[it].x / G, gx1 = (r[it].z - 1) / G, gy0 = r[it].y / G;
      const int wdt = gx1 - gx0 + 1;
      int gy = gy0 + (int)(j / (uint32_t)wdt), gx = gx0 + (int)(j % (uint32_t)wdt);
      bool in = true;
      if (bb.xy && s_pos[l[it] + 1] - s_pos[l[it]] < rect_blocks(r[it])) {
        gx = gx0;
        gy = gy0;
        in = culled_block(bb, s_g[l[it]], r[it], j, &gx, &gy);
      }
      const uint32_t bin = (uint32_t)(gy * GX + gx);
      // (desc_shift > 0: group bins without culling, the member-tile rectangle above the bin bits)
      bin_keys[e] = desc_shift ? bin | (in ? rect_desc(r[it], G, gx, gy) : kEmptyDesc) << desc_shift : bin;
      vals[e] = first + l[it];   // the Gaussian's rank in depth order; the last sort pass turns it into its index
      if (fc.counts) atomicAdd(&h[bin & dmask], 1u);
    }
  }
  if (fc.counts) {
    block_sync();
    for (int d = threadIdx.x; d < (1 << fc.nbits0); d += kBlock) fc.counts[(uint64_t)d * fc.tiles + tile] = h[d];
  }
}

// Binning under opacity-aware culling: a Gaussian's entries follow its tile rows (group
// rows), each a span from tight_row_span (a union of group-column ranges); entry j walks the
// rows until its own.  (Measured on the 1M-Gaussian 1080p frame, this beat an LDS table of
// row spans built per workgroup: the span of a row is a few instructions, the table's
// dependent loads and prefix pass are not.)
template <int ITEMS>
__global__ __launch_bounds__(kBlock) void k_binning_tight(const uint32_t *order, const uint64_t *dpos,
                                                          const uint32_t *block_first, uint32_t nvis_host,
                                                          uint64_t K_host, const uint32_t *nvis_dev,
                                                          const uint32_t *K_dev, const ushort4 *rect,
                                                          const double2 *xy, const float4 *conic, int TX, int G,
                                                          int GX, uint32_t *bin_keys, uint32_t *vals,
                                                          uint32_t *ranges, uint64_t nranges, FirstCounts fc) {
  __shared__ uint64_t s_pos[ITEMS + 1];
  __shared__ uint32_t s_g[ITEMS];
  __shared__ uint32_t s_first;
  __shared__ uint32_t h[kWideDigits];
  const uint32_t nvis = (uint32_t)count_of(nvis_host, nvis_dev);
  const uint64_t K = count_of(K_host, K_dev);
  const uint32_t tile = xcd_sort_tile(blockIdx.x, (K + ITEMS - 1) / ITEMS);
  const uint64_t e0 = (uint64_t)tile * ITEMS;
  const int lane = threadIdx.x & 63;
  clear_ranges(ranges, nranges);
  if (tile == ~0u) return;
  for (int d = threadIdx.x; d < kWideDigits; d += kBlock) h[d] = 0;
  uint32_t first, span;
  stage_block_gaussians<ITEMS>(dpos, block_first, nvis, e0, s_pos, &s_first, &first, &span, order, s_g);
  const uint32_t dmask = (1u << fc.nbits0) - 1u;
#pragma unroll
  for (int it = 0; it < ITEMS / kBlock; ++it) {
    const uint64_t e = e0 + (uint64_t)it * kBlock + threadIdx.x;
    const bool valid = e < K;
    if (__ballot(valid) == 0) continue;
    uint32_t rank = 0, g = 0, left = 0;
    if (valid) {
      const uint32_t l = local_gaussian_fixed<ITEMS>(s_pos, span, e);
      rank = first + l;
      g = s_g[l];
      left = (uint32_t)(e - s_pos[l]);
    }
    uint32_t bin = 0;   // (the walks always end early for counts from the preprocess)
    bool placed = false;
    // A wave whose entries all belong to one Gaussian (the large ones, where walking the rows
    // per entry costs most) shares the walk: lane k takes tile (group) row k, a wave prefix
    // sum of the row counts gives each row's first entry, and each lane finds its row by
    // bisection over those sums.  Same spans as the preprocess counted.
    const uint32_t g0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)g);
    if (__ballot(valid && g != g0) == 0) {
      const ushort4 r = rect[g0];
      const int row0 = r.y / G;
      const int R = (r.w - 1) / G - row0 + 1;   // tile rows (G = 1) or group rows
      if (R <= 64) {
        const double2 m = xy[g0];
        const float4 co = conic[g0];
        const TightEllipse el = tight_ellipse(m.x, m.y, co.x, co.y, co.z, co.w, r.x, r.z - 1, r.y);
        int lo = 0, hi = -1;
        uint32_t cnt = 0;
        if (lane < R) {
          if (G == 1) {
            tight_row_span(el, r.y + lane, &lo, &hi);
            cnt = (uint32_t)(hi - lo + 1);
          } else {
            cnt = tight_group_count(tight_group_row(el, G, row0 + lane, r.w - 1));
          }
        }
        uint32_t incl = cnt;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const uint32_t u = __shfl_up(incl, off, 64);
          if (lane >= off) incl += u;
        }
        int pos = 0;   // rows whose entries all precede this lane's entry
#pragma unroll
        for (int step = 32; step > 0; step >>= 1) {
          const uint32_t v = __shfl(incl, pos + step - 1, 64);
          if (v <= left) pos += step;
        }
        const uint32_t ip = __shfl(incl, pos, 64), cp = __shfl(cnt, pos, 64);
        const uint32_t within = left - (ip - cp);
        if (G == 1) {
          const int lop = __shfl(lo, pos, 64);
          bin = (uint32_t)((r.y + pos) * TX + lop) + within;
        } else if (valid) {
          const TightGroupRow row = tight_group_row(el, G, row0 + pos, r.w - 1);
          bin = (uint32_t)((row0 + pos) * GX + tight_group_nth(row, within));
        }
        placed = true;
      }
    }
    if (valid && !placed) {
      const ushort4 r = rect[g];
      const double2 m = xy[g];
      const float4 co = conic[g];
      const TightEllipse el = tight_ellipse(m.x, m.y, co.x, co.y, co.z, co.w, r.x, r.z - 1, r.y);
      if (G == 1) {
        for (int ty = r.y; ty < r.w; ++ty) {
          int lo, hi;
          tight_row_span(el, ty, &lo, &hi);
          const uint32_t cnt = (uint32_t)(hi - lo + 1);
          if (left < cnt) {
            bin = (uint32_t)(ty * TX + lo) + left;
            break;
          }
          left -= cnt;
        }
      } else {
        for (int gy = r.y / G; gy <= (r.w - 1) / G; ++gy) {
          const TightGroupRow row = tight_group_row(el, G, gy, r.w - 1);
          const uint32_t cnt = tight_group_count(row);
          if (left < cnt) {
            bin = (uint32_t)(gy * GX + tight_group_nth(row, left));
            break;
          }
          left -= cnt;
        }
      }
    }
    if (valid) {
      bin_keys[e] = bin;
      vals[e] = rank;   // the Gaussian's rank in depth order; the last sort pass turns it into its index
      if (fc.counts) atomicAdd(&h[bin & dmask], 1u);
    }
  }
  if (fc.counts) {
    block_sync();
    for (int d = threadIdx.x; d < (1 << fc.nbits0); d += kBlock) fc.counts[(uint64_t)d * fc.tiles + tile] = h[d];
  }
}

// Bin ranges (cleared beforehand), tile-membership masks and the 64-bit keys.  Entry i holds
// its Gaussian's rank r in the depth-sorted visible list; the Gaussian index order[r] and the
// depth bits dkeys[r] come from those two V-sized arrays (cache-resident), not from the
// per-Gaussian records.  A workgroup takes kRangeItems x 256 consecutive entries, thread t
// the entries t, t + 256, ... (coalesced), and issues all their loads before the dependent
// gathers, so several round trips are in flight at once.
constexpr int kRangeItems = 4;

__global__ __launch_bounds__(kBlock) void k_ranges(const uint32_t *bin_keys, const uint32_t *ranks, uint64_t n_host,
                                                   const uint32_t *n_dev, const uint32_t *order, const uint32_t *dkeys,
                                                   const ushort4 *rect, const double2 *xy, const float4 *conic,
                                                   int tight, int G, int GX, int desc_shift, uint32_t *vals,
                                                   uint32_t *ranges, void *masks, uint64_t *keys) {
  const uint64_t n = count_of(n_host, n_dev);
  const uint32_t bmask = desc_shift ? (1u << desc_shift) - 1u : ~0u;
  const uint64_t base = (uint64_t)blockIdx.x * kBlock * kRangeItems + threadIdx.x;
  uint32_t bin[kRangeItems], prev[kRangeItems], next[kRangeItems], r[kRangeItems];
#pragma unroll
  for (int j = 0; j < kRangeItems; ++j) {
    const uint64_t i = base + (uint64_t)j * kBlock;
    const bool in = i < n;
    bin[j] = in ? bin_keys[i] : 0u;
    prev[j] = (in && i > 0) ? bin_keys[i - 1] & bmask : 0xFFFFFFFFu;
    next[j] = (in && i + 1 < n) ? bin_keys[i + 1] & bmask : 0xFFFFFFFFu;
    r[j] = in ? ranks[i] : 0u;
  }
  uint32_t g[kRangeItems], d[kRangeItems];
#pragma unroll
  for (int j = 0; j < kRangeItems; ++j) {
    const bool in = base + (uint64_t)j * kBlock < n;
    g[j] = in ? order[r[j]] : 0u;
    d[j] = in ? dkeys[r[j]] : 0u;
  }
#pragma unroll
  for (int j = 0; j < kRangeItems; ++j) {
    const uint64_t i = base + (uint64_t)j * kBlock;
    if (i >= n) break;
    const uint32_t b = bin[j] & bmask;
    if (prev[j] != b) ranges[2 * (uint64_t)b] = (uint32_t)i;
    if (next[j] != b) ranges[2 * (uint64_t)b + 1] = (uint32_t)(i + 1);
    keys[i] = ((uint64_t)b << 32) | d[j];
    vals[i] = g[j];
    if (G > 1 && masks) {
      const ushort4 rc = rect[g[j]];
      const int gx = (int)(b % (uint32_t)GX), gy = (int)(b / (uint32_t)GX);
      uint64_t m = 0;
      if (desc_shift) {
        m = rect_desc_mask(bin[j] >> desc_shift, G);
      } else if (tight) {
        // member tiles the alpha-cut ellipse meets
        const double2 mu = xy[g[j]];
        const float4 co = conic[g[j]];
        const TightEllipse el = tight_ellipse(mu.x, mu.y, co.x, co.y, co.z, co.w, rc.x, rc.z - 1, rc.y);
        m = tight_group_mask(el, G, gx, gy, rc.w - 1);
      } else {
        // member tiles inside the footprint: a rectangle of rows [y0, y1) and columns [x0, x1)
        const int x0 = max((int)rc.x - gx * G, 0), x1 = min((int)rc.z - gx * G, G);
        const int y0 = max((int)rc.y - gy * G, 0), y1 = min((int)rc.w - gy * G, G);
        const uint64_t row = ((1ull << (x1 - x0)) - 1ull) << x0;   // x1 - x0 <= G <= 8
        for (int ly = y0; ly < y1; ++ly) m |= row << (ly * G);
      }
      if (G == 8) static_cast<uint64_t *>(masks)[i] = m;
      else static_cast<uint16_t *>(masks)[i] = (uint16_t)m;
    }
  }
}

// Bin ranges and (MASKS: group > 1) membership masks once the last bin pass has placed the
// final Gaussian indices and 64-bit keys: only the sorted bin keys are read for the ranges.
template <bool MASKS>
__global__ __launch_bounds__(kBlock) void k_ranges_final(const uint32_t *bin_keys, uint64_t n_host,
                                                         const uint32_t *n_dev, const uint32_t *vals,
                                                         const ushort4 *rect, const double2 *xy, const float4 *conic,
                                                         int tight, int G, int GX, int desc_shift, uint32_t *ranges,
                                                         void *masks) {
  const uint64_t n = count_of(n_host, n_dev);
  const uint32_t bmask = desc_shift ? (1u << desc_shift) - 1u : ~0u;
  const uint64_t base = (uint64_t)blockIdx.x * kBlock * kRangeItems + threadIdx.x;
  uint32_t bin[kRangeItems], prev[kRangeItems], next[kRangeItems];
#pragma unroll
  for (int j = 0; j < kRangeItems; ++j) {
    const uint64_t i = base + (uint64_t)j * kBlock;
    const bool in = i < n;
    bin[j] = in ? bin_keys[i] : 0u;
    prev[j] = (in && i > 0) ? bin_keys[i - 1] & bmask : 0xFFFFFFFFu;
    next[j] = (in && i + 1 < n) ? bin_keys[i + 1] & bmask : 0xFFFFFFFFu;
  }
#pragma unroll
  for (int j = 0; j < kRangeItems; ++j) {
    const uint64_t i = base + (uint64_t)j * kBlock;
    if (i >= n) break;
    const uint32_t b = bin[j] & bmask;
    if (prev[j] != b) ranges[2 * (uint64_t)b] = (uint32_t)i;
    if (next[j] != b) ranges[2 * (uint64_t)b + 1] = (uint32_t)(i + 1);
    if (MASKS && desc_shift) {
      const uint64_t m = rect_desc_mask(bin[j] >> desc_shift, G);
      if (G == 8) static_cast<uint64_t *>(masks)[i] = m;
      else static_cast<uint16_t *>(masks)[i] = (uint16_t)m;
    } else if (MASKS) {
      const uint32_t g = vals[i];
      const ushort4 rc = rect[g];
      const int gx = (int)(b % (uint32_t)GX), gy = (int)(b / (uint32_t)GX);
      uint64_t m = 0;
      if (tight) {
        const double2 mu = xy[g];
        const float4 co = conic[g];
        const TightEllipse el = tight_ellipse(mu.x, mu.y, co.x, co.y, co.z, co.w, rc.x, rc.z - 1, rc.y);
        m = tight_group_mask(el, G, gx, gy, rc.w - 1);
      } else {
        const int x0 = max((int)rc.x - gx * G, 0), x1 = min((int)rc.z - gx * G, G);
        const int y0 = max((int)rc.y - gy * G, 0), y1 = min((int)rc.w - gy * G, G);
        const uint64_t row = ((1ull << (x1 - x0)) - 1ull) << x0;
        for (int ly = y0; ly < y1; ++ly) m |= row << (ly * G);
      }
      if (G == 8) static_cast<uint64_t *>(masks)[i] = m;
      else static_cast<uint16_t *>(masks)[i] = (uint16_t)m;
    }
  }
}

inline unsigned grid_for(uint64_t n, uint64_t per = kBlock) {
  const uint64_t b = (n + per - 1) / per;
  return (unsigned)(b ? b : 1);
}

}  // namespace

hipError_t launch_fill_u32(uint32_t *p, uint64_t n, uint32_t v, hipStream_t st) {
  if (n == 0) return hipSuccess;
  uint64_t b = (n + kBlock - 1) / kBlock;
  if (b > 8192) b = 8192;
  hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)b), dim3(kBlock), 0, st, p, n, v);
  return hipGetLastError();
}

// tiles of a sort of n keys, and the most tiles of any sort of at most n keys
inline uint64_t sort_tiles(uint64_t n) {
  return n <= kSmallSort ? (n + SortTile<kSmallR>::kTile - 1) / SortTile<kSmallR>::kTile
                         : (n + SortTile<kLargeR>::kTile - 1) / SortTile<kLargeR>::kTile;
}

// Digit width of the passes over key bits [lo, hi): passes of (nearly) equal width, at most
// maxw bits each (13 bits -> 7 + 6 and 32 -> 4 x 8 with 8; 31 -> 11 + 11 + 9 with 11).
constexpr int pass_width(int lo, int hi, int maxw = 8) {
  return (hi - lo + (hi - lo + maxw - 1) / maxw - 1) / ((hi - lo + maxw - 1) / maxw);
}

// first_counted: the per-tile digit counts of the first pass are already in tmp (written where
// the keys were produced).  fin: the last pass places final Gaussian indices and 64-bit keys.
template <typename KT, int R, int DIG>
hipError_t radix_passes_r(KT *keys, uint32_t *vals, KT *keys_alt, uint32_t *vals_alt, uint64_t n,
                          const uint32_t *n_dev, int lo, int hi, void *tmp, hipStream_t st, bool *in_alt,
                          const FinalOut *fin, bool first_counted) {
  const uint32_t tiles = (uint32_t)((n + SortTile<R>::kTile - 1) / SortTile<R>::kTile);
  uint32_t *counts = static_cast<uint32_t *>(tmp);
  uint32_t *totals = counts + (uint64_t)DIG * tiles;
  KT *kin = keys, *kout = keys_alt;
  uint32_t *vin = vals, *vout = vals_alt;
  const int width = DIG == kWideDigits ? kWideBits : pass_width(lo, hi);
  const FinalOut none{nullptr, nullptr, nullptr, nullptr};
  const DigitWeights now{};
  const FirstEntries nofe{nullptr, nullptr, 0, nullptr, nullptr};
  for (int shift = lo; shift < hi; shift += width) {
    const int bits = (hi - shift) < width ? (hi - shift) : width;
    const bool last = shift + width >= hi;
    if (!(first_counted && shift == lo))
      hipLaunchKernelGGL((k_radix_count<KT, R, DIG, false>), dim3(xcd_sort_grid(tiles)), dim3(kBlock), 0, st, kin,
                         n, n_dev, shift, bits, tiles, counts, now);
    hipLaunchKernelGGL(k_radix_digit_scan, dim3(1u << bits), dim3(kBlock), 0, st, counts, tiles, totals, n, n_dev,
                       (uint32_t)SortTile<R>::kTile, now);
    hipLaunchKernelGGL((k_radix_scatter<KT, R, DIG, false, false>), dim3(xcd_sort_grid(tiles)), dim3(kBlock), 0, st, kin,
                       vin, kout, vout, n, n_dev, shift, bits, tiles, counts, totals, (last && fin) ? *fin : none,
                       now, nofe, ChunkTable{nullptr, 0}, DigitRows{});
    std::swap(kin, kout);
    std::swap(vin, vout);
    *in_alt = !*in_alt;
  }
  return hipGetLastError();
}

// n: the number of keys, or (with n_dev) an upper bound of *n_dev.
template <typename KT>
hipError_t radix_passes_t(KT *keys, uint32_t *vals, KT *keys_alt, uint32_t *vals_alt, uint64_t n,
                          const uint32_t *n_dev, int lo, int hi, void *tmp, hipStream_t st, bool *in_alt,
                          const FinalOut *fin = nullptr, bool first_counted = false) {
  *in_alt = false;
  if (hi <= lo || n <= 1) return hipSuccess;
  if (n <= kSmallSort)
    return radix_passes_r<KT, kSmallR, kDigits>(keys, vals, keys_alt, vals_alt, n, n_dev, lo, hi, tmp, st, in_alt,
                                                fin, first_counted);
  if (hi - lo == kWideBits)
    return radix_passes_r<KT, kLargeR, kWideDigits>(keys, vals, keys_alt, vals_alt, n, n_dev, lo, hi, tmp, st,
                                                    in_alt, fin, first_counted);
  return radix_passes_r<KT, kLargeR, kDigits>(keys, vals, keys_alt, vals_alt, n, n_dev, lo, hi, tmp, st, in_alt,
                                              fin, first_counted);
}

hipError_t radix_sort(uint64_t *keys, uint32_t *vals, uint64_t *keys_alt, uint32_t *vals_alt, uint64_t n, int lo,
                      int hi, void *tmp, hipStream_t st, bool *in_alt) {
  return radix_passes_t<uint64_t>(keys, vals, keys_alt, vals_alt, n, nullptr, lo, hi, tmp, st, in_alt);
}

// ---- depth sort -----------------------------------------------------------------------
// Four passes over the 31 bits of a positive depth (8, 8, 8 and 7 bits), the last one weighted.
constexpr int kDepthWidth = pass_width(0, kDepthBits);
constexpr int kDepthPasses = (kDepthBits + kDepthWidth - 1) / kDepthWidth;
constexpr int kDepthLastBits = kDepthBits - (kDepthPasses - 1) * kDepthWidth;
constexpr int kDepthLastDigits = 1 << kDepthLastBits;
static_assert(kDepthWidth == 8 && kDepthPasses == 4 && kDepthLastBits == 7, "depth passes of 8, 8, 8 and 7 bits");
// Sorts of up to this many tiles count in rows (DigitRows).  All of them visible, the first pass's
// rows (one per tile) take 13 us to add up and a scan 5, and the later ones' (one per 4) 4; at a fifth, 1 us.
constexpr uint64_t kRowTiles = 1024;

// Scratch of the depth sort over tiles sort tiles (the same for every pass): per-tile digit
// counts and digit totals, and the last pass's weights per tile and digit with their 64-bit
// scans and totals.
struct DepthTmp {
  uint64_t *wprefix;
  uint64_t *wtotals;
  uint32_t *counts;
  uint32_t *totals;
  uint32_t *wcounts;
  size_t bytes;
};
inline DepthTmp depth_tmp(void *tmp, uint64_t tiles) {
  DepthTmp d;
  char *p = static_cast<char *>(tmp);
  size_t off = 0;
  auto take = [&](size_t bytes) -> char * {
    char *q = p ? p + off : nullptr;
    off += (bytes + 255) & ~(size_t)255;
    return q;
  };
  const uint64_t t = tiles ? tiles : 1;
  d.wprefix = reinterpret_cast<uint64_t *>(take(kDepthLastDigits * t * 8));
  d.wtotals = reinterpret_cast<uint64_t *>(take(kDepthLastDigits * 8));
  d.counts = reinterpret_cast<uint32_t *>(take(kDigits * t * 4));
  d.totals = reinterpret_cast<uint32_t *>(take(kDigits * 4));
  d.wcounts = reinterpret_cast<uint32_t *>(take(kDepthLastDigits * t * 4));
  d.bytes = off;
  return d;
}

// Keys ping-pong between keys and keys_alt; values run order -> vals_alt -> vals_b ->
// vals_alt -> order, so that the sorted list ends where it started.
// Passes [p0, p1).
template <int R>
hipError_t depth_passes(int p0, int p1, uint32_t *order, const uint32_t *nvis, uint64_t n_max, uint32_t *keys, uint32_t *keys_alt,
                        uint32_t *vals_alt, uint32_t *vals_b, void *tmp, hipStream_t st, const EntryCounts &count,
                        uint64_t *dpos, uint32_t *first, uint64_t nfirst, uint32_t *total, const uint32_t *limit) {
  const uint32_t tiles = (uint32_t)sort_tiles(n_max);
  const DepthTmp d = depth_tmp(tmp, tiles);
  const unsigned grid = xcd_sort_grid(tiles);
  const uint32_t tile_keys = (uint32_t)SortTile<R>::kTile;
  const FinalOut none{nullptr, nullptr, nullptr, nullptr};
  const DigitWeights now{};
  const FirstEntries nofe{nullptr, nullptr, 0, nullptr, nullptr};
  uint32_t *kbuf[2] = {keys, keys_alt};
  uint32_t *vbuf[kDepthPasses + 1];
  vbuf[0] = vbuf[kDepthPasses] = order;
  for (int p = 1; p < kDepthPasses; ++p) vbuf[p] = (p & 1) ? vals_alt : vals_b;
  const bool in_rows = R == kSmallR || tiles <= kRowTiles;
  static_assert(kSmallSort <= kRowTiles * SortTile<kSmallR>::kTile, "small sorts count in rows");
  // (16-bit rows and their prefixes side by side in the room of the 32-bit counts)
  uint16_t *r16 = reinterpret_cast<uint16_t *>(d.counts);
  const dim3 groups((tiles + (1u << kRowShift) - 1u) >> kRowShift);
  for (int p = p0; p < p1; ++p) {
    const int shift = p * kDepthWidth;
    uint32_t *kin = kbuf[p & 1], *kout = kbuf[(p + 1) & 1];
    if (p + 1 < kDepthPasses && in_rows) {
      // the first pass was counted by k_depth_keys, in rows of single tiles
      const DigitRows rows{r16, r16 + (uint64_t)kDigits * tiles, p > 0 ? kRowShift : 0};
      if (p > 0)
        hipLaunchKernelGGL(k_count_rows<R>, groups, dim3(kBlock << kRowShift), 0, st, kin, nvis, shift, kDepthWidth,
                           rows);
      hipLaunchKernelGGL((k_radix_scatter<uint32_t, R, kDigits, false, true>), dim3(grid), dim3(kBlock), 0, st, kin,
                         vbuf[p], kout, vbuf[p + 1], n_max, nvis, shift, kDepthWidth, tiles, d.counts, d.totals, none,
                         now, nofe, ChunkTable{nullptr, 0}, rows);
    } else if (p + 1 < kDepthPasses) {
      if constexpr (R != kSmallR) {
        if (p > 0)
          hipLaunchKernelGGL((k_radix_count<uint32_t, R, kDigits, false>), dim3(grid), dim3(kBlock), 0, st, kin, n_max,
                             nvis, shift, kDepthWidth, tiles, d.counts, now);
        hipLaunchKernelGGL(k_radix_digit_scan, dim3(1u << kDepthWidth), dim3(kBlock), 0, st, d.counts, tiles, d.totals,
                           n_max, nvis, tile_keys, now);
        hipLaunchKernelGGL((k_radix_scatter<uint32_t, R, kDigits, false, false>), dim3(grid), dim3(kBlock), 0, st, kin,
                           vbuf[p], kout, vbuf[p + 1], n_max, nvis, shift, kDepthWidth, tiles, d.counts, d.totals,
                           none, now, nofe, ChunkTable{nullptr, 0}, DigitRows{});
      }
    } else {
      // weighted by the Gaussians' entry counts, with the first entries and block firsts
      const DigitWeights wt{vbuf[p], count, vals_b, d.wcounts, d.wprefix, d.wtotals};   // (vals_b is free again)
      hipLaunchKernelGGL((k_radix_count<uint32_t, R, kDigits, true>), dim3(grid), dim3(kBlock), 0, st, kin, n_max,
                         nvis, shift, kDepthLastBits, tiles, d.counts, wt);
      hipLaunchKernelGGL(k_radix_digit_scan, dim3(1u << kDepthLastBits), dim3(kBlock), 0, st, d.counts, tiles,
                         d.totals, n_max, nvis, tile_keys, wt);
      hipLaunchKernelGGL((k_radix_scatter<uint32_t, R, kDigits, true, false>), dim3(grid), dim3(kBlock), 0, st, kin,
                         vbuf[p], kout, vbuf[p + 1], n_max, nvis, shift, kDepthLastBits, tiles, d.counts, d.totals,
                         none, wt, FirstEntries{dpos, first, nfirst, total, limit}, ChunkTable{nullptr, 0},
                         DigitRows{});
    }
  }
  return hipGetLastError();
}

size_t radix_tmp_bytes(uint64_t n) {
  // the most digit counts of any sort of at most n keys: 256 per 1,024-key tile up to
  // kSmallSort keys, 512 per 2,048-key tile above (the same 1 count per 4 keys), and the totals
  uint64_t counts = (uint64_t)kDigits * sort_tiles(n < kSmallSort ? n : kSmallSort);
  if (n > kSmallSort && (uint64_t)kWideDigits * sort_tiles(n) > counts) counts = (uint64_t)kWideDigits * sort_tiles(n);
  // (the two-level binning takes 512 digits per 2,048-key tile at any length: at most one 1,024-key
  // tile's counts more)
  return ((size_t)(counts ? counts : kDigits) + 2 * kWideDigits) * sizeof(uint32_t);
}

size_t depth_sort_tmp_bytes(uint64_t n) { return depth_tmp(nullptr, sort_tiles(n ? n : 1)).bytes; }

hipError_t launch_depth_keys(const uint32_t *order, const float4 *rgb, const uint32_t *nvis, uint64_t n_max,
                             uint32_t *keys, const uint64_t *K, uint64_t *counts, uint64_t *host_counts,
                             uint64_t capacity, void *tmp, hipStream_t st) {
  // one workgroup per tile of the depth sort that follows (sort_depth_begin, same n_max): its first
  // pass's digit counts are taken here
  const uint32_t tiles = (uint32_t)sort_tiles(n_max ? n_max : 1);
  uint32_t *dcounts = depth_tmp(tmp, tiles).counts;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(xcd_sort_grid(tiles)), dim3(kBlock), 0, st, order, rgb, nvis, keys, K, counts,
                       host_counts, capacity, kDepthWidth, dcounts, tiles);
  };
  if (n_max <= kSmallSort) launch(k_depth_keys<kSmallR, true>);
  else if (tiles <= kRowTiles) launch(k_depth_keys<kLargeR, true>);
  else launch(k_depth_keys<kLargeR, false>);
  return hipGetLastError();
}

bool depth_sort_one(uint64_t n_max) { return n_max <= kOneKeys; }

hipError_t launch_depth_sort_one(uint32_t *order, const float4 *rgb, const uint32_t *nvis, uint32_t *keys,
                                 const uint64_t *K, uint64_t *counts, uint64_t *host_counts, uint64_t capacity,
                                 const EntryCounts &bins, const EntryCounts &blocks, const BlockRule &rule,
                                 uint64_t *dpos, uint32_t *first, uint64_t nfirst, uint32_t *total, hipStream_t st) {
  hipLaunchKernelGGL(k_depth_sort_one, dim3(1), dim3(kOneThreads), 0, st, order, rgb, nvis, keys, K, counts,
                     host_counts, capacity, bins, blocks, rule, FirstEntries{dpos, first, nfirst, total, nullptr});
  return hipGetLastError();
}

hipError_t sort_depth_begin(uint32_t *order, const uint32_t *nvis, uint64_t n_max, uint32_t *keys, uint32_t *keys_alt,
                            uint32_t *vals_alt, uint32_t *vals_b, void *tmp, hipStream_t st) {
  if (n_max <= 1) return hipSuccess;
  auto passes = n_max <= kSmallSort ? depth_passes<kSmallR> : depth_passes<kLargeR>;
  return passes(0, kDepthPasses - 1, order, nvis, n_max, keys, keys_alt, vals_alt, vals_b, tmp, st, EntryCounts{},
                nullptr, nullptr, 0, nullptr, nullptr);
}

hipError_t sort_depth_end(uint32_t *order, const uint32_t *nvis, uint64_t n_max, uint32_t *keys, uint32_t *keys_alt,
                          uint32_t *vals_alt, uint32_t *vals_b, void *tmp, hipStream_t st, const EntryCounts &count,
                          uint64_t *dpos, uint32_t *first, uint64_t nfirst, uint32_t *total, const uint32_t *limit) {
  if (n_max <= 1) return hipSuccess;
  auto passes = n_max <= kSmallSort ? depth_passes<kSmallR> : depth_passes<kLargeR>;
  return passes(kDepthPasses - 1, kDepthPasses, order, nvis, n_max, keys, keys_alt, vals_alt, vals_b, tmp, st, count,
                dpos, first, nfirst, total, limit);
}

hipError_t bin_and_sort(const uint32_t *order, const uint32_t *dkeys, const uint64_t *dpos, const uint32_t *block_first,
                        uint32_t V, uint64_t K, const uint32_t *V_dev, const uint32_t *K_dev,
                        const uint16_t *rect, const double *xy, const float *conic, bool tight, const Grid &g,
                        uint32_t *bkey, uint32_t *bval, uint32_t *bkey_alt, uint32_t *bval_alt, uint32_t *ranges,
                        void *masks, uint32_t *vals, uint64_t *keys, void *tmp, hipStream_t st) {
  const uint64_t nranges = 2 * (uint64_t)g.nbins;
  if (K == 0) return launch_fill_u32(ranges, nranges, 0u, st);
  const ushort4 *r4 = reinterpret_cast<const ushort4 *>(rect);
  const double2 *m2 = reinterpret_cast<const double2 *>(xy);
  const float4 *c4 = reinterpret_cast<const float4 *>(conic);
  const int hi = bits_for((uint64_t)g.nbins);
  // group bins without culling carry their member-tile rectangle above the bin bits (they fit:
  // at most 2^18 groups); culled groups' masks are computed from the Gaussians' records again
  const int desc_shift = (g.G > 1 && !tight && masks && hi + kRectDescBits <= 32) ? hi : 0;
  // with a sort to follow (K > 1), the binning takes its first pass's digit counts; with the
  // counts on the device, K is the bound that sizes the grids and picks the tile size, as the
  // sort's own passes do
  const bool large = K > kSmallSort;
  const unsigned tiles = grid_for(K, large ? SortTile<kLargeR>::kTile : SortTile<kSmallR>::kTile);
  const int nbits0 = (large && hi == kWideBits) ? kWideBits : pass_width(0, hi);   // as radix_passes_t splits [0, hi)
  const FirstCounts fc{K > 1 ? static_cast<uint32_t *>(tmp) : nullptr, nbits0, tiles};
  const unsigned grid = xcd_sort_grid(tiles);   // the sort's tile order (k_radix_scatter)
  if (tight) {
    if (large)
      hipLaunchKernelGGL((k_binning_tight<SortTile<kLargeR>::kTile>), dim3(grid), dim3(kBlock), 0, st, order, dpos,
                         block_first, V, K, V_dev, K_dev, r4, m2, c4, g.TX, g.G, g.GX, bkey, bval, ranges, nranges, fc);
    else
      hipLaunchKernelGGL((k_binning_tight<SortTile<kSmallR>::kTile>), dim3(grid), dim3(kBlock), 0, st, order, dpos,
                         block_first, V, K, V_dev, K_dev, r4, m2, c4, g.TX, g.G, g.GX, bkey, bval, ranges, nranges, fc);
  } else {
    if (large)
      hipLaunchKernelGGL((k_binning<SortTile<kLargeR>::kTile>), dim3(grid), dim3(kBlock), 0, st, order, dpos,
                         block_first, V, K, V_dev, K_dev, r4, g.G, g.GX, desc_shift, bkey, bval, ranges, nranges,
                         fc, BlockBinning{nullptr, 0, nullptr, nullptr});
    else
      hipLaunchKernelGGL((k_binning<SortTile<kSmallR>::kTile>), dim3(grid), dim3(kBlock), 0, st, order, dpos,
                         block_first, V, K, V_dev, K_dev, r4, g.G, g.GX, desc_shift, bkey, bval, ranges, nranges,
                         fc, BlockBinning{nullptr, 0, nullptr, nullptr});
  }
  if (K <= 1) {
    // nothing to sort: the single entry's index, key and range directly
    hipLaunchKernelGGL(k_ranges, dim3(1), dim3(kBlock), 0, st, bkey, bval, K, K_dev, order, dkeys, r4, m2, c4,
                       tight ? 1 : 0, g.G, g.GX, desc_shift, vals, ranges, masks, keys);
    return hipGetLastError();
  }
  bool in_alt = false;
  const FinalOut fin{order, dkeys, vals, keys, desc_shift ? (1u << desc_shift) - 1u : ~0u};
  // the bin passes ping-pong between (bkey, bval) and (bkey_alt, bval_alt); the last one writes
  // the final indices and 64-bit keys, and its sorted bin keys land in kf
  hipError_t e = radix_passes_t<uint32_t>(bkey, bval, bkey_alt, bval_alt, K, K_dev, 0, hi, tmp, st, &in_alt, &fin,
                                          true);
  if (e != hipSuccess) return e;
  const uint32_t *kf = in_alt ? bkey_alt : bkey;
  const dim3 rgrid(grid_for(K, (uint64_t)kBlock * kRangeItems));
  if (g.G > 1 && masks)
    hipLaunchKernelGGL(k_ranges_final<true>, rgrid, dim3(kBlock), 0, st, kf, K, K_dev, vals, r4, m2, c4, tight ? 1 : 0,
                       g.G, g.GX, desc_shift, ranges, masks);
  else
    hipLaunchKernelGGL(k_ranges_final<false>, rgrid, dim3(kBlock), 0, st, kf, K, K_dev, vals, r4, m2, c4,
                       tight ? 1 : 0, g.G, g.GX, desc_shift, ranges, masks);
  return hipGetLastError();
}

hipError_t bin_and_sort_blocks(const uint32_t *order, const uint32_t *dkeys, const uint64_t *dpos,
                               const uint32_t *block_first, uint32_t V, uint64_t K, const uint32_t *V_dev,
                               const uint32_t *K_dev, const uint32_t *entries_dev, const uint16_t *rect,
                               const double *xy, const float *conic, bool tight, const Grid &g, uint32_t *bkey,
                               uint32_t *bval, uint32_t *bkey_alt, uint32_t *bval_alt, uint32_t *ranges, void *masks,
                               uint32_t *vals, uint64_t *keys, void *tmp, void *block_tmp, hipStream_t st) {
  const uint64_t nranges = 2 * (uint64_t)g.nbins;
  if (K == 0) return launch_fill_u32(ranges, nranges, 0u, st);
  const Grid b = make_grid(g.W, g.H, kBlockTiles);
  const ushort4 *r4 = reinterpret_cast<const ushort4 *>(rect);
  const double2 *m2 = reinterpret_cast<const double2 *>(xy);
  const float4 *c4 = reinterpret_cast<const float4 *>(conic);
  // one pass over the block bits.  9 bits take the 512-digit pass
  // (2,048-key tiles) at any length, so that its counts stay one per four keys.
  const int hi = bits_for((uint64_t)b.nbins);
  // (the block entries are a fifth to a tenth of the bin entries, so the larger sort tiles pay
  // from four times as many of those; where K is only a bound of them, from sixteen times: with a bound of
  // 12M entries 88 us with larger tiles and 80 with smaller ones at 100K entries, 119 and 113 at 3M)
  const bool wide = hi > 8, large = wide || K > (K_dev ? 16 : 4) * kSmallSort;
  const unsigned tiles = grid_for(K, large ? SortTile<kLargeR>::kTile : SortTile<kSmallR>::kTile);
  const unsigned grid = xcd_sort_grid(tiles);
  uint32_t *counts = static_cast<uint32_t *>(tmp);
  uint32_t *totals = counts + (uint64_t)(wide ? kWideDigits : kDigits) * tiles;
  const FirstCounts fc{counts, hi, tiles};
  const BlockTmp bt = block_tmp_layout(tmp, block_tmp, K);
  const BlockBinning bb{bt.sums, BlockTmp::nsums(g, b), tight ? m2 : nullptr, c4};
  const ChunkTable ct{bt.start, (uint32_t)kChunk};
  const dim3 dg(grid), db(kBlock);
  // V and K are upper bounds of the visible Gaussians and of the block entries *entries_dev
  if (large)
    hipLaunchKernelGGL((k_binning<SortTile<kLargeR>::kTile>), dg, db, 0, st, order, dpos, block_first, V, K, V_dev,
                       entries_dev, r4, b.G, b.GX, hi, bkey, bval, ranges, nranges, fc, bb);
  else
    hipLaunchKernelGGL((k_binning<SortTile<kSmallR>::kTile>), dg, db, 0, st, order, dpos, block_first, V, K, V_dev,
                       entries_dev, r4, b.G, b.GX, hi, bkey, bval, ranges, nranges, fc, bb);
  const FinalOut none{nullptr, nullptr, nullptr, nullptr};
  const DigitWeights now{};
  const FirstEntries nofe{nullptr, nullptr, 0, nullptr, nullptr};
  hipLaunchKernelGGL(k_radix_digit_scan, dim3(1u << hi), db, 0, st, counts, tiles, totals, K, entries_dev,
                     (uint32_t)(large ? SortTile<kLargeR>::kTile : SortTile<kSmallR>::kTile), now);
  if (wide)
    hipLaunchKernelGGL((k_radix_scatter<uint32_t, kLargeR, kWideDigits, false, false>), dg, db, 0, st, bkey, bval, bkey_alt,
                       bval_alt, K, entries_dev, 0, hi, tiles, counts, totals, none, now, nofe, ct, DigitRows{});
  else if (large)
    hipLaunchKernelGGL((k_radix_scatter<uint32_t, kLargeR, kDigits, false, false>), dg, db, 0, st, bkey, bval, bkey_alt,
                       bval_alt, K, entries_dev, 0, hi, tiles, counts, totals, none, now, nofe, ct, DigitRows{});
  else
    hipLaunchKernelGGL((k_radix_scatter<uint32_t, kSmallR, kDigits, false, false>), dg, db, 0, st, bkey, bval, bkey_alt,
                       bval_alt, K, entries_dev, 0, hi, tiles, counts, totals, none, now, nofe, ct, DigitRows{});
  BlockExpand x;
  x.ckey = bkey_alt;
  x.crank = bval_alt;
  x.mask_lo = bkey;   // the pair of work arrays that the sorted entries leave free
  x.mask_hi = bval;
  x.start = bt.start;
  x.entries = entries_dev;
  x.nb = 1 << hi;
  x.BX = b.GX;
  x.GX = g.GX;
  x.GY = g.GY;
  x.desc_shift = hi;
  x.order = order;
  x.dkeys = dkeys;
  x.rect = r4;
  x.xy = m2;
  x.conic = c4;
  x.sums = bt.sums;
  x.rowsum = bt.sums + g.nbins;
  x.ecount = bt.ecount;
  x.desc = bt.desc;
  x.rows = bt.rows;
  x.K = K;
  x.K_dev = K_dev;
  x.ranges = ranges;
  x.masks = masks;
  x.vals = vals;
  x.keys = keys;
  return launch_block_expand(x, g.G, tight, st);
}

}  // namespace gsi
