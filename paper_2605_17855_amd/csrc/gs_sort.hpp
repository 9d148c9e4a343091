// Device helpers shared by the sort (gs_sort.hip) and the two-level binning (gs_blocks.hip), and the
// latter's interface.
#pragma once

#include "gs_internal.hpp"

namespace gsi {

// Exclusive scan of v over the 256 threads of the workgroup (wave shuffles, one LDS
// exchange of the four wave totals); *total = the sum.  sh4 holds 4 values.
template <typename T>
__device__ __forceinline__ T block_exclusive_scan_t(T v, T *sh4, T *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  T incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const T u = __shfl_up(incl, off, 64);
    if (lane >= off) incl += u;
  }
  if (lane == 63) sh4[w] = incl;
  block_sync();
  T before = 0, all = 0;
#pragma unroll
  for (int k = 0; k < kBlock / 64; ++k) {
    const T x = sh4[k];
    before += k < w ? x : (T)0;
    all += x;
  }
  block_sync();
  *total = all;
  return before + incl - v;
}
// n is *n_dev when n_dev is given (the grid then covers an upper bound and the surplus
// workgroups return at once), else n_host.
__device__ __forceinline__ uint64_t count_of(uint64_t n_host, const uint32_t *n_dev) {
  return n_dev ? (uint64_t)*n_dev : n_host;
}

// Member tiles of a group entry without culling: the rectangle of the footprint's tiles inside
// group (gx, gy), [x0, x1) x [y0, y1) in member-tile units.  The binning packs it (x0, x1 - 1,
// y0, y1 - 1 at 3 bits each) above the bin bits of the entry's sort key, which the bin passes
// carry along without sorting on them, so the ranges kernel expands it into the mask without
// gathering the Gaussian's rect again.
constexpr int kRectDescBits = 12;
__device__ __forceinline__ uint32_t rect_desc(ushort4 rc, int G, int gx, int gy) {
  const int x0 = max((int)rc.x - gx * G, 0), x1 = min((int)rc.z - gx * G, G);
  const int y0 = max((int)rc.y - gy * G, 0), y1 = min((int)rc.w - gy * G, G);
  return (uint32_t)x0 | (uint32_t)(x1 - 1) << 3 | (uint32_t)y0 << 6 | (uint32_t)(y1 - 1) << 9;
}
__device__ __forceinline__ uint64_t rect_desc_mask(uint32_t desc, int G) {
  const int x0 = desc & 7, x1 = (int)((desc >> 3) & 7) + 1, y0 = (desc >> 6) & 7, y1 = (int)((desc >> 9) & 7) + 1;
  const uint64_t row = ((1ull << (x1 - x0)) - 1ull) << x0;   // x1 - x0 <= G <= 8
  uint64_t m = 0;
  for (int ly = y0; ly < y1; ++ly) m |= row << (ly * G);
  return m;
}

// ---- two-level binning: expansion of the sorted block entries (gs_blocks.hip) ----------------
// Entries of a chunk: the unit of the counting and expanding kernels' workgroups.  (256: 2160p frames
// of 3M Gaussians 106 instead of 86 us in the expansion.)
constexpr int kChunk = 512;

// Scratch of the expansion over at most K block entries.  In the radix scratch, free once the entries
// are sorted: per chunk and sub-bin the entry counts, then their prefix over the block's chunks,
// and the chunk descriptors.  Of its own: the entry sums per bin and per (bin row, block), and the
// chunk table.
struct BlockTmp {
  uint64_t rows;   // chunks of K' entries in at most 512 blocks, for any K' <= K
  uint32_t *ecount;
  uint2 *desc;
  size_t radix_bytes;
  uint32_t *sums;
  uint64_t *start;   // (kMaxBlocks + 1)
  size_t bytes;
  static uint64_t nsums(const Grid &g, const Grid &b) {
    return (uint64_t)g.nbins + (uint64_t)b.nbins * (kBlockTiles / g.G);
  }
};
inline BlockTmp block_tmp_layout(void *radix_tmp, void *tmp, uint64_t K) {
  BlockTmp t;
  t.rows = K / kChunk + (K < kMaxBlocks ? K : kMaxBlocks);
  const size_t ecount_bytes = t.rows * 64 * sizeof(uint32_t);
  t.ecount = static_cast<uint32_t *>(radix_tmp);
  t.desc = reinterpret_cast<uint2 *>(static_cast<char *>(radix_tmp) + ecount_bytes);
  t.radix_bytes = ecount_bytes + t.rows * sizeof(uint2);
  const size_t sums_bytes = (size_t)kMaxBlocks * (kBlockTiles * kBlockTiles + kBlockTiles) * sizeof(uint32_t);
  t.sums = static_cast<uint32_t *>(tmp);
  t.start = reinterpret_cast<uint64_t *>(static_cast<char *>(tmp) + sums_bytes);
  t.bytes = sums_bytes + (kMaxBlocks + 1) * sizeof(uint64_t);
  return t;
}

struct BlockExpand {
  const uint32_t *ckey, *crank;    // block entries in (block, depth) order: sort key, depth rank
  uint32_t *mask_lo, *mask_hi;     // their tile masks (opacity-aware culling only)
  const uint64_t *start;           // before each block: entries (high word), chunks (low word)
  const uint32_t *entries;         // all block entries
  int nb, BX;                      // blocks (rounded up to a power of two), blocks per row
  int GX, GY;                      // grid of the bins
  int desc_shift;                  // the footprint's tiles in the block lie above this many key bits
  const uint32_t *order, *dkeys;
  const ushort4 *rect;
  const double2 *xy;
  const float4 *conic;
  uint32_t *sums, *rowsum;         // entries per bin; per (bin row, block)
  uint32_t *ecount;                // entries per (chunk, sub-bin), then those of the block's earlier chunks
  uint2 *desc;                     // per chunk: first entry; block, entries << 9, first of its block << 31
  uint64_t rows;                   // chunks the two hold
  uint64_t K;                      // entries of the bins: their count, or with K_dev an upper bound of *K_dev
  const uint32_t *K_dev;
  uint32_t *ranges;
  void *masks;
  uint32_t *vals;
  uint64_t *keys;
};
hipError_t launch_block_expand(const BlockExpand &x, int G, bool tight, hipStream_t st);

}  // namespace gsi
