// Two-level binning, second half: block entries to bin entries.
//
// Background ("Gaussian sorting") duplicates every Gaussian once per tile it overlaps and sorts
// the copies.  Here the copies that are sorted are per 8x8-tile block (bin_and_sort_blocks in
// gs_sort.hip: a fifth to a tenth of the tile entries, and one radix pass over the block bits
// instead of two or more over the bin bits).  The sorted list of a block holds its Gaussians in
// depth order, so the list of any bin inside the block is the sublist of the entries whose tile
// mask reaches it, in the same order: the bins are expanded by compaction, with no sort.
//
// A block's list is cut into chunks of 512 entries, one workgroup each:
//   k_block_count   tile mask of each entry (from the rectangle in its sort key, or the alpha-cut
//                   ellipse under opacity-aware culling) and entries per (chunk, sub-bin) by ballot;
//   k_block_sums    (one workgroup per block) those counts to their prefix over the block's chunks,
//                   the sums per bin and per (bin row, block), and the chunks' descriptors;
//   k_block_expand  first place of each (chunk, sub-bin) from those sums, the compacted entries
//                   (index, key, membership mask) and the bin ranges.
// All are bound by chains of dependent loads on a 1M-Gaussian frame (each trip to data that another
// kernel wrote costs ~0.8 us), the last by its stores on large ones.  (Sums by integer atomics in
// k_block_count saved the second launch, but atomics on one address from several XCDs take ~0.2 us
// each: 88 us instead of 22 on the dense scene's ~80 chunks per block.)
#include "gs_sort.hpp"

namespace gsi {
namespace {

constexpr int CH = kChunk;

// Chunk of the whole sorted list: block `block`, entries [e0, e0 + cnt).
struct Chunk {
  int block, cnt;
  uint32_t e0;
};

// Chunks of the list (none without entries: the table of an empty sort is not written).
__device__ __forceinline__ uint32_t chunk_total(const BlockExpand &x) {
  const uint32_t n = *x.entries, total = (uint32_t)x.start[x.nb];
  return n == 0 ? 0u : total;
}

// Chunk `item` by the chunk table.  Every wave searches for itself: 64 probes eight blocks apart, then
// the eight blocks of one (two round trips, no barrier).
__device__ __forceinline__ Chunk find_chunk(const BlockExpand &x, uint32_t item) {
  static_assert(kMaxBlocks == 64 * 8, "two search steps");
  const int lane = threadIdx.x & 63;
  const uint64_t s0 = x.start[min(8 * lane, x.nb)];
  const uint64_t m0 = __ballot(8 * lane < x.nb && (uint32_t)s0 <= item);
  const int b0 = 8 * (63 - __clzll(m0));
  const uint64_t s1 = x.start[min(b0 + min(lane, 8), x.nb)];
  // last block whose first chunk is <= item: it has chunks (an empty block shares its start)
  const uint64_t m1 = __ballot(lane < 8 && b0 + lane < x.nb && (uint32_t)s1 <= item);
  const int l = 63 - __clzll(m1);
  const uint32_t c = item - (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)s1, l);
  const uint32_t e = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(s1 >> 32), l);
  const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(s1 >> 32), l + 1);
  return Chunk{b0 + l, (int)min((uint32_t)CH, end - e - c * CH), e + c * CH};
}

// Chunks of a workgroup: number b of the grid, then with the grid's stride; runs of 16 neighbouring
// chunks, which write side by side into the same bins, go to one XCD.  The chunks' number is
// known only on the device and usually far below the bound that would size a grid of one each (the
// block entries are bounded by the bin entries): tens of thousands of workgroups with nothing to do
// cost 20 us of dispatch on a 4K frame.
constexpr unsigned kChunkRun = 16, kRunGrid = kXcds * kChunkRun;
inline unsigned chunk_grid(uint64_t chunks, unsigned most) {
  const uint64_t g = (chunks + kRunGrid - 1) / kRunGrid * kRunGrid;
  return (unsigned)(g < most ? g : most);
}
struct ChunkLoop {
  uint32_t b, total;
  __device__ __forceinline__ explicit ChunkLoop(uint32_t n) : b(blockIdx.x), total(n) {}
  __device__ __forceinline__ uint32_t item() const {
    return (b / kRunGrid * kXcds + b % kXcds) * kChunkRun + b / kXcds % kChunkRun;
  }
  // (the items of kRunGrid consecutive numbers are kRunGrid consecutive chunks)
  __device__ __forceinline__ bool more() const { return b / kRunGrid * kRunGrid < total; }
  __device__ __forceinline__ bool valid() const { return item() < total; }
  __device__ __forceinline__ void next() { b += gridDim.x; }
};

// Sub-bins: a block holds S x S bins of G = 8 / S tiles a side, shared evenly by the waves in order,
// so that each wave's tiles lie in one 32-bit half of the tile mask (rows 0..3 or 4..7): sub_mask
// is sub-bin s's tiles in that half.
template <int S>
__device__ __forceinline__ uint32_t sub_mask(int s) {
  constexpr int G = kBlockTiles / S;
  const int row = (s / S) * G % 4, col = (s % S) * G;
  const uint32_t r = (1u << G) - 1u;
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < G; ++i) m |= r << (8 * i);
  return m << (8 * row + col);
}

// Membership mask of sub-bin s (bit ly G + lx) from a block's tile mask.
template <int S>
__device__ __forceinline__ uint32_t member_mask(uint64_t m, int s) {
  constexpr int G = kBlockTiles / S;
  const uint64_t v = m >> (8 * (s / S) * G + (s % S) * G);
  uint32_t out = 0;
#pragma unroll
  for (int i = 0; i < G; ++i) out |= ((uint32_t)(v >> (8 * i)) & ((1u << G) - 1u)) << (i * G);
  return out;
}

// Tiles of block (bx, by) that the ellipse meets, of its tile rows ly0..ly1 (the footprint's).
__device__ __forceinline__ uint64_t tight_block_mask(const TightEllipse &e, int bx, int by, int ly0, int ly1) {
  uint64_t m = 0;
  for (int ly = ly0; ly <= ly1; ++ly) {
    int lo, hi;
    tight_row_span(e, by * kBlockTiles + ly, &lo, &hi);
    lo = max(lo - bx * kBlockTiles, 0);
    hi = min(hi - bx * kBlockTiles, kBlockTiles - 1);
    if (lo <= hi) m |= (uint64_t)(((1u << (hi - lo + 1)) - 1u) << lo) << (8 * ly);
  }
  return m;
}

template <int S, bool TIGHT>
__global__ __launch_bounds__(kBlock) void k_block_count(BlockExpand x) {
  constexpr int NS = S * S, kSubs = NS / 4, kWords = CH / 64;
  __shared__ uint64_t s_mask[CH];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  bool again = false;
  for (ChunkLoop at(chunk_total(x)); at.more(); at.next()) {
    if (!at.valid()) continue;
    if (again) block_sync();   // the masks of the chunk before are read
    again = true;
    const uint32_t item = at.item();
    const Chunk k = find_chunk(x, item);
    const int bx = k.block % x.BX, by = k.block / x.BX;
#pragma unroll
    for (int it = 0; it < CH / kBlock; ++it) {
      const int i = it * kBlock + t;
      uint64_t m = 0;
      if (i < k.cnt) {
        const uint32_t e = k.e0 + (uint32_t)i;
        const uint32_t desc = x.ckey[e] >> x.desc_shift;
        m = rect_desc_mask(desc, kBlockTiles);
        if (TIGHT) {
          const uint32_t g = x.order[x.crank[e]];
          if (m) {
            const ushort4 rc = x.rect[g];
            const double2 mu = x.xy[g];
            const float4 co = x.conic[g];
            const TightEllipse el = tight_ellipse(mu.x, mu.y, co.x, co.y, co.z, co.w, rc.x, rc.z - 1, rc.y);
            m = tight_block_mask(el, bx, by, (int)((desc >> 6) & 7u), (int)((desc >> 9) & 7u));
          }
          x.mask_lo[e] = (uint32_t)m;
          x.mask_hi[e] = (uint32_t)(m >> 32);
        }
      }
      s_mask[i] = m;
    }
    block_sync();
    uint32_t h[kWords];
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
      const uint64_t m = s_mask[i * 64 + lane];
      h[i] = w >= 2 ? (uint32_t)(m >> 32) : (uint32_t)m;
    }
    uint32_t mine = 0;   // lane q: entries of sub-bin w kSubs + q
    for (int q = 0; q < kSubs; ++q) {
      const uint32_t sm = sub_mask<S>(w * kSubs + q);
      uint32_t n = 0;
#pragma unroll
      for (int i = 0; i < kWords; ++i) n += (uint32_t)__popcll(__ballot((h[i] & sm) != 0u));
      mine = lane == q ? n : mine;
    }
    if (lane < kSubs) x.ecount[(uint64_t)item * NS + w * kSubs + lane] = mine;
  }
}

// One workgroup per block.
template <int S>
__global__ __launch_bounds__(kBlock) void k_block_sums(BlockExpand x) {
  constexpr int NS = S * S, P = kBlock / NS;   // P parts of the block's chunks side by side
  __shared__ uint32_t s_part[kBlock];
  const int b = blockIdx.x, t = threadIdx.x, s = t % NS, p = t / NS;
  const uint32_t total = *x.entries;
  const uint64_t s0 = x.start[b], s1 = x.start[b + 1];
  const uint32_t c0 = (uint32_t)s0, nc = (uint32_t)s1 - c0, e0 = (uint32_t)(s0 >> 32), e1 = (uint32_t)(s1 >> 32);
  if (total == 0 || nc == 0) return;
  for (uint32_t c = t; c < nc; c += kBlock)
    x.desc[c0 + c] = make_uint2(e0 + c * CH, (uint32_t)b | min((uint32_t)CH, e1 - e0 - c * CH) << 9 | (c == 0 ? 1u << 31 : 0u));
  const uint32_t per = (nc + P - 1) / P, a = min(nc, p * per), e = min(nc, a + per);
  uint32_t *cnt = x.ecount + (uint64_t)c0 * NS + s;
  uint32_t sum = 0;
#pragma unroll 8
  for (uint32_t c = a; c < e; ++c) sum += cnt[(uint64_t)c * NS];
  s_part[t] = sum;
  block_sync();
  uint32_t run = 0;
  for (int q = 0; q < p; ++q) run += s_part[q * NS + s];
#pragma unroll 4
  for (uint32_t c = a; c < e; ++c) {
    const uint32_t n = cnt[(uint64_t)c * NS];
    cnt[(uint64_t)c * NS] = run;
    run += n;
  }
  if (t < 64) {   // the sums: lane s of the first wave
    uint32_t n = 0;
    const int ss = t < NS ? t : 0;
    for (int q = 0; q < P; ++q) n += s_part[q * NS + ss];
    const int gx = (b % x.BX) * S + ss % S, gy = (b / x.BX) * S + ss / S;
    uint32_t row = n;
#pragma unroll
    for (int off = 1; off < S; off <<= 1) row += (uint32_t)__shfl_xor((int)row, off, 64);
    if (t < NS && gx < x.GX && gy < x.GY) x.sums[gy * x.GX + gx] = n;
    if (t < NS && ss % S == 0 && gy < x.GY) x.rowsum[gy * x.BX + b % x.BX] = row;
  }
}

template <int S, bool TIGHT>
__global__ __launch_bounds__(kBlock) void k_block_expand(BlockExpand x) {
  constexpr int NS = S * S, kSubs = NS / 4, kWords = CH / 64, G = kBlockTiles / S, kItems = CH / kBlock;
  constexpr int kGroup = kSubs < 4 ? kSubs : 4;                    // sub-bins compacted together
  constexpr int kRows = (int)kMaxBlocks * S / kBlock;              // (row, block) sums per thread
  __shared__ uint64_t s_mask[CH];
  __shared__ uint2 s_gd[CH];                      // Gaussian index, depth bits
  __shared__ uint16_t s_list[4][kGroup * CH];     // per wave: entry | sub-bin (of the group) << 9
  __shared__ uint32_t s_row[S], s_base[NS], s_first[4][kGroup];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  // first round trip: the first chunk, their number, and every (row, block) sum
  ChunkLoop at(0);
  uint2 desc = x.desc[min((uint64_t)at.item(), x.rows - 1)];
  const int nr = x.GY * x.BX;
  uint32_t rs[kRows];
#pragma unroll
  for (int j = 0; j < kRows; ++j) rs[j] = j * kBlock + t < nr ? x.rowsum[j * kBlock + t] : 0u;
  at.total = chunk_total(x);
  const uint32_t K = x.K_dev ? *x.K_dev : (uint32_t)x.K;   // (below 2^32)
  bool again = false;
  for (; at.more(); at.next()) {
    if (!at.valid()) continue;
    const uint32_t item = at.item();
    if (again) {
      desc = x.desc[item];
      block_sync();   // the LDS of the chunk before is read to the end
    }
    again = true;
    const uint32_t e0 = desc.x;
    const int block = (int)(desc.y & 511u), cnt = (int)(desc.y >> 9 & 1023u);
    const int bx = block % x.BX, by = block / x.BX;
    // second: the chunk's entries, its places and its bins' sums
    const int s = t < NS ? t : 0, gx = bx * S + s % S, gy = by * S + s / S;
    const bool bin_in = t < NS && gx < x.GX && gy < x.GY;
    const uint32_t bin_n = bin_in ? x.sums[gy * x.GX + gx] : 0u;
    const uint32_t before = t < NS ? x.ecount[(uint64_t)item * NS + s] : 0u;
    uint32_t rank[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
      const int i = it * kBlock + t;
      uint64_t m = 0;
      rank[it] = 0;
      if (i < cnt) {
        const uint32_t e = e0 + (uint32_t)i;
        rank[it] = x.crank[e];
        m = TIGHT ? (uint64_t)x.mask_hi[e] << 32 | x.mask_lo[e] : rect_desc_mask(x.ckey[e] >> x.desc_shift, kBlockTiles);
      }
      s_mask[i] = m;
    }
    if (t < S) s_row[t] = 0;
    block_sync();
    // third: their Gaussians and depths; meanwhile the first place of the block's part of each of
    // its bin rows: the (row, block) sums before it, row by row.  s_row[r] holds what lies between the
    // parts of rows r - 1 and r, s_row[0] all before.
    uint2 gd[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it)
      gd[it] = it * kBlock + t < cnt ? make_uint2(x.order[rank[it]], x.dkeys[rank[it]]) : make_uint2(0u, 0u);
    {
      const int i0 = by * S * x.BX + bx, i1 = i0 + (S - 1) * x.BX;
      uint32_t sum = 0;
#pragma unroll
      for (int j = 0; j < kRows; ++j) {
        const int i = j * kBlock + t;
        sum += i < i0 ? rs[j] : 0u;
        if (i >= i0 && i < i1 && rs[j]) atomicAdd(&s_row[(i - i0) / x.BX + (S > 1)], rs[j]);
      }
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) sum += (uint32_t)__shfl_xor((int)sum, off, 64);
      if (lane == 0 && sum) atomicAdd(&s_row[0], sum);
    }
#pragma unroll
    for (int it = 0; it < kItems; ++it) s_gd[it * kBlock + t] = gd[it];
    block_sync();
    // first place of each sub-bin, and of the chunk's entries in it; the ranges
    if (t < 64) {
      uint32_t incl = bin_n;
#pragma unroll
      for (int off = 1; off < S; off <<= 1) {
        const uint32_t u = __shfl_up(incl, off, 64);
        if (s % S >= off) incl += u;
      }
      uint32_t first = incl - bin_n;
      for (int r = 0; r <= s / S; ++r) first += s_row[r];
      if (t < NS) s_base[s] = first + before;
      if ((desc.y >> 31) && bin_n) {
        const int bin = gy * x.GX + gx;
        x.ranges[2 * bin] = min(first, K);
        x.ranges[2 * bin + 1] = min(first + bin_n, K);
      }
    }
    block_sync();
    uint32_t h[kWords];
#pragma unroll
    for (int i = 0; i < kWords; ++i) {
      const uint64_t m = s_mask[i * 64 + lane];
      h[i] = w >= 2 ? (uint32_t)(m >> 32) : (uint32_t)m;
    }
    uint16_t *list = s_list[w];
#pragma unroll 1
    for (int q0 = 0; q0 < kSubs; q0 += kGroup) {
      int n = 0;
      uint32_t first = 0;   // lane q: place of list position 0 in sub-bin q0 + q's entries
#pragma unroll
      for (int q = 0; q < kGroup; ++q) {
        const int sq = w * kSubs + q0 + q;
        const uint32_t sm = sub_mask<S>(sq);
        first = lane == q ? s_base[sq] - (uint32_t)n : first;
#pragma unroll
        for (int i = 0; i < kWords; ++i) {
          const bool in = (h[i] & sm) != 0u;
          const uint64_t m = __ballot(in);
          if (in)
            list[n + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))] =
                (uint16_t)(i * 64 + lane | q << 9);
          n += __popcll(m);
        }
      }
      if (lane < kGroup) s_first[w][lane] = first;
      // (list and places are written and read by lanes of this wave only)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const int sq0 = w * kSubs + q0;
      const uint32_t bin0 = (uint32_t)((by * S + sq0 / S) * x.GX + bx * S + sq0 % S);
      // (U at a time: the two LDS reads behind each other and the stores of several overlap)
      constexpr int U = 2;
      for (int j0 = 0; j0 < n; j0 += U * 64) {
        uint32_t v[U], p[U];
        uint2 g[U];
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const int j = j0 + i * 64 + lane;
          v[i] = j < n ? list[j] : 0u;
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const int j = j0 + i * 64 + lane;
          p[i] = j < n ? s_first[w][v[i] >> 9] + (uint32_t)j : ~0u;
          g[i] = s_gd[v[i] & 511u];
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const uint32_t q = v[i] >> 9;
          if (p[i] < K) {   // (holds for counts and footprints that agree)
            x.vals[p[i]] = g[i].x;
            *reinterpret_cast<uint2 *>(x.keys + p[i]) = make_uint2(g[i].y, bin0 + q);
            if (G > 1)
              static_cast<uint16_t *>(x.masks)[p[i]] = (uint16_t)member_mask<S>(s_mask[v[i] & 511u], sq0 + (int)q);
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
}

template <int S, bool TIGHT>
hipError_t launch_t(const BlockExpand &x, hipStream_t st) {
  // chunks of at most K entries in nb blocks; the grids hold about what the CUs do, twice over
  const uint64_t chunks = x.K / CH + ((uint64_t)x.nb < x.K ? (uint64_t)x.nb : x.K);
  const dim3 grid(chunk_grid(chunks, 4096)), block(kBlock);
  hipLaunchKernelGGL((k_block_count<S, TIGHT>), grid, block, 0, st, x);
  hipLaunchKernelGGL((k_block_sums<S>), dim3((unsigned)x.nb), block, 0, st, x);
  hipLaunchKernelGGL((k_block_expand<S, TIGHT>), grid, block, 0, st, x);
  return hipGetLastError();
}

template <int S>
hipError_t launch_s(const BlockExpand &x, bool tight, hipStream_t st) {
  return tight ? launch_t<S, true>(x, st) : launch_t<S, false>(x, st);
}

}  // namespace

size_t block_tmp_bytes() { return block_tmp_layout(nullptr, nullptr, 0).bytes; }
size_t block_radix_tmp_bytes(uint64_t K) { return block_tmp_layout(nullptr, nullptr, K).radix_bytes; }

hipError_t launch_block_expand(const BlockExpand &x, int G, bool tight, hipStream_t st) {
  switch (G) {
    case 1: return launch_s<8>(x, tight, st);
    case 2: return launch_s<4>(x, tight, st);
    case 4: return launch_s<2>(x, tight, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace gsi
