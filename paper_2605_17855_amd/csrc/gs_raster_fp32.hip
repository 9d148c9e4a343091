// Plain FP32 rasterizer (paper, Background: tile-based rasterization, eq. power_d, eq. power).
//
// One 256-lane workgroup per tile; lane = pixel, wave = 8x8 quadrant.  The tile's depth-sorted
// list is streamed through LDS in chunks of 256 entries.  Per (entry, pixel):
//   d = x - mu'                       (eq. power_d)
//   log2(alpha_raw) = log2(o) + log2(e) * (-1/2 d^T conic d)   (eq. power)
//   skip when alpha_raw < 1/255, alpha = min(0.99, alpha_raw)
//   T' = T (1 - alpha); stop (without blending) when T' < 1e-4; else C += alpha T c, T = T'.
// The pixel's offset to the centre is formed from a bin-relative FP32 copy of the FP64
// centre, so |d| stays small and exact.
//
// Each wave walks only the rows whose alpha can reach the 1/255 cut in its own quadrant (the
// quadrant mask of the tensorized rasterizer, with a margin that follows the FP32 power's rounding,
// so no output changes).  A row's nine floats are LDS reads broadcast to 64
// pixels, ~20 LDS cycles per wave and row at 128 B per cycle, and four SIMDs share one LDS:
// running every row in every quadrant was bound by exactly that (6.3M wave-rows of a 1M-Gaussian
// 1080p frame, 242 us).  The lists keep about a third of them: 107 us, bound by vector issue (94 % of the
// SIMD cycles).
//
// Tile groups (G > 1): one workgroup per member tile, walking the group's list and keeping the
// entries whose mask holds its tile, in list order, in a row buffer that fills over several
// steps (the member-tile rasterizer of gs_raster_mfma.hip); centres stay relative to the group.
// (One workgroup per 2x2 group, four pixels a lane, takes 261 us instead of 105 on a 1M-Gaussian 1080p
// frame, culled: the longest groups' serial walks.  Large culled frames still take it, see there.)
#include <type_traits>

#include "gs_mfma.hpp"

namespace gsi {
namespace {

template <int CAP_>
struct Fp32Shared {
  static constexpr int CAP = CAP_;
  float4 a[CAP + 1];     // (u, v, -a/2 log2e, -b log2e); row CAP never passes the cut
  float4 b[CAP + 1];     // (-c/2 log2e, log2 o, r, g)
  float c[CAP + 1];      // b
  uint32_t alive[2][4];
  __align__(16) uint32_t wcnt[2][4];   // groups: the tile's entries per wave in a step, by step parity
  uint8_t qm[CAP];       // quadrant masks
  uint16_t wl[4][CAP];   // each wave's row list
};

struct PixelState {
  float T, C0, C1, C2, W, cut;
  uint32_t nstop, nblend, last;   // last: 1 + list position of the last Gaussian blended
};

// Runs the rows wl[0, n) (ascending buffer indices) for this lane's pixel (X, Y).  Rows go in
// blocks of four, all their LDS reads and powers ahead of the blends.  row_base: list position
// of buffer row 0.
template <bool AUX, typename SM>
__device__ __forceinline__ void blend_rows(const SM &sm, const uint16_t *wl, int n, float X, float Y, PixelState &st,
                                           uint32_t row_base) {
  constexpr int U = 4;
  const int lane = threadIdx.x & 63;
  for (int r0 = 0; r0 < n; r0 += 64) {
    // a wave whose pixels have all stopped leaves its list
    if (__ballot(st.cut != INFINITY) == 0) return;
    const int idx = r0 + lane < n ? (int)wl[r0 + lane] : SM::CAP;
    const int m = min(64, n - r0);
    for (int k = 0; k < m; k += U) {
      float D[U];
      float4 B[U];
      float c2[U];
      int ri[U];
#pragma unroll
      for (int j = 0; j < U; ++j) {
        ri[j] = __builtin_amdgcn_readlane(idx, k + j);
        const float4 A = sm.a[ri[j]];
        B[j] = sm.b[ri[j]];
        c2[j] = sm.c[ri[j]];
        const float dx = X - A.x, dy = Y - A.y;
        D[j] = fmaf(dx, fmaf(A.z, dx, A.w * dy), fmaf(B[j].x * dy, dy, B[j].y));
      }
#pragma unroll
      for (int j = 0; j < U; ++j) {
        if (D[j] >= st.cut) {
          // branch-free body: T' = T (1 - alpha) as one FMA; a stop (T' < 1e-4) blends
          // nothing, keeps T and disables the pixel
          const float al = fminf(kAlphaMax, __builtin_amdgcn_exp2f(D[j]));
          const float Tn = fmaf(-st.T, al, st.T);
          const bool ok = Tn >= kTMin;
          const float wgt = ok ? al * st.T : 0.0f;
          st.C0 = fmaf(wgt, B[j].z, st.C0);
          st.C1 = fmaf(wgt, B[j].w, st.C1);
          st.C2 = fmaf(wgt, c2[j], st.C2);
          st.T = ok ? Tn : st.T;
          st.cut = ok ? st.cut : INFINITY;
          if (AUX) {
            st.W += wgt;
            st.nblend += ok ? 1u : 0u;
            st.nstop = ok ? st.nstop : row_base + (uint32_t)ri[j] + 1u;
            st.last = ok ? row_base + (uint32_t)ri[j] + 1u : st.last;
          }
        }
      }
    }
  }
}

// Stages Gaussian g as row `pos`: centre relative to (ox, oy); the quadrant test in the frame of
// the tile at (tx0, ty0).
template <typename SM>
__device__ __forceinline__ void stage_row(SM &sm, int pos, double2 m, float4 co, float4 cl, int ox, int oy, int tx0,
                                          int ty0, bool all_rows) {
  sm.a[pos] = make_float4((float)(m.x - ox), (float)(m.y - oy), -0.5f * kLog2e * co.x, -kLog2e * co.y);
  sm.b[pos] = make_float4(-0.5f * kLog2e * co.z, __log2f(co.w), cl.x, cl.y);
  sm.c[pos] = cl.z;
  const float ut = (float)(m.x - ((double)tx0 + 8.5)), vt = (float)(m.y - ((double)ty0 + 8.5));
  sm.qm[pos] = all_rows ? (uint8_t)0xF
                        : (uint8_t)mfma::quad_mask_fp32(ut, vt, co.x, co.y, co.z, mfma::log2_opacity(co.w));
}

template <bool AUX>
__device__ __forceinline__ void write_pixel(const RasterJob &J, const RasterParams &P, int xx, int yy,
                                            const PixelState &st, uint32_t rows_done) {
  if (xx >= J.W || yy >= J.H) return;
  const int64_t HW = (int64_t)J.W * J.H;
  const int64_t pix = (int64_t)yy * J.W + xx;
  J.image[pix] = st.C0 + st.T * P.bg[0];
  J.image[HW + pix] = st.C1 + st.T * P.bg[1];
  J.image[2 * HW + pix] = st.C2 + st.T * P.bg[2];
  if (AUX) {
    int plane = 0;
    if (P.aux_flags & GS_AUX_TFINAL) J.aux[(plane++) * HW + pix] = st.T;
    if (P.aux_flags & GS_AUX_WSUM) J.aux[(plane++) * HW + pix] = st.W;
    if (P.aux_flags & GS_AUX_NEVAL) {
      const bool stopped = (st.cut == INFINITY);
      J.aux[(plane++) * HW + pix] = (float)(stopped ? st.nstop : rows_done);
    }
    if (P.aux_flags & GS_AUX_NBLEND) J.aux[(plane++) * HW + pix] = (float)st.nblend;
    if (P.aux_flags & GS_AUX_LAST) J.aux[(plane++) * HW + pix] = (float)st.last;
  }
}

// Renders work item `item` of job J (one workgroup): a tile (G == 1) or member tile
// item % G^2 (row-major) of group item / G^2.  Shared by the single-image and batched kernels.
template <int G, bool AUX, typename SM>
__device__ __forceinline__ void raster_item_fp32(const RasterJob &J, const RasterParams &P, int item, SM &sm) {
  constexpr int NT = G * G, CAP = SM::CAP;
  const int bin = item / NT, k = item % NT;
  const int ox = (bin % J.GX) * G * kTile, oy = (bin / J.GX) * G * kTile;
  const int tx0 = ox + (k % G) * kTile, ty0 = oy + (k / G) * kTile;
  if (G > 1 && (tx0 >= J.W || ty0 >= J.H)) return;   // a member tile past the image (uniform)
  const uint32_t start = J.ranges[2 * bin], end = J.ranges[2 * bin + 1];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int px = (w & 1) * 8 + (lane & 7), py = (w >> 1) * 8 + (lane >> 3);
  const float X = (float)(tx0 - ox + px) + 0.5f, Y = (float)(ty0 - oy + py) + 0.5f;
  PixelState st;
  st.T = 1.0f; st.C0 = st.C1 = st.C2 = 0.0f; st.W = 0.0f;
  st.cut = (tx0 + px < J.W) && (ty0 + py < J.H) ? kCutLog2 : INFINITY;
  st.nstop = 0; st.nblend = 0; st.last = 0;
  uint32_t rows_done = 0;   // uniform: entries of the tile's list blended so far
  if (t == 0) {             // the row of the list slots past a wave's last row
    sm.a[CAP] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    sm.b[CAP] = make_float4(0.0f, -INFINITY, 0.0f, 0.0f);
    sm.c[CAP] = 0.0f;
  }
  int it = 0;

  if constexpr (G == 1) {
    for (uint32_t cs = start; cs < end; cs += kBlock) {
      const int cnt = (int)min((uint32_t)kBlock, end - cs);
      if (it > 0) {
        // every wave is done with the previous chunk and has posted whether it still blends
        block_sync();
        const uint32_t *al = sm.alive[(it - 1) & 1];
        if (!(al[0] | al[1] | al[2] | al[3])) break;
      }
      if (t < cnt) {
        const uint32_t g = J.vals[cs + t];
        stage_row(sm, t, J.xy[g], J.conic[g], J.rgb[g], ox, oy, tx0, ty0, P.all_rows);
      }
      block_sync();
      const int nw = mfma::wave_list(sm.qm, cnt, sm.wl[w]);
      blend_rows<AUX>(sm, sm.wl[w], nw, X, Y, st, rows_done);
      rows_done += (uint32_t)cnt;
      const uint64_t bal = __ballot(st.cut != INFINITY);
      if (lane == 0) sm.alive[it & 1][w] = bal != 0;
      ++it;
    }
  } else {
    int filled = 0;   // uniform: rows in the buffer
    auto blend = [&]() {
      const int nw = mfma::wave_list(sm.qm, filled, sm.wl[w]);
      blend_rows<AUX>(sm, sm.wl[w], nw, X, Y, st, rows_done);
      rows_done += (uint32_t)filled;
      filled = 0;
    };
    bool live = true;
    for (uint32_t cs = start; cs < end; cs += kBlock) {
      if (filled > CAP - kBlock) {   // another step might not fit
        block_sync();
        blend();
        const uint64_t ab = __ballot(st.cut != INFINITY);
        if (lane == 0) sm.alive[0][w] = ab != 0;
        block_sync();
        if (!(sm.alive[0][0] | sm.alive[0][1] | sm.alive[0][2] | sm.alive[0][3])) {
          live = false;
          break;
        }
      }
      const int cnt = (int)min((uint32_t)kBlock, end - cs);
      bool mine = false;
      double2 m = make_double2(0.0, 0.0);
      float4 co = make_float4(0.0f, 0.0f, 0.0f, 0.0f), cl = co;
      if (t < cnt) {
        mine = (static_cast<const uint16_t *>(J.masks)[cs + t] >> k) & 1u;
        if (mine) {
          const uint32_t g = J.vals[cs + t];
          m = J.xy[g];
          co = J.conic[g];
          cl = J.rgb[g];
        }
      }
      const uint64_t bk = __ballot(mine);
      if (lane == 0) sm.wcnt[it & 1][w] = (uint32_t)__popcll(bk);
      block_sync();
      const uint4 ck = *reinterpret_cast<const uint4 *>(sm.wcnt[it & 1]);
      if (mine) {
        const uint32_t woff = (w > 0 ? ck.x : 0u) + (w > 1 ? ck.y : 0u) + (w > 2 ? ck.z : 0u);
        const int pos = filled + (int)(woff + __builtin_amdgcn_mbcnt_hi((uint32_t)(bk >> 32),
                                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)bk, 0u)));
        stage_row(sm, pos, m, co, cl, ox, oy, tx0, ty0, P.all_rows);
      }
      filled += (int)(ck.x + ck.y + ck.z + ck.w);
      ++it;
    }
    if (live && filled > 0) {
      block_sync();
      blend();
    }
  }
  write_pixel<AUX>(J, P, tx0 + px, ty0 + py, st, rows_done);
}

// Renders a whole 2x2 group (one workgroup): a lane has its pixel in each of the four tiles, so that a
// row is read from LDS once for all of them, and every row runs in all quadrants of its tiles.  Where
// culling has left the lists short of rows to skip and the frame has groups enough to hide the longest,
// that beats the quadrant lists, which are bound by those reads: 3840x2160, culled, 1M Gaussians of
// the dense scene 397 us against 535 per member tile, 3M of the clustered one 378 against 472.
struct Fp32GroupShared {
  float4 a[kBlock];   // (u, v, -a/2 log2e, -b log2e)
  float4 b[kBlock];   // (-c/2 log2e, log2 o, r, g)
  float2 c[kBlock];   // (b, mask bits)
  uint32_t alive[2][4];
};

template <bool AUX>
__device__ __forceinline__ void raster_group_fp32(const RasterJob &J, const RasterParams &P, int bin,
                                                  Fp32GroupShared &sm) {
  constexpr int G = 2, NT = 4;
  const int ox = (bin % J.GX) * G * kTile, oy = (bin / J.GX) * G * kTile;
  const uint32_t start = J.ranges[2 * bin], end = J.ranges[2 * bin + 1];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int px = (w & 1) * 8 + (lane & 7), py = (w >> 1) * 8 + (lane >> 3);
  float X[NT], Y[NT];
  // (the state of PixelState in arrays: as four structs the compiler copies it around every row)
  float T[NT], C0[NT], C1[NT], C2[NT], W[NT], cut[NT];
  uint32_t seen[NT], nstop[NT], nblend[NT], last[NT];   // seen: entries of the tile's list so far
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    T[k] = 1.0f; C0[k] = C1[k] = C2[k] = 0.0f; W[k] = 0.0f;
    cut[k] = (ox + px + (k % G) * kTile < J.W) && (oy + py + (k / G) * kTile < J.H) ? kCutLog2 : INFINITY;
    seen[k] = 0; nstop[k] = 0; nblend[k] = 0; last[k] = 0;
    X[k] = (float)(px + (k % G) * kTile) + 0.5f;
    Y[k] = (float)(py + (k / G) * kTile) + 0.5f;
  }
  auto blending = [&]() { return __ballot(fminf(fminf(cut[0], cut[1]), fminf(cut[2], cut[3])) != INFINITY) != 0; };
  int it = 0;
  for (uint32_t cs = start; cs < end; cs += kBlock) {
    const int cnt = (int)min((uint32_t)kBlock, end - cs);
    if (it > 0) {
      // every wave is done with the previous chunk and has posted whether it still blends
      block_sync();
      const uint32_t *al = sm.alive[(it - 1) & 1];
      if (!(al[0] | al[1] | al[2] | al[3])) break;
    }
    if (t < cnt) {
      const uint32_t g = J.vals[cs + t], mk = static_cast<const uint16_t *>(J.masks)[cs + t];
      const double2 m = J.xy[g];
      const float4 co = J.conic[g];
      const float4 cl = J.rgb[g];
      sm.a[t] = make_float4((float)(m.x - ox), (float)(m.y - oy), -0.5f * kLog2e * co.x, -kLog2e * co.y);
      sm.b[t] = make_float4(-0.5f * kLog2e * co.z, __log2f(co.w), cl.x, cl.y);
      sm.c[t] = make_float2(cl.z, __uint_as_float(mk));
    }
    block_sync();
    for (int j = 0; j < cnt; ++j) {
      if ((j & 31) == 0) {
        bool any = false;
#pragma unroll
        for (int k = 0; k < NT; ++k) any |= cut[k] != INFINITY;
        if (__ballot(any) == 0) break;
      }
      const float4 a = sm.a[j], b = sm.b[j];
      const float2 c = sm.c[j];
      const uint32_t mk = __float_as_uint(c.y);
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        if (!((mk >> k) & 1u)) continue;   // (uniform)
        if (AUX) ++seen[k];
        const float dx = X[k] - a.x, dy = Y[k] - a.y;
        const float D = fmaf(dx, fmaf(a.z, dx, a.w * dy), fmaf(b.x * dy, dy, b.y));
        if (D >= cut[k]) {   // as in blend_rows
          const float al = fminf(kAlphaMax, __builtin_amdgcn_exp2f(D));
          const float Tn = fmaf(-T[k], al, T[k]);
          const bool ok = Tn >= kTMin;
          const float wgt = ok ? al * T[k] : 0.0f;
          C0[k] = fmaf(wgt, b.z, C0[k]);
          C1[k] = fmaf(wgt, b.w, C1[k]);
          C2[k] = fmaf(wgt, c.x, C2[k]);
          T[k] = ok ? Tn : T[k];
          cut[k] = ok ? cut[k] : INFINITY;
          if (AUX) {
            W[k] += wgt;
            nblend[k] += ok ? 1u : 0u;
            nstop[k] = ok ? nstop[k] : seen[k];
            last[k] = ok ? seen[k] : last[k];
          }
        }
      }
    }
    const bool live = blending();
    if (lane == 0) sm.alive[it & 1][w] = live;
    ++it;
  }
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    const PixelState st{T[k], C0[k], C1[k], C2[k], W[k], cut[k], nstop[k], nblend[k], last[k]};
    write_pixel<AUX>(J, P, ox + px + (k % G) * kTile, oy + py + (k / G) * kTile, st, seen[k]);
  }
}

// rows of LDS: one chunk for a tile, a buffer that takes a step of 256 on top of up to 192 for a
// member tile (as in gs_raster_mfma.hip)
template <int G>
using SharedOf = Fp32Shared<G == 1 ? kBlock : 448>;

// One workgroup per tile, in the XCD-aware order of the MFMA rasterizer, or per member tile, group by
// group.  (Member tiles in that order too, a group's on one XCD: 3840x2160 frames of 3M Gaussians 496 ->
// 483 us, but 1M at 2560x1440 158 -> 163 and 50K at 3840x2160 62 -> 73.)
template <int G, bool AUX>
__global__ __launch_bounds__(kBlock) void k_raster_fp32(RasterJob J, RasterParams P) {
  __shared__ SharedOf<G> sm;
  const int item = G == 1 ? xcd_raster_bin((int)blockIdx.x, J.GX, J.GY) : (int)blockIdx.x;
  if (item < 0) return;
  raster_item_fp32<G, AUX>(J, P, item, sm);
}

// One workgroup per 2x2 group, in the XCD-aware order.
template <bool AUX>
__global__ __launch_bounds__(kBlock) void k_raster_fp32_groups(RasterJob J, RasterParams P) {
  __shared__ Fp32GroupShared sm;
  const int bin = xcd_raster_bin((int)blockIdx.x, J.GX, J.GY);
  if (bin >= 0) raster_group_fp32<AUX>(J, P, bin, sm);
}

// Persistent batched rasterizer (see the MFMA variant); GROUPS: its items are whole 2x2 groups.
template <int G, bool AUX, bool GROUPS>
__global__ __launch_bounds__(kBlock) void k_raster_fp32_batch(const BatchTable tb,
                                                              RasterParams P, uint32_t *counter) {
  __shared__ std::conditional_t<GROUPS, Fp32GroupShared, SharedOf<G>> sm;
  __shared__ int s_item;
  batch_items(counter, tb.total, &s_item, [&](int item) {
    int lo = 0, hi = tb.n_jobs;   // last job with bin0 <= item
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (tb.jobs[mid].bin0 <= item) lo = mid; else hi = mid;
    }
    const RasterJob J = tb.jobs[lo];
    if constexpr (GROUPS)
      raster_group_fp32<AUX>(J, P, item - J.bin0, sm);
    else
      raster_item_fp32<G, AUX>(J, P, item - J.bin0, sm);
  });
}

struct BatchArgs {
  const BatchTable *table;
  int grid;
  uint32_t *counter;
};

template <int G, bool AUX, bool GROUPS = false>
hipError_t launch_g(const RasterJob &j, const RasterParams &p, const BatchArgs *b, hipStream_t st) {
  if (b)
    hipLaunchKernelGGL((k_raster_fp32_batch<G, AUX, GROUPS>), dim3((unsigned)b->grid), dim3(kBlock), 0, st, *b->table,
                       p, b->counter);
  else if constexpr (GROUPS)
    hipLaunchKernelGGL((k_raster_fp32_groups<AUX>), dim3(xcd_raster_grid(j.GX, j.GY)), dim3(kBlock), 0, st, j, p);
  else
    hipLaunchKernelGGL((k_raster_fp32<G, AUX>), dim3(G == 1 ? xcd_raster_grid(j.GX, j.GY) : (unsigned)j.items),
                       dim3(kBlock), 0, st, j, p);
  return hipGetLastError();
}

hipError_t dispatch(const RasterJob &j, const RasterParams &p, const BatchArgs *b, hipStream_t st) {
  const bool aux = p.aux_flags != 0;
  const int parts = b ? b->table->jobs[0].parts : j.parts;   // (the same for all jobs)
  switch (p.G) {
    case 1: return aux ? launch_g<1, true>(j, p, b, st) : launch_g<1, false>(j, p, b, st);
    case 2:
      if (parts == 1) return aux ? launch_g<2, true, true>(j, p, b, st) : launch_g<2, false, true>(j, p, b, st);
      return aux ? launch_g<2, true>(j, p, b, st) : launch_g<2, false>(j, p, b, st);
    case 4: return aux ? launch_g<4, true>(j, p, b, st) : launch_g<4, false>(j, p, b, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_raster_fp32(const RasterJob &j, const RasterParams &p, hipStream_t st) {
  if (j.items == 0) return hipSuccess;
  return dispatch(j, p, nullptr, st);
}

hipError_t launch_raster_fp32_batch(const BatchTable &table, int grid, const RasterParams &p, uint32_t *counter,
                                    hipStream_t st) {
  if (table.total == 0) return hipSuccess;
  BatchArgs b{&table, grid, counter};
  RasterJob dummy{};
  return dispatch(dummy, p, &b, st);
}

}  // namespace gsi
