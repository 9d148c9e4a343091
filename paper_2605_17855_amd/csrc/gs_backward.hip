// Backward pass of the compositing: the derivative of the forward recurrence (paper,
// Background: eq. power_d, eq. power, the 1/255 cut, the 0.99 clamp, the 1e-4 stop) on the
// branch the forward takes.
//
// One 256-lane workgroup per 16x16 tile, one pixel per lane, 8x8 quadrants per wave as in the
// forward; each wave walks only the rows whose alpha can reach the cut in its quadrant (the
// forward's masks).  The tile's list is taken back to front in chunks of 256 entries.  Per
// (row, pixel) pair, T_i = T_{i+1} / (1 - alpha_i) (a 1-ulp hardware reciprocal) recovers the
// transmittance in front of a blended Gaussian, and s, the upstream gradient's product with the
// colour that the later Gaussians and the background add, grows by alpha_i T_i (g . c_i):
//   dL/dalpha_i = T_i (g . c_i) - s / (1 - alpha_i),   p_i = dL/dpower_i = alpha_i dL/dalpha_i.
//
// Sums over pixels.  A row's nine gradients are linear in nine sums over the wave's pixels: p times
// (1, dx, dy, dx^2, dx dy, dy^2), d the pixel's offset from the Gaussian's centre, and alpha T times
// the three channels of g.  Both are formed for 8 rows at a time from a wave-private LDS buffer
// that turns a lane per pixel into a lane per (row, line of 8 pixels).  The six of p are summed from
// the offsets themselves, each lane its own line, then over the 8 lines by lane swaps.  (As a matrix
// product with the pixels' monomials, moments about a point that all rows share, they have to be
// shifted to each centre afterwards, which costs a splat of half a pixel at a tile's edge two to three
// digits.)  The three of alpha T are one FP32 matrix product, (8 rows x 2 halves of the quadrant) x 32
// pixels by 32 pixels x (3 channels x 2 halves): v_mfma_f32_16x16x4_f32, FP32 in, FP32 accumulate.
// The four waves of a tile add their sums in LDS and one thread per entry turns them into
// gradients and adds them with hardware FP32 atomics, once per (entry, tile).  Wave sums of every row
// by lane swaps and DPP took ~45 vector instructions per row and one nine-lane global atomic per
// (row, quadrant).
//
// What bounds it: vector issue (67 % of the SIMD cycles in FP32, 52 % in the MFMA variant) and LDS (61 and
// 63 %) together, and the waves of unequal lists that meet at the chunk barriers.  One buffer for p and then
// alpha T, instead of one each, brings the FP32 kernel from 38 to 29.5 KB: five workgroups per CU instead of
// four.  1M Gaussians at 1920x1080: FP32 438 -> 400 us, FP16 327 -> 324 us, with all sums as moments before.
#include "gs_backward.hpp"
#include "gs_mfma.hpp"

namespace gsi {
namespace {

typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int kRowBlock = 8;         // rows summed at a time
constexpr int kVStride = 68;         // floats per line of the transposing buffer: conflict-free 16-byte reads
constexpr int kTerms = 9;

// LDS of both kernels' sums.  acc: per staged entry, the six sums of p and the three colour
// sums; after the conversion, its nine gradients.
struct SumShared {
  __align__(16) float v[4][kRowBlock * kVStride];   // wave-private: the rows' p, then their alpha T
  float acc[kBlock * kTerms];
  uint32_t g[kBlock];                               // the entries' Gaussians
  __align__(4) uint8_t wl[4][kBlock];               // each wave's row list
  uint8_t qm[kBlock];
  uint32_t last;                                    // end of the longest blended prefix of the tile
};

// A value the compiler takes as new: what is computed from it stays where it is used, instead of
// being kept in registers across the row loops (the flush's indices alone took ~25).
__device__ __forceinline__ int fresh(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The line of 8 pixels of the wave's quadrant that this lane sums (of row lane % 8): lines 0..3 and
// 4..7 are the two halves of the colour product.
__device__ __forceinline__ int sum_line(int lane) { return 4 * ((lane >> 3) & 1) + (lane >> 4); }

// This lane's share of the pixel-side operand of the colour product: column n = lane % 16, pixels
// (j, lane / 16) of the half for j < 8.  Columns 0..2 are the channels of the upstream gradient in the
// upper half, 3..5 in the lower, the others zero.  A pixel whose upstream gradient is not finite has
// zeros there and adds its terms by itself, so that it reaches only the Gaussians it blends.
struct PixelSide {
  float b[8];
};

__device__ __forceinline__ PixelSide pixel_side(const BackwardJob &J, int ox, int oy) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int n = lane & 15;
  const int64_t HW = (int64_t)J.W * J.H;
  const int py = (w >> 1) * 8 + 4 * (n >= 3) + (lane >> 4);
  PixelSide s;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int px = (w & 1) * 8 + j;
    s.b[j] = 0.0f;
    if (n < 6 && ox + px < J.W && oy + py < J.H) {
      const int64_t pix = (int64_t)(oy + py) * J.W + (ox + px);
      const float g0 = J.dimage[pix], g1 = J.dimage[HW + pix], g2 = J.dimage[2 * HW + pix];
      const bool fin = fabsf(g0) < INFINITY && fabsf(g1) < INFINITY && fabsf(g2) < INFINITY;
      const int c = n % 3;
      s.b[j] = !fin ? 0.0f : c == 0 ? g0 : c == 1 ? g1 : g2;
    }
  }
  return s;
}

// One entry's nine sums to its gradients: rgb (3), opacity, conic (3), xy (2), in place.
__device__ __forceinline__ void convert_sums(float *a, const float4 co) {
  const float m0 = a[0], sx = a[1], sy = a[2], sxx = a[3], sxy = a[4], syy = a[5];
  const float r0 = a[6], r1 = a[7], r2 = a[8];
  // an entry that no pixel blended (its record may be anything) adds nothing
  const bool none = m0 == 0.0f && sx == 0.0f && sy == 0.0f && sxx == 0.0f && sxy == 0.0f && syy == 0.0f;
  a[0] = r0;
  a[1] = r1;
  a[2] = r2;
  a[3] = none ? 0.0f : m0 / co.w;
  a[4] = -0.5f * sxx;
  a[5] = -sxy;
  a[6] = -0.5f * syy;
  a[7] = none ? 0.0f : co.x * sx + co.y * sy;
  a[8] = none ? 0.0f : co.y * sx + co.z * sy;
}

// Adds the gradients of the staged entries [0, cnt) to the Gaussians', neighbouring lanes taking
// neighbouring addresses.  Entries that no pixel blended hold zeros and are left out.
__device__ __forceinline__ void flush_entries(const BackwardJob &J, const SumShared &sm, int cnt) {
  const int t = fresh(threadIdx.x);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int i = t + q * kBlock;
    if (i < 3 * cnt) {
      const int e = i / 3, f = i - 3 * e;
      const size_t g = sm.g[e];
      const float a = sm.acc[e * kTerms + f], b = sm.acc[e * kTerms + 4 + f];
      if (a != 0.0f) unsafeAtomicAdd(J.g_rgb + 3 * g + f, a);
      if (b != 0.0f) unsafeAtomicAdd(J.g_conic + 3 * g + f, b);
    }
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int i = t + q * kBlock;
    if (i < 2 * cnt) {
      const float a = sm.acc[(i >> 1) * kTerms + 7 + (i & 1)];
      if (a != 0.0f) unsafeAtomicAdd(J.g_xy + 2 * (size_t)sm.g[i >> 1] + (i & 1), a);
    }
  }
  if (t < cnt) {
    const float a = sm.acc[t * kTerms + 3];
    if (a != 0.0f) unsafeAtomicAdd(J.g_op + sm.g[t], a);
  }
}

// This lane's pixel in the back-to-front walk.
struct PixelBack {
  float T;             // transmittance behind the row reached
  float s;             // g . (colour the rows behind it and the background add)
  float g0, g1, g2;    // upstream gradient
  bool bad;            // it is not finite
};

__device__ __forceinline__ PixelBack pixel_back(const BackwardJob &J, int ox, int oy, int px, int py, bool inside,
                                                float T) {
  const int64_t HW = (int64_t)J.W * J.H;
  const int64_t pix = (int64_t)(oy + py) * J.W + (ox + px);
  PixelBack b;
  b.T = T;
  b.g0 = inside ? J.dimage[pix] : 0.0f;
  b.g1 = inside ? J.dimage[HW + pix] : 0.0f;
  b.g2 = inside ? J.dimage[2 * HW + pix] : 0.0f;
  b.bad = !(fabsf(b.g0) < INFINITY && fabsf(b.g1) < INFINITY && fabsf(b.g2) < INFINITY);
  b.s = b.g0 * (J.bg[0] * T) + b.g1 * (J.bg[1] * T) + b.g2 * (J.bg[2] * T);
  return b;
}

// One blended pair: steps the pixel in front of the row; *wgt = alpha T, *p = dL/dpower.
__device__ __forceinline__ void back_step(PixelBack &b, float D, float cr, float cg, float cb, float *wgt, float *p) {
  const float raw = __builtin_amdgcn_exp2f(D);
  const float al = fminf(kAlphaMax, raw);
  const float inv = __builtin_amdgcn_rcpf(1.0f - al);   // 1 - alpha >= 0.01
  const float Ti = b.T * inv;
  const float gc = fmaf(b.g0, cr, fmaf(b.g1, cg, b.g2 * cb));
  *wgt = al * Ti;
  const float dLda = fmaf(Ti, gc, -(b.s * inv));
  *p = raw < kAlphaMax ? dLda * al : 0.0f;
  b.s = fmaf(*wgt, gc, b.s);
  b.T = Ti;
}

// largest value of the wave (uniform)
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, 64));
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// The colour gradients of one (Gaussian, pixel) pair, added by this lane alone: pairs kept out of
// the matrix product because their upstream gradient is not finite.
__device__ __forceinline__ void direct_colour_terms(const BackwardJob &J, uint32_t gi, float wgt, float g0, float g1,
                                                    float g2) {
  const size_t g = gi;
  unsafeAtomicAdd(J.g_rgb + 3 * g, g0 * wgt);
  unsafeAtomicAdd(J.g_rgb + 3 * g + 1, g1 * wgt);
  unsafeAtomicAdd(J.g_rgb + 3 * g + 2, g2 * wgt);
}

// Reduce-scatter steps of two registers at once.  swap32_add: lanes 0..31 get a[i] + a[i+32],
// lanes 32..63 get b[i-32] + b[i].  swap16_add (rows of 16 lanes): row 0 gets a's rows 0 + 1,
// row 1 b's rows 0 + 1, row 2 a's rows 2 + 3, row 3 b's rows 2 + 3.
__device__ __forceinline__ float swap32_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_add(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// v plus the lane eight further in its row of 16
__device__ __forceinline__ float ror8_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false));
}

// Adds to acc the nine sums over the wave's pixels of 8 rows.  This lane's row (lane % 8) is staged
// entry `e` (none, its p and alpha T zero, unless `valid`) with its centre at (u, v); (X0, Y0): the
// quadrant's first pixel centre in the same frame.  Lines 0..7 of vbuf hold the rows' p and wgt[m] row
// m's alpha T, one value per lane, zero where a pixel did not blend the row.  special (uniform):
// some lane's upstream gradient is not finite; the colours of its pairs are kept out of the product
// (0 x inf) and added singly.
__device__ __forceinline__ void add_row_sums(const BackwardJob &J, float *vbuf, const PixelSide &s, SumShared &sm,
                                             int e, bool valid, float u, float v, float X0, float Y0,
                                             const float (&wgt)[kRowBlock], const PixelBack &pb, bool special) {
  const int lane = threadIdx.x & 63, line = sum_line(lane);
  float *mine = vbuf + (lane & (kRowBlock - 1)) * kVStride + 8 * line;
  const float4v *rp = reinterpret_cast<const float4v *>(mine);
  wave_fence();
  const float4v p0 = rp[0], p1 = rp[1];
  wave_fence();
#pragma unroll
  for (int m = 0; m < kRowBlock; ++m) vbuf[m * kVStride + lane] = wgt[m];
  wave_fence();
  const float4v w0 = rp[0], w1 = rp[1];
  // p (1, dx, dx^2) over the line, then dy, which it shares
  float m0 = 0.0f, mx = 0.0f, mxx = 0.0f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float p = j < 4 ? p0[j & 3] : p1[j & 3], dx = (X0 + (float)j) - u, pdx = p * dx;
    m0 += p;
    mx += pdx;
    mxx = fmaf(pdx, dx, mxx);
  }
  const float dy = (Y0 + (float)line) - v;
  const float my = m0 * dy, mxy = mx * dy, myy = my * dy;
  // over the lines: lane bits 5, 4 and 3
  const float z0 = ror8_add(swap16_add(swap32_add(m0, mx), swap32_add(my, mxx)));
  const float x2 = swap32_add(mxy, myy);
  const float z1 = ror8_add(swap16_add(x2, x2));
  // rows of 16 lanes: z0 holds sums 0, 2, 1, 3, z1 holds 4, 4, 5, 5
  const int row = lane >> 4;
  const bool second = (lane & 8) != 0;
  const int f = second ? 4 + (row >> 1) : row == 1 ? 2 : row == 2 ? 1 : row;
  if (valid && !(second && (row & 1))) unsafeAtomicAdd(&sm.acc[e * kTerms + f], second ? z1 : z0);
  float4v d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < 8; ++j)
    d = __builtin_amdgcn_mfma_f32_16x16x4f32(j < 4 ? w0[j & 3] : w1[j & 3], s.b[j], d, 0, 0, 0);
  // lane l holds column l % 16 of lines 4 (l / 16) + i: row 4 (l / 16 % 2) + i, half l / 32
  const int col = (lane & 15) - 3 * (lane >> 5);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * (row & 1) + i;   // (lane r's row)
    const int er = __shfl(valid ? e : -1, r, 64);
    if (col >= 0 && col < 3 && er >= 0) unsafeAtomicAdd(&sm.acc[er * kTerms + 6 + col], d[i]);
  }
  if (__builtin_expect(special, 0)) {
#pragma unroll 1
    for (int m = 0; m < kRowBlock; ++m) {
      const float wm = vbuf[m * kVStride + lane];
      const int em = __shfl(e, m, 64);
      if (pb.bad && wm != 0.0f) direct_colour_terms(J, sm.g[em], wm, pb.g0, pb.g1, pb.g2);
    }
  }
  wave_fence();   // the buffer is free for the next rows
}

// ---- backward of the FP32 forward ---------------------------------------------------------
// Two passes over the list: the forward recurrence again, in the forward rasterizer's FP32
// arithmetic (so every cut, clamp and stop is decided the same way), for the pixel's final
// transmittance and the end of its blended prefix, then the walk back.  The rows of a chunk
// stay in LDS between the passes where the walk back starts in the chunk staged last.
struct BwdShared {
  float4 a[kBlock + 1];   // (u, v, -a/2 log2e, -b log2e): centre relative to the tile; row kBlock never blends
  float4 b[kBlock + 1];   // (-c/2 log2e, log2 o, r, g)
  float c[kBlock + 1];    // b
  uint32_t alive[2][4];
  SumShared s;
};

__global__ __launch_bounds__(kBlock, 4) void k_raster_backward(BackwardJob J, int all_rows) {
  __shared__ BwdShared sm;
  const int tile = xcd_raster_bin((int)blockIdx.x, J.TX, J.TY);
  if (tile < 0) return;
  const int ox = (tile % J.TX) * kTile, oy = (tile / J.TX) * kTile;
  const uint32_t start = J.ranges[2 * tile], end = J.ranges[2 * tile + 1];
  if (start >= end) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int px = (w & 1) * 8 + (lane & 7), py = (w >> 1) * 8 + (lane >> 3);
  const float X = px + 0.5f, Y = py + 0.5f;
  const bool inside = (ox + px < J.W) && (oy + py < J.H);

  float4 eco = make_float4(0.0f, 0.0f, 0.0f, 1.0f);        // this thread's staged entry
  auto stage = [&](uint32_t cs, int cnt) {
    if (t < cnt) {
      const uint32_t g = J.vals[cs + t];
      const double2 m = J.xy[g];
      const float4 co = J.conic[g];
      const float4 cl = J.rgb[g];
      sm.a[t] = make_float4((float)(m.x - ox), (float)(m.y - oy), -0.5f * kLog2e * co.x, -kLog2e * co.y);
      sm.b[t] = make_float4(-0.5f * kLog2e * co.z, __log2f(co.w), cl.x, cl.y);
      sm.c[t] = cl.z;
      sm.s.g[t] = g;
      eco = co;
      sm.s.qm[t] = all_rows ? (uint8_t)0xF
                            : (uint8_t)mfma::quad_mask_fp32((float)(m.x - ((double)ox + 8.5)),
                                                            (float)(m.y - ((double)oy + 8.5)), co.x, co.y, co.z,
                                                            mfma::log2_opacity(co.w));
    }
  };

  // pass 1: the forward recurrence.  stop: list position of the row that stops this pixel;
  // wave_last (uniform): end of the longest blended prefix of the wave's pixels.
  float T = 1.0f;
  float cut = inside ? kCutLog2 : INFINITY;
  uint32_t stop = inside ? ~0u : start, wave_last = start;
  if (t == 0) {
    sm.s.last = start;
    sm.a[kBlock] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    sm.b[kBlock] = make_float4(0.0f, -INFINITY, 0.0f, 0.0f);
    sm.c[kBlock] = 0.0f;
  }
  uint32_t staged = start;   // first entry of the chunk in LDS
  int it = 0;
  for (uint32_t cs = start; cs < end; cs += kBlock) {
    const int cnt = (int)min((uint32_t)kBlock, end - cs);
    if (it > 0) {
      block_sync();
      const uint32_t *al = sm.alive[(it - 1) & 1];
      if (!(al[0] | al[1] | al[2] | al[3])) break;
    }
    stage(cs, cnt);
    staged = cs;
    block_sync();
    const int n = mfma::wave_list(sm.s.qm, cnt, sm.s.wl[w]);
    for (int r0 = 0; r0 < n; r0 += 64) {
      if (__ballot(cut != INFINITY) == 0) break;
      const int idx = r0 + lane < n ? (int)sm.s.wl[w][r0 + lane] : kBlock;
      const int mm = min(64, n - r0);
      for (int k = 0; k < mm; k += 4) {
        float D[4];
        int ri[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          ri[j] = __builtin_amdgcn_readlane(idx, k + j);
          const float4 A = sm.a[ri[j]];
          const float2 B = *reinterpret_cast<const float2 *>(&sm.b[ri[j]]);
          const float dx = X - A.x, dy = Y - A.y;
          D[j] = fmaf(dx, fmaf(A.z, dx, A.w * dy), fmaf(B.x * dy, dy, B.y));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (D[j] >= cut) {
            // T' = T (1 - alpha); a stop (T' < 1e-4) keeps T and disables the pixel, once per
            // pixel, so its selects run only when a lane stops on this row
            const float al = fminf(kAlphaMax, __builtin_amdgcn_exp2f(D[j]));
            const float Tn = fmaf(-T, al, T);
            wave_last = cs + (uint32_t)ri[j] + 1u;
            if (__builtin_expect(__ballot(!(Tn >= kTMin)) != 0, 0)) {
              const bool ok = Tn >= kTMin;
              T = ok ? Tn : T;
              stop = ok ? stop : cs + (uint32_t)ri[j];
              cut = ok ? cut : INFINITY;
            } else {
              T = Tn;
            }
          }
        }
      }
    }
    const uint64_t bal = __ballot(cut != INFINITY);
    if (lane == 0) sm.alive[it & 1][w] = bal != 0;
    ++it;
  }
  wave_last = wave_max(wave_last);
  block_sync();
  if (lane == 0) atomicMax(&sm.s.last, wave_last);
  block_sync();
  const uint32_t tile_last = sm.s.last;
  if (tile_last == start) return;

  // pass 2: back to front
  PixelBack pb = pixel_back(J, ox, oy, px, py, inside, T);
  const PixelSide side = pixel_side(J, ox, oy);
  const bool special = __ballot(pb.bad) != 0;
  float *vbuf = sm.s.v[w];
  for (uint32_t cs = start + (tile_last - 1 - start) / kBlock * kBlock;; cs -= kBlock) {
    const int cnt = (int)min((uint32_t)kBlock, end - cs);
    if (cs != staged) {
      block_sync();
      stage(cs, cnt);
    }
#pragma unroll
    for (int f = 0; f < kTerms; ++f) sm.s.acc[t * kTerms + f] = 0.0f;
    block_sync();
    const int rows = (int)min((uint32_t)cnt, wave_last > cs ? wave_last - cs : 0u);
    const int lim = stop > cs ? (int)min(stop - cs, (uint32_t)kBlock) : 0;   // this pixel's rows [0, lim)
    const int n = mfma::wave_list(sm.s.qm, rows, sm.s.wl[w]);
    for (int r0 = ((n + kRowBlock - 1) / kRowBlock - 1) * kRowBlock; r0 >= 0; r0 -= kRowBlock) {
      const int sl = r0 + (lane & (kRowBlock - 1));
      const int idx = sl < n ? (int)sm.s.wl[w][sl] : kBlock;
      bool any = false;
      float wgt[kRowBlock];
#pragma unroll
      for (int k = kRowBlock - 4; k >= 0; k -= 4) {
        float D[4], cr[4], cg[4], cb[4];
        int ri[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          ri[j] = __builtin_amdgcn_readlane(idx, k + j);
          const float4 A = sm.a[ri[j]], B = sm.b[ri[j]];
          cr[j] = B.z;
          cg[j] = B.w;
          cb[j] = sm.c[ri[j]];
          const float dx = X - A.x, dy = Y - A.y;
          D[j] = fmaf(dx, fmaf(A.z, dx, A.w * dy), fmaf(B.x * dy, dy, B.y));
        }
#pragma unroll
        for (int j = 3; j >= 0; --j) {
          float p = 0.0f;
          wgt[k + j] = 0.0f;
          const bool act = ri[j] < lim && D[j] >= kCutLog2;
          any |= act;
          if (act) back_step(pb, D[j], cr[j], cg[j], cb[j], &wgt[k + j], &p);
          vbuf[(k + j) * kVStride + lane] = p;
        }
      }
      if (__ballot(any) != 0) {
        const float2 c = *reinterpret_cast<const float2 *>(&sm.a[idx]);
        add_row_sums(J, vbuf, side, sm.s, idx, sl < n, c.x, c.y, (w & 1) * 8 + 0.5f, (w >> 1) * 8 + 0.5f, wgt, pb,
                     special);
      }
    }
    block_sync();
    if (t < cnt) convert_sums(sm.s.acc + t * kTerms, eco);
    block_sync();
    flush_entries(J, sm.s, cnt);
    if (cs == start) break;
    staged = ~0u;
    block_sync();
  }
}

// ---- backward of the MFMA forward ------------------------------------------------------
// The power of each (Gaussian, pixel) pair comes from the forward's own MFMA contraction (the
// Gaussian-side row and the pixel-side operand built by the same functions, so D =
// log2(alpha_raw) is bit-identical to the forward's and every cut, clamp and stop is decided the
// same way), and the forward's final transmittance and blended-prefix end (GS_AUX_TFINAL,
// GS_AUX_LAST) replace the replay pass.  Each wave takes its rows as 32-row MFMA blocks; after
// the lane swap a lane holds the 32 rows' D for its pixel and walks them back to front.  A row is
// active for a pixel when it lies before the pixel's blended-prefix end and D reaches the cut
// (the forward blended exactly those).
template <int S>
struct BwdMfmaShared {
  static constexpr int RS = (S == 3) ? 32 : 16;
  __align__(16) uint16_t A[kBlock * RS];   // Gaussian-side rows
  float col[3][kBlock];                    // r, g, b
  float2 uv[kBlock];                       // centre in the tile frame
  SumShared s;
};

template <int PREC, int S>
__global__ __launch_bounds__(kBlock, S == 3 ? 3 : 4) void k_raster_backward_mfma(BackwardJob J, int all_rows) {
  using N = mfma::Narrow<PREC>;
  constexpr int RS = BwdMfmaShared<S>::RS;
  __shared__ BwdMfmaShared<S> sm;
  const int tile = xcd_raster_bin((int)blockIdx.x, J.TX, J.TY);
  if (tile < 0) return;
  const int ox = (tile % J.TX) * kTile, oy = (tile / J.TX) * kTile;
  const uint32_t start = J.ranges[2 * tile], len = J.ranges[2 * tile + 1] - start;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int px = (w & 1) * 8 + (lane & 7), py = (w >> 1) * 8 + (lane >> 3);
  const bool inside = (ox + px < J.W) && (oy + py < J.H);
  const int64_t pix = (int64_t)(oy + py) * J.W + (ox + px);
  const float T = inside ? J.t_final[pix] : 1.0f;
  // (a blended-prefix end beyond the tile's list cannot come from the forward; clamped so that no
  // entry outside the tile is read)
  const uint32_t last = inside ? min((uint32_t)J.last[pix], len) : 0u;
  const uint32_t wave_last = wave_max(last);
  if (t == 0) sm.s.last = 0;
  block_sync();
  if (lane == 0) atomicMax(&sm.s.last, wave_last);
  block_sync();
  const uint32_t tile_last = sm.s.last;
  if (tile_last == 0) return;

  mfma::short8 B0, B1, B20, B21;
  mfma::make_pixel_operand<PREC>(B0, B1, B20, B21);
  PixelBack pb = pixel_back(J, ox, oy, px, py, inside, T);
  const PixelSide side = pixel_side(J, ox, oy);
  const bool special = __ballot(pb.bad) != 0;
  float *vbuf = sm.s.v[w];
  mfma::short8 pad = {}, zero = {};
  if (lane < 32) pad[5] = (short)N::enc(-1000.0f);

  for (uint32_t ce = tile_last; ce > 0;) {
    const int cnt = (int)min((uint32_t)kBlock, ce);
    const uint32_t cs = ce - (uint32_t)cnt;   // positions in the tile's list
    float4 eco = make_float4(0.0f, 0.0f, 0.0f, 1.0f);
    block_sync();
    if (t < cnt) {
      const uint32_t g = J.vals[start + cs + t];
      const double2 m = J.xy[g];
      const float4 co = J.conic[g];
      const float u = (float)(m.x - ((double)ox + 8.5)), v = (float)(m.y - ((double)oy + 8.5));
      const float l2o = mfma::log2_opacity(co.w);
      mfma::build_row<PREC, S>(&sm.A[t * RS], u, v, co.x, co.y, co.z, l2o);
      const float4 cl = J.rgb[g];
      sm.col[0][t] = cl.x;
      sm.col[1][t] = cl.y;
      sm.col[2][t] = cl.z;
      sm.s.g[t] = g;
      sm.s.qm[t] = all_rows ? (uint8_t)0xF : (uint8_t)mfma::quad_mask(u, v, co.x, co.y, co.z, l2o);
      sm.uv[t] = make_float2(u, v);
      eco = co;
    }
#pragma unroll
    for (int f = 0; f < kTerms; ++f) sm.s.acc[t * kTerms + f] = 0.0f;
    block_sync();
    const int rows = (int)min((uint32_t)cnt, wave_last > cs ? wave_last - cs : 0u);
    const int lim = last > cs ? (int)min(last - cs, (uint32_t)kBlock) : 0;   // this pixel's rows [0, lim)
    const int n = mfma::wave_list(sm.s.qm, rows, sm.s.wl[w]);
    for (int blk = ((n + 31) >> 5) - 1; blk >= 0; --blk) {
      const int slot = 32 * blk + (lane & 31);
      const bool real = slot < n;
      const int rr = real ? (int)sm.s.wl[w][slot] : 0;
      const uint16_t *rp = sm.A + (size_t)rr * RS + 8 * (lane >> 5);
      const mfma::short8 a = real ? *reinterpret_cast<const mfma::short8 *>(rp) : pad;
      mfma::float16v z = {};
      mfma::float16v d0 = N::mma(a, B0, z);
      mfma::float16v d1 = N::mma(a, B1, z);
      if (S == 3) {
        const mfma::short8 a2 = real ? *reinterpret_cast<const mfma::short8 *>(rp + 16) : zero;
        d0 = N::mma(a2, B20, d0);
        d1 = N::mma(a2, B21, d1);
      }
      // the last rows first: registers 4 r .. 4 r + 3 of the two accumulators hold rows 8 r .. 8 r + 7
#pragma unroll
      for (int r = 3; r >= 0; --r) {
        const int first = 32 * blk + kRowBlock * r;
        if (first >= n) continue;   // (uniform)
        float D[kRowBlock];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          auto pr = __builtin_amdgcn_permlane32_swap(__float_as_uint(d0[4 * r + j]), __float_as_uint(d1[4 * r + j]),
                                                     false, false);
          D[j] = __uint_as_float(pr[0]);
          D[4 + j] = __uint_as_float(pr[1]);
        }
        bool any = false;
        float wgt[kRowBlock];
#pragma unroll
        for (int m = kRowBlock - 1; m >= 0; --m) {
          const int ri = __builtin_amdgcn_readlane(rr, kRowBlock * r + m);   // (a slot past n: D = -1000)
          float p = 0.0f;
          wgt[m] = 0.0f;
          const bool act = ri < lim && D[m] >= kCutLog2;
          any |= act;
          if (act) back_step(pb, D[m], sm.col[0][ri], sm.col[1][ri], sm.col[2][ri], &wgt[m], &p);
          vbuf[m * kVStride + lane] = p;
        }
        if (__ballot(any) != 0) {
          const int e = __shfl(rr, kRowBlock * r + (lane & (kRowBlock - 1)), 64);
          const float2 c = sm.uv[e];
          add_row_sums(J, vbuf, side, sm.s, e, first + (lane & (kRowBlock - 1)) < n, c.x, c.y, (w & 1) * 8 - 8.0f,
                       (w >> 1) * 8 - 8.0f, wgt, pb, special);
        }
      }
    }
    block_sync();
    if (t < cnt) convert_sums(sm.s.acc + t * kTerms, eco);
    block_sync();
    flush_entries(J, sm.s, cnt);
    ce = cs;
  }
}

template <int PREC>
hipError_t launch_bwd_mfma_p(const BackwardJob &j, int splits, int all_rows, hipStream_t st) {
  switch (splits) {
    case 1: hipLaunchKernelGGL((k_raster_backward_mfma<PREC, 1>), dim3(xcd_raster_grid(j.TX, j.TY)), dim3(kBlock), 0, st, j, all_rows); break;
    case 2: hipLaunchKernelGGL((k_raster_backward_mfma<PREC, 2>), dim3(xcd_raster_grid(j.TX, j.TY)), dim3(kBlock), 0, st, j, all_rows); break;
    case 3:
      if (PREC == GS_PREC_FP16_MFMA) return hipErrorInvalidValue;
      hipLaunchKernelGGL((k_raster_backward_mfma<PREC, 3>), dim3(xcd_raster_grid(j.TX, j.TY)), dim3(kBlock), 0, st, j, all_rows);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_raster_backward_mfma(const BackwardJob &j, int prec, int splits, bool all_rows, hipStream_t st) {
  const int tiles = j.TX * j.TY;
  if (tiles == 0) return hipSuccess;
  if (prec == GS_PREC_FP16_MFMA) return launch_bwd_mfma_p<GS_PREC_FP16_MFMA>(j, splits, all_rows ? 1 : 0, st);
  if (prec == GS_PREC_BF16_MFMA) return launch_bwd_mfma_p<GS_PREC_BF16_MFMA>(j, splits, all_rows ? 1 : 0, st);
  return hipErrorInvalidValue;
}

hipError_t launch_raster_backward(const BackwardJob &j, bool all_rows, hipStream_t st) {
  const int tiles = j.TX * j.TY;
  if (tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(k_raster_backward, dim3(xcd_raster_grid(j.TX, j.TY)), dim3(kBlock), 0, st, j, all_rows ? 1 : 0);
  return hipGetLastError();
}

}  // namespace gsi
