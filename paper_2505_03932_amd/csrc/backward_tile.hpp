// Backward pass of the FP32 reprojection (not in the paper: it turns the
// reprojection into a differentiable step so WCS alignment can be refined
// by gradient descent on image residuals).
//
// For a loss L with g = dL/dout:
//   dL/dsrc_k = sum_p g_p w_kp / F_p       -- adjoint of the interpolation, a
//                                            scatter-add of contributions
//                                            rounded to a fixed grid and
//                                            summed exactly in 64-bit
//                                            integers (in an LDS copy of the
//                                            tile's source box, then one
//                                            global atomic per touched source
//                                            pixel), so the result does not
//                                            depend on the order of the adds;
//   dL/dpos_p  = g_p (dS/dpos - out dF/dpos) / F
// and through the map pos = (U, V) + SIP(U, V) + CRPIX - 1 with
// (U, V) = (p/w, q/w), (p, q, w) = H t:
//   dL/dH_1j = sum a t_j / w,  dL/dH_2j = sum b t_j / w,
//   dL/dH_3j = -sum (a U + b V) t_j / w,
// a = dL/dU, b = dL/dV; plus dL/dCRPIX and the AP/BP monomial sums.  These
// are reduced per wave, then per work-group into FP64 partials, then in a
// fixed order (deterministic), and chained to CRVAL and CD on the device
// with the FP64 Jacobian dH/d(CRVAL, CD) composed on the host.
#pragma once

#include "forward_body.hpp"
#include "launch.hpp"

namespace dfr {

// Up to kRun consecutive values (n of them, the others 0): one 16-byte load
// at any alignment where all are there.
__device__ __forceinline__ void load_run(const float *__restrict__ p, int n, float v[kRun]) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
  if (n >= kRun) {
    const f4u q = *reinterpret_cast<const f4u *>(p);
    v[0] = q.x;
    v[1] = q.y;
    v[2] = q.z;
    v[3] = q.w;
  } else {
#pragma unroll
    for (int e = 0; e < kRun; ++e) v[e] = e < n ? p[e] : 0.0f;
  }
}

// ---- tile set-up of the backward kernel (anchors, exact tap box, staging)

// LDS scratch of a tile kernel besides the dynamic source tile.
struct TileShared {
  Anchor anchor[kMaxAnchors];
  int box[4];     // imin, imax, jmin, jmax of the source box
  int touch;      // any anchor cell can reach the source
  int bounded;    // the box bounds every tap (from the anchors), all positions valid
};

// Geometry of a tile and of the calling thread inside it.
struct TileCtx {
  int x0, y0;    // tile origin (output pixels)
  int RP;        // rows per pass
  int cx0, cy0;  // first anchor cell
  int ncx;       // anchor cells per tile row
  int ty;        // thread row in the tile
  int xr;        // first output column of the thread's runs
};

// A backward tile works from its cells' FP64 anchors (the WCS gradient
// needs the projective intermediates of every pixel).  Where the anchors bound
// every pixel's taps (no target SIP, the projective denominator certainly
// positive), that bound is the tile's source box, and its copy into LDS is
// under way while the positions are computed; elsewhere the positions come
// first and give the exact box of the in-image taps.
//
// Phase 1.  Returns false when no pixel of the tile can reach the source
// (and skipping is allowed): the caller then only writes "uncovered".
template <int INTERP, int SORD, bool TSIP, int NP>
__device__ __forceinline__ bool tile_anchors(const FramePlan &P, const TileGeom &G, int tile,
                                             const Anchor *__restrict__ anchors, TileShared &sh,
                                             TileCtx &c) {
  const int tid = threadIdx.x;
  const int lg = G.txt_log2;
  const int TW = kRun << lg;
  c.RP = kThreads >> lg;
  const int TH = c.RP * NP;
  const int trow = tile / G.tiles_x;
  c.x0 = (tile - trow * G.tiles_x) * TW;
  c.y0 = trow * TH;
  c.cx0 = c.x0 / kCell;
  c.ncx = TW / kCell;
  c.cy0 = c.y0 / kCell;
  const int ncy = TH >= kCell ? TH / kCell : 1;
  const int nA = c.ncx * ncy;
  c.ty = tid >> lg;
  c.xr = c.x0 + (tid & ((1 << lg) - 1)) * kRun;
  if (tid < 64) {
    int t = 0;
    bool bounded = !TSIP;
    int imn = 0x3fffffff, imx = -0x3fffffff, jmn = 0x3fffffff, jmx = -0x3fffffff;
    if (tid < nA) {
      const int cy = c.cy0 + tid / c.ncx, cx = c.cx0 + tid % c.ncx;
      Anchor &A = sh.anchor[tid];
      if (anchors && cx * kCell < G.out_w && cy * kCell < G.out_h) {
        typedef unsigned u4v __attribute__((ext_vector_type(4)));
        const u4v *from = reinterpret_cast<const u4v *>(
            anchors + (int64_t)cy * ((G.out_w + kCell - 1) >> kCellLog2) + cx);
#pragma unroll
        for (int part = 0; part < (int)(sizeof(Anchor) / 16); ++part)
          reinterpret_cast<u4v *>(&A)[part] = from[part];
      } else if (anchors) {
        A = Anchor{};  // a cell outside the output: no pixel of it is computed
      } else {
        compute_anchor<SORD, TSIP>(P, cx * kCell, cy * kCell, TapSupport<INTERP>::hi, A);
      }
      t = A.touch;
      if constexpr (!TSIP) {
        // the part of the cell inside the tile and the output, as offsets from
        // the anchor; the extremes of the linear model there, grown by the
        // anchor's bound on the model's error
        const int xa = cx * kCell, ya = cy * kCell;
        const int xe = min(xa + kCell, min(c.x0 + TW, G.out_w)), ys = max(ya, c.y0);
        const int ye = min(ya + kCell, min(c.y0 + TH, G.out_h));
        if (xe > xa && ye > ys) {
          const float ux = (float)(xe - 1 - xa), v0 = (float)(ys - ya), v1 = (float)(ye - 1 - ya);
          const float xl =
              A.sx0 + fminf(0.0f, A.jx[0] * ux) + fminf(A.jx[1] * v0, A.jx[1] * v1) - A.ex;
          const float xh =
              A.sx0 + fmaxf(0.0f, A.jx[0] * ux) + fmaxf(A.jx[1] * v0, A.jx[1] * v1) + A.ex;
          const float yl =
              A.sy0 + fminf(0.0f, A.jy[0] * ux) + fminf(A.jy[1] * v0, A.jy[1] * v1) - A.ey;
          const float yh =
              A.sy0 + fmaxf(0.0f, A.jy[0] * ux) + fmaxf(A.jy[1] * v0, A.jy[1] * v1) + A.ey;
          bounded = A.ok && fabsf(xl) < 1.0e7f && fabsf(xh) < 1.0e7f && fabsf(yl) < 1.0e7f &&
                    fabsf(yh) < 1.0e7f;
          if (bounded) {
            constexpr int lo = TapSupport<INTERP>::lo + 2, hi = TapSupport<INTERP>::hi + 2;
            imn = A.bx + (int)floorf(xl) - lo;
            imx = A.bx + (int)floorf(xh) + hi;
            jmn = A.by + (int)floorf(yl) - lo;
            jmx = A.by + (int)floorf(yh) + hi;
          }
        }
      }
    }
#pragma unroll
    for (int m = kMaxAnchors / 2; m >= 1; m >>= 1) {
      imn = min(imn, __shfl_xor(imn, m, 64));
      imx = max(imx, __shfl_xor(imx, m, 64));
      jmn = min(jmn, __shfl_xor(jmn, m, 64));
      jmx = max(jmx, __shfl_xor(jmx, m, 64));
    }
    const unsigned long long any = __ballot(t != 0), loose = __ballot(tid < nA && !bounded);
    if (tid == 0) {
      const bool b = loose == 0ull;
      sh.touch = any != 0ull;
      sh.bounded = b;
      sh.box[0] = b ? imn : 0x7fffffff;
      sh.box[1] = b ? imx : -0x7fffffff;
      sh.box[2] = b ? jmn : 0x7fffffff;
      sh.box[3] = b ? jmx : -0x7fffffff;
    }
  }
  __syncthreads();
  return sh.touch || !G.allow_skip;
}

template <int NP>
struct TilePos {
  float rx[NP][kRun], ry[NP][kRun];
  int abx[NP], aby[NP];  // anchor base of each run
  int aidx[NP];          // anchor index of each run
  unsigned valid;        // bit k*kRun+e: pixel (run k, element e) has a position
  int bi0, bi1, bj0, bj1;
  bool empty;            // no pixel of the tile has a tap inside the source
};

// Phase 2: every pixel's position; without a bound from the anchors also the
// exact box of the in-image taps (then it ends with a barrier).
template <int INTERP, int SORD, bool TSIP, int NP>
__device__ __forceinline__ void anchor_positions(const FramePlan &P, const TileGeom &G,
                                               TileShared &sh, const TileCtx &c,
                                               TilePos<NP> &T) {
  constexpr int SLO = TapSupport<INTERP>::lo, SHI = TapSupport<INTERP>::hi;
  const int W = P.src_w, Hs = P.src_h;
  const float tinv = (float)P.t_inv_scale, sinv = (float)P.s_inv_scale;
  int imin = 0x7fffffff, imax = -0x7fffffff, jmin = 0x7fffffff, jmax = -0x7fffffff;
  const bool bounded = sh.bounded;
  T.valid = 0u;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int y = c.y0 + c.ty + k * c.RP;
    const int a = ((y >> kCellLog2) - c.cy0) * c.ncx + ((c.xr >> kCellLog2) - c.cx0);
    const Anchor &A = sh.anchor[a];
    T.aidx[k] = a;
    T.abx[k] = A.bx;
    T.aby[k] = A.by;
    const float dy = (float)(y & (kCell - 1));
#pragma unroll
    for (int e = 0; e < kRun; ++e) {
      const int x = c.xr + e;
      const float dx = (float)((c.xr & (kCell - 1)) + e);
      float px, py;
      bool ok = pixel_position<SORD, TSIP>(P, A, tinv, sinv, dx, dy, px, py);
      ok = ok && (y < G.out_h) && (x < G.out_w);
      double dbx = 0.0, dby = 0.0;
      bool exact = false;
      if constexpr (INTERP == DFR_NEAREST) {
        // a rounding decision within reach of the FP32 error: decide in FP64
        float tx_ = px - floorf(px), ty_ = py - floorf(py);
        if (ok && (fabsf(tx_ - 0.5f) < 1e-4f || fabsf(ty_ - 0.5f) < 1e-4f)) {
          double xs, ys;
          ok = position_f64_ct<SORD, TSIP>(P, (double)x, (double)y, xs, ys) && fabs(xs - A.bx) < 1.0e7 &&
               fabs(ys - A.by) < 1.0e7;
          if (ok) {
            px = (float)(rint(xs) - (double)A.bx);
            py = (float)(rint(ys) - (double)A.by);
            exact = true;
            dbx = xs;
            dby = ys;
          }
        }
      }
      T.rx[k][e] = px;
      T.ry[k][e] = py;
      if (G.debug && y < G.out_h && x < G.out_w) {
        double2 d;
        if (!ok) {
          d.x = __builtin_nan("");
          d.y = d.x;
        } else if (exact) {
          d.x = dbx;
          d.y = dby;
        } else {
          d.x = (double)A.bx + (double)px;
          d.y = (double)A.by + (double)py;
        }
        reinterpret_cast<double2 *>(G.debug)[(int64_t)y * G.out_w + x] = d;
      }
      if (ok) T.valid |= 1u << (k * kRun + e);
      if (ok && !bounded) {
        int ic, jc;
        if constexpr (INTERP == DFR_NEAREST) {
          ic = A.bx + (int)rintf(px);
          jc = A.by + (int)rintf(py);
        } else {
          ic = A.bx + (int)floorf(px);
          jc = A.by + (int)floorf(py);
        }
        int ilo = ic - SLO, ihi = ic + SHI, jlo = jc - SLO, jhi = jc + SHI;
        if (ihi >= 0 && ilo < W && jhi >= 0 && jlo < Hs) {
          imin = min(imin, max(ilo, 0));
          imax = max(imax, min(ihi, W - 1));
          jmin = min(jmin, max(jlo, 0));
          jmax = max(jmax, min(jhi, Hs - 1));
        }
      }
    }
  }
  if (bounded) return;
  imin = wave_min(imin);
  imax = wave_max(imax);
  jmin = wave_min(jmin);
  jmax = wave_max(jmax);
  if ((threadIdx.x & 63) == 0 && imin <= imax) {
    atomicMin(&sh.box[0], imin);
    atomicMax(&sh.box[1], imax);
    atomicMin(&sh.box[2], jmin);
    atomicMax(&sh.box[3], jmax);
  }
  __syncthreads();
}

// ---- per-pixel adjoint

// The taps of a pixel all of whose taps are inside the source, from a staged
// box through `flat` (value(idx) and add_scaled(idx, v) at base + l * pitch +
// k): no per-tap test, one address per row.
template <int NT, typename Flat>
__device__ __forceinline__ void flat_taps(int base, const float wx[4], const float wy[4],
                                          const float dx[4], const float dy[4], float g,
                                          const Flat &flat, float &gx, float &gy) {
  const float gs = flat.scaled(g);
  float gw[NT];
#pragma unroll
  for (int k = 0; k < NT; ++k) gw[k] = gs * wx[k];
  // every value first: between the adds, which may alias them as far as the
  // compiler knows, each read would be waited for on its own
  float v[NT][NT];
#pragma unroll
  for (int l = 0; l < NT; ++l)
#pragma unroll
    for (int k = 0; k < NT; ++k) v[l][k] = flat.value(base + l * flat.pitch() + k);
  float S = 0.0f, Sx = 0.0f, Sy = 0.0f;
#pragma unroll
  for (int l = 0; l < NT; ++l) {
    const int rb = base + l * flat.pitch();
    float row = 0.0f, rowd = 0.0f;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      row = fmaf(wx[k], v[l][k], row);
      rowd = fmaf(dx[k], v[l][k], rowd);
      flat.add_scaled(rb + k, gw[k] * wy[l]);
    }
    S = fmaf(wy[l], row, S);
    Sx = fmaf(wy[l], rowd, Sx);
    Sy = fmaf(dy[l], row, Sy);
  }
  gx = g * Sx;
  gy = g * Sy;
}

// Interpolation weights at fractions (t, s) and their derivatives.
template <int INTERP>
__device__ __forceinline__ void tap_weights(float t, float s, float a, float wx[4], float wy[4],
                                            float dx[4], float dy[4]) {
  if constexpr (INTERP == DFR_BILINEAR) {
    wx[0] = 1.0f - t; wx[1] = t; dx[0] = -1.0f; dx[1] = 1.0f;
    wy[0] = 1.0f - s; wy[1] = s; dy[0] = -1.0f; dy[1] = 1.0f;
  } else {
    keys_weights(t, a, wx);
    keys_weights(s, a, wy);
    keys_dweights(t, a, dx);
    keys_dweights(s, a, dy);
  }
}

// A pixel of an interior tile (every tap in the staged box and in the
// source) at position (rx, ry) relative to the box coordinates (ox, oy).  A
// zero output gradient contributes nothing, whatever the values there.
template <int INTERP, typename Flat>
__device__ __forceinline__ void interior_backward(int ox, int oy, float rx, float ry, float a,
                                                  float g, const Flat &flat, float &gx,
                                                  float &gy) {
  int i0, j0;
  float t, s;
  tap_origin<INTERP>(rx, ox, i0, t);
  tap_origin<INTERP>(ry, oy, j0, s);
  const int base = __umul24(j0, flat.pitch()) + i0;
  if constexpr (INTERP == DFR_NEAREST) {
    flat.add_nearest(base, flat.scaled(g));
    gx = gy = 0.0f;
  } else {
    float wx[4], wy[4], dx[4], dy[4];
    tap_weights<INTERP>(t, s, a, wx, wy, dx, dy);
    flat_taps<INTERP == DFR_BILINEAR ? 2 : 4>(base, wx, wy, dx, dy, g, flat, gx, gy);
    gx = g == 0.0f ? 0.0f : gx;
    gy = g == 0.0f ? 0.0f : gy;
  }
}

// FLAT: a staged box is there (`flat`), used where every tap is inside the
// source.  The same arithmetic in the same order as the general loop, so the
// same bits.
template <int INTERP, bool FLAT, typename Fetch, typename Scatter, typename Flat>
__device__ __forceinline__ bool interp_backward(int bx, int by, float rx, float ry, int W, int H,
                                                float a, float g, const Fetch &fetch,
                                                const Scatter &scatter, const Flat &flat,
                                                float &gx, float &gy) {
  gx = 0.0f;
  gy = 0.0f;
  if constexpr (INTERP == DFR_NEAREST) {
    int i = bx + (int)rintf(rx), j = by + (int)rintf(ry);
    bool in = ((unsigned)i < (unsigned)W) && ((unsigned)j < (unsigned)H);
    if (in) scatter(0, 0, i, j, flat.scaled(g));
    return in;
  } else {
    constexpr int NT = INTERP == DFR_BILINEAR ? 2 : 4;
    float fx = floorf(rx), fy = floorf(ry);
    float t = rx - fx, s = ry - fy;
    int i0 = bx + (int)fx - (NT == 4 ? 1 : 0), j0 = by + (int)fy - (NT == 4 ? 1 : 0);
    float wx[4], wy[4], dx[4], dy[4];
    tap_weights<INTERP>(t, s, a, wx, wy, dx, dy);
    if constexpr (FLAT) {
      if (W >= NT && H >= NT && (unsigned)i0 <= (unsigned)(W - NT) &&
          (unsigned)j0 <= (unsigned)(H - NT)) {
        flat_taps<NT>(flat.index(i0, j0), wx, wy, dx, dy, g, flat, gx, gy);
        return true;
      }
    }
    bool inx[NT], iny[NT];
    bool all_in = true;
    float Fx = 0.0f, Fy = 0.0f, dFx = 0.0f, dFy = 0.0f;
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      inx[k] = (unsigned)(i0 + k) < (unsigned)W;
      iny[k] = (unsigned)(j0 + k) < (unsigned)H;
      all_in = all_in && inx[k] && iny[k];
      wx[k] = inx[k] ? wx[k] : 0.0f;
      dx[k] = inx[k] ? dx[k] : 0.0f;
      wy[k] = iny[k] ? wy[k] : 0.0f;
      dy[k] = iny[k] ? dy[k] : 0.0f;
      Fx += wx[k];
      Fy += wy[k];
      dFx += dx[k];
      dFy += dy[k];
    }
    float F = all_in ? 1.0f : Fx * Fy;
    if (!(F > 0.0f)) return false;
    float iF = all_in ? 1.0f : __builtin_amdgcn_rcpf(F);
    float c = g * iF;
    const float cs = flat.scaled(c);  // the source adjoint's contributions, times 2^Q
    // Where taps leave the source, d out = (dS - out dF) / F cancels the
    // level of the values; taking every value relative to one in-bounds tap
    // (exact: the in-bounds taps form a product set, so both dS and out dF
    // move by vr dF) leaves a rounding relative to the local contrast
    // instead.  Interior pixels use vr = 0.
    float vr = 0.0f;
    if (!all_in) {
      int kr = 0, lr = 0;
#pragma unroll
      for (int k = NT - 1; k >= 0; --k) {
        if (inx[k]) kr = k;
        if (iny[k]) lr = k;
      }
      vr = fetch(i0 + kr, j0 + lr);  // F > 0: some tap is in bounds on each axis
    }
    float S = 0.0f, Sx = 0.0f, Sy = 0.0f;
#pragma unroll
    for (int l = 0; l < NT; ++l) {
      float row = 0.0f, rowd = 0.0f;
#pragma unroll
      for (int k = 0; k < NT; ++k) {
        if (inx[k] && iny[l]) {
          float v = fetch(i0 + k, j0 + l) - vr;
          row = fmaf(wx[k], v, row);
          rowd = fmaf(dx[k], v, rowd);
          scatter(k, l, i0 + k, j0 + l, cs * wx[k] * wy[l]);
        }
      }
      S = fmaf(wy[l], row, S);
      Sx = fmaf(wy[l], rowd, Sx);
      Sy = fmaf(dy[l], row, Sy);
    }
    float out = S * iF;
    float Fdx = all_in ? 0.0f : dFx * Fy, Fdy = all_in ? 0.0f : Fx * dFy;
    gx = g * (Sx - out * Fdx) * iF;
    gy = g * (Sy - out * Fdy) * iF;
    return true;
  }
}

// Source adjoint: every contribution v = g w / F is rounded to a
// multiple of 2^-Q (Q fixed per call from max |g|: 2^-Q = 2^-30 max |g|,
// rounded to a power of two) and the multiples are summed in 64-bit
// integers.  Integer sums do not depend on the order or the grouping of
// the additions, so the result is the same bits for every run and every
// tile shape; 64-bit LDS integer adds are also much faster here than
// ds_add_f32 on contended addresses (measured: 148 against 382 us per
// 2048^2 bicubic backward with one add per tap).  The rounding (at most
// 2^-31 max |g| per contribution) stays far below an FP32 sum's; where
// every tap is inside the source |v| 2^Q < 2^31, one 32-bit conversion;
// |v| beyond 2^32 max |g| (footprints below ~2.3e-10 at frame edges)
// saturates at +-2^62.
constexpr int kDetBits = 30;
__device__ __forceinline__ double det_scale(const int *__restrict__ gmax_bits) {
  const float m = __int_as_float(*gmax_bits);
  return m > 0.0f ? ldexp(1.0, kDetBits - ilogbf(m)) : 1.0;
}

// The same scale as an exponent: 2^Q.
__device__ __forceinline__ int det_exponent(const int *__restrict__ gmax_bits) {
  const float m = __int_as_float(*gmax_bits);
  return m > 0.0f ? kDetBits - ilogbf(m) : 0;
}

// An FP32 integer of at most 63 bits as a 64-bit integer, split exactly
// into 32-bit halves.
__device__ __forceinline__ unsigned long long det_int(float y) {
  const double d = (double)y;
  const double hi = floor(d * 0x1p-32);
  const double lo = fma(hi, -0x1p32, d);
  return ((unsigned long long)(unsigned)(int)hi << 32) | (unsigned long long)(unsigned)lo;
}

// A contribution already scaled by 2^Q (formed as (g/F 2^Q) wx wy: the
// scaling of g/F is exact), rounded to the nearest integer in FP32 and
// saturated at +-2^62.
__device__ __forceinline__ unsigned long long det_quant(float y) {
  return det_int(rintf(__builtin_amdgcn_fmed3f(y, -0x1p62f, 0x1p62f)));
}

// A pixel's taps in the staged box and, for the source adjoint, its 64-bit
// integer accumulation copy (same index, same row stride).  On this path
// every tap is inside the source (F = 1): |g| 2^Q < 2^31 and |wx wy| <= 1,
// and each rounded product is at most |g| 2^Q, so a contribution is an
// integer below 2^31 in magnitude: one 32-bit conversion, no saturation.
// The contributions are formed exactly as on the general path, so a pixel
// gives the same integers on either.
template <bool SRC>
struct BwdFlat {
  const float *vals;
  unsigned long long *qacc;
  int lp, bi0, bj0, Q;
  __device__ int index(int i, int j) const { return (j - bj0) * lp + (i - bi0); }
  __device__ int pitch() const { return lp; }
  __device__ float value(int idx) const { return vals[idx]; }
  __device__ float scaled(float g) const { return ldexpf(g, Q); }
  // y = (g 2^Q wx) wy
  __device__ void add_scaled(int idx, float y) const {
    if constexpr (SRC)
      atomicAdd(&qacc[idx], (unsigned long long)(long long)(int)rintf(y));
  }
  // Nearest, y = g 2^Q: a gradient that is not finite gives the integer of the
  // general path, so it too does not depend on the tile a pixel falls into.
  __device__ void add_nearest(int idx, float y) const {
    if constexpr (SRC)
      atomicAdd(&qacc[idx], fabsf(y) < 0x1p31f ? (unsigned long long)(long long)(int)rintf(y)
                                               : det_quant(y));
  }
};

// The two halves of a lane-swap pair summed: permlane32 (lanes 0-31 get
// a(i) + a(i + 32), lanes 32-63 get b(i - 32) + b(i)) or permlane16 (rows
// 0 and 2 of 16 lanes get a's pairs of rows 0+1 and 2+3, rows 1 and 3 get
// b's).  The empty asm makes the swap's two results opaque: without it
// this compiler folds r[0] + r[1] into r[0] + r[0].
template <bool ROWS16>
__device__ __forceinline__ float swap_sum(float a, float b) {
  const auto r = ROWS16 ? __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a),
                                                           __builtin_bit_cast(unsigned, b),
                                                           false, false)
                        : __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a),
                                                           __builtin_bit_cast(unsigned, b),
                                                           false, false);
  unsigned r0 = r[0], r1 = r[1];
  asm volatile("" : "+v"(r0), "+v"(r1));
  return __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1);
}

// anchors: the cells' FP64 anchors from bwd_prepare_kernel, or null: each
// group computes those of its tile.
// SRC: the source gradient is wanted (its integer sums go to gq,
// [src_h][src_w] dense; bwd_finish_kernel converts them); without it the
// kernel carries no scatter code at all.
template <int INTERP, int SORD, int NP, bool TSIP, bool SRC>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(NP == 1 || INTERP != DFR_BICUBIC ? 5 : 1)))
void reproject_bwd(FramePlan P, TileGeom G,
                                                          const float *__restrict__ gout,
                                                          double *__restrict__ partials,
                                                          unsigned long long *__restrict__ gq,
                                                          const int *__restrict__ gmax_bits,
                                                          const Anchor *__restrict__ anchors) {
  constexpr int NC = (SORD + 1) * (SORD + 2) / 2;
  constexpr int NS = 11 + 2 * NC;
  extern __shared__ __align__(16) float lds[];
  __shared__ TileShared sh;
  __shared__ float wsum[kThreads / 64][NS];
  const int tile = xcd_tile(blockIdx.x, G.n_tiles);
  const int tid = threadIdx.x;
  float acc[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) acc[s] = 0.0f;

  TileCtx c;
  // the thread's output gradients, on their way while the anchors are computed
  float gr[NP][kRun];
  {
    const int lg = G.txt_log2, trow = tile / G.tiles_x;
    const int xr = (tile - trow * G.tiles_x) * (kRun << lg) + (tid & ((1 << lg) - 1)) * kRun;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int y = trow * (kThreads >> lg) * NP + (tid >> lg) + k * (kThreads >> lg);
      load_run(gout + (int64_t)y * G.out_w + xr, y < G.out_h ? G.out_w - xr : 0, gr[k]);
    }
  }
  if (tile_anchors<INTERP, SORD, TSIP, NP>(P, G, tile, anchors, sh, c)) {
    TilePos<NP> T;
    const int W = P.src_w, Hs = P.src_h;
    constexpr bool want_src = SRC;
    const bool bounded = sh.bounded;
    int bw, bh, lp;
    bool use_lds, interior;
    float *vals = lds;
    unsigned long long *qacc;
    // LDS: the staged box, then the 64-bit integer accumulation box (16-byte
    // aligned, two floats per entry)
    auto stage = [&]() {
      // the box, clamped to the source where it comes from the anchors
      const int u0 = sh.box[0], u1 = sh.box[1], u2 = sh.box[2], u3 = sh.box[3];
      T.bi0 = max(u0, 0);
      T.bi1 = min(u1, W - 1);
      T.bj0 = max(u2, 0);
      T.bj1 = min(u3, Hs - 1);
      T.empty = T.bi0 > T.bi1 || T.bj0 > T.bj1;
      bw = T.empty ? 0 : T.bi1 - T.bi0 + 1;
      bh = T.empty ? 0 : T.bj1 - T.bj0 + 1;
      lp = lds_pitch(bw);  // padded row stride (bank spread)
      use_lds = !T.empty && (want_src ? 3 : 1) * (int64_t)lp * bh + 8 <= (int64_t)G.lds_cap;
      // every tap of every pixel lies in the staged box and in the source
      interior = use_lds && bounded && u0 == T.bi0 && u1 == T.bi1 && u2 == T.bj0 &&
                 u3 == T.bj1 && c.x0 + (kRun << G.txt_log2) <= G.out_w &&
                 c.y0 + c.RP * NP <= G.out_h;
      float *gacc = lds + (use_lds ? ((lp * bh + 3) & ~3) : 0);
      qacc = reinterpret_cast<unsigned long long *>(gacc);
      if (!use_lds) return;
      dma_box(P, T.bi0, T.bj0, bw, bh, lp, vals);
      if (want_src) {
        typedef unsigned u4v __attribute__((ext_vector_type(4)));
        for (int i = tid; i < (lp * bh + 1) / 2; i += kThreads)
          reinterpret_cast<u4v *>(gacc)[i] = u4v{0u, 0u, 0u, 0u};
      }
    };
    if (bounded) stage();
    anchor_positions<INTERP, SORD, TSIP, NP>(P, G, sh, c, T);
    if (!bounded) stage();
    if (T.empty) T.valid = 0u;  // no tap inside the source: every pixel is uncovered
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const int qs = SRC ? det_exponent(gmax_bits) : 0;
    const int bi0 = T.bi0, bj0 = T.bj0;
    auto fetch_lds = [&](int i, int j) -> float { return vals[(j - bj0) * lp + (i - bi0)]; };
    auto fetch_glb = [&](int i, int j) -> float { return P.src[(int64_t)j * P.pitch + i]; };
    auto scat_lds = [&](int, int, int i, int j, float v) {
      if (want_src) atomicAdd(&qacc[(j - bj0) * lp + (i - bi0)], det_quant(v));
    };
    auto scat_glb = [&](int, int, int i, int j, float v) {
      if (want_src) atomicAdd(&gq[(int64_t)j * W + i], det_quant(v));
    };
    const BwdFlat<SRC> flat{vals, qacc, lp, bi0, bj0, qs};
    const float tinv = (float)P.t_inv_scale, sinv = (float)P.s_inv_scale;
    const float S_s = (float)P.s_scale;
    constexpr unsigned kAllValid = (1u << (NP * kRun)) - 1u;
    // A wave without any output gradient (a masked residual) passes over its
    // pixels: bicubic, 2048^2, us per call without the look and with it, no
    // gradient at all 79.5 and 52.8, three tenths of the blocks kept 81.6 and
    // 73.7, a full gradient 88.1 and 88.0.  Not for bilinear, whose interior
    // pixels cost little more than the look (4000x3000, full gradient: 191.5 and
    // 192.5).
    if constexpr (INTERP == DFR_BICUBIC) {
      bool live = false;
#pragma unroll
      for (int k = 0; k < NP; ++k)
#pragma unroll
        for (int e = 0; e < kRun; ++e) live = live || gr[k][e] != 0.0f;
      if (!__any(live)) T.valid = 0u;
    }
    // Every tap's contribution is quantised and added on its own (64-bit
    // integer LDS adds are cheap; summing a run's taps in a register window
    // first measured slower, the window's registers costing occupancy).
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const int y = c.y0 + c.ty + k * c.RP;
      // the run's interpolant gradients; the WCS terms are formed from them
      // after the run's scatter, so the scatter's and the WCS sums'
      // registers are not live together
      float gxs[kRun], gys[kRun];
      unsigned covm = 0u;
      if (interior && T.valid == kAllValid) {
        // no per-pixel test: box-relative tap coordinates
        covm = (1u << kRun) - 1u;
        const int ox = T.abx[k] - bi0, oy = T.aby[k] - bj0;
#pragma unroll
        for (int e = 0; e < kRun; ++e)
          interior_backward<INTERP>(ox, oy, T.rx[k][e], T.ry[k][e], G.cubic_a, gr[k][e], flat,
                                    gxs[e], gys[e]);
      } else {
#pragma unroll
        for (int e = 0; e < kRun; ++e) {
          gxs[e] = 0.0f;
          gys[e] = 0.0f;
          if (!(T.valid & (1u << (k * kRun + e)))) continue;
          const float g = gr[k][e];
          if (g == 0.0f) continue;
          float gx, gy;
          bool cov;
          if (use_lds)
            cov = interp_backward<INTERP, true>(T.abx[k], T.aby[k], T.rx[k][e], T.ry[k][e], W, Hs,
                                                G.cubic_a, g, fetch_lds, scat_lds, flat, gx, gy);
          else
            cov = interp_backward<INTERP, false>(T.abx[k], T.aby[k], T.rx[k][e], T.ry[k][e], W,
                                                 Hs, G.cubic_a, g, fetch_glb, scat_glb, flat, gx,
                                                 gy);
          if (cov) {
            gxs[e] = gx;
            gys[e] = gy;
            covm |= 1u << e;
          }
        }
      }
      if constexpr (INTERP != DFR_NEAREST) {
        // the WCS terms of the run's covered pixels, in pixel order
        const Anchor &A = sh.anchor[T.aidx[k]];
#pragma unroll
        for (int e = 0; e < kRun; ++e) {
          if (!(covm & (1u << e))) continue;
          const float gx = gxs[e], gy = gys[e];
          // the projective intermediates of the pixel (its position is known)
          PixelGeom pg;
          float den;
          pixel_geom<TSIP>(P, A, tinv, sinv, (float)((c.xr & (kCell - 1)) + e),
                           (float)(y & (kCell - 1)), pg, den);
          float fa, fau, fav, fb, fbu, fbv;
          sip_f32_grad<SORD>(P.fsA, pg.us, pg.vs, fa, fau, fav);
          sip_f32_grad<SORD>(P.fsB, pg.us, pg.vs, fb, fbu, fbv);
          const float da = gx * fmaf(fau, sinv, 1.0f) + gy * (fbu * sinv);  // dL/dU
          const float db = gx * (fav * sinv) + gy * fmaf(fbv, sinv, 1.0f);  // dL/dV
          const float U = pg.us * S_s, V = pg.vs * S_s;
          const float iw = A.inv_w0 * pg.r;
          const float t0 = A.tu0 + pg.du, t1 = A.tv0 + pg.dv;
          const float a1 = da * iw, b1 = db * iw, c1 = -(da * U + db * V) * iw;
          acc[0] = fmaf(a1, t0, acc[0]);
          acc[1] = fmaf(a1, t1, acc[1]);
          acc[2] += a1;
          acc[3] = fmaf(b1, t0, acc[3]);
          acc[4] = fmaf(b1, t1, acc[4]);
          acc[5] += b1;
          acc[6] = fmaf(c1, t0, acc[6]);
          acc[7] = fmaf(c1, t1, acc[7]);
          acc[8] += c1;
          acc[9] += gx;
          acc[10] += gy;
          if constexpr (SORD > 0) {
            float up = 1.0f;
#pragma unroll
            for (int p = 0; p <= SORD; ++p) {
              float m = up;
#pragma unroll
              for (int q = 0; p + q <= SORD; ++q) {
                acc[11 + tri_n(SORD, p, q)] = fmaf(gx, m, acc[11 + tri_n(SORD, p, q)]);
                acc[11 + NC + tri_n(SORD, p, q)] = fmaf(gy, m, acc[11 + NC + tri_n(SORD, p, q)]);
                m *= pg.vs;
              }
              up *= pg.us;
            }
          }
        }
      }
    }
    __syncthreads();
    if (SRC && use_lds) {
      const int wave = tid >> 6, lane = tid & 63;
      for (int r = wave; r < bh; r += kThreads / 64)
        for (int col = lane; col < bw; col += 64) {
          const unsigned long long q = qacc[r * lp + col];
          if (q != 0ull) atomicAdd(&gq[(int64_t)(bj0 + r) * W + bi0 + col], q);
        }
    }
  }
  // per-wave, then per-group sums of the WCS terms (skipped tiles give 0):
  // a transposing butterfly halves the number of live sums at each lane
  // exchange (lanes i, i + 32, then rows 0/1 and 2/3 of 16 lanes), so each
  // row of the wave ends with a quarter of the sums, which DPP shifts
  // reduce within the row (lane 15 holds the row's total).  Fixed order.
  {
    constexpr int NSP = NS <= 16 ? 16 : (NS <= 32 ? 32 : 64);
    constexpr int H = NSP / 2, Q = NSP / 4;
    static_assert(NS <= 64, "WCS sums per wave");
    float x[H];
#pragma unroll
    for (int s = 0; s < H; ++s) {
      // lanes 0-31: sum s over lanes i and i + 32; lanes 32-63: sum s + H
      x[s] = swap_sum<false>(acc[s], s + H < NS ? acc[s + H] : 0.0f);
    }
    float y[Q];
#pragma unroll
    for (int s = 0; s < Q; ++s) {
      // row 0: sum s, row 1: s + Q, row 2: s + H, row 3: s + H + Q
      float v = swap_sum<true>(x[s], x[s + Q]);
      v = dpp_add<0x111, 0xf>(v);  // row_shr:1
      v = dpp_add<0x112, 0xf>(v);  // row_shr:2
      v = dpp_add<0x114, 0xf>(v);  // row_shr:4
      y[s] = dpp_add<0x118, 0xf>(v);  // row_shr:8
    }
    const int lane = tid & 63, row = lane >> 4;
    if ((lane & 15) == 15) {
      const int off = row == 0 ? 0 : (row == 1 ? Q : (row == 2 ? H : H + Q));
#pragma unroll
      for (int s = 0; s < Q; ++s)
        if (s + off < NS) wsum[tid >> 6][s + off] = y[s];
    }
  }
  __syncthreads();
  if (tid < NS) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) t += (double)wsum[w][tid];
    partials[(int64_t)tid * G.n_tiles + tile] = t;  // column-major: one column per sum
  }
}

using BwdKernel = void (*)(FramePlan, TileGeom, const float *, double *, unsigned long long *,
                          const int *, const Anchor *);

template <int INTERP, int NP, bool TSIP, bool SRC>
BwdKernel bwd_sord(int sord) {
  switch (sord) {
    case 0: return reproject_bwd<INTERP, 0, NP, TSIP, SRC>;
    case 1: return reproject_bwd<INTERP, 1, NP, TSIP, SRC>;
    case 2: return reproject_bwd<INTERP, 2, NP, TSIP, SRC>;
    case 3: return reproject_bwd<INTERP, 3, NP, TSIP, SRC>;
    case 4: return reproject_bwd<INTERP, 4, NP, TSIP, SRC>;
    default: return reproject_bwd<INTERP, 5, NP, TSIP, SRC>;
  }
}

// The backward kernel runs 1 or 2 rows per thread (the host picks such
// tiles); the target SIP is compiled in only where the target has one.
template <int INTERP>
BwdKernel bwd_pick(int np, int sord, bool tsip, bool src) {
  if (src) {
    if (tsip) return np == 1 ? bwd_sord<INTERP, 1, true, true>(sord) : bwd_sord<INTERP, 2, true, true>(sord);
    return np == 1 ? bwd_sord<INTERP, 1, false, true>(sord) : bwd_sord<INTERP, 2, false, true>(sord);
  }
  if (tsip) return np == 1 ? bwd_sord<INTERP, 1, true, false>(sord) : bwd_sord<INTERP, 2, true, false>(sord);
  return np == 1 ? bwd_sord<INTERP, 1, false, false>(sord) : bwd_sord<INTERP, 2, false, false>(sord);
}

extern template BwdKernel bwd_pick<DFR_NEAREST>(int, int, bool, bool);
extern template BwdKernel bwd_pick<DFR_BILINEAR>(int, int, bool, bool);
extern template BwdKernel bwd_pick<DFR_BICUBIC>(int, int, bool, bool);

}  // namespace dfr
