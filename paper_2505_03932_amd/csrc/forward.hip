// Forward reprojection launchers: the FP32 tiled path (kernels in
// tile_kernels.hpp: FP64 anchors, FP32 per-pixel offsets, LDS-staged source
// boxes) and the two FP64 comparison forms (composed projective map;
// explicit two-stage trigonometry of the paper's section 3.2).
#include "tile_kernels.hpp"

namespace dfr {

using TileKernel = void (*)(FramePlan, TileGeom);

static TileKernel pick_tile_kernel(int interp, int np, int sord) {
  const void *k = interp == DFR_NEAREST    ? tile_kernel_for<DFR_NEAREST>(np, sord)
                  : interp == DFR_BILINEAR ? tile_kernel_for<DFR_BILINEAR>(np, sord)
                                           : tile_kernel_for<DFR_BICUBIC>(np, sord);
  return reinterpret_cast<TileKernel>(const_cast<void *>(k));
}

bool forward_small(const FramePlan &P, const TileGeom &G, int np) {
  const int most = P.s_order == 5 ? kSmallTilesOrder5 : kSmallTiles;
  return np == 1 && G.n_tiles <= most && P.t_order == 0 && P.s_order <= 5;
}

hipError_t launch_forward_small(const FramePlan &P, const TileGeom &G, int interp,
                                hipStream_t stream) {
  if (G.n_tiles <= 0) return hipSuccess;
  const void *k = interp == DFR_NEAREST    ? small_kernel_for<DFR_NEAREST>(P.s_order)
                  : interp == DFR_BILINEAR ? small_kernel_for<DFR_BILINEAR>(P.s_order)
                                           : small_kernel_for<DFR_BICUBIC>(P.s_order);
  FramePlan plan = P;
  TileGeom geom = G;
  void *args[] = {&plan, &geom};
  return launch_kernel(k, dim3(G.n_tiles), dim3(kThreads), args,
                       (size_t)G.lds_cap * sizeof(float), stream);
}

hipError_t launch_forward_f32(const FramePlan &P, const TileGeom &G, int interp, int np,
                              hipStream_t stream) {
  if (G.n_tiles <= 0) return hipSuccess;
  // a target with SIP A/B needs the kernel that compiles the target SIP in
  TileKernel k = pick_tile_kernel(interp, np, P.t_order > 0 ? kRtOrder : P.s_order);
  size_t lds = (size_t)G.lds_cap * sizeof(float);
  hipLaunchKernelGGL(k, dim3(G.n_tiles), dim3(kThreads), lds, stream, P, G);
  return hipGetLastError();
}

// ------------------------------------------------------ cell models

// One lane per 32x32 cell of the output grid: the certified cubic model of
// the cell's position map (cell_model.hpp), written to the model table.
template <int SORD, int TN>
__global__ __launch_bounds__(64) void cell_models_kernel(FramePlan P, int ncx, int n,
                                                        CellModel *__restrict__ out) {
  __shared__ LdsCoefs<(TN > 0 ? 4 : 2)> L;
  const SipCoefs C = stage_coefs(plan_argument(), L);
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= n) return;
  const int cy = i / ncx, cx = i - cy * ncx;
  CellModel M;
  cell_model<SORD, TN>(P, C, cx, cy, M);
  out[i] = M;
}

// The same for every frame of a batch: block b holds 8x8 cells of frame
// b / bpf (bpf blocks per frame, bcols of them to a row; the frame's table
// starts at frame * ncells).  Most of a stack's grid lies outside any one
// frame: those cells are told apart first, from a bound that costs a fraction
// of the model, and in 8x8 blocks, so that most waves hold only cells of one
// kind; they get no model, only the mark kCellOut.  A block belongs to one
// frame, so the frame's plan is read with scalar loads; with cells numbered across frames the plan's address differed
// per lane as far as the compiler knew, and every coefficient was a vector load
// (64 frames on 8192^2, order 5: 541 us so and with every cell modelled, 397 us
// with scalar loads and the cheaper models, 306 us with the test, 200 us since
// reach_kernel folds the boxes, 161 us with the coefficients in LDS).
template <int SORD, int TN>
__global__ __launch_bounds__(64) void cell_models_batch_kernel(const FramePlan *__restrict__ plans,
                                                              int ncx, int ncy, int bcols,
                                                              int bpf,
                                                              CellModel *__restrict__ out,
                                                              int4 *__restrict__ parts) {
  const int frame = blockIdx.x / bpf, block = blockIdx.x - frame * bpf;
  const int by = block / bcols;
  const int cx = (block - by * bcols) * 8 + (threadIdx.x & 7), cy = by * 8 + (threadIdx.x >> 3);
  const int64_t c = (int64_t)frame * ncx * ncy + (int64_t)cy * ncx + cx;
  // the frame table is read-only here: scalar loads through the constant
  // address space
  using ConstPlan = const __attribute__((address_space(4))) FramePlan;
  ConstPlan *cp = (ConstPlan *)(plans + frame);
  const FramePlan &P = *(const FramePlan *)cp;
  __shared__ LdsCoefs<(TN > 0 ? 4 : 2)> L;
  const SipCoefs C = stage_coefs(cp, L);
  int reach = 0;
  const bool in = cx < ncx && cy < ncy;
  if (in && TN == 0 && cell_out_of_reach<SORD>(P, L.f, cx, cy)) {
    if (out) out[c].certified = kCellOut;
  } else if (in) {
    CellModel M;
    cell_model<SORD, TN>(P, C, cx, cy, M);
    if (out) out[c] = M;  // null: only the reach boxes are wanted
    // can any pixel of the cell have a tap inside the source?  From the
    // model's range over the whole cell, grown by 4 px (more than any tap
    // support and the tile kernel's guard); without a model, the anchor's
    // rigorous test with the widest support
    if (P.src_w <= 0 || P.src_h <= 0 || !parts) {
      reach = 0;
    } else if (!M.certified) {
      Anchor A;
      compute_anchor<SORD, (TN > 0)>(P, cx * kCell, cy * kCell, 4, A);
      reach = A.touch;
    } else {
      const float h = (float)kHalfCell;
      const float rx = (fabsf(M.mx[4]) + fabsf(M.mx[1])) * h + M.ex + 4.0f;
      const float ry = (fabsf(M.my[4]) + fabsf(M.my[1])) * h + M.ey + 4.0f;
      const float xc = (float)M.bx + M.mx[0], yc = (float)M.by + M.my[0];
      reach = (xc + rx >= 0.0f && xc - rx <= (float)(P.src_w - 1) && yc + ry >= 0.0f &&
               yc - ry <= (float)(P.src_h - 1)) ? 1 : 0;
    }
  }
  if (!parts) return;  // no reach boxes wanted
  // the block's box, for reach_kernel
  const int v0 = wave_max(reach ? kReachBig - cx : 0), v1 = wave_max(reach ? cx + 1 : 0);
  const int v2 = wave_max(reach ? kReachBig - cy : 0), v3 = wave_max(reach ? cy + 1 : 0);
  if (threadIdx.x == 0) parts[blockIdx.x] = make_int4(v0, v1, v2, v3);
}

// A frame's reach box from those of its blocks, one group per frame.  (Blocks
// folding theirs into the frame's with atomics, or only with a look at it
// before, met on one line that every XCD reads and writes in memory: the
// models of 64 frames on 8192^2 took 297 us so, 195 and 5 us without.)
__global__ __launch_bounds__(256) void reach_kernel(const FramePlan *__restrict__ plans,
                                                    const int4 *__restrict__ parts, int bpf) {
  __shared__ int4 wm[4];
  int4 m = make_int4(0, 0, 0, 0);
  for (int i = threadIdx.x; i < bpf; i += 256) {
    const int4 v = parts[(int64_t)blockIdx.x * bpf + i];
    m.x = max(m.x, v.x);
    m.y = max(m.y, v.y);
    m.z = max(m.z, v.z);
    m.w = max(m.w, v.w);
  }
  m = make_int4(wave_max(m.x), wave_max(m.y), wave_max(m.z), wave_max(m.w));
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t *r = plans[blockIdx.x].reach;
    r[0] = max(max(wm[0].x, wm[1].x), max(wm[2].x, wm[3].x));
    r[1] = max(max(wm[0].y, wm[1].y), max(wm[2].y, wm[3].y));
    r[2] = max(max(wm[0].z, wm[1].z), max(wm[2].z, wm[3].z));
    r[3] = max(max(wm[0].w, wm[1].w), max(wm[2].w, wm[3].w));
  }
}
const void *reach_kernel_ptr() { return reinterpret_cast<const void *>(reach_kernel); }

// Instances: source orders 0 .. 5 (and any) for a target without SIP; with
// target SIP both orders up to 5, or any (padding with zero coefficients is
// exact, and one instance keeps the library small).  A distorted 2048^2 target,
// orders 3 and 4, bilinear: 128 us per call when every pixel took the chain
// from anchors, 26 us with models (5.5 us of it this kernel).
template <template <int, int> class K>
static const void *pick_models(int sord, int tord) {
  if (tord > 0) return sord >= 0 && sord <= 5 && tord <= 5 ? K<5, 5>::ptr() : K<-1, kMaxOrder>::ptr();
  switch (sord) {
    case 0: return K<0, 0>::ptr();
    case 1: return K<1, 0>::ptr();
    case 2: return K<2, 0>::ptr();
    case 3: return K<3, 0>::ptr();
    case 4: return K<4, 0>::ptr();
    case 5: return K<5, 0>::ptr();
    default: return K<-1, 0>::ptr();
  }
}

template <int SORD, int TN>
struct ModelsK {
  static const void *ptr() { return reinterpret_cast<const void *>(cell_models_kernel<SORD, TN>); }
};
template <int SORD, int TN>
struct ModelsBatchK {
  static const void *ptr() { return reinterpret_cast<const void *>(cell_models_batch_kernel<SORD, TN>); }
};

const void *cell_models_batch_ptr(int sord, int tord) { return pick_models<ModelsBatchK>(sord, tord); }

hipError_t launch_cell_models(const FramePlan &P, int ncx, int ncy, CellModel *out,
                              hipStream_t stream) {
  int n = ncx * ncy;
  if (n <= 0) return hipSuccess;
  FramePlan plan = P;
  void *args[] = {&plan, &ncx, &n, &out};
  return launch_kernel(pick_models<ModelsK>(P.s_order, P.t_order), dim3((n + 63) / 64), dim3(64),
                       args, 0, stream);
}

// ------------------------------------------------------ FP64 comparison forms

// FP64 interpolation at (xs, ys) with zero padding; same rules as the FP32
// path (interior footprint exactly 1, out = S/F where F > 0).
template <int INTERP>
__device__ __forceinline__ void interp_f64(const FramePlan &P, double xs, double ys, double a,
                                           double &out, double &fp) {
  const int W = P.src_w, H = P.src_h;
  auto val = [&](int64_t i, int64_t j) -> double {
    return (double)P.src[j * P.pitch + i];
  };
  if constexpr (INTERP == DFR_NEAREST) {
    double fi = rint(xs), fj = rint(ys);
    bool in = fi >= 0.0 && fi < W && fj >= 0.0 && fj < H;
    out = in ? val((int64_t)fi, (int64_t)fj) : 0.0;
    fp = in ? 1.0 : 0.0;
  } else {
    double fx = floor(xs), fy = floor(ys);
    double t = xs - fx, s = ys - fy;
    int n = INTERP == DFR_BILINEAR ? 2 : 4;
    int64_t i0 = (int64_t)fx - (INTERP == DFR_BICUBIC ? 1 : 0);
    int64_t j0 = (int64_t)fy - (INTERP == DFR_BICUBIC ? 1 : 0);
    double wx[4], wy[4];
    if constexpr (INTERP == DFR_BILINEAR) {
      wx[0] = 1.0 - t; wx[1] = t; wy[0] = 1.0 - s; wy[1] = s;
      wx[2] = wx[3] = wy[2] = wy[3] = 0.0;
    } else {
      double u = 1.0 - t, v = 1.0 - s;
      wx[0] = a * t * u * u;
      wx[1] = fma(fma(a + 2.0, t, -(a + 3.0)), t * t, 1.0);
      wx[2] = fma(fma(a + 2.0, u, -(a + 3.0)), u * u, 1.0);
      wx[3] = a * t * t * u;
      wy[0] = a * s * v * v;
      wy[1] = fma(fma(a + 2.0, s, -(a + 3.0)), s * s, 1.0);
      wy[2] = fma(fma(a + 2.0, v, -(a + 3.0)), v * v, 1.0);
      wy[3] = a * s * s * v;
    }
    double S = 0.0, Fx = 0.0, Fy = 0.0;
    bool all_in = true;
    for (int k = 0; k < n; ++k) {
      bool ix = i0 + k >= 0 && i0 + k < W, iy = j0 + k >= 0 && j0 + k < H;
      all_in = all_in && ix && iy;
      Fx += ix ? wx[k] : 0.0;
      Fy += iy ? wy[k] : 0.0;
    }
    for (int l = 0; l < n; ++l) {
      if (j0 + l < 0 || j0 + l >= H) continue;
      double row = 0.0;
      for (int k = 0; k < n; ++k)
        if (i0 + k >= 0 && i0 + k < W) row = fma(wx[k], val(i0 + k, j0 + l), row);
      S = fma(wy[l], row, S);
    }
    double F = all_in ? 1.0 : Fx * Fy;
    out = all_in ? S : (F > 0.0 ? S / F : 0.0);
    fp = F > 0.0 ? F : 0.0;
  }
}

// Paper section 3.2 literally (trigonometric two-stage form, FP64), with
// the arcsines evaluated as atan2 of the same unit vector.
__device__ __forceinline__ bool position_trig(const FramePlan &P, const TrigPlan &T, double x,
                                              double y, double &xs, double &ys) {
  const double R0 = 57.295779513082320876798;  // 180 / pi
  double u = x - P.tcr[0], v = y - P.tcr[1];
  if (P.t_order > 0) {
    double du = sip_f64_dev(P.tA, P.t_order, u, v);
    double dv = sip_f64_dev(P.tB, P.t_order, u, v);
    u += du;
    v += dv;
  }
  double up = T.tcd[0] * u + T.tcd[1] * v;
  double vp = T.tcd[2] * u + T.tcd[3] * v;
  double r = hypot(up, vp);
  double phi = atan2(-up, vp);
  double theta = atan2(R0, r);
  double st, ct, sp, cp, sd0, cd0;
  sincos(theta, &st, &ct);
  sincos(phi, &sp, &cp);
  sincos(T.tcrval[1], &sd0, &cd0);
  double Z = st * sd0 + ct * cd0 * cp;
  double X = -ct * sp;
  double Y = st * cd0 - ct * sd0 * cp;
  double dec = atan2(Z, hypot(X, Y));
  double ra = T.tcrval[0] + atan2(X, Y);
  // to the source plane
  double sde, cde, sdr, cdr, ss0, cs0;
  sincos(dec, &sde, &cde);
  sincos(ra - T.scrval[0], &sdr, &cdr);
  sincos(T.scrval[1], &ss0, &cs0);
  double X2 = -cde * sdr;
  double Y2 = sde * cs0 - cde * ss0 * cdr;
  double Z2 = sde * ss0 + cde * cs0 * cdr;
  if (!(Z2 > 0.0)) return false;
  double phi2 = atan2(X2, Y2);
  double theta2 = atan2(Z2, hypot(X2, Y2));
  double st2, ct2, sp2, cp2;
  sincos(theta2, &st2, &ct2);
  sincos(phi2, &sp2, &cp2);
  double r2 = R0 * ct2 / st2;
  double xp = -r2 * sp2, yp = r2 * cp2;
  double U = T.scdi[0] * xp + T.scdi[1] * yp;
  double V = T.scdi[2] * xp + T.scdi[3] * yp;
  if (P.s_order > 0) {
    double dU = sip_f64_dev(P.sA, P.s_order, U, V);
    double dV = sip_f64_dev(P.sB, P.s_order, U, V);
    U += dU;
    V += dV;
  }
  xs = U + P.scr[0];
  ys = V + P.scr[1];
  return isfinite(xs) && isfinite(ys);
}

template <int INTERP, bool TRIG>
__global__ __launch_bounds__(kThreads) void reproject_f64(FramePlan P, TrigPlan T, TileGeom G) {
  const int64_t n = (int64_t)G.out_h * G.out_w;
  const float miss = G.nan_outside ? __builtin_nanf("") : 0.0f;
  for (int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x; idx < n;
       idx += (int64_t)gridDim.x * kThreads) {
    const int y = (int)(idx / G.out_w), x = (int)(idx - (int64_t)y * G.out_w);
    double xs = 0.0, ys = 0.0;
    bool ok = TRIG ? position_trig(P, T, x, y, xs, ys) : position_f64_ct<kRtOrder, true>(P, x, y, xs, ys);
    ok = ok && fabs(xs) < 4.0e15 && fabs(ys) < 4.0e15;
    double o = 0.0, f = 0.0;
    if (ok && P.src_h > 0 && P.src_w > 0) interp_f64<INTERP>(P, xs, ys, (double)G.cubic_a, o, f);
    bool cov = f > 0.0;
    P.out[idx] = cov ? (float)o : miss;
    if (P.fp) P.fp[idx] = cov ? (float)f : 0.0f;
    if (G.debug) {
      double2 d;
      d.x = ok ? xs : __builtin_nan("");
      d.y = ok ? ys : __builtin_nan("");
      reinterpret_cast<double2 *>(G.debug)[idx] = d;
    }
  }
}

hipError_t launch_forward_f64(const FramePlan &P, const TrigPlan &T, const TileGeom &G,
                              int interp, bool trig, hipStream_t stream) {
  int64_t n = (int64_t)G.out_h * G.out_w;
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + kThreads - 1) / kThreads;
  if (blocks > 65536 * 8) blocks = 65536 * 8;
  void (*k)(FramePlan, TrigPlan, TileGeom);
  if (trig) {
    k = interp == DFR_NEAREST ? reproject_f64<DFR_NEAREST, true>
        : interp == DFR_BILINEAR ? reproject_f64<DFR_BILINEAR, true>
                                 : reproject_f64<DFR_BICUBIC, true>;
  } else {
    k = interp == DFR_NEAREST ? reproject_f64<DFR_NEAREST, false>
        : interp == DFR_BILINEAR ? reproject_f64<DFR_BILINEAR, false>
                                 : reproject_f64<DFR_BICUBIC, false>;
  }
  hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(kThreads), 0, stream, P, T, G);
  return hipGetLastError();
}

// ------------------------------------------------------------ small kernels

__global__ void zero_i32_kernel(int *p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

hipError_t launch_zero_i32(int *p, int64_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(zero_i32_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, p, n);
  return hipGetLastError();
}

}  // namespace dfr
