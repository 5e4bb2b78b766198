// Certified local models of the position map (forward path).
//
// For a 32x32 cell of output pixels with centre (xc, yc), the source
// position of pixel (xc + a, yc + b), |a|, |b| <= 15.5, is written as
//     X = bx + sum_{i+j<=3} mx[a^i b^j] a^i b^j   (and Y likewise)
// plus a remainder bounded rigorously over the whole cell.  The model comes
// from Taylor-model arithmetic in FP64 (a degree-3 polynomial in (a, b) and
// an interval for everything it leaves out) applied to the two stages of
// section 3.2 in their composed form:
//   0. a target with SIP: its A/B re-expanded about the cell centre give the
//      corrected target offset d as a Taylor model (d = (a, b) without SIP);
//   1. the projective step: dU = (g.d) / (1 + e), e = k.d;
//      1/(1 + e) = 1 - e + e^2 - e^3 + e^4/(1 + e), |e| <= kap < 1/4;
//   2. the source SIP AP/BP re-expanded about the cell centre's (U, V)
//      (Taylor shift of the polynomial: exact up to rounding) and composed
//      with (dU, dV); terms of degree >= 4 in (dU, dV) go to the remainder.
// A cell is certified when the remainder is below kModelTol; the bound it
// reports adds the FP32 rounding of the stored coefficients.  Certification
// also proves the projective denominator positive over the cell (every
// pixel valid).
#pragma once

#include "common.hpp"

namespace dfr {

constexpr double kHalfCell = 0.5 * (kCell - 1);  // 15.5: |a|, |b| over a cell
constexpr double kModelTol = 1.0e-6;             // px: accepted model error
constexpr double kModelSlack = 1.0e-3;           // px: FP32 evaluation margin in box bounds

// Per-cell model (device table, 112 bytes).  Coefficient k of mx/my
// multiplies a^cm_i(k) b^cm_j(k); the layout groups powers of a so a row of
// pixels (fixed b) reduces to a cubic in a.
struct alignas(16) CellModel {
  float mx[10], my[10];  // source position minus (bx, by)
  float ex, ey;          // bound on |position - (constant + linear part)| over the cell
  int32_t bx, by;        // integer part of the source position at the cell centre
  float err;             // certified bound on |model - map| over the cell (px)
  int32_t certified;     // 1: truncation <= kModelTol and every pixel has a valid position;
                         // kCellOut: no pixel reaches the source (the rest of the record is not set)
  float tie;             // nearest: FP32 positions this close to a rounding tie are decided in FP64
  int32_t pad_;
};
static_assert(sizeof(CellModel) == 112, "CellModel layout");
constexpr int32_t kCellOut = 2;

__host__ __device__ constexpr int cm_i(int k) { return k < 4 ? 0 : (k < 7 ? 1 : (k < 9 ? 2 : 3)); }
__host__ __device__ constexpr int cm_j(int k) { return k < 4 ? k : (k < 7 ? k - 4 : (k < 9 ? k - 7 : 0)); }
__host__ __device__ constexpr int cm_idx(int i, int j) {
  return i == 0 ? j : (i == 1 ? 4 + j : (i == 2 ? 7 + j : 9));
}

// Taylor model: degree-3 polynomial in (a, b) plus a bound r on the rest.
// The functions below are told at compile time which degrees of their
// arguments can be non-zero (LO .. HI: a linear form is <1, 1>, a quantity
// without a constant term <1, 3>) and leave out the products and norms of the
// others: without that the compiler, which may not drop a multiplication by
// zero, keeps all of them.  The terms that remain are combined in the same
// order, so the result has the same bits (order 4: 718 FP64 instructions per
// lane instead of 988; the models of a 6000x4000 grid 5.5 us instead of 6.0).
struct Tm3 {
  double c[10];
  double r;
};

__host__ __device__ constexpr int cm_deg(int k) { return cm_i(k) + cm_j(k); }

__host__ __device__ inline void tm_zero(Tm3 &t) {
#pragma unroll
  for (int k = 0; k < 10; ++k) t.c[k] = 0.0;
  t.r = 0.0;
}

// Sum of |c| h^d over the terms of each degree d.
template <int LO, int HI>
__host__ __device__ inline void tm_norms(const Tm3 &t, double n[4]) {
  const double h = kHalfCell;
  const double hp[4] = {1.0, h, h * h, h * h * h};
#pragma unroll
  for (int d = 0; d < 4; ++d) n[d] = 0.0;
#pragma unroll
  for (int k = 0; k < 10; ++k)
    if (cm_deg(k) >= LO && cm_deg(k) <= HI) n[cm_deg(k)] += __builtin_fabs(t.c[k]) * hp[cm_deg(k)];
}

// Bound on |t| over the cell.
template <int LO, int HI>
__host__ __device__ inline double tm_bound(const Tm3 &t) {
  double n[4], b = t.r;
  tm_norms<LO, HI>(t, n);
  double s = 0.0;
#pragma unroll
  for (int d = LO; d <= HI; ++d) s += n[d];
  return s + b;
}

// z = x * y: product terms of degree <= 3 kept, the others bounded.
template <int XLO, int XHI, int YLO, int YHI>
__host__ __device__ inline void tm_mul(const Tm3 &x, const Tm3 &y, Tm3 &z) {
#pragma unroll
  for (int k = 0; k < 10; ++k) z.c[k] = 0.0;
#pragma unroll
  for (int kx = 0; kx < 10; ++kx)
#pragma unroll
    for (int ky = 0; ky < 10; ++ky) {
      const int dx = cm_deg(kx), dy = cm_deg(ky);
      if (dx < XLO || dx > XHI || dy < YLO || dy > YHI || dx + dy > 3) continue;
      double &t = z.c[cm_idx(cm_i(kx) + cm_i(ky), cm_j(kx) + cm_j(ky))];
      t = __builtin_fma(x.c[kx], y.c[ky], t);
    }
  double nx[4], ny[4];
  tm_norms<XLO, XHI>(x, nx);
  tm_norms<YLO, YHI>(y, ny);
  double drop = 0.0, bx = 0.0, by = 0.0;
#pragma unroll
  for (int d1 = XLO; d1 <= XHI; ++d1)
#pragma unroll
    for (int d2 = YLO; d2 <= YHI; ++d2)
      if (d1 + d2 >= 4) drop += nx[d1] * ny[d2];
#pragma unroll
  for (int d = XLO; d <= XHI; ++d) bx += nx[d];
#pragma unroll
  for (int d = YLO; d <= YHI; ++d) by += ny[d];
  z.r = drop + bx * y.r + by * x.r + x.r * y.r;
}

// z += s * x
template <int LO, int HI>
__host__ __device__ inline void tm_axpy(double s, const Tm3 &x, Tm3 &z) {
#pragma unroll
  for (int k = 0; k < 10; ++k)
    if (cm_deg(k) >= LO && cm_deg(k) <= HI) z.c[k] = __builtin_fma(s, x.c[k], z.c[k]);
  z.r += __builtin_fabs(s) * x.r;
}

// Taylor coefficients of the SIP polynomial c (packed by tri9, order <= N,
// zero past its order) about (U0, V0): t[tri9(i, j)] multiplies dU^i dV^j.
// Repeated synthetic division along U for every power of V, then along V.
template <int N>
__host__ __device__ inline void sip_taylor(const double *__restrict__ c, double U0, double V0,
                                           double t[kMaxCoef]) {
#pragma unroll
  for (int k = 0; k < kMaxCoef; ++k) t[k] = 0.0;
#pragma unroll
  for (int p = 0; p <= N; ++p)
#pragma unroll
    for (int q = 0; p + q <= N; ++q) t[tri9(p, q)] = c[tri9(p, q)];
#pragma unroll
  for (int q = 0; q <= N; ++q) {
    const int m = N - q;
#pragma unroll
    for (int k = 0; k < m; ++k)
#pragma unroll
      for (int p = m - 1; p >= k; --p) t[tri9(p, q)] = __builtin_fma(U0, t[tri9(p + 1, q)], t[tri9(p, q)]);
  }
#pragma unroll
  for (int p = 0; p <= N; ++p) {
    const int m = N - p;
#pragma unroll
    for (int k = 0; k < m; ++k)
#pragma unroll
      for (int q = m - 1; q >= k; --q) t[tri9(p, q)] = __builtin_fma(V0, t[tri9(p, q + 1)], t[tri9(p, q)]);
  }
}

// Position model of cell (cx, cy) of the output grid.  SORD: source SIP
// order at compile time (< 0: any order up to kMaxOrder; the padded
// coefficients make both give the same model).  TN: highest target SIP order
// the instance covers (0: a target with SIP gets no model).  C: the
// polynomials' coefficients, from the plan or a copy of it in LDS.
struct SipCoefs {
  const double *sA, *sB;  // source AP, BP
  const double *tA, *tB;  // target A, B (TN > 0)
};

template <int SORD, int TN = 0>
__host__ __device__ inline void cell_model(const FramePlan &P, const SipCoefs &C, int cx, int cy,
                                           CellModel &M) {
  constexpr int N = SORD >= 0 ? SORD : kMaxOrder;
  const double h = kHalfCell;
#pragma unroll
  for (int k = 0; k < 10; ++k) {
    M.mx[k] = 0.0f;
    M.my[k] = 0.0f;
  }
  M.ex = M.ey = 0.0f;
  M.bx = M.by = 0;
  M.err = 1.0e30f;
  M.certified = 0;
  M.tie = 0.5f;
  M.pad_ = 0;
  if (P.t_order > TN) return;

  double uc = (double)cx * kCell + h - P.tcr[0], vc = (double)cy * kCell + h - P.tcr[1];
  Tm3 du, dv;  // SIP-corrected target offset from the centre's
  if constexpr (TN > 0) {
    double t[kMaxCoef];
    auto correct = [&](const double *c, int main, Tm3 &d) {
      sip_taylor<TN>(c, uc, vc, t);
      tm_zero(d);
      double hp[TN + 1];
      hp[0] = 1.0;
#pragma unroll
      for (int i = 1; i <= TN; ++i) hp[i] = hp[i - 1] * h;
#pragma unroll
      for (int i = 0; i <= TN; ++i)
#pragma unroll
        for (int j = 0; i + j <= TN; ++j) {
          if (i + j == 0) continue;
          if (i + j <= 3)
            d.c[cm_idx(i, j)] = t[tri9(i, j)];
          else
            d.r += __builtin_fabs(t[tri9(i, j)]) * hp[i + j];
        }
      d.c[main] += 1.0;
      return t[0];
    };
    const double a0 = correct(C.tA, cm_idx(1, 0), du), b0 = correct(C.tB, cm_idx(0, 1), dv);
    uc += a0;
    vc += b0;
  }
  const double *H = P.H;
  const double pc = __builtin_fma(H[0], uc, __builtin_fma(H[1], vc, H[2]));
  const double qc = __builtin_fma(H[3], uc, __builtin_fma(H[4], vc, H[5]));
  const double wc = __builtin_fma(H[6], uc, __builtin_fma(H[7], vc, H[8]));
  if (!(wc > 0.0)) return;
  const double iw = 1.0 / wc;
  const double Uc = pc * iw, Vc = qc * iw;
  const double g1 = (H[0] - Uc * H[6]) * iw, g2 = (H[1] - Uc * H[7]) * iw;
  const double f1 = (H[3] - Vc * H[6]) * iw, f2 = (H[4] - Vc * H[7]) * iw;
  const double k1 = H[6] * iw, k2 = H[7] * iw;

  // e = k.d, g.d and f.d: linear in (a, b), or Taylor models with target SIP
  constexpr int LH = TN > 0 ? 3 : 1;
  auto dot = [&](double c1, double c2, Tm3 &z) {
    tm_zero(z);
    if constexpr (TN > 0) {
      tm_axpy<1, 3>(c1, du, z);
      tm_axpy<1, 3>(c2, dv, z);
    } else {
      z.c[cm_idx(1, 0)] = c1;
      z.c[cm_idx(0, 1)] = c2;
    }
  };
  Tm3 eps, e2, e3, rho;
  dot(k1, k2, eps);
  const double kap = TN > 0 ? tm_bound<1, LH>(eps) : (__builtin_fabs(k1) + __builtin_fabs(k2)) * h;
  if (!(kap < 0.25)) return;

  // 1 / (1 + e) as a Taylor model
  constexpr int H2 = TN > 0 ? 3 : 2;  // e^2: degrees 2 .. H2
  tm_mul<1, LH, 1, LH>(eps, eps, e2);
  tm_mul<2, H2, 1, LH>(e2, eps, e3);
#pragma unroll
  for (int k = 0; k < 10; ++k) {
    const int d = cm_deg(k);
    if (d == 0)
      rho.c[k] = 1.0;
    else if (d == 1)
      rho.c[k] = -eps.c[k];
    else if (d == 2)
      rho.c[k] = TN > 0 ? e2.c[k] - eps.c[k] : e2.c[k];
    else
      rho.c[k] = TN > 0 ? e2.c[k] - eps.c[k] - e3.c[k] : -e3.c[k];
  }
  rho.r = kap * kap * kap * kap / (1.0 - kap);
  if constexpr (TN > 0) rho.r += eps.r + e2.r + e3.r;

  Tm3 gd, fd, al, be;
  dot(g1, g2, gd);
  dot(f1, f2, fd);
  tm_mul<1, LH, 0, 3>(gd, rho, al);  // dU
  tm_mul<1, LH, 0, 3>(fd, rho, be);  // dV

  Tm3 X = al, Y = be;
  double sa0 = 0.0, sb0 = 0.0;
  if (N > 0 && P.s_order > 0) {
    double ta[kMaxCoef], tb[kMaxCoef];
    sip_taylor<N>(C.sA, Uc, Vc, ta);
    sip_taylor<N>(C.sB, Uc, Vc, tb);
    sa0 = ta[0];
    sb0 = tb[0];
    // degree 1..3 in (dU, dV): Taylor-model powers of al, be
    tm_axpy<1, 3>(ta[tri9(1, 0)], al, X);
    tm_axpy<1, 3>(ta[tri9(0, 1)], be, X);
    tm_axpy<1, 3>(tb[tri9(1, 0)], al, Y);
    tm_axpy<1, 3>(tb[tri9(0, 1)], be, Y);
    if (N >= 2) {
      Tm3 p2[3];  // al^2, al be, be^2
      tm_mul<1, 3, 1, 3>(al, al, p2[0]);
      tm_mul<1, 3, 1, 3>(al, be, p2[1]);
      tm_mul<1, 3, 1, 3>(be, be, p2[2]);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        tm_axpy<2, 3>(ta[tri9(2 - i, i)], p2[i], X);
        tm_axpy<2, 3>(tb[tri9(2 - i, i)], p2[i], Y);
      }
      if (N >= 3) {
        Tm3 p3;  // al^(3-i) be^i
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (i == 0)
            tm_mul<2, 3, 1, 3>(p2[0], al, p3);
          else
            tm_mul<2, 3, 1, 3>(p2[i - 1], be, p3);
          tm_axpy<3, 3>(ta[tri9(3 - i, i)], p3, X);
          tm_axpy<3, 3>(tb[tri9(3 - i, i)], p3, Y);
        }
      }
    }
    // degree >= 4 in (dU, dV): bounded term by term
    const double A = tm_bound<1, 3>(al), B = tm_bound<1, 3>(be);
    double apow[N + 1], bpow[N + 1];
    apow[0] = bpow[0] = 1.0;
#pragma unroll
    for (int i = 1; i <= N; ++i) {
      apow[i] = apow[i - 1] * A;
      bpow[i] = bpow[i - 1] * B;
    }
#pragma unroll
    for (int i = 0; i <= N; ++i)
#pragma unroll
      for (int j = 0; i + j <= N; ++j)
        if (i + j >= 4) {
          X.r += __builtin_fabs(ta[tri9(i, j)]) * apow[i] * bpow[j];
          Y.r += __builtin_fabs(tb[tri9(i, j)]) * apow[i] * bpow[j];
        }
  }

  const double X0 = Uc + sa0 + P.scr[0], Y0 = Vc + sb0 + P.scr[1];
  if (!(__builtin_fabs(X0) < kFar) || !(__builtin_fabs(Y0) < kFar)) return;  // also rejects NaN
  const double fx = __builtin_floor(X0), fy = __builtin_floor(Y0);
  M.bx = (int32_t)fx;
  M.by = (int32_t)fy;
  // constant terms of al, be are zero: the constant is the centre's position
  X.c[0] = X0 - fx;
  Y.c[0] = Y0 - fy;
  double rx = 0.0, ry = 0.0, nlx = 0.0, nly = 0.0;
  const double hp[4] = {1.0, h, h * h, h * h * h};
#pragma unroll
  for (int k = 0; k < 10; ++k) {
    M.mx[k] = (float)X.c[k];
    M.my[k] = (float)Y.c[k];
    const double hd = hp[cm_i(k) + cm_j(k)];
    rx += __builtin_fabs((double)M.mx[k] - X.c[k]) * hd;
    ry += __builtin_fabs((double)M.my[k] - Y.c[k]) * hd;
    if (cm_i(k) + cm_j(k) >= 2) {
      nlx += __builtin_fabs((double)M.mx[k]) * hd;
      nly += __builtin_fabs((double)M.my[k]) * hd;
    }
  }
  // FP64 rounding of this construction, generously
  const double slack = 1.0e-12 * (1.0 + __builtin_fabs(Uc) + __builtin_fabs(Vc) + tm_bound<1, 3>(al) + tm_bound<1, 3>(be));
  const double tx = X.r + slack, ty = Y.r + slack;  // truncation of the map
  const double errx = tx + rx, erry = ty + ry;       // plus FP32 rounding of the coefficients
  const double err = __builtin_fmax(errx, erry);
  if (!(err < 1.0e6)) return;
  M.err = (float)(err * (1.0 + 1.0e-6));
  // The FP32 evaluation of the stored cubic (Horner's rule with fused
  // multiply-adds in b, then in a) is within gamma_6 * S of the cubic's exact
  // value, S = sum_k |m_k| h^(i+j) (the Horner bound gamma_n sum |c_j| |x|^j
  // for each level, composed), so an FP32 position is within
  // E = err + gamma_6 * S of the map; nearest decides the pixels within 2E of
  // a rounding tie in FP64.
  {
    double sx = 0.0, sy = 0.0;
#pragma unroll
    for (int k = 0; k < 10; ++k) {
      const double hd = hp[cm_i(k) + cm_j(k)];
      sx += __builtin_fabs((double)M.mx[k]) * hd;
      sy += __builtin_fabs((double)M.my[k]) * hd;
    }
    const double u = 0x1p-24, g6 = 6.0 * u / (1.0 - 6.0 * u);
    const double t = 2.0 * (err + g6 * __builtin_fmax(sx, sy)) * (1.0 + 1.0e-6);
    M.tie = (float)__builtin_fmin(0.5, __builtin_fmax(t, 1.0e-6));  // >= 1e-6: 0.5f - tie rounds by < 3e-8
  }
  M.ex = (float)((nlx + errx + kModelSlack) * (1.0 + 1.0e-6));
  M.ey = (float)((nly + erry + kModelSlack) * (1.0 + 1.0e-6));
  // the coefficient rounding is the FP32 evaluation error every FP32 path has
  // (the anchored chain rounds its own coefficients alike); the tolerance
  // applies to what the cubic leaves out of the map
  M.certified = __builtin_fmax(tx, ty) <= kModelTol ? 1 : 0;
}

// The coefficients of a frame copied into LDS by one wave (POLYS: 2 without,
// 4 with the target's).  From the plan the compiler reads them with scalar
// loads, and as the scalar registers hold few, in small pieces as it goes: 128
// waits in the order-5 kernel, several us of a wave's time.  From LDS they are
// vector loads in flight together.  Models of one image, order 5, target with
// SIP (2048^2): 7.5 -> 5.5 us; without (8192^2): 8.6 -> 8.0; of 64 frames on
// 8192^2: 195 -> 156.  Not in the launch whose groups make their own models
// (forward_tile): it measured the same either way.
template <int POLYS>
struct LdsCoefs {
  double c[POLYS][kMaxCoef];
  float f[2][kMaxCoef];  // the source's scaled FP32 copies (cell_out_of_reach)
};
template <int POLYS, class PlanPtr>
__device__ __forceinline__ SipCoefs stage_coefs(PlanPtr P, LdsCoefs<POLYS> &L) {
  const int lane = threadIdx.x & 63;
  if (lane < kMaxCoef) {
    L.c[0][lane] = P->sA[lane];
    L.c[1][lane] = P->sB[lane];
    L.f[0][lane] = P->fsA[lane];
    L.f[1][lane] = P->fsB[lane];
    if constexpr (POLYS == 4) {
      L.c[2][lane] = P->tA[lane];
      L.c[3][lane] = P->tB[lane];
    }
  }
  // the wave's own LDS accesses are performed in order
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  return SipCoefs{L.c[0], L.c[1], L.c[POLYS - 2], L.c[POLYS - 1]};
}

// A kernel's first argument, a plan by value, as the memory it is passed in
// (indexing the argument itself by lane would copy the plan to private memory).
__device__ __forceinline__ const __attribute__((address_space(4))) FramePlan *plan_argument() {
  return (const __attribute__((address_space(4))) FramePlan *)__builtin_amdgcn_kernarg_segment_ptr();
}

// Whether cell (cx, cy) of a target without SIP is certain to be found
// without a tap in the source by both tests that follow a model (its range
// grown by 4 px; without a certified model the anchor's test), from far fewer
// operations than the model: |dU| <= A over the cell, and |AP| there is at
// most SA = sum |c| (|Uc| + A)^p (|Vc| + B)^q, which bounds the constant and all
// Taylor terms of the model together, so its range lies within A + SA + 4 of
// the centre's affine position.  The anchor's test asks for kk < 1/2 (kap < 0.1
// implies it), a slope below 1/4 (the same majorant differentiated) and a
// distance of 64 |g| (1 + 2 L) + 12 at the cell's corner, where |g| is at most
// 1.5 times the centre's: 144 |g| + 12.
template <int SORD>
__device__ __forceinline__ bool cell_out_of_reach(const FramePlan &P,
                                                  const float (&f)[2][kMaxCoef], int cx, int cy) {
  constexpr int N = SORD >= 0 ? SORD : kMaxOrder;
  const double h = kHalfCell;
  const double *H = P.H;
  const double uc = (double)cx * kCell + h - P.tcr[0], vc = (double)cy * kCell + h - P.tcr[1];
  const double pc = fma(H[0], uc, fma(H[1], vc, H[2]));
  const double qc = fma(H[3], uc, fma(H[4], vc, H[5]));
  const double wc = fma(H[6], uc, fma(H[7], vc, H[8]));
  if (!(wc > 0.0)) return false;
  const double iw = 1.0 / wc;
  const double Uc = pc * iw, Vc = qc * iw;
  const float gs = (float)((fabs(H[0] - Uc * H[6]) + fabs(H[1] - Uc * H[7])) * iw);
  const float fs = (float)((fabs(H[3] - Vc * H[6]) + fabs(H[4] - Vc * H[7])) * iw);
  const float kap = (float)((fabs(H[6]) + fabs(H[7])) * iw * h);
  if (!(kap < 0.1f)) return false;
  const float A = gs * (float)h / (1.0f - kap), B = fs * (float)h / (1.0f - kap);
  const float sinv = (float)P.s_inv_scale;
  const float u = ((float)fabs(Uc) + A) * sinv, v = ((float)fabs(Vc) + B) * sinv;
  float sa = 0.0f, sb = 0.0f, slope = 0.0f;  // majorants of |AP|, |BP| and of all their slopes
  float up = 1.0f, upd = 0.0f;               // u^p, p u^(p-1)
#pragma unroll
  for (int p = 0; p <= N; ++p) {
    float vq = 1.0f, vqd = 0.0f;
#pragma unroll
    for (int q = 0; p + q <= N; ++q) {
      const float a = fabsf(f[0][tri9(p, q)]), b = fabsf(f[1][tri9(p, q)]);
      const float m = up * vq;
      sa = fmaf(a, m, sa);
      sb = fmaf(b, m, sb);
      slope = fmaf(a + b, fmaf(upd, vq, up * vqd), slope);
      vqd = fmaf(vqd, v, vq);
      vq *= v;
    }
    upd = fmaf(upd, u, up);
    up *= u;
  }
  if (!(slope * sinv < 0.24f)) return false;
  // FP32 rounding of the sums and positions, generously
  const float grow = 1.0f + 1.0e-4f;
  const float dx = (A + sa + 144.0f * gs) * grow + 24.0f + 1.0e-5f * (float)fabs(Uc);
  const float dy = (B + sb + 144.0f * fs) * grow + 24.0f + 1.0e-5f * (float)fabs(Vc);
  const double X = Uc + P.scr[0], Y = Vc + P.scr[1];
  return X + dx < 0.0 || X - dx > (double)(P.src_w - 1) || Y + dy < 0.0 ||
         Y - dy > (double)(P.src_h - 1);
}

}  // namespace dfr
