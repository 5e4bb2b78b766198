// Host-side launch helpers shared by the translation units of libdfr.
#pragma once

#include <hip/hip_runtime.h>

#include "common.hpp"

namespace dfr {

// Tile shapes: id 1..kTileCount.  id-1 = li*3 + ni with threads-per-row
// 8 << li (tile width 32 << li px) and NP = 1 << ni rows per thread.
constexpr int kTileCount = 12;
constexpr int kDefaultTile = 5;  // 64 x 32
constexpr int kCoaddTile = 5;    // coadd default
constexpr int kSquareTile = 6;   // 64 x 64, four rows per thread
constexpr int kFlatTile = 8;     // 128 x 16

// Untuned default tile of the forward kernels for n images of out_h x out_w
// (1 for a single image or a plan).  Tile kernel alone, us, by tile shape:
//                         32x32  64x16  64x32  32x64  128x16
//   256^2      bilinear     6.4    6.3    8.9    9.1    9.1
//   256^2      bicubic      8.5    8.2   13.5   13.2   13.9
//   2048^2     nearest     18.2   18.5   15.9   15.1   16.2
//   2048^2     bilinear    14.5   14.8   17.4   14.8   17.6
//   2048^2     bicubic     19.0   20.2   21.0   20.0   25.8
//   2900x2400  bilinear    25.8   21.3   25.6   33.4   22.9
//   2900x2400  bicubic     29.5   28.6   30.0   37.0   35.1
//   5003x3301  bicubic     76.1   69.5   65.8   96.6   70.0
//   6000x4000  bilinear    76.8   73.2   67.1   71.7   64.6
//   6000x4000  bicubic     94.7   98.8   79.3   76.3   96.1
// Up to a few rounds of groups on the chip (256 CUs x 8 groups x 1024 pixels a
// round) a call is as long as one group's chain of phases: the smallest tiles,
// one row per thread, win (nearest, with the least to do per pixel, only below
// one round).  Beyond, bytes count: tiles with fewer halo rows, and wide ones
// where output rows are not multiples of 128 bytes (a narrow tile then splits
// a line at both ends of every row).
inline int forward_default_tile(int interp, int64_t n, int64_t out_h, int64_t out_w) {
  const int64_t px = n * out_h * out_w;
  const bool lines = (out_w & 31) == 0;
  if (px <= (interp == DFR_NEAREST ? int64_t(1) << 20 : int64_t(1) << 23)) return lines ? 1 : 4;
  return interp == DFR_BICUBIC ? (lines ? 2 : kDefaultTile) : kFlatTile;
}
// The backward's, measured on the 2048^2 bicubic and 6000x4000 bilinear
// cases: 64 x 16 (one row per thread) for bicubic with the source gradient
// (its LDS adds), else 64 x 32.
inline int backward_default_tile(int interp, bool src_grad) {
  return interp == DFR_BICUBIC && src_grad ? 4 : kDefaultTile;
}

struct TileShape {
  int txt_log2;  // threads per tile row, log2
  int np;        // rows per thread
  int width, height;
};

inline bool tile_shape(int id, TileShape &s) {
  if (id < 1 || id > kTileCount) return false;
  int li = (id - 1) / 3, ni = (id - 1) % 3;
  s.txt_log2 = 3 + li;
  s.np = 1 << ni;
  s.width = kRun << s.txt_log2;
  s.height = (kThreads >> s.txt_log2) * s.np;
  return true;
}

// Extra per-frame data the FP64 comparison forms need (trig form: the
// explicit two-stage formulas of section 3.2).
struct TrigPlan {
  double tcd[4];     // target CD (deg/px)
  double scdi[4];    // inverse of the source CD (px/deg)
  double tcrval[2];  // target (RA, Dec) in radians
  double scrval[2];  // source (RA, Dec) in radians
};

// Launch a kernel by its address.  A failure is returned and also taken from the
// runtime, whose last error would otherwise fail the next checked launch.
inline hipError_t launch_kernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t lds,
                                hipStream_t stream) {
  const hipError_t e = hipLaunchKernel(kernel, grid, block, args, lds, stream);
  if (e != hipSuccess) (void)hipGetLastError();
  return e;
}

hipError_t launch_forward_f32(const FramePlan &P, const TileGeom &G, int interp, int np,
                              hipStream_t stream);
// Whether a call with cell models takes the one-launch form for few tiles
// (launch_forward_small, no model table): tiles of one row per thread, up to
// the groups that run at once beside the FP64 registers: three per CU and 768
// where the instance takes at most 170 of them (orders 0 to 4), two and 512 at
// order 5 (182 to 184).  Above, a second round of groups pays the models' chain
// again.  us per call at order 5, nearest, bilinear, bicubic: one launch at 704^2
// (484 groups) 13.7, 10.9, 13.2; at 768^2 (576) 16.8, 13.4, 16.5 and with the
// table 14.4, 13.1, 13.5.  At order 4 one launch at 864^2 (729) 12.2, 11.0, 13.6,
// the table at 880^2 (784) 13.7, 13.0, 13.8.
constexpr int kSmallTiles = 768;
constexpr int kSmallTilesOrder5 = 512;
bool forward_small(const FramePlan &P, const TileGeom &G, int np);
hipError_t launch_forward_small(const FramePlan &P, const TileGeom &G, int interp,
                                hipStream_t stream);
// Per-cell position models of the output grid (ncx x ncy cells of 32x32).
hipError_t launch_cell_models(const FramePlan &P, int ncx, int ncy, CellModel *out,
                              hipStream_t stream);
// Kernel (plans, ncx, ncy, bcols, bpf, out, parts) modelling every cell of
// every frame of a batch, bpf blocks of 8x8 cells per frame, bcols to a row; sord as for the batch
// kernel, tord the target SIP order.
const void *cell_models_batch_ptr(int sord, int tord);
// Kernel (plans, parts, bpf) folding its blocks' reach boxes, a group per frame.
const void *reach_kernel_ptr();
hipError_t launch_forward_f64(const FramePlan &P, const TrigPlan &T, const TileGeom &G,
                              int interp, bool trig, hipStream_t stream);
hipError_t launch_batch_f32(const FramePlan *plans_dev, int n_frames, int max_sord,
                            const TileGeom &G, int interp, int np, hipStream_t stream);
const void *batch_kernel_ptr(int interp, int np, int sord);
// The batch into per-frame windows (FramePlan crop, item0, tile0, ntx):
// `total` items over the frames.
hipError_t launch_batch_cropped(const FramePlan *plans_dev, int n_frames, int total, int max_sord,
                                const TileGeom &G, int interp, int np, hipStream_t stream);
// Coadd of a frame table: one work-group per target tile (G.n_tiles).
hipError_t launch_coadd_f32(const FramePlan *plans_dev, int n_frames, int max_sord,
                            const TileGeom &G, int interp, int np, const CoaddOut &C,
                            hipStream_t stream);
constexpr int kBatchItems = 1 << 23;  // items of one launch of a batch kernel
// Number of per-tile FP64 partial sums the backward kernel produces for a
// source SIP order (9 for H, 2 for CRPIX, AP and BP monomial sums).
inline int backward_sums(int s_order) { return 11 + (s_order + 1) * (s_order + 2); }

struct WcsJacobian {
  double dh[54];  // dH_i / d theta_k at [k * 9 + i], theta = CRVAL1..2, CD1_1..CD2_2
};

// src_acc non-null: the source adjoint too, as integer sums into src_acc
// [src_h][src_w] (zeroed by launch_bwd_prepare), quantised with the scale
// from max|g| in gmax_bits; launch_backward_finish then writes grad_src.
hipError_t launch_backward(const FramePlan &P, const TileGeom &G, int interp, int np,
                           const float *grad_out, double *partials, unsigned long long *src_acc,
                           const int *gmax_bits, const Anchor *anchors, hipStream_t stream);
// What precedes it: the cells' anchors (anchors non-null), and for the source
// adjoint (q non-null) q[0 .. nq) and *gmax_next zeroed and max |g| folded into
// *gmax (which must start at 0).
hipError_t launch_bwd_prepare(const FramePlan &P, const TileGeom &G, int interp, Anchor *anchors,
                              const float *grad_out, int64_t n, unsigned long long *q, int64_t nq,
                              int *gmax, int *gmax_next, hipStream_t stream);
// A backward call without the source adjoint needs that launch only for the
// anchors: above this many tiles it pays (one round of groups on the chip).
constexpr int kBwdAnchorTiles = 1024;
// What follows the backward kernel: the WCS partials reduced and chained
// into grad_wcs (nr = ns - 10 blocks when grad_wcs is wanted, else 0), and
// the integer sums q (if non-null) converted into grad_src with the scale
// from *gmax.
constexpr int kBwdMaxOrder = 5;  // highest source SIP order the backward takes
constexpr int kBwdSipCols = (kBwdMaxOrder + 1) * (kBwdMaxOrder + 2);  // AP and BP
constexpr int kBwdSipEntries = 2 * (kBwdMaxOrder + 1) * (kBwdMaxOrder + 1);
struct FinishArgs {
  const double *partials;
  int n_blocks, ns, nr;
  WcsJacobian J;
  double S;
  double *grad_wcs;
  int col_entry[kBwdSipCols];   // grad entry of SIP column 11 + k, or -1
  int col_deg[kBwdSipCols];     // its p + q
  int above[kBwdSipEntries];    // grad entries above their polynomial's order
  int n_above;
  const unsigned long long *q;
  int64_t h, w;
  float *gsrc;
  int64_t gpitch;
  const int *gmax;
};
hipError_t launch_backward_finish(const FinishArgs &args, hipStream_t stream);
hipError_t launch_zero_i32(int *p, int64_t n, hipStream_t stream);
hipError_t launch_sq_residual(const float *out, const float *ref, const float *mask, int64_t n,
                              double *partials, int n_blocks, double *loss, float *grad_out,
                              hipStream_t stream);

}  // namespace dfr
