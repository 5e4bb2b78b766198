// The tiled forward kernels (single image, batch, coadd) as
// templates; each interpolation is instantiated in two translation units of
// its own (tiles_*.hip: single image; stacks_*.hip: the others) so the library
// builds in parallel.
#pragma once

#include "forward_tile.hpp"
#include "launch.hpp"

namespace dfr {

// Waves per SIMD the compiler is asked to leave registers for.
constexpr int tile_waves(int interp, int np) {
  return np >= 4 ? 4 : (interp == DFR_BICUBIC ? 6 : 8);
}

template <int INTERP, int SORD, int NP>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(tile_waves(INTERP, NP))))
void reproject_tiles(FramePlan P, TileGeom G) {
  extern __shared__ float lds[];
  __shared__ FwdShared sh;
  StoreSink sink;
  forward_tile<INTERP, SORD, NP>(P, G, xcd_tile(blockIdx.x, G.n_tiles), lds, sh, sink);
}

// The same with each group making the models of its own cells (32x32 and
// 64x16 tiles: one or two of them; 128x8 and 256x4, where they are asked for: four
// and eight, a lane each), for outputs of few tiles: one launch and no
// table.  The FP64 chain is then on every group's path, but while the groups
// are few they all run at once, so it costs its own latency (about 2 us) in
// place of a launch that waits for another one (256x256 bilinear: 15.2 us per
// call with the table, 12.4 so; 487x500 alignment step 43.6 and 40.1).
template <int INTERP, int SORD>
__global__ __launch_bounds__(kThreads) void reproject_small(FramePlan P, TileGeom G) {
  extern __shared__ float lds[];
  __shared__ FwdShared sh;
  StoreSink sink;
  forward_tile<INTERP, SORD, 1, true>(P, G, xcd_tile(blockIdx.x, G.n_tiles), lds, sh, sink);
}

// Order in which the work-groups of a batch take its items ((frame, tile)
// pairs): groups are dealt round-robin to the 8 XCDs, each with its own L2, so
// each XCD gets runs of `chunk` consecutive items (a few rows of tiles, which
// share source rows), and the runs go round the XCDs, turned by `turn` in each
// round, so work that varies over the target still spreads over the whole chip (the
// coadd; full-grid outputs of 24 frames took 707 us turned, 675 not turned).
// A permutation of 0 .. total - 1: the items past the last whole round keep
// their order.
__device__ __forceinline__ int batch_item(int b, int chunk, int turn, int total) {
  const int round = 8 * chunk, r = b / round;
  if ((r + 1) * (int64_t)round > total) return b;
  const int k = b - r * round;
  return r * round + ((k + turn * r) & 7) * chunk + (k >> 3);
}

// Batched reprojection: many source frames of uneven sizes onto one target
// grid in one launch (the paper's stacking use case, section 1), one
// work-group per (frame, tile) item; each item runs exactly the single-image
// tile body, so every frame's result is bit-identical to a single-image call.
// One group per item and not resident groups that loop over items: a group
// that ends with its stores never waits for them, while one that goes on has
// its next loads queue behind them (one in-order counter covers both), and the
// loop's state cost registers.  24 frames bicubic into their windows on
// 8192^2: 2,240 us looping, 1,400 us so; 24 frames
// bilinear as full 4096^2 images: 685 and 620 us.  (`first`: a batch beyond the launch
// limit takes several launches.)
template <int INTERP, int SORD, int NP>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(tile_waves(INTERP, NP))))
void reproject_batch(const FramePlan *__restrict__ plans, int first, int total, TileGeom G) {
  extern __shared__ float lds[];
  __shared__ FwdShared sh;
  const int item = batch_item(first + blockIdx.x, 4 * G.tiles_x, 0, total);
  const int frame = item / G.n_tiles;
  // read the frame table through the constant address space: it is not
  // written during the launch, so its fields can be scalar (SGPR) loads
  using ConstPlan = const __attribute__((address_space(4))) FramePlan;
  const FramePlan &P = *(const FramePlan *)((ConstPlan *)(plans + frame));
  const int tile = item - frame * G.n_tiles;
  StoreSink sink;
  // (also where frames cover all of the grid: without the look at the box the
  // launch of 24 frames bilinear on 4096^2 took 684 us instead of 606)
  if (tile_out_of_reach<NP>(P, G, tile))
    tile_uncovered<NP>(P, G, tile);  // most of a frame that covers part of the grid
  else
    forward_tile<INTERP, SORD, NP>(P, G, tile, lds, sh, sink);
}

// The batch into per-frame windows of the target grid (cropped outputs):
// frame i has items item0 .. item0 + (tiles of its window) - 1, the tiles of
// the global tile grid that meet its window, so every pixel is computed
// exactly as in the full batch; only the window's pixels are stored.
template <int INTERP, int SORD, int NP>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(tile_waves(INTERP, NP))))
void reproject_batch_cropped(const FramePlan *__restrict__ plans, int n_frames, int first,
                             int total, TileGeom G) {
  extern __shared__ float lds[];
  __shared__ FwdShared sh;
  using ConstPlan = const __attribute__((address_space(4))) FramePlan;
  const int item = batch_item(first + blockIdx.x, 4 * G.tiles_x, 0, total);
  // the last frame whose first item is <= item (frames without items share
  // the next frame's item0 and are passed over)
  int lo = 0, hi = n_frames - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (((ConstPlan *)(plans + mid))->item0 <= item)
      lo = mid;
    else
      hi = mid - 1;
  }
  const FramePlan &P = *(const FramePlan *)((ConstPlan *)(plans + lo));
  const int k = item - P.item0;
  const int tile = (P.tile0[1] + k / P.ntx) * G.tiles_x + P.tile0[0] + k % P.ntx;
  CropSink sink;
  forward_tile<INTERP, SORD, NP>(P, G, tile, lds, sh, sink);
}

// Coadd (stacking) of many frames onto one target grid, the paper's
// motivating use (section 1): per target pixel the sums over the frames of
// out * F and of F, and their ratio.  One work-group owns one target tile for
// the whole stack and visits the frames in index order, so the sums stay in
// registers, every output pixel is written once, and the result is
// deterministic (no atomics).  Each frame's per-pixel out and F are exactly
// those of a single-image call.
template <int INTERP, int SORD, int NP>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(NP >= 4 ? 3 : 4)))  // room for the sums
void coadd_tiles(const FramePlan *__restrict__ plans, int n_frames, TileGeom G, CoaddOut C) {
  extern __shared__ float lds[];
  __shared__ FwdShared sh;
  // Work per tile follows the stack's depth there, which varies across the
  // target (deep in the middle, zero at the edges): short runs of tiles, which
  // share source rows, go round the XCDs (contiguous per-XCD bands would leave
  // the XCDs holding the edges idle).  With the shorter DMA loop 64 frames on
  // 8192^2 take this kernel 2,260 us, from 2,690 with tile b for block b.
  const int tile = batch_item(blockIdx.x, 16, 1, G.n_tiles);
  const int lg = G.txt_log2;
  const int TW = kRun << lg, RP = kThreads >> lg, TH = RP * NP;
  const int trow = tile / G.tiles_x;
  const int x0 = (tile - trow * G.tiles_x) * TW, y0 = trow * TH;
  const int ty = threadIdx.x >> lg, xr = x0 + (threadIdx.x & ((1 << lg) - 1)) * kRun;
  StackSink<NP> acc;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int y = y0 + ty + k * RP;
    const int64_t off = (int64_t)y * G.out_w + xr;
#pragma unroll
    for (int e = 0; e < kRun; ++e) {
      const bool in = C.accumulate && y < G.out_h && xr + e < G.out_w;
      acc.s[k][e] = in ? C.sum_wf[off + e] : 0.0f;
      acc.w[k][e] = in ? C.sum_f[off + e] : 0.0f;
    }
  }
  using ConstPlan = const __attribute__((address_space(4))) FramePlan;
#pragma unroll 1
  for (int i = 0; i < n_frames; ++i) {
    const FramePlan &P = *(const FramePlan *)((ConstPlan *)(plans + i));
    if (tile_out_of_reach<NP>(P, G, tile)) continue;  // uniform over the group
    forward_tile<INTERP, SORD, NP>(P, G, tile, lds, sh, acc);
    __syncthreads();  // LDS and the per-tile state are reused by the next frame
  }
  const float miss = G.nan_outside ? __builtin_nanf("") : 0.0f;
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    const int y = y0 + ty + k * RP;
    if (y >= G.out_h || xr >= G.out_w) continue;
    const int64_t off = (int64_t)y * G.out_w + xr;
    store_run(C.sum_wf, off, xr, G.out_w, acc.s[k]);
    store_run(C.sum_f, off, xr, G.out_w, acc.w[k]);
    if (C.coadd) {
      float q[kRun];
#pragma unroll
      for (int e = 0; e < kRun; ++e) q[e] = acc.w[k][e] > 0.0f ? acc.s[k][e] / acc.w[k][e] : miss;
      store_run(C.coadd, off, xr, G.out_w, q);
    }
  }
}

// Source SIP orders 0..5 have compile-time kernels; higher orders, and any
// target with SIP A/B (sord < 0 here), use the run-time-order kernel.
template <template <int, int, int> class K, int INTERP, int NP>
const void *pick_sord(int sord) {
  switch (sord) {
    case 0: return K<INTERP, 0, NP>::ptr();
    case 1: return K<INTERP, 1, NP>::ptr();
    case 2: return K<INTERP, 2, NP>::ptr();
    case 3: return K<INTERP, 3, NP>::ptr();
    case 4: return K<INTERP, 4, NP>::ptr();
    case 5: return K<INTERP, 5, NP>::ptr();
    default: return K<INTERP, kRtOrder, NP>::ptr();
  }
}

template <int INTERP, int SORD, int NP>
struct TileK {
  static const void *ptr() { return reinterpret_cast<const void *>(reproject_tiles<INTERP, SORD, NP>); }
};
template <int INTERP, int SORD, int NP>
struct SmallK {
  static const void *ptr() { return reinterpret_cast<const void *>(reproject_small<INTERP, SORD>); }
};
template <int INTERP, int SORD, int NP>
struct BatchK {
  static const void *ptr() { return reinterpret_cast<const void *>(reproject_batch<INTERP, SORD, NP>); }
};

template <int INTERP, int SORD, int NP>
struct CropK {
  static const void *ptr() { return reinterpret_cast<const void *>(reproject_batch_cropped<INTERP, SORD, NP>); }
};
template <int INTERP, int SORD, int NP>
struct CoaddK {
  static const void *ptr() { return reinterpret_cast<const void *>(coadd_tiles<INTERP, SORD, NP>); }
};

// Kernel for (rows per thread, source SIP order) of one interpolation.
template <int INTERP>
const void *tile_kernel_for(int np, int sord) {
  switch (np) {
    case 1: return pick_sord<TileK, INTERP, 1>(sord);
    case 2: return pick_sord<TileK, INTERP, 2>(sord);
    default: return pick_sord<TileK, INTERP, 4>(sord);
  }
}

// reproject_small for source orders 0 .. 5.
template <int INTERP>
const void *small_kernel_for(int sord) {
  switch (sord) {
    case 0: return SmallK<INTERP, 0, 1>::ptr();
    case 1: return SmallK<INTERP, 1, 1>::ptr();
    case 2: return SmallK<INTERP, 2, 1>::ptr();
    case 3: return SmallK<INTERP, 3, 1>::ptr();
    case 4: return SmallK<INTERP, 4, 1>::ptr();
    default: return SmallK<INTERP, 5, 1>::ptr();
  }
}

template <int INTERP>
const void *batch_kernel_for(int np, int sord) {
  switch (np) {
    case 1: return pick_sord<BatchK, INTERP, 1>(sord);
    case 2: return pick_sord<BatchK, INTERP, 2>(sord);
    default: return pick_sord<BatchK, INTERP, 4>(sord);
  }
}

template <int INTERP>
const void *crop_kernel_for(int np, int sord) {
  switch (np) {
    case 1: return pick_sord<CropK, INTERP, 1>(sord);
    case 2: return pick_sord<CropK, INTERP, 2>(sord);
    default: return pick_sord<CropK, INTERP, 4>(sord);
  }
}

template <int INTERP>
const void *coadd_kernel_for(int np, int sord) {
  switch (np) {
    case 1: return pick_sord<CoaddK, INTERP, 1>(sord);
    case 2: return pick_sord<CoaddK, INTERP, 2>(sord);
    default: return pick_sord<CoaddK, INTERP, 4>(sord);
  }
}

extern template const void *tile_kernel_for<DFR_NEAREST>(int, int);
extern template const void *tile_kernel_for<DFR_BILINEAR>(int, int);
extern template const void *tile_kernel_for<DFR_BICUBIC>(int, int);
extern template const void *small_kernel_for<DFR_NEAREST>(int);
extern template const void *small_kernel_for<DFR_BILINEAR>(int);
extern template const void *small_kernel_for<DFR_BICUBIC>(int);
extern template const void *batch_kernel_for<DFR_NEAREST>(int, int);
extern template const void *batch_kernel_for<DFR_BILINEAR>(int, int);
extern template const void *batch_kernel_for<DFR_BICUBIC>(int, int);
extern template const void *crop_kernel_for<DFR_NEAREST>(int, int);
extern template const void *crop_kernel_for<DFR_BILINEAR>(int, int);
extern template const void *crop_kernel_for<DFR_BICUBIC>(int, int);
extern template const void *coadd_kernel_for<DFR_NEAREST>(int, int);
extern template const void *coadd_kernel_for<DFR_BILINEAR>(int, int);
extern template const void *coadd_kernel_for<DFR_BICUBIC>(int, int);

}  // namespace dfr
