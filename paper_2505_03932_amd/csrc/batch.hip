// Launch helpers of the batch and the coadd kernels (defined in
// tile_kernels.hpp).
#include "tile_kernels.hpp"

#include <algorithm>

namespace dfr {

const void *batch_kernel_ptr(int interp, int np, int sord) {
  return interp == DFR_NEAREST    ? batch_kernel_for<DFR_NEAREST>(np, sord)
         : interp == DFR_BILINEAR ? batch_kernel_for<DFR_BILINEAR>(np, sord)
                                  : batch_kernel_for<DFR_BICUBIC>(np, sord);
}

const void *crop_kernel_ptr(int interp, int np, int sord) {
  return interp == DFR_NEAREST    ? crop_kernel_for<DFR_NEAREST>(np, sord)
         : interp == DFR_BILINEAR ? crop_kernel_for<DFR_BILINEAR>(np, sord)
                                  : crop_kernel_for<DFR_BICUBIC>(np, sord);
}

const void *coadd_kernel_ptr(int interp, int np, int sord) {
  return interp == DFR_NEAREST    ? coadd_kernel_for<DFR_NEAREST>(np, sord)
         : interp == DFR_BILINEAR ? coadd_kernel_for<DFR_BILINEAR>(np, sord)
                                  : coadd_kernel_for<DFR_BICUBIC>(np, sord);
}

// One work-group per item; a launch has fewer than 2^32 threads.
static hipError_t launch_items(const void *kernel, int total, int &first, void **args, size_t lds,
                               hipStream_t stream) {
  for (first = 0; first < total; first += kBatchItems) {
    const hipError_t e = launch_kernel(kernel, dim3(std::min(total - first, kBatchItems)),
                                       dim3(kThreads), args, lds, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_batch_f32(const FramePlan *plans_dev, int n_frames, int max_sord,
                            const TileGeom &G, int interp, int np, hipStream_t stream) {
  int first = 0, total = n_frames * G.n_tiles;
  TileGeom geom = G;
  void *args[] = {&plans_dev, &first, &total, &geom};
  return launch_items(batch_kernel_ptr(interp, np, max_sord), total, first, args,
                      (size_t)G.lds_cap * sizeof(float), stream);
}

hipError_t launch_batch_cropped(const FramePlan *plans_dev, int n_frames, int total, int max_sord,
                                const TileGeom &G, int interp, int np, hipStream_t stream) {
  int first = 0;
  TileGeom geom = G;
  void *args[] = {&plans_dev, &n_frames, &first, &total, &geom};
  return launch_items(crop_kernel_ptr(interp, np, max_sord), total, first, args,
                      (size_t)G.lds_cap * sizeof(float), stream);
}

hipError_t launch_coadd_f32(const FramePlan *plans_dev, int n_frames, int max_sord,
                            const TileGeom &G, int interp, int np, const CoaddOut &C,
                            hipStream_t stream) {
  using CoaddKernel = void (*)(const FramePlan *, int, TileGeom, CoaddOut);
  CoaddKernel k = reinterpret_cast<CoaddKernel>(const_cast<void *>(coadd_kernel_ptr(interp, np, max_sord)));
  size_t lds = (size_t)G.lds_cap * sizeof(float);
  hipLaunchKernelGGL(k, dim3(G.n_tiles), dim3(kThreads), lds, stream, plans_dev, n_frames, G, C);
  return hipGetLastError();
}

}  // namespace dfr
