// Launchers and small kernels of the backward pass (the tile kernel is in
// backward_tile.hpp) and the alignment loss.
#include "backward_tile.hpp"

namespace dfr {

hipError_t launch_backward(const FramePlan &P, const TileGeom &G, int interp, int np,
                           const float *grad_out, double *partials, unsigned long long *src_acc,
                           const int *gmax_bits, const Anchor *anchors, hipStream_t stream) {
  if (G.n_tiles <= 0) return hipSuccess;
  const bool tsip = P.t_order > 0;
  const bool src = src_acc != nullptr;
  BwdKernel k = interp == DFR_NEAREST    ? bwd_pick<DFR_NEAREST>(np, P.s_order, tsip, src)
                : interp == DFR_BILINEAR ? bwd_pick<DFR_BILINEAR>(np, P.s_order, tsip, src)
                                         : bwd_pick<DFR_BICUBIC>(np, P.s_order, tsip, src);
  size_t lds = (size_t)G.lds_cap * sizeof(float);
  hipLaunchKernelGGL(k, dim3(G.n_tiles), dim3(kThreads), lds, stream, P, G, grad_out, partials,
                     src_acc, gmax_bits, anchors);
  return hipGetLastError();
}

// Before the backward kernel, in one launch:
//  - the first nab blocks: the FP64 anchor of every cell, a lane each, into
//    `anchors`.  Computed by the tiles themselves, two lanes of one wave ran
//    that chain (about 1,500 instructions) in every group, with the other
//    waves waiting (2048^2 bicubic: backward kernel 68.6 us that way, 64.2 so;
//    4000x3000 bilinear 158 and 149);
//  - the others, for the source adjoint: the 64-bit integer image is zeroed
//    and max |g| over the output gradient is folded into *gmax as the bits of
//    a non-negative float (their integer order is the float order, so atomicMax
//    gives the same result in any order).  *gmax is 0 on entry; *gmax_next, the
//    slot the next call uses, is zeroed here (the previous call's kernels,
//    which read it, have finished).
template <int SORD, bool TSIP>
__global__ __launch_bounds__(256) void bwd_prepare_kernel(FramePlan P, int ncx, int ncells,
                                                          int support, int nab,
                                                          Anchor *__restrict__ anchors,
                                                          const float *__restrict__ g, int64_t n,
                                                          unsigned long long *__restrict__ q,
                                                          int64_t nq, int *__restrict__ gmax,
                                                          int *__restrict__ gmax_next) {
  if ((int)blockIdx.x < nab) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= ncells) return;
    const int cy = i / ncx, cx = i - cy * ncx;
    Anchor A = Anchor{};
    compute_anchor<SORD, TSIP>(P, cx * kCell, cy * kCell, support, A);
    anchors[i] = A;
    return;
  }
  __shared__ float wm[4];
  const int64_t stride = (int64_t)(gridDim.x - nab) * 256;
  const int64_t i0 = (int64_t)(blockIdx.x - nab) * 256 + threadIdx.x;
  if (i0 == 0) *gmax_next = 0;
  // the image is 16-byte aligned (a 256-byte aligned workspace offset)
  typedef unsigned long long u2v __attribute__((ext_vector_type(2)));
#pragma unroll 4
  for (int64_t i = i0; i < nq / 2; i += stride) reinterpret_cast<u2v *>(q)[i] = u2v{0ull, 0ull};
  if (i0 == 0 && (nq & 1)) q[nq - 1] = 0ull;
  float m = 0.0f;
  // 16-byte loads where the gradient is aligned, then the tail
  typedef float f4v __attribute__((ext_vector_type(4)));
  const int64_t n4 = (reinterpret_cast<uintptr_t>(g) & 15) == 0 ? n / 4 : 0;
#pragma unroll 4
  for (int64_t i = i0; i < n4; i += stride) {
    const f4v v = reinterpret_cast<const f4v *>(g)[i];
    m = fmaxf(fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w)));
  }
  for (int64_t i = 4 * n4 + i0; i < n; i += stride) m = fmaxf(m, fabsf(g[i]));
  m = wave_max_f(m);
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = fmaxf(fmaxf(wm[0], wm[1]), fmaxf(wm[2], wm[3]));
    // one atomic per block, few blocks: atomics on one address serialise
    if (m > 0.0f) atomicMax(gmax, __float_as_int(m));
  }
}

template <bool TSIP>
static const void *prepare_pick(int sord) {
  switch (sord) {
    case 0: return reinterpret_cast<const void *>(bwd_prepare_kernel<0, TSIP>);
    case 1: return reinterpret_cast<const void *>(bwd_prepare_kernel<1, TSIP>);
    case 2: return reinterpret_cast<const void *>(bwd_prepare_kernel<2, TSIP>);
    case 3: return reinterpret_cast<const void *>(bwd_prepare_kernel<3, TSIP>);
    case 4: return reinterpret_cast<const void *>(bwd_prepare_kernel<4, TSIP>);
    default: return reinterpret_cast<const void *>(bwd_prepare_kernel<5, TSIP>);
  }
}

hipError_t launch_bwd_prepare(const FramePlan &P, const TileGeom &G, int interp, Anchor *anchors,
                              const float *grad_out, int64_t n, unsigned long long *q, int64_t nq,
                              int *gmax, int *gmax_next, hipStream_t stream) {
  int ncx = (G.out_w + kCell - 1) / kCell, ncells = ncx * ((G.out_h + kCell - 1) / kCell);
  int nab = anchors ? (ncells + 255) / 256 : 0;
  int support = interp == DFR_NEAREST ? 0 : (interp == DFR_BILINEAR ? 1 : 2);
  const int64_t work = std::max<int64_t>(n / 4, nq / 2);
  const int blocks = q ? (int)std::min<int64_t>(512, std::max<int64_t>(1, (work + 255) / 256)) : 0;
  if (nab + blocks == 0) return hipSuccess;
  FramePlan plan = P;
  void *args[] = {&plan, &ncx, &ncells, &support, &nab, &anchors,
                  &grad_out, &n, &q, &nq, &gmax, &gmax_next};
  const void *k = P.t_order > 0 ? prepare_pick<true>(P.s_order) : prepare_pick<false>(P.s_order);
  return launch_kernel(k, dim3(nab + blocks), dim3(256), args, 0, stream);
}

// Column c of the partials ([ns][n_blocks], column-major), summed by one
// block in a fixed order (256 strided partial sums, then a tree); the
// result is in sm[0].
__device__ __forceinline__ void column_sum(const FinishArgs &A, int c, double *sm) {
  const int tid = threadIdx.x;
  double a = 0.0;
  const double *col = A.partials + (int64_t)c * A.n_blocks;
#pragma unroll 4
  for (int k = tid; k < A.n_blocks; k += 256) a += col[k];
  sm[tid] = a;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) sm[tid] += sm[tid + w];
    __syncthreads();
  }
}

// After the backward kernel, in one launch with no block depending on
// another.  With WCS gradients (nr = ns - 10 blocks): block 0 sums the nine
// dH and two CRPIX columns and applies the chain rule to CRVAL, CRPIX and CD
// (dH/dtheta), and writes the AP/BP entries of the square layouts that lie
// above their order (zero); block 1 + k sums SIP column 11 + k and writes its
// entry, scaled by S^(p+q) (A.col_entry / A.col_deg; -1: a padded column).
// The remaining blocks convert rows of the integer sums to grad_src =
// q 2^-Q.  Grad entries follow dfr_wcs_grad_size: CRVAL(2), CRPIX(2), CD(4),
// AP, BP.
__global__ __launch_bounds__(256) void bwd_finish_kernel(FinishArgs A) {
  __shared__ double sm[11 * 256];
  __shared__ double tot[11];
  const int b = blockIdx.x, tid = threadIdx.x;
  if (b >= A.nr) {
    const double inv = 1.0 / det_scale(A.gmax);
    const int nc = (int)gridDim.x - A.nr;
    for (int64_t r = b - A.nr; r < A.h; r += nc) {
      const unsigned long long *qr = A.q + r * A.w;
      float *gr = A.gsrc + r * A.gpitch;
      for (int64_t c = tid; c < A.w; c += 256) gr[c] = (float)((double)(long long)qr[c] * inv);
    }
    return;
  }
  if (b > 0) {
    const int k = b - 1;
    column_sum(A, 11 + k, sm);
    if (tid == 0 && A.col_entry[k] >= 0) {
      double sc = 1.0;
      for (int i = 0; i < A.col_deg[k]; ++i) sc *= A.S;
      A.grad_wcs[A.col_entry[k]] = sm[0] * sc;
    }
    return;
  }
  // the 11 leading columns side by side (one load of each per row, so
  // eleven are in flight together), then 11 trees side by side
  double a[11];
#pragma unroll
  for (int c = 0; c < 11; ++c) a[c] = 0.0;
  const int64_t nb = A.n_blocks;
#pragma unroll 2
  for (int k = tid; k < A.n_blocks; k += 256) {
#pragma unroll
    for (int c = 0; c < 11; ++c) a[c] += A.partials[c * nb + k];
  }
#pragma unroll
  for (int c = 0; c < 11; ++c) sm[c * 256 + tid] = a[c];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (tid < w) {
#pragma unroll
      for (int c = 0; c < 11; ++c) sm[c * 256 + tid] += sm[c * 256 + tid + w];
    }
    __syncthreads();
  }
  if (tid < 11) tot[tid] = sm[tid * 256];
  __syncthreads();
  if (tid < 8) {
    if (tid < 2 || tid >= 4) {
      // CRVAL_k (tid < 2) or CD_kl (tid = 4 + kl) through dH/dtheta
      const int row = tid < 2 ? tid : 2 + (tid - 4);
      double g = 0.0;
      for (int i = 0; i < 9; ++i) g += tot[i] * A.J.dh[row * 9 + i];
      A.grad_wcs[tid] = g;
    } else {
      A.grad_wcs[tid] = tot[9 + (tid - 2)];  // CRPIX
    }
  }
  for (int t = tid; t < A.n_above; t += 256) A.grad_wcs[A.above[t]] = 0.0;
}

hipError_t launch_backward_finish(const FinishArgs &A, hipStream_t stream) {
  const int nc = A.q ? (int)std::min<int64_t>(2048, A.h) : 0;
  if (A.nr + nc == 0) return hipSuccess;
  hipLaunchKernelGGL(bwd_finish_kernel, dim3(A.nr + nc), dim3(256), 0, stream, A);
  return hipGetLastError();
}

// ------------------------------------------------------ alignment loss

__global__ __launch_bounds__(256) void sq_residual_kernel(const float *__restrict__ out,
                                                          const float *__restrict__ ref,
                                                          const float *__restrict__ mask,
                                                          int64_t n, double *__restrict__ partials,
                                                          float *__restrict__ gout) {
  __shared__ double ws[4];
  double acc = 0.0;
  // four elements per step with 16-byte loads and stores when every buffer
  // is 16-byte aligned; element by element otherwise and for the tail
  typedef float f4v __attribute__((ext_vector_type(4)));
  const bool vec = ((reinterpret_cast<uintptr_t>(out) | reinterpret_cast<uintptr_t>(ref) |
                     reinterpret_cast<uintptr_t>(mask) | reinterpret_cast<uintptr_t>(gout)) &
                    15) == 0;
  const int64_t n4 = vec ? n / 4 : 0;
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride) {
    const f4v o = reinterpret_cast<const f4v *>(out)[i];
    const f4v r0 = reinterpret_cast<const f4v *>(ref)[i];
    const f4v m = mask ? reinterpret_cast<const f4v *>(mask)[i] : (f4v){1.0f, 1.0f, 1.0f, 1.0f};
    const f4v r = o - r0;
    acc += (double)m.x * (double)r.x * (double)r.x;
    acc += (double)m.y * (double)r.y * (double)r.y;
    acc += (double)m.z * (double)r.z * (double)r.z;
    acc += (double)m.w * (double)r.w * (double)r.w;
    if (gout) reinterpret_cast<f4v *>(gout)[i] = 2.0f * m * r;
  }
  for (int64_t i = 4 * n4 + (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    float r = out[i] - ref[i];
    float m = mask ? mask[i] : 1.0f;
    acc += (double)m * (double)r * (double)r;
    if (gout) gout[i] = 2.0f * m * r;
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

__global__ __launch_bounds__(256) void sum_partials_kernel(const double *__restrict__ partials,
                                                           int n, double *__restrict__ loss) {
  __shared__ double sm[256];
  double a = 0.0;
  for (int b = threadIdx.x; b < n; b += 256) a += partials[b];
  sm[threadIdx.x] = a;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = sm[0];
}

hipError_t launch_sq_residual(const float *out, const float *ref, const float *mask, int64_t n,
                              double *partials, int n_blocks, double *loss, float *grad_out,
                              hipStream_t stream) {
  hipLaunchKernelGGL(sq_residual_kernel, dim3(n_blocks), dim3(256), 0, stream, out, ref, mask, n,
                     partials, grad_out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, stream, partials, n_blocks,
                     loss);
  return hipGetLastError();
}

}  // namespace dfr
