// Window sums and a fixed-order reduction of FP64 planes, for the FLR adjoint.
//
// The adjoint recomputes the window moments as FP64 sums of anchored input
// products, and sums its per-pixel fields over the same clipped window (the
// window sum is its own adjoint). The window-sum tile is box_tile
// (flr_box.hpp): one workgroup per strip of kThreads input columns of one
// plane and segment of rows, running vertical sums per lane, horizontal sums
// by segmented prefixes.
#include <hip/hip_runtime.h>

#include "flr_avg.hpp"
#include "flr_box.hpp"
#include "flr_launch.hpp"
#include "flr_prefix.hpp"

namespace flr {

template <int SRC, bool WIDE, bool RING>
__global__ void __launch_bounds__(256) adj_box_kernel(AdjBoxArgs a) {
  box_tile<SRC, WIDE, RING>(a, blockIdx.x, blockIdx.y);
}

struct AdjPairArgs {
  const double* src;
  double* dst;
  int n;
};

__global__ void __launch_bounds__(256) adj_pair_sum_kernel(AdjPairArgs a) {
  extern __shared__ float lds[];
  double* part = reinterpret_cast<double*>(lds);  // [2][kThreads]
  const int tid = threadIdx.x;
  double s0 = 0.0, s1 = 0.0;
  for (int i = tid; i < a.n; i += kThreads) {
    s0 += a.src[2 * i];
    s1 += a.src[2 * i + 1];
  }
  part[tid] = s0;
  part[kThreads + tid] = s1;
  __syncthreads();
  for (int s = kThreads / 2; s > 0; s >>= 1) {
    if (tid < s) {
      part[tid] += part[tid + s];
      part[kThreads + tid] += part[kThreads + tid + s];
    }
    __syncthreads();
  }
  if (tid == 0) {
    a.dst[0] = part[0];
    a.dst[1] = part[kThreads];
  }
}

template <bool WIDE, bool RING>
static void box_dispatch(const AdjBoxArgs& a, dim3 grid, size_t lds, hipStream_t s) {
  if (a.srcf)
    hipLaunchKernelGGL((adj_box_kernel<BOX_MEAN32, WIDE, RING>), grid, dim3(kThreads), lds, s, a);
  else if (a.src && a.count_first)  // count_first marks a mean of FP64 planes here
    hipLaunchKernelGGL((adj_box_kernel<BOX_MEAN64, WIDE, RING>), grid, dim3(kThreads), lds, s, a);
  else if (a.src)
    hipLaunchKernelGGL((adj_box_kernel<BOX_SUM64, WIDE, RING>), grid, dim3(kThreads), lds, s, a);
  else if (a.gout)
    hipLaunchKernelGGL((adj_box_kernel<BOX_AVGFIELDS, WIDE, RING>), grid, dim3(kThreads), lds, s,
                       a);
  else
    hipLaunchKernelGGL((adj_box_kernel<BOX_PRODUCTS, WIDE, RING>), grid, dim3(kThreads), lds, s,
                       a);
}

static hipError_t box_launch(AdjBoxArgs a, int planes, hipStream_t s) {
  // windows of up to 2r + 1 = 65 columns: at most two 64-lane prefix segments
  if (planes <= 0 || planes > 65535 || a.H < 1 || a.W < 1 || a.r < 0 || a.r > 32)
    return hipErrorInvalidValue;
  const dim3 grid(box_plan(a, planes), planes);
  a.ring = box_lds_bytes(a.r, true) <= kBoxLdsMax ? 1 : 0;
  const size_t lds = box_lds_bytes(a.r, a.ring != 0);
  if (wide_segments(a.r)) {
    if (a.ring)
      box_dispatch<true, true>(a, grid, lds, s);
    else
      box_dispatch<true, false>(a, grid, lds, s);
  } else {
    if (a.ring)
      box_dispatch<false, true>(a, grid, lds, s);
    else
      box_dispatch<false, false>(a, grid, lds, s);
  }
  return hipGetLastError();
}

hipError_t launch_mean_planes(const float* src, float* dst, int planes, int H, int W, int r,
                              hipStream_t s) {
  if (!src || !dst) return hipErrorInvalidValue;
  AdjBoxArgs a = {};
  a.srcf = src;
  a.dstf = dst;
  a.H = H;
  a.W = W;
  a.r = r;
  return box_launch(a, planes, s);
}

hipError_t launch_box(const double* src, double* dst, int planes, int H, int W, int r,
                      hipStream_t s) {
  if (!src) return hipErrorInvalidValue;
  AdjBoxArgs a = {};
  a.src = src;
  a.dst = dst;
  a.H = H;
  a.W = W;
  a.r = r;
  return box_launch(a, planes, s);
}

hipError_t launch_box_products(const float* guides, const float* noisy, int Q, int C, int H,
                               int W, int r, double* dst, hipStream_t s, bool with_count) {
  AdjBoxArgs a = {};
  a.guides = guides;
  a.noisy = noisy;
  a.dst = dst;
  a.H = H;
  a.W = W;
  a.r = r;
  a.Q = Q;
  a.C = C;
  a.count_first = with_count ? 1 : 0;
  return box_launch(a, num_sums(Q, C) + a.count_first, s);
}

hipError_t launch_box_avgfields(const float* guides, const float* gout, int Q, int C, int H,
                                int W, int r, double* dst, hipStream_t s) {
  if (!guides || !gout || !dst) return hipErrorInvalidValue;
  AdjBoxArgs a = {};
  a.guides = guides;
  a.gout = gout;
  a.dst = dst;
  a.H = H;
  a.W = W;
  a.r = r;
  a.Q = Q;
  a.C = C;
  return box_launch(a, C + Q * C, s);
}

hipError_t launch_mean_planes64(const double* src, double* dst, int planes, int H, int W, int r,
                                hipStream_t s) {
  if (!src || !dst) return hipErrorInvalidValue;
  AdjBoxArgs a = {};
  a.src = src;
  a.dst = dst;
  a.count_first = 1;
  a.H = H;
  a.W = W;
  a.r = r;
  return box_launch(a, planes, s);
}

// The coefficient average (it needs no per-(Q, C) code, so it is built here
// once, beside the other window sums).
// Frames of a batch may differ in tile height and width: TH is the tallest,
// NARROW set where one is narrower than four columns. A frame of two-row tiles
// beside one of four rows then forms twice the rows it stores (15 frames of 200 x
// 260 and one of 1080p, r = 8, Q = 8, C = 3: 808 us in one batch, 423 and 339 in
// batches of their own).
template <int RAD, int TH, bool BATCH, bool NARROW>
__global__ void __launch_bounds__(kThreads, 2) apply_avg_kernel(LaunchArgs ain) {
  int bid = blockIdx.x;
  const LaunchArgs a = BATCH ? batch_frame(ain, &bid) : ain;
  const int n = avg_workgroups(a.tiles_x * a.n_seg, a.nc, a.avg_solo);
  const int t = avg_group_xcd(bid, n);
  if (t >= n) return;  // padding
  avg_group_th<TH, RAD, NARROW>(a, t);
}

template <int RAD, int TH, bool NARROW>
static void avg_launch(const LaunchArgs& a, bool batch, int blocks, hipStream_t s) {
  const size_t l = avg_lds_bytes(TH);
  if (batch)
    hipLaunchKernelGGL((apply_avg_kernel<RAD, TH, true, NARROW>), dim3(blocks), dim3(kThreads), l,
                       s, a);
  else
    hipLaunchKernelGGL((apply_avg_kernel<RAD, TH, false, NARROW>), dim3(blocks), dim3(kThreads), l,
                       s, a);
}

// The kernel of the tile height: one for both heights would take the taller
// one's registers on every frame.
template <int RAD>
static void avg_dispatch(const LaunchArgs& a, bool batch, int blocks, hipStream_t s) {
  if (a.seg_rows > 2)
    a.W < 4 ? avg_launch<RAD, 4, true>(a, batch, blocks, s)
            : avg_launch<RAD, 4, false>(a, batch, blocks, s);
  else
    a.W < 4 ? avg_launch<RAD, 2, true>(a, batch, blocks, s)
            : avg_launch<RAD, 2, false>(a, batch, blocks, s);
}

hipError_t launch_avg(const LaunchArgs& a, bool batch, hipStream_t s) {
  if (a.r < 0 || a.r > 32) return hipErrorInvalidValue;
  if (a.seg_rows < 1 || a.seg_rows > kAvgTileRows || (!batch && a.nc < 1))
    return hipErrorInvalidValue;
  const int blocks = batch ? a.batch_blocks : avg_groups(a.tiles_x * a.n_seg, a.nc, a.avg_solo);
  switch (avg_variant(a.r)) {
    case AVG_R8: avg_dispatch<AVG_R8>(a, batch, blocks, s); break;
    case AVG_R64: avg_dispatch<AVG_R64>(a, batch, blocks, s); break;
    default: avg_dispatch<AVG_R16>(a, batch, blocks, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_pair_sum(const double* src, int n, double* dst, hipStream_t s) {
  if (n < 0) return hipErrorInvalidValue;
  AdjPairArgs a;
  a.src = src;
  a.dst = dst;
  a.n = n;
  hipLaunchKernelGGL(adj_pair_sum_kernel, dim3(1), dim3(kThreads), 2 * kThreads * sizeof(double), s,
                     a);
  return hipGetLastError();
}

}  // namespace flr
