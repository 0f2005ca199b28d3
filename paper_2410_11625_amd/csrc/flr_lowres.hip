// Separable Gaussian blur of the low-resolution moment planes of the
// downsampled-moment variant. A workgroup blurs one 16 x 16 tile of one
// plane: it stages the tile with an R-wide border in LDS (zero outside the
// grid), runs the pass along the rows into a second LDS buffer, then the
// pass along the columns.
#include <hip/hip_runtime.h>

#include "flr_launch.hpp"

namespace flr {

constexpr int kLrTile = 16;

struct LrBlurArgs {
  const double* src;
  double* dst;
  int Hl, Wl, tiles_x;
  double taps[2 * kMaxLowresRadius + 1];
};

// What bounds it: the tile's loads, its halo read from L2 (2.25 loads per output
// at radius 4). The radius is a template parameter so that every tap's LDS read
// is in flight at once (with a loop over a runtime radius each waited for the
// one before) and positions need no division: 23.0 -> 13.9 us at 1080p, 8 x 8
// blocks, 72 planes. Tiles of 32 and 64 rows took 13.8 and 14.0.
template <int R>
__global__ void __launch_bounds__(kThreads) lr_blur_kernel(LrBlurArgs a) {
  constexpr int SX = kLrTile + 2 * R, SY = kLrTile + 2 * R;
  constexpr int NL = (SX * SY + kThreads - 1) / kThreads;
  __shared__ double tile[SX * SY];
  __shared__ double mid[SY * kLrTile];
  const int tid = threadIdx.x;
  const int bx = blockIdx.x % a.tiles_x, by = blockIdx.x / a.tiles_x;
  const int64_t pll = (int64_t)a.Hl * a.Wl;
  const double* src = a.src + (int64_t)blockIdx.y * pll;
  const int I0 = by * kLrTile - R, J0 = bx * kLrTile - R;
  // loads from clamped positions, issued together, zero outside the grid
  double v[NL];
  bool in[NL];
#pragma unroll
  for (int u = 0; u < NL; ++u) {
    const int t = tid + u * kThreads;
    const int ii = t / SX, jj = t - (t / SX) * SX;
    const int I = I0 + ii, J = J0 + jj;
    in[u] = t < SX * SY && I >= 0 && I < a.Hl && J >= 0 && J < a.Wl;
    const int Ic = I < 0 ? 0 : (I >= a.Hl ? a.Hl - 1 : I);
    const int Jc = J < 0 ? 0 : (J >= a.Wl ? a.Wl - 1 : J);
    v[u] = src[(int64_t)Ic * a.Wl + Jc];
  }
#pragma unroll
  for (int u = 0; u < NL; ++u) {
    const int t = tid + u * kThreads;
    if (t < SX * SY) tile[t] = in[u] ? v[u] : 0.0;
  }
  __syncthreads();
  for (int t = tid; t < SY * kLrTile; t += kThreads) {
    const int ii = t / kLrTile, jj = t - (t / kLrTile) * kLrTile;
    double s = 0.0;
#pragma unroll
    for (int d = 0; d <= 2 * R; ++d) s = fma(a.taps[d], tile[ii * SX + jj + d], s);
    mid[t] = s;
  }
  __syncthreads();
  const int ii = tid / kLrTile, jj = tid - (tid / kLrTile) * kLrTile;
  const int I = by * kLrTile + ii, J = bx * kLrTile + jj;
  if (I < a.Hl && J < a.Wl) {
    double s = 0.0;
#pragma unroll
    for (int d = 0; d <= 2 * R; ++d) s = fma(a.taps[d], mid[(ii + d) * kLrTile + jj], s);
    a.dst[(int64_t)blockIdx.y * pll + (int64_t)I * a.Wl + J] = s;
  }
}

template <int R>
hipError_t launch_blur(const LrBlurArgs& a, int rad, int blocks, int planes, hipStream_t s) {
  if constexpr (R < kMaxLowresRadius)
    if (rad > R) return launch_blur<R + 1>(a, rad, blocks, planes, s);
  hipLaunchKernelGGL(lr_blur_kernel<R>, dim3(blocks, planes), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_lr_blur(const double* src, double* dst, int planes, int Hl, int Wl, int R,
                          const double* taps, hipStream_t s) {
  if (planes <= 0 || planes > 65535 || Hl < 1 || Wl < 1 || R < 0 || R > kMaxLowresRadius)
    return hipErrorInvalidValue;
  LrBlurArgs a;
  a.src = src;
  a.dst = dst;
  a.Hl = Hl;
  a.Wl = Wl;
  a.tiles_x = (Wl + kLrTile - 1) / kLrTile;
  const int tiles_y = (Hl + kLrTile - 1) / kLrTile;
  for (int k = 0; k < 2 * kMaxLowresRadius + 1; ++k) a.taps[k] = k <= 2 * R ? taps[k] : 0.0;
  return launch_blur<0>(a, R, a.tiles_x * tiles_y, planes, s);
}

}  // namespace flr
