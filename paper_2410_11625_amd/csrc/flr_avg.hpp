// Window average of the coefficient planes and reconstruction (flr_apply,
// the second kernel of the two-pass path and of a batch), for any guide and
// channel count.
//
// Sec. 3.1: each pixel's output uses the mean of the coefficients of the
// windows that contain it,
//   out_c = (sum b_c + sum_q g_q * sum a_qc) / n.
// One workgroup (with few planes and many tiles one wavefront, plan_avg_solo)
// owns one channel of a tile of output rows by avg_cols(r) output columns; that
// channel's planes (b, a_q, and with a.coef_lo the intercepts' lo parts) are
// taken one at a time. Lane l of a wavefront holds
// four adjacent columns X0 - r + 4 l .. + 3: vertical window sums slide down
// each column in FP64 registers, an exclusive prefix of the lanes' totals
// (segments of 16 columns for r <= 8, 64 columns otherwise; DPP moves) turns a
// row of them into segment prefixes, which the wavefront exchanges through
// its own LDS rows, and a window [s, s + 2r] (output column X0 + s) is
//   P[s + 2r] - P[s - 1] (+ the segment's total where it crosses its end).
// Four columns per lane make every load 16 bytes per lane and share the
// prefix's lane moves between four columns.
//
// What bounds it: on small frames the chain of planes (load, sum, exchange),
// hence the planes dealt to the four wavefronts; on large ones the plane rows
// fetched again by the tile below, from L2 and beyond (1080p, Q = 8, C = 3:
// 30 planes of 8.3 MB, five times each, in 135 us = 9.2 TB/s). Measured
// against one workgroup per tile and all channels, 17 rows, one column per
// lane, planes in turn: 256 x 256, Q = 12 144 -> 17 us; 540p, Q = 8 121 ->
// 37 us; 720p, Q = 12 177 -> 83 us; 1080p, Q = 8 149 -> 135 us; 540p, r = 16,
// Q = 6, C = 1 86 -> 27 us. Staging a tile's rows of a plane in LDS for four
// wavefronts (16 rows, each fetched twice) took 176 us at 1080p: its barriers
// leave too few loads in flight.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "flr_launch.hpp"
#include "flr_prefix.hpp"

namespace flr {

// Buffer descriptor of one FP32 plane of `bytes` bytes (raw: stride 0,
// GFX9 dword-3 format word), and a dword load at vector offset `vo` plus
// scalar offset `so`.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const float* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, bytes, 0x00020000);
}
__device__ __forceinline__ float plane_load(__amdgpu_buffer_rsrc_t rs, int vo, int so) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, vo, so, 0));
}

// Four dwords at 4-byte aligned offset vo + so.
__device__ __forceinline__ void plane_load4(__amdgpu_buffer_rsrc_t rs, int vo, int so,
                                            float (&v)[4]) {
#if __has_builtin(__builtin_amdgcn_raw_buffer_load_b128)
  const auto t = __builtin_amdgcn_raw_buffer_load_b128(rs, vo, so, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(t[i]);
#else
  for (int i = 0; i < 4; ++i) v[i] = plane_load(rs, vo + 4 * i, so);
#endif
}

// Four floats at a 4-byte aligned address (one 16-byte store).
typedef float f32x4u __attribute__((vector_size(16), aligned(4)));

// Exclusive prefix of x over aligned groups of G lanes (4 or 16), 0 at the
// first lane of each group. Every lane of the wavefront must take part.
constexpr int kDppQuadShr1 = 0x90;  // quad_perm [0, 0, 1, 2]
constexpr int kDppQuadShr2 = 0x40;  // quad_perm [0, 0, 0, 1]
constexpr int kDppQuadLast = 0xFF;  // quad_perm [3, 3, 3, 3]
// x where the lane mask m is all ones, 0 where it is 0 (two AND instructions,
// half the cycles of two selects).
__device__ __forceinline__ double keep64(double x, unsigned m) {
  const unsigned long long v = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = (unsigned)v & m, hi = (unsigned)(v >> 32) & m;
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// m1, m2: all ones in lanes 1.. and 2.. of each group of four, else 0.
template <int G>
__device__ __forceinline__ double group_exclusive(double x, unsigned m1, unsigned m2) {
  if constexpr (G == 4) {
    double e = keep64(dpp_move<kDppQuadShr1, 0xf>(x), m1);
    e += keep64(dpp_move<kDppQuadShr1, 0xf>(e), m1);
    e += keep64(dpp_move<kDppQuadShr2, 0xf>(e), m2);
    return e;
  } else {
    double e = dpp_move<kDppRowShr + 1, 0xf>(x);
    e += dpp_move<kDppRowShr + 1, 0xf>(e);
    e += dpp_move<kDppRowShr + 2, 0xf>(e);
    e += dpp_move<kDppRowShr + 4, 0xf>(e);
    e += dpp_move<kDppRowShr + 8, 0xf>(e);
    return e;
  }
}

// c ? a : b, both in registers.
__device__ __forceinline__ double pick(bool c, double a, double b) { return c ? a : b; }

// One wavefront's columns of a tile (see above). RAD: AVG_R8 (r = 8), AVG_R16
// (r <= 8) or AVG_R64 (r > 8). EDGE: 0 when every column and row the tile
// reads lies inside the image, 1 when not, 2 for images narrower than four
// columns.
template <int RAD, int EDGE>
struct AvgLane {
  static constexpr int RB = kAvgRowBatch;
  static constexpr int SEG = RAD == AVG_R64 ? 64 : 16;  // columns per prefix segment
  // a row of 128 pairs of columns in LDS, even pairs then odd pairs, so that
  // the 16-byte accesses of consecutive lanes are contiguous
  struct alignas(16) Pair {
    double u, v;
  };
  int lane, r, H, W, Q, C, np, pbytes, x, xo, xs, shift, xg0;
  int xg[4];
  int ia, ib, it;
  unsigned m1, m2;
  int64_t pl;
  const float* planes;
  const float* guides;
  Pair* pr0;

  __device__ __forceinline__ AvgLane(const LaunchArgs& a, int c, int X0, double* row) {
    lane = threadIdx.x & 63;
    r = RAD == AVG_R8 ? 8 : a.r;
    H = a.H;
    W = a.W;
    Q = a.nq;
    C = a.nc;
    np = Q + 1 + (a.coef_lo ? 1 : 0);
    pl = (int64_t)H * W;
    planes = a.planes + (int64_t)c * pl;
    guides = a.guides;
    x = X0 - r + 4 * lane;  // the lane's first column (a multiple of 4)
    xo = X0 + 4 * lane;     // and its first output column
    // Raw buffer loads: a descriptor per plane, the lane's column byte offset
    // (vector) and the row's (scalar); planes hold at most 2^28 pixels, so
    // offsets fit in 32 bits. At the image's edges a lane loads four columns
    // inside the row (only the right end may cut a lane's columns: it then
    // holds columns W - 4 .. W - 1, and its vertical sums move down by `shift`
    // columns), rows are clamped and zeroed.
    pbytes = (int)(pl * 4);
    xs = EDGE == 0 ? x : min(max(x, 0), W - 4);
    shift = x - xs;
    // guide columns of the lane's outputs (clamped; what lies outside is not
    // stored)
#pragma unroll
    for (int i = 0; i < 4; ++i) xg[i] = min(max(xo + i, 0), W - 1) * 4;
    xg0 = min(xo, W - 4) * 4;  // EDGE == 0: xo >= 0 and W >= 256
    // pairs 2 l + r and 2 l + r + 1 hold columns 4 l + 2r .. + 3 (lanes past
    // the tile's columns: clamped), pair pt the last column of the lane's
    // segment (SEG = 64)
    const int pa = min(2 * lane + r, 127), pb = min(2 * lane + r + 1, 127);
    const int pt = (4 * lane | 63) >> 1;
    ia = (pa & 1) * 64 + (pa >> 1);
    ib = (pb & 1) * 64 + (pb >> 1);
    it = (pt & 1) * 64 + (pt >> 1);
    pr0 = reinterpret_cast<Pair*>(row);
    m1 = (lane & 3) >= 1 ? 0xffffffffu : 0u;
    m2 = (lane & 3) >= 2 ? 0xffffffffu : 0u;
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t plane(int f) const {
    return plane_rsrc(planes + (int64_t)f * C * pl, pbytes);
  }
  __device__ __forceinline__ bool is_guide(int f) const { return f >= 1 && f <= Q; }
  // plane f's guide (any valid descriptor for the intercepts)
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t guide_plane(int f) const {
    return plane_rsrc(guides + (int64_t)(is_guide(f) ? f - 1 : 0) * pl, pbytes);
  }
  __device__ __forceinline__ void load_row(__amdgpu_buffer_rsrc_t p, int y, float (&v)[4]) const {
    const int so = (EDGE ? min(max(y, 0), H - 1) : y) * W * 4;
    if constexpr (EDGE == 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = plane_load(p, min(max(x + i, 0), W - 1) * 4, so);
    } else {
      plane_load4(p, xs * 4, so, v);
    }
    if constexpr (EDGE != 0) {
      const unsigned keep = y >= 0 && y < H ? 0xffffffffu : 0u;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = __uint_as_float(__float_as_uint(v[i]) & keep);
    }
  }
  __device__ __forceinline__ void load_guide(__amdgpu_buffer_rsrc_t p, int y, float (&g)[4]) const {
    const int so = (EDGE ? min(y, H - 1) : y) * W * 4;
    if constexpr (EDGE == 0) {
      plane_load4(p, xg0, so, g);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) g[i] = plane_load(p, xg[i], so);
    }
  }
  // vertical sums of the lane's columns x .. x + 3, 0 outside the image
  __device__ __forceinline__ void columns(const double (&s)[4], double (&v)[4]) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double t = s[i];
      if constexpr (EDGE == 1) {
        if (i < 3) t = pick(shift == 1, s[(i + 1) & 3], t);
        if (i < 2) t = pick(shift == 2, s[(i + 2) & 3], t);
        if (i < 1) t = pick(shift == 3, s[(i + 3) & 3], t);
      }
      v[i] = EDGE == 0 ? t : pick(x + i >= 0 && x + i < W, t, 0.0);
    }
  }
  // Horizontal window sums of RB rows of vertical sums, times the guides (1
  // for the intercepts: fma(1, v, s) is v + s), into acc[k0 ..].
  template <int N, int TH>
  __device__ __forceinline__ void rows_out(const int k0, const double (&vs)[N][4],
                                           const float (&g)[TH][4], bool guide,
                                           double (&acc)[TH][4]) const {
    const unsigned gm = guide ? 0xffffffffu : 0u, go = guide ? 0u : 0x3f800000u;  // 1.0f
    double A[N][4];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      double l[4];
      l[0] = vs[j][0];
#pragma unroll
      for (int i = 1; i < 4; ++i) l[i] = l[i - 1] + vs[j][i];
      const double ex = group_exclusive<SEG / 4>(l[3], m1, m2);
      double P[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) P[i] = ex + l[i];
      Pair* pr = pr0 + j * 128;
      pr[lane] = Pair{P[0], P[1]};
      pr[64 + lane] = Pair{P[2], P[3]};
      if constexpr (SEG == 16) {
        const double T = dpp_move<kDppQuadLast, 0xf>(P[3]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool cross = RAD == AVG_R8 || ((4 * lane + i) & 15) + 2 * r > 15;
          A[j][i] = pick(cross, T, 0.0) - (i == 0 ? ex : P[i - 1]);
        }
      } else {
        A[j][0] = ex;
#pragma unroll
        for (int i = 1; i < 4; ++i) A[j][i] = P[i - 1];
      }
    }
    // this wavefront's LDS operations complete in order; the compiler must
    // keep the reads behind the writes
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const int ja = lane_opaque(ia), jb = lane_opaque(ib);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const Pair* pr = pr0 + j * 128;
      const Pair ea = pr[ja], eb = pr[jb];
      const double e[4] = {ea.u, ea.v, eb.u, eb.v};
      double T = 0.0;
      if constexpr (SEG == 64) T = pr[it].v;
      double v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (SEG == 16) {
          v[i] = e[i] + A[j][i];
        } else {
          const bool cross = ((4 * lane + i) & 63) + 2 * r > 63;
          v[i] = (e[i] - A[j][i]) + pick(cross, T, 0.0);
        }
      }
      if constexpr (RAD == AVG_R8) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float w = __uint_as_float((__float_as_uint(g[k0 + j][i]) & gm) | go);
          acc[k0 + j][i] = fma((double)w, v[i], acc[k0 + j][i]);
        }
      } else if (guide) {  // uniform (measured: faster here, slower at r = 8)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[k0 + j][i] = fma((double)g[k0 + j][i], v[i], acc[k0 + j][i]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[k0 + j][i] += v[i];
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  // the means of TH rows from Y (rows y < yend)
  template <int TH>
  __device__ __forceinline__ void store(float* out, const int Y, const int yend,
                                        const double (&acc)[TH][4]) const {
    if (4 * lane >= avg_cols(r)) return;  // a multiple of 4
#pragma unroll
    for (int k = 0; k < TH; ++k) {
      const int y = Y + k;
      if (y >= yend) break;
      const int ny = min(y + r, H - 1) - max(y - r, 0) + 1;
      float* o = out + ((int64_t)y * W + xo);
      float m[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int xi = xo + i;
        const int nx = min(xi + r, W - 1) - max(xi - r, 0) + 1;
        m[i] = (float)(acc[k][i] * recip_count(ny * max(nx, 1), 0.0));
      }
      if constexpr (EDGE) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (xo + i >= 0 && xo + i < W) o[i] = m[i];
      } else {
        *reinterpret_cast<f32x4u*>(o) = f32x4u{m[0], m[1], m[2], m[3]};
      }
    }
  }
};

// One channel of a tile of TH rows. The workgroup's wavefronts take every
// fourth plane each (the chain of planes is what a small frame waits for) and
// add their sums in LDS at the end; SOLO: this wavefront takes every plane
// alone (no barrier), the workgroup's others have tiles of their own.
template <int TH, int RAD, int EDGE, bool SOLO>
__device__ __forceinline__ void avg_tile(const LaunchArgs& a, const int c, const int X0,
                                         const int Y0, const int yend, double* base,
                                         const int wv) {
  constexpr int RB = kAvgRowBatch;
  static_assert(TH % RB == 0, "rows are exchanged RB at a time");
  const AvgLane<RAD, EDGE> L(a, c, X0, base + wv * RB * 256);
  const int r = L.r;
  double acc[TH][4];
#pragma unroll
  for (int k = 0; k < TH; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[k][i] = 0.0;
  for (int f = SOLO ? 0 : wv; f < L.np; f += SOLO ? 1 : kAvgWaves) {
    const __amdgpu_buffer_rsrc_t p = L.plane(f);
    const __amdgpu_buffer_rsrc_t gp = L.guide_plane(f);
    // all loads of the plane first: rows of the first window, then the rows
    // entering (and, where they are not in registers, leaving) it, guides
    constexpr bool R8 = RAD == AVG_R8;
    constexpr int NV = R8 ? TH + 16 : 1, NE = R8 ? 1 : TH;
    float g[TH][4], v[NV][4], ve[NE][4], vl[NE][4];
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    if constexpr (R8) {
#pragma unroll
      for (int j = 0; j < NV; ++j) L.load_row(p, Y0 - 8 + j, v[j]);
    } else {
#pragma unroll
      for (int k = 1; k < TH; ++k) {
        L.load_row(p, Y0 + r + k, ve[k]);
        L.load_row(p, Y0 - r - 1 + k, vl[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < TH; ++k) L.load_guide(gp, Y0 + k, g[k]);
    if constexpr (R8) {
#pragma unroll
      for (int j = 0; j < 17; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) s[i] += (double)v[j][i];
    } else {
      constexpr int B = 8;
      for (int y = Y0 - r; y <= Y0 + r; y += B) {
        float t[B][4];
#pragma unroll
        for (int j = 0; j < B; ++j) L.load_row(p, min(y + j, Y0 + r), t[j]);
#pragma unroll
        for (int j = 0; j < B; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[i] += y + j <= Y0 + r ? (double)t[j][i] : 0.0;
      }
    }
#pragma unroll
    for (int k0 = 0; k0 < TH; k0 += RB) {
      double vs[RB][4];
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        const int k = k0 + j;
        if (k > 0) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (R8)
              s[i] += (double)v[k + 16][i] - (double)v[k - 1][i];
            else
              s[i] += (double)ve[k][i] - (double)vl[k][i];
          }
        }
        L.columns(s, vs[j]);
      }
      L.template rows_out<RB, TH>(k0, vs, g, L.is_guide(f), acc);
    }
  }
  if constexpr (SOLO) {
    L.template store<TH>(a.out + (int64_t)c * L.pl, Y0, yend, acc);
    return;
  }
  __syncthreads();  // every wavefront is done with its exchange rows
  double* red = base + (threadIdx.x & 63);
#pragma unroll
  for (int k = 0; k < TH; ++k)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[((wv * TH + k) * 4 + i) * 64] = acc[k][i];
  __syncthreads();
  // wavefront w stores rows w, w + 4, ...
  for (int k = wv; k < TH; k += kAvgWaves) {
    double sum[1][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      double t = 0.0;
#pragma unroll
      for (int w = 0; w < kAvgWaves; ++w) t += red[((w * TH + k) * 4 + i) * 64];
      sum[0][i] = t;
    }
    L.template store<1>(a.out + (int64_t)c * L.pl, Y0 + k, yend, sum);
  }
}

// Unit u of a frame: one channel of one tile. Channels run fastest, then
// down a strip, so that a tile's channels (which read the same guides) and
// vertically adjacent tiles (which share 2r rows of every plane) follow each
// other. NARROW: the image may be (1) or is (2) narrower than four columns (a
// kernel of its own: its loads would take the four-row form at r = 8 from 163 to
// 252 registers).
template <int TH, int RAD, int NARROW, bool SOLO>
__device__ __forceinline__ void avg_unit(const LaunchArgs& a, const int u, double* base,
                                         const int wv) {
  const int tile = u / a.nc, c = u - tile * a.nc;
  const int sx = tile / a.n_seg, sy = tile - sx * a.n_seg;
  const int X0 = avg_col0(sx, a.r), Y0 = sy * a.seg_rows;
  const int yend = min(Y0 + a.seg_rows, a.H);
  const bool edge = X0 - a.r < 0 || X0 - a.r + 256 > a.W || Y0 - a.r < 0 ||
                    Y0 + TH - 1 + a.r >= a.H;
  if constexpr (NARROW == 2)
    avg_tile<TH, RAD, 2, SOLO>(a, c, X0, Y0, yend, base, wv);
  else if (!edge)
    avg_tile<TH, RAD, 0, SOLO>(a, c, X0, Y0, yend, base, wv);
  else if (!NARROW || a.W >= 4)
    avg_tile<TH, RAD, 1, SOLO>(a, c, X0, Y0, yend, base, wv);
  else
    avg_tile<TH, RAD, 2, SOLO>(a, c, X0, Y0, yend, base, wv);
}

// Workgroup t of a frame: a unit, or one for each wavefront (avg_solo).
template <int TH, int RAD, int NARROW>
__device__ __forceinline__ void avg_group_th(const LaunchArgs& a, const int t) {
  extern __shared__ float lds[];
  double* base = reinterpret_cast<double*>(lds);
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (a.avg_solo) {
    const int u = t * kAvgWaves + wv;
    if (u < a.tiles_x * a.n_seg * a.nc) avg_unit<TH, RAD, NARROW, true>(a, u, base, wv);
  } else {
    avg_unit<TH, RAD, NARROW, false>(a, t, base, wv);
  }
}

// Workgroup t with the frame's tile height and width.
template <int RAD>
__device__ __forceinline__ void avg_group(const LaunchArgs& a, const int t) {
  if (a.W < 4)
    a.seg_rows > 2 ? avg_group_th<4, RAD, 2>(a, t) : avg_group_th<2, RAD, 2>(a, t);
  else
    a.seg_rows > 2 ? avg_group_th<4, RAD, 0>(a, t) : avg_group_th<2, RAD, 0>(a, t);
}

// Workgroup of a frame for workgroup b of its launch range. Workgroups are
// dealt to the XCDs round-robin, and a frame's range starts at a multiple
// of kXcds and has avg_groups(n) workgroups, so XCD k runs the frame's
// workgroups k, k + kXcds, ... in order; it gets the k-th run of
// ceil(n / kXcds) groups, whose shared plane rows stay in that XCD's L2.
// The last ones may lie past the end (padding).
__device__ __forceinline__ int avg_group_xcd(int b, int n) {
  const int m = (n + kXcds - 1) / kXcds;
  return (b % kXcds) * m + b / kXcds;
}

}  // namespace flr
