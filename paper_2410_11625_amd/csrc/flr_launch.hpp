// Launch geometry and the interface between the host dispatcher and the
// per-guide-count kernel instantiations. Host and device code share it.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace flr {

// One workgroup = one column strip of kThreads input columns walking down a
// segment of rows. Four 64-wide wavefronts.
constexpr int kThreads = 256;
// MI355X compute units; the automatic segment choice aims for whole waves of
// workgroups over this many CUs (workgroups_per_cu of a walker on each).
constexpr int kCUs = 256;
// Numeric types. Products of the FP32 inputs are summed in sum_t; central
// moments, intercepts, the coefficient average and the reconstruction run in
// solve_t; the centred, regularised system is factorised and solved in
// chol_t (it is well conditioned once centred in solve_t). (With packed FP32 unused, an FP64 FMA
// issues at the same rate as an FP32 one on CDNA4; FP64 costs registers and
// LDS bytes, not ALU slots.)
#ifndef FLR_SUM_T
#define FLR_SUM_T double
#endif
#ifndef FLR_SOLVE_T
#define FLR_SOLVE_T double
#endif
// Element type of the fused kernel's coefficient ring (coefficients relative
// to the workgroup anchor).
#ifndef FLR_RING_T
#define FLR_RING_T float
#endif
// Factorisation and triangular solves of the per-pixel system. FP64: with
// the regulariser at 1e-3 of unit-scale guides, windows of near-constant
// guides make the centred system's condition number reach 1e4 and more, and
// an FP32 factorisation then errs by up to 2e-4 relative in the output
// (measured on 40 x 270 frames of the RGB workload); in FP64 it is below 2e-5.
#ifndef FLR_CHOL_T
#define FLR_CHOL_T double
#endif
typedef FLR_CHOL_T chol_t;
typedef FLR_SUM_T sum_t;
typedef FLR_SOLVE_T solve_t;
typedef FLR_RING_T ring_t;
// Running vertical sums of the ring values in the fused kernel.
#ifndef FLR_AVG_T
#define FLR_AVG_T double
#endif
typedef FLR_AVG_T avg_t;
// LDS row stride in elements: kThreads + 1 keeps lanes that read
// consecutive channel rows of one column on distinct banks.
constexpr int kLdsStride = kThreads + 1;
// LDS per workgroup (gfx950: 160 KiB).
constexpr int kLdsBytes = 163840;
// Channel rows of element size `elem` that fit twice (source and
// destination of the horizontal pass) in LDS.
__host__ __device__ constexpr int max_lds_rows(int elem) {
  return kLdsBytes / (2 * kLdsStride * elem);
}
__host__ __device__ constexpr int group_count(int rows, int elem) {
  return (rows + max_lds_rows(elem) - 1) / max_lds_rows(elem);
}
__host__ __device__ constexpr int group_size(int rows, int elem) {
  return (rows + group_count(rows, elem) - 1) / group_count(rows, elem);
}

enum Kind : int {
  K_MOMENTS = 0,      // window moments -> moment planes
  K_SOLVE = 1,        // moment planes -> coefficient planes
  K_APPLY_POINT = 2,  // coefficient planes + guides -> output (no averaging)
  K_APPLY_AVG = 3,    // coefficient planes -> window average -> output
  K_FUSED0 = 4,       // moments -> solve -> apply, no averaging, one kernel
  K_FUSED1 = 5,       // moments -> solve -> average -> apply, one kernel
  K_COEFFS = 6,       // moments -> solve -> coefficient planes, one kernel
  K_MOMENTS_A = 7,    // K_MOMENTS over the first slice of the product channels
  K_MOMENTS_B = 8,    // K_MOMENTS over the rest (split walks)
  // adjoint (flr_denoise_backward)
  K_ADJ_COEF = 9,     // coefficients from FP64 moment sums + the averaging fields
  K_ADJ_SOLVE = 10,   // per-pixel solve adjoint -> fields whose window sums give dL/dg, dL/dy
  K_ADJ_GATHER = 11,  // window sums of those fields contracted with g and y
  // the downsampled-moment variant (flr_denoise_lowres)
  K_LR_BLOCK = 12,    // block sums of the anchored products -> low-resolution planes
  K_LR_SOLVE = 13,    // Gaussian pass along columns + solve per low-resolution pixel
  K_LR_APPLY = 14,    // bilinear model interpolation + reconstruction
  // batched serving
  K_COEFFS_BATCH = 15,     // K_COEFFS over the tiles of several frames
  K_APPLY_AVG_BATCH = 16,  // K_APPLY_AVG over the tiles of several frames
  K_UP_APPLY_BATCH = 17,   // bilinear upsampling of coefficient planes + reconstruction
  K_BATCH_PERSISTENT = 18, // every stage of a batch in one launch over a work queue
  K_SPLIT_COEFFS = 19,     // split walks: the walk over the second slice, with the first
                           // slice's moment planes read back -> solve -> coefficient planes
};

// One persistent launch for a batch (flr_batch_run): workgroups take items
// from a queue counter in order; an item is one workgroup's tile of one
// stage of one frame. Stages, in queue order: the coefficient walk of the
// plain frames; per joint frame the FP64 window sums of its products, the
// per-pixel solve and the window mean of the models; the averaging and
// reconstruction of the plain frames; the upsampling of the joint frames.
// An item only waits on items earlier in the queue (taken by workgroups
// that are running), through counters that finished items increment.
enum BatchItemKind : int {
  BI_WALK = 0, BI_JBOX = 1, BI_JSOLVE = 2, BI_JMEAN = 3, BI_AVG = 4, BI_UP = 5
};
struct BatchStage {
  int kind;      // BatchItemKind
  int arg;       // index into the launch-argument table (largs) or, box passes, bargs
  int first;     // first queue item of the stage
  int count;     // its items
  int nx;        // box passes: workgroups per plane
  int wait;      // counter its items wait on (-1: none); BI_AVG: the frame's
                 // first walk-segment counter
  int need;      // the value that counter must reach (BI_AVG: strips per walk segment)
  int done;      // counter a finished item increments (-1: none); BI_WALK: the
                 // frame's first walk-segment counter (one per segment)
  int seg_rows;  // BI_WALK, BI_AVG: rows per walk segment of the frame
  int nseg;      // BI_AVG: walk segments of the frame
};
// Arguments of one box pass (flr_box.hpp).
struct AdjBoxArgs {
  const float* srcf;   // BOX_MEAN32: FP32 planes, averaged into dstf
  float* dstf;
  const double* src;   // FP64 planes, or NULL for the product channels below
  const float* guides; // product channels: guides [Q][H][W]
  const float* noisy;  // product channels: noisy [C][H][W]
  const float* gout;   // BOX_AVGFIELDS: dL/d(output) [C][H][W]
  double* dst;
  int64_t plane;  // elements per plane
  int H, W, r, seg_rows, tiles_x;
  int Q, C;
  int count_first;  // BOX_PRODUCTS: plane 0 is the window pixel count, channels follow
  int ring;         // 1: the leaving rows come from an LDS ring of 2r + 1 rows
};

// LDS bytes of a box pass: two FP64 prefix rows of kThreads + 1, and with
// the ring 2r + 1 FP64 rows of kThreads.
inline size_t box_lds_bytes(int r, bool ring) {
  return (size_t)(2 * (kThreads + 1) + (ring ? (2 * r + 1) * kThreads : 0)) * sizeof(double);
}
// Largest LDS of a standalone box launch with the ring (so that several
// workgroups share a CU); larger radii load the leaving row again.
constexpr size_t kBoxLdsMax = 64 * 1024;

// Rows per workgroup segment of a box pass, and its tiling: sets plane,
// seg_rows, tiles_x; returns the workgroups per plane. Segments of up to
// kBoxSegRows rows (each repeats 2r warm-up rows), halved while the
// `planes` planes of the pass would give fewer than kBoxMinGroups
// workgroups.
constexpr int kBoxSegRows = 128;
constexpr int kBoxMinGroups = 2048;
inline int box_plan(AdjBoxArgs& a, int planes = 1) {
  a.plane = (int64_t)a.H * a.W;
  a.tiles_x = (a.W + (kThreads - 2 * a.r) - 1) / (kThreads - 2 * a.r);
  int seg = kBoxSegRows;
  while (seg > 16 && (int64_t)a.tiles_x * ((a.H + seg - 1) / seg) * planes < kBoxMinGroups)
    seg /= 2;
  a.seg_rows = seg < a.H ? seg : a.H;
  return a.tiles_x * ((a.H + a.seg_rows - 1) / a.seg_rows);
}

struct BatchPlanDev {
  const BatchStage* stages;
  int nstages, nitems, ncounters, pad;
  const struct LaunchArgs* largs;
  const AdjBoxArgs* bargs;
  int* ctl;       // [0] queue head, [1] workgroups finished, [2] waits given up (kept)
  int* counters;  // [ncounters]
};
// Longest wait of an item before it gives up and flags the run as failed
// (iterations of a short sleep; far beyond any item's duration).
constexpr int kBatchSpinLimit = 1 << 24;

// Longest Gaussian of the downsampled-moment variant (taps -R..R).
constexpr int kMaxLowresRadius = 8;

struct LaunchArgs {
  const float* guides;   // [Q][H][W]
  const float* noisy;    // [C][H][W]
  const float* planes;   // K_SOLVE: moments; K_APPLY_*: coefficients
  float* out;            // moments / coefficients / output image
  void* ring;            // K_FUSED1 workspace (ring_t elements)
  int H, W, r;
  int nq, nc;    // guides and channels
  int avg_solo;  // averaging: a tile and channel per wavefront (plan_avg)
  int seg_rows, tiles_x, n_seg;
  int hchunk_m, hchunk_a;  // horizontal-pass chunk lengths (moments, averaging)
  float eps, eps_mul;
  const float* eps_dev;  // when set: (eps, eps_mul) read from device memory instead
  int reg_mode;
  int raw;
  // K_COEFFS / K_SPLIT_COEFFS / K_APPLY_AVG (and their batched forms): the
  // coefficient image carries each intercept as an FP32 pair, hi in plane c
  // and lo in plane (Q + 1) C + c, formed in FP64 from the slopes as stored
  // (FP32), so that the model's value at the window mean is kept to FP64
  // accuracy where a fit's intercept and slope terms cancel
  int coef_lo;
  // adjoint kernels only
  const float* gout;     // dL/d(output) [C][H][W]
  const float* coeffs;   // unaveraged coefficient planes (b | a)
  const double* sums;    // FP64 window sums of the anchored input products
  const double* fin;     // FP64 field planes read (window sums)
  const double* fin2;    // K_ADJ_GATHER: window sums of the averaging fields
  double* fout;          // FP64 field planes written
  double* red;           // K_ADJ_SOLVE: per-workgroup sums of dL/deps, dL/deps_mul
  float* out2;           // K_ADJ_GATHER: dL/d(noisy)
  int average;
  // downsampled-moment variant only
  int block, Hl, Wl, lr_R;
  int lr_rows;  // K_LR_APPLY: full-resolution rows per workgroup (0: one lane per pixel)
  // batched launches (K_COEFFS_BATCH, K_APPLY_AVG_BATCH, K_UP_APPLY_BATCH):
  // workgroup b belongs to the frame f with wg_start[f] <= b < wg_start[f + 1]
  // and runs as workgroup b - wg_start[f] of frames[f]
  const struct LaunchArgs* frames;
  const int* wg_start;
  const BatchPlanDev* bplan;  // K_BATCH_PERSISTENT
  int nframes;
  int batch_blocks;  // total workgroups of the launch
  int up;            // K_UP_APPLY: upsampling factor (coefficient grid = H / up)
  const float* guides_low;  // K_UP_APPLY: the guides the models were fitted on (anchors)
  double taps[2 * kMaxLowresRadius + 1];
};

// LDS of the staged model interpolation: rows x models x low-resolution
// columns of FP64 (a workgroup's kThreads columns span at most
// (kThreads - 1) / block + 3 low-resolution columns).
__host__ __device__ constexpr size_t lr_apply_lds_bytes(int Q, int C, int block, int rows) {
  return (size_t)rows * (Q + 1) * C * ((kThreads - 1) / block + 3) * sizeof(double);
}
// Rows per workgroup of the staged interpolation: the most of 8, 4, 2 whose
// staging fits in 32 KiB (five or more workgroups per CU: a workgroup stages,
// then computes, and others fill either half's waits), else one row where
// that fits in 64 KiB; 0 when it does not (one lane per pixel then). Measured at
// 1080p, Q = 8, C = 3, 8 x 8 blocks: 8 rows in 59 KB 44.5 us, 4 in 29 KB 32.3, 2
// in 15 KB 33.2.
inline int lr_apply_rows(int Q, int C, int block) {
  for (int rows = 8; rows > 1; rows /= 2)
    if (lr_apply_lds_bytes(Q, C, block, rows) <= 32768) return rows;
  return lr_apply_lds_bytes(Q, C, block, 1) <= 65536 ? 1 : 0;
}

// Upsampling tiles have one row: staged at 2 x it takes 28 KB at Q = 8, C = 3
// (two rows, 57 KB: 114 against 88 us at 1080p). Frames of up to half a
// workgroup's columns take as many rows as fit in it side by side, in no more
// LDS (the staged columns of a row are at most half its pixels).
__host__ __device__ constexpr int up_rows(int W) {
  int rows = 1;
  while (2 * rows * W <= kThreads) rows *= 2;
  return rows;
}
inline int up_items(int H, int W) {
  return ((W + kThreads - 1) / kThreads) * ((H + up_rows(W) - 1) / up_rows(W));
}

// The downsampled-moment variant's low-resolution planes: the pixel count
// n then the num_sums(Q, C) anchored product sums (FP64, [planes][Hl][Wl]);
// models b~ (C) then a (Q*C) in anchored units (FP64).
// dst[p][I][J] = sum_{|d|, |e| <= R} taps[d + R] taps[e + R] src[p][I + d][J + e]
// (zero outside the grid): the separable low-resolution blur.
hipError_t launch_lr_blur(const double* src, double* dst, int planes, int Hl, int Wl, int R,
                          const double* taps, hipStream_t s);

// Adjoint field planes (FP64, [planes][H][W]).
//  averaging fields: G_c / n (C), g~_q G_c / n (Q*C), a_qc (Q*C) (K_ADJ_COEF
//  writes the a_qc; the window-sum pass forms the others from the inputs);
//  solve fields, K_ADJ_SOLVE: 2 dW / n (upper triangle), Gv / n (Q*C),
//  e (Q), f (C) -- num_sums(Q, C) planes.
__host__ __device__ constexpr int num_avg_fields(int Q, int C) { return C + 2 * Q * C; }

// FP64 clipped window sums of `planes` planes of H x W (separable: running
// column sums, then a row pass through LDS). src and dst must not overlap.
hipError_t launch_box(const double* src, double* dst, int planes, int H, int W, int r,
                      hipStream_t s);
// FP32 window means (clipped window, FP64 sums) of `planes` planes of H x W.
hipError_t launch_mean_planes(const float* src, float* dst, int planes, int H, int W, int r,
                              hipStream_t s);
// The same for FP64 planes, FP64 means.
hipError_t launch_mean_planes64(const double* src, double* dst, int planes, int H, int W, int r,
                                hipStream_t s);
// FP64 clipped window sums of the num_sums(Q, C) anchored products of the
// inputs, in the moment order g_q | y_c | g_p g_q (p <= q) | g_q y_c, each
// input plane shifted by its value at pixel (0, 0).
// With with_count, plane 0 is the window pixel count and the channels follow
// (the plane order of the downsampled-moment variant's solve).
hipError_t launch_box_products(const float* guides, const float* noisy, int Q, int C, int H,
                               int W, int r, double* dst, hipStream_t s,
                               bool with_count = false);
// FP64 clipped window sums of the adjoint's averaging products, formed from
// the inputs: G_c / n (C planes) then g~_q G_c / n (Q*C planes), with G =
// dL/d(output), n the pixel's window count and g~ each guide shifted by its
// value at pixel (0, 0).
hipError_t launch_box_avgfields(const float* guides, const float* gout, int Q, int C, int H,
                                int W, int r, double* dst, hipStream_t s);
// dst[0..1] = sums over n entries of the interleaved pairs src[2i], src[2i+1]
// (fixed order; one workgroup).
hipError_t launch_pair_sum(const double* src, int n, double* dst, hipStream_t s);
// Window average of the coefficient planes and reconstruction (a.planes ->
// a.out, tiles of plan_avg), of one frame or (batch) of a.frames.
hipError_t launch_avg(const LaunchArgs& a, bool batch, hipStream_t s);

__host__ __device__ constexpr int num_sums(int Q, int C) {
  return Q + C + Q * (Q + 1) / 2 + Q * C;
}

// Output columns per strip for a walker kernel.
inline int strip_out_cols(int kind, int r) {
  if (kind == K_FUSED1) return kThreads - 4 * r;
  return kThreads - 2 * r;  // K_MOMENTS, K_FUSED0, K_COEFFS
}

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// The coefficient-averaging kernel (flr_avg.hpp): wavefronts per workgroup,
// rows a wavefront exchanges through LDS at a time, the output columns of a
// tile (256 input columns, four per lane, less the window's 2r, in whole
// lanes) and the largest tile height.
// Prefix segments of 16 lanes (or columns) serve windows up to 2r + 1 = 17
// columns wide.
__host__ __device__ constexpr bool wide_segments(int r) { return r > 8; }
constexpr int kAvgWaves = 4;
constexpr int kAvgRowBatch = 2;
constexpr int kAvgTileRows = 4;
__host__ __device__ constexpr int avg_cols(int r) { return (256 - 2 * r) & ~3; }
// First output column of strip sx: its input columns start r to the left, at
// a multiple of 4 (strip 0's first outputs may lie left of the image).
__host__ __device__ constexpr int avg_col0(int sx, int r) {
  return sx * avg_cols(r) + r - ((r + 3) & ~3);
}
// LDS of a workgroup with tiles of `rows` rows: the wavefronts' exchange
// rows, reused for their closing sums of `rows` rows.
inline size_t avg_lds_bytes(int rows) {
  return (size_t)kAvgWaves * (rows > 2 ? 4 : 2) * 256 * sizeof(double);
}
// Its forms by radius: r = 8 keeps a plane's rows of the tile in registers;
// other radii load the rows entering and leaving the window; r > 8 needs
// prefix segments of 64 columns.
enum AvgVariant : int { AVG_R16 = 0, AVG_R64 = 1, AVG_R8 = 2 };
__host__ __device__ constexpr int avg_variant(int r) {
  return r == 8 ? AVG_R8 : (wide_segments(r) ? AVG_R64 : AVG_R16);
}

// XCDs of the GPU (workgroups are dealt to them round-robin), the averaging
// workgroups of `tiles` tiles of C channels, and their launch range: whole
// rounds of the XCDs, so that each XCD runs a contiguous run of them.
constexpr int kXcds = 8;
// Tiles of an averaging item of the persistent batch queue, all channels of
// each: an item costs a queue step and its wait, a tile of four rows alone is
// too little work for one (16 frames, 35 Mpixel: 16.7 -> 13.5 ms).
constexpr int kAvgItemTiles = 4;
static_assert(kAvgItemTiles % kAvgWaves == 0, "an item holds whole workgroups of plan_avg_solo");
inline int avg_items(int tiles) { return (tiles + kAvgItemTiles - 1) / kAvgItemTiles; }
__host__ __device__ constexpr int avg_workgroups(int tiles, int C, int solo) {
  return solo ? (tiles * C + kAvgWaves - 1) / kAvgWaves : tiles * C;
}
inline int avg_groups(int tiles, int C, int solo) {
  return (avg_workgroups(tiles, C, solo) + kXcds - 1) / kXcds * kXcds;
}

// Rows of coefficient halo a walker recomputes above and below its segment.
inline int row_halo(int kind, int r) { return kind == K_FUSED1 ? r : 0; }

// Tiles of the averaging kernel: tile_rows, when set; else four rows where
// they give kAvgMinGroups workgroups (tile and channel), so that a plane row is
// fetched (4 + 2r) / 4 times instead of (2 + 2r) / 2, and two rows below, where
// the shorter chain and the workgroup count win. Measured, 2 / 4 rows: 256 x
// 256, Q = 12, C = 3 16.8 / 17.9 us; 540p, Q = 8 45 / 37; 1080p, Q = 8 177 / 135;
// r = 16, 540p, C = 1 35 / 27; 1080p, C = 3 261 / 181. (Eight rows: 242
// registers, two wavefronts per SIMD; 1080p, Q = 8 132, r = 16 221.)
constexpr int kAvgMinGroups = 600;
// A wavefront takes a tile's planes (np of them) alone where four would share
// too few: with 2, 3 or 5 planes some idle through a quarter to half of the
// tile, and the closing sum costs two barriers. It takes several tiles per
// wavefront slot of the chip to make up for the longer chain. Measured, shared /
// alone: r = 8, 1080p, 2 planes, C = 1 (2160 tiles) 17.3 / 13.2 us; 4K, C = 3 154
// / 107; 3 planes, 1080p, C = 3 45 / 38; 5 planes, 1080p, C = 3 (6480 tiles) 65.5 /
// 58.1, C = 1 26.5 / 27.7; 7 planes, 1080p, C = 3 within 3 %; other radii hold fewer
// registers and more wavefronts: 2 planes, 4K, r = 16, C = 3 0.77, 3 planes
// 0.89 to 1.19.
inline int plan_avg_solo(int r, int np, int64_t units) {
  if (r == 8) return (np <= 3 && units >= 2048) || (np <= 6 && units >= 6144);
  return np == 2 && units >= 3072;
}
inline void plan_avg(int H, int W, int r, int Q, int C, bool coef_lo, int tile_rows, int* tiles_x,
                     int* n_seg, int* seg_rows, int* solo) {
  *tiles_x = ceil_div(W - avg_col0(0, r), avg_cols(r));
  constexpr int tall = kAvgTileRows;
  int t = 2;
  if (tile_rows > 0)
    t = tile_rows < kAvgTileRows ? tile_rows : kAvgTileRows;
  else if ((int64_t)*tiles_x * ceil_div(H, tall) * C >= kAvgMinGroups)
    t = tall;
  *seg_rows = t < H ? t : H;
  *n_seg = ceil_div(H, *seg_rows);
  *solo = plan_avg_solo(r, Q + 1 + (coef_lo ? 1 : 0), (int64_t)*tiles_x * *n_seg * C);
}

// Chunk length for the LDS horizontal pass over `rows` channel rows and
// `nout` outputs: minimise (task passes) x (window taps + 2 per output). A
// pass runs two tasks per thread side by side, so its latency is that of one.
inline int plan_chunk(int rows, int nout, int r) {
  int best = nout;
  double bestc = 1e300;
  for (int nch = 1; nch <= nout; ++nch) {
    const int chunk = ceil_div(nout, nch);
    if (nch > 1 && ceil_div(nout, nch - 1) == chunk) continue;
    const int passes = ceil_div(rows * ceil_div(nout, chunk), 2 * kThreads);
    const double cost = passes * (2.0 * r + 1 + 2.0 * (chunk - 1));
    if (cost < bestc) {
      bestc = cost;
      best = chunk;
    }
  }
  return best;
}

// LDS layout of the walker kernels (bytes, rows of kLdsStride elements):
//   [0, a)            source rows of the horizontal pass (one moment group);
//   [a, a + b)        destination rows (moment group, or coefficient sums);
//   [a + b, + va)     K_FUSED1 only, when it fits: the persistent vertical
//                     window sums of the coefficients, F*C rows of solve_t,
//                     read directly by the horizontal averaging pass.
// Moment channels are processed in groups of `mg` rows; the first group
// always holds all Q + C first moments.
struct WalkLayout {
  int mg;          // moment rows per group
  int ag;          // coefficient rows per averaging group (va_lds: all F*C)
  bool va_lds;     // coefficient sums live in LDS
  size_t a, b, va; // region sizes in bytes
};

__host__ __device__ constexpr WalkLayout walk_layout(int Q, int C, int kind, int ns_walk = -1) {
  const int ns = ns_walk > 0 ? ns_walk : num_sums(Q, C);
  const int fc = (Q + 1) * C;
  const int row_s = kLdsStride * (int)sizeof(sum_t);
  const int row_t = kLdsStride * (int)sizeof(solve_t);
  WalkLayout L{0, 0, false, 0, 0, 0};
  if (kind == K_FUSED1) {
    const int va = fc * row_t;
    const int left = kLdsBytes - 2 * va;  // Va region + destination sized for F*C rows
    const int mg_max = left > 0 ? left / row_s : 0;
    if (mg_max >= Q + C) {
      const int ng = (ns + mg_max - 1) / mg_max;
      L.mg = (ns + ng - 1) / ng;
      L.ag = fc;
      L.va_lds = true;
      L.a = (size_t)L.mg * row_s;
      const size_t bm = (size_t)L.mg * row_s;
      L.b = bm > (size_t)va ? bm : (size_t)va;
      L.va = (size_t)va;
      return L;
    }
  }
  L.mg = group_size(ns, sizeof(sum_t));
  L.ag = group_size(fc, sizeof(solve_t));
  const size_t m = (size_t)L.mg * row_s;
  const size_t c = (size_t)L.ag * row_t;
  L.a = L.b = m > c ? m : c;
  // all channels in one group, resident in LDS: the second buffer is not used
  if (kind != K_FUSED1 && L.mg >= ns) L.b = 0;
  return L;
}

inline size_t walk_lds_bytes(int kind, int Q, int C, int ns_walk = -1) {
  const WalkLayout L = walk_layout(Q, C, kind, ns_walk);
  return L.a + L.b + L.va;
}

// Vector registers of a walker of ns moment channels in one LDS group: its
// vertical sums, two registers each, and what a mode holds beside them (the
// built kernels': W_MOMENTS 68 at 4 channels, 176 at 19, 276 at 34; W_COEFFS and
// W_FUSED0 56, 138 and 212).
__host__ __device__ constexpr int walk_registers(int kind, int ns) {
  return kind == K_MOMENTS ? 54 + (13 * ns + 1) / 2 : 44 + 5 * ns;
}
// Workgroups of a walker kernel that share a CU: by LDS, and by the 512
// registers of a SIMD lane, on which each has one wave. Counting LDS alone
// planned two workgroups of 276 registers as if both ran at once: moments at
// Q = 6, C = 1, 540p, r = 24 94.7 us, counted as one 67.6.
inline int workgroups_per_cu(int kind, int Q, int C) {
  if (kind == K_FUSED1) return 1;
  const int lds = (int)(kLdsBytes / walk_lds_bytes(kind, Q, C));
  const int regs = 512 / walk_registers(kind, num_sums(Q, C));
  const int n = lds < regs ? lds : regs;
  return n < 1 ? 1 : (n > 4 ? 4 : n);
}
// Time of a row step with k workgroups on a CU, against one alone. Measured
// at 1080p, Q = 4, C = 1: one workgroup per CU 2.24 us per row, two 2.8, four
// (three of them at a time) 5: one wave per SIMD leaves most issue slots empty.
inline double shared_step(int k) { return k <= 1 ? 1.0 : 0.15 + 0.55 * k; }

// Pick tiles and segments. With tile_rows > 0 the caller fixes the segment
// length; otherwise minimise the rounds of workgroups, each the rows walked
// per segment at the speed of the workgroups that then share a CU. Measured,
// coefficients at 1080p, Q = 4, C = 1: segments of 34 rows (one workgroup per
// CU) 88.7 us, of 17 (two) 62.8, of 9 (four) 68.9; Q = 6, C = 1 130 / 96.5. The
// same line serves the moments and the fused walk without averaging: 14 pairs
// of guides and channels, six sizes, r = 2, 8 and 24, none slower than with one
// workgroup per CU.
// K_MOMENTS, K_FUSED0 and K_COEFFS have no coefficient-row halo.
inline void plan_walk(int kind, int H, int W, int Q, int C, int r, int tile_rows, int* tiles_x,
                      int* n_seg, int* seg_rows) {
  const int tout = strip_out_cols(kind, r);
  *tiles_x = ceil_div(W, tout);
  if (tile_rows > 0) {
    *seg_rows = tile_rows < H ? tile_rows : H;
    *n_seg = ceil_div(H, *seg_rows);
    return;
  }
  const int hc = row_halo(kind, r);
  const int per_cu = workgroups_per_cu(kind, Q, C);
  double best = 1e300;
  int best_n = 1;
  const int nmax = H < 4096 ? H : 4096;
  for (int n = 1; n <= nmax; ++n) {
    const int R = ceil_div(H, n);
    if (n > 1 && ceil_div(H, n - 1) == R) continue;
    const int wgs = *tiles_x * n;
    const int full = wgs / (kCUs * per_cu), rest = wgs - full * kCUs * per_cu;
    const double rounds = full * shared_step(per_cu) +
                          (rest > 0 ? shared_step(ceil_div(rest, kCUs)) : 0.0);
    // rows solved per segment plus a share for the moment warm-up rows
    const double cost = rounds * ((double)R + 2.0 * hc + 0.5 * r) + 1e-3 * n;
    if (cost < best) {
      best = cost;
      best_n = n;
    }
  }
  *seg_rows = ceil_div(H, best_n);
  *n_seg = ceil_div(H, *seg_rows);
}

// LDS of the persistent batch kernel: the larger of the walk's and the
// averaging kernel's (its box items use the ring where it fits in that).
inline size_t batch_lds_bytes(int Q, int C) {
  const size_t w = walk_lds_bytes(K_COEFFS, Q, C), v = avg_lds_bytes(kAvgTileRows);
  const size_t u = lr_apply_lds_bytes(Q, C, 2, 1), m = w > v ? w : v;
  return u > m ? u : m;
}

// Split walks: when a moment walker's channels exceed what stays resident in
// LDS between rows (two groups of max_lds_rows FP64 rows for 256 columns),
// the product channels are walked in two slices, each with the first
// moments: [0, split_first) then the rest. Only where both slices fit.
__host__ __device__ constexpr int num_products(int Q, int C) { return Q * (Q + 1) / 2 + Q * C; }
__host__ __device__ constexpr int resident_channels() { return 2 * max_lds_rows(8); }
__host__ __device__ constexpr int split_first(int Q, int C) { return (num_products(Q, C) + 1) / 2; }
__host__ __device__ constexpr bool split_walk(int Q, int C) {
  return num_sums(Q, C) > resident_channels() &&
         Q + C + split_first(Q, C) <= resident_channels();
}

inline size_t ring_bytes_per_block(int Q, int C, int r) {
  return (size_t)(2 * r + 1) * (Q + 1) * C * kThreads * sizeof(ring_t);
}

// Per-guide-count dispatch entry points (one translation unit each).
#define FLR_DECLARE_Q(q) \
  hipError_t launch_q##q(int C, int kind, const LaunchArgs& a, hipStream_t s);
FLR_DECLARE_Q(1)
FLR_DECLARE_Q(2)
FLR_DECLARE_Q(3)
FLR_DECLARE_Q(4)
FLR_DECLARE_Q(5)
FLR_DECLARE_Q(6)
FLR_DECLARE_Q(7)
FLR_DECLARE_Q(8)
FLR_DECLARE_Q(9)
FLR_DECLARE_Q(10)
FLR_DECLARE_Q(11)
FLR_DECLARE_Q(12)
#undef FLR_DECLARE_Q

}  // namespace flr
