// The FLNR guide network (Sec. 3.3, the three-level 16/32/64 variant
// declared in include/flr_net.h) on the gfx950 matrix cores, and FLNR
// denoising (network, then FLR over the 12 guides).
//
// Every 3x3 layer is one implicit-GEMM kernel. Activations are BF16 in HWC order
// (channels innermost, a multiple of 16), so the 16 channels of one K step
// of a pixel are 32 contiguous bytes. With A = weights (c_out x k) and
// B = input (k x pixels), v_mfma_f32_16x16x16_bf16 gives lane l the
// accumulators of output channels 4*(l/16) .. +3 of pixel l % 16: four
// consecutive channels, stored as one 8-byte write, and exactly the B
// operand layout of a following 1x1 layer, which is therefore fused into the
// producing kernel (in3 + in1, out3 + out1). Upsampling and concatenation
// are folded into the consumer's staging. A workgroup of four waves computes
// four output rows from an input tile in LDS; weights are packed once into the
// per-lane fragment order, so each A operand is one contiguous 512-byte read
// per wave.
//
// What bounds it: 668 bytes per full-resolution pixel between the layers (270
// us at 1080p at the 5.2 TB/s of a large copy) and, per layer, staging and
// epilogue instructions beside few matrix instructions. Measured against
// 8-byte staging with per-chunk clamps, a separate pass for the input and the
// 64- and 96-channel layers reading operands from L2, 64 pixels per wave at
// every size: 1080p 802 -> 608 us (569 with the decoder's upsampled half staged
// at its own resolution); 256 x 256 137 -> 75 us (its half and quarter grids
// left most CUs idle).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>

#include "flr.h"
#include "flr_net.h"

// The workgroup's dynamic LDS (one array shared by every kernel of the library).
namespace flr {
extern __shared__ float lds[];
}

namespace flrnet {

typedef short bf16x4_t __attribute__((vector_size(8)));
typedef float f32x4_t __attribute__((vector_size(16)));

enum InKind : int { IN_HWC = 0, IN_PLANES = 1, IN_UPCAT = 2 };
enum Fuse : int { FUSE_NONE = 0, FUSE_1X1_RELU = 1, FUSE_1X1_SIGMOID = 2 };

struct ConvArgs {
  const uint16_t* in0;  // HWC BF16 input (IN_UPCAT: the low-resolution part)
  const uint16_t* in1;  // IN_UPCAT: the skip connection, on the conv's input grid
  const bf16x4_t* w;    // packed weight fragments of the layer
  const float* b;       // BF16-rounded bias (padded output channels)
  const bf16x4_t* w2;   // fused 1x1 layer
  const float* b2;
  uint16_t* out;        // HWC BF16 output
  float* outf;          // FUSE_1X1_SIGMOID: planar FP32 output
  uint16_t* mid;        // fused layers: when set, the first layer's BF16
                        // activations are stored here too (HWC, 16 channels)
  const float* guides;  // IN_PLANES: the network's input planes,
  const float* noisy;
  uint16_t* x0;         // and, when set, its compressed BF16 copy (HWC, 16 channels)
  int Hi, Wi;           // input grid
  int Hl, Wl;           // IN_UPCAT: grid of in0
  int Ho, Wo;           // output grid
};

// FP32 -> BF16, round to nearest, ties to even (NaN stays NaN).
__device__ __forceinline__ uint16_t f2bf(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Four FP32 values rounded to BF16 (as f2bf; two conversion instructions).
__device__ __forceinline__ bf16x4_t round4(float a, float b, float c, float d);

__device__ __forceinline__ bf16x4_t pack4(uint16_t a, uint16_t b, uint16_t c, uint16_t d) {
  bf16x4_t v;
  v[0] = (short)a;
  v[1] = (short)b;
  v[2] = (short)c;
  v[3] = (short)d;
  return v;
}

#if defined(__gfx950__)
__device__ __forceinline__ bf16x4_t round4(float a, float b, float c, float d) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  typedef __bf16 h2 __attribute__((ext_vector_type(2)));
  const h2 v[2] = {__builtin_convertvector(f2{a, b}, h2), __builtin_convertvector(f2{c, d}, h2)};
  bf16x4_t r;
  __builtin_memcpy(&r, v, sizeof r);
  return r;
}
#else
__device__ __forceinline__ bf16x4_t round4(float a, float b, float c, float d) {
  return pack4(f2bf(a), f2bf(b), f2bf(c), f2bf(d));
}
#endif

// Network input at one pixel, channels c0 .. c0 + 7 of the 16 (8 guides, 3
// noisy planes, zero): sign(v) log(1 + |v|), rounded to BF16.
// (The hardware logarithm with a rounding correction took 35 us less of a
// 1080p forward, and moved 7 in a million of the BF16 values: not kept.)
__device__ __forceinline__ float compress(float v) { return copysignf(log1pf(fabsf(v)), v); }

__device__ __forceinline__ f32x4_t load_bias(const float* b) {
  return *reinterpret_cast<const f32x4_t*>(b);
}
__device__ __forceinline__ bf16x4_t relu_round(f32x4_t v) {
  return round4(fmaxf(v[0], 0.f), fmaxf(v[1], 0.f), fmaxf(v[2], 0.f), fmaxf(v[3], 0.f));
}

// Bias, ReLU and store of TPW tiles of one output row (lane l: channels
// 4*(l/16)..+3 of each 16-channel block, pixel px0 + 16 t + l % 16), or the
// fused 1x1 layer on those activations.
template <int COUT, int FUSE, int COUT2, int TPW>
__device__ __forceinline__ void epilogue(const ConvArgs& a, int y, int px0, int lane,
                                         const f32x4_t (&acc)[TPW][COUT / 16]) {
  constexpr int NB = COUT / 16;
  const int kq = lane >> 4;
  const size_t row = (size_t)y * a.Wo;
  if constexpr (FUSE == FUSE_NONE) {
    f32x4_t bias[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) bias[nb] = load_bias(a.b + nb * 16 + 4 * kq);
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const int px = px0 + t * 16 + (lane & 15);
      if (px >= a.Wo) continue;
      uint16_t* o = a.out + (row + px) * COUT + 4 * kq;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        *reinterpret_cast<bf16x4_t*>(o + nb * 16) = relu_round(acc[t][nb] + bias[nb]);
    }
  } else {
    static_assert(COUT == 16, "a fused 1x1 layer reads 16 channels");
    const f32x4_t bias = load_bias(a.b + 4 * kq);
    if constexpr (FUSE == FUSE_1X1_RELU) {
      constexpr int NB2 = COUT2 / 16;
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const int px = px0 + t * 16 + (lane & 15);
        // this layer's activations are the B operand of the 1x1 layer as they are
        const bf16x4_t hv = relu_round(acc[t][0] + bias);
        if (a.mid && px < a.Wo)
          *reinterpret_cast<bf16x4_t*>(a.mid + (row + px) * 16 + 4 * kq) = hv;
#pragma unroll
        for (int nb = 0; nb < NB2; ++nb) {
          f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f};
          d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a.w2[nb * 64 + lane], hv, d, 0, 0, 0);
          if (px < a.Wo)
            *reinterpret_cast<bf16x4_t*>(a.out + (row + px) * COUT2 + nb * 16 + 4 * kq) =
                relu_round(d + load_bias(a.b2 + nb * 16 + 4 * kq));
        }
      }
    } else {
      // Four output channels: the A operand repeats their rows in every row
      // group, so that each lane group holds all four at its pixel; group g
      // then finishes tile g: one sigmoid per lane and channel, and stores of
      // whole rows of pixels.
      static_assert(COUT2 == 4, "the head has four channels");
      const bf16x4_t w2 = a.w2[(lane & 48) | (lane & 3)];
      f32x4_t d = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        const int px = px0 + t * 16 + (lane & 15);
        const bf16x4_t hv = relu_round(acc[t][0] + bias);
        if (a.mid && px < a.Wo)
          *reinterpret_cast<bf16x4_t*>(a.mid + (row + px) * 16 + 4 * kq) = hv;
        f32x4_t e = f32x4_t{0.f, 0.f, 0.f, 0.f};
        e = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w2, hv, e, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = kq == t ? e[i] : d[i];
      }
      const int px = px0 + kq * 16 + (lane & 15);
      if (kq < TPW && px < a.Wo) {
        const size_t pl = (size_t)a.Ho * a.Wo;
#pragma unroll
        for (int c = 0; c < 4; ++c)
          a.outf[c * pl + row + px] = 1.f / (1.f + expf(-(d[c] + a.b2[c])));
      }
    }
  }
}

// One 3x3 layer (CIN, COUT multiples of 16; stride ST), bias and ReLU,
// optionally followed by a fused 1x1 layer to COUT2 channels (ReLU to HWC
// BF16, or sigmoid to planar FP32).
//
// A workgroup computes four output rows (one per wave) of 16 TPW pixels for
// all output channels. It first stages the input pixels of the tile with all
// their channels in LDS (16-byte chunks, zero outside the image; the network
// input's compression and the decoder's upsampling and concatenation happen
// here), then reads the MFMA B fragments from there. LDS holds one plane per
// 16-channel block, 32 bytes a pixel, so that the 16 pixels x 4 channel quads
// of a fragment are 512 consecutive bytes; at stride 2 the even columns of a
// row come first, then the odd ones, for the same reason. K steps run over
// taps, then channel blocks, whatever the tile: results do not depend on it.
template <int CIN, int ST, int TPW>
struct ConvTile {
  static constexpr int NCB = CIN / 16;
  static constexpr int SR = 3 * ST + 3, SP = (16 * TPW - 1) * ST + 3;  // staged rows, columns
  static constexpr int SPH = (SP + 1) / 2, SPL = ST == 2 ? 2 * SPH : SP;
  static constexpr size_t lds_bytes() { return (size_t)NCB * SR * SPL * 32; }
  // 16-channel unit of block cb, staged row sr, column sx
  __device__ static int unit(int cb, int sr, int sx) {
    return (cb * SR + sr) * SPL + (ST == 2 ? (sx & 1) * SPH + (sx >> 1) : sx);
  }
};

template <int CIN, int ST, int TPW, bool EDGE>
__device__ __forceinline__ void stage_tile(const ConvArgs& a, const int x0, const int y0) {
  using T = ConvTile<CIN, ST, TPW>;
  constexpr int NCH = CIN / 8;  // chunks per pixel
  constexpr int NIT = T::SR * T::SP * NCH, B = 4;
  uint4* st = reinterpret_cast<uint4*>(flr::lds);
  const int tid = threadIdx.x;
  const int yb = y0 * ST - 1, xb = x0 * ST - 1;  // the tile's first input pixel
#pragma unroll 1
  for (int b0 = 0; b0 < NIT; b0 += B * 256) {
    uint4 v[B];
    int dst[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int i = b0 + u * 256 + tid, ic = i < NIT ? i : NIT - 1;
      const int pix = ic / NCH, ch = ic - pix * NCH;
      const int sr = pix / T::SP, sx = pix - sr * T::SP;
      dst[u] = i < NIT ? T::unit(ch >> 1, sr, sx) * 2 + (ch & 1) : -1;
      int y = yb + sr, x = xb + sx;
      bool ok = true;
      if constexpr (EDGE) {
        ok = y >= 0 && y < a.Hi && x >= 0 && x < a.Wi;
        y = min(max(y, 0), a.Hi - 1);
        x = min(max(x, 0), a.Wi - 1);
      }
      const uint16_t* src = a.in0 + ((size_t)y * a.Wi + x) * CIN + ch * 8;
      v[u] = *reinterpret_cast<const uint4*>(src);
      if constexpr (EDGE) {
        const uint32_t keep = ok ? 0xffffffffu : 0u;
        v[u] = uint4{v[u].x & keep, v[u].y & keep, v[u].z & keep, v[u].w & keep};
      }
    }
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (dst[u] >= 0) st[dst[u]] = v[u];
  }
}

// [up2(in0), in1] of a tile: in0's pixels are staged at their own resolution,
// once instead of up to four times (4 rows of 8 TPW + 2 pixels), block after
// block, then in1's at full resolution. At the image's edge (EDGE) what lies
// outside is staged from clamped addresses and zeroed where fragments are read
// (a fine pixel past an odd edge shares its coarse pixel with one inside).
template <int CIN, int CUP, int TPW>
struct UpTile {
  using T = ConvTile<CIN - CUP, 1, TPW>;
  static constexpr int LR = 4, LP = 8 * TPW + 2, NCBL = CUP / 16;
  static constexpr int base = NCBL * LR * LP;  // units of in0, before in1's
  __device__ static int low(int cb, int lr, int lx) { return (cb * LR + lr) * LP + lx; }
  static constexpr size_t lds_bytes() { return (size_t)base * 32 + T::lds_bytes(); }
};
template <int CIN, int CUP, int TPW, bool EDGE>
__device__ __forceinline__ void stage_up(const ConvArgs& a, const int x0, const int y0) {
  using U = UpTile<CIN, CUP, TPW>;
  using T = typename U::T;
  constexpr int CL = CUP / 8, CS = (CIN - CUP) / 8;  // chunks per pixel
  constexpr int NL = U::LR * U::LP * CL, NIT = NL + T::SR * T::SP * CS, B = 6;
  uint4* st = reinterpret_cast<uint4*>(flr::lds);
  const int tid = threadIdx.x;
  const int ly = y0 / 2 - 1, lx0 = x0 / 2 - 1, hy = y0 - 1, hx = x0 - 1;  // first pixels
  const uint16_t* lo = a.in0 + (EDGE ? 0 : ((size_t)ly * a.Wl + lx0) * CUP);
  const uint16_t* hi = a.in1 + (EDGE ? 0 : ((size_t)hy * a.Wi + hx) * (CIN - CUP));
#pragma unroll 1
  for (int b0 = 0; b0 < NIT; b0 += B * 256) {
    uint4 v[B];
    int dst[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int i = b0 + u * 256 + tid, ic = i < NIT ? i : NIT - 1;
      const uint16_t* src;
      int d;
      if (ic < NL) {
        const int pix = ic / CL, ch = ic - pix * CL, lr = pix / U::LP, lx = pix - lr * U::LP;
        if constexpr (EDGE)
          src = lo + ((size_t)min(max(ly + lr, 0), a.Hl - 1) * a.Wl +
                      min(max(lx0 + lx, 0), a.Wl - 1)) * CUP + ch * 8;
        else
          src = lo + (unsigned)((lr * a.Wl + lx) * CUP + ch * 8);
        d = U::low(ch >> 1, lr, lx) * 2 + (ch & 1);
      } else {
        const int j = ic - NL, pix = j / CS, ch = j - pix * CS, sr = pix / T::SP,
                  sx = pix - sr * T::SP;
        if constexpr (EDGE)
          src = hi + ((size_t)min(max(hy + sr, 0), a.Hi - 1) * a.Wi +
                      min(max(hx + sx, 0), a.Wi - 1)) * (CIN - CUP) + ch * 8;
        else
          src = hi + (unsigned)((sr * a.Wi + sx) * (CIN - CUP) + ch * 8);
        d = (U::base + T::unit(ch >> 1, sr, sx)) * 2 + (ch & 1);
      }
      v[u] = *reinterpret_cast<const uint4*>(src);
      dst[u] = i < NIT ? d : -1;
    }
#pragma unroll
    for (int u = 0; u < B; ++u)
      if (dst[u] >= 0) st[dst[u]] = v[u];
  }
}

// The network's input (IN_PLANES): compressed while it is staged, one pixel
// per lane; x0, when set, receives the tile's own pixels (HWC, 16 channels).
template <int TPW>
__device__ __forceinline__ void stage_input(const ConvArgs& a, const int x0, const int y0) {
  using T = ConvTile<16, 1, TPW>;
  constexpr int NPX = T::SR * T::SP, NIN = FLR_NET_IN_GUIDES + FLR_NET_IN_NOISY;
  bf16x4_t* st = reinterpret_cast<bf16x4_t*>(flr::lds);
  const size_t pl = (size_t)a.Hi * a.Wi;
#pragma unroll 1
  for (int i = threadIdx.x; i < NPX; i += 256) {
    const int sr = i / T::SP, sx = i - sr * T::SP;
    const int y = y0 - 1 + sr, x = x0 - 1 + sx;
    const bool ok = y >= 0 && y < a.Hi && x >= 0 && x < a.Wi;
    const size_t p = (size_t)min(max(y, 0), a.Hi - 1) * a.Wi + min(max(x, 0), a.Wi - 1);
    float v[12];
#pragma unroll
    for (int c = 0; c < NIN; ++c)
      v[c] = c < FLR_NET_IN_GUIDES ? a.guides[c * pl + p] : a.noisy[(c - FLR_NET_IN_GUIDES) * pl + p];
#pragma unroll
    for (int c = 0; c < 12; ++c) v[c] = c < NIN && ok ? compress(v[c]) : 0.f;
    bf16x4_t h[4];
#pragma unroll
    for (int q = 0; q < 3; ++q) h[q] = round4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    h[3] = pack4(0, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) st[T::unit(0, sr, sx) * 4 + q] = h[q];
    if (a.x0 && ok && sr >= 1 && sr <= 4 && sx >= 1 && sx <= 16 * TPW) {
      bf16x4_t* o = reinterpret_cast<bf16x4_t*>(a.x0 + p * 16);
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = h[q];
    }
  }
}

// The matrix products of one wave's output row from the staged tile, and the
// epilogue. LOW: staged by stage_up, EDGE: at the image's edge.
template <int CIN, int COUT, int ST, int CUP, int FUSE, int COUT2, int TPW, bool LOW,
          bool EDGE>
__device__ __forceinline__ void conv_row(const ConvArgs& a, const int x0, const int y0,
                                         const int wv) {
  using T = ConvTile<CIN, ST, TPW>;
  constexpr int NCB = T::NCB, NB = COUT / 16;
  const int lane = threadIdx.x & 63, kq = lane >> 4, lx = lane & 15;
  const bf16x4_t* st = reinterpret_cast<const bf16x4_t*>(flr::lds);
  auto frag = [&](int ky, int kx, int cb, int t) {
    if constexpr (LOW) {
      using U = UpTile<CIN, CUP, TPW>;
      const int u = cb < U::NCBL
                        ? U::low(cb, (wv + ky + 1) >> 1, ((lx + kx + 1) >> 1) + t * 8)
                        : U::base + U::T::unit(cb - U::NCBL, wv + ky, kx) + t * 16 + lx;
      bf16x4_t v = st[u * 4 + kq];
      if constexpr (EDGE) {
        const int y = y0 + wv + ky - 1, x = x0 + t * 16 + lx + kx - 1;
        const bool in = y >= 0 && y < a.Hi && x >= 0 && x < a.Wi;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = in ? v[j] : (short)0;
      }
      return v;
    } else {
      return st[(T::unit(cb, wv * ST + ky, kx) + t * 16 + lx) * 4 + kq];
    }
  };
  // partial sums (K steps round-robin) for layers of one output block, so
  // that enough independent MFMA chains are in flight per wave
  constexpr int KSPL = NB >= 2 ? 1 : 2;
  f32x4_t acc[TPW][NB][KSPL];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int k = 0; k < KSPL; ++k) acc[t][nb][k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ky = 0; ky < 3; ++ky) {
#pragma unroll
    for (int kx = 0; kx < 3; ++kx) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const int tap = ky * 3 + kx;
        const int ks = (tap * NCB + cb) % KSPL;
        bf16x4_t bv[TPW];
#pragma unroll
        for (int t = 0; t < TPW; ++t) bv[t] = frag(ky, kx, cb, t);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const bf16x4_t av = a.w[((tap * NCB + cb) * NB + nb) * 64 + lane];
#pragma unroll
          for (int t = 0; t < TPW; ++t)
            acc[t][nb][ks] =
                __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, bv[t], acc[t][nb][ks], 0, 0, 0);
        }
      }
    }
  }
  f32x4_t sum[TPW][NB];
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      sum[t][nb] = acc[t][nb][0];
#pragma unroll
      for (int k = 1; k < KSPL; ++k) sum[t][nb] += acc[t][nb][k];
    }
  epilogue<COUT, FUSE, COUT2, TPW>(a, y0 + wv, x0, lane, sum);
}

template <int CIN, int COUT, int ST, int IN, int CUP, int FUSE, int COUT2, int TPW>
__global__ void __launch_bounds__(256) conv_kernel(ConvArgs a) {
  using T = ConvTile<CIN, ST, TPW>;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int x0 = blockIdx.x * 16 * TPW, y0 = blockIdx.y * 4;
  const bool edge = x0 == 0 || y0 == 0 || x0 * ST - 1 + T::SP > a.Wi ||
                    y0 * ST - 1 + T::SR > a.Hi;
  if constexpr (IN == IN_PLANES) {
    stage_input<TPW>(a, x0, y0);
  } else if constexpr (IN == IN_UPCAT) {
    if (edge)  // uniform across the workgroup
      stage_up<CIN, CUP, TPW, true>(a, x0, y0);
    else
      stage_up<CIN, CUP, TPW, false>(a, x0, y0);
    __syncthreads();
    if (y0 + wv >= a.Ho) return;
    if (edge)
      conv_row<CIN, COUT, ST, CUP, FUSE, COUT2, TPW, true, true>(a, x0, y0, wv);
    else
      conv_row<CIN, COUT, ST, CUP, FUSE, COUT2, TPW, true, false>(a, x0, y0, wv);
    return;
  } else {
    if (edge)
      stage_tile<CIN, ST, TPW, true>(a, x0, y0);
    else
      stage_tile<CIN, ST, TPW, false>(a, x0, y0);
  }
  __syncthreads();
  if (y0 + wv >= a.Ho) return;  // uniform across the wave; no barrier follows
  conv_row<CIN, COUT, ST, CUP, FUSE, COUT2, TPW, false, false>(a, x0, y0, wv);
}

// Packing: FP32 weight [cout][cin][k][k] -> fragments (tap, cin block,
// cout block, lane) of 4 BF16, lane l holding output channel 16*nb + l%16
// and input channels 16*cb + 4*(l/16) .. +3; zero in the padding.
struct PackArgs {
  const float* w;  // [cout][cin][ks][ks]
  const float* b;  // [cout]
  int cin, cout, ks, ncb, nb;
  bf16x4_t* wp;    // fragments
  float* bp;       // [16 * nb]
};
__global__ void pack_kernel(PackArgs p) {
  const float* w = p.w;
  const float* b = p.b;
  const int cin = p.cin, cout = p.cout, ks = p.ks, ncb = p.ncb, nb = p.nb;
  bf16x4_t* wp = p.wp;
  float* bp = p.bp;
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  const int nfrag = ks * ks * ncb * nb * 64;
  if (idx < nfrag) {
    const int lane = idx % 64;
    const int n = (idx / 64) % nb;
    const int cb = (idx / 64 / nb) % ncb;
    const int tap = idx / (64 * nb * ncb);
    const int ky = tap / ks, kx = tap % ks;
    const int co = n * 16 + lane % 16;
    uint16_t h[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int ci = cb * 16 + 4 * (lane / 16) + j;
      h[j] = (co < cout && ci < cin) ? f2bf(w[((co * cin + ci) * ks + ky) * ks + kx]) : (uint16_t)0;
    }
    wp[idx] = pack4(h[0], h[1], h[2], h[3]);
  }
  if (idx < nb * 16) bp[idx] = idx < cout ? bf2f(f2bf(b[idx])) : 0.f;
}

// ---------------------------------------------------------------------------
// Host side: layer table, packed-block and workspace layout, launches.

struct Layer {
  int cin, cout, k, stride;
};
constexpr Layer kLayers[12] = {
    {11, 16, 3, 1},  // in3
    {16, 16, 1, 1},  // in1
    {16, 32, 3, 1},  // e1a
    {32, 32, 3, 2},  // e1b
    {32, 64, 3, 1},  // e2a
    {64, 64, 3, 2},  // e2b
    {96, 32, 3, 1},  // d1a
    {32, 32, 3, 1},  // d1b
    {48, 16, 3, 1},  // d0a
    {16, 16, 3, 1},  // d0b
    {16, 16, 3, 1},  // out3
    {16, 4, 1, 1},   // out1
};
constexpr int pad16(int n) { return (n + 15) / 16 * 16; }
inline size_t frag_count(const Layer& L) {
  return (size_t)L.k * L.k * (pad16(L.cin) / 16) * (pad16(L.cout) / 16) * 64;
}
inline size_t packed_layer_bytes(const Layer& L) {
  return frag_count(L) * sizeof(bf16x4_t) + pad16(L.cout) * sizeof(float);
}
inline size_t param_offset(int i) {
  size_t o = 0;
  for (int j = 0; j < i; ++j) o += (size_t)kLayers[j].cout * kLayers[j].cin * kLayers[j].k * kLayers[j].k + kLayers[j].cout;
  return o;
}
inline size_t packed_offset(int i) {
  size_t o = 0;
  for (int j = 0; j < i; ++j) o += packed_layer_bytes(kLayers[j]);
  return o;
}
inline const bf16x4_t* layer_w(const void* packed, int i) {
  return reinterpret_cast<const bf16x4_t*>(static_cast<const char*>(packed) + packed_offset(i));
}
inline const float* layer_b(const void* packed, int i) {
  return reinterpret_cast<const float*>(static_cast<const char*>(packed) + packed_offset(i) +
                                        frag_count(kLayers[i]) * sizeof(bf16x4_t));
}

// Activation buffers in the workspace, in order: x0 (the prepared input,
// 16, full), e0 (16, full), t1 (32, full), e1 (32, half), t2 (64, half),
// e2 (64, quarter), t3 (32, half), d1 (32, half), t4 (16, full), t5 (16,
// full).
struct Grids {
  int H, W, Hh, Wh, Hq, Wq;
};
inline Grids grids(int H, int W) {
  Grids g{H, W, (H + 1) / 2, (W + 1) / 2, 0, 0};
  g.Hq = (g.Hh + 1) / 2;
  g.Wq = (g.Wh + 1) / 2;
  return g;
}
inline size_t align256(size_t n) { return (n + 255) / 256 * 256; }
constexpr int kActBufs = 10;
inline void act_layout(const Grids& g, size_t off[kActBufs + 1]) {
  const size_t full = (size_t)g.H * g.W * 2, half = (size_t)g.Hh * g.Wh * 2,
               quarter = (size_t)g.Hq * g.Wq * 2;
  const size_t sz[kActBufs] = {16 * full, 16 * full, 32 * full, 32 * half, 64 * half,
                               64 * quarter, 32 * half, 32 * half, 16 * full, 16 * full};
  off[0] = 0;
  for (int i = 0; i < kActBufs; ++i) off[i + 1] = off[i] + align256(sz[i]);
}

// Forward trace (flr_net_forward_trace): every layer's output activation,
// in the order of the header's layer table: x0 (the prepared input), in3,
// e0, e1a, e1, e2a, e2, d1a, d1, d0a, d0b, out3. The forward's own buffers
// (act_layout) come first; in3's and out3's outputs follow them.
constexpr int kTraceTensors = 12;
constexpr int kTraceChannels[kTraceTensors] = {16, 16, 16, 32, 32, 64, 64, 32, 32, 16, 16, 16};
constexpr int kTraceGrid[kTraceTensors] = {0, 0, 0, 0, 1, 1, 2, 1, 1, 0, 0, 0};
// trace index -> act_layout buffer (-1: the two stored after them)
constexpr int kTraceAct[kTraceTensors] = {0, -1, 1, 2, 3, 4, 5, 6, 7, 8, 9, -1};
inline void trace_layout(const Grids& g, size_t off[kTraceTensors + 1]) {
  size_t act[kActBufs + 1];
  act_layout(g, act);
  const size_t full16 = align256((size_t)g.H * g.W * 2 * 16);
  for (int i = 0; i < kTraceTensors; ++i)
    if (kTraceAct[i] >= 0) off[i] = act[kTraceAct[i]];
  off[1] = act[kActBufs];
  off[11] = act[kActBufs] + full16;
  off[kTraceTensors] = act[kActBufs] + 2 * full16;
}

bool valid_dims(int H, int W) {
  return H >= 1 && W >= 1 && H <= FLR_MAX_DIM && W <= FLR_MAX_DIM &&
         (int64_t)H * W <= ((int64_t)1 << 28);
}
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
  return a0 < b0 + nb && b0 < a0 + na;
}

template <int CIN, int ST, int IN, int CUP, int TPW>
constexpr size_t conv_lds_bytes() {
  if constexpr (IN == IN_UPCAT)
    return UpTile<CIN, CUP, TPW>::lds_bytes();
  else
    return ConvTile<CIN, ST, TPW>::lds_bytes();
}
// Tiles of 64 pixels where they give kConvMinGroups workgroups (two per CU),
// else 32, else 16: at training-crop sizes the half and quarter grids would
// otherwise leave most CUs idle. Stride 2 and the 96-channel layer: at most 32
// pixels (their staged tiles would keep too few workgroups on a CU).
constexpr int kConvMinGroups = 512;
template <int CIN, int COUT, int ST, int IN, int CUP, int FUSE, int COUT2, int TPW>
hipError_t launch_tpw(const ConvArgs& a, hipStream_t s) {
  auto k = conv_kernel<CIN, COUT, ST, IN, CUP, FUSE, COUT2, TPW>;
  const size_t lds = conv_lds_bytes<CIN, ST, IN, CUP, TPW>();
  if (lds > 65536) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3((a.Wo + 16 * TPW - 1) / (16 * TPW), (a.Ho + 3) / 4), dim3(256), lds, s,
                     a);
  return hipGetLastError();
}
template <int CIN, int COUT, int ST, int IN, int CUP, int FUSE, int COUT2>
hipError_t launch(const ConvArgs& a, hipStream_t s) {
  constexpr int MAX = CIN * ST >= 64 ? 2 : 4;
  const int rows = (a.Ho + 3) / 4;
  if constexpr (MAX == 4)
    if ((a.Wo + 63) / 64 * rows >= kConvMinGroups)
      return launch_tpw<CIN, COUT, ST, IN, CUP, FUSE, COUT2, 4>(a, s);
  if ((a.Wo + 31) / 32 * rows >= kConvMinGroups)
    return launch_tpw<CIN, COUT, ST, IN, CUP, FUSE, COUT2, 2>(a, s);
  return launch_tpw<CIN, COUT, ST, IN, CUP, FUSE, COUT2, 1>(a, s);
}

// The forward pass into the activation buffers at the start of ws (the
// act_layout offsets), the sigmoid output planar FP32 into out. When set,
// mid_in3 and mid_out3 receive the activations of in3 and out3, which the
// fused kernels otherwise keep in registers (HWC BF16, 16 channels, full
// resolution).
flr_status run_forward(const Grids& g, const float* guides, const float* noisy, const void* packed,
                       float* out, char* ws, hipStream_t s, uint16_t* mid_in3 = nullptr,
                       uint16_t* mid_out3 = nullptr) {
  size_t off[kActBufs + 1];
  act_layout(g, off);
  auto buf = [&](int i) { return reinterpret_cast<uint16_t*>(ws + off[i]); };
  uint16_t *x0 = buf(0), *e0 = buf(1), *t1 = buf(2), *e1 = buf(3), *t2 = buf(4), *e2 = buf(5),
           *t3 = buf(6), *d1 = buf(7), *t4 = buf(8), *t5 = buf(9);
  auto args = [&](int layer, int Hi, int Wi, int Ho, int Wo) {
    ConvArgs a = {};
    a.w = layer_w(packed, layer);
    a.b = layer_b(packed, layer);
    a.Hi = Hi;
    a.Wi = Wi;
    a.Ho = Ho;
    a.Wo = Wo;
    return a;
  };
  hipError_t e;
  {  // in3 + in1 -> e0
    ConvArgs a = args(0, g.H, g.W, g.H, g.W);
    a.guides = guides;
    a.noisy = noisy;
    a.x0 = mid_in3 ? x0 : nullptr;  // the backward and the trace read it
    a.w2 = layer_w(packed, 1);
    a.b2 = layer_b(packed, 1);
    a.out = e0;
    a.mid = mid_in3;
    if ((e = launch<16, 16, 1, IN_PLANES, 0, FUSE_1X1_RELU, 16>(a, s)) != hipSuccess) return FLR_ERR_HIP;
  }
  {  // e1a
    ConvArgs a = args(2, g.H, g.W, g.H, g.W);
    a.in0 = e0;
    a.out = t1;
    if ((e = launch<16, 32, 1, IN_HWC, 0, FUSE_NONE, 0>(a, s)) != hipSuccess) return FLR_ERR_HIP;
  }
  {  // e1b (stride 2)
    ConvArgs a = args(3, g.H, g.W, g.Hh, g.Wh);
    a.in0 = t1;
    a.out = e1;
    if ((e = launch<32, 32, 2, IN_HWC, 0, FUSE_NONE, 0>(a, s)) != hipSuccess) return FLR_ERR_HIP;
  }
  {  // e2a
    ConvArgs a = args(4, g.Hh, g.Wh, g.Hh, g.Wh);
    a.in0 = e1;
    a.out = t2;
    if ((e = launch<32, 64, 1, IN_HWC, 0, FUSE_NONE, 0>(a, s)) != hipSuccess) return FLR_ERR_HIP;
  }
  {  // e2b (stride 2)
    ConvArgs a = args(5, g.Hh, g.Wh, g.Hq, g.Wq);
    a.in0 = t2;
    a.out = e2;
    if ((e = launch<64, 64, 2, IN_HWC, 0, FUSE_NONE, 0>(a, s)) != hipSuccess) return FLR_ERR_HIP;
  }
  {  // d1a: [up2(e2), e1]
    ConvArgs a = args(6, g.Hh, g.Wh, g.Hh, g.Wh);
    a.in0 = e2;
    a.Hl = g.Hq;
    a.Wl = g.Wq;
    a.in1 = e1;
    a.out = t3;
    if ((e = launch<96, 32, 1, IN_UPCAT, 64, FUSE_NONE, 0>(a, s)) != hipSuccess) return FLR_ERR_HIP;
  }
  {  // d1b
    ConvArgs a = args(7, g.Hh, g.Wh, g.Hh, g.Wh);
    a.in0 = t3;
    a.out = d1;
    if ((e = launch<32, 32, 1, IN_HWC, 0, FUSE_NONE, 0>(a, s)) != hipSuccess) return FLR_ERR_HIP;
  }
  {  // d0a: [up2(d1), e0]
    ConvArgs a = args(8, g.H, g.W, g.H, g.W);
    a.in0 = d1;
    a.Hl = g.Hh;
    a.Wl = g.Wh;
    a.in1 = e0;
    a.out = t4;
    if ((e = launch<48, 16, 1, IN_UPCAT, 32, FUSE_NONE, 0>(a, s)) != hipSuccess) return FLR_ERR_HIP;
  }
  {  // d0b
    ConvArgs a = args(9, g.H, g.W, g.H, g.W);
    a.in0 = t4;
    a.out = t5;
    if ((e = launch<16, 16, 1, IN_HWC, 0, FUSE_NONE, 0>(a, s)) != hipSuccess) return FLR_ERR_HIP;
  }
  {  // out3 + out1 (sigmoid) -> planar FP32
    ConvArgs a = args(10, g.H, g.W, g.H, g.W);
    a.in0 = t5;
    a.w2 = layer_w(packed, 11);
    a.b2 = layer_b(packed, 11);
    a.outf = out;
    a.mid = mid_out3;
    if ((e = launch<16, 16, 1, IN_HWC, 0, FUSE_1X1_SIGMOID, FLR_NET_OUT>(a, s)) != hipSuccess)
      return FLR_ERR_HIP;
  }
  return FLR_OK;
}


}  // namespace flrnet

#include "flr_net_bwd.hpp"

namespace flrnet {

// Backward workspace: the forward's activation buffers (act_layout), then
// in3's and out3's activations (fused away in the forward), the sigmoid
// output, the data-gradient weights, the FP32 gradient tensors and the
// weight gradients' partial sums (every layer's: they are formed in one
// launch).
enum BwdBuf : int {
  B_A, B_T6, B_SIG, B_WD, B_DZ1, B_GT6, B_GT5, B_GT4, B_G48, B_GT3, B_G96, B_GT2, B_GE1, B_GT1,
  B_GE0, B_GA, B_PART, B_COUNT
};
// Input and output grid of each layer: 0 full, 1 half, 2 quarter.
constexpr int kInGrid[12] = {0, 0, 0, 0, 1, 1, 1, 1, 0, 0, 0, 0};
constexpr int kOutGrid[12] = {0, 0, 0, 1, 1, 2, 1, 1, 0, 0, 0, 0};

inline int grid_h(const Grids& g, int which) { return which == 0 ? g.H : which == 1 ? g.Hh : g.Hq; }
inline int grid_w(const Grids& g, int which) { return which == 0 ? g.W : which == 1 ? g.Wh : g.Wq; }

// Layers with a data gradient through dgrad_kernel: all but the first (its
// input is the network's) and the last (head_bwd_kernel).
inline bool has_dgrad(int li) { return li >= 1 && li <= 10; }
// First data-gradient fragment of layer i (i = 12: their count).
inline size_t dfrag_offset(int i) {
  size_t o = 0;
  for (int j = 0; j < i; ++j)
    if (has_dgrad(j)) o += frag_count(kLayers[j]);
  return o;
}

inline void bwd_layout(const Grids& g, size_t off[B_COUNT + 1]) {
  size_t act[kActBufs + 1];
  act_layout(g, act);
  const size_t F = (size_t)g.H * g.W, Hf = (size_t)g.Hh * g.Wh;
  size_t part = 0;
  for (int li = 0; li < 12; ++li) {
    const WgradPlan wp = wgrad_plan(kLayers[li], grid_h(g, kOutGrid[li]), grid_w(g, kOutGrid[li]));
    part += wgrad_part_floats(kLayers[li], wp);
  }
  const size_t sz[B_COUNT] = {16 * F * 2,  16 * F * 2,  4 * F * 4,   dfrag_offset(12) * 8,
                              4 * F * 4,   16 * F * 4,  16 * F * 4,  16 * F * 4,
                              48 * F * 4,  32 * Hf * 4, 96 * Hf * 4, 64 * Hf * 4,
                              32 * Hf * 4, 32 * F * 4,  16 * F * 4,  16 * F * 4,
                              part * 4};
  off[0] = act[kActBufs];
  for (int i = 0; i < B_COUNT; ++i) off[i + 1] = off[i] + align256(sz[i]);
}

// Data gradient of a layer. Workgroups take two 16-channel blocks of dx
// (the staged tile serves both) and 64 pixels of four rows; on grids that
// would leave most CUs idle 32 pixels (kDgNarrowGroups workgroups of 64). A
// dx's sums are the same either way. FLR_DGRAD_WIDE_PX in the environment, when
// it holds a number, sets the line in pixels of dx instead (a tuning knob).
constexpr int kDgNarrowGroups = 256;
inline int64_t dgrad_wide_px() {
  const char* e = getenv("FLR_DGRAD_WIDE_PX");
  if (e && *e) {
    char* end = nullptr;
    const long long v = strtoll(e, &end, 10);
    if (end && *end == 0 && v >= 0) return v;
  }
  return -1;
}
template <int CIN, int COUT, int KS, int ST, int CBG, int NT>
hipError_t launch_dgrad_nt(const DgradArgs& a, hipStream_t s) {
  // tiles of dx pixels (stride 2: of the coarse grid covering dx)
  const int Ht = (a.Hi + ST - 1) / ST, Wt = (a.Wi + ST - 1) / ST;
  hipLaunchKernelGGL((dgrad_kernel<CIN, COUT, KS, ST, CBG, NT>),
                     dim3((Wt + 16 * NT - 1) / (16 * NT) * (CIN / 16 / CBG), (Ht + 3) / 4), dim3(256),
                     (dgrad_lds_bytes<KS, ST, NT>()), s, a);
  return hipGetLastError();
}
template <int CIN, int COUT, int KS, int ST>
hipError_t launch_dgrad(const DgradArgs& a, int64_t wide_px, hipStream_t s) {
  constexpr int CBG = CIN % 32 == 0 ? 2 : 1;
  const int Ht = (a.Hi + ST - 1) / ST, Wt = (a.Wi + ST - 1) / ST;
  const bool wide = wide_px >= 0 ? (int64_t)a.Hi * a.Wi >= wide_px
                                 : (Wt + 63) / 64 * ((Ht + 3) / 4) * (CIN / 16 / CBG) >=
                                       kDgNarrowGroups;
  if constexpr (ST == 1) {
    if (wide) return launch_dgrad_nt<CIN, COUT, KS, ST, CBG, 4>(a, s);
    return launch_dgrad_nt<CIN, COUT, KS, ST, CBG, 2>(a, s);
  } else {  // four parities' sums per pixel: 32 pixels, or 16
    if (wide) return launch_dgrad_nt<CIN, COUT, KS, ST, CBG, 2>(a, s);
    return launch_dgrad_nt<CIN, COUT, KS, ST, CBG, 1>(a, s);
  }
}

flr_status run_backward(const Grids& g, const float* guides, const float* noisy,
                        const float* params, const void* packed, const float* dout, float* grad,
                        int accumulate, char* ws, hipStream_t s) {
  size_t act[kActBufs + 1], off[B_COUNT + 1];
  act_layout(g, act);
  bwd_layout(g, off);
  auto abuf = [&](int i) { return reinterpret_cast<uint16_t*>(ws + act[i]); };
  auto fbuf = [&](int i) { return reinterpret_cast<float*>(ws + off[i]); };
  uint16_t *x0 = abuf(0), *e0 = abuf(1), *t1 = abuf(2), *e1 = abuf(3), *t2 = abuf(4),
           *e2 = abuf(5), *t3 = abuf(6), *d1 = abuf(7), *t4 = abuf(8), *t5 = abuf(9);
  uint16_t* a16 = reinterpret_cast<uint16_t*>(ws + off[B_A]);
  uint16_t* t6 = reinterpret_cast<uint16_t*>(ws + off[B_T6]);
  bf16x4_t* wd = reinterpret_cast<bf16x4_t*>(ws + off[B_WD]);
  float* sig = fbuf(B_SIG);
  const int F = g.H * g.W;

  BwdPackArgs pk = {};
  pk.params = params;
  pk.out = wd;
  for (int li = 0; li < 12; ++li) {
    pk.first[li] = (int)dfrag_offset(li);
    pk.param[li] = (int)param_offset(li);
    pk.cin[li] = kLayers[li].cin;
    pk.cout[li] = kLayers[li].cout;
    pk.k[li] = kLayers[li].k;
  }
  pk.first[12] = (int)dfrag_offset(12);
  hipLaunchKernelGGL(bwd_pack_kernel, dim3((pk.first[12] + 255) / 256), dim3(256), 0, s, pk);
  if (hipGetLastError() != hipSuccess) return FLR_ERR_HIP;
  // the forward, also storing in3's and out3's activations
  flr_status st = run_forward(g, guides, noisy, packed, sig, ws, s, a16, t6);
  if (st != FLR_OK) return st;
  const HeadBwdArgs ha = {dout, sig, params + param_offset(11), fbuf(B_DZ1), fbuf(B_GT6), F};
  hipLaunchKernelGGL(head_bwd_kernel, dim3((F + 255) / 256), dim3(256), 0, s, ha);
  if (hipGetLastError() != hipSuccess) return FLR_ERR_HIP;

  // each layer's dz (output gradient and ReLU mask) and input
  auto dzs = [](const float* go, const uint16_t* ac, int cout) {
    return DzSrc{go, ac, cout, cout, 0, 0, 0};
  };
  auto up2 = [](const float* go, const uint16_t* ac, int cs, int cout, int Hf, int Wf) {
    return DzSrc{go, ac, cs, cout, 1, Hf, Wf};
  };
  auto plain = [](const uint16_t* in, int cs) { return BwdSrc{in, nullptr, cs, cs, 0, 0}; };
  const DzSrc dz[12] = {
      dzs(fbuf(B_GA), a16, 16),  dzs(fbuf(B_GE0), e0, 16), dzs(fbuf(B_GT1), t1, 32),
      dzs(fbuf(B_GE1), e1, 32),  dzs(fbuf(B_GT2), t2, 64),
      up2(fbuf(B_G96), e2, 96, 64, g.Hh, g.Wh),  // e2 through up2 and d1a
      dzs(fbuf(B_GT3), t3, 32),
      up2(fbuf(B_G48), d1, 48, 32, g.H, g.W),    // d1 through up2 and d0a
      dzs(fbuf(B_GT4), t4, 16),  dzs(fbuf(B_GT5), t5, 16), dzs(fbuf(B_GT6), t6, 16),
      dzs(fbuf(B_DZ1), nullptr, FLR_NET_OUT)};
  const BwdSrc src[12] = {
      plain(x0, 16), plain(a16, 16), plain(e0, 16), plain(t1, 32), plain(e1, 32), plain(t2, 64),
      BwdSrc{e2, e1, 64, 64, 32, g.Wq}, plain(t3, 32), BwdSrc{d1, e0, 32, 32, 16, g.Wh},
      plain(t4, 16), plain(t5, 16), plain(t6, 16)};
  bool ok = true;
  const int64_t wide_px = dgrad_wide_px();
  auto D = [&](auto kernel, int li, float* dx, const float* add = nullptr, int add_cs = 0,
               int add_off = 0) {
    DgradArgs a = {};
    a.dz = dz[li];
    a.w = wd + dfrag_offset(li);
    a.Hi = grid_h(g, kInGrid[li]);
    a.Wi = grid_w(g, kInGrid[li]);
    a.Ho = grid_h(g, kOutGrid[li]);
    a.Wo = grid_w(g, kOutGrid[li]);
    a.dx = dx;
    a.add = add;
    a.add_cs = add_cs;
    a.add_off = add_off;
    ok = ok && kernel(a, wide_px, s) == hipSuccess;
  };
  // from out3 back to in1, as in the forward reversed
  D(launch_dgrad<16, 16, 3, 1>, 10, fbuf(B_GT5));
  D(launch_dgrad<16, 16, 3, 1>, 9, fbuf(B_GT4));
  D(launch_dgrad<48, 16, 3, 1>, 8, fbuf(B_G48));
  D(launch_dgrad<32, 32, 3, 1>, 7, fbuf(B_GT3));
  D(launch_dgrad<96, 32, 3, 1>, 6, fbuf(B_G96));
  D(launch_dgrad<64, 64, 3, 2>, 5, fbuf(B_GT2));
  D(launch_dgrad<32, 64, 3, 1>, 4, fbuf(B_GE1), fbuf(B_G96), 96, 64);
  D(launch_dgrad<32, 32, 3, 2>, 3, fbuf(B_GT1));
  D(launch_dgrad<16, 32, 3, 1>, 2, fbuf(B_GE0), fbuf(B_G48), 48, 32);
  D(launch_dgrad<16, 16, 1, 1>, 1, fbuf(B_GA));
  // every layer's weight and bias gradients
  WgradArgs w = {};
  w.accumulate = accumulate;
  float* part = fbuf(B_PART);
  for (int li = 0; li < 12; ++li) {
    const Layer& L = kLayers[li];
    const int Ho = grid_h(g, kOutGrid[li]), Wo = grid_w(g, kOutGrid[li]);
    const WgradPlan p = wgrad_plan(L, Ho, Wo);
    w.layer[li] = WgradLayer{dz[li], src[li], grid_h(g, kInGrid[li]), grid_w(g, kInGrid[li]), Ho,
                             Wo, p.ncb, p.npair, L.k, L.stride, p.tiles_x, p.ntile, p.chunk,
                             p.nchunk, part, L.cin, L.cout, grad + param_offset(li)};
    part += wgrad_part_floats(L, p);
    w.first[li + 1] = w.first[li] + p.nchunk * p.npair;
    w.rfirst[li + 1] = w.rfirst[li] + p.npair * (L.k * L.k * 256 + 16);
  }
  hipLaunchKernelGGL(wgrad_kernel, dim3(w.first[12]), dim3(256), wgrad_lds_bytes(), s, w);
  ok = ok && hipGetLastError() == hipSuccess;
  hipLaunchKernelGGL(wreduce_kernel, dim3((w.rfirst[12] + 63) / 64), dim3(256),
                     4 * 64 * sizeof(float), s, w);
  ok = ok && hipGetLastError() == hipSuccess;
  return ok ? FLR_OK : FLR_ERR_HIP;
}
}  // namespace flrnet

using namespace flrnet;

extern "C" {

size_t flr_net_num_params(void) { return param_offset(12); }

size_t flr_net_packed_bytes(void) { return packed_offset(12); }

flr_status flr_net_pack(const float* params, void* packed, void* stream) {
  if (!params || !packed) return FLR_ERR_NULL;
  if (!aligned16(params) || !aligned16(packed)) return FLR_ERR_ALIGN;
  if (overlaps(params, flr_net_num_params() * sizeof(float), packed, flr_net_packed_bytes()))
    return FLR_ERR_ALIAS;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  for (int i = 0; i < 12; ++i) {
    const Layer& L = kLayers[i];
    const float* w = params + param_offset(i);
    const float* b = w + (size_t)L.cout * L.cin * L.k * L.k;
    const int n = (int)frag_count(L);
    const PackArgs pa = {w, b, L.cin, L.cout, L.k, pad16(L.cin) / 16, pad16(L.cout) / 16,
                         const_cast<bf16x4_t*>(layer_w(packed, i)),
                         const_cast<float*>(layer_b(packed, i))};
    hipLaunchKernelGGL(pack_kernel, dim3((n + 255) / 256), dim3(256), 0, s, pa);
    if (hipGetLastError() != hipSuccess) return FLR_ERR_HIP;
  }
  return FLR_OK;
}

size_t flr_net_workspace_bytes(int32_t height, int32_t width) {
  if (!valid_dims(height, width)) return 0;
  size_t off[kActBufs + 1];
  act_layout(grids(height, width), off);
  return off[kActBufs];
}

flr_status flr_net_forward(int32_t height, int32_t width, const float* guides, const float* noisy,
                           const void* packed, float* out, void* workspace, size_t workspace_bytes,
                           void* stream) {
  if (!valid_dims(height, width)) return FLR_ERR_SHAPE;
  if (!guides || !noisy || !packed || !out) return FLR_ERR_NULL;
  if (!aligned16(guides) || !aligned16(noisy) || !aligned16(packed) || !aligned16(out))
    return FLR_ERR_ALIGN;
  const size_t need = flr_net_workspace_bytes(height, width);
  if (!workspace || workspace_bytes < need) return FLR_ERR_WORKSPACE;
  if (!aligned16(workspace)) return FLR_ERR_ALIGN;
  const size_t pb = (size_t)height * width * sizeof(float);
  const size_t gb = FLR_NET_IN_GUIDES * pb, nb = FLR_NET_IN_NOISY * pb, ob = FLR_NET_OUT * pb;
  const size_t kb = flr_net_packed_bytes();
  if (overlaps(out, ob, guides, gb) || overlaps(out, ob, noisy, nb) || overlaps(out, ob, packed, kb) ||
      overlaps(workspace, need, guides, gb) || overlaps(workspace, need, noisy, nb) ||
      overlaps(workspace, need, packed, kb) || overlaps(workspace, need, out, ob))
    return FLR_ERR_ALIAS;
  return run_forward(grids(height, width), guides, noisy, packed, out,
                     static_cast<char*>(workspace), reinterpret_cast<hipStream_t>(stream));
}

size_t flr_net_trace_bytes(int32_t height, int32_t width) {
  if (!valid_dims(height, width)) return 0;
  size_t off[kTraceTensors + 1];
  trace_layout(grids(height, width), off);
  return off[kTraceTensors];
}

flr_status flr_net_trace_tensor(int32_t height, int32_t width, int32_t index, size_t* offset,
                                int32_t* channels, int32_t* tensor_height, int32_t* tensor_width) {
  if (!valid_dims(height, width)) return FLR_ERR_SHAPE;
  if (!offset || !channels || !tensor_height || !tensor_width) return FLR_ERR_NULL;
  if (index < 0 || index >= kTraceTensors) return FLR_ERR_MODE;
  const Grids g = grids(height, width);
  size_t off[kTraceTensors + 1];
  trace_layout(g, off);
  const int which = kTraceGrid[index];
  *offset = off[index];
  *channels = kTraceChannels[index];
  *tensor_height = which == 0 ? g.H : which == 1 ? g.Hh : g.Hq;
  *tensor_width = which == 0 ? g.W : which == 1 ? g.Wh : g.Wq;
  return FLR_OK;
}

flr_status flr_net_forward_trace(int32_t height, int32_t width, const float* guides,
                                 const float* noisy, const void* packed, float* out, void* trace,
                                 size_t trace_bytes, void* stream) {
  if (!valid_dims(height, width)) return FLR_ERR_SHAPE;
  if (!guides || !noisy || !packed || !out) return FLR_ERR_NULL;
  if (!aligned16(guides) || !aligned16(noisy) || !aligned16(packed) || !aligned16(out))
    return FLR_ERR_ALIGN;
  const size_t need = flr_net_trace_bytes(height, width);
  if (!trace || trace_bytes < need) return FLR_ERR_WORKSPACE;
  if (!aligned16(trace)) return FLR_ERR_ALIGN;
  const size_t pb = (size_t)height * width * sizeof(float);
  const size_t gb = FLR_NET_IN_GUIDES * pb, nb = FLR_NET_IN_NOISY * pb, ob = FLR_NET_OUT * pb;
  const size_t kb = flr_net_packed_bytes();
  if (overlaps(out, ob, guides, gb) || overlaps(out, ob, noisy, nb) || overlaps(out, ob, packed, kb) ||
      overlaps(trace, need, guides, gb) || overlaps(trace, need, noisy, nb) ||
      overlaps(trace, need, packed, kb) || overlaps(trace, need, out, ob))
    return FLR_ERR_ALIAS;
  const Grids g = grids(height, width);
  size_t off[kTraceTensors + 1];
  trace_layout(g, off);
  char* t = static_cast<char*>(trace);
  return run_forward(g, guides, noisy, packed, out, t, reinterpret_cast<hipStream_t>(stream),
                     reinterpret_cast<uint16_t*>(t + off[1]),
                     reinterpret_cast<uint16_t*>(t + off[11]));
}

size_t flr_net_backward_workspace_bytes(int32_t height, int32_t width) {
  if (!valid_dims(height, width)) return 0;
  size_t off[B_COUNT + 1];
  bwd_layout(grids(height, width), off);
  return off[B_COUNT];
}

flr_status flr_net_backward(int32_t height, int32_t width, const float* guides, const float* noisy,
                            const float* params, const void* packed, const float* grad_out,
                            float* grad_params, int32_t accumulate, void* workspace,
                            size_t workspace_bytes, void* stream) {
  if (!valid_dims(height, width)) return FLR_ERR_SHAPE;
  if (!guides || !noisy || !params || !packed || !grad_out || !grad_params) return FLR_ERR_NULL;
  if (!aligned16(guides) || !aligned16(noisy) || !aligned16(params) || !aligned16(packed) ||
      !aligned16(grad_out) || !aligned16(grad_params))
    return FLR_ERR_ALIGN;
  if (accumulate != 0 && accumulate != 1) return FLR_ERR_MODE;
  const size_t need = flr_net_backward_workspace_bytes(height, width);
  if (!workspace || workspace_bytes < need) return FLR_ERR_WORKSPACE;
  if (!aligned16(workspace)) return FLR_ERR_ALIGN;
  const size_t pb = (size_t)height * width * sizeof(float);
  const size_t gb = FLR_NET_IN_GUIDES * pb, nb = FLR_NET_IN_NOISY * pb, ob = FLR_NET_OUT * pb;
  const size_t kb = flr_net_packed_bytes(), wb = flr_net_num_params() * sizeof(float);
  const void* ins[5] = {guides, noisy, params, packed, grad_out};
  const size_t inb[5] = {gb, nb, wb, kb, ob};
  for (int i = 0; i < 5; ++i)
    if (overlaps(workspace, need, ins[i], inb[i]) || overlaps(grad_params, wb, ins[i], inb[i]))
      return FLR_ERR_ALIAS;
  if (overlaps(workspace, need, grad_params, wb)) return FLR_ERR_ALIAS;
  return run_backward(grids(height, width), guides, noisy, params, packed, grad_out, grad_params,
                      accumulate, static_cast<char*>(workspace),
                      reinterpret_cast<hipStream_t>(stream));
}

size_t flr_flnr_workspace_bytes(const flr_params* p) {
  if (!p || flr_validate_params(p) != FLR_OK) return 0;
  if (p->num_guides != FLR_NET_IN_GUIDES + FLR_NET_OUT || p->num_channels != FLR_NET_IN_NOISY)
    return 0;
  return align256(flr_denoise_workspace_bytes(p)) + flr_net_workspace_bytes(p->height, p->width);
}

flr_status flr_flnr_denoise(const flr_params* p, float* guides12, const float* noisy,
                            const void* packed, float* out, void* workspace,
                            size_t workspace_bytes, void* stream) {
  flr_status st = flr_validate_params(p);
  if (st != FLR_OK) return st;
  if (p->num_guides != FLR_NET_IN_GUIDES + FLR_NET_OUT || p->num_channels != FLR_NET_IN_NOISY)
    return FLR_ERR_CHANNELS;
  if (p->flags & FLR_FLAG_RAW_MOMENTS) return FLR_ERR_MODE;
  if (!guides12 || !noisy || !packed || !out) return FLR_ERR_NULL;
  // the regression's part, then the network's: the fused path also takes a
  // workspace that only holds its smaller form
  const size_t pl = (size_t)p->height * p->width;
  const size_t nw = flr_net_workspace_bytes(p->height, p->width);
  size_t fw = align256(flr_denoise_workspace_bytes(p));
  if (workspace_bytes < fw + nw) fw = align256(flr_denoise_min_workspace_bytes(p));
  const size_t need = fw + nw;
  if (!workspace || workspace_bytes < need) return FLR_ERR_WORKSPACE;
  char* ws = static_cast<char*>(workspace);
  st = flr_net_forward(p->height, p->width, guides12, noisy, packed,
                       guides12 + FLR_NET_IN_GUIDES * pl, ws + fw, need - fw, stream);
  if (st != FLR_OK) return st;
  return flr_denoise(p, guides12, noisy, out, fw ? ws : nullptr, fw, stream);
}

}  // extern "C"
