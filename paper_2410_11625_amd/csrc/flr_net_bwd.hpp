// Gradients of the FLNR guide network (Sec. 3.3 trains the network by
// backpropagating the loss through the regression into it).
//
// Straight-through reading of the BF16 network: the backward treats every
// BF16 rounding of the forward as the identity, so the gradients are those of
// the exact network evaluated at the BF16 weights and activations the forward
// produced. Gradients between layers are FP32 HWC tensors ([pixel][channel]),
// products and sums FP32 on the matrix cores.
//
//   ReLU layer      dz = g * [a > 0], a the stored BF16 activation (a > 0
//                   exactly when the FP32 pre-activation is > 0: BF16 keeps
//                   the FP32 exponent range)
//   sigmoid head    dz = g * s (1 - s), s the FP32 output
//   conv            db[o] = sum_q dz[q][o]
//                   dW[o][c][u][v] = sum_(i,j) dz[(i,j)][o] x[(s i + u - p, s j + v - p)][c]
//                   dx[(y,x)][c] = sum_(o,u,v) W[o][c][u][v] dz[((y + p - u)/s, (x + p - v)/s)][o]
//                   over the terms whose division is exact and in range
//   up2 + concat    the coarse tensor collects the gradients of the 2x2 fine
//                   pixels that copied it; the skip takes its channels as is
//
// Launches: the head, one data gradient per layer (each needs the one before),
// then every layer's weight gradient in one launch (they only need the stored
// dz and activations), and one launch that adds the weight gradients' partial
// sums in a fixed order, so the result does not depend on scheduling.
//
// What bounds it: at a training crop's sizes the chain of data gradients (ten
// launches of 5 to 36 us, most of them with fewer workgroups than the chip has
// room for) and the FP32 matrix instructions of both gradients. Measured at
// 256 x 256 against FP32 vector kernels (one thread per pixel and 8 channels of
// dx, one wave per 4 x 8 channels of a weight gradient's taps, 48 launches):
// data gradients 435 -> 161 us, weight gradients and their sums 480 -> 102 us,
// the whole call 963 -> 342 us, 72 us of it the recomputed forward.

namespace flrnet {

// Data-gradient weights: BF16 fragments of W^T (rows: input channels c, K:
// output channels o), layer after layer, (tap, o block, c block, lane) of 4
// BF16: lane l holds input channel 16 cb + l % 16 and output channels
// 16 ob + 4 (l / 16) .. + 3.
struct BwdPackArgs {
  const float* params;
  bf16x4_t* out;
  int first[13];  // first fragment of each layer (equal: none)
  int param[12];  // first parameter of each layer
  int cin[12], cout[12], k[12];
};
__global__ void __launch_bounds__(256) bwd_pack_kernel(BwdPackArgs a) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= a.first[12]) return;
  int li = 0;
  while (idx >= a.first[li + 1]) ++li;
  const int i = idx - a.first[li];
  const int cin = a.cin[li], cout = a.cout[li], k = a.k[li];
  const int ncb = (cin + 15) / 16, nob = (cout + 15) / 16;
  const int lane = i & 63, cb = (i >> 6) % ncb, ob = (i >> 6) / ncb % nob;
  const int tap = (i >> 6) / ncb / nob;
  const int c = cb * 16 + (lane & 15);
  const float* w = a.params + a.param[li];
  uint16_t h[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int o = ob * 16 + 4 * (lane >> 4) + j;
    h[j] = o < cout && c < cin ? f2bf(w[((size_t)o * cin + c) * k * k + tap]) : (uint16_t)0;
  }
  a.out[idx] = pack4(h[0], h[1], h[2], h[3]);
}

// dz1[q][o] = dout[o][q] s (1 - s), s = sig[o][q] (planar in, HWC out): the
// sigmoid head's gradient; and the gradient of its input, the 16 channels
// of out3's output, gt[q][c] = sum_o W[o][c] dz1[q][o] with the BF16-rounded
// weights.
struct HeadBwdArgs {
  const float* dout;
  const float* sig;
  const float* w;  // [4][16]
  float* dz1;
  float* gt;
  int npx;
};
__global__ void __launch_bounds__(256) head_bwd_kernel(HeadBwdArgs a) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= a.npx) return;
  float d[FLR_NET_OUT];
#pragma unroll
  for (int o = 0; o < FLR_NET_OUT; ++o) {
    const float s = a.sig[(size_t)o * a.npx + q];
    d[o] = a.dout[(size_t)o * a.npx + q] * s * (1.f - s);
  }
  *reinterpret_cast<float4*>(a.dz1 + (size_t)q * FLR_NET_OUT) = float4{d[0], d[1], d[2], d[3]};
#pragma unroll
  for (int c = 0; c < 16; c += 4) {
    float g[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float s = 0.f;
#pragma unroll
      for (int o = 0; o < FLR_NET_OUT; ++o) s += bf2f(f2bf(a.w[o * 16 + c + i])) * d[o];
      g[i] = s;
    }
    *reinterpret_cast<float4*>(a.gt + (size_t)q * 16 + c) = float4{g[0], g[1], g[2], g[3]};
  }
}

// dz of a layer: the gradient g of its output activation (HWC, channel stride
// cs), masked by the stored activation where act is given. up: g is the
// gradient of the 2x upsampled copy, on a grid of Hf x Wf pixels; the coarse
// pixel takes the sum of its (up to four) fine pixels.
struct DzSrc {
  const float* g;
  const uint16_t* act;  // [pixel][cout]
  int cs, cout;
  int up, Hf, Wf;
};

// Four channels o .. o + 3 at pixel (y, x) of the H x W grid (clamped by the
// caller); zero past cout.
__device__ __forceinline__ float4 load_dz4(const DzSrc& s, int y, int x, int W, int o) {
  if (o >= s.cout) return float4{0.f, 0.f, 0.f, 0.f};
  float4 d;
  if (s.up) {
    d = float4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int di = 0; di < 2; ++di)
#pragma unroll
      for (int dj = 0; dj < 2; ++dj) {
        const int fy = 2 * y + di, fx = 2 * x + dj;
        const bool ok = fy < s.Hf && fx < s.Wf;
        const size_t q = (size_t)(fy < s.Hf ? fy : s.Hf - 1) * s.Wf + (fx < s.Wf ? fx : s.Wf - 1);
        const float4 t = *reinterpret_cast<const float4*>(s.g + q * s.cs + o);
        d.x += ok ? t.x : 0.f;
        d.y += ok ? t.y : 0.f;
        d.z += ok ? t.z : 0.f;
        d.w += ok ? t.w : 0.f;
      }
  } else {
    d = *reinterpret_cast<const float4*>(s.g + ((size_t)y * W + x) * s.cs + o);
  }
  if (s.act) {
    const uint2 a = *reinterpret_cast<const uint2*>(s.act + ((size_t)y * W + x) * s.cout + o);
    d.x = (a.x & 0xffffu) != 0 && !(a.x & 0x8000u) ? d.x : 0.f;
    d.y = (a.x >> 16) != 0 && !(a.x & 0x80000000u) ? d.y : 0.f;
    d.z = (a.y & 0xffffu) != 0 && !(a.y & 0x8000u) ? d.z : 0.f;
    d.w = (a.y >> 16) != 0 && !(a.y & 0x80000000u) ? d.w : 0.f;
  }
  return d;
}

// x = hi + mid + lo exactly (24 bits in three BF16, each the truncation of
// what is left); infinities and NaN stay in hi alone.
__device__ __forceinline__ void split3(float x, uint16_t (&h)[3]) {
  const uint32_t u = __float_as_uint(x);
  const bool fin = (u & 0x7f800000u) != 0x7f800000u;
  const float r1 = fin ? x - __uint_as_float(u & 0xffff0000u) : 0.f;
  const uint32_t u1 = __float_as_uint(r1);
  const float r2 = r1 - __uint_as_float(u1 & 0xffff0000u);
  // a NaN whose set bits all lie in the low half must stay one
  h[0] = (uint16_t)((u >> 16) | ((u & 0x7fffffffu) > 0x7f800000u ? 0x40u : 0u));
  h[1] = (uint16_t)(u1 >> 16);
  h[2] = (uint16_t)(__float_as_uint(r2) >> 16);
}

// D = A B + C of 16 x 16 x 4 FP32 (lane l: A row l % 16, k = l / 16; B k =
// l / 16, column l % 16; C, D as the BF16 instruction). One of a and b holds
// BF16 values (A32: b does).
template <bool A32>
__device__ __forceinline__ f32x4_t mfma_f32(float a, float b, f32x4_t c) {
#if __has_builtin(__builtin_amdgcn_mfma_f32_16x16x4f32)
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
#else  // hosts that emulate the BF16 instruction only: the same products in three parts
  uint16_t h[3];
  split3(A32 ? a : b, h);
  const bf16x4_t v = pack4((uint16_t)(__float_as_uint(A32 ? b : a) >> 16), 0, 0, 0);
  for (int s = 2; s >= 0; --s) {
    const bf16x4_t part = pack4(h[s], 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(A32 ? part : v, A32 ? v : part, c, 0, 0, 0);
  }
  return c;
#endif
}

struct DgradArgs {
  DzSrc dz;
  const bf16x4_t* w;  // the layer's data-gradient fragments
  int Hi, Wi, Ho, Wo;
  float* dx;          // [Hi*Wi][cin]
  const float* add;   // optional addend add[p * add_cs + add_off + c]
  int add_cs, add_off;
};

// Data gradient of one layer (CIN channels of dx from COUT of dz, both
// multiples of 16; kernel KS, stride ST) as an implicit GEMM on the FP32
// matrix cores: D (c x pixels) += W^T (c x o) dz (o x pixels). The weights'
// BF16 values are widened in registers. (Three BF16 products of dz split
// exactly into three parts take a third of the matrix time, but the BF16
// instruction's sums lean to minus infinity, by about 0.05 * 2^-24 of the
// accumulator each: over a frame that bias adds up where the gradients
// cancel. Relative rms error of in3's weights under a loss gradient of random
// signs, in 2^-24: three BF16 products 429 at 256 x 256 and 1847 at 1080p,
// FP32 15 and 27; the whole call at 256 x 256 320 -> 343 us.)
//
// A workgroup of four waves computes CBG 16-channel blocks of dx for four
// rows (stride 2: four coarse rows, both row and both column parities) of
// 16 NT pixels; per 16 output channels it stages the dz tile with its halo in
// LDS (HWC FP32, zero outside the grid) and runs the taps.
template <int CIN, int COUT, int KS, int ST, int CBG, int NT>
__global__ void __launch_bounds__(256) dgrad_kernel(DgradArgs a) {
  constexpr int NCB = CIN / 16, NOB = COUT / 16;
  constexpr int HALO = KS == 1 ? 0 : (ST == 1 ? 2 : 1);  // staged rows and columns beyond the tile
  constexpr int LO = KS == 3 && ST == 1 ? 1 : 0;         // of which before it
  constexpr int SR = 4 + HALO, SP = 16 * NT + HALO;
  constexpr int NPAR = ST * ST, NCG = NCB / CBG;
  float4* st = reinterpret_cast<float4*>(flr::lds);  // [SR][SP][4]
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, kq = lane >> 4;
  const int x0 = blockIdx.x / NCG * 16 * NT, y0 = blockIdx.y * 4, cb0 = blockIdx.x % NCG * CBG;
  f32x4_t acc[NPAR][NT][CBG];
#pragma unroll
  for (int p = 0; p < NPAR; ++p)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int cb = 0; cb < CBG; ++cb) acc[p][t][cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int ob = 0; ob < NOB; ++ob) {
    if (ob > 0) __syncthreads();  // the previous block's tile has been read
    constexpr int NIT = SR * SP * 4, B = 4;
    for (int b0 = 0; b0 < NIT; b0 += B * 256) {
      float4 d[B];
      bool ok[B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int i = b0 + u * 256 + tid, ic = i < NIT ? i : NIT - 1;
        const int pix = ic >> 2, q = ic & 3;
        const int sr = pix / SP, sx = pix - sr * SP;
        const int y = y0 - LO + sr, x = x0 - LO + sx;
        ok[u] = y >= 0 && y < a.Ho && x >= 0 && x < a.Wo;
        d[u] = load_dz4(a.dz, min(max(y, 0), a.Ho - 1), min(max(x, 0), a.Wo - 1), a.Wo,
                        ob * 16 + 4 * q);
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int i = b0 + u * 256 + tid;
        if (i < NIT)
          st[i] = float4{ok[u] ? d[u].x : 0.f, ok[u] ? d[u].y : 0.f, ok[u] ? d[u].z : 0.f,
                         ok[u] ? d[u].w : 0.f};
      }
    }
    __syncthreads();
    // tap (u, v): stride 1 reads dz at (+1 - u, +1 - v); stride 2 reads, for
    // output parity (py, px), (py + 1 - u) / 2 where that is whole
#pragma unroll
    for (int u = 0; u < KS; ++u) {
#pragma unroll
      for (int v = 0; v < KS; ++v) {
        const int tap = u * KS + v;
        const int par = ST == 1 ? 0 : ((u + 1) & 1) * 2 + ((v + 1) & 1);
        const int dy = KS == 1 ? 0 : (ST == 1 ? 2 - u : (u == 0 ? 1 : 0));
        const int dx = KS == 1 ? 0 : (ST == 1 ? 2 - v : (v == 0 ? 1 : 0));
        float av[CBG][4];  // lane: output channels 4 kq + j, as dz below
#pragma unroll
        for (int cb = 0; cb < CBG; ++cb) {
          const bf16x4_t w = a.w[((tap * NOB + ob) * NCB + cb0 + cb) * 64 + lane];
#pragma unroll
          for (int j = 0; j < 4; ++j) av[cb][j] = bf2f((uint16_t)w[j]);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const float4 z = st[((wv + dy) * SP + t * 16 + (lane & 15) + dx) * 4 + kq];
          const float b[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int cb = 0; cb < CBG; ++cb)
              acc[par][t][cb] = mfma_f32<false>(av[cb][j], b[j], acc[par][t][cb]);
        }
      }
    }
  }
  // lane: channels 4 kq .. + 3 of each block at one pixel
#pragma unroll
  for (int p = 0; p < NPAR; ++p) {
    const int y = (y0 + wv) * ST + (p >> 1);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int x = (x0 + t * 16 + (lane & 15)) * ST + (p & 1);
      if (y >= a.Hi || x >= a.Wi) continue;
      const size_t q = (size_t)y * a.Wi + x;
#pragma unroll
      for (int cb = 0; cb < CBG; ++cb) {
        const int c = (cb0 + cb) * 16 + 4 * kq;
        const f32x4_t s = acc[p][t][cb];
        float4 o{s[0], s[1], s[2], s[3]};
        if (a.add) {
          const float4 e = *reinterpret_cast<const float4*>(a.add + q * a.add_cs + a.add_off + c);
          o = float4{o.x + e.x, o.y + e.y, o.z + e.z, o.w + e.w};
        }
        *reinterpret_cast<float4*>(a.dx + q * CIN + c) = o;
      }
    }
  }
}
template <int KS, int ST, int NT>
constexpr size_t dgrad_lds_bytes() {
  constexpr int halo = KS == 1 ? 0 : (ST == 1 ? 2 : 1);
  return (size_t)(4 + halo) * (16 * NT + halo) * 4 * sizeof(float4);
}

// Input of a layer as the backward reads it: one HWC BF16 tensor, or
// [up2(in0), in1] with in0 on a grid of width Wl (Wl = 0: plain).
struct BwdSrc {
  const uint16_t* in0;
  const uint16_t* in1;
  int cs0, cup, cs1;  // in0 channel stride, channels taken from in0, in1 channel stride
  int Wl;
};

// One layer of the weight-gradient launch. Its workgroups are (16 x 16 block
// of output x input channels, pixel chunk), chunk-major.
struct WgradLayer {
  DzSrc dz;
  BwdSrc src;
  int Hi, Wi, Ho, Wo;
  int ncb, npair;    // input channel blocks, block pairs
  int k, stride;
  int tiles_x, ntile, chunk;  // tiles of 4 x 64 output pixels; tiles per chunk
  int nchunk;
  float* part;       // [nchunk][npair][k k 256 + 16]: sums, then the bias sums
  int cin, cout;
  float* grad;       // the layer's weights [cout][cin][k][k] then bias [cout]
};
struct WgradArgs {
  WgradLayer layer[12];
  int first[13];      // first workgroup of each layer's weight gradients
  int rfirst[13];     // first element of each layer in the reduction
  int accumulate;
};

// Weight gradients as GEMMs over pixels on the matrix cores: D (o x c) += dz
// (o x pixels) x (pixels x c), one accumulator per tap. A workgroup stages a
// tile of 4 x 64 output pixels' dz (16 channels, FP32) and the input pixels
// its taps read (16 channels, BF16) in LDS, HWC: the FP32 instruction takes
// one pixel and one channel per lane, so both operands are read as they lie,
// 64 consecutive values. Wave w sums row w; the four sums are added in wave
// order at the end of the chunk.
//
// A wave's sums are closed into a second set every kWgClose tiles (32 pixels
// per lane and tap), so that a chain of FP32 sums does not grow with the frame.
// Relative error of the head's weight gradient at 1080p under a loss gradient
// of random signs, in 2^-24: one chain per chunk (51 tiles) 23, closed every
// 4 tiles 7.4, every 2 tiles 6.8; closing after every tile needs more
// registers than three workgroups per CU have (1080p 5.26 -> 5.58 ms).
constexpr int kWgClose = 2;
template <int KS, int ST>
__device__ __forceinline__ void wgrad_tile(const WgradLayer& a, const int wg) {
  constexpr int KK = KS * KS, PD = KS / 2;
  constexpr int XR = 3 * ST + KS, XP = 63 * ST + KS;  // staged input rows and columns
  float* zs = flr::lds;                               // [4][64][16]
  uint16_t* xs = reinterpret_cast<uint16_t*>(flr::lds + 4 * 64 * 16);  // [XR][XP][16]
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int chunk = wg / a.npair, pair = wg - chunk * a.npair;
  const int ob = pair / a.ncb, cb = pair - ob * a.ncb;
  f32x4_t acc[KK], bacc = f32x4_t{0.f, 0.f, 0.f, 0.f}, sum[KK], bsum = bacc;
#pragma unroll
  for (int t = 0; t < KK; ++t) acc[t] = sum[t] = bacc;
  auto close = [&]() {
#pragma unroll
    for (int t = 0; t < KK; ++t) {
      sum[t] += acc[t];
      acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    }
    bsum += bacc;
    bacc = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  const float one = (lane & 15) == 0 ? 1.f : 0.f;
  const int t0 = chunk * a.chunk, t1 = min(t0 + a.chunk, a.ntile);
  for (int tile = t0; tile < t1; ++tile) {
    const int ty = tile / a.tiles_x, tx = tile - ty * a.tiles_x;
    const int y0 = ty * 4, x0 = tx * 64;
    if (tile > t0) __syncthreads();  // the previous tile has been read
    {
      float4 d[4];
      bool ok[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = u * 256 + tid, pix = i >> 2, q = i & 3;
        const int y = y0 + (pix >> 6), x = x0 + (pix & 63);
        ok[u] = y < a.Ho && x < a.Wo;
        d[u] = load_dz4(a.dz, min(y, a.Ho - 1), min(x, a.Wo - 1), a.Wo, ob * 16 + 4 * q);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        *reinterpret_cast<float4*>(zs + (u * 256 + tid) * 4) =
            float4{ok[u] ? d[u].x : 0.f, ok[u] ? d[u].y : 0.f, ok[u] ? d[u].z : 0.f,
                   ok[u] ? d[u].w : 0.f};
      }
    }
    // input pixels: two 16-byte halves each
    constexpr int NIT = XR * XP * 2, B = 4;
    const int c0 = cb * 16;
    const bool low = a.src.Wl > 0 && c0 < a.src.cup;
    for (int b0 = 0; b0 < NIT; b0 += B * 256) {
      uint4 v[B];
      bool ok[B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int i = b0 + u * 256 + tid, ic = i < NIT ? i : NIT - 1;
        const int pix = ic >> 1, hf = ic & 1;
        const int sr = pix / XP, sx = pix - sr * XP;
        const int y = y0 * ST - PD + sr, x = x0 * ST - PD + sx;
        ok[u] = y >= 0 && y < a.Hi && x >= 0 && x < a.Wi;
        const int yc = min(max(y, 0), a.Hi - 1), xc = min(max(x, 0), a.Wi - 1);
        const uint16_t* p =
            low ? a.src.in0 + ((size_t)(yc >> 1) * a.src.Wl + (xc >> 1)) * a.src.cs0 + c0
            : a.src.Wl > 0
                ? a.src.in1 + ((size_t)yc * a.Wi + xc) * a.src.cs1 + (c0 - a.src.cup)
                : a.src.in0 + ((size_t)yc * a.Wi + xc) * a.src.cs0 + c0;
        v[u] = *reinterpret_cast<const uint4*>(p + 8 * hf);
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int i = b0 + u * 256 + tid;
        const uint32_t keep = ok[u] ? 0xffffffffu : 0u;
        if (i < NIT)
          *reinterpret_cast<uint4*>(xs + i * 8) =
              uint4{v[u].x & keep, v[u].y & keep, v[u].z & keep, v[u].w & keep};
      }
    }
    __syncthreads();
    const float* zr = zs + wv * 64 * 16 + lane;  // pixel 4 s + lane / 16, channel lane % 16
    const uint16_t* xr = xs + ((wv * ST) * XP + (lane >> 4) * ST) * 16 + (lane & 15);
#pragma unroll 4
    for (int s = 0; s < 16; ++s) {
      const float z = zr[s * 64];
      if (cb == 0) bacc = mfma_f32<true>(z, one, bacc);
#pragma unroll
      for (int u = 0; u < KS; ++u)
#pragma unroll
        for (int v = 0; v < KS; ++v) {
          const float x = bf2f(xr[(u * XP + 4 * s * ST + v) * 16]);
          acc[u * KS + v] = mfma_f32<true>(z, x, acc[u * KS + v]);
        }
    }
    if ((tile - t0) % kWgClose == kWgClose - 1) close();
  }
  close();
  // add the four waves' sums: [wave][tap][o][c], then the bias [wave][o]
  __syncthreads();
  float* red = flr::lds;
  constexpr int S = KK * 256 + 16;
#pragma unroll
  for (int t = 0; t < KK; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      red[wv * S + t * 256 + (4 * (lane >> 4) + i) * 16 + (lane & 15)] = sum[t][i];
  if ((lane & 15) == 0)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wv * S + KK * 256 + 4 * (lane >> 4) + i] = bsum[i];
  __syncthreads();
  float* out = a.part + ((size_t)chunk * a.npair + pair) * S;
  for (int i = tid; i < S; i += 256)
    out[i] = ((red[i] + red[S + i]) + red[2 * S + i]) + red[3 * S + i];
}
constexpr size_t wgrad_lds_bytes() {
  // the stride-2 tile (9 x 129 input pixels) or the closing sums, whichever is larger
  return 4 * 64 * 16 * sizeof(float) + (size_t)9 * 129 * 16 * sizeof(uint16_t);
}
static_assert(wgrad_lds_bytes() >= 4 * (9 * 256 + 16) * sizeof(float), "closing sums fit");

__global__ void __launch_bounds__(256) wgrad_kernel(WgradArgs a) {
  const int b = blockIdx.x;
  int li = 0;
  while (b >= a.first[li + 1]) ++li;
  const WgradLayer& L = a.layer[li];
  if (L.k == 1)
    wgrad_tile<1, 1>(L, b - a.first[li]);
  else if (L.stride == 1)
    wgrad_tile<3, 1>(L, b - a.first[li]);
  else
    wgrad_tile<3, 2>(L, b - a.first[li]);
}

// grad = (accumulate ? grad : 0) + the chunks' partial sums in chunk order:
// 64 elements per workgroup, each wave a quarter of the chunks (16 loads in
// flight), then the four quarters in order.
__global__ void __launch_bounds__(256) wreduce_kernel(WgradArgs a) {
  float* red = flr::lds;  // [4][64]
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane;
  const int total = a.rfirst[12];
  int li = 0;
  while (li < 11 && e >= a.rfirst[li + 1]) ++li;
  const WgradLayer& L = a.layer[li];
  const int i = e - a.rfirst[li];
  const int kk = L.k * L.k, S = kk * 256 + 16;
  const int pair = i / S, s = i - pair * S;
  const int per = (L.nchunk + 3) / 4;
  const int c0 = wv * per, c1 = min(c0 + per, L.nchunk);
  float sum = 0.f;
  if (e < total) {
    const size_t step = (size_t)L.npair * S;
    const float* p = L.part + i + (size_t)c0 * step;
    int c = c0;
    for (; c + 16 <= c1; c += 16) {
      float t[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) t[k] = p[k * step];
#pragma unroll
      for (int k = 0; k < 16; ++k) sum += t[k];
      p += 16 * step;
    }
    for (; c < c1; ++c, p += step) sum += *p;
  }
  red[wv * 64 + lane] = sum;
  __syncthreads();
  if (wv != 0 || e >= total) return;
  const float t = ((red[lane] + red[64 + lane]) + red[128 + lane]) + red[192 + lane];
  const int ob = pair / L.ncb, cb = pair - ob * L.ncb;
  int dst;
  if (s < kk * 256) {
    const int tap = s >> 8, o = ob * 16 + ((s >> 4) & 15), c = cb * 16 + (s & 15);
    if (o >= L.cout || c >= L.cin) return;  // padding channels
    dst = (o * L.cin + c) * kk + tap;
  } else {
    const int o = ob * 16 + (s - kk * 256);
    if (cb != 0 || o >= L.cout) return;
    dst = L.cout * L.cin * kk + o;
  }
  L.grad[dst] = a.accumulate ? L.grad[dst] + t : t;
}

// Chunking of a layer's weight gradient: about kWgTarget workgroups.
constexpr int kWgTarget = 160;
struct WgradPlan {
  int ncb, npair, tiles_x, ntile, chunk, nchunk;
};
inline WgradPlan wgrad_plan(const Layer& L, int Ho, int Wo) {
  WgradPlan p;
  p.ncb = (L.cin + 15) / 16;
  p.npair = p.ncb * ((L.cout + 15) / 16);
  p.tiles_x = (Wo + 63) / 64;
  p.ntile = p.tiles_x * ((Ho + 3) / 4);
  const int want = kWgTarget / p.npair > 1 ? kWgTarget / p.npair : 1;
  p.chunk = (p.ntile + want - 1) / want;
  p.nchunk = (p.ntile + p.chunk - 1) / p.chunk;
  return p;
}
inline size_t wgrad_part_floats(const Layer& L, const WgradPlan& p) {
  return (size_t)p.nchunk * p.npair * (L.k * L.k * 256 + 16);
}

}  // namespace flrnet
