// Learned descriptor network kernels: 3x3 convolutions in NHWC with bf16
// operands and float32 accumulation on matrix cores, their backward passes,
// the Adam update, and the quantisation of learned features to bytes.
//
// Convolution as an implicit GEMM: 32 output pixels x 32 output channels per
// wave, K = 9 taps x Cin in chunks of 16 (one v_mfma_f32_32x32x16_bf16 per
// chunk).  A lane holds 8 consecutive input channels of one tap of one pixel
// (16 bytes, zero outside the image: "same" zero padding) and the matching 8
// weights of one output channel.  Layout: activations [B][H][W][C], weights
// [Cout][9][Cin] (tap = 3 * (dy + 1) + (dx + 1)).
//
// The data gradient is the same convolution with the weights rotated by 180
// degrees and transposed ([Cin][9][Cout]).  The weight gradient is a
// contraction over all pixels, also on matrix cores; each workgroup writes
// a partial sum of its rows and a second kernel adds the partials in a fixed
// order, so it is deterministic.
#include <algorithm>

#include "ff_device.h"
#include "ff_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  // round to nearest even (finite inputs)
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// Two at once, the first in the low half (v_cvt_pk_bf16_f32; the same
// rounding for every non-NaN input, denormals included).
__device__ __forceinline__ uint32_t f32x2_to_bf16(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 h = __builtin_convertvector((f32x2){lo, hi}, bf16x2);
  uint32_t u;
  __builtin_memcpy(&u, &h, 4);
  return u;
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) {
  bf16x8 r;
  __builtin_memcpy(&r, &v, sizeof(r));
  return r;
}

// The 16 features of one pixel scaled to unit length; returns the scale.
__device__ __forceinline__ float l2norm16(float4 v[4], float delta) {
  float s = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) s += v[k].x * v[k].x + v[k].y * v[k].y + v[k].z * v[k].z + v[k].w * v[k].w;
  const float r = 1.0f / sqrtf(s + delta);
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = make_float4(v[k].x * r, v[k].y * r, v[k].z * r, v[k].w * r);
  return r;
}

// Epilogue of a transposed product D = W X (weights the first operand, 32
// pixels the columns): a lane holds the output channels 8 g + 4 kh .. 8 g + 4
// kh + 3, g < COUT / 8, of one pixel.  Every output element is the same sum
// of the same products as in X W, bit for bit.  A run of 32 pixels is one
// contiguous piece of the output; the lanes' parts go through a wave's own
// 2 KB of LDS (16-byte chunks permuted against bank conflicts) so that a
// store instruction writes 1 KB of it: storing from the lanes' registers
// touches every 64-byte pixel four times.  (Float32 outputs of 32 channels: 64 of
// a pixel's 128 bytes at a time.  Two 640 x 480 images, 32 -> 32: 65 us from the
// registers, 29 this way.)
enum ConvEpilogue {
  kConvPlain,  // bias, optional ReLU; float32 and / or bf16, aligned for 16-byte stores
  kConvAny,    // the same for outputs aligned to an element only: from X W (below)
  kConvMask,   // gradient through the ReLU whose output is a.act, split into two bf16 parts
  kConvNorm,   // bias, unit length per pixel (COUT = 16), float32 and the scale
};

// A wave's LDS accesses stay in order; keeps the compiler from moving them.
__device__ __forceinline__ void lds_in_order() { asm volatile("" ::: "memory"); }

// 16-byte chunk c (0 .. 3) of pixel px (0 .. 31) of a 64-byte-per-pixel run.
__device__ __forceinline__ int run_chunk(int px, int c) { return px * 64 + ((c ^ ((px >> 2) & 3)) << 4); }

__device__ __forceinline__ uint2 pack4(const uint32_t (&h)[4]) {
  return make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
}

// Writes the run's first n pixels from LDS to `dst` (64 bytes per pixel,
// STRIDE bytes from pixel to pixel), 16-bit lanes zeroed where `act` (nullable)
// is not positive.
template <int STRIDE = 64>
__device__ __forceinline__ void store_run(const uint8_t *tr, uint8_t *dst, int n, int lane, const uint8_t *act) {
  const int px = lane >> 2, c = lane & 3;  // and pixel px + 16
  uint4 v0 = *reinterpret_cast<const uint4 *>(tr + run_chunk(px, c));
  uint4 v1 = *reinterpret_cast<const uint4 *>(tr + run_chunk(px + 16, c));
  if (act) {
    uint4 m0 = make_uint4(0, 0, 0, 0), m1 = m0;
    if (px < n) m0 = *reinterpret_cast<const uint4 *>(act + px * 64 + 16 * c);
    if (px + 16 < n) m1 = *reinterpret_cast<const uint4 *>(act + (px + 16) * 64 + 16 * c);
    auto mask = [](uint32_t x, uint32_t a) {  // bf16 > 0: a bit pattern in [1, 0x7F80]
      const uint32_t l = a & 0xFFFFu, h = a >> 16;
      return (l - 1u < 0x7F80u ? x & 0xFFFFu : 0u) | (h - 1u < 0x7F80u ? x & 0xFFFF0000u : 0u);
    };
    auto mask4 = [&](uint4 x, uint4 m) {
      return make_uint4(mask(x.x, m.x), mask(x.y, m.y), mask(x.z, m.z), mask(x.w, m.w));
    };
    v0 = mask4(v0, m0);
    v1 = mask4(v1, m1);
  }
  lds_in_order();
  if (px < n) *reinterpret_cast<uint4 *>(dst + px * STRIDE + 16 * c) = v0;
  if (px + 16 < n) *reinterpret_cast<uint4 *>(dst + (px + 16) * STRIDE + 16 * c) = v1;
}

// q0: the run's first pixel; n: its pixels in the image (at most 32, the lane's
// is row); tr: the wave's 2 KB.
template <int COUT, ConvEpilogue EPI>
__device__ __forceinline__ void conv_store(const ffh::ConvArgs &a, size_t q0, int n, int lane, const f32x16 &acc,
                                           const float (&bias)[COUT / 2], uint8_t *tr) {
  constexpr int G = COUT / 8;
  const int row = lane & 31, kh = lane >> 5;
  float v[G][4];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int c = 0; c < 4; ++c) v[g][c] = acc[4 * g + c] + bias[4 * g + c];
  if constexpr (EPI == kConvNorm) {
    static_assert(COUT == 16, "the normalisation is over 16 channels");
    // all 16 channels: the other lane half holds the other 8
    float o[2][4];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int c = 0; c < 4; ++c) o[g][c] = __shfl_xor(v[g][c], 32);
    auto quad = [&](int g, bool own) {
      return make_float4(own ? v[g][0] : o[g][0], own ? v[g][1] : o[g][1], own ? v[g][2] : o[g][2],
                         own ? v[g][3] : o[g][3]);
    };
    float4 f[4] = {quad(0, kh == 0), quad(0, kh == 1), quad(1, kh == 0), quad(1, kh == 1)};
    const float r = l2norm16(f, a.delta);
#pragma unroll
    for (int g = 0; g < 2; ++g)
      *reinterpret_cast<float4 *>(tr + run_chunk(row, 2 * g + kh)) =
          make_float4(v[g][0] * r, v[g][1] * r, v[g][2] * r, v[g][3] * r);
    lds_in_order();
    store_run(tr, reinterpret_cast<uint8_t *>(a.out_f32 + q0 * 16), n, lane, nullptr);
    if (kh == 0 && row < n) a.inv_norm[q0 + row] = r;
  } else if constexpr (EPI == kConvMask) {
    static_assert(COUT == 32, "data gradients have 32 channels");
    uint2 lo[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      uint32_t h[2], l[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const float a0 = v[g][2 * c], a1 = v[g][2 * c + 1];
        h[c] = f32x2_to_bf16(a0, a1);
        l[c] = f32x2_to_bf16(a0 - bf16_to_f32((uint16_t)h[c]), a1 - __uint_as_float(h[c] & 0xFFFF0000u));
      }
      *reinterpret_cast<uint2 *>(tr + run_chunk(row, g) + 8 * kh) = make_uint2(h[0], h[1]);
      lo[g] = make_uint2(l[0], l[1]);
    }
    lds_in_order();
    const uint8_t *act = reinterpret_cast<const uint8_t *>(a.act + q0 * 32);
    store_run(tr, reinterpret_cast<uint8_t *>(a.out_bf16 + q0 * 32), n, lane, act);
#pragma unroll
    for (int g = 0; g < G; ++g) *reinterpret_cast<uint2 *>(tr + run_chunk(row, g) + 8 * kh) = lo[g];
    lds_in_order();
    store_run(tr, reinterpret_cast<uint8_t *>(a.out_lo + q0 * 32), n, lane, act);
  } else {
    if (a.relu)
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int c = 0; c < 4; ++c) v[g][c] = fmaxf(v[g][c], 0.0f);
    if (a.out_f32) {
#pragma unroll
      for (int h = 0; h < G; h += 2) {  // 16 channels at a time: 64 bytes of every pixel
#pragma unroll
        for (int g = 0; g < 2; ++g)
          *reinterpret_cast<float4 *>(tr + run_chunk(row, 2 * g + kh)) =
              make_float4(v[h + g][0], v[h + g][1], v[h + g][2], v[h + g][3]);
        lds_in_order();
        store_run<4 * COUT>(tr, reinterpret_cast<uint8_t *>(a.out_f32 + q0 * COUT + 8 * h), n, lane, nullptr);
        lds_in_order();
      }
    }
    if (a.out_bf16) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const uint2 h = make_uint2(f32x2_to_bf16(v[g][0], v[g][1]), f32x2_to_bf16(v[g][2], v[g][3]));
        if constexpr (COUT == 32)
          *reinterpret_cast<uint2 *>(tr + run_chunk(row, g) + 8 * kh) = h;
        else if (row < n)
          *reinterpret_cast<uint2 *>(a.out_bf16 + (q0 + row) * COUT + 8 * g + 4 * kh) = h;
      }
      if constexpr (COUT == 32) {
        lds_in_order();
        store_run(tr, reinterpret_cast<uint8_t *>(a.out_bf16 + q0 * 32), n, lane, nullptr);
      }
    }
  }
  lds_in_order();
}

// Epilogue of the product X W: a lane holds output channel col = lane & 31 of
// the pixels 8 g + 4 kh + c, so that 32 lanes store 32 channels of a pixel
// element by element, one after another.
template <int COUT>
__device__ __forceinline__ void conv_store_any(const ffh::ConvArgs &a, size_t q0, int n, int lane, const f32x16 &acc,
                                               float bias) {
  const int col = lane & 31, kh = lane >> 5;
  if (col >= COUT) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int px = 8 * (r >> 2) + 4 * kh + (r & 3);
    float v = acc[r] + bias;
    if (a.relu) v = fmaxf(v, 0.0f);
    if (px >= n) continue;
    if (a.out_f32) a.out_f32[(q0 + px) * COUT + col] = v;
    if (a.out_bf16) a.out_bf16[(q0 + px) * COUT + col] = (uint16_t)f32x2_to_bf16(v, 0.0f);
  }
}

// The biases of a lane's output channels.
template <int COUT>
__device__ __forceinline__ void conv_bias(const float *bias, int kh, float (&b)[COUT / 2]) {
#pragma unroll
  for (int r = 0; r < COUT / 2; ++r) b[r] = bias ? bias[8 * (r >> 2) + 4 * kh + (r & 3)] : 0.0f;
}

// Single input channel (the first layer): K = 9 taps padded to 16, lane
// half kh holds taps 8 * kh .. 8 * kh + 7 of one pixel.  Bound by its stores
// (64 bytes a pixel, 45 us for 3.6 Mpx at copy rate) and the 2-byte loads of
// the taps: 89 us with one bf16 per lane and store, 99 with the 8 bytes that a
// lane holds, 92 in 1 KB pieces, 87 with two values rounded at a time.
template <int CIN, int COUT, ConvEpilogue EPI>
__global__ __launch_bounds__(256) void k_conv_fwd(ffh::ConvArgs a) {
  static_assert(CIN == 1, "Cin 1 (wider inputs: k_conv_fwd_tile)");
  static_assert(COUT == 32, "Cout 32");
  __shared__ __attribute__((aligned(16))) uint8_t s_tr[4][2048];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane & 31, kh = lane >> 5;
  const long long P = (long long)a.B * a.H * a.W;
  const long long p0 = ((long long)blockIdx.x * 4 + wave) * 32;
  if (p0 >= P) return;  // wave-uniform
  const long long p = p0 + row;
  const bool pv = p < P;
  const int x = pv ? (int)(p % a.W) : 0, y = pv ? (int)((p / a.W) % a.H) : 0;
  const long long img = pv ? p / ((long long)a.W * a.H) : 0;
  const uint16_t *in = a.in;
  f32x16 acc = {0};
  uint16_t av[8], bv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int tap = 8 * kh + e;
    uint16_t va = 0, vb = 0;
    if (tap < 9) {
      const int sx = x + tap % 3 - 1, sy = y + tap / 3 - 1;
      if (pv && sx >= 0 && sx < a.W && sy >= 0 && sy < a.H) va = in[((img * a.H + sy) * a.W + sx)];
      vb = a.w[row * 9 + tap];
    }
    av[e] = va;
    bv[e] = vb;
  }
  uint4 ua, ub;
  __builtin_memcpy(&ua, av, 16);
  __builtin_memcpy(&ub, bv, 16);
  const int n = (int)min(32ll, P - p0);
  if constexpr (EPI == kConvAny) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ua), as_bf16x8(ub), acc, 0, 0, 0);
    conv_store_any<COUT>(a, (size_t)p0, n, lane, acc, a.bias ? a.bias[row] : 0.0f);
  } else {
    float bias[COUT / 2];
    conv_bias<COUT>(a.bias, kh, bias);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ub), as_bf16x8(ua), acc, 0, 0, 0);
    conv_store<COUT, kConvPlain>(a, (size_t)p0, n, lane, acc, bias, s_tr[wave]);
  }
}

// Tiled form for Cin >= 16: a workgroup takes kConvRows image rows x 32
// pixels of one image.  The input tile with a one-pixel border (zeros
// outside the image: the "same" padding) is staged in LDS once, instead of
// every tap of every pixel being read from global memory; a pixel occupies
// Cin * 2 + 16 bytes there, so the 16-byte reads of 32 consecutive pixels hit
// distinct banks.  Each wave keeps its weight operands in registers and runs
// every fourth row of the tile.  The products are accumulated in the same
// order as in k_conv_fwd (taps, then channel chunks), so the results are
// identical.  The epilogues that a training step needs run here instead of as
// passes over memory of their own: the last layer's normalisation, and the
// data gradient's ReLU and its split into two bf16 parts.  3.6 Mpx: 32 -> 32
// with bf16 outputs 172 -> 123 us, 32 -> 16 with the normalisation 156 + 96 ->
// 120 us, data gradient with mask and split 32 -> 32 172 + 383 -> 228 us and
// 16 -> 32 115 + 383 -> 167 us.  Bound by memory: 89, 92, 178 and 156 us at
// copy rate.
//
// A workgroup runs down up to kConvStrips such tiles: its weights are loaded once,
// and the next tile's pixels are in flight while this one is computed (not with
// element stores, which leave no registers for them: 168 -> 139 us without).
// Without both the four kernels took 186, 155, 307 and 268 us (stores
// straight from the lanes' registers included); rounding value by value 132,
// 122, 239 and 173 us.
constexpr int kConvRows = 8, kConvStrips = 4;  // rows of a tile, most tiles of a workgroup

template <int CIN, int COUT, ConvEpilogue EPI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, EPI == kConvAny ? 4 : 3))) void k_conv_fwd_tile(ffh::ConvArgs a) {
  static_assert(CIN % 16 == 0, "Cin must be a multiple of 16");
  static_assert(COUT == 16 || COUT == 32, "Cout 16 or 32");
  constexpr int KC = CIN / 16, TW = 32, TR = kConvRows, LW = TW + 2;
  constexpr int PX16 = CIN / 8 + 1;  // 16-byte slots per staged pixel (one of padding)
  constexpr int NL = (TR + 2) * LW * (CIN / 8), NI = (NL + 255) / 256;  // 16-byte loads of a tile, per thread
  __shared__ uint4 s_in[(TR + 2) * LW * PX16];
  __shared__ __attribute__((aligned(16))) uint8_t s_tr[4][2048];
  const int rows = TR * a.strips, tiles_x = (a.W + TW - 1) / TW, strips = (a.H + rows - 1) / rows;
  const int img = blockIdx.x / (tiles_x * strips), t = blockIdx.x % (tiles_x * strips);
  const int x0 = (t % tiles_x) * TW, ys = (t / tiles_x) * rows, ye = min(ys + rows, a.H);
  uint4 px[NI];
  auto load = [&](int y0) {
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int k = threadIdx.x + 256 * it, c16 = k % (CIN / 8), p = (k / (CIN / 8)) % LW, ry = k / ((CIN / 8) * LW);
      const int sx = x0 - 1 + p, sy = y0 - 1 + ry;
      px[it] = make_uint4(0, 0, 0, 0);
      if (k < NL && sx >= 0 && sx < a.W && sy >= 0 && sy < a.H)
        px[it] = reinterpret_cast<const uint4 *>(a.in + (((size_t)img * a.H + sy) * a.W + sx) * CIN)[c16];
    }
  };
  load(ys);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row = lane & 31, kh = lane >> 5, col = row;  // weights: output channel col; pixels: x0 + row
  uint4 ub[9 * KC];
  const uint32_t wmask = col < COUT ? 0xFFFFFFFFu : 0u;  // channels beyond Cout multiply by zero
#pragma unroll
  for (int tap = 0; tap < 9; ++tap) {
    const uint4 *wsrc = reinterpret_cast<const uint4 *>(a.w + ((size_t)min(col, COUT - 1) * 9 + tap) * CIN);
#pragma unroll
    for (int cc = 0; cc < KC; ++cc) {
      const uint4 w = wsrc[cc * 2 + kh];
      ub[tap * KC + cc] = make_uint4(w.x & wmask, w.y & wmask, w.z & wmask, w.w & wmask);
    }
  }
  [[maybe_unused]] float bias[COUT / 2], bias_col = 0.0f;
  if constexpr (EPI == kConvAny)
    bias_col = a.bias && col < COUT ? a.bias[col] : 0.0f;
  else
    conv_bias<COUT>(a.bias, kh, bias);
  for (int y0 = ys; y0 < ye; y0 += TR) {
    if (y0 > ys) __syncthreads();  // the previous tile is read
    if (EPI == kConvAny && y0 > ys) load(y0);
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int k = threadIdx.x + 256 * it, c16 = k % (CIN / 8), p = (k / (CIN / 8)) % LW, ry = k / ((CIN / 8) * LW);
      if (k < NL) s_in[(ry * LW + p) * PX16 + c16] = px[it];
    }
    __syncthreads();
    if (EPI != kConvAny && y0 + TR < ye) load(y0 + TR);
    for (int rr = wave; rr < TR && y0 + rr < a.H; rr += 4) {
      f32x16 acc = {0};
#pragma unroll
      for (int tap = 0; tap < 9; ++tap) {
        const uint4 *src = s_in + ((rr + tap / 3) * LW + row + tap % 3) * PX16;
#pragma unroll
        for (int cc = 0; cc < KC; ++cc) {
          const bf16x8 w = as_bf16x8(ub[tap * KC + cc]), x = as_bf16x8(src[cc * 2 + kh]);
          acc = EPI == kConvAny ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, w, acc, 0, 0, 0)
                                : __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, x, acc, 0, 0, 0);
        }
      }
      const size_t q0 = ((size_t)img * a.H + y0 + rr) * a.W + x0;
      const int n = min(TW, a.W - x0);
      if constexpr (EPI == kConvAny)
        conv_store_any<COUT>(a, q0, n, lane, acc, bias_col);
      else
        conv_store<COUT, EPI>(a, q0, n, lane, acc, bias, s_tr[wave]);
    }
  }
}

// The whole network for inference in one launch (1 -> 32 -> 32 -> 16, ReLU
// after the first two layers, optionally unit length per pixel).  A workgroup
// walks down columns of 60 pixels, kNetRows image rows a step; the first
// layer's outputs (60 + 4 columns) and the second's stay in LDS in rings of
// kNetRows + 2 rows (zero outside the image: the "same" padding of the next
// layer), so the activations never leave the chip and only the columns'
// borders and the two rows a run starts with are computed twice.  A wave
// computes one row (two blocks of 32 pixels) per layer and step.  Every layer
// issues the matrix-core products of k_conv_fwd (first layer) and
// k_conv_fwd_tile (32 pixels of a row per product, taps then channel chunks,
// the same operands) and the same bias, ReLU and bf16 rounding, and the
// normalisation is l2norm16: the features are bit for bit those of the three
// convolution launches and the normalisation launch.
//
// Bound by the matrix cores (74 products a wave and step), the LDS reads that
// feed them (one 16-byte read per lane and product) and the epilogues' vector
// instructions, which overlap only between the two workgroups of a compute
// unit (registers: 36 weight operands).  Tiles of 60 x 4 with their borders
// computed for each took 523 us for ten 1024 x 436 images; this takes 210.
constexpr int kNetRows = 4, kNetTW = 60, kNetCols = 64, kNetRing = kNetRows + 2;
constexpr int kNetPX = 80, kNetRowB = kNetCols * kNetPX;  // bytes per staged pixel (16 of padding) and row
constexpr int kNetInC = kNetCols + 2;

__global__ __launch_bounds__(256, 2) void k_descnet_fwd(ffh::NetArgs a) {
  // two pixels more: blocks read past a row's last column (results not used)
  __shared__ __attribute__((aligned(16))) uint8_t s_a1[kNetRing * kNetRowB + 2 * kNetPX];
  __shared__ __attribute__((aligned(16))) uint8_t s_a2[kNetRing * kNetRowB + 2 * kNetPX];
  __shared__ __attribute__((aligned(16))) uint8_t s_tr[4][2048];
  __shared__ __attribute__((aligned(16))) float s_bias[80];
  // input rows of a step; two rows and two pixels more for the lanes that
  // hold the ninth tap only
  __shared__ uint16_t s_in[(kNetRows + 4) * kNetInC + 4];
  const int W = a.W, H = a.H, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = lane & 31, kh = lane >> 5, col = row;
  const int tiles_x = (W + kNetTW - 1) / kNetTW, steps = (H + kNetRows - 1) / kNetRows;
  const long long i0 = blockIdx.x * a.per_wg, i1 = min(i0 + a.per_wg, (long long)a.B * tiles_x * steps);
  uint16_t bw1[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int tap = 8 * kh + e;
    bw1[e] = tap < 9 ? a.w1[col * 9 + tap] : (uint16_t)0;
  }
  uint4 ub1, ub2[18], ub3[18];
  __builtin_memcpy(&ub1, bw1, 16);
  const uint32_t wmask = col < 16 ? 0xFFFFFFFFu : 0u;  // third layer: rows beyond the 16 outputs multiply by zero
#pragma unroll
  for (int tap = 0; tap < 9; ++tap)
#pragma unroll
    for (int cc = 0; cc < 2; ++cc) {
      ub2[tap * 2 + cc] = reinterpret_cast<const uint4 *>(a.w2 + ((size_t)col * 9 + tap) * 32)[cc * 2 + kh];
      const uint4 w = reinterpret_cast<const uint4 *>(a.w3 + ((size_t)min(col, 15) * 9 + tap) * 32)[cc * 2 + kh];
      ub3[tap * 2 + cc] = make_uint4(w.x & wmask, w.y & wmask, w.z & wmask, w.w & wmask);
    }
  if (tid < 80) s_bias[tid] = tid < 32 ? a.b1[tid] : tid < 64 ? a.b2[tid - 32] : a.b3[tid - 64];

  // bias, ReLU and bf16 of one pixel's 16 channels of this lane (8 g + 4 kh +
  // q), zero where `keep` is (outside the image)
  auto store_bf16 = [&](uint8_t *px, const f32x16 &acc, const float *bias, uint32_t keep) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 b = *reinterpret_cast<const float4 *>(bias + 8 * g + 4 * kh);
      const uint32_t h0 = f32x2_to_bf16(fmaxf(acc[4 * g] + b.x, 0.0f), fmaxf(acc[4 * g + 1] + b.y, 0.0f));
      const uint32_t h1 = f32x2_to_bf16(fmaxf(acc[4 * g + 2] + b.z, 0.0f), fmaxf(acc[4 * g + 3] + b.w, 0.0f));
      *reinterpret_cast<uint2 *>(px + 16 * g + 8 * kh) = make_uint2(h0 & keep, h1 & keep);
    }
  };
  auto ring = [](int slot) { return slot >= kNetRing ? slot - kNetRing : slot; };
  // both blocks of row `wave`: the map's rows base + wave .. base + wave + 2
  auto products = [&](const uint8_t *map, int base, const uint4(&ub)[18], f32x16 &acc0, f32x16 &acc1) {
    acc0 = acc1 = f32x16{0};
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
      const uint8_t *p = map + ring(base + wave + dy) * kNetRowB + row * kNetPX + 16 * kh;
#pragma unroll
      for (int k = 0; k < 6; ++k) {  // dx, then channel chunk
        const uint4 v0 = *reinterpret_cast<const uint4 *>(p + (k >> 1) * kNetPX + 32 * (k & 1));
        const uint4 v1 = *reinterpret_cast<const uint4 *>(p + (32 + (k >> 1)) * kNetPX + 32 * (k & 1));
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ub[dy * 6 + k]), as_bf16x8(v0), acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ub[dy * 6 + k]), as_bf16x8(v1), acc1, 0, 0, 0);
      }
    }
  };

  for (long long i = i0; i < i1;) {
    const int c = (int)(i / steps), s0 = (int)(i % steps), s1 = (int)min((long long)steps, s0 + (i1 - i));
    i += s1 - s0;
    const int img = c / tiles_x, x0 = (c % tiles_x) * kNetTW;
    const size_t plane = (size_t)img * H * W;
    uint16_t nx[2];
    auto load = [&](int s) {  // input rows 4 s + 1 .. 4 s + 6, columns from x0 - 3
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int k = tid + 256 * j, y = kNetRows * s + 1 + k / kNetInC, x = x0 - 3 + k % kNetInC;
        nx[j] = 0;
        if (k < (kNetRows + 2) * kNetInC && y >= 0 && y < H && x >= 0 && x < W) nx[j] = a.in[plane + (size_t)y * W + x];
      }
    };
    auto put = [&] {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        if (tid + 256 * j < (kNetRows + 2) * kNetInC) s_in[tid + 256 * j] = nx[j];
    };
    load(s0 - 1);
    put();  // the previous run's input is read (its last step's first barrier)
    __syncthreads();
    // The step before the first computes the rows above: with y = 4 s, a step
    // adds rows y + 2 .. y + 5 of the first layer and y + 1 .. y + 4 of the
    // second (two of them from rows that a run's first step does not have;
    // they are not used), and writes y .. y + 3.  Slot `base` holds row y of
    // the first layer's ring and y - 1 of the second's.
    int base = 0;
    for (int s = s0 - 1; s < s1; ++s, base = ring(base + kNetRows)) {
      const int y = kNetRows * s;
      const int put_row = ring(base + 2 + wave) * kNetRowB;
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) {
        // K = 9 taps padded to 16, lane half kh holds taps 8 kh .. 8 kh + 7
        const uint16_t *p = s_in + (wave + 2 * kh) * kNetInC + 32 * blk + row + 2 * kh;
        uint16_t av[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) av[e] = p[(e / 3) * kNetInC + e % 3];
        uint4 ua;
        __builtin_memcpy(&ua, av, 16);
        const uint32_t rest = kh ? 0u : 0xFFFFFFFFu;
        ua = make_uint4(ua.x & (rest | 0xFFFFu), ua.y & rest, ua.z & rest, ua.w & rest);
        f32x16 acc = {0};
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(ub1), as_bf16x8(ua), acc, 0, 0, 0);
        const int py = y + 2 + wave, px = x0 - 2 + 32 * blk + row;
        store_bf16(s_a1 + put_row + (32 * blk + row) * kNetPX, acc, s_bias,
                   py >= 0 && py < H && px >= 0 && px < W ? 0xFFFFFFFFu : 0u);
      }
      if (s + 1 < s1) load(s + 1);
      __syncthreads();
      f32x16 acc0, acc1;
      products(s_a1, base, ub2, acc0, acc1);
      {
        const int py = y + 1 + wave, px = x0 - 1 + row;
        const bool in = py >= 0 && py < H;
        uint8_t *q = s_a2 + put_row + row * kNetPX;
        store_bf16(q, acc0, s_bias + 32, in && px >= 0 && px < W ? 0xFFFFFFFFu : 0u);
        store_bf16(q + 32 * kNetPX, acc1, s_bias + 32, in && px + 32 < W ? 0xFFFFFFFFu : 0u);
      }
      if (s + 1 < s1) put();
      __syncthreads();
      if (s < s0) continue;
      products(s_a2, base, ub3, acc0, acc1);
      const int n = y + wave < H ? min(kNetTW, W - x0) : 0;
#pragma unroll
      for (int blk = 0; blk < 2; ++blk) {
        const f32x16 &acc = blk ? acc1 : acc0;
        float v[2][4], o[2][4];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const float4 b = *reinterpret_cast<const float4 *>(s_bias + 64 + 8 * g + 4 * kh);
          v[g][0] = acc[4 * g] + b.x;
          v[g][1] = acc[4 * g + 1] + b.y;
          v[g][2] = acc[4 * g + 2] + b.z;
          v[g][3] = acc[4 * g + 3] + b.w;
        }
        if (a.normalize) {  // over all 16 channels: the other lane half holds the other 8
#pragma unroll
          for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) o[g][q] = __shfl_xor(v[g][q], 32);
          float4 f[4];
#pragma unroll
          for (int g = 0; g < 2; ++g) {
            const float4 mine = make_float4(v[g][0], v[g][1], v[g][2], v[g][3]);
            const float4 theirs = make_float4(o[g][0], o[g][1], o[g][2], o[g][3]);
            f[2 * g] = kh ? theirs : mine;
            f[2 * g + 1] = kh ? mine : theirs;
          }
          const float r = l2norm16(f, a.delta);
#pragma unroll
          for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int q = 0; q < 4; ++q) v[g][q] *= r;
        }
#pragma unroll
        for (int g = 0; g < 2; ++g)
          *reinterpret_cast<float4 *>(s_tr[wave] + run_chunk(row, 2 * g + kh)) =
              make_float4(v[g][0], v[g][1], v[g][2], v[g][3]);
        lds_in_order();
        store_run(s_tr[wave], reinterpret_cast<uint8_t *>(a.out + (plane + (size_t)(y + wave) * W + x0 + 32 * blk) * 16),
                  n - 32 * blk, lane, nullptr);
        lds_in_order();
      }
    }
  }
}

// W'[ci][tap][co] = W[co][8 - tap][ci]
__global__ __launch_bounds__(256) void k_flip(const uint16_t *w, uint16_t *wf, int cin, int cout) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= cin * 9 * cout) return;
  const int co = i % cout, tap = (i / cout) % 9, ci = i / (cout * 9);
  wf[i] = w[((size_t)co * 9 + (8 - tap)) * cin + ci];
}

// Partial weight and bias gradients of a run of pixels on matrix cores.
// gw[co][tap][ci] = sum over pixels p of g[p][co] * x[p + d(tap)][ci] is a
// contraction over pixels: per tap, D[co][ci] (32 x 32) += A[co][16 pixels]
// x B[16 pixels][ci] with v_mfma_f32_32x32x16_bf16.  x is bf16 already; the
// float32 gradient is split as g_hi = bf16(g) and g_lo = bf16(g - g_hi) (by the
// caller's epilogues, kSplit, or here) and both parts are multiplied (bf16
// products are exact in float32, and |g - g_hi - g_lo| <= 2^-17 |g|), so
// every term keeps float32-level accuracy.  The bias gradient sum_p g is one
// more product with B = 1 (for Cin = 1 the nine taps and the bias are the
// columns of one product).  With Cout = 16 both parts are the rows of one
// operand and are added at the end.
//
// An operand's lane holds 8 pixels of one channel, memory holds the channels
// of a pixel: the LDS transpose reads (ds_read_b64_tr_b16: 16 lanes read 4
// pixels x 16 channels, lane i gets channel i) give that from rows stored as
// they come, and a tap one pixel aside is the same read 64 bytes on.  A wave
// walks down a column of 16 pixels by itself: it loads one row of x (18
// pixels) and of g ahead, keeps the operands of three rows of x in
// registers, and needs no barrier; every value is read from memory once (x:
// 18/16 times).  Bound by that traffic and by the 18 products a row.  Staging
// transposed with 2-byte LDS stores, three rows of x for every row of g, one
// barrier pair per 64 pixels, took 576 us (32 -> 32), 487 (32 -> 16) and 152
// (1 -> 32) for 3.6 Mpx; this takes 175, 132 and 132.
//
// The four waves' sums are added in LDS in a fixed order and each workgroup
// writes one partial; k_wgrad_reduce adds the partials in a fixed order, so
// the result is deterministic.
typedef short s16x4 __attribute__((ext_vector_type(4)));

// Operand of 16 pixels (k) x 32 channels from LDS rows of 64 bytes per pixel,
// the first pixel at `p`: this lane's channel (lane & 31), its 8 pixels.
__device__ __forceinline__ bf16x8 read_pixels_tr(const uint8_t *p, int lane) {
  const int j = lane & 15;
  const uint8_t *q = p + (8 * (lane >> 5) + (j >> 2)) * 64 + 32 * ((lane >> 4) & 1) + 8 * (j & 3);
  union {
    s16x4 h[2];
    bf16x8 v;
  } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)q);
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(q + 256));
  return u.v;
}

// the 8 bf16 at entries e0 + s .. e0 + s + 7 (s = -1, 0, 1) of an LDS row,
// from the aligned reads lo = [e0 - 8, e0), mid = [e0, e0 + 8), hi = [e0 + 8,
// e0 + 16)
__device__ __forceinline__ uint4 shifted8(uint4 lo, uint4 mid, uint4 hi, int s) {
  if (s == 0) return mid;
  if (s > 0)
    return make_uint4(__builtin_amdgcn_alignbyte(mid.y, mid.x, 2), __builtin_amdgcn_alignbyte(mid.z, mid.y, 2),
                      __builtin_amdgcn_alignbyte(mid.w, mid.z, 2), __builtin_amdgcn_alignbyte(hi.x, mid.w, 2));
  return make_uint4(__builtin_amdgcn_alignbyte(mid.x, lo.w, 2), __builtin_amdgcn_alignbyte(mid.y, mid.x, 2),
                    __builtin_amdgcn_alignbyte(mid.z, mid.y, 2), __builtin_amdgcn_alignbyte(mid.w, mid.z, 2));
}

// Items: (image, column of 16 pixels, row), row fastest; wave w takes items
// [w * per_wave, (w + 1) * per_wave).
template <int CIN, int COUT, bool kSplit>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_wgrad_partial(ffh::ConvArgs a,
                                                                                               long long per_wave) {
  static_assert((CIN == 1 || CIN == 32) && (COUT == 16 || COUT == 32), "Cin 1 or 32, Cout 16 or 32");
  constexpr int NP = CIN == 1 ? 1 : 10;  // products per pixel block: 9 taps and the bias
  constexpr int XB = CIN == 1 ? 3 * 64 : 18 * 64;  // x: three rows of 32 bf16 (ring) or one row of 18 pixels
  constexpr int GB = COUT == 32 ? 2048 : 1024;     // g: 16 pixels of both parts
  constexpr int WAVE_LDS = XB + GB;
  static_assert(WAVE_LDS % 16 == 0 && 4 * WAVE_LDS <= 4 * 32 * 32 * 4, "the reduction reuses the staging");
  __shared__ __attribute__((aligned(16))) float s_red[4][32 * 32];  // the four waves' sums of one product
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, kh = lane >> 5;
  uint8_t *sx = reinterpret_cast<uint8_t *>(s_red) + wave * WAVE_LDS, *sg = sx + XB;
  f32x16 acc[NP];
#pragma unroll
  for (int t = 0; t < NP; ++t) acc[t] = f32x16{0};
  const bf16x8 ones = as_bf16x8(make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));  // bf16 1.0
  const int cx = (a.W + 15) >> 4, W = a.W, H = a.H;
  const long long total = (long long)a.B * cx * H;
  const long long i0 = min(((long long)blockIdx.x * 4 + wave) * per_wave, total), i1 = min(i0 + per_wave, total);

  int y = (int)(i0 % H), c = (int)((i0 / H) % cx), img = (int)(i0 / ((long long)H * cx));
  const uint4 zero4 = make_uint4(0u, 0u, 0u, 0u);
  // next row of x and g, in flight
  uint4 xr[2] = {zero4, zero4}, gr[2] = {zero4, zero4};
  uint32_t xs = 0;
  auto load_x = [&](int row) {  // pixels 16 c - 1 .. 16 c + 16 of a row; zeros outside the image
    const bool in_row = row >= 0 && row < H;
    const size_t base = ((size_t)img * H + (in_row ? row : 0)) * W;
    if constexpr (CIN == 32) {
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        const int k = lane + 64 * it, x = 16 * c - 1 + (k >> 2);
        xr[it] = zero4;
        if (in_row && k < 72 && x >= 0 && x < W)
          xr[it] = *reinterpret_cast<const uint4 *>(a.in + (base + x) * 32 + 8 * (k & 3));
      }
    } else {
      const int x = 16 * c - 1 + lane;
      xs = in_row && lane < 18 && x >= 0 && x < W ? a.in[base + x] : 0u;
    }
  };
  auto store_x = [&](int row) {
    if constexpr (CIN == 32) {
      *reinterpret_cast<uint4 *>(sx + 16 * lane) = xr[0];
      if (lane < 8) *reinterpret_cast<uint4 *>(sx + 1024 + 16 * lane) = xr[1];
    } else if (lane < 18) {  // pixel 16 c - 8 + i at entry i of the row's slot
      reinterpret_cast<uint16_t *>(sx)[((row + 3) % 3) * 32 + 7 + lane] = (uint16_t)xs;
    }
  };
  auto load_g = [&](int row) {
    const size_t base = ((size_t)img * H + row) * W;
    gr[0] = gr[1] = zero4;
    if constexpr (kSplit) {
      if constexpr (COUT == 32) {
        const int x = 16 * c + (lane >> 2);
        if (x < W) {
          gr[0] = *reinterpret_cast<const uint4 *>(a.g_hi + (base + x) * 32 + 8 * (lane & 3));
          gr[1] = *reinterpret_cast<const uint4 *>(a.g_lo + (base + x) * 32 + 8 * (lane & 3));
        }
      } else {
        const int x = 16 * c + ((lane & 31) >> 1);
        if (x < W) gr[0] = *reinterpret_cast<const uint4 *>((kh ? a.g_lo : a.g_hi) + (base + x) * 16 + 8 * (lane & 1));
      }
    } else {
#pragma unroll
      for (int it = 0; it < COUT / 16; ++it) {
        const int k = lane + 64 * it, x = 16 * c + k / (COUT / 4);
        if (x < W) gr[it] = *reinterpret_cast<const uint4 *>(a.gout + (base + x) * COUT + 4 * (k % (COUT / 4)));
      }
    }
  };
  // LDS rows of 64 bytes per pixel: Cout = 32: the high parts, then the low
  // ones 1 KB on; Cout = 16: a pixel's high parts and low parts side by side
  auto store_g = [&]() {
    if constexpr (kSplit) {
      if constexpr (COUT == 32) {
        *reinterpret_cast<uint4 *>(sg + 16 * lane) = gr[0];
        *reinterpret_cast<uint4 *>(sg + 1024 + 16 * lane) = gr[1];
      } else {
        *reinterpret_cast<uint4 *>(sg + ((lane & 31) >> 1) * 64 + 32 * kh + 16 * (lane & 1)) = gr[0];
      }
    } else {
#pragma unroll
      for (int it = 0; it < COUT / 16; ++it) {
        const int k = lane + 64 * it, px = k / (COUT / 4), v = k % (COUT / 4);
        const uint32_t w[4] = {gr[it].x, gr[it].y, gr[it].z, gr[it].w};
        uint32_t hi[4], lo[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float g = __uint_as_float(w[e]);
          hi[e] = f32_to_bf16(g);
          lo[e] = f32_to_bf16(g - bf16_to_f32((uint16_t)hi[e]));
        }
        *reinterpret_cast<uint2 *>(sg + px * 64 + 8 * v) = pack4(hi);
        *reinterpret_cast<uint2 *>(sg + (COUT == 32 ? 1024 : 32) + px * 64 + 8 * v) = pack4(lo);
      }
    }
  };
  bf16x8 xb[3][3];  // operands of rows y - 1, y, y + 1 at dx = -1, 0, 1
  auto read_x = [&](int slot) {
    if constexpr (CIN == 32) {
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) xb[slot][dx] = read_pixels_tr(sx + 64 * dx, lane);
    }
  };
  bool fresh = true;
  for (long long i = i0; i < i1; ++i) {
    lds_in_order();
    if (fresh) {  // a new column: rows y - 1 and y first
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        load_x(y - 1 + k);
        store_x(y - 1 + k);
        lds_in_order();
        read_x(k);
        lds_in_order();
      }
      load_x(y + 1);
      load_g(y);
    }
    store_x(y + 1);
    store_g();
    lds_in_order();
    read_x(2);
    const bf16x8 ahi = read_pixels_tr(sg, lane);
    bf16x8 alo = ahi;
    if constexpr (COUT == 32) alo = read_pixels_tr(sg + 1024, lane);
    [[maybe_unused]] bf16x8 b1 = ones;
    if constexpr (CIN == 1) {
      // column n of B: tap n (n < 9), the bias (n = 9), nothing beyond
      uint4 bv = zero4;
      const int dy = min(col / 3, 2);
      const uint16_t *r = reinterpret_cast<const uint16_t *>(sx) + ((y + dy + 2) % 3) * 32 + 8 * kh;
      const uint4 lo = *reinterpret_cast<const uint4 *>(r), mid = *reinterpret_cast<const uint4 *>(r + 8),
                  hi = *reinterpret_cast<const uint4 *>(r + 16);
      if (col < 9) bv = shifted8(lo, mid, hi, col % 3 - 1);
      b1 = col == 9 ? ones : as_bf16x8(bv);
    }
    lds_in_order();
    // the next row's loads, in flight during the products
    const bool down = y + 1 < H;
    if (i + 1 < i1 && down) {
      load_x(y + 2);
      load_g(y + 1);
    }
    if constexpr (CIN == 1) {
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi, b1, acc[0], 0, 0, 0);
      if constexpr (COUT == 32) acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo, b1, acc[0], 0, 0, 0);
    } else {
#pragma unroll
      for (int t = 0; t < 10; ++t) {
        const bf16x8 b = t < 9 ? xb[t / 3][t % 3] : ones;
        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ahi, b, acc[t], 0, 0, 0);
        if constexpr (COUT == 32) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(alo, b, acc[t], 0, 0, 0);
      }
#pragma unroll
      for (int dx = 0; dx < 3; ++dx) {
        xb[0][dx] = xb[1][dx];
        xb[1][dx] = xb[2][dx];
      }
    }
    fresh = !down;
    if (down) {
      ++y;
    } else {
      y = 0;
      if (++c == cx) {
        c = 0;
        ++img;
      }
    }
  }
  // D[co][n]: a lane holds column n = col, rows co = 8 (r / 4) + 4 kh + r % 4.
  // The four waves' sums of each product are added in a fixed order.
  float *part = a.partial + (size_t)blockIdx.x * (COUT * 9 * CIN + COUT);
#pragma unroll
  for (int t = 0; t < NP; ++t) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) s_red[wave][(8 * (r >> 2) + 4 * kh + (r & 3)) * 32 + col] = acc[t][r];
    __syncthreads();
    for (int e = tid; e < COUT * 32; e += 256) {
      const int co = e >> 5, n = e & 31;
      float v = ((s_red[0][e] + s_red[1][e]) + s_red[2][e]) + s_red[3][e];
      if constexpr (COUT == 16) {  // the low parts' rows
        const int f = e + 16 * 32;
        v += ((s_red[0][f] + s_red[1][f]) + s_red[2][f]) + s_red[3][f];
      }
      if constexpr (CIN == 1) {
        if (n < 9) part[co * 9 + n] = v;
        else if (n == 9) part[COUT * 9 + co] = v;
      } else if (t < 9) {
        part[((size_t)co * 9 + t) * CIN + n] = v;
      } else if (n == 0) {
        part[COUT * 9 * CIN + co] = v;
      }
    }
  }
}

// Sum of the per-workgroup partials: 32 threads per output, each adding a
// contiguous 1/32 of the partials in order, then the 32 sums in a fixed tree
// (deterministic).  Latency-bound chains of loads: eight threads per output
// took 43 us for 1024 partials of 9248 values, 32 and half the partials 9.
__global__ __launch_bounds__(1024) void k_wgrad_reduce(const float *partial, int nblocks, int len, float *gw,
                                                       float *gbias, int nw) {
  __shared__ float s[32][33];
  const int o = threadIdx.x & 31, seg = threadIdx.x >> 5, i = blockIdx.x * 32 + o;
  float v = 0.0f;
  if (i < len) {
    const int b0 = (int)((long long)nblocks * seg / 32), b1 = (int)((long long)nblocks * (seg + 1) / 32);
#pragma unroll 4
    for (int b = b0; b < b1; ++b) v += partial[(size_t)b * len + i];
  }
  s[seg][o] = v;
  __syncthreads();
  for (int w = 16; w > 0; w >>= 1) {
    if (seg < w) s[seg][o] += s[seg + w][o];
    __syncthreads();
  }
  if (seg == 0 && i < len) {
    if (i < nw) gw[i] = s[0][o];
    else if (gbias) gbias[i - nw] = s[0][o];
  }
}

// grad_pre = grad_post where the post-activation is positive, else 0; also
// the bf16 copy for the next matrix-core pass.
__global__ __launch_bounds__(256) void k_relu_bwd(const uint16_t *act, const float *g, float *gout, uint16_t *gout_bf16,
                                                  long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float v = (act == nullptr || bf16_to_f32(act[i]) > 0.0f) ? g[i] : 0.0f;
  if (gout) gout[i] = v;
  if (gout_bf16) gout_bf16[i] = f32_to_bf16(v);
}

__global__ __launch_bounds__(256) void k_f32_to_bf16(const float *x, uint16_t *y, long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) y[i] = f32_to_bf16(x[i]);
}

// Image bytes -> network input v / 255 - 0.5 (bf16).
__global__ __launch_bounds__(256) void k_image_to_bf16(const uint8_t *img, uint16_t *out, long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) out[i] = f32_to_bf16((float)img[i] * (1.0f / 255.0f) - 0.5f);
}

// Adam (Kingma and Ba 2015) with bias correction; writes the bf16 copy.
__global__ __launch_bounds__(256) void k_adam(float *p, const float *g, float *m, float *v, int count, float lr,
                                              float b1, float b2, float eps, float c1, float c2, uint16_t *p_bf16) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  if (p_bf16) p_bf16[i] = f32_to_bf16(pi);
}

// Unit length per pixel of 16-channel features: y = f / sqrt(|f|^2 + delta).
__global__ __launch_bounds__(256) void k_l2norm16_fwd(const float4 *f, long long P, float delta, float4 *y,
                                                      float *inv_norm) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P) return;
  float4 v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = f[p * 4 + k];
  const float r = l2norm16(v, delta);
#pragma unroll
  for (int k = 0; k < 4; ++k) y[p * 4 + k] = v[k];
  if (inv_norm) inv_norm[p] = r;
}

// dL/df = r * (g - y * <g, y>) with r = 1 / sqrt(|f|^2 + delta).
__global__ __launch_bounds__(256) void k_l2norm16_bwd(const float4 *y, const float *inv_norm, const float4 *g,
                                                      long long P, float4 *gin) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= P) return;
  float4 yv[4], gv[4];
  float d = 0.0f;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    yv[k] = y[p * 4 + k];
    gv[k] = g[p * 4 + k];
    d += yv[k].x * gv[k].x + yv[k].y * gv[k].y + yv[k].z * gv[k].z + yv[k].w * gv[k].w;
  }
  const float r = inv_norm[p];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    gin[p * 4 + k] = make_float4(r * (gv[k].x - yv[k].x * d), r * (gv[k].y - yv[k].y * d),
                                 r * (gv[k].z - yv[k].z * d), r * (gv[k].w - yv[k].w * d));
}

// A float32 gradient as two bf16 parts (hi + lo), 4 values per thread.
__device__ __forceinline__ void store_split(float4 g, uint16_t *hi, uint16_t *lo) {
  const float v[4] = {g.x, g.y, g.z, g.w};
  uint32_t h[4], l[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    h[c] = f32_to_bf16(v[c]);
    l[c] = f32_to_bf16(v[c] - bf16_to_f32((uint16_t)h[c]));
  }
  *reinterpret_cast<uint2 *>(hi) = pack4(h);
  *reinterpret_cast<uint2 *>(lo) = pack4(l);
}

// k_l2norm16_bwd with its result split, four lanes per pixel (coalesced 16-
// byte accesses); y nullptr: the split alone.  The inner product is taken by
// every lane over all 16 channels in k_l2norm16_bwd's order (the other lanes'
// values by shuffles), so the gradient has the same bits.
__global__ __launch_bounds__(256) void k_l2norm16_bwd_split(const float4 *y, const float *inv_norm, const float4 *g,
                                                            long long P, uint16_t *hi, uint16_t *lo) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x, p = min(i >> 2, P - 1);
  const int k = (int)(i & 3), base = (threadIdx.x & 63) & ~3;
  float4 v = g[p * 4 + k];
  if (y) {
    const float4 yk = y[p * 4 + k];
    float d = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      float4 a, b;
      a.x = __shfl(yk.x, base + q), a.y = __shfl(yk.y, base + q), a.z = __shfl(yk.z, base + q), a.w = __shfl(yk.w, base + q);
      b.x = __shfl(v.x, base + q), b.y = __shfl(v.y, base + q), b.z = __shfl(v.z, base + q), b.w = __shfl(v.w, base + q);
      d += a.x * b.x + a.y * b.y + a.z * b.z + a.w * b.w;
    }
    const float r = inv_norm[p];
    v = make_float4(r * (v.x - yk.x * d), r * (v.y - yk.y * d), r * (v.z - yk.z * d), r * (v.w - yk.w * d));
  }
  if ((i >> 2) < P) store_split(v, hi + p * 16 + 4 * k, lo + p * 16 + 4 * k);
}

// Triplet hinge of m (positive, negative) cost pairs: cost[0..m) positives,
// cost[m..2m) negatives.  Loss = weight * sum_k max(0, margin + scale *
// (cost[k] - cost[m + k])); grad[k] = +weight*scale and grad[m + k] =
// -weight*scale where the hinge is active, else 0.  One workgroup: the
// loss is summed in a fixed order (thread-strided partials, then a tree),
// so it is deterministic.
__global__ __launch_bounds__(1024) void k_triplet_hinge(const float *cost, int m, float margin, float scale,
                                                        float weight, float *grad, float *loss) {
  __shared__ float s_part[1024];
  float acc = 0.0f;
  for (int k = threadIdx.x; k < m; k += 1024) {
    const float h = margin + scale * (cost[k] - cost[m + k]);
    const bool on = h > 0.0f;
    acc += on ? h : 0.0f;
    grad[k] = on ? weight * scale : 0.0f;
    grad[m + k] = on ? -weight * scale : 0.0f;
  }
  s_part[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 512; w > 0; w >>= 1) {
    if (threadIdx.x < w) s_part[threadIdx.x] += s_part[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) *loss = weight * s_part[0];
}

// One map or the two of a pair, quantised with one range.
struct QuantMaps {
  const float *f[2];
  uint8_t *q[2];
  long long count;
  int wide;  // 16-byte aligned maps, 4-byte aligned outputs
};

// Per-map range of float features (block partials, then one block).
// (blockIdx.y selects the map; both maps of a pair in one launch and four
// floats a load: two of 1024 x 436 x 16 in 13 instead of 24 us.)
__global__ __launch_bounds__(256) void k_minmax_partial(QuantMaps m, float *part) {
  __shared__ float s_lo[256], s_hi[256];
  const float *f = m.f[blockIdx.y];
  part += 2 * (size_t)blockIdx.y * gridDim.x;
  float lo = INFINITY, hi = -INFINITY;
  const long long first = (long long)blockIdx.x * 256 + threadIdx.x, step = (long long)gridDim.x * 256;
  const long long n4 = m.wide ? m.count >> 2 : 0;
#pragma unroll 4
  for (long long i = first; i < n4; i += step) {
    const float4 v = reinterpret_cast<const float4 *>(f)[i];
    lo = fminf(lo, fminf(fminf(v.x, v.y), fminf(v.z, v.w)));
    hi = fmaxf(hi, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
  }
  for (long long i = 4 * n4 + first; i < m.count; i += step) {
    lo = fminf(lo, f[i]);
    hi = fmaxf(hi, f[i]);
  }
  s_lo[threadIdx.x] = lo;
  s_hi[threadIdx.x] = hi;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) {
      s_lo[threadIdx.x] = fminf(s_lo[threadIdx.x], s_lo[threadIdx.x + s]);
      s_hi[threadIdx.x] = fmaxf(s_hi[threadIdx.x], s_hi[threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = s_lo[0];
    part[2 * blockIdx.x + 1] = s_hi[0];
  }
}

// The range over the partials (min and max are order-independent), into
// part[2 * nparts], part[2 * nparts + 1].
__global__ __launch_bounds__(256) void k_minmax_final(float *part, int nparts) {
  __shared__ float s_lo[256], s_hi[256];
  float lo = INFINITY, hi = -INFINITY;
  for (int k = threadIdx.x; k < nparts; k += 256) {  // min and max: any order gives the same result
    lo = fminf(lo, part[2 * k]);
    hi = fmaxf(hi, part[2 * k + 1]);
  }
  s_lo[threadIdx.x] = lo;
  s_hi[threadIdx.x] = hi;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      s_lo[threadIdx.x] = fminf(s_lo[threadIdx.x], s_lo[threadIdx.x + w]);
      s_hi[threadIdx.x] = fmaxf(s_hi[threadIdx.x], s_hi[threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    part[2 * nparts] = s_lo[0];
    part[2 * nparts + 1] = s_hi[0];
  }
}

// q = clamp(rint((f - lo) * (255 / (hi - lo))), 0, 255).  Four values a
// thread, the maps of a pair in one launch (as above: 26 -> 13 us).
__global__ __launch_bounds__(256) void k_quantize(QuantMaps m, const float *range) {
  const float lo = range[0], hi = range[1];
  const float s = hi > lo ? 255.0f / (hi - lo) : 0.0f;
  const float *f = m.f[blockIdx.y];
  uint8_t *q = m.q[blockIdx.y];
  auto level = [&](float v) { return (uint8_t)fminf(fmaxf(rintf((v - lo) * s), 0.0f), 255.0f); };
  const long long i = 4 * ((long long)blockIdx.x * blockDim.x + threadIdx.x);
  if (m.wide && i + 4 <= m.count) {
    const float4 v = *reinterpret_cast<const float4 *>(f + i);
    *reinterpret_cast<uint32_t *>(q + i) = (uint32_t)level(v.x) | (uint32_t)level(v.y) << 8 |
                                           (uint32_t)level(v.z) << 16 | (uint32_t)level(v.w) << 24;
    return;
  }
  for (int e = 0; e < 4; ++e)
    if (i + e < m.count) q[i + e] = level(f[i + e]);
}

}  // namespace

namespace ffh {

static unsigned blocks_of(long long n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_conv_fwd(const ConvArgs &args, hipStream_t stream) {
  ConvArgs a = args;
  const long long P = (long long)a.B * a.H * a.W;
  const unsigned grid = (unsigned)((P + 127) / 128);
  if (P == 0) return hipSuccess;
  const bool wide = (((uintptr_t)a.out_f32 | (uintptr_t)a.out_bf16) & 15) == 0;
  // Tiles that a workgroup runs down (k_conv_fwd_tile): what the 256 compute
  // units have each, at most kConvStrips.  32 -> 32 with bf16 outputs, us a call:
  // 150 tiles (two of 160 x 120) 8.4 with one a workgroup and 11.5 with four; 600
  // (two of 320 x 240) 11.0, 10.8 and 10.5 with one, two and three, 12.7 with four;
  // 8100 (1920 x 1080) 84, 70 and 68, 62 with four.  Stores element by element
  // gain less from it, four times as many tiles each: 600 tiles 11.7 with one
  // and 12.8 with three, 8100 tiles 89 and, with four, 71.
  const long long single = (long long)a.B * ((a.W + 31) / 32) * ((a.H + kConvRows - 1) / kConvRows);
  a.strips = (int)std::min<long long>(wide ? (single + 255) / 256 : single / 1024 + 1, kConvStrips);
  const int rows = kConvRows * a.strips;
  const long long tiles = (long long)a.B * ((a.W + 31) / 32) * ((a.H + rows - 1) / rows);
  if (tiles > 0x7FFFFFFF) return hipErrorInvalidValue;
  auto launch = [&](auto kernel, unsigned groups) {
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(256), 0, stream, a);
    return hipGetLastError();
  };
#define TILE(CIN, COUT, EPI) launch(k_conv_fwd_tile<CIN, COUT, EPI>, (unsigned)tiles)
  if (a.inv_norm)  // the last layer with the normalisation
    return a.cin == 32 && a.cout == 16 ? TILE(32, 16, kConvNorm) : hipErrorInvalidValue;
  if (a.act) {  // a data gradient through a ReLU
    if (a.cout != 32 || (a.cin != 32 && a.cin != 16)) return hipErrorInvalidValue;
    return a.cin == 32 ? TILE(32, 32, kConvMask) : TILE(16, 32, kConvMask);
  }
  if (a.cin == 1 && a.cout == 32)
    return wide ? launch(k_conv_fwd<1, 32, kConvPlain>, grid) : launch(k_conv_fwd<1, 32, kConvAny>, grid);
  if (a.cin == 32 && a.cout == 32) return wide ? TILE(32, 32, kConvPlain) : TILE(32, 32, kConvAny);
  if (a.cin == 32 && a.cout == 16) return wide ? TILE(32, 16, kConvPlain) : TILE(32, 16, kConvAny);
  if (a.cin == 16 && a.cout == 32) return wide ? TILE(16, 32, kConvPlain) : TILE(16, 32, kConvAny);
#undef TILE
  return hipErrorInvalidValue;
}

hipError_t launch_descnet_fwd(NetArgs a, hipStream_t stream) {
  // two workgroups per compute unit, each with one run of steps
  const long long items = (long long)a.B * ((a.W + kNetTW - 1) / kNetTW) * ((a.H + kNetRows - 1) / kNetRows);
  if (items <= 0 || items > INT32_MAX) return hipErrorInvalidValue;
  a.per_wg = (items + 511) / 512;
  hipLaunchKernelGGL(k_descnet_fwd, dim3((unsigned)((items + a.per_wg - 1) / a.per_wg)), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_weight_flip(const uint16_t *w, uint16_t *wf, int cin, int cout, hipStream_t stream) {
  hipLaunchKernelGGL(k_flip, dim3(blocks_of((long long)cin * 9 * cout)), dim3(256), 0, stream, w, wf, cin, cout);
  return hipGetLastError();
}

int wgrad_blocks(int B, int H) { return std::min(B * H, 1024); }

template <int CIN, int COUT>
static void wgrad_kernel(const ConvArgs &a, int blocks, long long per_wave, hipStream_t stream) {
  if (a.g_hi)
    hipLaunchKernelGGL((k_wgrad_partial<CIN, COUT, true>), dim3(blocks), dim3(256), 0, stream, a, per_wave);
  else
    hipLaunchKernelGGL((k_wgrad_partial<CIN, COUT, false>), dim3(blocks), dim3(256), 0, stream, a, per_wave);
}

hipError_t launch_wgrad(const ConvArgs &a, float *gw, float *gbias, hipStream_t stream) {
  // two workgroups per compute unit (two waves per SIMD), each with one run of
  // items per wave; at least two items a wave: the three rows a run starts with
  // and the partials cost less than idle units (32 -> 32, us a call with at least
  // 16, 4 and 2: 64 x 48 21.8, 12.9 and 11.3; two of 160 x 120 24.4, 15.5 and
  // 16.7; two of 320 x 240 24.9, 23.0 and 22.9)
  const long long items = (long long)a.B * ((a.W + 15) / 16) * a.H;
  const int nb = (int)std::max<long long>(1, std::min<long long>(std::min(wgrad_blocks(a.B, a.H), 512), items / 8));
  const long long per_wave = (items + 4ll * nb - 1) / (4ll * nb);
  if (a.cin == 1 && a.cout == 32) wgrad_kernel<1, 32>(a, nb, per_wave, stream);
  else if (a.cin == 32 && a.cout == 32) wgrad_kernel<32, 32>(a, nb, per_wave, stream);
  else if (a.cin == 32 && a.cout == 16) wgrad_kernel<32, 16>(a, nb, per_wave, stream);
  else return hipErrorInvalidValue;
  const int nw = a.cout * 9 * a.cin, len = nw + a.cout;
  hipLaunchKernelGGL(k_wgrad_reduce, dim3((unsigned)((len + 31) / 32)), dim3(1024), 0, stream, a.partial, nb, len, gw,
                     gbias, nw);
  return hipGetLastError();
}

hipError_t launch_relu_bwd(const uint16_t *act, const float *g, float *gout, uint16_t *gout_bf16, long long count,
                           hipStream_t stream) {
  if (count > 0)
    hipLaunchKernelGGL(k_relu_bwd, dim3(blocks_of(count)), dim3(256), 0, stream, act, g, gout, gout_bf16, count);
  return hipGetLastError();
}

hipError_t launch_f32_to_bf16(const float *x, uint16_t *y, long long count, hipStream_t stream) {
  if (count > 0) hipLaunchKernelGGL(k_f32_to_bf16, dim3(blocks_of(count)), dim3(256), 0, stream, x, y, count);
  return hipGetLastError();
}

hipError_t launch_image_to_bf16(const uint8_t *img, uint16_t *out, long long count, hipStream_t stream) {
  if (count > 0) hipLaunchKernelGGL(k_image_to_bf16, dim3(blocks_of(count)), dim3(256), 0, stream, img, out, count);
  return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, int count, float lr, float b1, float b2,
                       float eps, int step, uint16_t *p_bf16, hipStream_t stream) {
  const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
  if (count > 0)
    hipLaunchKernelGGL(k_adam, dim3(blocks_of(count)), dim3(256), 0, stream, p, g, m, v, count, lr, b1, b2, eps, c1,
                       c2, p_bf16);
  return hipGetLastError();
}

hipError_t launch_l2norm16_fwd(const float *f, long long P, float delta, float *y, float *inv_norm,
                               hipStream_t stream) {
  if (P > 0)
    hipLaunchKernelGGL(k_l2norm16_fwd, dim3(blocks_of(P)), dim3(256), 0, stream, reinterpret_cast<const float4 *>(f),
                       P, delta, reinterpret_cast<float4 *>(y), inv_norm);
  return hipGetLastError();
}

hipError_t launch_l2norm16_bwd(const float *y, const float *inv_norm, const float *g, long long P, float *gin,
                               hipStream_t stream) {
  if (P > 0)
    hipLaunchKernelGGL(k_l2norm16_bwd, dim3(blocks_of(P)), dim3(256), 0, stream, reinterpret_cast<const float4 *>(y),
                       inv_norm, reinterpret_cast<const float4 *>(g), P, reinterpret_cast<float4 *>(gin));
  return hipGetLastError();
}

hipError_t launch_l2norm16_bwd_split(const float *y, const float *inv_norm, const float *g, long long P, uint16_t *hi,
                                     uint16_t *lo, hipStream_t stream) {
  constexpr long long kMost = 1ll << 29;  // pixels of a launch: four threads each, fewer than 2^32
  for (long long p = 0; p < P; p += kMost) {
    const long long n = std::min(P - p, kMost);
    hipLaunchKernelGGL(k_l2norm16_bwd_split, dim3(blocks_of(4 * n)), dim3(256), 0, stream,
                       reinterpret_cast<const float4 *>(y ? y + 16 * p : nullptr), y ? inv_norm + p : nullptr,
                       reinterpret_cast<const float4 *>(g + 16 * p), n, hi + 16 * p, lo + 16 * p);
  }
  return hipGetLastError();
}

hipError_t launch_triplet_hinge(const float *cost, int m, float margin, float scale, float weight, float *grad,
                                float *loss, hipStream_t stream) {
  hipLaunchKernelGGL(k_triplet_hinge, dim3(1), dim3(1024), 0, stream, cost, m, margin, scale, weight, grad, loss);
  return hipGetLastError();
}

constexpr int kQuantParts = 1024;

static void quantize_maps(QuantMaps m, int maps, float *part, hipStream_t stream) {
  m.wide = (((uintptr_t)m.f[0] | (uintptr_t)m.f[1]) & 15) == 0 && (((uintptr_t)m.q[0] | (uintptr_t)m.q[1]) & 3) == 0;
  float *range = part + 2 * maps * kQuantParts;
  hipLaunchKernelGGL(k_minmax_partial, dim3(kQuantParts, maps), dim3(256), 0, stream, m, part);
  hipLaunchKernelGGL(k_minmax_final, dim3(1), dim3(256), 0, stream, part, maps * kQuantParts);
  hipLaunchKernelGGL(k_quantize, dim3(blocks_of((m.count + 3) / 4), maps), dim3(256), 0, stream, m, range);
}

hipError_t launch_quantize(const float *f, long long count, float *part, uint8_t *q, hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  quantize_maps({{f, f}, {q, q}, count, 0}, 1, part, stream);
  return hipGetLastError();
}

// Two maps with the range of their union: partials of map 1, then of map 2,
// one final reduction over both, both quantised with that range.
hipError_t launch_quantize_pair(const float *f1, const float *f2, long long count, float *part, uint8_t *q1,
                                uint8_t *q2, hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  quantize_maps({{f1, f2}, {q1, q2}, count, 0}, 2, part, stream);
  return hipGetLastError();
}

size_t quantize_scratch_bytes() { return (size_t)(2 * kQuantParts + 1) * 2 * sizeof(float); }

}  // namespace ffh
