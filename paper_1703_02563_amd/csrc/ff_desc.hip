// Scale-space low-pass and per-pixel descriptors (Sec. 3.2 scale spaces,
// Sec. 3.6 low-pass filtering and replicate border condition).
//
// I^n: integer box filter of half-width h = max(1, n/2), rounded half up,
// computed separably (row sums, then column sums of the row sums; both are
// exact in integers), per 64 x 64 tile in LDS.  Descriptor of scale n: the 16 samples of I^n on a 4x4
// grid with spacing 2n around the pixel, stored as one 16-byte vector per
// pixel so that a patch position costs one 128-bit load; the pixels of each
// row are stored in phase order (x mod n, then x / n), and the map carries a
// replicated border of 3n pixels (desc_col, desc_index).
//
// All (image, scale) jobs of a call run in one launch per stage: blockIdx.z
// selects the job.
#include <algorithm>

#include "ff_device.h"
#include "ff_internal.h"

namespace {

using ffk::clampi;

// Box filter of one (image, scale) job on a 64 x 64 tile of outputs: the
// input tile with its h-wide border (edge pixels replicated) is staged in
// LDS, every staged row gets the row sums of the tile's 64 columns by a
// sliding window over 8 consecutive columns, then every output takes the
// column sum of 2h + 1 row sums, also sliding over 8 rows, rounded half up
// over the box area.  These are the integer sums of the separable
// definition (exact in any order), in one pass over the image.  Row sums read
// four samples at a time, and the rounded quotient is a multiplication: with
// byte reads and a division per pixel ten 1024 x 436 images took 15.6 us and
// twelve of 1920 x 1080 52, now 13 and 42.
constexpr int kBT = 64, kBHmax = 32, kBS = kBT + 2 * kBHmax;  // tile, largest half-width (n <= 64), staged side

struct BlurTile {
  __attribute__((aligned(16))) uint8_t in[kBS * kBS + 16];  // rows of a multiple of 4 bytes; the last dword read ends past one
  uint16_t row[kBS * kBT];  // (2h + 1) * 255 fits 16 bits
};

__device__ __forceinline__ void blur_tile(BlurTile &sm, const uint8_t *img, uint8_t *blurred, int W, int H, int n,
                                          int x0, int y0) {
  uint8_t *s_in = sm.in;
  uint16_t *s_row = sm.row;
  const int h = max(1, n >> 1), S = kBT + 2 * h;  // staged rows and columns
  const int Sp = (S + 3) & ~3;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  // staged rows ty + 4u, columns tx and tx + 64: 16 loads in flight per
  // thread before their LDS stores (rows past S read a clamped row, unused)
  const int xa = clampi(x0 - h + tx, W - 1), xb = clampi(x0 - h + tx + 64, W - 1);
  for (int u0 = 0; u0 < S; u0 += 32) {
    uint32_t va[8], vb[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint8_t *row = img + (size_t)clampi(y0 - h + u0 + ty + 4 * u, H - 1) * W;
      va[u] = row[xa];
      vb[u] = row[xb];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = u0 + ty + 4 * u;
      if (r < S) {
        s_in[r * Sp + tx] = (uint8_t)va[u];
        if (tx + 64 < S) s_in[r * Sp + tx + 64] = (uint8_t)vb[u];
      }
    }
  }
  __syncthreads();
  // row sums of staged row r for output columns c0 .. c0 + 7 (window of
  // output column c: staged columns c .. c + 2h)
  for (int k = threadIdx.x; k < S * (kBT / 8); k += 256) {
    const int r = k >> 3, c0 = (k & 7) * 8;
    const uint32_t *row = reinterpret_cast<const uint32_t *>(s_in + r * Sp + c0);  // four samples each
    const int full = (2 * h + 1) >> 2, rest = (2 * h + 1) & 3;  // of the first window
    uint32_t sum = 0;
    for (int k4 = 0; k4 < full; ++k4) sum = __builtin_amdgcn_sad_u8(row[k4], 0u, sum);
    const uint32_t t0 = row[full], t1 = row[full + 1], t2 = row[full + 2];
    sum = __builtin_amdgcn_sad_u8(t0 & ((1u << (8 * rest)) - 1u), 0u, sum);
    // samples 2h + 1 .. 2h + 7 enter, 0 .. 6 leave
    const uint32_t in[2] = {__builtin_amdgcn_alignbyte(t1, t0, rest), __builtin_amdgcn_alignbyte(t2, t1, rest)};
    const uint32_t lv[2] = {row[0], row[1]};
    uint32_t w[4] = {sum, 0, 0, 0};
#pragma unroll
    for (int c = 1; c < 8; ++c) {
      sum += (in[(c - 1) >> 2] >> (8 * ((c - 1) & 3))) & 0xFFu;
      sum -= (lv[(c - 1) >> 2] >> (8 * ((c - 1) & 3))) & 0xFFu;
      w[c >> 1] |= sum << (16 * (c & 1));
    }
    *reinterpret_cast<uint4 *>(s_row + r * kBT + c0) = make_uint4(w[0], w[1], w[2], w[3]);
  }
  __syncthreads();
  // column sums for output column c, rows r0 .. r0 + 7 (window of output
  // row r: staged rows r .. r + 2h)
  const uint32_t area = (uint32_t)((2 * h + 1) * (2 * h + 1));
  const uint32_t recip = 0xFFFFFFFFu / area + 1;  // exact for every sum of every h <= 32
  for (int k = threadIdx.x; k < kBT * (kBT / 8); k += 256) {
    const int c = k & (kBT - 1), r0 = (k / kBT) * 8, x = x0 + c;
    const uint16_t *col = s_row + r0 * kBT + c;
    uint32_t sum = 0;
#pragma unroll 8
    for (int dy = 0; dy <= 2 * h; ++dy) sum += col[dy * kBT];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if (r > 0) {
        sum += col[(r + 2 * h) * kBT];
        sum -= col[(r - 1) * kBT];
      }
      const int y = y0 + r0 + r;
      if (x < W && y < H) blurred[(size_t)y * W + x] = (uint8_t)__umulhi(sum + area / 2, recip);
    }
  }
}

__global__ __launch_bounds__(256) void k_blur(ffh::DescJobs jobs) {
  __shared__ BlurTile sm;
  const ffh::DescJob &jb = jobs.job[blockIdx.z];
  blur_tile(sm, jb.img, jb.blurred, jobs.W, jobs.H, jb.n, blockIdx.x * kBT, blockIdx.y * kBT);
}

// Weight-class row entry (wform_index) of pixel x of blurred row `row`, for
// patch radius r.
__device__ __forceinline__ uint4 wform_entry(const uint8_t *row, int W, int n, int x, int r = 3) {
  auto at = [&](int a) { return (uint32_t)row[clampi(x + n * a, W - 1)]; };
  if (r == 4)
    return make_uint4(at(-7) | at(-6) << 8 | at(6) << 16 | at(7) << 24, at(-5) | at(-4) << 8 | at(4) << 16 | at(5) << 24,
                      at(-3) | at(-2) << 8 | at(2) << 16 | at(3) << 24, at(-1) | at(0) << 8 | at(1) << 16);
  if (r == 2)
    return make_uint4(at(-5) | at(-4) << 8 | at(4) << 16 | at(5) << 24, at(-3) | at(-2) << 8 | at(2) << 16 | at(3) << 24,
                      at(-1) | at(1) << 8, at(0));
  return make_uint4(at(-6) | at(-5) << 8 | at(5) << 16 | at(6) << 24, at(-4) | at(-3) << 8 | at(3) << 16 | at(4) << 24,
                    at(-2) | at(-1) << 8 | at(1) << 16 | at(2) << 24, at(0));
}

// One workgroup per stored row yp of one map: the four blurred rows its
// descriptors sample (y + n(2gy - 3), clamped) are staged in LDS once, then
// every entry of the padded row (coalesced 16-byte stores) takes its 16
// samples from there.  Entries that are image pixels also go to the
// row-major copy when one is requested.  The weight-class row map has the
// same rows (y + 3n); its row yp is written from a fifth staged row, the
// blurred row y itself.  Dynamic LDS: five rows of Ws bytes.
//
// Bound by the stores and by the vector instructions that gather an entry.
// Rows are read in aligned dwords whatever their width (a staged row keeps its
// address modulo 4), and an entry's pixel is found with multiplications by
// reciprocals.  Before: 33 us for 741 x 497 (5 scales, both images), 38 for
// 1242 x 375, 230 for eight pairs of 2.1 Mpx; now 25, 25
// and 191 (and 25 -> 23 for 1024 x 436, 145 -> 132 for 1920 x 1080, six scales).  Rows staged in phase
// order, so that the samples of a row gy are adjacent bytes (two aligned LDS
// reads, two shifts and a permute), cost more in staging than they save (30, 32
// and 233 us), with unaligned LDS reads much more (46, 55 and 333).
__host__ __device__ __forceinline__ int desc_row_stride(int W) { return (W + 15) & ~15; }

__device__ __forceinline__ void desc_row(uint8_t *s_rows, int Ws, const ffh::DescJob &jb, int W, int H, int yp) {
  const int n = jb.n, l2 = ffk::map_log2(n);
  const int P = ffk::desc_pad(n), Wp = W + 2 * P;
  const int yr = yp - P, y = clampi(yr, H - 1);
  // staged rows g = 0..3: y + n(2g - 3); g = 4: y itself (weight-class map)
  const int nrows = jb.wform ? 5 : 4;
  const uint8_t *src[5];
  int off[5], mis = 0;  // a row's address modulo 4
#pragma unroll
  for (int g = 0; g < 5; ++g) {
    src[g] = jb.blurred + (size_t)(g < 4 ? clampi(y + n * (2 * g - 3), H - 1) : y) * W;
    off[g] = (int)(reinterpret_cast<uintptr_t>(src[g]) & 3);
    mis |= off[g];
  }
  if (!mis && (W & 3) == 0) {
    for (int q = threadIdx.x; 4 * q < W; q += blockDim.x)
#pragma unroll
      for (int g = 0; g < 5; ++g)
        if (g < nrows)
          reinterpret_cast<uint32_t *>(s_rows + g * Ws)[q] = reinterpret_cast<const uint32_t *>(src[g])[q];
  } else if (Ws >= W + 3) {
    for (int q = threadIdx.x; 4 * q < W + 3; q += blockDim.x) {
      uint32_t v[5];
#pragma unroll
      for (int g = 0; g < 5; ++g) {
        const int x = 4 * q - off[g];
        v[g] = 0;
        if (g >= nrows) continue;
        if (x >= 0 && x + 4 <= W) {
          v[g] = *reinterpret_cast<const uint32_t *>(src[g] + x);
        } else {  // the row's own bytes of its first and last dword
          for (int j = 0; j < 4; ++j)
            if (x + j >= 0 && x + j < W) v[g] |= (uint32_t)src[g][x + j] << (8 * j);
        }
      }
#pragma unroll
      for (int g = 0; g < 5; ++g)
        if (g < nrows) reinterpret_cast<uint32_t *>(s_rows + g * Ws)[q] = v[g];
    }
  } else {
#pragma unroll
    for (int g = 0; g < 5; ++g) off[g] = 0;
    for (int k = threadIdx.x; k < nrows * W; k += blockDim.x) {
      const int g = k / W, x = k - g * W;
      s_rows[g * Ws + x] = jb.blurred[(size_t)(g < 4 ? clampi(y + n * (2 * g - 3), H - 1) : y) * W + x];
    }
  }
  __syncthreads();
  // the weight-class map's rows y in [-3n, H + 3n) are a band of the
  // descriptor map's rows [-4n, H + 4n): stored row y + 3n
  const int ywf = yr + ffk::kWformPad * n;
  if (jb.wform && ywf >= 0 && ywf < H + 2 * ffk::kWformPad * n) {
    uint4 *wout = reinterpret_cast<uint4 *>(jb.wform) + (size_t)ywf * W;
    for (int x = threadIdx.x; x < W; x += blockDim.x) wout[x] = wform_entry(s_rows + 4 * Ws + off[4], W, n, x, jb.wradius);
  }
  uint4 *out = reinterpret_cast<uint4 *>(jb.desc) + (size_t)yp * Wp;
  // desc_pixel with its quotients by reciprocals, exact for columns below 2^16
  const int q = Wp >> l2, m = Wp & ((1 << l2) - 1);
  const uint32_t rq = 0xFFFFFFFFu / (uint32_t)q + 1, rq1 = 0xFFFFFFFFu / (uint32_t)(q + 1) + 1;
  for (int c = threadIdx.x; c < Wp; c += blockDim.x) {
    const bool lead = c < (q + 1) * m;  // phases with one entry more
    const int c2 = lead ? c : c - (q + 1) * m;
    const int f = (int)__umulhi((uint32_t)c2, lead ? rq1 : rq);
    const int xr = (lead ? f : m + f) + ((c2 - f * (lead ? q + 1 : q)) << l2) - P, x = clampi(xr, W - 1);
    uint32_t w[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const uint8_t *row = s_rows + g * Ws + off[g];
      uint32_t v = 0;
#pragma unroll
      for (int gx = 0; gx < 4; ++gx) v |= (uint32_t)row[clampi(x + n * (2 * gx - 3), W - 1)] << (8 * gx);
      w[g] = v;
    }
    const uint4 d = make_uint4(w[0], w[1], w[2], w[3]);
    if (jb.desc) out[c] = d;
    if (jb.compact && xr >= 0 && xr < W && yr >= 0 && yr < H)
      reinterpret_cast<uint4 *>(jb.compact)[(size_t)yr * W + xr] = d;
  }
}

__global__ __launch_bounds__(256) void k_desc(ffh::DescJobs jobs, int Ws) {
  extern __shared__ uint8_t s_rows[];
  const ffh::DescJob &jb = jobs.job[blockIdx.y];
  if ((int)blockIdx.x >= jobs.H + 2 * ffk::desc_pad(jb.n)) return;  // workgroup-uniform
  desc_row(s_rows, Ws, jb, jobs.W, jobs.H, blockIdx.x);
}

// ---- batches: the same work units, one workgroup each --------------------
// (pixel-wise separable sums through a row-sum buffer and descriptors straight
// from global memory took 624 us for eight pairs of 2.1 Mpx in all, weight-class
// maps of every scale included; the units of the single-pair kernels, and
// those maps only where a variant reads them, 242 us; 2048 or 4096 workgroups
// striding through the items cost 28 us more than one for each)

// Items (pair, image * L + scale, 64 x 64 tile).
__global__ __launch_bounds__(256) void k_blur_batch(ffh::BatchStage st) {
  __shared__ BlurTile sm;
  ffk::for_items(st.total, [&](int item) {
    const int p = ffk::batch_pair(st.prefix, st.npairs, item);
    const ffh::BatchPair &bp = st.pairs[p];
    const int tx = (bp.W + kBT - 1) / kBT, tiles = tx * ((bp.H + kBT - 1) / kBT);
    const int local = item - st.prefix[p], z = local / tiles, t = local % tiles, im = z / st.L, lv = z % st.L;
    blur_tile(sm, bp.img[im], bp.blur[im][lv], bp.W, bp.H, 1 << lv, (t % tx) * kBT, (t / tx) * kBT);
    __syncthreads();  // the next item stages its tile
  });
}

// Items (pair, scale, image, stored row).
__global__ __launch_bounds__(256) void k_desc_batch(ffh::BatchStage st, int Ws) {
  extern __shared__ uint8_t s_rows[];
  ffk::for_items(st.total, [&](int item) {
    const int p = ffk::batch_pair(st.prefix, st.npairs, item);
    const ffh::BatchPair &bp = st.pairs[p];
    int local = item - st.prefix[p], lv = 0;
    while (local >= 2 * (bp.H + 2 * ffk::desc_pad(1 << lv))) local -= 2 * (bp.H + 2 * ffk::desc_pad(1 << lv++));
    const int Hp = bp.H + 2 * ffk::desc_pad(1 << lv), im = local / Hp;
    const ffh::DescJob jb = {bp.img[im], bp.blur[im][lv], bp.desc[im][lv], lv == 0 ? bp.desc1[im] : nullptr,
                             (st.wform_scales >> lv) & 1 ? bp.wform[im][lv] : nullptr, 1 << lv, 3};
    desc_row(s_rows, Ws, jb, bp.W, bp.H, local % Hp);
    __syncthreads();  // the next item stages its rows
  });
}

}  // namespace

namespace ffh {

int batch_blur_items(int W, int H, int L) { return 2 * L * ((W + kBT - 1) / kBT) * ((H + kBT - 1) / kBT); }

int batch_desc_items(int H, int L) {
  int rows = 0;
  for (int lv = 0; lv < L; ++lv) rows += 2 * (H + 2 * ffk::desc_pad(1 << lv));
  return rows;
}

// Dynamic LDS of the descriptor rows of a W-wide image.
// *Ws: bytes per row, with three for its alignment where they fit.
static hipError_t desc_lds(const void *kernel, int W, int *Ws, size_t *lds) {
  *Ws = desc_row_stride(W + 3);
  if (5 * (size_t)*Ws > 160 * 1024) *Ws = desc_row_stride(W);
  *lds = 5 * (size_t)*Ws;
  if (*lds > 160 * 1024) return hipErrorInvalidValue;
  if (*lds > 64 * 1024)  // rows wider than 12 K pixels
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)*lds);
  return hipSuccess;
}

hipError_t launch_batch_descriptors(const BatchStage &tiles, const BatchStage &rows, int max_width,
                                    hipStream_t stream) {
  if (tiles.total <= 0 || rows.total <= 0) return hipSuccess;
  size_t lds;
  int Ws;
  const hipError_t e = desc_lds(reinterpret_cast<const void *>(k_desc_batch), max_width, &Ws, &lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_blur_batch, dim3(item_groups(tiles.total)), dim3(256), 0, stream, tiles);
  hipLaunchKernelGGL(k_desc_batch, dim3(item_groups(rows.total)), dim3(256), lds, stream, rows, Ws);
  return hipGetLastError();
}

// Five scales of two 1024 x 436 images in one launch: 13 us; a blur and a
// descriptor launch for each, of which only the blurred image is wanted, 140.
hipError_t launch_blur(const DescJobs &jobs, hipStream_t stream) {
  if (jobs.count <= 0) return hipSuccess;
  for (int k = 0; k < jobs.count; ++k)
    if (jobs.job[k].n < 1 || jobs.job[k].n > 2 * kBHmax + 1) return hipErrorInvalidValue;
  if (5 * (size_t)desc_row_stride(jobs.W) > 160 * 1024) return hipErrorInvalidValue;  // as launch_descriptors
  const dim3 gb((jobs.W + kBT - 1) / kBT, (jobs.H + kBT - 1) / kBT, jobs.count);
  hipLaunchKernelGGL(k_blur, gb, dim3(256), 0, stream, jobs);
  return hipGetLastError();
}

hipError_t launch_descriptors(const DescJobs &jobs, hipStream_t stream) {
  if (jobs.count <= 0) return hipSuccess;
  size_t lds;
  int Ws;
  hipError_t e = desc_lds(reinterpret_cast<const void *>(k_desc), jobs.W, &Ws, &lds);
  if (e != hipSuccess || (e = launch_blur(jobs, stream)) != hipSuccess) return e;
  int pmax = 0;
  for (int k = 0; k < jobs.count; ++k) pmax = std::max(pmax, ffk::desc_pad(jobs.job[k].n));
  const dim3 gpad(jobs.H + 2 * pmax, jobs.count);
  hipLaunchKernelGGL(k_desc, gpad, dim3(256), lds, stream, jobs, Ws);
  return hipGetLastError();
}

}  // namespace ffh
