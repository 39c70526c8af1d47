// Float patch cost of learned 16-channel features and its gradient.
//
// Cost of entry (x, y, fx, fy) at scale n, patch radius r (Eq. 3 with a
// squared-difference data term for learned features, Sec. 3.5; replicate
// border of Sec. 3.6):
//   C = sum_{v=-r..r} sum_{u=-r..r} sum_{c<16} (f1(clamp(p+n(u,v)))[c] - f2(clamp(p+f+n(u,v)))[c])^2
// accumulated in float32 as four partial sums, one per group of channels
// 4k .. 4k+3, each with one fused multiply-add per term in the order v, u, c,
// then added as (s0 + s1) + (s2 + s3) (fixed, so that every caller sees the
// same rounding).
//
// Backward: dL/df1[q] += 2g(f1(q) - f2(t)), dL/df2[t] -= 2g(f1(q) - f2(t))
// per patch position.  Many entries touch the same pixels, and float
// atomics would make the sums depend on arrival order; each contribution is
// therefore rounded once to 64-bit fixed point (2^-32 units) and added with
// integer atomics, which are associative: the result is deterministic.  A
// term of magnitude 2^31 or more, or a sum that leaves the int64 range,
// would wrap: both are detected (the atomic returns the previous value, so
// the adding thread sees a signed overflow) and counted in an overflow word
// after the accumulators; a nonzero count turns every gradient output into
// NaN instead of a wrapped value.
#include <algorithm>

#include "ff_device.h"
#include "ff_internal.h"

namespace {

using ffk::clampi;

constexpr double kFix = 4294967296.0;  // 2^32

// A quad of lanes per entry: lane k owns channels 4k .. 4k+3, so one load of a
// quad covers a pixel's 64 bytes and the four partial sums of the fixed order
// are the four lanes' own.  Latency-bound (49 dependent additions per lane) with
// few entries: 2,048 at radius 3 on 1024 x 436 62 us with one thread per entry,
// 12 with four.  With many, scattered, bound by the pixels' cache lines, whose
// halves more waves read at different times: up to radius 3 the next row is in
// flight instead (65,536 entries 64.3 -> 62.3 us, one thread per entry 62.3; a
// million 947 -> 912 and 1363); beyond, its registers cost more than they give
// (radius 4, 16,384 entries: 46 against 44).
template <int R>
__global__ __launch_bounds__(256) void k_cost_fwd(ffh::CostArgs a) {
  constexpr int K = 2 * R + 1, D = R <= 3 ? 2 : 1;  // rows in flight
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int e = (int)min(gid >> 2, (long long)a.count - 1), k = (int)(gid & 3);
  const int4 en = a.entries[e];
  const int n = a.n, Wm = a.W - 1, Hm = a.H - 1;
  const float4 *f1 = reinterpret_cast<const float4 *>(a.f1) + k;
  const float4 *f2 = reinterpret_cast<const float4 *>(a.f2) + k;
  float acc = 0.0f;
  float4 x[D][K], y[D][K];
  auto load = [&](int v, float4 (&xr)[K], float4 (&yr)[K]) {
    const size_t qrow = (size_t)clampi(en.y + n * v, Hm) * a.W;
    const size_t trow = (size_t)clampi(en.y + en.w + n * v, Hm) * a.W;
#pragma unroll
    for (int u = -R; u <= R; ++u) {
      xr[u + R] = f1[(qrow + clampi(en.x + n * u, Wm)) * 4];
      yr[u + R] = f2[(trow + clampi(en.x + en.z + n * u, Wm)) * 4];
    }
  };
  auto add = [&](const float4 (&xr)[K], const float4 (&yr)[K]) {
#pragma unroll
    for (int u = 0; u < K; ++u) {
      float d = xr[u].x - yr[u].x;
      acc = __fmaf_rn(d, d, acc);
      d = xr[u].y - yr[u].y;
      acc = __fmaf_rn(d, d, acc);
      d = xr[u].z - yr[u].z;
      acc = __fmaf_rn(d, d, acc);
      d = xr[u].w - yr[u].w;
      acc = __fmaf_rn(d, d, acc);
    }
  };
  if constexpr (D == 2) {
    load(-R, x[0], y[0]);
#pragma unroll
    for (int v = 0; v < K; ++v) {
      if (v + 1 < K) load(v + 1 - R, x[(v + 1) & 1], y[(v + 1) & 1]);
      add(x[v & 1], y[v & 1]);
    }
  } else {
    for (int v = -R; v <= R; ++v) {
      load(v, x[0], y[0]);
      add(x[0], y[0]);
    }
  }
  acc += __shfl_xor(acc, 1);  // s0 + s1 (and s2 + s3 in the quad's upper half)
  acc += __shfl_xor(acc, 2);
  if (k == 0 && (gid >> 2) < a.count) a.cost[e] = acc;
}

// Atomic form (see launch_cost_bwd for when it runs): one thread per (entry,
// patch position).
__global__ __launch_bounds__(256) void k_cost_bwd(ffh::CostArgs a) {
  const int side = 2 * a.radius + 1, P = side * side;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long long)a.count * P) return;
  const int e = (int)(gid / P), k = (int)(gid % P);
  const int v = k / side - a.radius, u = k % side - a.radius;
  const int4 en = a.entries[e];
  const double g2 = 2.0 * (double)a.grad_cost[e];
  if (g2 == 0.0) return;
  unsigned long long *over = reinterpret_cast<unsigned long long *>(a.overflow);
  const int Wm = a.W - 1, Hm = a.H - 1, n = a.n;
  const size_t q = (size_t)clampi(en.y + n * v, Hm) * a.W + clampi(en.x + n * u, Wm);
  const size_t t = (size_t)clampi(en.y + en.w + n * v, Hm) * a.W + clampi(en.x + en.z + n * u, Wm);
  const float *pa = a.f1 + q * 16, *pb = a.f2 + t * 16;
  unsigned long long *acc1 = reinterpret_cast<unsigned long long *>(a.acc1) + q * 16;
  unsigned long long *acc2 = reinterpret_cast<unsigned long long *>(a.acc2) + t * 16;
#pragma unroll
  for (int c = 0; c < 16; ++c) {
    const double d = g2 * ((double)pa[c] - (double)pb[c]);
    if (!(fabs(d) < 2147483648.0)) {  // |term| >= 2^31 (or NaN): no int64 fixed-point value
      atomicAdd(over, 1ull);
      continue;
    }
    const long long fx = __double2ll_rn(d * kFix);
    if (fx != 0) {
      // signed overflow of old + x: both operands of one sign, the sum of the other
      const long long o1 = (long long)atomicAdd(acc1 + c, (unsigned long long)fx);
      const long long o2 = (long long)atomicAdd(acc2 + c, (unsigned long long)(-fx));
      const long long n1 = (long long)((unsigned long long)o1 + (unsigned long long)fx);
      const long long n2 = (long long)((unsigned long long)o2 - (unsigned long long)fx);
      if ((((o1 ^ n1) & (fx ^ n1)) | ((o2 ^ n2) & (-fx ^ n2))) < 0) atomicAdd(over, 1ull);
    }
  }
}

__global__ __launch_bounds__(256) void k_fixed_to_float(const int64_t *acc, const int64_t *overflow, float *out,
                                                        long long count) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) out[i] = *overflow ? __builtin_nanf("") : (float)((double)acc[i] * (1.0 / kFix));
}

// ---- backward by gathering ------------------------------------------------
//
// The atomic form issues 2 * 16 64-bit atomics per entry and patch position
// (103 M for 65,536 entries at radius 3: 4.54 ms, bound by the L2's atomic
// rate).  The sums are integers, so any order gives the same bits: here the
// entries are sorted into bins by their patch centre (p for f1's gradient, the
// target p + f for f2's), and every pixel adds the entries whose patch covers
// it in registers and writes its gradient once.
//
// Bins: one per centre of [-rn, W + rn) x [-rn, H + rn) (rn = radius * n; a
// centre further out is binned at the edge, which reaches the same border
// pixels), each row in phase order (desc_col), so that the 2 radius + 1 centres
// x - n u of a patch row are adjacent bins and their entries one range of
// records.  A row's records are contiguous, the rows' places are handed out by
// an atomic cursor.
struct CostBins {
  int32_t *start[2];  // [Hb][Wb + 1]: counts, then first records (last column: end of the row)
  int32_t *rank[2];   // [count]: the entry's place inside its bin, -1: no contribution;
                      // once the records stand: the crowded pixels
  int4 *rec[2];       // [count]: (flow to the other map, gradient bits, entry)
  int32_t *cursor;    // [5]: records placed, then crowded pixels, per side; workgroups done with them
  int Wb, Hb, rn, log2n;
};

// Index of the entry's bin on one side.
__device__ __forceinline__ size_t cost_bin(const CostBins &b, int4 en, int side, int W, int H) {
  const int cx = side ? en.x + en.z : en.x, cy = side ? en.y + en.w : en.y;
  const int x = clampi(cx + b.rn, b.Wb - 1), y = clampi(cy + b.rn, b.Hb - 1);
  return (size_t)y * (b.Wb + 1) + ffk::desc_col(x, b.log2n, b.Wb);
}

__global__ __launch_bounds__(256) void k_cost_count(ffh::CostArgs a, CostBins b) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x, side = blockIdx.y;
  if (e == 0 && side == 0) *a.overflow = 0;
  if (e >= a.count) return;
  b.rank[side][e] =
      a.grad_cost[e] == 0.0f ? -1 : atomicAdd(b.start[side] + cost_bin(b, a.entries[e], side, a.W, a.H), 1);
}

// One workgroup per row of bins: exclusive sums of its counts from a place
// of its own.
__global__ __launch_bounds__(256) void k_cost_rows(CostBins b) {
  __shared__ int wsum[4], base;
  const int side = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int32_t *row = b.start[side] + (size_t)blockIdx.x * (b.Wb + 1);
  const int per = (b.Wb + 255) / 256, c0 = min(tid * per, b.Wb), c1 = min(c0 + per, b.Wb);
  int sum = 0;
  for (int c = c0; c < c1; ++c) sum += row[c];
  int incl = sum;
  for (int off = 1; off < 64; off <<= 1) {
    const int o = __shfl_up(incl, off);
    if (lane >= off) incl += o;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  if (tid == 0) {
    const int total = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    base = total ? atomicAdd(b.cursor + side, total) : 0;
    row[b.Wb] = base + total;
  }
  __syncthreads();
  int at = base + incl - sum;
  for (int w = 0; w < wave; ++w) at += wsum[w];
  for (int c = c0; c < c1; ++c) {
    const int k = row[c];
    row[c] = at;
    at += k;
  }
}

__global__ __launch_bounds__(256) void k_cost_fill(ffh::CostArgs a, CostBins b) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x, side = blockIdx.y;
  if (e >= a.count) return;
  const int rank = b.rank[side][e];
  if (rank < 0) return;
  const int4 en = a.entries[e];
  const int at = b.start[side][cost_bin(b, en, side, a.W, a.H)] + rank;
  const int g = __float_as_int(a.grad_cost[e]);
  b.rec[side][at] = side ? make_int4(-en.z, -en.w, g, e) : make_int4(en.z, en.w, g, e);
}

// Sum of one lane's four channels with the checks of the atomic form.
struct CostSum {
  long long s[4] = {0, 0, 0, 0};
  unsigned terms = 0, sums = 0;  // terms out of range; sums that left the int64 range
  __device__ __forceinline__ void put(int c, long long fx) {
    const long long t = (long long)((unsigned long long)s[c] + (unsigned long long)fx);
    sums += ((s[c] ^ t) & (fx ^ t)) < 0;
    s[c] = t;
  }
  __device__ __forceinline__ void add(float g, float4 own, float4 other) {
    const double g2 = 2.0 * (double)g;
    const float p[4] = {own.x, own.y, own.z, own.w}, q[4] = {other.x, other.y, other.z, other.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double d = g2 * ((double)p[c] - (double)q[c]);
      if (!(fabs(d) < 2147483648.0)) {  // |term| >= 2^31 (or NaN): no int64 fixed-point value
        ++terms;
        continue;
      }
      put(c, __double2ll_rn(d * kFix));
    }
  }
  __device__ __forceinline__ void merge(const CostSum &o) {
    terms += o.terms;
    sums += o.sums;
#pragma unroll
    for (int c = 0; c < 4; ++c) put(c, o.s[c]);
  }
  // The sums of the wave's 16 quads, in every quad.
  __device__ __forceinline__ void wave_sum() {
#pragma unroll
    for (int off = 4; off < 64; off <<= 1) {
      CostSum o;
#pragma unroll
      for (int c = 0; c < 4; ++c) o.s[c] = __shfl_xor(s[c], off);
      o.terms = __shfl_xor(terms, off);
      o.sums = __shfl_xor(sums, off);
      merge(o);
    }
  }
};

constexpr double kMagic = 6755399441055744.0;  // 3 * 2^51: adding it rounds to an integer
constexpr double kSmall = 2251799813685248.0;  // 2^51: terms of 2^19 in fixed point

// The same with short additions for terms below 2^19 (kMagic's bits summed as
// they are), at most 2047 of them before they join the checked sum.
struct CostFastSum {
  CostSum sum;
  unsigned long long acc[4] = {0, 0, 0, 0};
  unsigned n = 0;
  __device__ __forceinline__ void flush() {
    const unsigned long long bias = (unsigned long long)__double_as_longlong(kMagic) * n;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      sum.put(c, (long long)(acc[c] - bias));
      acc[c] = 0;
    }
    n = 0;
  }
  __device__ __forceinline__ void add(float g, float4 own, float4 other) {
#pragma clang fp contract(off)
    const double g2 = (double)g * (2.0 * kFix);
    const double d0 = g2 * ((double)own.x - (double)other.x), d1 = g2 * ((double)own.y - (double)other.y);
    const double d2 = g2 * ((double)own.z - (double)other.z), d3 = g2 * ((double)own.w - (double)other.w);
    if (fabs(d0) < kSmall && fabs(d1) < kSmall && fabs(d2) < kSmall && fabs(d3) < kSmall) {
      acc[0] += (unsigned long long)__double_as_longlong(d0 + kMagic);
      acc[1] += (unsigned long long)__double_as_longlong(d1 + kMagic);
      acc[2] += (unsigned long long)__double_as_longlong(d2 + kMagic);
      acc[3] += (unsigned long long)__double_as_longlong(d3 + kMagic);
      if (++n == 2047) flush();
    } else {
      sum.add(g, own, other);
    }
  }
};

// A finished pixel: this lane's four channels, and what left the range (a
// term out of range is seen from both sides and counted on the first).
__device__ __forceinline__ void cost_write(const ffh::CostArgs &a, int side, size_t px, const CostSum &sum) {
  const unsigned bad = sum.sums + (side == 0 ? sum.terms : 0u);
  if (bad) atomicAdd(reinterpret_cast<unsigned long long *>(a.overflow), (unsigned long long)bad);
  constexpr double inv = 1.0 / kFix;
  reinterpret_cast<float4 *>(side ? a.grad_f2 : a.grad_f1)[px] =
      make_float4((float)((double)sum.s[0] * inv), (float)((double)sum.s[1] * inv), (float)((double)sum.s[2] * inv),
                  (float)((double)sum.s[3] * inv));
}

// Terms of an interior pixel that its quad sums alone; more make it crowded.
// At least the 225 samples of the largest patch, so that the crowded pixels of a
// side are no more than its entries (the length of their list).
constexpr int kCrowded = 256;
constexpr int kTailGroups = 512;  // workgroups for them (1024: the same, 2048: 20 % slower)

// The terms of interior pixel (x, y): every sample that lands there is exactly
// (x, y), one term per entry of 2R + 1 ranges of records.  Term i of the
// sequence in row v is record first[v] + i, at[v] <= i < at[v + 1].
template <int K>
__device__ __forceinline__ void cost_terms(const CostBins &b, int side, int n, int x, int y, int (&first)[K],
                                           int (&at)[K + 1]) {
  const int stride = b.Wb + 1;
  const int32_t *row = b.start[side] + (size_t)y * stride + ffk::desc_col(x, b.log2n, b.Wb);
  at[0] = 0;
#pragma unroll
  for (int v = 0; v < K; ++v) {
    const int lo = row[(size_t)v * n * stride], hi = row[(size_t)v * n * stride + K];
    first[v] = lo - at[v];
    at[v + 1] = at[v] + (hi - lo);
  }
}
template <int K>
__device__ __forceinline__ int cost_record(const int (&first)[K], const int (&at)[K + 1], int i) {
  int f = first[0];
#pragma unroll
  for (int v = 1; v < K; ++v) f = i >= at[v] ? first[v] : f;
  return f + i;
}

// A border pixel, by a wave.  It also takes the samples outside the image that
// clamp to it: the records of all bins within rn of the pixel along the axis it
// borders.  The ranges of 16 bins at a time, their records dealt out to the 16
// quads, so that neither many empty bins nor one crowded bin is walked by one
// quad.  (Short additions as for the inner pixels would take 34 registers more,
// which the inner pixels pay for: 127 -> 148 us where the corner case below gains
// a fifth.)
template <int R>
__device__ __forceinline__ void cost_border(const ffh::CostArgs &a, const CostBins &b, int side, int x, int y) {
  constexpr int K = 2 * R + 1;
  const int lane = threadIdx.x & 63, quad = lane >> 2, k = lane & 3;
  const int W = a.W, Wm = W - 1, Hm = a.H - 1, n = a.n;
  const size_t px = ((size_t)y * W + x) * 4 + k;
  const float4 *fo = reinterpret_cast<const float4 *>(side ? a.f1 : a.f2) + k;
  const float4 own = reinterpret_cast<const float4 *>(side ? a.f2 : a.f1)[px];
  const int4 *rec = b.rec[side];
  CostSum sum;
  const int sy = (y == 0 || y == Hm) ? 1 : n, np = R > 0 && (x == 0 || x == Wm) ? n : 1;
  const int ranges = (2 * b.rn / sy + 1) * np;
  for (int base = 0; base < ranges; base += 16) {
    const int j = base + quad;
    int lo = 0, len = 0;
    if (j < ranges) {
      // centres x - rn + ph, then every n-th: at most K adjacent bins, one more for phase 0
      const int ph = j % np;
      const int32_t *p =
          b.start[side] + (size_t)(y + j / np * sy) * (b.Wb + 1) + ffk::desc_col(x + ph, b.log2n, b.Wb);
      lo = p[0];
      len = p[ph == 0 ? K : K - 1] - lo;
    }
    int incl = len;
#pragma unroll
    for (int off = 4; off < 64; off <<= 1) {
      const int o = __shfl_up(incl, off);
      if (lane >= off) incl += o;
    }
    const int total = __shfl(incl, 63), at = lo - (incl - len);  // item i of a range is record at + i
    for (int i0 = 0; i0 < total; i0 += 16) {
      const int i = i0 + quad;
      int z = 0;  // the range that holds item i
#pragma unroll
      for (int step = 8; step > 0; step >>= 1) z += __shfl(incl, 4 * (z + step - 1)) <= i ? step : 0;
      const int record = __shfl(at, 4 * z) + i;
      if (i >= total) continue;
      const int4 r = rec[record], en = a.entries[r.w];
      const int cx = side ? en.x + en.z : en.x, cy = side ? en.y + en.w : en.y;
      const float g = __int_as_float(r.z);
      for (int v = -R; v <= R; ++v) {
        if (clampi(cy + n * v, Hm) != y) continue;
        const size_t orow = (size_t)clampi(cy + n * v + r.y, Hm) * W;
        for (int u = -R; u <= R; ++u)
          if (clampi(cx + n * u, Wm) == x) sum.add(g, own, fo[(orow + clampi(cx + n * u + r.x, Wm)) * 4]);
      }
    }
  }
  sum.wave_sum();
  if (quad == 0) cost_write(a, side, px, sum);
}

// Border pixels of an image, and the i-th.
inline __host__ __device__ long long cost_border_count(int W, int H) {
  return W == 1 || H == 1 ? (long long)W * H : 2ll * (W + H - 2);
}
__device__ __forceinline__ void cost_border_pixel(int i, int W, int H, int &x, int &y) {
  if (W == 1 || H == 1) {
    x = W == 1 ? 0 : i;
    y = W == 1 ? i : 0;
  } else if (i < 2 * W) {
    x = i < W ? i : i - W;
    y = i < W ? 0 : H - 1;
  } else {
    x = (i & 1) ? W - 1 : 0;  // 2 W is even
    y = 1 + ((i - 2 * W) >> 1);
  }
}

// Gradient of one side (blockIdx.z).  The first `border_rows` rows of
// workgroups take the border pixels, a wave each; the others 16 x 4 inner pixels,
// four lanes per pixel with four channels each; crowded ones are listed for
// k_cost_tail.  Bound by its vector instructions, issued in 98 % of the cycles
// where every pixel has terms (a term is formed and rounded in float64 as in the
// atomic form and added in 64 bits); record and other map's pixel are both
// prefetched one term ahead.
// The terms of the 2R + 1 ranges run as one sequence, so that the 16 pixels
// of a wave differ only in their total.  With every |term| below 2^19 (51
// bits of fixed point) adding 3 * 2^51 rounds it to an integer whose bits are
// summed as they are; a pixel with a larger term takes the checked additions.
// 65,536 entries at radius 3 on 1024 x 436: the whole backward, sorting
// included, 4.59 ms in the atomic form, 0.33 with border and crowded pixels
// walked by one quad each (waves wait for it), now 0.13.
template <int R>
__global__ __launch_bounds__(256) void k_cost_gather(ffh::CostArgs a, CostBins b, int border_rows) {
  constexpr int K = 2 * R + 1;
  const int k = threadIdx.x & 3, side = blockIdx.z;
  if ((int)blockIdx.y < border_rows) {
    const long long i = ((long long)blockIdx.y * gridDim.x + blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (i >= cost_border_count(a.W, a.H)) return;
    int bx, by;
    cost_border_pixel((int)i, a.W, a.H, bx, by);
    cost_border<R>(a, b, side, bx, by);
    return;
  }
  const int x = blockIdx.x * 16 + ((threadIdx.x >> 2) & 15), y = (blockIdx.y - border_rows) * 4 + (threadIdx.x >> 6);
  const int W = a.W, H = a.H, Wm = W - 1, Hm = H - 1;
  if (x <= 0 || x >= Wm || y <= 0 || y >= Hm) return;
  const size_t px = ((size_t)y * W + x) * 4 + k;
  const float4 *fo = reinterpret_cast<const float4 *>(side ? a.f1 : a.f2) + k;
  const float4 own = reinterpret_cast<const float4 *>(side ? a.f2 : a.f1)[px];
  const int4 *rec = b.rec[side];
  int first[K], at[K + 1];
  cost_terms<K>(b, side, a.n, x, y, first, at);
  const int total = at[K];
  if (total > kCrowded) {
    if (k == 0) b.rank[side][atomicAdd(b.cursor + 2 + side, 1)] = y * W + x;
    return;
  }
  auto record = [&](int i) { return rec[cost_record<K>(first, at, i)]; };
  auto other = [&](int4 r) { return fo[((size_t)clampi(y + r.y, Hm) * W + clampi(x + r.x, Wm)) * 4]; };
  CostSum sum;
  bool checked = false;
  if (total > 0) {
    const double o0 = own.x, o1 = own.y, o2 = own.z, o3 = own.w;
    int4 r0 = record(0), r1 = record(min(1, total - 1));
    float4 q0 = other(r0);
    bool small = true;
    unsigned long long acc[4] = {0, 0, 0, 0};
    for (int i = 0; i < total; ++i) {
      const float4 q1 = other(r1);
      const int4 r2 = record(min(i + 2, total - 1));
      {
#pragma clang fp contract(off)
        const double g = (double)__int_as_float(r0.z) * (2.0 * kFix);
        const double d0 = g * (o0 - (double)q0.x), d1 = g * (o1 - (double)q0.y);
        const double d2 = g * (o2 - (double)q0.z), d3 = g * (o3 - (double)q0.w);
        small = small && fabs(d0) < kSmall && fabs(d1) < kSmall && fabs(d2) < kSmall && fabs(d3) < kSmall;
        acc[0] += (unsigned long long)__double_as_longlong(d0 + kMagic);
        acc[1] += (unsigned long long)__double_as_longlong(d1 + kMagic);
        acc[2] += (unsigned long long)__double_as_longlong(d2 + kMagic);
        acc[3] += (unsigned long long)__double_as_longlong(d3 + kMagic);
      }
      r0 = r1;
      r1 = r2;
      q0 = q1;
    }
    const unsigned long long bias = (unsigned long long)__double_as_longlong(kMagic) * (unsigned long long)total;
#pragma unroll
    for (int c = 0; c < 4; ++c) sum.s[c] = (long long)(acc[c] - bias);
    checked = !small;
  }
  if (checked) {
    sum = CostSum();
    for (int i = 0; i < total; ++i) {
      const int4 r = record(i);
      sum.add(__int_as_float(r.z), own, other(r));
    }
  }
  cost_write(a, side, px, sum);
}

// The crowded pixels, which would keep one quad busy while the others wait: a
// workgroup each, striding through the two sides' lists (integer sums: any order
// gives the same bits).  Then, with the overflow word nonzero, NaN over both
// gradients: by every workgroup where there are no crowded pixels, else by the last
// one that had any, once their gradients are written.
//
// The whole backward at radius 3 with a quad for every pixel, with waves for the
// border and workgroups for crowded pixels, and in the atomic form: 65,536
// entries on a corner 709, 27 and 129 ms, on one inner pixel of 1024 x 436 37, 1.7
// and 22 ms, in 16 x 16 pixels of 160 x 120 7.3, 0.29 and 6.5 ms; 8,192 along an
// edge of 160 x 120 3.0, 0.15 and 0.82 ms; 512 spread over 64 x 48 at n = 4 222, 35
// and 64 us.  Where neither happens: 8,192 in 64 x 64 inner pixels of 1024 x 436
// 110, 115 us.
template <int R>
__global__ __launch_bounds__(256) void k_cost_tail(ffh::CostArgs a, CostBins b, long long count) {
  constexpr int K = 2 * R + 1, T = 4;  // terms in flight
  __shared__ long long s_sum[4][4][5];  // of a wave's quads: four channels; terms and sums out of range
  __shared__ int s_last;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, k = lane & 3;
  const int W = a.W, Wm = W - 1, Hm = a.H - 1, groups = (int)gridDim.x;
  const int crowded = b.cursor[2] + b.cursor[3];  // side 0's, then side 1's
  for (int c = blockIdx.x; c < crowded; c += groups) {
    const int side = c >= b.cursor[2], p = b.rank[side][side ? c - b.cursor[2] : c], x = p % W, y = p / W;
    const float4 *fo = reinterpret_cast<const float4 *>(side ? a.f1 : a.f2) + k;
    const int4 *rec = b.rec[side];
    const float4 own = reinterpret_cast<const float4 *>(side ? a.f2 : a.f1)[(size_t)p * 4 + k];
    int first[K], at[K + 1];
    cost_terms<K>(b, side, a.n, x, y, first, at);
    const int total = at[K];
    CostFastSum fast;
    for (int i0 = threadIdx.x >> 2; i0 < total; i0 += 64 * T) {
      int4 r[T];
      float4 q[T];
#pragma unroll
      for (int j = 0; j < T; ++j) r[j] = rec[cost_record<K>(first, at, min(i0 + 64 * j, total - 1))];
#pragma unroll
      for (int j = 0; j < T; ++j) q[j] = fo[((size_t)clampi(y + r[j].y, Hm) * W + clampi(x + r[j].x, Wm)) * 4];
#pragma unroll
      for (int j = 0; j < T; ++j)
        if (i0 + 64 * j < total) fast.add(__int_as_float(r[j].z), own, q[j]);
    }
    fast.flush();
    CostSum &sum = fast.sum;
    sum.wave_sum();
    if (lane < 4) {
      for (int e = 0; e < 4; ++e) s_sum[wave][k][e] = sum.s[e];
      s_sum[wave][k][4] = (long long)sum.terms << 32 | sum.sums;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
      for (int w = 1; w < 4; ++w) {
        CostSum o;
        for (int e = 0; e < 4; ++e) o.s[e] = s_sum[w][k][e];
        o.terms = (unsigned)(s_sum[w][k][4] >> 32);
        o.sums = (unsigned)s_sum[w][k][4];
        sum.merge(o);
      }
      cost_write(a, side, (size_t)p * 4 + k, sum);
    }
    __syncthreads();  // the next pixel's sums
  }
  long long first = (long long)blockIdx.x * 256, step = (long long)groups * 256;
  if (crowded > 0) {
    if ((int)blockIdx.x >= crowded) return;
    if (threadIdx.x == 0) s_last = 0;
    __syncthreads();
    if (threadIdx.x < 4) {  // the threads that wrote
      __threadfence();
      if (threadIdx.x == 0) {
        s_last = atomicAdd(b.cursor + 4, 1) == min(groups, crowded) - 1;
        __threadfence();
      }
    }
    __syncthreads();
    if (!s_last) return;
    first = 0;
    step = 256;
  }
  if (__hip_atomic_load(a.overflow, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) return;
  for (long long i = first + threadIdx.x; i < count; i += step) {
    a.grad_f1[i] = __builtin_nanf("");
    a.grad_f2[i] = __builtin_nanf("");
  }
}

// Copy of a float feature map with the pixels of every row in phase order
// (desc_col): one thread per 16-byte quarter of an entry, so consecutive lanes
// store consecutive bytes.  All maps of a call in one launch: eight of
// 1024 x 436, a launch each 8 x 14.9 us, together 89 us, the rate of a copy.
__global__ __launch_bounds__(256) void k_phase_features(ffh::PhaseJobs jobs) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x, c = q >> 2, W = jobs.W;
  if (c >= W) return;
  const ffh::PhaseJob &jb = jobs.job[blockIdx.z];
  const float4 *f = reinterpret_cast<const float4 *>(jb.f);
  const size_t row = (size_t)blockIdx.y * W;
  reinterpret_cast<float4 *>(jb.out)[(row + c) * 4 + (q & 3)] =
      f[(row + ffk::desc_pixel(c, jb.log2n, W)) * 4 + (q & 3)];
}

}  // namespace

namespace ffh {

hipError_t launch_phase_features(const PhaseJobs &jobs, hipStream_t stream) {
  if (jobs.count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_phase_features, dim3((4 * jobs.W + 255) / 256, jobs.H, jobs.count), dim3(256), 0, stream, jobs);
  return hipGetLastError();
}

hipError_t launch_cost_fwd(const CostArgs &all, hipStream_t stream) {
  if (all.count <= 0) return hipSuccess;
  constexpr int kMost = 1 << 29;  // entries of a launch: four threads each, fewer than 2^32
  CostArgs a = all;
  if (all.count > kMost) {
    a.entries += kMost;
    a.cost += kMost;
    a.count -= kMost;
    const hipError_t e = launch_cost_fwd(a, stream);
    if (e != hipSuccess) return e;
    a = all;
    a.count = kMost;
  }
  const dim3 grid((unsigned)(((long long)a.count * 4 + 255) / 256));
  switch (a.radius) {
    case 0: hipLaunchKernelGGL(k_cost_fwd<0>, grid, dim3(256), 0, stream, a); break;
    case 1: hipLaunchKernelGGL(k_cost_fwd<1>, grid, dim3(256), 0, stream, a); break;
    case 2: hipLaunchKernelGGL(k_cost_fwd<2>, grid, dim3(256), 0, stream, a); break;
    case 3: hipLaunchKernelGGL(k_cost_fwd<3>, grid, dim3(256), 0, stream, a); break;
    case 4: hipLaunchKernelGGL(k_cost_fwd<4>, grid, dim3(256), 0, stream, a); break;
    case 5: hipLaunchKernelGGL(k_cost_fwd<5>, grid, dim3(256), 0, stream, a); break;
    case 6: hipLaunchKernelGGL(k_cost_fwd<6>, grid, dim3(256), 0, stream, a); break;
    case 7: hipLaunchKernelGGL(k_cost_fwd<7>, grid, dim3(256), 0, stream, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Places the bins in the accumulator scratch (2 * W * H * 16 words, whose
// last word, the overflow count, lies behind them); false if they do not fit.
static bool cost_bins(const CostArgs &a, CostBins *b, size_t *clear_words) {
  b->rn = a.radius * a.n;
  b->Wb = a.W + 2 * b->rn;
  b->Hb = a.H + 2 * b->rn;
  b->log2n = __builtin_ctz(a.n);
  const size_t bins = ((size_t)b->Hb * (b->Wb + 1) + 1) & ~(size_t)1, entries = ((size_t)a.count + 1) & ~(size_t)1;
  // records first (16-byte aligned), then the counts and the cursor, then the ranks
  const uintptr_t base = ((uintptr_t)a.acc1 + 15) & ~(uintptr_t)15;
  const size_t total = (base - (uintptr_t)a.acc1) + 2 * entries * 16 + (2 * bins + 6) * 4 + 2 * entries * 4;
  if (total > (size_t)2 * a.W * a.H * 16 * 8) return false;
  b->rec[0] = reinterpret_cast<int4 *>(base);
  b->rec[1] = b->rec[0] + entries;
  b->start[0] = reinterpret_cast<int32_t *>(b->rec[1] + entries);
  b->start[1] = b->start[0] + bins;
  b->cursor = b->start[1] + bins;
  b->rank[0] = b->cursor + 6;
  b->rank[1] = b->rank[0] + entries;
  *clear_words = bins + 3;
  return true;
}

template <int R>
static void launch_cost_sums(const CostArgs &a, const CostBins &b, hipStream_t stream) {
  const int tx = (a.W + 15) / 16;
  const int border_rows = (int)((cost_border_count(a.W, a.H) + 4ll * tx - 1) / (4ll * tx));
  hipLaunchKernelGGL(k_cost_gather<R>, dim3(tx, (a.H + 3) / 4 + border_rows, 2), dim3(256), 0, stream, a, b,
                     border_rows);
  hipLaunchKernelGGL(k_cost_tail<R>, dim3(kTailGroups), dim3(256), 0, stream, a, b, (long long)a.W * a.H * 16);
}

static hipError_t launch_cost_gather(const CostArgs &a, const CostBins &b, hipStream_t stream) {
  switch (a.radius) {
    case 0: launch_cost_sums<0>(a, b, stream); break;
    case 1: launch_cost_sums<1>(a, b, stream); break;
    case 2: launch_cost_sums<2>(a, b, stream); break;
    case 3: launch_cost_sums<3>(a, b, stream); break;
    case 4: launch_cost_sums<4>(a, b, stream); break;
    case 5: launch_cost_sums<5>(a, b, stream); break;
    case 6: launch_cost_sums<6>(a, b, stream); break;
    case 7: launch_cost_sums<7>(a, b, stream); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_cost_bwd(const CostArgs &a, hipStream_t stream) {
  const long long px = (long long)a.W * a.H * 16;
  // Gathering needs the bins to fit the scratch (they do unless the image is
  // tiny against the patch or holds more than about 6 entries per pixel), 16-byte loads of
  // the maps, and few phases: a corner pixel walks n (2 n radius + 1) ranges.
  // Radius 3, 160 x 120, atomics against gathering: 512 entries 57 and 74 us at n =
  // 8, 85 and 163 at n = 16; 1024 x 436 at n = 64 108 and 1006 us, and with 8,192
  // entries 875 and 2083 (at n = 8, many entries: 662 and 127).
  CostBins b;
  size_t clear = 0;
  const uintptr_t align = (uintptr_t)a.f1 | (uintptr_t)a.f2 | (uintptr_t)a.grad_f1 | (uintptr_t)a.grad_f2;
  if (a.n <= 4 && (align & 15) == 0 && cost_bins(a, &b, &clear)) {
    hipError_t e = launch_fill_u64(reinterpret_cast<uint64_t *>(b.start[0]), 0, (int64_t)clear, stream);
    if (e != hipSuccess) return e;
    const dim3 ge((unsigned)std::max(((long long)a.count + 255) / 256, 1ll), 2);
    hipLaunchKernelGGL(k_cost_count, ge, dim3(256), 0, stream, a, b);
    hipLaunchKernelGGL(k_cost_rows, dim3(b.Hb, 2), dim3(256), 0, stream, b);
    hipLaunchKernelGGL(k_cost_fill, ge, dim3(256), 0, stream, a, b);
    return launch_cost_gather(a, b, stream);
  }
  // acc1, acc2 and the overflow word after them are one array
  hipError_t e = launch_fill_u64(reinterpret_cast<uint64_t *>(a.acc1), 0, 2 * px + 1, stream);
  if (e != hipSuccess) return e;
  const int side = 2 * a.radius + 1;
  const long long work = (long long)a.count * side * side;
  if (work > 0)
    hipLaunchKernelGGL(k_cost_bwd, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, stream, a);
  const dim3 g((unsigned)((px + 255) / 256));
  hipLaunchKernelGGL(k_fixed_to_float, g, dim3(256), 0, stream, a.acc1, a.overflow, a.grad_f1, px);
  hipLaunchKernelGGL(k_fixed_to_float, g, dim3(256), 0, stream, a.acc2, a.overflow, a.grad_f2, px);
  return hipGetLastError();
}

}  // namespace ffh
