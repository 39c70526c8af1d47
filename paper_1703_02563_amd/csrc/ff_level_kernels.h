// Kernels and launchers of the temporally blocked level kernel; included by
// the per-scale translation units ff_level_s*.hip (each instantiates the
// kernels of one scale, so that they compile in parallel).
//
// Temporally blocked level kernel: a run of propagation steps (Eq. 2) and
// random-search steps (Sec. 3.1) of one scale in one launch (Sec. 3.2
// schedule), for patch radius 3.
//
// Each workgroup owns a TW x TH tile of the level grid and keeps the flow
// and cost of the tile plus a halo in LDS.  A half-sweep that reads sources
// on one side can only update correctly the cells whose source lies inside
// the currently valid window, so the valid window loses one cell on every
// side the half-sweep reads from.  The halo of a run equals the number of
// half-sweeps that read each side, so after the last step exactly the owned
// tile is valid and is written back.  Cells of the halo are computed
// redundantly by the neighbouring workgroups; evaluations are counted only
// for owned cells, so the count equals the unblocked schedule's.
//
// The scale-n descriptors of image a are staged in LDS on the level
// lattice (virtual cell (i+u, j+v) -> pixel clamp((i+u)n, (j+v)n)), which is
// exactly where E_n reads them.  Image b is read at p + f + n(u, v) with f
// per cell, straight from global memory.  The descriptor maps are padded
// with a replicated border of 3n pixels and their rows are in phase order,
// so every patch read is unclamped and contiguous at every scale.
//
// A half-sweep checks every cell's sources and queues the evaluations that
// can matter, evaluates the queue densely (one lane, or a quad of lanes, per
// evaluation) and then decodes each cell's best candidate; a random-search
// step evaluates one queued candidate per cell.
#pragma once

#include <algorithm>
#include <type_traits>

#include "ff_device.h"
#include "ff_internal.h"

namespace {

using ffk::clampi;
using ffk::kUnset;

constexpr int kR = 3;
constexpr int kHalo = ffh::kLevelHalo;

template <int TW, int TH, int HALO = kHalo, int RR = kR>
struct Geo {
  static constexpr int LW = TW + 2 * HALO, LH = TH + 2 * HALO;  // state window
  static constexpr int DW = LW + 2 * RR, DH = LH + 2 * RR;        // descriptor window (patch radius RR)
  static_assert(2 * LW * LH < 65536, "queue entries are 16-bit: cell * 2 + vertical");
};

// E_n(p, f) with image-a descriptors from LDS.  `pa` points at the LDS
// descriptor of the cell itself; (bx, by) = p + f in pixels, inside the
// image, so the whole patch lies in the padded map of image b: no clamps,
// and the samples of a patch row are consecutive stored columns (phase
// order) loaded with immediate offsets.  EV selects the load schedule:
// 0 rows one after another, 1 rows unrolled (the compiler interleaves),
// 2 all 49 loads issued before any arithmetic (needs ~200 registers); EV 3
// evaluates with a quad of lanes instead (eval_quad).
template <int LOG2N, int DW, int EV, int RR = kR>
__device__ __forceinline__ uint32_t eval_cell(const uint4 *pa, const uint4 *__restrict__ Db, int W, int bx, int by) {
  constexpr int n = 1 << LOG2N, P = ffk::kDescPad * n, K = 2 * RR + 1;
  const int Wp = W + 2 * P;
  uint32_t s = 0;
  const uint4 *pb = Db + ffk::desc_index(bx - RR * n, by - RR * n, LOG2N, W);
  if constexpr (EV == 2) {
    uint4 b[K * K];
#pragma unroll
    for (int v = 0; v < K; ++v)
#pragma unroll
      for (int u = 0; u < K; ++u) b[v * K + u] = pb[(size_t)v * n * Wp + u];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < K; ++v) {
      const uint4 *ra = pa + (v - RR) * DW - RR;
#pragma unroll
      for (int u = 0; u < K; ++u) s = ffk::sad16(ra[u], b[v * K + u], s);
    }
  } else {
#pragma unroll EV ? K : 1
    for (int v = 0; v < K; ++v) {
      const uint4 *ra = pa + (v - RR) * DW - RR;
#pragma unroll
      for (int u = 0; u < K; ++u) s = ffk::sad16(ra[u], pb[u], s);
      pb += (size_t)n * Wp;
    }
  }
  return s;
}

// E_n(p, f) evaluated by the four lanes of a quad (lanes 4k .. 4k+3 of a
// wave, all active): lane r takes patch columns u = r and u = r + 4 (none for
// r = 3) of all seven rows, so one load instruction of a quad covers four
// consecutive samples (64 contiguous bytes of a patch row) instead of one
// sample per lane spread over 64 patches.  Image b is read through a buffer
// resource over its padded map (the row offset rides in the scalar offset);
// the partial sums are added across the quad, every lane returns the total.
// Requires a map of less than 2^31 bytes.
// E_n(p, f) of a radius-4 patch (9 x 9) by a quad: lane r takes columns
// r, r + 4 and r + 8 (the last for lane 0 only), one column after another.
template <int LOG2N, int DW>
__device__ __forceinline__ uint32_t eval_quad9(const uint4 *pa, __amdgpu_buffer_rsrc_t db, int W, int bx, int by,
                                               int r) {
  constexpr int n = 1 << LOG2N, P = ffk::kDescPad * n, RR = 4, K = 2 * RR + 1;
  const int rowb = n * (W + 2 * P) * 16;
  const int off = (int)ffk::desc_index(bx - RR * n, by - RR * n, LOG2N, W) * 16;
  uint32_t s = 0;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int u = min(r + 4 * c, K - 1);
    uint4 b[K];
#pragma unroll
    for (int v = 0; v < K; ++v) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b128(db, off + u * 16, v * rowb, 0);
      b[v] = make_uint4(x[0], x[1], x[2], x[3]);
    }
    const uint4 *ra = pa - RR * DW - RR + u;
    uint32_t t = 0;
#pragma unroll
    for (int v = 0; v < K; ++v) t = ffk::sad16(ra[v * DW], b[v], t);
    s += (r + 4 * c < K) ? t : 0u;
  }
  s += (uint32_t)__builtin_amdgcn_mov_dpp((int)s, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
  s += (uint32_t)__builtin_amdgcn_mov_dpp((int)s, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  return s;
}

template <int LOG2N, int DW, int RR = kR>
__device__ __forceinline__ uint32_t eval_quad(const uint4 *pa, __amdgpu_buffer_rsrc_t db, int W, int bx, int by,
                                              int r) {
  if constexpr (RR == 4) {
    return eval_quad9<LOG2N, DW>(pa, db, W, bx, by, r);
  } else {
    constexpr int n = 1 << LOG2N, P = ffk::kDescPad * n, K = 2 * RR + 1;
    const int rowb = n * (W + 2 * P) * 16;
    const int u1 = r, u2 = min(r + 4, K - 1);
    const int off = (int)ffk::desc_index(bx - RR * n, by - RR * n, LOG2N, W) * 16;
    uint4 b1[K], b2[K], a1[K], a2[K];
#pragma unroll
    for (int v = 0; v < K; ++v) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b128(db, off + u1 * 16, v * rowb, 0);
      const auto y = __builtin_amdgcn_raw_buffer_load_b128(db, off + u2 * 16, v * rowb, 0);
      b1[v] = make_uint4(x[0], x[1], x[2], x[3]);
      b2[v] = make_uint4(y[0], y[1], y[2], y[3]);
    }
    // image a's samples from LDS while the global loads are in flight: the
    // first column's now, the second's once half of the first is summed (so
    // that fewer than 128 registers hold the whole evaluation)
    const uint4 *ra1 = pa - RR * DW - RR + u1, *ra2 = pa - RR * DW - RR + u2;
#pragma unroll
    for (int v = 0; v < K; ++v) a1[v] = ra1[v * DW];
    __builtin_amdgcn_sched_barrier(0);
    uint32_t s1 = 0, s2 = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) s1 = ffk::sad16(a1[v], b1[v], s1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 0; v < K; ++v) a2[v] = ra2[v * DW];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = 4; v < K; ++v) s1 = ffk::sad16(a1[v], b1[v], s1);
#pragma unroll
    for (int v = 0; v < K; ++v) s2 = ffk::sad16(a2[v], b2[v], s2);
    uint32_t s = s1 + (r < K - 4 ? s2 : 0u);
    s += (uint32_t)__builtin_amdgcn_mov_dpp((int)s, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
    s += (uint32_t)__builtin_amdgcn_mov_dpp((int)s, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
    return s;
}
}
// The same with image a's patch also read from its padded map (a quad per
// evaluation; the cells the weight-class evaluation does not cover).
template <int LOG2N, int RR = kR>
__device__ __forceinline__ uint32_t eval_quad_gg(__amdgpu_buffer_rsrc_t da, __amdgpu_buffer_rsrc_t db, int W, int ax,
                                                 int ay, int bx, int by, int r) {
  constexpr int n = 1 << LOG2N, P = ffk::kDescPad * n, K = 2 * RR + 1;
  const int rowb = n * (W + 2 * P) * 16;
  const int u1 = r, u2 = min(r + 4, K - 1);
  const int offa = (int)ffk::desc_index(ax - RR * n, ay - RR * n, LOG2N, W) * 16;
  const int offb = (int)ffk::desc_index(bx - RR * n, by - RR * n, LOG2N, W) * 16;
  uint32_t s1 = 0, s2 = 0;
#pragma unroll
  for (int v = 0; v < K; ++v) {
    const auto a1 = __builtin_amdgcn_raw_buffer_load_b128(da, offa + u1 * 16, v * rowb, 0);
    const auto a2 = __builtin_amdgcn_raw_buffer_load_b128(da, offa + u2 * 16, v * rowb, 0);
    const auto b1 = __builtin_amdgcn_raw_buffer_load_b128(db, offb + u1 * 16, v * rowb, 0);
    const auto b2 = __builtin_amdgcn_raw_buffer_load_b128(db, offb + u2 * 16, v * rowb, 0);
    s1 = ffk::sad16(make_uint4(a1[0], a1[1], a1[2], a1[3]), make_uint4(b1[0], b1[1], b1[2], b1[3]), s1);
    s2 = ffk::sad16(make_uint4(a2[0], a2[1], a2[2], a2[3]), make_uint4(b2[0], b2[1], b2[2], b2[3]), s2);
  }
  uint32_t s = s1 + (r < K - 4 ? s2 : 0u);
  if constexpr (K > 8) {  // radius 4: the ninth column, by lane 0
    if (r == 0) {
#pragma unroll
      for (int v = 0; v < K; ++v) {
        const auto a3 = __builtin_amdgcn_raw_buffer_load_b128(da, offa + 8 * 16, v * rowb, 0);
        const auto b3 = __builtin_amdgcn_raw_buffer_load_b128(db, offb + 8 * 16, v * rowb, 0);
        s = ffk::sad16(make_uint4(a3[0], a3[1], a3[2], a3[3]), make_uint4(b3[0], b3[1], b3[2], b3[3]), s);
      }
    }
  }
  s += (uint32_t)__builtin_amdgcn_mov_dpp((int)s, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
  s += (uint32_t)__builtin_amdgcn_mov_dpp((int)s, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  return s;
}

// E(p, f) at the patch scale m of a sub-scale stage (Sec. 3.3) by a quad,
// both images read from their image-order maps of scale m (border
// P = kDescPad * m, rows of W + 2P entries; a sample p + m (u, v) of a patch
// around an in-image pixel lies inside the border, so no clamping): lane r
// sums columns r and r + 4 of the 7 x 7 samples, the quad adds the lanes.
// Integer sums: the value is that of the per-step kernels' patch_cost.
template <int RR = kR>
__device__ __forceinline__ uint32_t eval_quad_sub(__amdgpu_buffer_rsrc_t da, __amdgpu_buffer_rsrc_t db, int W, int m,
                                                  int ax, int ay, int bx, int by, int r) {
  constexpr int K = 2 * RR + 1;
  const int P = ffk::desc_pad(m), Wp = W + 2 * P;
  const int rowb = m * Wp * 16, colb = m * 16;
  const int u1 = r, u2 = min(r + 4, K - 1);
  const int offa = ((ay - RR * m + P) * Wp + (ax - RR * m + P)) * 16;
  const int offb = ((by - RR * m + P) * Wp + (bx - RR * m + P)) * 16;
  uint32_t s1 = 0, s2 = 0;
#pragma unroll
  for (int v = 0; v < K; ++v) {
    const auto a1 = __builtin_amdgcn_raw_buffer_load_b128(da, offa + u1 * colb, v * rowb, 0);
    const auto a2 = __builtin_amdgcn_raw_buffer_load_b128(da, offa + u2 * colb, v * rowb, 0);
    const auto b1 = __builtin_amdgcn_raw_buffer_load_b128(db, offb + u1 * colb, v * rowb, 0);
    const auto b2 = __builtin_amdgcn_raw_buffer_load_b128(db, offb + u2 * colb, v * rowb, 0);
    s1 = ffk::sad16(make_uint4(a1[0], a1[1], a1[2], a1[3]), make_uint4(b1[0], b1[1], b1[2], b1[3]), s1);
    s2 = ffk::sad16(make_uint4(a2[0], a2[1], a2[2], a2[3]), make_uint4(b2[0], b2[1], b2[2], b2[3]), s2);
  }
  uint32_t s = s1 + (r < K - 4 ? s2 : 0u);
  s += (uint32_t)__builtin_amdgcn_mov_dpp((int)s, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
  s += (uint32_t)__builtin_amdgcn_mov_dpp((int)s, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  return s;
}

// The subpixel form of eval_quad_gg (radius 3): target (bx, by) in 1/8
// pixel, image b's descriptors mixed from the four pixels around it with
// integer weights (sad_bilinear4); a corner of weight 0 is read at its
// neighbour's column or row.
template <int LOG2N>
__device__ __forceinline__ uint32_t eval_quad_spx(__amdgpu_buffer_rsrc_t da, __amdgpu_buffer_rsrc_t db, int W, int ax,
                                                  int ay, int bx, int by, int r) {
  constexpr int n = 1 << LOG2N, P = ffk::kDescPad * n, K = 7;
  const int Wp = W + 2 * P, rowb = n * Wp * 16;
  const int x0 = bx >> 3, y0 = by >> 3, fx = bx & 7, fy = by & 7, dy = fy != 0 ? Wp * 16 : 0;
  const uint32_t w00 = (8 - fx) * (8 - fy), w10 = fx * (8 - fy), w01 = (8 - fx) * fy, w11 = fx * fy;
  const int offa = (int)ffk::desc_index(ax - 3 * n, ay - 3 * n, LOG2N, W) * 16;
  const int off0 = (int)ffk::desc_index(x0 - 3 * n, y0 - 3 * n, LOG2N, W) * 16;
  const int off1 = (int)ffk::desc_index(x0 + (fx != 0) - 3 * n, y0 - 3 * n, LOG2N, W) * 16;
  uint32_t s[2] = {0, 0};
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int u = 16 * (c == 0 ? r : min(r + 4, K - 1));
#pragma unroll
    for (int v = 0; v < K; ++v) {
      const auto a = __builtin_amdgcn_raw_buffer_load_b128(da, offa + u, v * rowb, 0);
      const auto b00 = __builtin_amdgcn_raw_buffer_load_b128(db, off0 + u, v * rowb, 0);
      const auto b10 = __builtin_amdgcn_raw_buffer_load_b128(db, off1 + u, v * rowb, 0);
      const auto b01 = __builtin_amdgcn_raw_buffer_load_b128(db, off0 + dy + u, v * rowb, 0);
      const auto b11 = __builtin_amdgcn_raw_buffer_load_b128(db, off1 + dy + u, v * rowb, 0);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        s[c] = ffk::sad_bilinear4(a[k], b00[k], b10[k], b01[k], b11[k], w00, w10, w01, w11, s[c]);
    }
  }
  uint32_t e = s[0] + (r < K - 4 ? s[1] : 0u);
  e += (uint32_t)__builtin_amdgcn_mov_dpp((int)e, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
  e += (uint32_t)__builtin_amdgcn_mov_dpp((int)e, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  return e;
}

// Sum of the class accumulators: T[l][k] collects rows of weight l + 1,
// dword k.
template <int RR>
__device__ __forceinline__ uint32_t wclass_sum(const uint32_t (&T)[4][4]) {
  using C = ffk::WClass<RR>;
  uint32_t e = 0;
#pragma unroll
  for (int l = 0; l < 4; ++l) {
    uint32_t r = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) r += (uint32_t)C::dword[k] * T[l][k];
    e += (uint32_t)(l + 1) * r;
  }
  return e;
}

// E_n(p, f) by one lane from the weight-class row maps of radius RR
// (wform_index, WClass), for a cell p and a target (bx, by) both at least RR n
// inside the image: the K = 2 RR + 7 rows y + n b of image a come from LDS
// (`pa`: the cell's entry of the first row, `step` entries between rows),
// those of image b from its map (one 16-byte load per row, the row step in
// the scalar offset); four byte SADs per row go to the accumulator of its
// (row weight, column weight) class, and E = sum_{l,k} l k T[l][k].  m: the
// patch scale (n, or a sub-scale stage's).
template <int RR>
__device__ __forceinline__ uint32_t eval_wform(const uint4 *pa, int step, __amdgpu_buffer_rsrc_t wb, int W, int m,
                                               int bx, int by) {
  using C = ffk::WClass<RR>;
  constexpr int K = C::K;
  const int rowb = m * W * 16;
  const int off = (int)ffk::wform_index(bx, by - (RR + 3) * m, m, W) * 16;
  uint4 B[K];
#pragma unroll
  for (int b = 0; b < K; ++b) {
    const auto x = __builtin_amdgcn_raw_buffer_load_b128(wb, off, b * rowb, 0);
    B[b] = make_uint4(x[0], x[1], x[2], x[3]);
  }
  uint32_t T[4][4] = {};
#pragma unroll
  for (int b = 0; b < K; ++b) {
    const uint4 A = pa[b * step];
    const int l = C::row[b] - 1;
    T[l][0] = __builtin_amdgcn_sad_u8(A.x, B[b].x, T[l][0]);
    T[l][1] = __builtin_amdgcn_sad_u8(A.y, B[b].y, T[l][1]);
    T[l][2] = __builtin_amdgcn_sad_u8(A.z, B[b].z, T[l][2]);
    T[l][3] = __builtin_amdgcn_sad_u8(A.w, B[b].w, T[l][3]);
  }
  return wclass_sum<RR>(T);
}

// The subpixel form (radius 3): target (bx, by) in 1/8 pixel, both of its
// pixel columns and rows at least 3n inside.  A bilinear mix of descriptors is
// the descriptor of the mixed image, so the classes stay: E = sum of w(b) k
// |64 a - mix| over the 13 x 13 samples, four row entries per row instead of
// the 4 x 49 descriptors of the direct form (about 77 operations per row
// against 88 per descriptor).  An evaluation is some thousand operations: FL
// = 4 lets a quad share its rows where the tile's workgroup has lanes to spare
// and one lane's chain would be a phase's critical path (1024 x 436, per
// launch at scale 16: 117 -> 70 us, scale 4: 144 -> 113 us); on the 256-thread
// tiles of the fine scales one lane per evaluation does less work in all
// (scale 1: 232 against 318 us).  At n = 1 the lower corners of a row are the
// upper ones of the next, so a quad's lanes take adjacent rows there, else
// every fourth.
template <int LOG2N, int FL>
__device__ __forceinline__ uint32_t eval_wform_spx(const uint4 *pa, int step, __amdgpu_buffer_rsrc_t wb, int W, int bx,
                                                   int by, int r) {
  constexpr int n = 1 << LOG2N, K = 13, ROWS = FL == 4 ? 4 : K;  // rows per lane
  const int rowb = n * W * 16;
  const int fx = bx & 7, fy = by & 7, dx = fx != 0 ? 16 : 0, dy = fy != 0 ? W * 16 : 0;
  const int off = (int)ffk::wform_index(bx >> 3, (by >> 3) - 6 * n, n, W) * 16;
  // row i of this lane, and its weight w(b) = (8 - |b - 6|) / 2 (0 past the
  // lane's last row)
  auto row_of = [&](int i) { return FL == 1 ? i : LOG2N == 0 ? min((r == 0 ? 0 : 3 * r + 1) + i, 12) : min(r + 4 * i, 12); };
  auto weight = [&](int i) {
    const bool there = FL == 1 || i < 3 || r == 0;
    return there ? (uint32_t)(8 - abs(row_of(i) - 6)) >> 1 : 0u;
  };
  // The mixed entry in even and odd 16-bit lanes: dword k holds samples of
  // weight k + 1, the last one a single sample in its even lanes.
  uint32_t e = 0;
  auto add = [&](int i, const uint32_t (&mix)[7]) {
    const uint4 A = pa[row_of(i) * step];
    const uint32_t w[4] = {A.x, A.y, A.z, A.w};
    uint32_t s[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      s[k] = __builtin_amdgcn_sad_u16(ffk::even_bytes(w[k]) << 6, mix[2 * k], 0);
      if (k < 3) s[k] = __builtin_amdgcn_sad_u16(ffk::odd_bytes(w[k]) << 6, mix[2 * k + 1], s[k]);
    }
    e = ffk::mad24(s[0] + 2 * s[1] + 3 * s[2] + 4 * s[3], weight(i), e);
  };
  auto lanes = [](const auto &v, int k) {
    return (k & 1) ? ffk::odd_bytes(v[k >> 1]) : ffk::even_bytes(v[k >> 1]);
  };
  auto load = [&](int row, int o) {
    if constexpr (FL == 1)
      return __builtin_amdgcn_raw_buffer_load_b128(wb, off + o, row * rowb, 0);
    else
      return __builtin_amdgcn_raw_buffer_load_b128(wb, off + row * rowb + o, 0, 0);
  };
  if constexpr (LOG2N == 0) {
    const uint32_t wx0 = 8 - fx, wx1 = fx, wy0 = (8 - fy) * 0x10001u, wy1 = fy * 0x10001u;
    auto hmix = [&](int row, uint32_t (&h)[7]) {
      const auto p = load(row, 0);
      const auto q = load(row, dx);
#pragma unroll
      for (int k = 0; k < 7; ++k) h[k] = ffk::mad24(lanes(q, k), wx1, __umul24(lanes(p, k), wx0));
    };
    uint32_t h0[7], h1[7], mix[7];
    hmix(row_of(0), h0);
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      hmix(row_of(i) + 1, h1);  // (past the target's own rows only with weight 0)
#pragma unroll
      for (int k = 0; k < 7; ++k) {
        mix[k] = ffk::mix16(h0[k], wy0, h1[k], wy1);  // at most 8 * 2040 a lane
        h0[k] = h1[k];
      }
      add(i, mix);
    }
  } else {
    const uint32_t w00 = (8 - fx) * (8 - fy), w10 = fx * (8 - fy), w01 = (8 - fx) * fy, w11 = fx * fy;
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int b = row_of(i);
      const auto p = load(b, 0), q = load(b, dx), t = load(b, dy), u = load(b, dx + dy);
      uint32_t mix[7];
#pragma unroll
      for (int k = 0; k < 7; ++k)
        mix[k] = ffk::mad24(lanes(u, k), w11,
                            ffk::mad24(lanes(t, k), w01, ffk::mad24(lanes(q, k), w10, __umul24(lanes(p, k), w00))));
      add(i, mix);
    }
  }
  if constexpr (FL == 4) {
    e += (uint32_t)__builtin_amdgcn_mov_dpp((int)e, 0xB1, 0xF, 0xF, false);  // quad_perm [1,0,3,2]
    e += (uint32_t)__builtin_amdgcn_mov_dpp((int)e, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  }
  return e;
}

// Float learned-feature cost (Eq. 3 with the squared-difference data term)
// by a quad of lanes: lane r owns channels 4r .. 4r+3 and sums their terms
// with one fused multiply-add each in the order v, u, c; the quad then adds
// the four partial sums as (s0 + s1) + (s2 + s3) (every lane returns the
// total, as a bit pattern).  Image a's lattice samples come from LDS (`pa`:
// the cell's 4 float4 in a window of row length DW cells), image b's from
// its feature map, [H][W][16] with the pixels of a row in phase order
// (desc_col; at n = 1 image order), positions clamped: a quad reads one whole
// 64-byte entry per load, the samples of a patch row next to each other.
//
// Bound by those reads (49 entries of 64 bytes per evaluation through the
// vector L1), so they stop once the value cannot be used: `limit` holds the
// bits of the cost an evaluation has to stay at or below, terms are not
// negative and rounding keeps the order, so a partial sum above it decides.
// The wave leaves together, after the row that puts its last quad above; the
// value returned is then some number above the limit.  A row's loads are
// issued before the previous row is summed.  Infinities and NaN never decide.
//
// Targets 3n inside the image (a wave of them takes eval_quad_f32_rows with
// kInside) need one address per patch row: the samples of a row are adjacent
// and the rows n image rows apart.  Clamping and addressing every sample
// doubles the vector instructions (16 a sample instead of 8): 142 -> 139 us a
// launch at 1024x436, n = 1, and 68 -> 64 us at n = 2.
template <int LOG2N, int DW, bool kInside>
__device__ __forceinline__ uint32_t eval_quad_f32_rows(const float4 *pa, const float4 *__restrict__ B, int W, int H,
                                                       int bx, int by, int r, uint32_t limit) {
  constexpr int n = 1 << LOG2N, K = 2 * kR + 1;
  const float4 *ra = pa + (-kR * DW - kR) * 4 + r;
  int xo[K];
  const float4 *next = B;
  if constexpr (kInside) {
    next += ((size_t)(by - kR * n) * W + ffk::desc_col(bx - kR * n, LOG2N, W)) * 4 + r;
  } else {
#pragma unroll
    for (int u = 0; u < K; ++u) xo[u] = 4 * ffk::desc_col(clampi(bx + (u - kR) * n, W - 1), LOG2N, W) + r;
  }
  constexpr int D = 3;  // rows in flight, the summed one included
  float4 y[D][K];
  auto fetch = [&](int v, float4 (&row)[K]) {  // rows in turn
    if constexpr (kInside) {
#pragma unroll
      for (int u = 0; u < K; ++u) row[u] = next[4 * u];
      next += (size_t)n * W * 4;
    } else {
      const float4 *p = B + (size_t)clampi(by + (v - kR) * n, H - 1) * W * 4;
#pragma unroll
      for (int u = 0; u < K; ++u) row[u] = p[xo[u]];
    }
  };
  auto total = [](float s) {
    s += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(s), 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
    s += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(s), 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
    return s;
  };
  const float lim = __uint_as_float(limit);
  float s = 0.0f;
#pragma unroll
  for (int v = 0; v + 1 < D; ++v) fetch(v, y[v]);
#pragma unroll
  for (int v = 0; v < K; ++v) {
    if (v + D - 1 < K) fetch(v + D - 1, y[(v + D - 1) % D]);
#pragma unroll
    for (int u = 0; u < K; ++u) {
      const float4 x = ra[(v * DW + u) * 4], z = y[v % D][u];
      float e = x.x - z.x;
      s = __fmaf_rn(e, e, s);
      e = x.y - z.y;
      s = __fmaf_rn(e, e, s);
      e = x.z - z.z;
      s = __fmaf_rn(e, e, s);
      e = x.w - z.w;
      s = __fmaf_rn(e, e, s);
    }
    if (LOG2N <= 2 && v + D < K) {
      const float t = total(s);
      if (!__ballot(!(t > lim && t < __builtin_inff()))) return __float_as_uint(t);
    }
  }
  return __float_as_uint(total(s));
}

template <int LOG2N, int DW>
__device__ __forceinline__ uint32_t eval_quad_f32(const float4 *pa, const float4 *__restrict__ B, int W, int H, int bx,
                                                  int by, int r, uint32_t limit) {
  constexpr int m = kR << LOG2N;
  if (!__ballot(bx < m || bx >= W - m || by < m || by >= H - m))
    return eval_quad_f32_rows<LOG2N, DW, true>(pa, B, W, H, bx, by, r, limit);
  return eval_quad_f32_rows<LOG2N, DW, false>(pa, B, W, H, bx, by, r, limit);
}

// The run of passes for tile `tile` of one direction `d` (a holds the
// pair's sizes and the schedule).  All threads of the workgroup call it.
template <int LOG2N, int TW, int TH, int kThreads, int EV, bool F32 = false, int HALO = kHalo, int RR = kR,
          bool SUB = false, bool SPX = false>
__device__ __forceinline__ void level_body(const ffh::LevelKArgs &a, const ffh::LevelKDir &d, int tile) {
  // SUB: a sub-scale stage (patch scale a.sub_m = 3n/2, maps of that scale);
  // SPX: flows in 1/8 pixel, bilinear targets
  static_assert((!SUB && !SPX) || (EV == 4 && !F32 && RR == kR && !(SUB && SPX) && !(SUB && LOG2N == 0)),
                "sub-scale and subpixel stages run the radius-3 weight-class kernels");
  // patch radius RR: 3, or 2 and 4 with the descriptor-quad or weight-class
  // evaluations (the float path holds radius-3 patches)
  static_assert(Geo<TW, TH, HALO, RR>::LW * Geo<TW, TH, HALO, RR>::LH + kThreads < 65536,
                "the cell index of a half-sweep must stay below 2^16 (cell_of's division)");
  static_assert(RR == kR || ((RR == 2 || RR == 4) && EV >= 3 && !F32),
                "radii 2 and 4 run the descriptor-quad and weight-class kernels only");
  constexpr int SB = SPX ? 3 : 0;  // flows in 1/2^SB pixel
  constexpr int FL = SPX && kThreads > 256 ? 4 : 1;  // lanes per weight-class evaluation
  using G = Geo<TW, TH, HALO, RR>;
  constexpr int n = 1 << LOG2N;
  // EV 3 and float features: every evaluation by a quad of lanes
  // (eval_quad, eval_quad_f32); the candidate flows of a random-search step
  // are then parked in s_flags.  EV 4: evaluations whose cell and target lie
  // 3n inside the image by one lane each on the weight-class row maps
  // (eval_wform, image a's rows staged in LDS), the others by a quad
  // reading both descriptor maps (eval_quad_gg); such queues fill from the
  // front (weight-class) and from the back (descriptor quads).
  constexpr bool WF = EV == 4;
  constexpr bool QUAD = EV == 3 || F32 || WF;
  constexpr int QCAP = G::LH * G::LW + G::LH;
  constexpr int kQuads = kThreads / 4;
  using FlagT = std::conditional_t<QUAD, uint32_t, uint8_t>;
  __shared__ int32_t s_flow[G::LH * G::LW];
  __shared__ uint32_t s_cost[G::LH * G::LW];
  // byte descriptors of image a on the level lattice; 64-bit keys for float
  // costs
  __shared__ uint4 s_da[(F32 || WF) ? 1 : G::DH * G::DW];
  // weight-class row entries of image a: window rows gj0 - (RR + 3) ... gj0 +
  // LH + RR + 2; the rows of a sub-scale patch lie 3/2 cells apart, so its
  // window holds rows half a cell apart from gj0 - 9 on (patch row b of cell
  // row j is window row 2 (j - gj0) + 3 (b + 6))
  constexpr int WROWS = SUB ? 2 * G::LH + 35 : G::LH + 2 * (RR + 3);
  __shared__ uint4 s_wa[WF ? WROWS * G::LW : 1];
  __shared__ float4 s_daf[F32 ? 4 * G::DH * G::DW : 1];
  __shared__ unsigned long long s_key[F32 ? G::LH * G::LW : 1];
  __shared__ uint16_t s_queue[QCAP];  // queued evaluations: cell * 2 + vertical
  // candidate flags of the current half-sweep; with quads also the parked
  // random-search candidate flows
  __shared__ FlagT s_flags[G::LH * G::LW];
  __shared__ unsigned int s_cnt, s_qlen, s_rlen, s_blen, s_rblen;
  __shared__ unsigned int s_work[2];  // evaluations computed: owned cells, all cells

  const int tid = threadIdx.x, qr = tid & 3;
  const int W = a.W, H = a.H, Wn = a.Wn, Hn = a.Hn;
  const int ti0 = (tile % a.tiles_x) * TW, tj0 = (tile / a.tiles_x) * TH;
  const int oi1 = min(ti0 + TW, Wn), oj1 = min(tj0 + TH, Hn);
  const int gi0 = ti0 - HALO, gj0 = tj0 - HALO;  // grid coords of window cell (0, 0)
  auto owned = [&](int i, int j) { return i >= ti0 && i < oi1 && j >= tj0 && j < oj1; };
  const uint4 *Db = reinterpret_cast<const uint4 *>(d.Db);
  if (tid == 0) {
    s_cnt = 0;
    s_qlen = 0;
    s_rlen = 0;
    s_blen = 0;
    s_rblen = 0;
    s_work[0] = 0;
    s_work[1] = 0;
  }

  // image-a descriptors on the level lattice around the window: every load
  // of a thread is issued before the first LDS store (one memory round trip)
  constexpr int NSTAGE = F32 ? 4 * G::DH * G::DW : (WF ? WROWS * G::LW : G::DH * G::DW);
  constexpr int NS = (NSTAGE + kThreads - 1) / kThreads;
  uint4 sv[F32 ? 1 : NS];
  float4 sf[F32 ? NS : 1];
  if constexpr (WF) {
    const uint4 *Wa = reinterpret_cast<const uint4 *>(d.Wa);
#pragma unroll
    for (int it = 0; it < NS; ++it) {
      const int k = min(it * kThreads + tid, NSTAGE - 1);
      const int vi = gi0 + k % G::LW, vr = k / G::LW;
      const int y = SUB ? gj0 * n + (vr - 18) * (n / 2) : (gj0 - (RR + 3) + vr) * n;
      // rows of a patch reach 3 of its scale past the image (kWformPad); the
      // windows of cells without weight-class evaluations are clamped to that
      const int sc = SUB ? a.sub_m : n;
      sv[it] = Wa[ffk::wform_index(clampi(vi * n, W - 1), min(max(y, -3 * sc), H - 1 + 3 * sc), sc, W)];
    }
  } else if constexpr (!F32) {
    const uint4 *Da = reinterpret_cast<const uint4 *>(d.Da);
    uint4 *v = sv;
#pragma unroll
    for (int it = 0; it < NS; ++it) {
      const int k = min(it * kThreads + tid, G::DH * G::DW - 1);
      const int vi = gi0 - RR + k % G::DW, vj = gj0 - RR + k / G::DW;
      v[it] = Da[ffk::desc_index(clampi(vi * n, W - 1), clampi(vj * n, H - 1), LOG2N, W)];
    }
  } else {
    const float4 *Da = reinterpret_cast<const float4 *>(d.Da);
    float4 *v = sf;
#pragma unroll
    for (int it = 0; it < NS; ++it) {
      const int k = min(it * kThreads + tid, 4 * G::DH * G::DW - 1);
      const int c = k >> 2, vi = gi0 - RR + c % G::DW, vj = gj0 - RR + c / G::DW;
      v[it] = Da[4 * ((size_t)clampi(vj * n, H - 1) * W + ffk::desc_col(clampi(vi * n, W - 1), LOG2N, W)) + (k & 3)];
    }
  }
  const int pscale = SUB ? a.sub_m : n;  // patch scale
  // E_n of grid cell (i, j) and target pixel (bx, by), one lane per
  // evaluation (byte descriptors, EV 0-2)
  auto evalc = [&](int i, int j, int bx, int by) -> uint32_t {
    const uint4 *pa = s_da + (j - gj0 + RR) * G::DW + (i - gi0 + RR);
    return eval_cell<LOG2N, G::DW, (EV < 3 ? EV : 1), RR>(pa, Db, W, bx, by);
  };
  // the same by a quad of lanes (QUAD only)
  [[maybe_unused]] const int map_bytes =
      (int)((size_t)(H + 2 * ffk::desc_pad(pscale)) * (W + 2 * ffk::desc_pad(pscale)) * 16);
  [[maybe_unused]] const __amdgpu_buffer_rsrc_t db_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(d.Db), (short)0, map_bytes, 0x00020000);
  auto evalq = [&](int i, int j, int bx, int by, [[maybe_unused]] uint32_t limit) -> uint32_t {
    if constexpr (F32) {
      const float4 *pa = s_daf + 4 * ((j - gj0 + RR) * G::DW + (i - gi0 + RR));
      return eval_quad_f32<LOG2N, G::DW>(pa, reinterpret_cast<const float4 *>(d.Db), W, H, bx, by, qr, limit);
    } else {
      const uint4 *pa = s_da + (j - gj0 + RR) * G::DW + (i - gi0 + RR);
      return eval_quad<LOG2N, G::DW, RR>(pa, db_rsrc, W, bx, by, qr);
    }
  };
  // evaluations computed (the work counters; a no-op without them), called
  // by every lane of a wave
  auto count_work = [&](bool did, bool own) {
    if (d.n_work == nullptr) return;
    const int all = __popcll(__ballot(did)), mine = __popcll(__ballot(did && own));
    if ((tid & 63) == 0 && all) {
      atomicAdd(&s_work[0], (unsigned)mine);
      atomicAdd(&s_work[1], (unsigned)all);
    }
  };
  // the weight-class path: interior test, one-lane and all-global quad
  // evaluations; (bx, by): target in 1/2^SB pixel
  [[maybe_unused]] const __amdgpu_buffer_rsrc_t wb_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t *>(d.Wb), (short)0, WF ? (int)ffk::wform_bytes(W, H, pscale) : 0, 0x00020000);
  [[maybe_unused]] const __amdgpu_buffer_rsrc_t da_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(d.Da), (short)0, WF ? map_bytes : 0, 0x00020000);
  [[maybe_unused]] auto inner = [&](int i, int j, int bx, int by) {
    const int lo = RR * pscale, xh = (W - 1 - lo) << SB, yh = (H - 1 - lo) << SB;
    return i * n >= lo && i * n <= W - 1 - lo && j * n >= lo && j * n <= H - 1 - lo && bx >= (lo << SB) && bx <= xh &&
           by >= (lo << SB) && by <= yh;
  };
  [[maybe_unused]] auto evalw = [&](int i, int j, int bx, int by) -> uint32_t {
    if constexpr (SPX)
      return eval_wform_spx<LOG2N, FL>(s_wa + (j - gj0) * G::LW + (i - gi0), G::LW, wb_rsrc, W, bx, by, qr);
    else
      return eval_wform<RR>(s_wa + (SUB ? 2 : 1) * (j - gj0) * G::LW + (i - gi0), (SUB ? 3 : 1) * G::LW, wb_rsrc, W,
                            pscale, bx, by);
  };
  [[maybe_unused]] auto evalg = [&](int i, int j, int bx, int by) -> uint32_t {
    if constexpr (SUB)
      return eval_quad_sub<RR>(da_rsrc, db_rsrc, W, pscale, i * n, j * n, bx, by, qr);
    else if constexpr (SPX)
      return eval_quad_spx<LOG2N>(da_rsrc, db_rsrc, W, i * n, j * n, bx, by, qr);
    else
      return eval_quad_gg<LOG2N, RR>(da_rsrc, db_rsrc, W, i * n, j * n, bx, by, qr);
  };
  // append of the lanes with `on` set, at the front (inn) or the back (!inn)
  // of the queue: one LDS atomic per wave and end
  [[maybe_unused]] auto enqueue2 = [&](bool on, bool inn, uint16_t e, unsigned int &flen, unsigned int &blen) {
    const uint64_t bi = __ballot(on && inn), bb = __ballot(on && !inn);
    int q0 = 0, q1 = 0;
    if ((tid & 63) == 0) {
      if (bi) q0 = (int)atomicAdd(&flen, (unsigned)__popcll(bi));
      if (bb) q1 = (int)atomicAdd(&blen, (unsigned)__popcll(bb));
    }
    q0 = __shfl(q0, 0);
    q1 = __shfl(q1, 0);
    const int lane = tid & 63;
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    if (on && inn) s_queue[q0 + __popcll(bi & below)] = e;
    if (on && !inn) s_queue[QCAP - 1 - (q1 + __popcll(bb & below))] = e;
  };
  // evaluations of a front/back queue pair in one sequence over the threads:
  // the front entries one lane each (weight-class; a quad each for subpixel
  // flows) in whole waves, then the back entries a quad each, so that both
  // kinds run side by side on different waves.  decode(e, l, i, j, bx, by)
  // gives an entry's window cell l, grid cell (i, j) and target; done(e, l,
  // cost) is called once per entry, on the evaluating lane (a quad's lane 0)
  [[maybe_unused]] auto run_queues = [&](int flen, int blen, auto decode, auto done) {
    const int fthreads = (flen * FL + 63) & ~63, total = fthreads + 4 * blen;
    for (int base = 0; base < total; base += kThreads) {
      const int q = base + tid;
      bool own = false, did = false;
      if (q < fthreads) {  // wave-uniform
        if (q < flen * FL) {
          const int e = s_queue[q / FL];
          int l, i, j, bx, by;
          decode(e, l, i, j, bx, by);
          const uint32_t c = evalw(i, j, bx, by);
          did = q % FL == 0;
          if (did) done(e, l, c);
          own = owned(i, j);
        }
      } else if (q < total) {
        const int e = s_queue[QCAP - 1 - ((q - fthreads) >> 2)];
        int l, i, j, bx, by;
        decode(e, l, i, j, bx, by);
        const uint32_t c = evalg(i, j, bx, by);
        did = qr == 0;
        if (did) done(e, l, c);
        own = owned(i, j);
      }
      count_work(did, own);
    }
  };
  // queue append of the lanes with `on` set (one LDS atomic per wave)
  auto enqueue = [&](bool on, uint16_t e, unsigned int &len) {
    const uint64_t b = __ballot(on);
    int q0 = 0;
    if ((tid & 63) == 0 && b) q0 = (int)atomicAdd(&len, (unsigned)__popcll(b));
    q0 = __shfl(q0, 0);
    const int lane = tid & 63;
    if (on) s_queue[q0 + __popcll(b & (lane ? (~0ull >> (64 - lane)) : 0ull))] = e;
  };

  int ml = a.halo[0], mr = a.halo[1], mt = a.halo[2], mb = a.halo[3];
  // a random search follows step t unless t ends its group (the R^+ steps
  // of Flow Fields+ end at P - 1, the scale at T - 1)
  auto rs_after = [&](int t) { return t != a.P - 1 && t != a.T - 1; };
  // random-search candidate of cell (i, j) at step t from its current state
  // (branch-free, so that two draws in one block can interleave)
  [[maybe_unused]] auto rs_candidate = [&](int i, int j, int l, int t, int32_t &fc) {
    const uint32_t c0 = s_cost[l];
    const int32_t f0 = s_flow[l];
    int ox, oy;
    ffk::rs_offset(a.seed, d.stream_id, a.level, t, j, i, (t < a.P ? a.Rnp : a.Rn) << SB, ox, oy);
    const int fx = ffk::flow_x(f0) + ox, fy = ffk::flow_y(f0) + oy;
    fc = ffk::pack_flow(fx, fy);
    return c0 != kUnset && (ox | oy) != 0 && ffk::target_in<SB>(W, H, i * n, j * n, fx, fy);
  };

  // initial state of the valid window: the state of every cell of a thread
  // is loaded first, then stored, evaluated (one lane per evaluation) or
  // queued (quads)
  {
    const int rl = max(ti0 - ml, 0), rr = min(oi1 + mr, Wn), rt = max(tj0 - mt, 0), rb = min(oj1 + mb, Hn);
    const int rw = rr - rl, rh = rb - rt;
    const int Wc = (Wn + 1) >> 1;
    constexpr int NI = (G::LH * G::LW + kThreads - 1) / kThreads;
    int32_t fv[NI];
    uint32_t cv[NI];
    bool ev[NI];
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int k = it * kThreads + tid;
      fv[it] = 0;
      cv[it] = kUnset;
      ev[it] = false;
      if (k < rw * rh) {
        const int i = rl + k % rw, j = rt + k / rw;
        if (a.mode == ffh::kLevelContinue) {
          fv[it] = d.flow_in[(size_t)j * Wn + i];
          cv[it] = d.cost_in[(size_t)j * Wn + i];
        } else if (a.mode == ffh::kLevelInit) {
          const uint32_t q = (uint32_t)d.nn_key[(size_t)j * Wn + i];
          fv[it] = ffk::pack_flow(((int)(q % (uint32_t)W) - i * n) * (1 << SB),
                                  ((int)(q / (uint32_t)W) - j * n) * (1 << SB));
          ev[it] = true;
        } else if (!((i | j) & 1)) {
          const int kc = (j >> 1) * Wc + (i >> 1);
          const uint32_t cc = d.ccost[kc];
          const int32_t cf = d.cflow[kc];
          if (cc != kUnset) {
            fv[it] = cf;
            ev[it] = true;
          }
        }
      }
    }
    // the staged descriptors go to LDS once both groups of loads are issued
    if constexpr (WF) {
#pragma unroll
      for (int it = 0; it < NS; ++it)
        if (it * kThreads + tid < NSTAGE) s_wa[it * kThreads + tid] = sv[it];
    } else if constexpr (!F32) {
#pragma unroll
      for (int it = 0; it < NS; ++it)
        if (it * kThreads + tid < G::DH * G::DW) s_da[it * kThreads + tid] = sv[it];
    } else {
#pragma unroll
      for (int it = 0; it < NS; ++it)
        if (it * kThreads + tid < 4 * G::DH * G::DW) s_daf[it * kThreads + tid] = sf[it];
    }
    // one-lane seed evaluations read the staged descriptors, and queueing
    // needs the counters cleared: a barrier, except for a continuing run of
    // the quad kernels, which neither evaluates nor queues here
    if (!QUAD || a.mode != ffh::kLevelContinue) __syncthreads();
#pragma unroll
    for (int it = 0; it < NI; ++it) {
      const int k = it * kThreads + tid;
      int cnt = 0, l = 0;
      bool inn = false;
      if (k < rw * rh) {
        const int i = rl + k % rw, j = rt + k / rw;
        l = (j - gj0) * G::LW + (i - gi0);
        s_flow[l] = fv[it];
        s_cost[l] = cv[it];
        if (ev[it]) {
          if constexpr (!QUAD) s_cost[l] = evalc(i, j, i * n + ffk::flow_x(fv[it]), j * n + ffk::flow_y(fv[it]));
          if constexpr (WF) inn = inner(i, j, ((i * n) << SB) + ffk::flow_x(fv[it]), ((j * n) << SB) + ffk::flow_y(fv[it]));
          cnt = owned(i, j);
        }
      }
      if constexpr (!QUAD) count_work(k < rw * rh && ev[it], cnt != 0);
      if constexpr (WF)
        enqueue2(k < rw * rh && ev[it], inn, (uint16_t)l, s_qlen, s_blen);
      else if constexpr (QUAD)
        enqueue(k < rw * rh && ev[it], (uint16_t)l, s_qlen);
      const int tot = __popcll(__ballot(cnt));
      if ((tid & 63) == 0 && tot) atomicAdd(&s_cnt, (unsigned)tot);
    }
  }
  __syncthreads();
  if constexpr (WF) {
    if (a.mode != ffh::kLevelContinue) {  // the seed evaluations
      run_queues(
          (int)s_qlen, (int)s_blen,
          [&](int e, int &l, int &i, int &j, int &bx, int &by) {
            l = e;
            i = gi0 + l % G::LW;
            j = gj0 + l / G::LW;
            const int32_t f = s_flow[l];
            bx = ((i * n) << SB) + ffk::flow_x(f);
            by = ((j * n) << SB) + ffk::flow_y(f);
          },
          [&](int, int l, uint32_t c) { s_cost[l] = c; });
      __syncthreads();
      if (tid == 0) s_qlen = s_blen = 0;
      __syncthreads();
    }
  } else if constexpr (QUAD) {
    if (a.mode != ffh::kLevelContinue) {  // the seed evaluations, a quad each
      const int qlen = (int)s_qlen;
      for (int base = 0; base < qlen; base += kQuads) {
        const int q = base + (tid >> 2);
        bool own = false;
        if (q < qlen) {
          const int l = s_queue[q], i = gi0 + l % G::LW, j = gj0 + l / G::LW;
          const int32_t f = s_flow[l];
          const uint32_t c = evalq(i, j, i * n + ffk::flow_x(f), j * n + ffk::flow_y(f), kUnset);
          if (qr == 0) s_cost[l] = c;
          own = owned(i, j);
        }
        count_work(q < qlen && qr == 0, own);
      }
      __syncthreads();
      if (tid == 0) s_qlen = 0;
      __syncthreads();
    }
  }

  for (int t = a.t_begin; t < a.t_end; ++t) {
    const int dir = t & 3;
    const int hdi = (dir == 0 || dir == 3) ? -1 : 1;
    const int vdj = (dir == 0 || dir == 2) ? -1 : 1;
    for (int colour = 1; colour >= 0; --colour) {
      if (hdi < 0) --ml; else --mr;
      if (vdj < 0) --mt; else --mb;
      const int rl = max(ti0 - ml, 0), rr = min(oi1 + mr, Wn), rt = max(tj0 - mt, 0), rb = min(oj1 + mb, Hn);
      const int hw = (rr - rl + 1) >> 1, rh = rb - rt;
      // k / hw as a multiply-high by ceil(2^32 / hw): exact for k, hw < 2^16
      // (the error term k (m - 2^32 / hw) / 2^32 stays below 1 / hw)
      const uint32_t hwm = hw > 1 ? 0xFFFFFFFFu / (uint32_t)hw + 1u : 0u;
      // Cells of this colour in the valid window, thread-strided.
      auto cell_of = [&](int c, int k, int &i, int &j) {
        const int q = hw > 1 ? (int)__umulhi((uint32_t)k, hwm) : k;
        j = rt + (k < hw * rh ? q : 0);
        i = rl + ((c + j + rl) & 1) + 2 * (hw > 1 ? k - q * hw : 0);
        return k < hw * rh && i < rr;
      };
      auto cell = [&](int k, int &i, int &j) { return cell_of(colour, k, i, j); };
      // (1) candidate checks (Eq. 2 with the skip rules).  Only evaluations
      // whose value can matter are queued: the vertical source is not
      // evaluated when it repeats the horizontal one or the cell's own flow
      // (its value is then known not to win).  The cell's cost slot holds
      // the key cost*4 + rank (own 0, horizontal 1, vertical 2; UNSET stays
      // all ones) and evaluations lower it with an LDS atomic min: the
      // smallest key is exactly the sequential strict-< choice with ties
      // kept by the earlier candidate.
      for (int base = 0; base < hw * rh; base += kThreads) {
        int i, j;
        const bool live = cell(base + tid, i, j);
        const int l = (j - gj0) * G::LW + (i - gi0);
        bool hv = false, vcomp = false;
        [[maybe_unused]] bool hin = false, vin = false;  // weight-class path: cell and target inside
        if (live) {
          // the state of the cell and of both sources in one round of LDS
          // reads: a source cell lies inside the window for every live cell
          // (the valid region shrinks towards it), so the reads need no
          // guard; an outside-grid source's slot holds nothing used
          const int lh = l + hdi, lv = l + vdj * G::LW;
          uint32_t c0 = s_cost[l], chs = s_cost[lh], cvs = s_cost[lv];
          int32_t f0 = s_flow[l], fhs = s_flow[lh], fvs = s_flow[lv];
          // keeps the compiler from sinking the reads into the branches below
          asm volatile("" : "+v"(c0), "+v"(chs), "+v"(cvs), "+v"(f0), "+v"(fhs), "+v"(fvs));
          const bool set0 = c0 != kUnset;
          const int x = (i * n) << SB, y = (j * n) << SB, xmax = (W - 1) << SB, ymax = (H - 1) << SB;
          bool vb = false, vsame_h = false, vsame_0 = false;
          int32_t fh = 0;
          if (i + hdi >= 0 && i + hdi < Wn && chs != kUnset) {
            fh = fhs;
            const int tx = x + ffk::flow_x(fh), ty = y + ffk::flow_y(fh);
            hv = !(set0 && fh == f0) && tx >= 0 && tx <= xmax && ty >= 0 && ty <= ymax;
            if constexpr (WF) hin = inner(i, j, tx, ty);
          }
          if (j + vdj >= 0 && j + vdj < Hn && cvs != kUnset) {
            const int32_t fv = fvs;
            const int tx = x + ffk::flow_x(fv), ty = y + ffk::flow_y(fv);
            vb = tx >= 0 && tx <= xmax && ty >= 0 && ty <= ymax;
            vsame_h = hv && fv == fh;
            vsame_0 = set0 && fv == f0;
            if constexpr (WF) vin = inner(i, j, tx, ty);
          }
          vcomp = vb && !vsame_h && !vsame_0;
          s_flags[l] = (uint8_t)(hv | (vb << 1) | (vsame_h << 2) | (vsame_0 << 3) | (vcomp << 4));
          if constexpr (F32)
            s_key[l] = set0 ? (unsigned long long)c0 << 2 : ~0ull;
          else
            s_cost[l] = set0 ? c0 << 2 : kUnset;
        }
        if constexpr (WF) {  // weight-class entries at the front, descriptor quads at the back
          const uint64_t bhi = __ballot(hv && hin), bvi = __ballot(vcomp && vin);
          const uint64_t bhb = __ballot(hv && !hin), bvb = __ballot(vcomp && !vin);
          const int nhi = __popcll(bhi), nvi = __popcll(bvi), nhb = __popcll(bhb), nvb = __popcll(bvb);
          int q0 = 0, q1 = 0;
          if ((tid & 63) == 0) {
            if (nhi + nvi) q0 = (int)atomicAdd(&s_qlen, (unsigned)(nhi + nvi));
            if (nhb + nvb) q1 = (int)atomicAdd(&s_blen, (unsigned)(nhb + nvb));
          }
          q0 = __shfl(q0, 0);
          q1 = __shfl(q1, 0);
          const int lane = tid & 63;
          const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
          if (hv && hin) s_queue[q0 + __popcll(bhi & below)] = (uint16_t)(l << 1);
          if (vcomp && vin) s_queue[q0 + nhi + __popcll(bvi & below)] = (uint16_t)((l << 1) | 1);
          if (hv && !hin) s_queue[QCAP - 1 - (q1 + __popcll(bhb & below))] = (uint16_t)(l << 1);
          if (vcomp && !vin) s_queue[QCAP - 1 - (q1 + nhb + __popcll(bvb & below))] = (uint16_t)((l << 1) | 1);
        } else {
          const uint64_t bh = __ballot(hv), bv = __ballot(vcomp);
          const int nh = __popcll(bh), nv = __popcll(bv);
          int q0 = 0;
          if ((tid & 63) == 0 && nh + nv) q0 = (int)atomicAdd(&s_qlen, (unsigned)(nh + nv));
          q0 = __shfl(q0, 0);
          const int lane = tid & 63;
          const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
          if (hv) s_queue[q0 + __popcll(bh & below)] = (uint16_t)(l << 1);
          if (vcomp) s_queue[q0 + nh + __popcll(bv & below)] = (uint16_t)((l << 1) | 1);
        }
      }
      __syncthreads();
      // (2) the queued evaluations, densely over all lanes
      if constexpr (WF) {
        run_queues(
            (int)s_qlen, (int)s_blen,
            [&](int e, int &l, int &i, int &j, int &bx, int &by) {
              l = e >> 1;
              i = gi0 + l % G::LW;
              j = gj0 + l / G::LW;
              const int32_t f = s_flow[(e & 1) ? l + vdj * G::LW : l + hdi];
              bx = ((i * n) << SB) + ffk::flow_x(f);
              by = ((j * n) << SB) + ffk::flow_y(f);
            },
            [&](int e, int l, uint32_t c) { atomicMin(&s_cost[l], (c << 2) | (uint32_t)(1 + (e & 1))); });
      } else if constexpr (QUAD) {
        const int qlen = (int)s_qlen;
        for (int base = 0; base < qlen; base += kQuads) {
          const int q = base + (tid >> 2);
          bool own = false;
          if (q < qlen) {
            const int e = s_queue[q], l = e >> 1, vert = e & 1;
            const int i = gi0 + l % G::LW, j = gj0 + l / G::LW;
            const int32_t f = s_flow[vert ? l + vdj * G::LW : l + hdi];
            uint32_t limit = kUnset;
            if constexpr (F32) {  // the cell's best so far (another candidate may lower it meanwhile)
              const unsigned long long key = s_key[l];
              limit = key == ~0ull ? kUnset : (uint32_t)(key >> 2);
            }
            const uint32_t c = evalq(i, j, i * n + ffk::flow_x(f), j * n + ffk::flow_y(f), limit);
            if (qr == 0) {
              if constexpr (F32)
                atomicMin(&s_key[l], ((unsigned long long)c << 2) | (unsigned long long)(1 + vert));
              else
                atomicMin(&s_cost[l], (c << 2) | (uint32_t)(1 + vert));
            }
            own = owned(i, j);
          }
          count_work(q < qlen && qr == 0, own);
        }
      } else {
        const int qlen = (int)s_qlen;
        for (int base = 0; base < qlen; base += kThreads) {
          const int q = base + tid;
          bool own = false;
          if (q < qlen) {
            const int e = s_queue[q], l = e >> 1, vert = e & 1;
            const int i = gi0 + l % G::LW, j = gj0 + l / G::LW;
            const int32_t f = s_flow[vert ? l + vdj * G::LW : l + hdi];
            const uint32_t c = evalc(i, j, i * n + ffk::flow_x(f), j * n + ffk::flow_y(f));
            atomicMin(&s_cost[l], (c << 2) | (uint32_t)(1 + vert));
            own = owned(i, j);
          }
          count_work(q < qlen, own);
        }
      }
      __syncthreads();
      if (tid == 0) s_qlen = s_blen = 0;
      // (3) new state and evaluation count of every cell
      for (int base = 0; base < hw * rh; base += kThreads) {
        int i, j;
        const bool live = cell(base + tid, i, j);
        const int l = (j - gj0) * G::LW + (i - gi0);
        int cnt = 0;
        if (live) {
          // both source flows read with the key and flags (one round of
          // LDS reads; the sources lie inside the window, as in the check)
          int32_t fhs = s_flow[l + hdi], fvs = s_flow[l + vdj * G::LW];
          asm volatile("" : "+v"(fhs), "+v"(fvs));
          bool unset;
          int rank;
          uint32_t cost;
          if constexpr (F32) {
            const unsigned long long key = s_key[l];
            unset = key == ~0ull;
            rank = unset ? 0 : (int)(key & 3);
            cost = unset ? kUnset : (uint32_t)(key >> 2);
          } else {
            const uint32_t key = s_cost[l];
            unset = key == kUnset;
            rank = unset ? 0 : (int)(key & 3);
            cost = unset ? kUnset : key >> 2;
          }
          const int fl = s_flags[l];
          const bool hv = fl & 1, vb = fl & 2, vsame_h = fl & 4, vsame_0 = fl & 8;
          cnt = hv;
          // the vertical source counts as evaluated unless it equals the
          // best flow after the horizontal step
          if (vb) cnt += vsame_h ? (rank == 0) : vsame_0 ? (rank == 1) : 1;
          if (rank) s_flow[l] = rank == 1 ? fhs : fvs;
          s_cost[l] = cost;
          if (!owned(i, j)) cnt = 0;
        }
        if constexpr (QUAD) {
          // after the second half-sweep of a step with a random search:
          // the cell is final, draw its candidate now, and that of the cell
          // of the other colour with the same index (final since the first
          // half-sweep; the same number of cells): the two hashes are
          // independent, so they run interleaved
          if (colour == 0 && rs_after(t)) {
            int i1, j1;
            const bool live1 = cell_of(1, base + tid, i1, j1);
            const int l1 = (j1 - gj0) * G::LW + (i1 - gi0);
            int32_t fc = 0, fc1 = 0;
            bool act = false, act1 = false;
            if (__ballot(live || live1)) {  // (a cell index past the valid region reads slot 0)
              act = rs_candidate(i, j, live ? l : 0, t, fc) && live;
              act1 = rs_candidate(i1, j1, live1 ? l1 : 0, t, fc1) && live1;
            }
            if (act) {
              s_flags[l] = (uint32_t)fc;
              cnt += owned(i, j);
            }
            if (act1) s_flags[l1] = (uint32_t)fc1;
            const int tot1 = __popcll(__ballot(act1 && owned(i1, j1)));
            if ((tid & 63) == 0 && tot1) atomicAdd(&s_cnt, (unsigned)tot1);
            if constexpr (WF) {
              enqueue2(act, act && inner(i, j, ((i * n) << SB) + ffk::flow_x(fc), ((j * n) << SB) + ffk::flow_y(fc)),
                       (uint16_t)l, s_rlen, s_rblen);
              enqueue2(act1,
                       act1 && inner(i1, j1, ((i1 * n) << SB) + ffk::flow_x(fc1), ((j1 * n) << SB) + ffk::flow_y(fc1)),
                       (uint16_t)l1, s_rlen, s_rblen);
            } else {
              enqueue(act, (uint16_t)l, s_rlen);
              enqueue(act1, (uint16_t)l1, s_rlen);
            }
          }
        }
        const int tot = __popcll(__ballot(cnt >= 1)) + __popcll(__ballot(cnt >= 2)) + __popcll(__ballot(cnt >= 3));
        if ((tid & 63) == 0 && tot) atomicAdd(&s_cnt, (unsigned)tot);
      }
      __syncthreads();
    }
    if (WF && rs_after(t)) {  // the candidates drawn in the second half-sweep
      run_queues(
          (int)s_rlen, (int)s_rblen,
          [&](int e, int &l, int &i, int &j, int &bx, int &by) {
            l = e;
            i = gi0 + l % G::LW;
            j = gj0 + l / G::LW;
            const int32_t fc = (int32_t)s_flags[l];
            bx = ((i * n) << SB) + ffk::flow_x(fc);
            by = ((j * n) << SB) + ffk::flow_y(fc);
          },
          [&](int, int l, uint32_t c) {
            if (c < s_cost[l]) {
              s_cost[l] = c;
              s_flow[l] = (int32_t)s_flags[l];
            }
          });
      __syncthreads();
      if (tid == 0) s_rlen = s_rblen = 0;  // next written after the next step's first half-sweep
    } else if (QUAD && rs_after(t)) {  // the candidates drawn in the second half-sweep, a quad each
      const int qlen = (int)s_rlen;
      for (int base = 0; base < qlen; base += kQuads) {
        const int q = base + (tid >> 2);
        bool own = false;
        if (q < qlen) {
          const int l = s_queue[q], i = gi0 + l % G::LW, j = gj0 + l / G::LW;
          const int32_t fc = (int32_t)s_flags[l];
          const uint32_t e = evalq(i, j, i * n + ffk::flow_x(fc), j * n + ffk::flow_y(fc), s_cost[l]);
          if (qr == 0 && e < s_cost[l]) {
            s_cost[l] = e;
            s_flow[l] = fc;
          }
          own = owned(i, j);
        }
        count_work(q < qlen && qr == 0, own);
      }
      __syncthreads();
      if (tid == 0) s_rlen = 0;  // next written after the next step's first half-sweep
    } else if (rs_after(t)) {  // random search over the whole valid window
      const int rl = max(ti0 - ml, 0), rr = min(oi1 + mr, Wn), rt = max(tj0 - mt, 0), rb = min(oj1 + mb, Hn);
      const int rw = rr - rl, rh = rb - rt;
      for (int base = 0; base < rw * rh; base += kThreads) {
        const int k = base + tid;
        const bool live = k < rw * rh;
        const int i = rl + (live ? k % rw : 0), j = rt + (live ? k / rw : 0);
        const int l = (j - gj0) * G::LW + (i - gi0);
        bool act = false;
        int fx = 0, fy = 0;
        uint32_t c0 = kUnset;
        if (live) {
          c0 = s_cost[l];
          if (c0 != kUnset) {
            int ox, oy;
            ffk::rs_offset(a.seed, d.stream_id, a.level, t, j, i, t < a.P ? a.Rnp : a.Rn, ox, oy);
            const int32_t f0 = s_flow[l];
            fx = ffk::flow_x(f0) + ox;
            fy = ffk::flow_y(f0) + oy;
            const int tx = i * n + fx, ty = j * n + fy;
            act = (ox | oy) != 0 && tx >= 0 && tx < W && ty >= 0 && ty < H;
          }
        }
        int cnt = 0;
        if (act) {
          const uint32_t e = evalc(i, j, i * n + fx, j * n + fy);
          cnt = owned(i, j);
          if (e < c0) {
            s_cost[l] = e;
            s_flow[l] = ffk::pack_flow(fx, fy);
          }
        }
        count_work(act, cnt != 0);
        const int tot = __popcll(__ballot(cnt));
        if ((tid & 63) == 0 && tot) atomicAdd(&s_cnt, (unsigned)tot);
      }
      __syncthreads();
    }
  }

  // write back the owned tile
  const int ow = oi1 - ti0, oh = oj1 - tj0;
  for (int k = tid; k < ow * oh; k += kThreads) {
    const int i = ti0 + k % ow, j = tj0 + k / ow;
    const int l = (j - gj0) * G::LW + (i - gi0);
    d.flow[(size_t)j * Wn + i] = s_flow[l];
    d.cost[(size_t)j * Wn + i] = s_cost[l];
  }
  if (tid == 0 && s_cnt && d.n_evals) atomicAdd(d.n_evals, (unsigned long long)s_cnt);
  if (tid == 0 && d.n_work && s_work[1]) {
    atomicAdd(d.n_work, (unsigned long long)s_work[0]);
    atomicAdd(d.n_work + 1, (unsigned long long)s_work[1]);
  }
}

// Waves per SIMD a kernel is compiled for: four (two with EV = 2), so that
// the register budget keeps the loads of a patch in flight together instead
// of one after another; five for the weight-class kernels (EV = 4) whose LDS
// window lets five waves per SIMD be resident (their 13 row loads fit 80
// registers; measured 1.6 % faster per pair at 1024x436), and up to seven
// for the smaller weight-class tiles whose window lets six or seven
// workgroups share a compute unit: the launch is bound by the latency of
// its barrier-separated phases, which more resident workgroups hide.
template <int TW, int TH, int kThreads, int EV, int HALO, int RR = kR, bool SUB = false, bool SPX = false>
constexpr int level_waves() {
  if constexpr (EV == 2) return 2;
  if constexpr (EV != 4 || (SPX && kThreads > 256)) return 4;  // (four entries of four rows in flight)
  using G = Geo<TW, TH, HALO>;
  // state, flags, queue; image a's rows
  constexpr int lds = G::LH * G::LW * 14 + (SUB ? 2 * G::LH + 35 : G::LH + 2 * (RR + 3)) * G::LW * 16;
  constexpr int fit = 160 * 1024 / lds * (kThreads / 64) / 4;           // waves per SIMD the LDS allows
  // a tile whose area is not a power of two (32x12) is sized for six or
  // seven resident workgroups
  if constexpr (kThreads == 256 && ((TW * TH) & (TW * TH - 1)) != 0) return fit < 5 ? 4 : (fit > 7 ? 7 : fit);
  return fit >= 5 ? 5 : 4;
}

// One workgroup per (direction, tile) of one pair; XCD-aware order.
template <int LOG2N, int TW, int TH, int kThreads, int EV, int HALO, int RR = kR>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(
    EV >= 3 ? level_waves<TW, TH, kThreads, EV, HALO, RR>() : 1, level_waves<TW, TH, kThreads, EV, HALO, RR>()))) void k_level(ffh::LevelKArgs a) {
  const int tiles = a.tiles_x * ((a.Hn + TH - 1) / TH);
  const int wg = ffk::xcd_remap(blockIdx.x, gridDim.x);
  level_body<LOG2N, TW, TH, kThreads, EV, false, HALO, RR>(a, a.dir[wg / tiles], wg % tiles);
}

// A sub-scale stage (Sec. 3.3: patch scale a.sub_m on the grid of scale n) or
// a subpixel scale (flows in 1/8 pixel), on the weight-class row maps.
template <int LOG2N, int TW, int TH, int kThreads, int HALO, bool SPX>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(
    level_waves<TW, TH, kThreads, 4, HALO, kR, !SPX, SPX>(),
    level_waves<TW, TH, kThreads, 4, HALO, kR, !SPX, SPX>()))) void k_level_sub(ffh::LevelKArgs a) {
  const int tiles = a.tiles_x * ((a.Hn + TH - 1) / TH);
  const int wg = ffk::xcd_remap(blockIdx.x, gridDim.x);
  level_body<LOG2N, TW, TH, kThreads, 4, false, HALO, kR, !SPX, SPX>(a, a.dir[wg / tiles], wg % tiles);
}

// Float learned features ([H][W][16] maps, rows in phase order, in
// LevelKDir::Da/Db).
template <int LOG2N, int TW, int TH, int kThreads, int HALO>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 3))) void k_level_f32(
    ffh::LevelKArgs a) {
  const int tiles = a.tiles_x * ((a.Hn + TH - 1) / TH);
  const int wg = ffk::xcd_remap(blockIdx.x, gridDim.x);
  level_body<LOG2N, TW, TH, kThreads, 1, true, HALO>(a, a.dir[wg / tiles], wg % tiles);
}

// Launch over the (pair, direction, tile) items of a batch.
template <int LOG2N, int TW, int TH, int kThreads, int EV, int HALO>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(
    EV >= 3 ? level_waves<TW, TH, kThreads, EV, HALO>() : 1, level_waves<TW, TH, kThreads, EV, HALO>()))) void k_level_batch(
    ffh::LevelKArgs base, ffh::BatchStage st) {
  constexpr int n = 1 << LOG2N;
  ffk::for_items(st.total, [&](int item) {
    const int p = ffk::batch_pair(st.prefix, st.npairs, item);
    const ffh::BatchPair &bp = st.pairs[p];
    ffh::LevelKArgs a = base;
    a.W = bp.W;
    a.H = bp.H;
    a.Wn = (bp.W + n - 1) / n;
    a.Hn = (bp.H + n - 1) / n;
    a.tiles_x = (a.Wn + TW - 1) / TW;
    const int tiles = a.tiles_x * ((a.Hn + TH - 1) / TH);
    const int local = item - st.prefix[p];
    const int dir = local / tiles, lv = st.lv;
    ffh::LevelKDir d;
    d.Da = bp.desc[dir][lv];
    d.Db = bp.desc[dir ^ 1][lv];
    d.Wa = bp.wform[dir][lv];
    d.Wb = bp.wform[dir ^ 1][lv];
    d.flow = st.dst ? bp.sflow[lv][dir] : bp.gflow[lv][dir];
    d.cost = st.dst ? bp.scost[lv][dir] : bp.gcost[lv][dir];
    d.flow_in = st.src ? bp.sflow[lv][dir] : bp.gflow[lv][dir];
    d.cost_in = st.src ? bp.scost[lv][dir] : bp.gcost[lv][dir];
    d.cflow = lv + 1 < st.L ? bp.gflow[lv + 1][dir] : nullptr;
    d.ccost = lv + 1 < st.L ? bp.gcost[lv + 1][dir] : nullptr;
    d.nn_key = bp.keys[dir];
    d.n_evals = bp.evals + dir;
    d.n_work = nullptr;
    d.stream_id = dir;
    level_body<LOG2N, TW, TH, kThreads, EV, false, HALO>(a, d, local % tiles);
    __syncthreads();  // the next item reuses the LDS window
  });
}

template <int LOG2N, int TW, int TH, int THREADS, int EV, int HALO = ffh::kLevelHalo, int RR = kR>
hipError_t launch_v(const ffh::LevelKArgs &a, const ffh::BatchStage *batch, hipStream_t stream) {
  if constexpr (RR != kR) {
    if (batch) return hipErrorInvalidValue;  // batches run radius 3
  } else if (batch) {
    if (batch->total <= 0) return hipSuccess;
    // a workgroup per item: 2048 workgroups, more than are resident at once,
    // left a second round a third full (n = 1, eight pairs of 2.1 Mpx in all:
    // 476 us a launch against 397)
    const dim3 grid(ffh::item_groups(batch->total));
    hipLaunchKernelGGL((k_level_batch<LOG2N, TW, TH, THREADS, EV, HALO>), grid, dim3(THREADS), 0, stream, a,
                       *batch);
    return hipGetLastError();
  }
  ffh::LevelKArgs b = a;
  b.tiles_x = (a.Wn + TW - 1) / TW;
  const int tiles = b.tiles_x * ((a.Hn + TH - 1) / TH);
  hipLaunchKernelGGL((k_level<LOG2N, TW, TH, THREADS, EV, HALO, RR>), dim3(tiles * a.ndir), dim3(THREADS), 0, stream,
                     b);
  return hipGetLastError();
}

template <int LOG2N, int TW, int TH, int THREADS, int HALO>
hipError_t launch_f32(const ffh::LevelKArgs &a, hipStream_t stream) {
  ffh::LevelKArgs b = a;
  b.tiles_x = (a.Wn + TW - 1) / TW;
  const int tiles = b.tiles_x * ((a.Hn + TH - 1) / TH);
  hipLaunchKernelGGL((k_level_f32<LOG2N, TW, TH, THREADS, HALO>), dim3(tiles * a.ndir), dim3(THREADS), 0, stream,
                     b);
  return hipGetLastError();
}

// Float-feature variant index -> kernel; kHaloF32 in ff_level.hip lists the
// window halo of every index, which must match.  16x16 or 8x8 tiles (the
// latter for the small grids of the coarse scales); a halo of 2 allows one
// step per launch, 4 two and 6 three.  Index 5, 4x4 tiles, is level_pick_f32's
// only.  Latency counts: with 512 or 1024 threads (and fewer rows in flight)
// the coarse scales of 1024x436 take 25 % longer, with all seven rows in
// flight they take the same.
template <int LOG2N>
hipError_t launch_nf32(const ffh::LevelKArgs &a, int variant, hipStream_t stream) {
  switch (variant) {
    case 0: return launch_f32<LOG2N, 16, 16, 256, 2>(a, stream);
    case 1: return launch_f32<LOG2N, 8, 8, 256, 2>(a, stream);
    case 2: return launch_f32<LOG2N, 8, 8, 256, 4>(a, stream);
    case 3: return launch_f32<LOG2N, 8, 8, 256, 6>(a, stream);
    case 4: return launch_f32<LOG2N, 16, 16, 256, 4>(a, stream);
    case 5: return launch_f32<LOG2N, 4, 4, 256, 2>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

// Variant index -> kernel; the tile and halo of every index are listed in
// kVariants (ff_level.hip), which must match.
template <int LOG2N>
hipError_t launch_n(const ffh::LevelKArgs &a, const ffh::BatchStage *batch, int variant, hipStream_t stream) {
  switch (variant) {
    case 0: return launch_v<LOG2N, 64, 32, 1024, 0>(a, batch, stream);
    case 1: return launch_v<LOG2N, 32, 16, 1024, 0>(a, batch, stream);
    case 2: return launch_v<LOG2N, 32, 16, 256, 1>(a, batch, stream);
    case 3: return launch_v<LOG2N, 16, 16, 256, 1>(a, batch, stream);
    case 4: return launch_v<LOG2N, 32, 32, 512, 1>(a, batch, stream);
    case 5: return launch_v<LOG2N, 32, 16, 256, 2>(a, batch, stream);
    case 6: return launch_v<LOG2N, 16, 16, 256, 2>(a, batch, stream);
    case 7: return launch_v<LOG2N, 32, 32, 512, 2>(a, batch, stream);
    case 8: return launch_v<LOG2N, 8, 8, 256, 2>(a, batch, stream);
    case 9: return launch_v<LOG2N, 16, 16, 512, 2>(a, batch, stream);
    case 10: return launch_v<LOG2N, 16, 16, 1024, 1>(a, batch, stream);
    case 11: return launch_v<LOG2N, 16, 16, 256, 3, 2>(a, batch, stream);
    case 12: return launch_v<LOG2N, 32, 16, 256, 3, 2>(a, batch, stream);
    case 13: return launch_v<LOG2N, 16, 16, 256, 3>(a, batch, stream);
    case 14: return launch_v<LOG2N, 8, 8, 256, 3>(a, batch, stream);
    case 15: return launch_v<LOG2N, 8, 8, 256, 3, 2>(a, batch, stream);
    case 16: return launch_v<LOG2N, 32, 16, 256, 3, 4>(a, batch, stream);
    case 17: return launch_v<LOG2N, 16, 16, 256, 3, 4>(a, batch, stream);
    case 18: return launch_v<LOG2N, 32, 16, 256, 4, 4>(a, batch, stream);
    case 19: return launch_v<LOG2N, 16, 16, 256, 4, 4>(a, batch, stream);
    case 20: return launch_v<LOG2N, 32, 16, 256, 4, 2>(a, batch, stream);
    case 21: return launch_v<LOG2N, 16, 16, 256, 4, 2>(a, batch, stream);
    case 22: return launch_v<LOG2N, 8, 8, 256, 4, 6>(a, batch, stream);
    case 23: return launch_v<LOG2N, 8, 8, 256, 4, 2>(a, batch, stream);
    case 24: return launch_v<LOG2N, 32, 16, 512, 4, 4>(a, batch, stream);
    case 25: return launch_v<LOG2N, 64, 32, 1024, 4, 4>(a, batch, stream);
    case 26: return launch_v<LOG2N, 8, 8, 1024, 3>(a, batch, stream);
    case 27: return launch_v<LOG2N, 8, 8, 1024, 3, 4>(a, batch, stream);
    case 28: return launch_v<LOG2N, 8, 8, 1024, 4>(a, batch, stream);
    case 29: return launch_v<LOG2N, 8, 8, 1024, 4, 4>(a, batch, stream);
    case 30: return launch_v<LOG2N, 16, 16, 1024, 3>(a, batch, stream);
    case 31: return launch_v<LOG2N, 32, 12, 256, 4, 2>(a, batch, stream);
    case 32: return launch_v<LOG2N, 4, 4, 1024, 3, 4>(a, batch, stream);
    default: return hipErrorInvalidValue;
  }
}

// Patch radii 2 and 4 (the second backward field of Sec. 3.7 in the
// conference setting, r2 = 2; the radius r = 4 of Flow Fields+, Sec. 4.1):
// the descriptor-quad variants, same tiles and halos as the indices of
// launch_n; quad_variant in ff_level.hip maps every other index onto one of
// these with the same window halo.
template <int LOG2N, int RR>
hipError_t launch_n_rx(const ffh::LevelKArgs &a, int variant, hipStream_t stream) {
  switch (variant) {
    case 11: return launch_v<LOG2N, 16, 16, 256, 3, 2, RR>(a, nullptr, stream);
    case 12: return launch_v<LOG2N, 32, 16, 256, 3, 2, RR>(a, nullptr, stream);
    case 13: return launch_v<LOG2N, 16, 16, 256, 3, ffh::kLevelHalo, RR>(a, nullptr, stream);
    case 14: return launch_v<LOG2N, 8, 8, 256, 3, ffh::kLevelHalo, RR>(a, nullptr, stream);
    case 15: return launch_v<LOG2N, 8, 8, 256, 3, 2, RR>(a, nullptr, stream);
    case 16: return launch_v<LOG2N, 32, 16, 256, 3, 4, RR>(a, nullptr, stream);
    case 17: return launch_v<LOG2N, 16, 16, 256, 3, 4, RR>(a, nullptr, stream);
    case 26: return launch_v<LOG2N, 8, 8, 1024, 3, ffh::kLevelHalo, RR>(a, nullptr, stream);
    case 27: return launch_v<LOG2N, 8, 8, 1024, 3, 4, RR>(a, nullptr, stream);
    case 30: return launch_v<LOG2N, 16, 16, 1024, 3, ffh::kLevelHalo, RR>(a, nullptr, stream);
    default: return hipErrorInvalidValue;
  }
}

// The weight-class kernels of the forms beside the plain radius-3 one:
// patch radii 2 and 4 (maps of that radius), sub-scale stages, subpixel
// flows.  `tile` is an index of wx_variant in ff_level.hip.
template <int LOG2N, int TW, int TH, int THREADS, int HALO>
hipError_t launch_wx_tile(const ffh::LevelKArgs &a, hipStream_t stream) {
  if (a.radius == 2) return launch_v<LOG2N, TW, TH, THREADS, 4, HALO, 2>(a, nullptr, stream);
  if (a.radius == 4) return launch_v<LOG2N, TW, TH, THREADS, 4, HALO, 4>(a, nullptr, stream);
  ffh::LevelKArgs b = a;
  b.tiles_x = (a.Wn + TW - 1) / TW;
  const dim3 grid(b.tiles_x * ((a.Hn + TH - 1) / TH) * a.ndir);
  if (a.spx) {
    hipLaunchKernelGGL((k_level_sub<LOG2N, TW, TH, THREADS, HALO, true>), grid, dim3(THREADS), 0, stream, b);
  } else if constexpr (LOG2N > 0) {
    if (!a.sub_m) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_level_sub<LOG2N, TW, TH, THREADS, HALO, false>), grid, dim3(THREADS), 0, stream, b);
  } else {
    return hipErrorInvalidValue;  // no sub-scale below the finest scale
  }
  return hipGetLastError();
}

template <int LOG2N>
hipError_t launch_wx(const ffh::LevelKArgs &a, int tile, hipStream_t stream) {
  switch (tile) {
    case 0: return launch_wx_tile<LOG2N, 32, 12, 256, 2>(a, stream);
    case 1: return launch_wx_tile<LOG2N, 16, 16, 256, 2>(a, stream);
    case 2: return launch_wx_tile<LOG2N, 16, 16, 1024, ffh::kLevelHalo>(a, stream);
    case 3: return launch_wx_tile<LOG2N, 8, 8, 1024, ffh::kLevelHalo>(a, stream);
    case 4: return launch_wx_tile<LOG2N, 8, 8, 1024, 4>(a, stream);
    case 5: return launch_wx_tile<LOG2N, 4, 4, 1024, 4>(a, stream);
    case 6: return launch_wx_tile<LOG2N, 8, 8, 256, ffh::kLevelHalo>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace
