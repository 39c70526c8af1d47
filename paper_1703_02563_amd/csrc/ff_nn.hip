// Exact brute-force nearest neighbour of the coarsest-grid cells (stands in
// for the kd-tree candidate search of Sec. 3.1 with one candidate; the
// initial flow of Eq. 1 / Eq. 4 is F = q - p), and the l nearest references
// (a kd-tree leaf of size l).
//
// ||a - b||^2 = |a|^2 + |b|^2 - 2 a.b is a dense contraction over the 16
// descriptor bytes.  Bytes v are shifted to int8 (v - 128, a plain xor with
// 0x80), which leaves the distance unchanged.  v_mfma_i32_32x32x32_i8 has
// K = 32: both halves of K hold the same 16 bytes, so one instruction gives
// 2 a.b, and with the accumulator initialised to -|b|^2 the score
//     s = 2 a.b - |b|^2 = |a|^2 - dist
// comes out of the matrix core finished.  References are the rows and queries
// the columns of the product: a lane then holds 16 references of one query,
// and the maximum over two tiles (64 references, a unit) is 16 v_max3 and one
// compare and select for the unit's index -- 0.6 VALU operations per pair
// instead of the 1.5 that scoring (index and distance in one word) and a
// running maximum per query row cost with queries as the rows.  Which of a
// unit's references it was is found afterwards for the one winning unit per
// query (k_nn_resolve).  1024 x 436, 16-pixel grid, both directions:
// norms + search 122 -> search + resolve 71 us; 1920 x 1080,
// 32-pixel grid: 534 -> 275 us.
//
// A workgroup takes 4 waves x 32 QB queries against one chunk of references,
// staged in LDS (stages of 32 tiles, double-buffered; the norms are computed
// while staging).  With QB = 8 query blocks per wave each tile's five 16-byte
// LDS reads feed eight products; the VALU is then busy 64 % of the time and
// the matrix cores 44 %, at the 1.94 GHz that the card holds under this load.
//
// Ties: within a lane the first unit that reaches the maximum is kept, units
// merge by (score, unit), and inside the unit the smallest index of that
// score is taken: the smallest reference index of the smallest distance.
// References at or beyond N score -(2^20 - 1), below every real one.
#include <algorithm>
#include <atomic>
#include <climits>

#include "ff_device.h"
#include "ff_internal.h"

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kWaves = 4;
constexpr int kStageTiles = 32, kStageRefs = kStageTiles * 32;
constexpr int kPad = -((1 << 20) - 1);  // score of a padding reference
constexpr int kMaxChunkTiles = 4096;    // a unit's index inside its chunk must fit 11 bits
constexpr int kBatchChunkTiles = 128;   // batches: reference tiles per work item
constexpr int kBatchQB = 8;
// Waves per SIMD a kernel of QB query blocks per wave is compiled for
constexpr int nn_waves(int qb) { return qb >= 4 ? 2 : qb == 2 ? 3 : 4; }

__global__ __launch_bounds__(256) void k_fill_u64(uint64_t *dst, uint64_t value, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) dst[i] = value;
}

__device__ __forceinline__ uint4 to_i8(uint4 v) {
  return make_uint4(v.x ^ 0x80808080u, v.y ^ 0x80808080u, v.z ^ 0x80808080u, v.w ^ 0x80808080u);
}
__device__ __forceinline__ int dot16(uint4 a, uint4 b) {
  int s = __builtin_amdgcn_sdot4((int)a.x, (int)b.x, 0, false);
  s = __builtin_amdgcn_sdot4((int)a.y, (int)b.y, s, false);
  s = __builtin_amdgcn_sdot4((int)a.z, (int)b.z, s, false);
  return __builtin_amdgcn_sdot4((int)a.w, (int)b.w, s, false);
}
__device__ __forceinline__ int max3(int a, int b, int c) { return max(max(a, b), c); }

struct NNStage {
  uint4 desc[2][kStageRefs];
  int norm[2][kStageRefs];  // -|b|^2
};

// int8 descriptor of query m.
__device__ __forceinline__ uint4 query_desc(const uint8_t *Dq, int W, int nc, int Wc, int m) {
  const int i = m % Wc, j = m / Wc;
  return to_i8(reinterpret_cast<const uint4 *>(Dq)[(size_t)(j * nc) * W + (size_t)(i * nc)]);
}

// 32 QB queries per wave (block qblk) against the reference tiles [t0, t1)
// (t0 even) of one direction; the whole workgroup calls it.  kTop: instead of
// the best unit, the largest score of every group of `group` tiles goes to
// gmax[group index][M] (t0 and group even, t0 a multiple of group).
template <int QB, bool kTop>
__device__ __forceinline__ void nn_body(NNStage &sm, const ffh::NNDir &d, int M, int N, int W, int nc, int Wc, int qblk,
                                        int t0, int t1, uint32_t *part, int group, int32_t *gmax) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 31, kh = lane >> 5;
  const int m0 = (qblk * kWaves + wave) * (32 * QB);
  const bool active = m0 < M;  // wave-uniform; idle waves still help staging
  const uint4 *Dr = reinterpret_cast<const uint4 *>(d.Dr);
  const int lim = min(N, t1 * 32);

  v4i bq[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    const uint4 q = query_desc(d.Dq, W, nc, Wc, min(m0 + qb * 32 + col, M - 1));
    bq[qb] = v4i{(int)q.x, (int)q.y, (int)q.z, (int)q.w};
  }
  int best[QB], unit[QB];
#pragma unroll
  for (int qb = 0; qb < QB; ++qb) {
    best[qb] = INT_MIN;
    unit[qb] = 0;
  }

  uint4 v[4];
  auto load = [&](int b) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int ref = b * 32 + tid + 256 * k;
      v[k] = Dr[min(ref, N - 1)];
    }
  };
  auto store = [&](int b, int buf) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = tid + 256 * k;
      const bool in = b * 32 + r < lim;
      uint4 w = to_i8(v[k]);
      if (!in) w = make_uint4(0, 0, 0, 0);
      sm.desc[buf][r] = w;
      sm.norm[buf][r] = in ? -dot16(w, w) : kPad;
    }
  };
  // Operands of one unit (two tiles): the tiles' descriptors and the
  // accumulators' initial values.
  struct Unit {
    v4i a0, a1;
    v16i c0, c1;
  };
  auto fetch = [&](Unit &u, int buf, int t) {
    const v4i *da = reinterpret_cast<const v4i *>(&sm.desc[buf][t * 32 + col]);
    u.a0 = da[0];
    u.a1 = da[32];
    const v4i *cn = reinterpret_cast<const v4i *>(&sm.norm[buf][t * 32 + 4 * kh]);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const v4i x = cn[2 * g], y = cn[8 + 2 * g];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        u.c0[4 * g + r] = x[r];
        u.c1[4 * g + r] = y[r];
      }
    }
  };
  // Products of query block qb + 1 are issued before block qb's maxima, so the
  // matrix core works while the VALU reduces.
  auto score = [&](const Unit &u, int tile) {
    v16i p = __builtin_amdgcn_mfma_i32_32x32x32_i8(u.a0, bq[0], u.c0, 0, 0, 0);
    v16i q = __builtin_amdgcn_mfma_i32_32x32x32_i8(u.a1, bq[0], u.c1, 0, 0, 0);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      v16i pn = p, qn = q;
      if (qb + 1 < QB) pn = __builtin_amdgcn_mfma_i32_32x32x32_i8(u.a0, bq[(qb + 1) % QB], u.c0, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      int x = max3(p[0], p[1], p[2]);
#pragma unroll
      for (int r = 3; r < 15; r += 2) x = max3(x, p[r], p[r + 1]);
      x = max(x, p[15]);
      __builtin_amdgcn_sched_barrier(0);
      if (qb + 1 < QB) qn = __builtin_amdgcn_mfma_i32_32x32x32_i8(u.a1, bq[(qb + 1) % QB], u.c1, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < 16; r += 2) x = max3(x, q[r], q[r + 1]);
      if constexpr (!kTop) unit[qb] = x > best[qb] ? tile >> 1 : unit[qb];
      best[qb] = max(best[qb], x);
      __builtin_amdgcn_sched_barrier(0);
      p = pn;
      q = qn;
    }
    if constexpr (kTop) {
      const int next = tile + 2;
      if (tile < t1 && (next % group == 0 || next >= t1)) {  // last unit of its group
        int32_t *out = gmax + (size_t)(tile / group) * M;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
          const int o = max(best[qb], __shfl_xor(best[qb], 32));
          const int m = m0 + qb * 32 + col;
          if (kh == 0 && m < M) out[m] = o;
          best[qb] = INT_MIN;
        }
      }
    }
  };
  load(t0);
  store(t0, 0);
  __syncthreads();
  int buf = 0;
  for (int b = t0; b < t1; b += kStageTiles, buf ^= 1) {
    const bool more = b + kStageTiles < t1;
    if (more) load(b + kStageTiles);
    if (active) {
      // Two operand sets: the next unit's LDS reads are in flight while this
      // one's products and maxima run.  Units of padding at the end of the
      // last stage only score kPad.
      const int tiles = min(kStageTiles, t1 - b);
      Unit u0, u1;
      fetch(u0, buf, 0);
      for (int t = 0; t < tiles; t += 4) {
        fetch(u1, buf, t + 2);
        score(u0, b + t);
        fetch(u0, buf, min(t + 4, kStageTiles - 2));
        score(u1, b + t + 2);
      }
    }
    if (more) store(b + kStageTiles, buf ^ 1);
    __syncthreads();
  }
  if constexpr (!kTop) {
    if (!active) return;
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
      // the two halves of a query's references: larger score, then smaller unit
      const int os = __shfl_xor(best[qb], 32), ou = __shfl_xor(unit[qb], 32);
      const bool take = os > best[qb] || (os == best[qb] && ou < unit[qb]);
      const int s = take ? os : best[qb], u = take ? ou : unit[qb];
      const int m = m0 + qb * 32 + col;
      if (kh != 0 || m >= M) continue;
      const uint32_t rank = (uint32_t)((1 << 20) - s);  // smaller is nearer, below 2^21
      if (part)
        part[m] = (rank << 11) | (uint32_t)(u - (t0 >> 1));
      else
        atomicMin(reinterpret_cast<unsigned long long *>(d.keys) + m, ((unsigned long long)rank << 32) | (uint32_t)u);
    }
  }
}

__host__ __device__ __forceinline__ int nn_qblocks(int M, int qb) { return (M + 32 * kWaves * qb - 1) / (32 * kWaves * qb); }

// One workgroup per (direction, reference chunk, query block) of one pair,
// query block fastest; XCD-aware order keeps the workgroups of one chunk on
// one L2.
template <int QB>
__global__ __launch_bounds__(256, nn_waves(QB)) void k_nn(ffh::NNArgs a) {
  __shared__ NNStage sm;
  const int nqb = nn_qblocks(a.M, QB), ntiles = (a.N + 31) >> 5;
  const int wg = ffk::xcd_remap(blockIdx.x, gridDim.x);
  const ffh::NNDir d = a.dir[wg / (nqb * a.nchunk)];
  const int chunk = (wg / nqb) % a.nchunk, t0 = chunk * a.chunk_tiles;
  nn_body<QB, false>(sm, d, a.M, a.N, a.W, a.nc, a.Wc, wg % nqb, t0, min(t0 + a.chunk_tiles, ntiles),
                     a.atomic ? nullptr : reinterpret_cast<uint32_t *>(d.nb) + (size_t)chunk * a.M, 0, nullptr);
}

// Reference index of the even-pixel subset (Flow Fields+ Fast x2: pixel
// (2a, 2b) is entry b * W2 + a) -> pixel index of the image.
__device__ __forceinline__ uint32_t even_pixel(uint32_t q, int W2, int W) {
  return (q / (uint32_t)W2) * 2u * (uint32_t)W + (q % (uint32_t)W2) * 2u;
}

// Merges the chunks' results of 16 queries (block qblk) and finds the
// reference inside the winning unit: keys[m] = (squared distance << 32) | q.
// The part words of a query lie M apart, so a block of 256 reads them 16
// queries wide; then a wave per query scores the unit's 64 references.
constexpr int kResolveQ = 16;
struct NNResolve {
  unsigned long long best[16][kResolveQ];
};
__device__ __forceinline__ void nn_resolve(NNResolve &sm, const ffh::NNDir &d, int M, int N, int W, int nc, int Wc,
                                           int qblk, int nchunk, int chunk_tiles, bool atomic, int even_refs) {
  const int tid = threadIdx.x, q = tid & 15, slot = tid >> 4;
  const int mq = qblk * kResolveQ + q;
  unsigned long long k = ~0ull;
  if (mq < M) {
    if (atomic) {
      if (slot == 0) k = d.keys[mq];
    } else {
      const uint32_t *part = reinterpret_cast<const uint32_t *>(d.nb) + mq;
      for (int c = slot; c < nchunk; c += 16) {
        const uint32_t p = part[(size_t)c * M];
        const unsigned long long o =
            ((unsigned long long)(p >> 11) << 32) | (uint32_t)(c * (chunk_tiles >> 1) + (int)(p & 2047u));
        k = o < k ? o : k;
      }
    }
  }
  sm.best[slot][q] = k;
  __syncthreads();
  const int lane = tid & 63, wave = tid >> 6;
  for (int z = wave; z < kResolveQ; z += kWaves) {
    const int m = qblk * kResolveQ + z;
    if (m >= M) break;
    unsigned long long b = sm.best[0][z];
#pragma unroll
    for (int s = 1; s < 16; ++s) b = sm.best[s][z] < b ? sm.best[s][z] : b;
    const uint4 qd = query_desc(d.Dq, W, nc, Wc, m);
    const int ref = (int)(uint32_t)b * 64 + lane;
    const int want = (1 << 20) - (int)(b >> 32);
    const uint4 rd = to_i8(reinterpret_cast<const uint4 *>(d.Dr)[min(ref, N - 1)]);
    const unsigned long long hit = __ballot(ref < N && 2 * dot16(qd, rd) - dot16(rd, rd) == want);
    if (lane == 0) {
      uint32_t r = (uint32_t)b * 64u + (uint32_t)(__ffsll((long long)hit) - 1);
      if (even_refs) r = even_pixel(r, (W + 1) >> 1, W);
      d.keys[m] = ((uint64_t)(uint32_t)(dot16(qd, qd) - want) << 32) | r;
    }
  }
}

__global__ __launch_bounds__(256) void k_nn_resolve(ffh::NNArgs a) {
  __shared__ NNResolve sm;
  nn_resolve(sm, a.dir[blockIdx.y], a.M, a.N, a.W, a.nc, a.Wc, blockIdx.x, a.nchunk, a.chunk_tiles, a.atomic != 0,
             a.even_refs);
}

// ---- batches -----------------------------------------------------------

// Chunks of one pair.  The part words of a direction, nchunk * M, lie in the
// Npad words of its nb scratch; where they do not fit, one 64-bit atomic per
// query and chunk merges them.  Fine seed grids leave room for few chunks (one
// where every pixel is a query): a search of its own (alone) takes the atomics
// where more than three times as many are wanted.  One scale, a direction, us a
// call: 160 x 120 46 against 164 with one chunk, 480 x 270 (four wanted) 555
// against 960; 256 x 192 at n = 8 (three times as many wanted) 85 against 82,
// the fill included.  Batches have other pairs to fill the units: 1920 x 1080
// at n = 4 17.0 ms against 17.7 with the atomics.
struct NNPlan {
  int chunk_tiles, nchunk, atomic;
};
__host__ __device__ __forceinline__ NNPlan nn_plan(int M, int N, int want_chunks, bool alone) {
  const int ntiles = (N + 31) >> 5;
  const int fit = (ntiles * 32) / M, need = (ntiles + kMaxChunkTiles - 1) / kMaxChunkTiles;
  NNPlan p;
  p.atomic = need > fit || (alone && want_chunks > 3 * fit);
  int c = p.atomic ? want_chunks : (want_chunks < fit ? want_chunks : fit);
  c = c < need ? need : c;
  c = c < 1 ? 1 : c;
  p.chunk_tiles = (((ntiles + c - 1) / c) + 1) & ~1;
  p.nchunk = (ntiles + p.chunk_tiles - 1) / p.chunk_tiles;
  return p;
}
__host__ __device__ __forceinline__ NNPlan nn_batch_plan(int M, int N) {
  return nn_plan(M, N, (((N + 31) >> 5) + kBatchChunkTiles - 1) / kBatchChunkTiles, false);
}

// Key initialisation (items: pair, direction, 256 queries); the first item of
// a pair also clears its counters.
__global__ __launch_bounds__(256) void k_nn_fill_batch(ffh::BatchStage st) {
  ffk::for_items(st.total, [&](int item) {
    const int p = ffk::batch_pair(st.prefix, st.npairs, item);
    const ffh::BatchPair &bp = st.pairs[p];
    const int M = ((bp.W + st.n - 1) / st.n) * ((bp.H + st.n - 1) / st.n);
    const int blocks = (M + 255) / 256;
    const int local = item - st.prefix[p];
    const int dir = local / blocks, m = (local % blocks) * 256 + threadIdx.x;
    if (local == 0 && threadIdx.x < 2) bp.evals[threadIdx.x] = 0;
    if (m < M) bp.keys[dir][m] = ~0ull;
  });
}

// NN of every pair (items: pair, direction, chunk, query block).
__global__ __launch_bounds__(256, nn_waves(kBatchQB)) void k_nn_batch(ffh::BatchStage st) {
  __shared__ NNStage sm;
  ffk::for_items(st.total, [&](int item) {
    const int p = ffk::batch_pair(st.prefix, st.npairs, item);
    const ffh::BatchPair &bp = st.pairs[p];
    const int nc = st.n, Wc = (bp.W + nc - 1) / nc;
    const int M = Wc * ((bp.H + nc - 1) / nc), N = bp.W * bp.H, ntiles = (N + 31) >> 5;
    const NNPlan pl = nn_batch_plan(M, N);
    const int nqb = nn_qblocks(M, kBatchQB);
    const int local = item - st.prefix[p];
    const int dir = local / (nqb * pl.nchunk), chunk = (local / nqb) % pl.nchunk, t0 = chunk * pl.chunk_tiles;
    const ffh::NNDir d = {bp.desc1[dir], bp.desc1[dir ^ 1], bp.nb[dir ^ 1], bp.keys[dir]};
    nn_body<kBatchQB, false>(sm, d, M, N, bp.W, nc, Wc, local % nqb, t0, min(t0 + pl.chunk_tiles, ntiles),
                             pl.atomic ? nullptr : reinterpret_cast<uint32_t *>(d.nb) + (size_t)chunk * M, 0, nullptr);
  });
}

__global__ __launch_bounds__(256) void k_nn_resolve_batch(ffh::BatchStage st) {
  __shared__ NNResolve sm;
  ffk::for_items(st.total, [&](int item) {
    const int p = ffk::batch_pair(st.prefix, st.npairs, item);
    const ffh::BatchPair &bp = st.pairs[p];
    const int nc = st.n, Wc = (bp.W + nc - 1) / nc;
    const int M = Wc * ((bp.H + nc - 1) / nc), N = bp.W * bp.H;
    const NNPlan pl = nn_batch_plan(M, N);
    const int blocks = (M + kResolveQ - 1) / kResolveQ, local = item - st.prefix[p], dir = local / blocks;
    const ffh::NNDir d = {bp.desc1[dir], bp.desc1[dir ^ 1], bp.nb[dir ^ 1], bp.keys[dir]};
    nn_resolve(sm, d, M, N, bp.W, nc, Wc, local % blocks, pl.nchunk, pl.chunk_tiles, pl.atomic != 0, 0);
    __syncthreads();  // the next item writes sm again
  });
}

// ---- the l nearest references (seed rerank, Eq. 1 / Eq. 4) -------------
//
// One pass of the search writes the largest score of every group of
// consecutive tiles per query.  The l nearest references (by distance, then
// index) lie in the l groups of largest score (equal scores: the earlier
// group): any other group's best reference has l better ones before it.  A
// wave per query then scores those groups' references and ranks the l
// nearest.  Against one exclusion pass of the search per rank: eight
// candidates per cell at 741 x 497, both directions, 1432 -> 102 us.
constexpr int kTopGroups = 512;  // groups per query at most (LDS of the ranking kernel)
constexpr size_t kTopBytes = (size_t)64 << 20;  // of group scores per direction, at least 16 groups
constexpr int kTopQ = 4, kTopList = 256;  // queries per workgroup (one per wave), list length
constexpr int kTopLoads = 8;              // 64 references each

__host__ __device__ __forceinline__ int topl_groups(int M, int ntiles) {
  const long long fit = (long long)(kTopBytes / 4) / M;
  const int g = fit < 16 ? 16 : fit > kTopGroups ? kTopGroups : (int)fit;
  return g < ntiles ? g : ntiles;
}

template <int QB>
__global__ __launch_bounds__(256, nn_waves(QB)) void k_nn_groups(ffh::TopLArgs a) {
  __shared__ NNStage sm;
  const int nqb = nn_qblocks(a.M, QB), ntiles = (a.N + 31) >> 5;
  const int wg = ffk::xcd_remap(blockIdx.x, gridDim.x);
  const ffh::TopLDir &t = a.dir[wg / (nqb * a.nchunk)];
  const ffh::NNDir d = {t.Dq, t.Dr, nullptr, nullptr};
  const int t0 = ((wg / nqb) % a.nchunk) * a.chunk_tiles;
  nn_body<QB, true>(sm, d, a.M, a.N, a.W, a.nc, a.Wc, wg % nqb, t0, min(t0 + a.chunk_tiles, ntiles), nullptr, a.group,
                    t.gmax);
}

__device__ __forceinline__ unsigned long long wave_min(unsigned long long v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const unsigned long long o = __shfl_xor(v, off);
    v = o < v ? o : v;
  }
  return v;
}

// Moves the l smallest of list[0, count) (distinct keys) to its front, ranked;
// returns how many there are.  A wave calls it; count <= kTopList.
__device__ __forceinline__ int rank_list(unsigned long long *list, int count, int l, int lane) {
  unsigned long long k[kTopList / 64];
#pragma unroll
  for (int z = 0; z < kTopList / 64; ++z) k[z] = lane + 64 * z < count ? list[lane + 64 * z] : ~0ull;
  const int n = min(l, count);
  for (int r = 0; r < n; ++r) {
    unsigned long long m = k[0];
#pragma unroll
    for (int z = 1; z < kTopList / 64; ++z) m = k[z] < m ? k[z] : m;
    m = wave_min(m);
    if (lane == 0) list[r] = m;
#pragma unroll
    for (int z = 0; z < kTopList / 64; ++z)
      if (k[z] == m) k[z] = ~0ull;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return n;
}

// cand[m * l + k] = (squared distance << 32) | q of the k-th nearest
// reference, ~0 past the last reference; queries from `first` on.
__global__ __launch_bounds__(256) void k_topl_rank(ffh::TopLArgs a, int first) {
  __shared__ int32_t score[kTopQ][kTopGroups + 1];
  __shared__ unsigned long long lists[kWaves][kTopList];
  const ffh::TopLDir d = a.dir[blockIdx.y];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = first + blockIdx.x * kTopQ;
  for (int g = tid / kTopQ; g < a.ngroups; g += 256 / kTopQ) {
    const int m = min(m0 + tid % kTopQ, a.M - 1);
    score[tid % kTopQ][g] = d.gmax[(size_t)g * a.M + m];
  }
  __syncthreads();
  const uint4 *Dr = reinterpret_cast<const uint4 *>(d.Dr);
  unsigned long long *list = lists[wave];
  const int refs = a.group * 32;  // references of a group
  static_assert(kTopQ == kWaves, "one query per wave");
  const int m = m0 + wave;
  if (m >= a.M) return;
  // the l best groups: keys (2^20 - score) << 32 | group, ascending
  unsigned long long gk[kTopGroups / 64], mine = ~0ull;  // lane r: the r-th best group
#pragma unroll
  for (int s = 0; s < kTopGroups / 64; ++s) {
    const int g = lane + 64 * s;
    gk[s] = g < a.ngroups ? ((unsigned long long)(uint32_t)((1 << 20) - score[wave][g]) << 32) | (uint32_t)g : ~0ull;
  }
  for (int r = 0; r < a.l; ++r) {
    unsigned long long b = gk[0];
#pragma unroll
    for (int s = 1; s < kTopGroups / 64; ++s) b = gk[s] < b ? gk[s] : b;
    b = wave_min(b);
    if (lane == r) mine = b;
#pragma unroll
    for (int s = 0; s < kTopGroups / 64; ++s)
      if (gk[s] == b) gk[s] = ~0ull;
  }
  const uint4 qd = query_desc(d.Dq, a.W, a.nc, a.Wc, m);
  const int qn = dot16(qd, qd);
  // each of the l groups has a reference as near as its score: one further
  // away than the last of them is not among the l nearest
  const unsigned long long last = __shfl(mine, a.l - 1);
  unsigned long long bound =
      last == ~0ull ? ~0ull
                    : ((unsigned long long)(uint32_t)((int)(last >> 32) - (1 << 20) + qn) << 32) | 0xFFFFFFFFull;
  int count = 0;
  for (int r = 0; r < a.l; ++r) {
    const unsigned long long group = __shfl(mine, r);
    if (group == ~0ull) break;  // wave-uniform
    const int base = (int)(uint32_t)group * refs, end = min(base + refs, a.N);
    for (int o = base; o < end; o += 64 * kTopLoads) {
      uint4 rd[kTopLoads];  // all in flight together
#pragma unroll
      for (int k = 0; k < kTopLoads; ++k) rd[k] = Dr[min(o + 64 * k + lane, a.N - 1)];
#pragma unroll
      for (int k = 0; k < kTopLoads; ++k) {
        const int ref = o + 64 * k + lane;
        const uint4 r = to_i8(rd[k]);
        const int dist = qn - 2 * dot16(qd, r) + dot16(r, r);
        const unsigned long long key = ((unsigned long long)(uint32_t)dist << 32) | (uint32_t)ref;
        const bool in = ref < end && key <= bound;
        const unsigned long long mask = __ballot(in);
        if (mask) {
          if (in) list[count + __popcll(mask & ((1ull << lane) - 1))] = key;
          count += __popcll(mask);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          if (count > kTopList - 64) {  // keep the l nearest so far; nothing past the l-th is needed any more
            count = rank_list(list, count, a.l, lane);
            bound = list[count - 1];
          }
        }
      }
    }
  }
  count = rank_list(list, count, a.l, lane);
  if (lane < a.l) {
    unsigned long long k = lane < count ? list[lane] : ~0ull;
    if (k != ~0ull && a.even_refs)
      k = (k & 0xFFFFFFFF00000000ull) | even_pixel((uint32_t)k, (a.W + 1) >> 1, a.W);
    d.cand[(size_t)m * a.l + lane] = k;
  }
}

// Level-1 descriptors of the pixels with even x and y, row-major [H2][W2].
__global__ __launch_bounds__(256) void k_gather_even(const uint4 *src, uint4 *dst, int W, int H) {
  const int W2 = (W + 1) >> 1, H2 = (H + 1) >> 1;
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= W2 * H2) return;
  dst[k] = src[(size_t)(k / W2) * 2 * W + (k % W2) * 2];
}

}  // namespace

namespace ffh {

int batch_nn_items(int W, int H, int L) {
  const int nc = 1 << (L - 1);
  const int M = ((W + nc - 1) / nc) * ((H + nc - 1) / nc), N = W * H;
  return 2 * nn_qblocks(M, kBatchQB) * nn_batch_plan(M, N).nchunk;
}

int batch_nn_resolve_items(int W, int H, int L) {
  const int nc = 1 << (L - 1);
  return 2 * ((((W + nc - 1) / nc) * ((H + nc - 1) / nc) + kResolveQ - 1) / kResolveQ);
}

static int strided_grid(int total, int cap) { return ((std::min(std::max(total, 1), cap) + 7) / 8) * 8; }

hipError_t launch_batch_nn(const BatchStage &fill, const BatchStage &nn, const BatchStage &resolve,
                           hipStream_t stream) {
  hipLaunchKernelGGL(k_nn_fill_batch, dim3(strided_grid(fill.total, 4096)), dim3(256), 0, stream, fill);
  hipLaunchKernelGGL(k_nn_batch, dim3(item_groups(nn.total)), dim3(64 * kWaves), 0, stream, nn);
  hipLaunchKernelGGL(k_nn_resolve_batch, dim3(strided_grid(resolve.total, 2048)), dim3(256), 0, stream, resolve);
  return hipGetLastError();
}

hipError_t launch_fill_u64(uint64_t *dst, uint64_t value, int64_t count, hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, stream, dst, value, count);
  return hipGetLastError();
}

// Workgroups of the search the current device holds at once (waves per SIMD
// the kernel is compiled for = workgroups of four waves per compute unit); the
// count of compute units is cached per device.
static int nn_resident_workgroups(int qb) {
  static std::atomic<int> cache[64] = {};  // calls of several threads fill it with the same value
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256 * nn_waves(qb);
  int cus = cache[dev].load(std::memory_order_relaxed);
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return 256 * nn_waves(qb);
    cus = std::max(cus, 1);
    cache[dev].store(cus, std::memory_order_relaxed);
  }
  return cus * nn_waves(qb);
}

// Query blocks of 32 per wave: 8 while that leaves a wave with work in every
// workgroup; small grids take fewer, for more workgroups.
static int nn_query_blocks(int M) { return M > 512 ? 8 : M > 256 ? 4 : M > 128 ? 2 : 1; }

// The number of chunks whose workgroups fill the device in the fewest rounds
// for the least work per workgroup (a grid of 1.2 rounds would leave most of
// the second round idle).  Each chunk also costs its first stage and its
// merge, about as much as kChunkOverhead tiles; at least 8 tiles per chunk.
static int nn_want_chunks(int ntiles, int per_chunk_wgs, int qb) {
  constexpr int kChunkOverhead = 16;
  const int cap = nn_resident_workgroups(qb);
  int best = 1;
  long long best_cost = LLONG_MAX;
  for (int k = 1; k <= 4; ++k) {
    const int c = std::max(1, std::min(ntiles / 8, (int)((long long)k * cap / per_chunk_wgs)));  // the most in k rounds
    const long long rounds = ((long long)c * per_chunk_wgs + cap - 1) / cap;
    const long long cost = rounds * ((ntiles + c - 1) / c + kChunkOverhead);
    if (cost < best_cost) {
      best_cost = cost;
      best = c;
    }
  }
  return best;
}

hipError_t launch_nn(const NNArgs &args_in, hipStream_t stream) {
  NNArgs args = args_in;
  const int qb = nn_query_blocks(args.M), nqb = nn_qblocks(args.M, qb);
  const NNPlan p = nn_plan(args.M, args.N, nn_want_chunks((args.N + 31) / 32, nqb * args.ndir, qb), true);
  args.chunk_tiles = p.chunk_tiles;
  args.nchunk = p.nchunk;
  args.atomic = p.atomic;
  if (p.atomic)
    for (int dr = 0; dr < args.ndir; ++dr) {
      hipError_t e = launch_fill_u64(args.dir[dr].keys, ~0ull, args.M, stream);
      if (e != hipSuccess) return e;
    }
  const dim3 grid((unsigned)(nqb * p.nchunk * args.ndir));
  if (qb == 8)
    hipLaunchKernelGGL(k_nn<8>, grid, dim3(64 * kWaves), 0, stream, args);
  else if (qb == 4)
    hipLaunchKernelGGL(k_nn<4>, grid, dim3(64 * kWaves), 0, stream, args);
  else if (qb == 2)
    hipLaunchKernelGGL(k_nn<2>, grid, dim3(64 * kWaves), 0, stream, args);
  else
    hipLaunchKernelGGL(k_nn<1>, grid, dim3(64 * kWaves), 0, stream, args);
  hipLaunchKernelGGL(k_nn_resolve, dim3((args.M + kResolveQ - 1) / kResolveQ, args.ndir), dim3(256), 0, stream, args);
  return hipGetLastError();
}

hipError_t launch_gather_even(const uint8_t *desc1, uint8_t *out, int W, int H, hipStream_t stream) {
  const int n2 = ((W + 1) >> 1) * ((H + 1) >> 1);
  hipLaunchKernelGGL(k_gather_even, dim3((n2 + 255) / 256), dim3(256), 0, stream,
                     reinterpret_cast<const uint4 *>(desc1), reinterpret_cast<uint4 *>(out), W, H);
  return hipGetLastError();
}

size_t topl_scratch_bytes(int M, long long N) {
  const int ntiles = (int)((N + 31) / 32);
  return (((size_t)topl_groups(M, ntiles) * M * sizeof(int32_t)) + 255) & ~(size_t)255;
}

hipError_t launch_topl(const TopLArgs &args_in, hipStream_t stream) {
  TopLArgs a = args_in;
  if (a.l < 1 || a.l > kTopLMax || a.M < 1 || a.N < 1) return hipErrorInvalidValue;
  const int ntiles = (a.N + 31) / 32;
  const int qb = nn_query_blocks(a.M), nqb = nn_qblocks(a.M, qb);
  // groups of an even number of tiles; a chunk is a whole number of groups
  const int groups = topl_groups(a.M, ntiles);
  a.group = (((ntiles + groups - 1) / groups) + 1) & ~1;
  a.ngroups = (ntiles + a.group - 1) / a.group;
  const int want = std::min(nn_want_chunks(ntiles, nqb * a.ndir, qb), a.ngroups);
  const int per = (a.ngroups + want - 1) / want;
  a.chunk_tiles = per * a.group;
  a.nchunk = (ntiles + a.chunk_tiles - 1) / a.chunk_tiles;
  const dim3 grid((unsigned)(nqb * a.nchunk * a.ndir));
  if (qb == 8)
    hipLaunchKernelGGL(k_nn_groups<8>, grid, dim3(64 * kWaves), 0, stream, a);
  else if (qb == 4)
    hipLaunchKernelGGL(k_nn_groups<4>, grid, dim3(64 * kWaves), 0, stream, a);
  else if (qb == 2)
    hipLaunchKernelGGL(k_nn_groups<2>, grid, dim3(64 * kWaves), 0, stream, a);
  else
    hipLaunchKernelGGL(k_nn_groups<1>, grid, dim3(64 * kWaves), 0, stream, a);
  // 64 threads a query: a launch of 2^26 queries would have 2^32 threads
  for (int first = 0; first < a.M; first += kItemsPerLaunch)
    hipLaunchKernelGGL(k_topl_rank, dim3((std::min(a.M - first, kItemsPerLaunch) + kTopQ - 1) / kTopQ, a.ndir),
                       dim3(256), 0, stream, a, first);
  return hipGetLastError();
}

}  // namespace ffh
