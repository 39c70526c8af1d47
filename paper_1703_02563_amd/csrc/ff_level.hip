// Host side of the temporally blocked level kernel: launch variants and
// run-length tables, and the dispatch to the per-scale translation units
// (ff_level_s0.hip ... ff_level_s6.hip; the kernels are in ff_level_kernels.h).
#include <algorithm>

#include "ff_device.h"
#include "ff_internal.h"

namespace {

constexpr int kH = ffh::kLevelHalo;
// Tile / workgroup variants of the level kernel (tile, threads, load
// schedule, window halo: launch_n in ff_level_kernels.h maps each index to
// its kernel; the tiles and halos here must match it).  Index kNumVariants of the
// per-scale table selects the step-wise schedule instead (one launch per
// half-sweep or random-search step over all cells, no halo): better where
// the grid is too small to give every compute unit a tile.  A variant with
// quad evaluations addresses image b with 32-bit offsets; for a larger map
// its fallback (a halo at least as wide; batches count their work items
// with level_tiles, which follows the fallback) runs instead.  Variants 18-25,
// 28, 29 and 31 evaluate interior cells on the weight-class row maps; without
// those maps (a caller that passes none) their descriptor-quad twin (`nowf`,
// same halo, the same tile where one exists) runs.
struct Variant {
  int tw, th, halo, fallback, nowf;
};
constexpr Variant kVariants[] = {
    {64, 32, kH, 0, 0},   {32, 16, kH, 1, 1},   {32, 16, kH, 2, 2},   {16, 16, kH, 3, 3},   {32, 32, kH, 4, 4},
    {32, 16, kH, 5, 5},   {16, 16, kH, 6, 6},   {32, 32, kH, 7, 7},   {8, 8, kH, 8, 8},     {16, 16, kH, 9, 9},
    {16, 16, kH, 10, 10}, {16, 16, 2, 3, 11},   {32, 16, 2, 2, 12},   {16, 16, kH, 3, 13},  {8, 8, kH, 8, 14},
    {8, 8, 2, 8, 15},     {32, 16, 4, 2, 16},   {16, 16, 4, 3, 17},   {32, 16, 4, 2, 16},   {16, 16, 4, 3, 17},
    {32, 16, 2, 2, 12},   {16, 16, 2, 3, 11},   {8, 8, kH, 8, 14},    {8, 8, 2, 8, 15},     {32, 16, 4, 2, 16},
    {64, 32, 4, 0, 16},   {8, 8, kH, 8, 26},    {8, 8, 4, 8, 27},     {8, 8, kH, 8, 26},    {8, 8, 4, 8, 27},
    {16, 16, kH, 10, 30}, {32, 12, 2, 2, 12},   {4, 4, 4, 8, 32}};
constexpr int kNumVariants = 33;
static_assert(sizeof(kVariants) / sizeof(kVariants[0]) == kNumVariants, "variant table");

using ScaleLaunch = hipError_t (*)(const ffh::LevelKArgs &, const ffh::BatchStage *, int, hipStream_t);
using ScaleLaunchF32 = hipError_t (*)(const ffh::LevelKArgs &, int, hipStream_t);
constexpr ScaleLaunchF32 kScaleR2[7] = {ffh::launch_level_r2_scale0, ffh::launch_level_r2_scale1,
                                        ffh::launch_level_r2_scale2, ffh::launch_level_r2_scale3,
                                        ffh::launch_level_r2_scale4, ffh::launch_level_r2_scale5,
                                        ffh::launch_level_r2_scale6};
constexpr ScaleLaunchF32 kScaleR4[7] = {ffh::launch_level_r4_scale0, ffh::launch_level_r4_scale1,
                                        ffh::launch_level_r4_scale2, ffh::launch_level_r4_scale3,
                                        ffh::launch_level_r4_scale4, ffh::launch_level_r4_scale5,
                                        ffh::launch_level_r4_scale6};

// Radius-2 / radius-4 kernel of a table entry: the descriptor-quad variant
// with the same window halo (the run lengths follow the table's halo) -- a
// weight-class variant's quad twin, 8x8 tiles for the 4x4 ones, or for a one-lane variant (all of halo
// kLevelHalo) the quad variant of that halo and a tile of the same class.
int quad_variant(int v) {
  v = kVariants[v].nowf;
  switch (v) {
    case 11: case 12: case 13: case 14: case 15: case 16: case 17: case 26: case 27: case 30: return v;
    case 32: return 27;
    default: return kVariants[v].tw >= 16 ? 13 : 14;
  }
}

constexpr ScaleLaunchF32 kScaleWx[7] = {ffh::launch_level_wx_scale0, ffh::launch_level_wx_scale1,
                                        ffh::launch_level_wx_scale2, ffh::launch_level_wx_scale3,
                                        ffh::launch_level_wx_scale4, ffh::launch_level_wx_scale5,
                                        ffh::launch_level_wx_scale6};

// Tile index of launch_wx for a table entry: the same window halo (the run
// lengths follow it) and a tile of the same class.
int wx_variant(int v) {
  const Variant t = kVariants[v];
  if (t.halo == 2) return t.tw >= 32 ? 0 : 1;
  if (t.halo == 4) return t.tw == 4 ? 5 : 4;
  if (t.tw >= 16) return 2;
  return v == 14 || v == 22 ? 6 : 3;  // 8x8 with 256 or 1024 threads
}

constexpr ScaleLaunch kScale[7] = {ffh::launch_level_scale0, ffh::launch_level_scale1, ffh::launch_level_scale2,
                                   ffh::launch_level_scale3, ffh::launch_level_scale4, ffh::launch_level_scale5,
                                   ffh::launch_level_scale6};
constexpr ScaleLaunchF32 kScaleF32[7] = {ffh::launch_level_f32_scale0, ffh::launch_level_f32_scale1,
                                         ffh::launch_level_f32_scale2, ffh::launch_level_f32_scale3,
                                         ffh::launch_level_f32_scale4, ffh::launch_level_f32_scale5,
                                         ffh::launch_level_f32_scale6};

hipError_t dispatch(const ffh::LevelKArgs &a, const ffh::BatchStage *batch, int log2n, int variant,
                    hipStream_t stream) {
  if (log2n < 0 || log2n >= 7 || variant < 0 || variant >= kNumVariants) return hipErrorInvalidValue;
  return kScale[log2n](a, batch, variant, stream);
}

// Window halo of every variant of the float-feature level kernel (image a's
// samples staged in LDS, 64 bytes each; launch_nf32 in ff_level_kernels.h
// maps each index to its tile and kernel): 16x16 / 8x8 / 8x8 / 8x8 / 16x16,
// and 4x4, which a caller's table cannot name.
constexpr int kHaloF32[] = {2, 2, 4, 6, 4, 2};
constexpr int kNumVariantsF32 = 5;
static_assert(sizeof(kHaloF32) / sizeof(kHaloF32[0]) == kNumVariantsF32 + 1, "float variant table");

// The built-in launch tables.  Byte descriptors: weight-class evaluations
// on 32x12 tiles (256 threads, six workgroups per compute unit; two steps
// per launch) at n = 1, descriptor quads on 16x16 tiles with 256 threads
// and a halo of 2 at n = 2, with 1024 threads on 16x16 tiles at n = 4, on
// 8x8 tiles at n = 8 and on 4x4 tiles at n = 16 (so that the small grid
// still gives most compute units a workgroup); at most three steps per
// launch (the table tuned at 1024x436, which also halves the time of the
// older one-lane table at 160x120 and 1242x375).
// Float features: 16x16 tiles at n <= 2, 8x8 tiles from n = 4
// on (16x16 tiles leave most compute units idle there), one step per launch
// (the float evaluations are expensive enough that this is fastest at every
// scale, measured at 1024x436).
constexpr ffh::Tuning kDefaultTuning = {{31, 11, 30, 26, 32, 3, 3},
                                        {3, 3, 3, 3, 3, 0, 0},
                                        {0, 0, 1, 1, 1, 1, 1},
                                        {1, 1, 1, 1, 1, 1, 1}};

}  // namespace

namespace ffh {

const Tuning &default_tuning() { return kDefaultTuning; }

// The variant of scale 2^log2n for a call's grids (its pairs and directions
// together), where the caller gives no table.  What decides is how many
// workgroups a tile gives the 256 compute units; per scale, the fastest of
// all variants in a sweep over frames from 96x64 to 1920x1080 (us per call):
//  * 4x4 tiles with 1024 threads while they fit one round of one workgroup
//    per unit (1792 cells of 1024x436 at n = 16: 655 against 664 on 8x8; 2040
//    cells, 270 workgroups: 423 against 398);
//  * 8x8 tiles with 1024 threads while those fit one round (4800 cells at
//    160x120, n = 2: 147 against 150 with 256 threads and 170 on 16x16; 8160
//    cells, 270 workgroups: 429 against 398);
//  * 16x16 tiles with 1024 threads where those fill three quarters of a round,
//    against the next, in workgroups: 192 to 256 at n = 1 and 2 2 to 6 %
//    (256x128, n = 1: 213 against 226; 320x320, n = 2: 294 against 302), at n =
//    4 1 to 2 % (1024x436: 652 against 659), at n = 8 equal; 162 to 180 2 % at n =
//    1 and 2, but at n = 4 and 8 1 % slower (640x570: 556 against 553); subpixel
//    flows 8 % at 256 (256x128: 430 against 468), 1 to 2 % slower up to 240;
//  * 8x8 tiles with 256 threads while four per unit are resident at once
//    (19200 cells at 160x120, n = 1: 146 against 158 on 16x16; 32400 cells at
//    480x270, n = 2: 398 against 418; 49152 cells at 256x192, n = 1: 310
//    against 288);
//  * above, 16x16 descriptor quads, and at n = 1 the weight-class kernel on
//    32x12 tiles once they give four workgroups per unit (640x480: 563 against
//    602; 480x270: 407 against 400).
static int level_pick_variant(int log2n, const int (*sizes)[2], int count, int ndir) {
  constexpr long long kUnits = 256;
  auto workgroups = [&](int tw, int th) {
    long long t = 0;
    for (int k = 0; k < count; ++k) {
      const int Wn = (sizes[k][0] + (1 << log2n) - 1) >> log2n, Hn = (sizes[k][1] + (1 << log2n) - 1) >> log2n;
      t += (long long)((Wn + tw - 1) / tw) * ((Hn + th - 1) / th);
    }
    return t * ndir;
  };
  if (workgroups(4, 4) <= kUnits) return 32;
  if (workgroups(8, 8) <= kUnits) return 27;
  const long long big = workgroups(16, 16);
  if (big <= kUnits && 4 * big >= 3 * kUnits) return 30;
  if (workgroups(8, 8) <= 4 * kUnits) return 14;
  return log2n == 0 && workgroups(32, 12) >= 4 * kUnits ? 31 : 11;
}

// Three steps per launch at most (the halo's redundant cells), but as many as
// the widest halo takes on grids of a single cell, which have none: 64x48 at n =
// 64, six and twelve steps, 18 and 38 against 24 and 49 (4x4 tiles) and 24 and
// 49 (8x8 ones).
void level_pick(int log2n, const int (*sizes)[2], int count, int ndir, int *variant, int *passes) {
  bool single = true;
  for (int k = 0; k < count; ++k) single = single && std::max(sizes[k][0], sizes[k][1]) <= 1 << log2n;
  *variant = single ? 13 : level_pick_variant(log2n, sizes, count, ndir);
  *passes = single ? 0 : 3;
}

// The same for float features (one step per launch), from how many workgroups
// a tile gives; us per call of six steps a scale, both sides:
//  * 16x16 tiles from two workgroups per unit on (600 workgroups at 320x240,
//    n = 1: 642 against 717 on 8x8; 896 at 1024x436, n = 2: 1826 against
//    1905; 224 at n = 4: 1862 against 1832; 160 at 320x240, n = 2: 711
//    against 642);
//  * 4x4 tiles where 8x8 ones give less than half of the units a workgroup (64
//    at 1024x436, n = 16: 1836 against 1857; 40 at 320x240, n = 8: 721 against
//    747; 160 at n = 4: 766 against 716).
int level_pick_f32(int log2n, int W, int H, int ndir) {
  constexpr long long kUnits = 256;
  const long long Wn = (W + (1 << log2n) - 1) >> log2n, Hn = (H + (1 << log2n) - 1) >> log2n;
  auto workgroups = [&](int t) { return (Wn + t - 1) / t * ((Hn + t - 1) / t) * ndir; };
  if (workgroups(16) >= 2 * kUnits) return 0;
  return 2 * workgroups(8) < kUnits ? 5 : 1;
}

int level_variant_count() { return kNumVariants + 1; }  // + the step-wise schedule

int level_variant_count_f32() { return kNumVariantsF32; }

bool level_stepwise(int variant) { return variant == kNumVariants; }

bool tuning_ok(const Tuning &t) {
  for (int k = 0; k < kTuneScales; ++k) {
    if (t.variant[k] < 0 || t.variant[k] >= level_variant_count()) return false;
    if (t.variant_f32[k] < 0 || t.variant_f32[k] >= kNumVariantsF32) return false;
    if (t.passes[k] < 0 || t.passes[k] > 64 || t.passes_f32[k] < 0 || t.passes_f32[k] > 64) return false;
  }
  return true;
}

// Blocked kernel variant used where the table asks for the step-wise
// schedule but the caller only has the blocked form (batches, ff_run_level).
static int blocked_variant(int variant) { return variant == kNumVariants ? 3 : variant; }

static int log2_of(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return l;
}

int level_window_halo_f32(int variant) {
  return (variant >= 0 && variant <= kNumVariantsF32) ? kHaloF32[variant] : 2;
}

int level_window_halo(int variant) {
  const int v = blocked_variant(variant);
  return (v >= 0 && v < kNumVariants) ? kVariants[v].halo : kLevelHalo;
}

bool level_map_fits(int W, int H, int log2n) {
  const size_t P = (size_t)ffk::desc_pad(1 << log2n);
  return ((size_t)W + 2 * P) * ((size_t)H + 2 * P) * 16 < ((size_t)1 << 31);
}

// Radii 2 and 4: scales whose launches run the weight-class kernels.
static bool level_wform_rx_scale(int radius, int log2n) { return log2n <= (radius == 4 ? 1 : 0); }

bool level_uses_wform(int variant, int radius, int log2n) {
  if (radius == 2 || radius == 4) return level_wform_rx_scale(radius, log2n);
  return variant >= 0 && variant < kNumVariants && kVariants[variant].nowf != variant;
}

// The table's variant, or its fallback where image b's map is too large
// for the 32-bit offsets of the quad evaluations, or its descriptor-quad
// twin where the weight-class maps are missing.
static int launch_variant(int variant, bool map_fits, bool has_wform) {
  int v = blocked_variant(variant);
  if (v < 0 || v >= kNumVariants) return v;
  if (!map_fits) return kVariants[v].fallback;
  if (!has_wform) v = kVariants[v].nowf;
  return v;
}

static bool dirs_have_wform(const LevelKArgs &a) {
  for (int d = 0; d < a.ndir; ++d)
    if (!a.dir[d].Wa || !a.dir[d].Wb) return false;
  return true;
}

bool level_blocked_ok(int W, int H, int L, int radius) {
  if (radius == 3) return true;
  if (radius != 2 && radius != 4) return false;
  for (int l = 0; l < L; ++l)
    if (!level_map_fits(W, H, l)) return false;
  return true;
}

hipError_t launch_level(LevelKArgs a, hipStream_t stream) {
  const int l2 = log2_of(a.n);
  if (a.fcost) {
    if (l2 < 0 || l2 >= 7) return hipErrorInvalidValue;
    return kScaleF32[l2](a, a.variant, stream);
  }
  if (a.sub_m || a.spx) {  // a sub-scale stage or subpixel flows: weight-class kernels only
    const int v = blocked_variant(a.variant);
    if (l2 < 0 || l2 >= 7 || v < 0 || v >= kNumVariants || (a.radius != 0 && a.radius != 3) || !dirs_have_wform(a))
      return hipErrorInvalidValue;
    return kScaleWx[l2](a, wx_variant(v), stream);
  }
  if (a.radius == 2 || a.radius == 4) {
    const int v = blocked_variant(a.variant);
    if (l2 < 0 || l2 >= 7 || v < 0 || v >= kNumVariants || !level_map_fits(a.W, a.H, l2))
      return hipErrorInvalidValue;
    // maps of another radius (a caller's, of radius 3) are of no use
    if (a.wradius == a.radius && dirs_have_wform(a)) return kScaleWx[l2](a, wx_variant(v), stream);
    return (a.radius == 2 ? kScaleR2 : kScaleR4)[l2](a, quad_variant(v), stream);
  }
  return dispatch(a, nullptr, l2, launch_variant(a.variant, level_map_fits(a.W, a.H, l2), dirs_have_wform(a)),
                  stream);
}

hipError_t launch_batch_level(const LevelKArgs &base, const BatchStage &st, bool maps_fit, hipStream_t stream) {
  const int l2 = log2_of(base.n);
  return dispatch(base, &st, l2, launch_variant(base.variant, maps_fit, true), stream);
}

int level_tiles(int Wn, int Hn, int variant, bool maps_fit) {
  const int v = launch_variant(variant, maps_fit, true);
  if (v < 0 || v >= kNumVariants) return 0;
  const Variant t = kVariants[v];
  return ((Wn + t.tw - 1) / t.tw) * ((Hn + t.th - 1) / t.th);
}

void level_halo(int t_begin, int t_end, int halo[4]) {
  halo[0] = halo[1] = halo[2] = halo[3] = 0;
  for (int t = t_begin; t < t_end; ++t) {
    const int d = t & 3;
    halo[(d == 0 || d == 3) ? 0 : 1] += 2;
    halo[(d == 0 || d == 2) ? 2 : 3] += 2;
  }
}

}  // namespace ffh
