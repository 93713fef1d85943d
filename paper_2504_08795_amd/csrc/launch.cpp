// Host side of the kernels: names, launch plans of the convolutions, and the encoders that turn a layer's arguments
// into ready-to-dispatch launches (kernel, geometry, argument bytes).
#include "kernels.h"

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "aql.h"

namespace daris {

static const char* const kNames[K_COUNT] = {
    "none",
    "conv_wave_f32_t1w2", "conv_wave_f32_t1w4", "conv_wave_f32_t1w8", "conv_wave_f32_t2w2", "conv_wave_f32_t2w4", "conv_wave_f32_t2w8",
    "conv_wave_bf16_t1w2", "conv_wave_bf16_t1w4", "conv_wave_bf16_t1w8", "conv_wave_bf16_t2w2", "conv_wave_bf16_t2w4", "conv_wave_bf16_t2w8",
    "conv_wave16_f32_t1w2", "conv_wave16_f32_t1w4", "conv_wave16_f32_t1w8", "conv_wave16_f32_t2w2", "conv_wave16_f32_t2w4", "conv_wave16_f32_t2w8",
    "conv_wave16_bf16_t1w2", "conv_wave16_bf16_t1w4", "conv_wave16_bf16_t1w8", "conv_wave16_bf16_t2w2", "conv_wave16_bf16_t2w4", "conv_wave16_bf16_t2w8",
    "conv_wave64_f32_t2w2", "conv_wave64_f32_t2w4", "conv_wave64_f32_t2w8",
    "splitk_reduce", "dwconv", "maxpool", "gavgpool", "fc", "ingest", "egress",
    "conv_wave_taps_f32_t1w2", "conv_wave_taps_f32_t1w4", "conv_wave_taps_f32_t1w8", "conv_wave_taps_f32_t2w2", "conv_wave_taps_f32_t2w8",
    "conv_wave_taps_bf16_t1w2", "conv_wave_taps_bf16_t1w4", "conv_wave_taps_bf16_t2w2", "conv_wave_taps_bf16_t2w4",
    "conv_wave16_taps_f32_t1w8", "conv_wave16_taps_f32_t2w8", "conv_wave16_taps_bf16_t1w4", "conv_wave16_taps_bf16_t1w8", "conv_wave16_taps_bf16_t2w4", "conv_wave16_taps_bf16_t2w8",
    "conv_wave64_taps_f32_t2w2", "conv_wave64_taps_f32_t2w4", "conv_wave64_taps_f32_t2w8",
    "conv_wave_image_f32_n1_t1w4", "conv_wave_image_f32_n2_t1w4", "conv_wave_image_bf16_n1_t1w4", "conv_wave_image_bf16_n2_t1w4",
    "conv_wave_image_pool_f32_n2_t1w10", "conv_wave_image_pool_bf16_n2_t1w10",
    "conv_wave16_expand_dw_f32", "conv_wave16_expand_dw_bf16", "conv_wave_chain_f32_t2w8", "conv_wave_chain_bf16_t2w4",
    "conv_wave64_pool_f32"};

const char* kernel_name(int32_t id) { return (id >= 0 && id < K_COUNT) ? kNames[id] : "?"; }

static inline int cdiv(int a, int b) { return (a + b - 1) / b; }

// Index of a tile variant in the tables of kernels.
static int variant_of(int tn, int nw) { return (tn - 1) * 3 + (nw == 2 ? 0 : nw == 4 ? 1 : 2); }

// The kernel that fetches rows once for three taps with a tile of `rows` pixels, or K_NONE: there is one for every tile and number of
// waves that the planner arrives at for 3 x 3 windows over whole rows.
static int32_t taps_kernel(int rows, int bf16, int tn, int nw) {
  static const int32_t k32[2][6] = {{K_TAPS_F32_T1W2, K_TAPS_F32_T1W4, K_TAPS_F32_T1W8, K_TAPS_F32_T2W2, K_NONE, K_TAPS_F32_T2W8},
                                    {K_TAPS_BF16_T1W2, K_TAPS_BF16_T1W4, K_NONE, K_TAPS_BF16_T2W2, K_TAPS_BF16_T2W4, K_NONE}};
  static const int32_t k16[2][6] = {{K_NONE, K_NONE, K_TAPS16_F32_T1W8, K_NONE, K_NONE, K_TAPS16_F32_T2W8},
                                    {K_NONE, K_TAPS16_BF16_T1W4, K_TAPS16_BF16_T1W8, K_NONE, K_TAPS16_BF16_T2W4, K_TAPS16_BF16_T2W8}};
  const int v = variant_of(tn, nw);
  return rows == 64 ? K_TAPS64_F32_T2W2 + v - 3 : rows == 16 ? k16[bf16][v] : k32[bf16][v];
}
// The kernel of a plan.
static int32_t conv_kernel(int rows, int bf16, int tn, int nw, bool taps) {
  if (taps) return taps_kernel(rows, bf16, tn, nw);
  const int v = variant_of(tn, nw);
  return rows == 64 ? K_CONV64_F32_T2W2 + v - 3 : rows == 16 ? (bf16 ? K_CONV16_BF16_T1W2 : K_CONV16_F32_T1W2) + v : (bf16 ? K_CONVW_BF16_T1W2 : K_CONVW_F32_T1W2) + v;
}

// Launches of equal workgroups run in ceil(workgroups / CUs) rounds: how many rounds' worth of time the grid needs per
// round's worth of work.  1 = perfectly even; 98 workgroups on 96 CUs: 1.96.
static double round_waste(int groups, int cus) { return (double)cdiv(groups, cus) * cus / groups; }

// Workgroups of a launch of MT pixel tiles and G weight groups in the order of conv_tile_of.
static uint32_t tile_order(int MT, int G, int* xmode) {
  *xmode = G % 8 == 0 ? 1 : 8 % G == 0 ? 2 : 0;
  return (uint32_t)(*xmode == 2 ? 8 * cdiv(MT, 8 / G) : G * MT);
}

// Waves of a workgroup of 32-pixel tiles, nw if there are no more tiles than CUs.  K is split so finely to shorten the launch of a workgroup a CU; where a CU has
// several, they fill it by themselves, and fewer waves have fewer partial tiles to sum and less LDS each.  us with eight waves / four, fp32: 3136 x 64
// x 576 on 96 CUs (196 tiles) 7.6 / 6.3, 784 x 128 x 512 on 96 (100) 5.5 / 5.0, 784 x 128 x 1152 on 48 12.4 / 11.6, 1520 x 256 x 512 on 160 8.0 / 7.4, 6000 x 64 x
// 256 on 160 6.0 / 5.0, 196 x 256 x 1024 on 48 8.05 / 7.35.  bf16 with four / two: 3136 x 64 x 576 on 32 CUs (98 tiles) 5.45 / 4.95, 3136 x 256 x 1152 on 128 (392)
// 8.3 / 7.6, 1364 x 512 x 1152 on 80 11.3 / 10.7, 2728 x 256 x 2304 on 232 9.7 / 8.6; with fewer tiles 784 x 256 x 512 beside 196 x 1024 x 512 on 128 (212) 4.2 / 4.5.  (Some layers of a long
// K lose alone, 840 x 512 x 4608 on 40 38.2 / 39.3; VGG-16's frames that have such layers of K >= 2304, 59 random sizes, are 0.8 % shorter with two waves in the geometric mean, 46 of them.)
// In fp32 the partial tiles are no matter for a long K of tiles one block of channels wide without three taps per fetch: 256 x 1024 x 4608 beside 256 x 1024 x 512 on 96 (256 and 256 tiles) 46.2 / 50.5, but with
// three taps per fetch 385 x 256 x 4608 on 48 49.0 / 39.5, and two blocks wide 300 x 1024 x 4608 beside 300 x 1024 x 512 on 48 166 / 124.
static int fewer_waves(int tiles, int cus, int bf16, int nw, int S, int tn, bool three_taps) {
  if (!bf16) return tiles > cus && (tn == 2 || three_taps || S <= 36 * nw) ? std::min(nw, 4) : nw;
  return 2 * tiles > 5 * cus && tiles < 6 * cus ? std::min(nw, 2) : nw;
}

static ConvPlan plan_conv_wave(int M, int N, int Kpad, int bf16, int step_align, int nominal_cus, bool allow_block, ThreeTaps three_taps, int force_tn = 0, int force_nw = 0) {
  const int kNominalWaveSlots = 4 * nominal_cus;  // SIMDs of the partition size the plan is balanced for
  // What a launch of few tiles pays for is its fixed cost and idle CUs.  Best found on a 128-CU partition (ResNet-18 shapes): 8
  // waves per workgroup splitting K, and enough grid.z slices that tiles * z is about the number of CUs, while a wave keeps
  // at least ~6 steps.
  ConvPlan pl = ConvPlan();
  const int ks = bf16 ? 16 : 8;  // k per step: two 16-byte vectors
  const int S = Kpad / ks;
  const int nb = cdiv(N, 32);
  // A wave tile two channel blocks wide halves the reads of the pixel operand, but also halves the number of tiles:
  // below about 3/4 of the partition's CUs it is better to keep 32-channel tiles and split K less (or not at all,
  // which saves the reduction launch).
  int tn = (nb % 2 == 0 && cdiv(M, 32) * (nb / 2) >= nominal_cus * 3 / 4) ? 2 : 1;
  // ... unless the 64-channel tiles are a few more than the CUs (98 on 96): the launch then takes two rounds for hardly more
  // than one round's work, and twice as many tiles of half the work take three half rounds
  if (tn == 2) {
    const int t2 = cdiv(M, 32) * (nb / 2);
    // (only for grids of one to two rounds: with more, the loss is smaller and the next round's workgroups overlap the tail -- measured: no gain)
    if (t2 > nominal_cus && t2 <= 2 * nominal_cus && round_waste(t2, nominal_cus) > 1.3 && round_waste(2 * t2, nominal_cus) < round_waste(t2, nominal_cus)) tn = 1;
  }
  if (force_tn) tn = force_tn;
  // Fetching the pixel operand as coalesced rows through LDS pays where a launch is bound by its loads.
  const int staged = step_align > 1;
  if (!bf16) step_align = 2;  // the fp32 kernels take K in chunks of two steps
  // 64 x 64 tiles (conv_block_*) once they nearly fill the partition, if K is at least 256 (3136 x 128 x 256: 7.5 us against
  // 8.8, 3072 x 64 x 576 on 64 CUs 9.9 against 12.7; but 784 x 512 x 128: 6.0 against 5.4)
  const bool block = allow_block && !bf16 && staged && nb % 2 == 0 && cdiv(M, 64) * (nb / 2) >= nominal_cus * 3 / 4 && S >= 32;
  if (block) tn = 2;
  const int tiles = (block ? cdiv(M, 64) : cdiv(M, 32)) * (nb / tn);
  int nw = bf16 ? 4 : 8;  // bf16 steps are short: fewer waves to sum through LDS beat a finer K split (measured 0.4-0.8 us per layer)
  while (nw > 2 && (S / nw < 4 || tiles * nw > 8 * kNominalWaveSlots)) nw /= 2;  // >= 4 steps per wave, <= 8 waves per SIMD
  nw = fewer_waves(tiles, nominal_cus, bf16, nw, S, tn, three_taps != kNoTaps);
  // ... whose workgroups are the smaller the more of them a CU gets: 104 tiles on 128 CUs 41 us with 8 waves, 51 with 4 (784 x
  // 512 x 4608); 196 tiles 46, 43 and, with 2 waves, 72 (3136 x 256 x 2304); 392 tiles 56, 47 and 43 (12544 x 128 x 1152)
  if (block) nw = tiles > nominal_cus * 5 / 2 ? 2 : tiles > nominal_cus * 3 / 2 ? 4 : 8;
  int z = nominal_cus / tiles;
  if (z < 1) z = 1;
  const int max_by_k = S / (nw * 6) > 0 ? S / (nw * 6) : 1;
  if (z > max_by_k) z = max_by_k;
  if (z > 16) z = 16;
  if (tiles > nominal_cus) {
    // More tiles than CUs: the launch runs in ceil(tiles * z / CUs) rounds of workgroups whose K loops take
    // (S / z) * tn * c cycles of MFMA time per SIMD, so a K split can even out the last round (200 tiles: z = 1 and 2
    // need the time of 2 whole tiles, z = 3 that of 5/3).  Estimate: loop time x 1.3 + a reduction pass of 3 us + its traffic at
    // 1.5 TB/s.  It was fitted to the fp32 matrix instruction; with the three-part products, which are not bound by the matrix pipe
    // alone, layers take 1.2 to 2.1 times as long, and for the 64 x 64 tiles it overrates the split.  us with the split that it takes
    // and without one: 784 x 512 x 4608 on 64 CUs 70.5, 73.9, on 96 77.2, 75.2, on 192 (32-pixel tiles) 47.1, 50.4; 784 x 512 x 2304 on
    // 96 47.2, 42.5; 3136 x 256 x 2304 on 64 82.9, 74.0, on 96 60.9, 59.7, on 192 51.2, 46.5.  On 128 CUs and in bf16 it splits none of
    // VGG-16's layers.
    const double cyc = block ? 96.0 : bf16 ? tn * 8.0 : (tn == 1 ? 40.0 : 64.0);
    double best = 1e30;
    for (int zz = 1; zz <= 6 && S / (nw * zz) >= 6; ++zz) {
      const double rounds = (double)cdiv(tiles * zz, nominal_cus);
      double us = 1.3 * rounds * cdiv(S, zz) * cyc / 2400.0;
      if (zz > 1) us += 3.0 + (double)zz * M * N * 4.0 / 1.5e6;
      if (us < best) {
        best = us;
        z = zz;
      }
    }
  }
  if (force_nw) {  // second problem of a two-problem launch: the first one's kernel variant, no split across workgroups
    nw = force_nw;
    z = 1;
  }
  // K slices of workgroups and waves in whole multiples of step_align steps (2 when the kernel fetches the pixel
  // operand in chunks of two steps; S is then even as well; 6 when a fetch serves three chunks, where every wave gets one at least)
  const bool taps = three_taps != kNoTaps && staged && (block || ((three_taps == kTaps || nw == 2) && S / 6 >= nw * z)) && taps_kernel(block ? 64 : 32, bf16, tn, nw) != K_NONE;
  if (taps) step_align = 6;
  const int sz = cdiv(cdiv(S, z), step_align) * step_align;
  z = cdiv(S, sz);
  pl.rows = block ? 64 : 32;
  pl.tn = tn;
  pl.nw = nw;
  pl.S = S;
  pl.sz = sz;
  pl.sw = cdiv(cdiv(sz, nw), step_align) * step_align;
  pl.step_align = step_align;
  pl.staged = staged;
  pl.gather = taps ? kGatherTaps : kGatherRows;
  pl.splitk = z;
  pl.tiles = tiles;
  pl.threads = nw * 64;
  pl.MT = cdiv(M, pl.rows);  // (the division multipliers are filled in by the caller, which knows Wo, Cin and kw)
  pl.NTn = nb / tn;
  pl.G = pl.NTn * z;
  pl.grid_x = tile_order(pl.MT, pl.G, &pl.xmode);
  pl.ws_bytes = z > 1 ? (size_t)z * M * N * sizeof(float) : 0;
  pl.kernel = conv_kernel(pl.rows, bf16, tn, nw, taps);
  return pl;
}

// 16-pixel tiles of tn 16-channel blocks, K split among the waves of a workgroup only.  Chosen for layers whose 32-row
// plan needs a reduction launch or leaves the partition idle (plan_conv); returns kernel == K_NONE when a wave would walk more than 18 steps while the shape does not fill
// three quarters of the nominal partition either, or when it is too shallow to split eight (four) ways.  Up to 18 steps the walk is
// shorter than the reduction launch, however few the tiles.  us with 32-pixel tiles and a reduction -> with 16-pixel tiles, 64 tiles
// (49 x 256) on 128 CUs and 128 tiles (49 x 512) on 192: fp32 of 8 steps 6.3 -> 4.0 and 6.5 -> 4.1, 16: 6.7 -> 5.3 and 7.0 -> 5.5, 18: 6.4 ->
// 5.6 and 6.7 -> 5.8, 24: 6.8 -> 6.6 and 7.4 -> 6.8, 28: 7.2 -> 7.3 and 7.7 -> 7.5, 32: 7.3 -> 7.9 and 8.2 -> 8.3, 36: 7.7 -> 8.5 and 8.3 -> 8.9;
// bf16 of 8 steps 5.3 -> 3.8 and 5.4 -> 3.8, 18: 5.7 -> 4.8 and 5.9 -> 5.0.  The two meet at 24 to 32 steps: 18 leaves room.  Tiles that
// fill three quarters are taken at any length, up to 32 steps with a gain (128 tiles on 128 CUs: 24 steps 7.5 -> 6.8, 32: 8.4 -> 8.2), at
// 36 without one (8.8 -> 8.8; 104 tiles 8.7 -> 9.6).
static ConvPlan plan_conv_wave16(int M, int N, int Kpad, int bf16, int nominal_cus, bool three_taps, int force_tn = 0, int force_nw = 0) {
  ConvPlan pl = ConvPlan();
  const int ks = bf16 ? 32 : 16;
  if (Kpad % 32) return pl;  // whole steps (bf16), pairs of steps (fp32)
  const int S = Kpad / ks;
  const int nb = cdiv(N, 16), mt = cdiv(M, 16);
  // two channel blocks per wave halve the reads of the pixel operand: taken when that still gives nearly one workgroup per CU
  // (and not a few more than one per CU, see plan_conv_wave)
  int tn = (nb % 2 == 0 && mt * (nb / 2) >= nominal_cus * 3 / 4) ? 2 : 1;
  if (tn == 2) {
    const int t2 = mt * (nb / 2);
    // (only for grids of one to two rounds: with more, the loss is smaller and the next round's workgroups overlap the tail -- measured: no gain)
    if (t2 > nominal_cus && t2 <= 2 * nominal_cus && round_waste(t2, nominal_cus) > 1.3 && round_waste(2 * t2, nominal_cus) < round_waste(t2, nominal_cus)) tn = 1;
  }
  if (force_tn) tn = force_tn;
  if (nb % tn) return pl;
  const int tiles = mt * (nb / tn);
  // bf16: 8 waves once K is 2048 or more (128 CUs, 4 -> 8 waves: 49 x 512 x 4608 6.4 -> 5.0 us, 49 x 512 x 2048 4.3 -> 3.9, 196 x
  // 256 x 2304 4.68 -> 4.53; but 196 x 256 x 1024 3.64 -> 3.72), unless CUs get two workgroups anyway (208 tiles planned for 192
  // CUs: ResNet-18 105.4 us with 4 waves, 107.1 with 8).  The 32-pixel tiles gain nothing from it.
  int nw = bf16 && (S < 64 || tiles > nominal_cus) ? 4 : 8;
  while (nw > 2 && S / nw < 4) nw /= 2;
  if (force_nw) {  // second problem of a two-problem launch: the first one's kernel variant, whatever its own shape
    nw = force_nw;
  } else if ((tiles < nominal_cus * 3 / 4 && S / nw > 18) || tiles > 4 * nominal_cus || S / nw < 2) {
    return pl;
  }
  pl.rows = 16;
  pl.tn = tn;
  pl.nw = nw;
  pl.S = S;
  pl.sz = S;
  const bool taps = three_taps && S % 6 == 0 && S / 6 >= nw && taps_kernel(16, bf16, tn, nw) != K_NONE;
  pl.gather = taps ? kGatherTaps : kGatherRows;
  pl.step_align = taps ? 6 : bf16 ? 1 : 2;
  pl.sw = pl.step_align * cdiv(S / pl.step_align, nw);
  pl.staged = 1;
  pl.splitk = 1;
  pl.tiles = tiles;
  pl.threads = nw * 64;
  pl.MT = mt;
  pl.NTn = nb / tn;
  pl.G = pl.NTn;
  pl.grid_x = tile_order(pl.MT, pl.G, &pl.xmode);
  pl.ws_bytes = 0;
  pl.kernel = conv_kernel(16, bf16, tn, nw, taps);
  return pl;
}

ConvPlan plan_conv(int M, int N, int Kpad, int bf16, int step_align, int cin_stride, int nominal_cus, bool allow_block, ThreeTaps three_taps) {
  if (nominal_cus < 8) nominal_cus = 8;
  if (nominal_cus > 256) nominal_cus = 256;
  const ConvPlan pl = plan_conv_wave(M, N, Kpad, bf16, step_align, nominal_cus, allow_block, three_taps);
  // Besides the plans with a reduction, what leaves half of the partition idle: half the pixels a tile, half the serial work of a wave and
  // its share of the launch.  us with 32-pixel tiles -> with 16, fp32 on 128 CUs: 196 x 64 x 384 (14 tiles) 3.63 -> 2.75, 196 x 96 x 576 (21)
  // 4.26 -> 3.41, 49 x 160 x 576 4.21 -> 3.35, 784 x 32 x 192 (25) 2.95 -> 2.60, 49 x 960 x 160 (60) 3.10 -> 2.83; bf16 2.37 -> 2.13, 2.68 -> 2.39,
  // 2.68 -> 2.32; 64 and 192 CUs alike.  Between half of the partition and all of it a short K gains (196 x 384 x 64, 84 tiles,
  // 2.73 -> 2.35; 196 x 576 x 96, 126, 2.97 -> 2.80), a longer one does not (784 x 128 x 512, 100, 4.10 -> 4.42; 196 x 1024 x 256 3.99 -> 4.54).
  // A single channel tile with a short K is taken up to half of the partition as well: there it gains with every K (196 x 32 x 64, 7 tiles, 2.53 ->
  // 2.02, 784 x 32 x 128, 25, 2.70 -> 2.40, bf16 2.22 -> 1.86), beyond less and less (2304 x 32 x 64, 72, 2.61 -> 2.29, x 128 2.80 -> 2.77; 3136, 98,
  // 2.64 -> 2.31 and 2.81 -> 2.92), and there the depthwise layer in front may join the launch, which 32-pixel tiles are for.  A launch of one tile
  // stays (9 x 20 x 128 2.45, 2.32).
  const bool narrow = pl.NTn == 1 && Kpad <= 128;
  const bool idle = pl.tiles <= (Kpad > 128 || narrow ? nominal_cus / 2 : nominal_cus) && !(narrow && pl.tiles == 1);
  if ((pl.splitk > 1 || idle) && cin_stride > 0 && cin_stride % (bf16 ? 32 : 16) == 0) {
    const ConvPlan p16 = plan_conv_wave16(M, N, Kpad, bf16, nominal_cus, three_taps == kTaps);
    if (p16.kernel != K_NONE) return p16;
  }
  return pl;
}

ConvPlan plan_conv_beside(const ConvPlan& own, const ConvPlan& light, int M, int N, int Kpad, int bf16, int step_align, int nominal_cus) {
  const int cus = std::min(std::max(nominal_cus, 8), 256);
  if (own.rows != 32 || own.splitk != 1 || own.gather == kGatherTaps || light.kernel == K_NONE) return own;
  // Beside a long K the tiles of a lighter one with a short K do not count: they are gone early and leave a CU to the few waves of one heavy tile.  us, fp32 with eight waves / four: 232 x
  // 512 x 2304 beside 232 x 512 x 256 on 128 CUs (128 tiles and 128) 9.9 / 12.4.  Not so with a shorter K or tiles two blocks of channels wide: ResNet-18's frames in which such
  // pairs have 0.9 to 1 heavy tile a CU, 40 random sizes, are 0.7 % longer with eight waves in the geometric mean, up to 3 % (two blocks: 316 x 174 on 56 CUs).
  const bool soon_done = !bf16 && own.tn == 1 && own.S >= 36 * own.nw && 2 * light.S < own.S;
  const int nw = fewer_waves(own.tiles + (soon_done ? 0 : (int)((int64_t)light.tiles * std::min(light.S, own.S) / own.S)), cus, bf16, own.nw, own.S, own.tn, false);
  return nw == own.nw ? own : plan_conv_wave(M, N, Kpad, bf16, step_align, cus, false, kNoTaps, own.tn, nw);
}

ConvPlan plan_conv_like(const ConvPlan& first, int M, int N, int Kpad, int bf16, int step_align, int nominal_cus) {
  ConvPlan none = ConvPlan();
  if (nominal_cus < 8) nominal_cus = 8;
  if (nominal_cus > 256) nominal_cus = 256;
  if (first.rows == 16) return plan_conv_wave16(M, N, Kpad, bf16, nominal_cus, false, first.tn, first.nw);
  if (cdiv(N, 32) % first.tn != 0) return none;
  return plan_conv_wave(M, N, Kpad, bf16, step_align, nominal_cus, false, kNoTaps, first.tn, first.nw);
}


// ---- kernel table ------------------------------------------------------------------------------------------------------------

namespace {

struct ReduceArgs {  // splitk_reduce_kernel(ws, bias, res, y, M, N, splitk, act)
  const float* ws;
  const float* bias;
  const void* res;
  void* y;
  int M, N, splitk, act;
};
struct IngestArgs {  // ingest_kernel / egress_kernel (x, y, C, Cs, HW)
  const void* x;
  void* y;
  int C, Cs, HW;
};
struct ProbeArgs {  // cu_probe_kernel(out, spin)
  uint32_t* out;
  int spin;
};
struct PairArgs {  // conv_wave_pair_kernel(p0, p1, n0)
  ConvArgs p0, p1;
  int n0;
};
struct ConvDwArgs {  // conv_wave_dw_kernel(p, d)
  ConvArgs p;
  DwFusedArgs d;
};
static_assert(sizeof(ImageConvArgs) == 160 && offsetof(ImageConvArgs, x) == kConvInputOffset, "the input is where every convolution has it");
constexpr uint32_t kIngestBytes = 28, kProbeBytes = 12, kPairBytes = 2 * sizeof(ConvArgs) + 4;
static_assert(sizeof(DwFusedArgs) == 32 && sizeof(ConvDwArgs) == 192 && offsetof(ConvDwArgs, d) == sizeof(ConvArgs), "fused depthwise arguments");
static_assert(sizeof(FcPooledArgs) == 64 && offsetof(FcPooledArgs, y) == kFcOutputOffset, "the logits are where every FC layer has them");
static_assert(sizeof(ExpandDwArgs) == 160 && sizeof(ChainArgs) == 88, "sizes that grab() reads");
struct ChainLaunchArgs {  // conv_chain_kernel(p, c)
  ConvArgs p;
  ChainArgs c;
};
static_assert(sizeof(ChainLaunchArgs) == 248 && offsetof(ChainLaunchArgs, c) == sizeof(ConvArgs), "chain arguments");
static_assert(sizeof(ConvArgs) == 160 && sizeof(DwArgs) == 72 && sizeof(PoolArgs) == 48 && sizeof(FcArgs) == 56 && sizeof(ReduceArgs) == 48 && sizeof(DwWindowArgs) == 88 && sizeof(PoolWindowArgs) == 64,
              "argument structures must match what the kernels were compiled for");
static_assert(offsetof(ConvArgs, x) == kConvInputOffset && offsetof(FcArgs, y) == kFcOutputOffset && offsetof(IngestArgs, x) == kIngestInputOffset &&
                  offsetof(IngestArgs, y) == kEgressOutputOffset && offsetof(PairArgs, p1) == sizeof(ConvArgs) &&
                  offsetof(PairArgs, n0) == 2 * sizeof(ConvArgs),
              "argument offsets");

bool push(std::vector<KernelLaunch>* out, const AqlKernel* k, int32_t id, uint32_t groups, uint32_t threads, const void* args, uint32_t nbytes) {
  if (!k || k->kernarg_size != nbytes || nbytes > sizeof(KernelLaunch::args) || groups == 0) return false;
  KernelLaunch l;
  l.k = k;
  l.kernel_id = id;
  l.groups = groups;
  l.threads = threads;
  l.nbytes = nbytes;
  std::memcpy(l.args, args, nbytes);
  out->push_back(l);
  return true;
}

}  // namespace

// A kernel by its name; missing keeps the first that is not there, or takes another argument block.
static const AqlKernel* find_kernel(const AqlRuntime& rt, const std::string& name, uint32_t want_bytes, std::string* missing) {
  const AqlKernel* k = rt.kernel(name);
  if ((!k || k->kernarg_size != want_bytes) && missing->empty())
    *missing = name + (k ? " (argument block of " + std::to_string(k->kernarg_size) + " bytes, expected " + std::to_string(want_bytes) + ")" : " (not in the code object)");
  return k;
}

std::string KernelTable::resolve(const AqlRuntime& rt) {
  std::string missing;
  auto get = [&](const std::string& name, uint32_t want_bytes) { return find_kernel(rt, name, want_bytes, &missing); };
  static const int tn_[6] = {1, 1, 1, 2, 2, 2}, nw_[6] = {2, 4, 8, 2, 4, 8};
  for (int b = 0; b < 2; ++b) {
    const std::string B = b ? "true" : "false";
    for (int v = 0; v < 6; ++v) {
      const std::string tp = B + ", " + std::to_string(tn_[v]) + ", " + std::to_string(nw_[v]) + ", ";
      // (fp32 has no kGatherAligned: what it would gain, a walk in scalars, kGatherGeneral does in closed form for quads of channels)
      if (taps_kernel(32, b, tn_[v], nw_[v]) != K_NONE) taps[b][v] = get("daris::conv_taps_kernel<" + B + ", " + std::to_string(tn_[v]) + ", " + std::to_string(nw_[v]) + ">", sizeof(ConvArgs));
      for (int m = b ? 0 : 1; m < 4; ++m) conv[b][v][m] = get("daris::conv_wave_kernel<" + tp + std::to_string(m) + ">", sizeof(ConvArgs));
      static const int pair_modes[3] = {0, 1, 3};
      for (int m = b ? 0 : 1; m < 3; ++m) pair[b][v][m] = get("daris::conv_wave_pair_kernel<" + tp + std::to_string(pair_modes[m]) + ">", kPairBytes);
    }
    for (int v = 0; v < 4; ++v) large[b][v / 2][v % 2] = get((v < 2 ? "daris::conv_large_kernel<" : "daris::conv_taps_large_kernel<") + B + ", " + std::to_string(v % 2 + 1) + ">", sizeof(ConvArgs));
    for (int v = 0; v < 2; ++v) image[b][v] = get("daris::conv_image_kernel<" + B + ", " + std::to_string(v + 1) + ">", sizeof(ImageConvArgs));
    for (int v = 0; v < 6; ++v) {
      for (int t = 0; t < (taps_kernel(16, b, tn_[v], nw_[v]) != K_NONE ? 2 : 1); ++t)
        conv16[b][t][v] = get((t ? "daris::conv_taps16_kernel<" : "daris::conv_wave16_kernel<") + B + ", " + std::to_string(tn_[v]) + ", " + std::to_string(nw_[v]) + ">", sizeof(ConvArgs));
      pair16[b][v] = get("daris::conv_wave16_pair_kernel<" + B + ", " + std::to_string(tn_[v]) + ", " + std::to_string(nw_[v]) + ">", kPairBytes);
      if (b ? nw_[v] != 8 : tn_[v] == 1)
        convdw[b][v] = get("daris::conv_wave_dw_kernel<" + B + ", " + std::to_string(tn_[v]) + ", " + std::to_string(nw_[v]) + ">", sizeof(ConvDwArgs));
    }
    reduce[b] = get("daris::splitk_reduce_kernel<" + B + ">", sizeof(ReduceArgs));
    dwconv[b] = get("daris::dwconv_kernel<" + B + ">", sizeof(DwArgs));
    maxpool[b] = get("daris::maxpool_kernel<" + B + ">", sizeof(PoolArgs));
    dwconv3[b] = get("daris::dwconv_window_kernel<" + B + ", 3>", sizeof(DwWindowArgs));
    for (int v = 0; v < 2; ++v) maxpool_k[b][v] = get("daris::maxpool_window_kernel<" + B + (v ? ", 3>" : ", 2>"), sizeof(PoolWindowArgs));
    gavgpool[b] = get("daris::gavgpool_kernel<" + B + ">", sizeof(PoolArgs));
    fc[b] = get("daris::fc_kernel<" + B + ">", sizeof(FcArgs));
    ingest[b] = get("daris::ingest_kernel<" + B + ">", kIngestBytes);
    egress[b] = get("daris::egress_kernel<" + B + ">", kIngestBytes);
  }
  for (int t = 0; t < 2; ++t)
    for (int v = 0; v < 3; ++v) block[t][v] = get("daris::conv_block_kernel<" + std::to_string(nw_[v]) + (t ? ", true>" : ", false>"), sizeof(ConvArgs));
  for (int b = 0; b < 2; ++b)
    for (int r = 0; r < 2; ++r)
      for (int v = 0; v < 6; ++v) {
        if (b && !r && nw_[v] == 8) continue;  // (no bf16 plan of 32-pixel tiles has eight waves)
        const std::string tp = std::string(b ? "true" : "false") + (r ? ", 16, " : ", 32, ") + std::to_string(tn_[v]) + ", " + std::to_string(nw_[v]) + ">";
        point[b][r][v] = get("daris::conv_point_kernel<" + tp, sizeof(ConvArgs));
        point_pair[b][r][v] = get("daris::conv_point_pair_kernel<" + tp, kPairBytes);
      }
  cu_probe = get("daris::cu_probe_kernel", kProbeBytes);
  return missing;
}

std::string JoinedTable::resolve(const AqlRuntime& rt) {
  std::string missing;
  auto get = [&](const std::string& name, uint32_t want_bytes) { return find_kernel(rt, name, want_bytes, &missing); };
  for (int b = 0; b < 2; ++b) {
    const std::string B = b ? "true" : "false";
    image_pool[b] = get("daris::conv_image_pool_kernel<" + B + ">", sizeof(ImageConvArgs));
    tall[b] = get("daris::conv_taps16_tall_kernel<" + B + ">", sizeof(ConvArgs));
    for (int v = 0; v < 3; ++v) block_pool[v] = get("daris::conv_block_pool_kernel<" + std::to_string(2 << v) + ">", sizeof(ConvArgs));
    chain[b] = get("daris::conv_chain_kernel<" + B + ", " + (b ? "4" : "8") + ">", sizeof(ChainLaunchArgs));
    fc_pooled[b] = get("daris::fc_pooled_kernel<" + B + ">", sizeof(FcPooledArgs));
    for (int v = 0; v < kExpandChunks; ++v) expand_dw[b][v] = get("daris::conv_expand_dw_kernel<" + B + ", " + std::to_string(v + 1) + ">", sizeof(ExpandDwArgs));
  }
  return missing;
}

// ---- encoders ----------------------------------------------------------------------------------------------------------------

static bool rows_take(const ConvArgs& a, int bf16) { return a.c_real == 0 && conv_rows_take(a.H, a.W, a.Cin, (uint64_t)a.M, a.Cout, a.Kpad, bf16); }

static bool rows_take_large(const ConvArgs& a, int bf16) { return a.c_real == 0 && a.kh == a.kw && conv_rows_take_large(a.H, a.W, a.Cin, a.Wo, a.Cout, a.kh, a.stride, a.Kpad, bf16); }

// 1x1 windows without padding, which kernels of their own take over whole rows: the same plans and sums, fewer instructions.  Alone, a bf16 layer whose waves walk two chunks (K =
// 128 on two waves) takes a little longer with them, 784 x 512 on 128 CUs 2.82 us -> 2.86, but not in a frame, where kernels change from launch to launch: ResNet-50's bf16 frame
// with the general kernel for such layers / with these, 48 random sizes on 32 to 208 CUs, 1.003 in the geometric mean, and longer in 39.
static bool point_window(const ConvArgs& a) { return a.kh == 1 && a.kw == 1 && a.pad == 0; }

static bool push_reduce(const KernelTable& kt, const ConvPlan& pl, const ConvArgs& a, int bf16, std::vector<KernelLaunch>* out) {
  if (pl.splitk <= 1) return true;
  const size_t total4 = (size_t)a.M * a.Cout / 4;
  ReduceArgs r{a.ws, a.bias, a.res, a.y, a.M, a.Cout, pl.splitk, a.act};
  return push(out, kt.reduce[bf16], K_SPLITK_REDUCE, (uint32_t)((total4 + 255) / 256), 256, &r, sizeof(ReduceArgs));
}

// What a fetch of rows for three taps assumes: the window, an output as large as the input, and K cut in threes of chunks.
static bool taps_agree(const ConvPlan& pl, const ConvArgs& a) {
  return conv_three_taps(a.kh, a.stride, a.pad) && a.kw == a.kh && a.Ho == a.H && a.Wo == a.W && pl.S % 6 == 0 && pl.sz % 6 == 0 && pl.sw % 6 == 0;
}

// Tiles and LDS places of conv_image_body; ok: it can run the convolution.
struct ImageTiles {
  bool ok;
  int nb, wn, rows, patch_w, phase, pitch, across;  // channel blocks, side by side in a workgroup, rows of a tile, see ImageConvArgs
  int64_t patch_h, tiles;
};
// The input pixels of a tile have to fit the patch (kernels of 7 x 7 up to stride 2, 11 x 11 with stride 1), its taps the table, byte
// offsets into the output 31 bits.
// pool: tiles that become pooled pixels where they are computed (two channel blocks and ten rows each).
static ImageTiles image_tiles(int Ho, int Wo, int cout_stride, int k, int stride, int S, int bf16, bool pool = false) {
  ImageTiles t = ImageTiles();
  if (stride > 64 || k > 64) return t;
  t.nb = cdiv(cout_stride, 32);
  t.wn = t.nb % 2 ? 1 : 2;
  t.rows = pool ? 2 * kImagePoolRows + 2 : 8 / t.wn;
  t.patch_w = (kImageCols - 1) * stride + k;
  t.phase = cdiv(t.patch_w, stride);
  t.pitch = t.phase * stride;  // made so that the two rows of a block lie in different banks
  for (int i = 0; i < 32 && t.pitch * stride % 32 != 16; ++i) ++t.pitch;
  t.patch_h = (int64_t)(t.rows - 1) * stride + k;
  t.across = pool ? cdiv((Wo - 1) / 2 + 1, kImagePoolCols) : cdiv(Wo, kImageCols);
  t.tiles = (int64_t)t.across * (pool ? cdiv((Ho - 1) / 2 + 1, kImagePoolRows) : cdiv(Ho, t.rows));
  const uint64_t M = (uint64_t)Ho * (uint64_t)Wo;
  t.ok = t.patch_h * t.pitch <= (pool ? kImagePoolPatch : kImagePatch) && S * 2 + 16 <= kImageTaps && M * cout_stride * (bf16 ? 2 : 4) < (1ull << 31) && (M + 16 * (uint64_t)Wo) * Wo < (1ull << 32) &&
         (uint64_t)t.tiles * (t.nb / t.wn) * (uint64_t)t.tiles < (1ull << 32) && (!pool || (t.wn == 2 && ((uint64_t)Ho + 16) * ((uint64_t)Wo + 17) * ((uint64_t)Wo + 1) < (1ull << 32)));
  return t;
}

// Patches where the gather would have more blocks of 32 pixels x 32 channels than there are CUs.  A workgroup of the gather splits K among its waves; one of
// the patches walks all of it in every wave and waits for its pixels first, so that the gather has the shorter launch while one
// round of it is enough.  us, means over 600 random layers, gather, patches with fewer blocks than CUs | with two to four times as many: 7 x 7 with stride 2 fp32 3.8,
// 4.4 | 6.8, 4.6, bf16 3.0, 3.7 | 5.6, 3.8; 5 x 5 with stride 2 fp32 3.55, 3.63 | 4.7, 3.7, bf16 2.85, 3.0 | 4.2, 3.3; 3 x 3 with stride 2 fp32 2.95, 3.15 | 4.2, 3.4,
// bf16 2.46, 2.6 | 3.4, 2.9.  Two exceptions in fp32: windows of 3 x 3 to 5 x 5 with stride 1, whose patches are small, are no slower in
// them on few blocks either (2.95, 2.93 and 3.55, 3.44); and a 1 x 1 window, which wants its pixels once, gains from four times as
// many blocks as CUs on (few 2.5, 2.9; two to four times 3.0, 3.1; four to eight 3.5, 3.4; over 32 12, 9).
void plan_input(ConvPlan* pl, int Ho, int Wo, int cout_stride, int k, int stride, int nominal_cus, int bf16) {
  pl->gather = kGatherInput;
  const ImageTiles t = image_tiles(Ho, Wo, cout_stride, k, stride, pl->S, bf16);
  const int cus = std::min(std::max(nominal_cus, 8), 256);
  const bool one_round = (int64_t)pl->tiles * pl->tn <= (int64_t)cus * (!bf16 && k == 1 ? 4 : 1);
  if (one_round && (bf16 || stride > 1 || k < 3 || k > 5)) return;
  if (pl->splitk != 1 || pl->rows != 32 || !t.ok) return;
  pl->gather = kGatherImage;
  pl->kernel = (bf16 ? K_IMAGE_BF16_N1 : K_IMAGE_F32_N1) + t.wn - 1;
  pl->tn = 1;
  pl->nw = 4;
  pl->sz = pl->sw = pl->S;
  pl->MT = (int)t.tiles;
  pl->NTn = t.nb;
  pl->G = t.nb / t.wn;
  pl->xmode = 0;
  pl->tiles = (int)t.tiles * pl->G;
  pl->grid_x = (uint32_t)pl->tiles;
  pl->threads = 256;
}

void plan_gather(ConvPlan* pl, int cin_stride, bool rows, int bf16) {
  if (pl->gather == kGatherTaps) return;
  pl->gather = pl->rows != 32 || (rows && pl->staged) ? kGatherRows : bf16 && cin_stride % 16 == 0 ? kGatherAligned : kGatherGeneral;
}

static void image_args(const ImageTiles& t, const ConvPlan& pl, const ConvArgs& a, ImageConvArgs* out) {
  ImageConvArgs& m = *out;
  m = ImageConvArgs();
  m.x = a.x; m.w = a.w; m.bias = a.bias; m.y = a.y;
  m.H = a.H; m.W = a.W; m.Ho = a.Ho; m.Wo = a.Wo; m.Cout = a.Cout; m.k = a.kh; m.stride = a.stride; m.pad = a.pad;
  m.act = a.act; m.S = pl.S; m.M = a.M; m.c_real = a.c_real; m.wave_prio = a.wave_prio;
  m.tiles = (int)t.tiles; m.across = t.across; m.patch_w = t.patch_w; m.patch = (int)t.patch_h * t.patch_w; m.phase = t.phase; m.pitch = t.pitch;
  m.mg_tiles = div_magic((uint32_t)t.tiles); m.mg_across = div_magic((uint32_t)t.across); m.mg_patch_w = div_magic((uint32_t)t.patch_w);
  m.mg_stride = div_magic((uint32_t)a.stride); m.mg_wo = div_magic((uint32_t)a.Wo); m.mg_k = div_magic((uint32_t)a.kw);
}

// What both launches of patches assume of a plan and its arguments.
static bool image_agrees(const ConvPlan& pl, const ConvArgs& a, int bf16) {
  return pl.gather == kGatherImage && a.kh == a.kw && !a.res && pl.splitk == 1 && pl.rows == 32 && pl.tn == 1 && pl.threads == 256 && a.c_real > 0 && a.c_real <= 4 &&
         a.Cin == (bf16 ? 8 : 4) && (uint64_t)a.c_real * a.H * a.W * 4 < (1ull << 31);
}

static bool encode_image(const KernelTable& kt, const ConvPlan& pl, const ConvArgs& a, int bf16, std::vector<KernelLaunch>* out) {
  const ImageTiles t = image_tiles(a.Ho, a.Wo, a.Cout, a.kh, a.stride, pl.S, bf16);
  if (!t.ok || !image_agrees(pl, a, bf16) || pl.kernel != (bf16 ? K_IMAGE_BF16_N1 : K_IMAGE_F32_N1) + t.wn - 1 || pl.grid_x != (uint64_t)t.tiles * (t.nb / t.wn)) return false;
  ImageConvArgs m;
  image_args(t, pl, a, &m);
  return push(out, kt.image[bf16][t.wn - 1], pl.kernel, pl.grid_x, (uint32_t)pl.threads, &m, sizeof(m));
}

bool image_pool_takes(const ConvPlan& pl, int Ho, int Wo, int cout_stride, int k, int stride, int nominal_cus, int bf16) {
  const ImageTiles t = image_tiles(Ho, Wo, cout_stride, k, stride, pl.S, bf16, true);
  if (pl.gather != kGatherImage || !t.ok) return false;
  const int64_t groups = t.tiles * (t.nb / t.wn), cus = nominal_cus;
  return bf16 || (cus % 32 == 0 ? groups <= cus : 9 * groups <= 8 * cus);
}

bool encode_image_pool(const JoinedTable& kt, const ConvPlan& pl, const ConvArgs& a, const PoolArgs& pool, int bf16, std::vector<KernelLaunch>* out) {
  const ImageTiles t = image_tiles(a.Ho, a.Wo, a.Cout, a.kh, a.stride, pl.S, bf16, true);
  if (!t.ok || !image_agrees(pl, a, bf16) || pool.k != 3 || pool.stride != 2 || pool.pad != 1 || pool.H != a.Ho || pool.W != a.Wo || pool.C != a.Cout ||
      pool.Ho != (a.Ho - 1) / 2 + 1 || pool.Wo != (a.Wo - 1) / 2 + 1)
    return false;
  ImageConvArgs m;
  image_args(t, pl, a, &m);
  m.y = pool.y;
  m.pool_h = pool.Ho;
  m.pool_w = pool.Wo;
  return push(out, kt.image_pool[bf16], bf16 ? K_IMAGE_POOL_BF16 : K_IMAGE_POOL_F32, (uint32_t)(t.tiles * (t.nb / t.wn)), 64 * 2 * (kImagePoolRows + 1), &m, sizeof(m));
}

bool block_pool_takes(const ConvPlan& pl, int Ho, int Wo) { return pl.rows == 64 && pl.gather == kGatherTaps && pl.splitk == 1 && pl.tn == 2 && Ho % 2 == 0 && Wo % 2 == 0; }

bool encode_block_pool(const JoinedTable& kt, const ConvPlan& pl, const ConvArgs& layer, const PoolArgs& pool, std::vector<KernelLaunch>* out) {
  if (!block_pool_takes(pl, layer.Ho, layer.Wo) || !taps_agree(pl, layer) || !conv_block_takes(layer.H, layer.W, layer.Cin, layer.kh, layer.pad, layer.Kpad) || layer.res || (layer.act & kActSumPixels) ||
      pl.threads != 64 * pl.nw || pool.k != 2 || pool.stride != 2 || pool.pad != 0 || pool.Ho != layer.Ho / 2 || pool.Wo != layer.Wo / 2 || pool.C != layer.Cout)
    return false;
  ConvArgs a = layer;
  a.y = pool.y;
  return push(out, kt.block_pool[variant_of(2, pl.nw) - 3], K_BLOCK_POOL_F32, pl.grid_x, (uint32_t)pl.threads, &a, sizeof(a));
}

bool encode_conv(const KernelTable& kt, const ConvPlan& pl, const ConvArgs& a, int bf16, std::vector<KernelLaunch>* out) {
  if (pl.tn < 1 || pl.tn > 2 || (pl.nw != 2 && pl.nw != 4 && pl.nw != 8) || pl.threads != 64 * pl.nw) return false;
  const bool input = pl.gather == kGatherInput || pl.gather == kGatherImage, taps = pl.gather == kGatherTaps;
  if (input != (a.c_real > 0)) return false;
  if (input && (a.Cin != (bf16 ? 8 : 4) || a.c_real > 4 || (uint64_t)a.c_real * a.H * a.W * 4 >= (1ull << 31))) return false;
  if (pl.gather == kGatherImage) return encode_image(kt, pl, a, bf16, out);
  if (pl.kernel != conv_kernel(pl.rows, bf16, pl.tn, pl.nw, taps)) return false;
  if ((pl.splitk > 1 && !a.ws) || (taps && !taps_agree(pl, a))) return false;
  const int v = variant_of(pl.tn, pl.nw);
  const AqlKernel* kernel;
  if (pl.rows == 16) {
    const int ks16 = bf16 ? 32 : 16;
    if ((pl.gather != kGatherRows && !taps) || !rows_take(a, bf16) || a.Kpad % 32 || pl.S * ks16 != a.Kpad || pl.sw % pl.step_align) return false;
    kernel = point_window(a) ? kt.point[bf16][1][v] : kt.conv16[bf16][taps][v];
  } else if (pl.rows == 64) {
    // what the kernel assumes: whole 64-byte rows, one bit per filter tap, byte offsets that fit 32 bits, K in whole chunks
    if ((pl.gather != kGatherRows && !taps) || bf16 || !pl.staged || pl.tn != 2 || pl.S % 2 || pl.sz % 2 || pl.sw % 2) return false;
    if (a.kh != a.kw || !conv_block_takes(a.H, a.W, a.Cin, a.kh, a.pad, a.Kpad)) return false;
    kernel = kt.block[taps][v - 3];
  } else {
    const bool rows = pl.gather == kGatherRows || taps;
    if (pl.rows != 32 || pl.gather == kGatherDepthwise) return false;
    const bool large = rows && !rows_take(a, bf16);
    if ((a.act & kActSumPixels) && (!rows || large)) return false;
    if (rows && (!pl.staged || (large && (pl.nw != 2 || !rows_take_large(a, bf16))))) return false;
    if (pl.gather == kGatherAligned && (!bf16 || a.Cin % 16)) return false;
    if ((rows || !bf16) && (pl.S % 2 || pl.sz % 2 || pl.sw % 2)) return false;
    kernel = large ? kt.large[bf16][taps][pl.tn - 1] : rows && point_window(a) ? kt.point[bf16][0][v] : taps ? kt.taps[bf16][v] : kt.conv[bf16][v][pl.gather];
  }
  return push(out, kernel, pl.kernel, pl.grid_x, (uint32_t)pl.threads, &a, sizeof(a)) && push_reduce(kt, pl, a, bf16, out);
}

bool tall_takes(const ConvPlan& pl, int M, int nominal_cus) {
  if (pl.gather != kGatherTaps || pl.tn != 2 || pl.nw != 8 || pl.S < 72 || pl.rows != 16 || pl.splitk != 1) return false;
  const int cus = std::min(std::max(nominal_cus, 8), 256);
  return cdiv(cdiv(M, 32) * pl.NTn * 2, cus) <= cdiv(pl.tiles, cus);
}

bool encode_conv_tall(const JoinedTable& kt, const ConvPlan& pl, const ConvArgs& layer, int bf16, std::vector<KernelLaunch>* out) {
  if (pl.gather != kGatherTaps || pl.tn != 2 || pl.nw != 8 || pl.rows != 16 || pl.splitk != 1 || pl.threads != 64 * pl.nw || pl.kernel != conv_kernel(16, bf16, 2, pl.nw, true) || !taps_agree(pl, layer) ||
      !rows_take(layer, bf16) || pl.S * (bf16 ? 32 : 16) != layer.Kpad)
    return false;
  ConvArgs a = layer;
  a.MT = cdiv(a.M, 32);
  a.NTn = a.G = pl.NTn * 2;
  const uint32_t groups = tile_order(a.MT, a.G, &a.xmode);
  a.mg_mt = tile_magic(groups, a.MT);
  return push(out, kt.tall[bf16], pl.kernel, groups, (uint32_t)pl.threads, &a, sizeof(a));
}

bool conv_dw_fusable(const ConvPlan& pl, int bf16) {
  if (pl.rows != 32 || !pl.staged || (!bf16 && pl.tn != 1) || (bf16 && pl.nw == 8)) return false;  // no such kernel variant
  return pl.MT >= 96 && pl.NTn == 1;
}

bool encode_conv_dw(const KernelTable& kt, const ConvPlan& pl, const ConvArgs& a, const DwFusedArgs& d, int bf16, std::vector<KernelLaunch>* out) {
  const int variant = pl.kernel - (bf16 ? K_CONVW_BF16_T1W2 : K_CONVW_F32_T1W2);
  if (pl.rows != 32 || variant < 0 || variant >= 6 || pl.threads != 64 * pl.nw || !conv_dw_fusable(pl, bf16)) return false;
  const AqlKernel* kernel = kt.convdw[bf16][variant];
  if (!kernel) return false;
  // what the kernel's producer assumes: a 1x1 / stride 1 / unpadded convolution over whole 64-byte rows, K cut in chunks of two steps,
  // a depthwise input that maps onto the convolution's pixels, and offsets that fit 32 bits
  if (a.kh != 1 || a.kw != 1 || a.stride != 1 || a.pad != 0 || a.c_real > 0 || a.Kpad != a.Cin || a.H != a.Ho || a.W != a.Wo) return false;
  if (!conv_rows_staged(a.Cin, bf16) || !pl.staged || pl.S % 2 || pl.sz % 2 || pl.sw % 2 || a.Cin < (bf16 ? 32 : 16)) return false;
  if (!d.w || !d.bias || (d.stride != 1 && d.stride != 2) || (d.H + 2 - 3) / d.stride + 1 != a.H || (d.W + 2 - 3) / d.stride + 1 != a.W) return false;
  if ((uint64_t)d.H * (uint64_t)d.W * (uint64_t)a.Cin >= (1ull << 31)) return false;
  if (pl.splitk > 1 && !a.ws) return false;
  ConvDwArgs args;
  std::memset(&args, 0, sizeof(args));
  args.p = a;
  args.d = d;
  if (!push(out, kernel, pl.kernel, pl.grid_x, (uint32_t)pl.threads, &args, sizeof(args))) return false;
  return push_reduce(kt, pl, a, bf16, out);
}

bool encode_conv_pair(const KernelTable& kt, const ConvPlan& pl0, const ConvArgs& a0, const ConvPlan& pl1, const ConvArgs& a1, int bf16,
                      std::vector<KernelLaunch>* out) {
  if (pl0.kernel != pl1.kernel || pl0.rows != pl1.rows || pl0.gather != pl1.gather || pl0.tn != pl1.tn || pl0.nw != pl1.nw || pl0.threads != 64 * pl0.nw || pl1.splitk != 1 || a0.c_real > 0 ||
      a1.c_real > 0 || pl0.rows == 64 || pl0.kernel != conv_kernel(pl0.rows, bf16, pl0.tn, pl0.nw, false))
    return false;
  const int v = variant_of(pl0.tn, pl0.nw);
  const AqlKernel* kernel;
  if (pl0.rows == 16) {
    const int ks16 = bf16 ? 32 : 16;
    if (pl0.gather != kGatherRows || pl0.splitk != 1 || !rows_take(a0, bf16) || !rows_take(a1, bf16) || a0.Kpad % 32 || a1.Kpad % 32 || pl0.sw % pl0.step_align || pl1.sw % pl1.step_align ||
        pl0.S * ks16 != a0.Kpad || pl1.S * ks16 != a1.Kpad)
      return false;
    kernel = point_window(a0) && point_window(a1) ? kt.point_pair[bf16][1][v] : kt.pair16[bf16][v];
  } else {
    const bool rows = pl0.gather == kGatherRows;
    if (rows && (!rows_take(a0, bf16) || !rows_take(a1, bf16) || !pl0.staged || !pl1.staged)) return false;
    if (pl0.gather == kGatherAligned && (!bf16 || a0.Cin % 16 || a1.Cin % 16)) return false;
    if (!rows && pl0.gather != kGatherAligned && pl0.gather != kGatherGeneral) return false;
    if ((rows || !bf16) && (pl0.S % 2 || pl0.sz % 2 || pl0.sw % 2 || pl1.S % 2 || pl1.sz % 2 || pl1.sw % 2)) return false;
    if (pl0.splitk > 1 && !a0.ws) return false;
    kernel = rows && point_window(a0) && point_window(a1) ? kt.point_pair[bf16][0][v] : kt.pair[bf16][v][rows ? 2 : pl0.gather];
  }
  PairArgs pa;
  std::memset(&pa, 0, sizeof(pa));
  pa.p0 = a0;
  pa.p1 = a1;
  pa.n0 = (int)((pl0.grid_x + 7) / 8 * 8);  // the second problem starts at a multiple of 8: its workgroup -> XCD relation is kept
  return push(out, kernel, pl0.kernel, (uint32_t)pa.n0 + pl1.grid_x, (uint32_t)pl0.threads, &pa, kPairBytes) && push_reduce(kt, pl0, a0, bf16, out);
}

// Bands of output rows that the workgroups of a channel block share: as many as fill the CUs once, and no band with more input pixels than LDS has room for.
static bool expand_bands(int H, int W, int c_stride, int dw_stride, int nominal_cus, int* band, int* bands) {
  const int Ho = (H - 1) / dw_stride + 1, groups = c_stride / 16, cus = std::min(std::max(nominal_cus, 8), 256);
  *band = cdiv(Ho, std::min(std::max(cus / groups, 1), Ho));
  const int most = (kExpandPixels / W - 3) / dw_stride + 1;  // rows of a band: (band - 1) * stride + 3 of the input
  if (kExpandPixels / W < 3 || most < 1) return false;
  *band = std::min(*band, most);
  *bands = cdiv(Ho, *band);
  return true;
}

// 16-pixel tiles of a band.
static int expand_tiles(int H, int W, int dw_stride, int band) { return cdiv(std::min((band - 1) * dw_stride + 3, H) * W, 16); }

bool plan_expand_dw(ConvPlan* pl, int H, int W, int cin_stride, int c_stride, int Kpad, int dw_stride, int nominal_cus, int bf16) {
  int band, bands;
  if (Kpad != cin_stride || Kpad % 32 || Kpad / 32 > kExpandChunks || c_stride % 16 || (uint64_t)H * W * std::max(cin_stride, c_stride) * 4 >= (1ull << 31) ||
      (uint64_t)H * W * W >= (1ull << 32) || !expand_bands(H, W, c_stride, dw_stride, nominal_cus, &band, &bands) || (uint64_t)bands * bands * (c_stride / 16) >= (1ull << 32))
    return false;
  // A workgroup computes all pixels of its band with eight waves at most, and the rows between bands twice, so that the joint launch wins while it is short.  Chunks of 32 k
  // that a CU takes through the matrix pipe (bf16, whose products take no time: tiles), over 260 random layers in fp32 and 260 in bf16 (K of 32 to 160, maps of 5 to 60 a
  // side, 32 to 256 CUs), us of the joint launch less those of the two: up to 24 (12) -1.7 to 1.3 (-2.1 to 1.3) and more than 0.6, what a launch costs in the chain of a
  // frame beside its own time, in 6 of 151 (2 of 175); above, up to 114 (28): 160 x 960 at 29 x 55 on 40 CUs 176.0 against 61.2.  MobileNetV2's frame at 307 x 240 on 40 CUs
  // joined everywhere 364, by this rule 320, with no expansion joined 326.
  const int cus = std::min(std::max(nominal_cus, 8), 256), tiles = expand_tiles(H, W, dw_stride, band);
  if ((int64_t)tiles * (bf16 ? 1 : Kpad / 32) * bands * (c_stride / 16) > (int64_t)(bf16 ? 12 : 24) * cus) return false;
  const ConvPlan own = plan_conv_wave16(H * W, c_stride, Kpad, bf16, cus, false, 0, 2);
  if (own.kernel == K_NONE) return false;
  *pl = own;
  return true;
}

bool encode_expand_dw(const JoinedTable& kt, const ConvPlan& pl, const ConvArgs& a, const DwArgs& d, int nominal_cus, int bf16, std::vector<KernelLaunch>* out) {
  ConvPlan own;
  if (a.kh != 1 || a.kw != 1 || a.stride != 1 || a.pad != 0 || a.res || a.c_real > 0 || d.k != 3 || d.pad != 1 || (d.stride != 1 && d.stride != 2) || d.H != a.Ho || d.W != a.Wo ||
      d.C != a.Cout || d.Ho != (d.H - 1) / d.stride + 1 || d.Wo != (d.W - 1) / d.stride + 1 || !plan_expand_dw(&own, a.H, a.W, a.Cin, a.Cout, a.Kpad, d.stride, nominal_cus, bf16))
    return false;
  if (pl.rows != 16 || pl.nw != 2 || pl.splitk != 1 || pl.S != own.S || pl.sw != own.sw) return false;  // (the order of the sums)
  ExpandDwArgs e = ExpandDwArgs();
  e.x = a.x; e.w = a.w; e.bias = a.bias; e.dw_w = d.w; e.dw_bias = d.bias; e.y = d.y;
  e.H = a.H; e.W = a.W; e.Cin = a.Cin; e.Ho = d.Ho; e.Wo = d.Wo; e.C = a.Cout; e.stride = d.stride; e.act = a.act; e.dw_act = d.act; e.S = pl.S; e.wave_prio = a.wave_prio;
  if (!expand_bands(a.H, a.W, a.Cout, d.stride, nominal_cus, &e.band, &e.bands)) return false;
  e.mg_bands = div_magic((uint32_t)e.bands); e.mg_w = div_magic((uint32_t)e.W); e.mg_wo = div_magic((uint32_t)e.Wo);
  // a wave for every tile, and a thread for every four channels of an output pixel (a second round of either takes as long as the first)
  const int tiles = expand_tiles(a.H, a.W, d.stride, e.band), chunks = a.Kpad / 32;
  e.threads = 64 * std::min(std::max(std::max(tiles, cdiv(std::min(e.band, e.Ho) * e.Wo * 4, 64)), 2), 8);
  return push(out, kt.expand_dw[bf16][chunks - 1], bf16 ? K_EXPAND_DW_BF16 : K_EXPAND_DW_F32, (uint32_t)(e.bands * (a.Cout / 16)), (uint32_t)e.threads, &e, sizeof(e));
}

// The kernel has one wave tile of 64 channels over all K slices of a workgroup, four waves in bf16 and eight in fp32, and takes the first 1x1 in two halves of K,
// as plans of few steps have it.
bool chain_takes(const ConvPlan& conv, int channels, const ConvPlan& wide, int wide_channels, const ConvPlan* narrow, int bf16) {
  const int nw = bf16 ? 4 : 8, unit = bf16 ? 1 : 2;  // steps of 16 k
  if (conv.rows != 32 || conv.gather != kGatherTaps || conv.splitk != 1 || conv.tn != 2 || conv.nw != nw || conv.NTn != 1 || channels != 64) return false;
  if (wide.rows != 32 || wide.gather != kGatherRows || wide.splitk != 1 || wide.S != 4 * unit || wide.nw != 2 || wide.sw != 2 * unit || wide_channels != kChainWide) return false;
  if (!narrow) return true;
  return narrow->rows == 32 && narrow->gather == kGatherRows && narrow->splitk == 1 && narrow->tn == 2 && narrow->NTn == 1 && narrow->nw == nw && narrow->S == kChainWide / 16 * unit && narrow->sw * nw == narrow->S;
}

bool encode_chain(const JoinedTable& kt, const ConvPlan& conv, const ConvArgs& a, const ConvPlan& wide, const ConvArgs& b, const ConvPlan* narrow, const ConvArgs* c, int bf16,
                  std::vector<KernelLaunch>* out) {
  if (!chain_takes(conv, a.Cout, wide, b.Cout, narrow, bf16) || !rows_take(a, bf16) || !rows_take(b, bf16) || !taps_agree(conv, a) || a.res || (a.act & kActSumPixels) || (b.act & kActSumPixels) || b.M != a.M ||
      b.kh != 1 || b.kw != 1 || b.stride != 1 || b.pad != 0 || b.Cin != a.Cout)
    return false;
  ChainLaunchArgs l = {a, ChainArgs()};
  l.p.y = nullptr;
  l.c.w3 = b.w; l.c.bias3 = b.bias; l.c.res3 = b.res; l.c.y3 = b.y;
  l.c.act3 = b.act;
  if (narrow) {
    if (!rows_take(*c, bf16) || c->res || (c->act & kActSumPixels) || c->M != a.M || c->kh != 1 || c->kw != 1 || c->stride != 1 || c->pad != 0 || c->Cin != b.Cout || c->Cout > 64) return false;
    l.c.w1 = c->w; l.c.bias1 = c->bias; l.c.y1 = c->y;
    l.c.n1 = c->Cout; l.c.act1 = c->act;
  }
  return push(out, kt.chain[bf16], K_CHAIN_F32 + bf16, conv.grid_x, (uint32_t)conv.threads, &l, sizeof(l));
}

// Grid and place finding of a window kernel (point_of): workgroups in multiples of 8, one band of them per XCD.
template <typename Args>
static uint32_t point_grid(const Args& a, int bf16, PointPlace* at) {
  const uint32_t cvn = (uint32_t)(a.C / (bf16 ? 8 : 4));
  const uint64_t total = (uint64_t)a.Ho * a.Wo * cvn;
  at->per_xcd = (uint32_t)((total + 2047) / 2048);
  const uint64_t threads = (uint64_t)at->per_xcd * 2048;
  at->mg_cv = tile_magic(threads, (int)cvn);
  at->mg_wo = tile_magic((threads + cvn - 1) / cvn, a.Wo);
  return threads < (1ull << 32) ? 8 * at->per_xcd : 0;
}
// Byte offsets into the input, padding included, fit a signed 32-bit number.
template <typename Args>
static bool offsets_fit(const Args& a, int bf16) {
  return (uint64_t)(a.H + 2 * a.pad + a.k) * (uint64_t)(a.W + 2 * a.pad + a.k) * a.C * (bf16 ? 2 : 4) < (1ull << 31);
}
bool encode_dwconv(const KernelTable& kt, const DwArgs& a, int bf16, std::vector<KernelLaunch>* out) {
  if (a.k == 3 && offsets_fit(a, bf16)) {
    DwWindowArgs w{a, PointPlace()};
    const uint32_t groups = point_grid(a, bf16, &w.at);
    return push(out, kt.dwconv3[bf16], K_DWCONV, groups, 256, &w, sizeof(w));
  }
  const size_t total = (size_t)a.Ho * a.Wo * (a.C / (bf16 ? 8 : 4));
  return push(out, kt.dwconv[bf16], K_DWCONV, (uint32_t)((total + 255) / 256), 256, &a, sizeof(a));
}
bool encode_maxpool(const KernelTable& kt, const PoolArgs& a, int bf16, std::vector<KernelLaunch>* out) {
  if ((a.k == 2 || a.k == 3) && offsets_fit(a, bf16)) {
    PoolWindowArgs w{a, PointPlace()};
    const uint32_t groups = point_grid(a, bf16, &w.at);
    return push(out, kt.maxpool_k[bf16][a.k - 2], K_MAXPOOL, groups, 256, &w, sizeof(w));
  }
  const size_t total = (size_t)a.Ho * a.Wo * (a.C / (bf16 ? 8 : 4));
  return push(out, kt.maxpool[bf16], K_MAXPOOL, (uint32_t)((total + 255) / 256), 256, &a, sizeof(a));
}
bool encode_gavgpool(const KernelTable& kt, const PoolArgs& layer, int bf16, std::vector<KernelLaunch>* out) {
  PoolArgs a = layer;
  a.k = a.H * a.W;  // what the sums are divided by
  return push(out, kt.gavgpool[bf16], K_GAVGPOOL, (uint32_t)cdiv(a.C, 64), 256, &a, sizeof(a));
}
bool sums_pixels(const ConvPlan& pl, int channels) {
  return (pl.rows == 16 || pl.rows == 32) && pl.splitk == 1 && (pl.gather == kGatherRows || pl.gather == kGatherTaps) && pl.MT <= kPooledTiles && channels <= kPooledInputs;
}
bool encode_pooled_sums(const KernelTable& kt, const float* x, float* y, int C, int tiles, int pixels, std::vector<KernelLaunch>* out) {
  if (tiles < 1 || tiles > kPooledTiles) return false;
  PoolArgs a = PoolArgs();
  a.x = x; a.y = y; a.H = tiles; a.W = 1; a.C = C; a.Ho = a.Wo = 1;
  a.k = pixels;
  return push(out, kt.gavgpool[0], K_GAVGPOOL, (uint32_t)cdiv(C, 64), 256, &a, sizeof(a));
}
bool encode_fc_pooled(const JoinedTable& kt, const FcArgs& f, int tiles, int pixels, int bf16, std::vector<KernelLaunch>* out) {
  if (tiles < 1 || tiles > kPooledTiles || f.K > kPooledInputs || f.K % (bf16 ? 8 : 4)) return false;
  FcPooledArgs a = FcPooledArgs();
  a.x = (const float*)f.x; a.w = f.w; a.bias = f.bias; a.y = f.y;
  a.K = f.K; a.N = f.N; a.Ns = f.Ns; a.act = f.act; a.out_f32 = f.out_f32; a.tiles = tiles; a.pixels = pixels;
  return push(out, kt.fc_pooled[bf16], K_FC, (uint32_t)cdiv(a.Ns, kPooledRows), 64 * kPooledRows, &a, sizeof(a));
}
bool encode_fc(const KernelTable& kt, const FcArgs& layer, int bf16, std::vector<KernelLaunch>* out) {
  FcArgs a = layer;
  // Half of the 256 MB last cache or more: what is left of it at the next frame is little (fc_row has the measurements).
  a.stream = (uint64_t)a.N * a.K * (bf16 ? 2 : 4) >= (128ull << 20) && a.K / (bf16 ? 8 : 4) > 2048;
  return push(out, kt.fc[bf16], K_FC, (uint32_t)cdiv(a.Ns, 4), 256, &a, sizeof(a));
}
bool encode_ingest(const KernelTable& kt, const float* x, void* y, int C, int Cs, int H, int W, int bf16, std::vector<KernelLaunch>* out) {
  IngestArgs a{x, y, C, Cs, H * W};
  const size_t total = (size_t)H * W * Cs;
  return push(out, kt.ingest[bf16], K_INGEST, (uint32_t)((total + 255) / 256), 256, &a, kIngestBytes);
}
bool encode_egress(const KernelTable& kt, const void* x, float* y, int C, int Cs, int H, int W, int bf16, std::vector<KernelLaunch>* out) {
  IngestArgs a{x, y, C, Cs, H * W};
  const size_t total = (size_t)H * W * C;
  return push(out, kt.egress[bf16], K_EGRESS, (uint32_t)((total + 255) / 256), 256, &a, kIngestBytes);
}
bool encode_cu_probe(const KernelTable& kt, uint32_t* out_dev, int n_groups, int spin, std::vector<KernelLaunch>* out) {
  ProbeArgs a{out_dev, spin};
  return push(out, kt.cu_probe, K_NONE, (uint32_t)n_groups, 64, &a, kProbeBytes);
}

}  // namespace daris
