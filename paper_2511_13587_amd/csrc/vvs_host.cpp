// Host side of libvvs: argument validation, buffer planning, tree tables and the C ABI entry
// points.  Everything here runs before any launch, so bad input never reaches a kernel.
#include "vvs_internal.h"

#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

namespace vvs {

constexpr size_t kStreamed = (size_t)24 << 20;   // bytes of a weight matrix from which on it is streamed rather than held near the CUs

static std::string g_last_error;   // for failures that have no context (query / create)

static vvs_status fail(std::string* err, vvs_status st, const std::string& msg) {
  if (err) *err = msg;
  g_last_error = msg;
  return st;
}

// Every launch of a projection and every prefetch of its weights takes its tiles from here (or from plan_resid), so that the two
// cannot disagree about which XCD reads which weight tile.
//
// Tiles whose operands are shared through LDS (k_gemm_shared_dma).  A CU is filled at about 64 GB/s whatever the tile, so a stage of 32
// contraction values costs about 1 ns per tile row and column until the matrix cores are the slower side (256 x 256); start and
// epilogue cost every round of tiles again, by the tile's area and what is written; a launch lasts as many rounds as its fullest CU works
// through, and no less than its weights take from HBM (6 TB/s).  The tile of least cost is taken.  us per launch, measured / by this
// table, at 3904 and 1920 rows of d 1280, d_ff 3456 and 388 of d 4096, d_ff 11008:
//   gate/up  128 x 128: 85, 44, 114 / 80, 44, 103   192 x 128: 100, 56, 133 / 96, 57, 139   256 x 128: 98, 48, 116 / 95, 48, 115   256 x 256: 79, 41, 94 / 80, 40, 95
//   q/k/v    128 x 128: 61, 30, 68 / 60, 30, 68     192 x 128: 76, 45, 99 / 77, 51, 106     256 x 128: 67, 34, 68 / 65, 33, 66     256 x 256: 57, 51, 98 / 58, 58, 112
// Launches of a d 4096 step with the rule before (64-row tiles up to 192 rows) / with this one: 126 rows gate/up 57.8 / 49.8 (128 x 128), O and
// down, mean, 22.4 / 21.4 (128 x 64, K in 4); 388 rows gate/up 112 / 94.6 (256 x 256), O 26 / 23.6, down 66 / 49.2 (both 128 x 128, K in 2).
static GemmPlan plan_shared(int M, int N, int K, int section, bool may_split, int min_bn) {
  struct Tile { int bm, bn; double stage, lone; bool pair; };      // pair: two workgroups fit a CU; lone: one of such a pair by itself
  static const Tile tiles[] = {{256, 256, 0.62, 0.62, false}, {256, 128, 0.385, 0.385, false}, {192, 128, 0.31, 0.31, false},
                               {192, 64, 0.23, 0.23, false},   {128, 128, 0.245, 0.245, false}, {128, 128, 0.215, 0.34, true},
                               {128, 64, 0.19, 0.19, true},    {64, 128, 0.21, 0.21, true},     {64, 64, 0.155, 0.155, true}};
  const double area = section ? 4.8e-4 : min_bn > 64 ? 2.1e-4 : 4.5e-4;   // us per value: q/k/v in cache order, one bf16 for two, fp32
  const int rows = (int)align_up(M, 32), nst = K / 32;             // limits on multiples of 32 rows (plan_sizes)
  const double stream = 2e-6 * N * K / 6.0, again = may_split ? 4e-6 * rows * N / 5.0 : 0.0;   // the weights from memory; the sums read again, per share
  GemmPlan best{0, 0, 1};
  double least = 1e30;
  for (const Tile& t : tiles) {
    if (t.bn < min_bn || N % t.bn || section % t.bn) continue;
    const int n = (rows + t.bm - 1) / t.bm * (N / t.bn);
    const double once = 1.5 + area * t.bm * t.bn;                  // start and epilogue
    const double even = std::max(t.stage * nst * n * (1.0 / 256), stream) + 1.5;   // no launch is shorter than its stages dealt evenly to all CUs
    for (int want = 1; want <= (may_split ? 8 : 1); ++want) {
      if ((want > 1 && n * (want - 1) >= 512) || even + want * again > least) break;   // two rounds of tiles need no further shares
      const int per = (nst + want - 1) / want, splits = (nst + per - 1) / per, all = n * splits;
      if (splits != want || (splits > 1 && per < 16)) continue;
      // 128 x 128 stands twice: 8 slots, one workgroup per CU, for a single round; 4 slots, two per CU, for more
      if (t.bm == 128 && t.bn == 128 && t.pair != (all > 256)) continue;
      double us;
      if (t.pair && all > 256) {                                   // rounds of two per CU; a rest of up to one per CU runs beside the others' epilogues
        const int pairs = all / 512 + (all % 512 > 256), rest = all % 512 > 256 ? 0 : all % 512;
        us = pairs * (2 * t.stage * per + 1.5 + 1.45 * area * t.bm * t.bn) + (rest ? t.lone * per : 0.0);
      } else {
        us = (all + 255) / 256 * (t.stage * per + once);
      }
      us = std::max(us, stream + once) + again * splits;
      if (us <= least) { least = us; best = GemmPlan{t.bm, t.bn, splits, false, true}; }
    }
  }
  return best;
}

// Beyond 512 tiles of 64 x 64 some CUs work through a third of them (as at plan_resid), whichever the projection.  us per pass, own / shared
// operands: d 768, 12 heads, 4 layers, 960 to 1024 rows (540 to 576 q/k/v tiles) 387 / 366 and 400 / 373, 880 rows (504) 347 / 348; d 512, 1584
// rows 704 / 647; d 1024, 672 rows 708 / 654; a prefix of d 1280 with 520 tiles 494 / 449.  (At 160 tiles of 128 x 128, where the line stood, calls of
// 896 to 1024 rows of d 768 with more (head, prompt) pairs than CUs had become up to 3.8 % slower when their projection left the attention's launch.)
// Large weights: from one row-block's end on, and with up to 32 rows where the contraction is long enough that a tile's stages outweigh its ramp.
// Step of 4 to 32 rows, shared against own operands: d 1536 (d_ff 4096) +4.5 to +2.5 %, 1792 (4864) +1.5 to -0.5, 2048 (5504) -0.8 to -4.2, 2560 (6912)
// -4.1 to -6.1, 4096 (11008) -7.5 to -1.8.
static bool takes_shared(int M, int N, int K) {
  return N % 128 == 0 && ((M > 192 && ((M + 63) / 64) * (N / 64) > 512) || ((size_t)N * K * 2 >= kStreamed && (M > 32 || K >= 2048)));
}

// Tiles whose waves stream operands of their own: 64 x 64 (32 x 64 for up to 32 rows); every workgroup already splits its K range over its 4
// waves.  Add grid-level K splits until there is about one workgroup per CU, keeping at least 8 k-steps of 16 per wave.
static GemmPlan plan_own(int M, int N, int K) {
  GemmPlan p{M <= 32 ? 32 : 64, 64, 1};
  // 64 x 128 tiles when they give one workgroup for (nearly) every CU and no second round: a CU then
  // pulls (64 + 128) K-rows through its L1 instead of 2 x (64 + 64)
  if (p.bm == 64 && N % 128 == 0) {
    const int t128 = ((M + 63) / 64) * (N / 128);
    if (t128 >= 160 && t128 <= 256) { p.bn = 128; return p; }
  }
  // up to 32 rows (weight streaming): 32 x 128 tiles under the same condition - with 64-column tiles such an
  // N gives between one and two workgroups per CU, and the kernel lasts as long as the CUs that got two
  if (p.bm == 32 && N % 128 == 0 && N / 128 >= 160 && N / 128 <= 256) { p.bn = 128; return p; }
  const int tiles = ((M + p.bm - 1) / p.bm) * (N / 64);
  const int kb = K / 16;
  if (tiles < 256) {
    const int want = std::min({(256 + tiles - 1) / tiles, 8, std::max(1, kb / 32)}), per = (kb + want - 1) / want;
    p.splits = (kb + per - 1) / per;
  }
  return p;
}

GemmPlan plan_gemm(const Ctx* c, int M, int N, int K, int section, bool may_split, int min_bn) {
  if (c->cfg.dtype != VVS_BF16) return GemmPlan{64, 64, 1};   // fp32 path: one wave per output column, no split
  // Operands shared through LDS where a launch has many 128 x 128 tiles, or where the weights are large and the rows more than one
  // row-block: a CU then has whole rows of stages to work through, and each weight byte feeds twice the MFMAs
  return takes_shared(M, N, K) ? plan_shared(M, N, K, section, may_split, min_bn) : plan_own(M, N, K);
}

// A projection that leaves partial sums for the kernel behind it (run_gemm)
GemmPlan plan_partial(const Ctx* c, int M, int N, int K) { return plan_gemm(c, M, N, K, 0, true); }

// q/k/v: 32 x 32 tiles on 8 waves while every tile has a CU of its own - a launch of few tiles lasts as long as one CU takes to pull its
// operands in.  us per launch, 64 x 64 on 4 waves / 32 x 32 on 8: d 1280, 54 rows 10.2 / 9.0 (240 tiles); a step of 96 rows (360 tiles) 1823 / 1913.
bool qkv_small_tiles(const Ctx* c, int M) {
  return c->cfg.dtype == VVS_BF16 && (size_t)6 * c->d * c->d < kStreamed && (M + 31) / 32 * (3 * c->d / 32) <= 256;
}
GemmPlan plan_qkv(const Ctx* c, int M) {
  if (qkv_small_tiles(c, M)) return GemmPlan{32, 32, 1};
  return plan_gemm(c, M, 3 * c->d, c->d, c->d);
}
// Gate/up of large weights on tiles with operands of their own.  A shared tile holds gate and up of its hidden units in one wave, 128 columns; its
// own has 64, so where these are one round of CUs the shared ones leave half of the CUs idle; and with up to 32 rows (both read one
// row-block) three 64-column tiles on the fullest CU are less than two of 128.  us per layer, shared / own whole sums / own split:
//   one round:  d 2048, d_ff 4096, 14 rows 67.0 / 62.3 / 65.7, 96 rows 71.7 / 69.0; d 2560, d_ff 5120, 64 rows 85.9 / 81.6 / 86.8; d 3072, d_ff 6144, 30 rows 94.3 /
//     87.2 / 91.9; d 4096, d_ff 8192, 30 rows 122.5 / 115.0, 40 rows 133.8 / 125.4; d_ff 4096, 30 rows 108.8 / 100.7 / 100.7, 40 rows 121.6 / 114.4 / 111.7
//   two:        d 3072, d_ff 8256, 28 rows 97.2 / 100.5; d 4096, d_ff 11008, 28 rows 124.6 / 125.1; d 2560, d_ff 5120, 96 rows 90.3 / 91.3
//   three:      d 4096, 2 layers, 30 rows, d_ff 18432 359 / 339, 20480 369 / 358; four: d_ff 32768 450 / 450
static int gate_up_own_tiles(const Ctx* c, int M) { return (M <= 32 ? 1 : (M + 63) / 64) * (2 * c->F / 64); }
static bool gate_up_own(const Ctx* c, int M) {
  const int n = gate_up_own_tiles(c, M);
  return c->cfg.dtype == VVS_BF16 && (n <= 256 || (M <= 32 && n > 512 && n <= 768));
}
GemmPlan plan_gate_up(const Ctx* c, int M) {
  const int N = 2 * c->F, K = c->d;
  if (!takes_shared(M, N, K) || !gate_up_own(c, M)) return plan_gemm(c, M, N, K, 0, false, 128);
  GemmPlan p = plan_own(M, N, K);
  // whole sums, unless half of the CUs have no tile and the contraction is long.  30 rows, whole / split: d 4096, d_ff 2048 (64 tiles) 94.9 / 91.5, d 8192,
  // d_ff 4096 (128) 217 / 209; d 3584, d_ff 3584 (112) 90.4 / 91.9; d 3072, d_ff 6144 (192) 87.2 / 91.9, d 4096, d_ff 5504 (172) 104 / 108
  if (gate_up_own_tiles(c, M) > 128 || K < 4096) p.splits = 1;
  return p;
}

// The projections that end in the residual epilogue (fused layer: O, down, a drafter's input map); d columns.
GemmPlan plan_resid(const Ctx* c, int M) {
  const int d = c->d;
  // many rows: 192 x 128 tiles with the operands shared through LDS (a quarter of the bytes per flop that 64 x 64 tiles pull
  // through a CU's L1), when they give most CUs a tile - at d = 1280 and 3904 rows: 210 tiles, one round.
  // Tile order by fabric traffic: the operand an XCD does not own is fetched by all 8 of them (M + 8 d rows against 8 M + d)
  if (d % 128 == 0 && ((M + 191) / 192) * (d / 128) >= 160) return GemmPlan{192, 128, 1, M > d, true};
  // Two 64 x 64 workgroups fit a CU, so up to 512 of them run at once; beyond that some CUs work through a third tile while the
  // others wait, and 128 x 128 tiles through LDS, which leave 90 to 130 CUs without a tile, are the better choice.  us per launch, mean of
  // O and down, 64 x 64 / 128 x 128:
  //   d 1280, d_ff 3456: 864 rows (280 tiles of 64 x 64) 17.9 / 28.7, 1296 (420) 22.0 / 27.3, 1586 (500) 24.1 / 29.0, 1620 (520) 29.3 / 30.3,
  //                      1728 (540) 30.7 / 29.1, 1920 (600) 33.2 / 30.8, 2304 (720) 37.7 / 31.8, 2560 (800) 44.7 / 32.0
  //   d 768, d_ff 2048:  2560 rows (480) 17.9 / 21.3, 2720 (516) 21.0 / 21.5, 2880 (540) 22.5 / 21.8, 3840 (720) 26.7 / 23.5
  //   d 1024, d_ff 2816: 2048 rows (512) 23.4 / 26.6, 2160 (544) 29.0 / 26.7;  d 1408, d_ff 3840: 1392 (484) 25.0 / 32.4, 1488 (528) 31.8 / 32.0,
  //   1568 (550) 32.8 / 30.8;  d 1536, d_ff 2048: 1280 (480) 19.6 / 25.2, 1360 (528) 24.1 / 24.9, 1440 (552) 25.0 / 24.2
  // (A whole pass is faster from 513 tiles on also where the two are level: the launches before have CUs free to read ahead.)
  // Column tiles per XCD: the transposed order took 3 % less (d 768, 3520 rows: 22.9 -> 22.2) to 2 % more (d 1280, 1920 rows: 30.8 -> 31.4).
  if (d % 128 == 0 && ((M + 63) / 64) * (d / 64) > 512) return GemmPlan{128, 128, 1, false, true};
  // 32 x 32 tiles on 8 waves while that gives at most 448 workgroups - a launch of few tiles lasts as long as one CU takes to
  // pull its operands in, so smaller tiles on more CUs win until two workgroups share most CUs - else 64 x 64 on 4.  us per launch,
  // O and down mean, 64 x 64 on 4 waves / 32 x 32 on 8: d 768, 48 rows 7.3 / 4.9; d 1280, 54 rows 10.4 / 7.2, 300 rows (400 tiles)
  // 10.8 / 10.1, 432 rows (560 tiles) 11.5 / 14.3.  (32 x 64 and 64 x 32 on 8 waves lie between.)
  const int bm = ((M + 31) / 32) * (d / 32) <= 448 ? 32 : 64;
  return GemmPlan{bm, bm, 1};
}

// The fused layer (5 kernels, no separate normalisation) is taken when a layer's weights are so small (below
// ~48 MB: the B and XL widths, a drafter) that a launch costs more than streaming them: then fewer launches
// win.  Wide layers stream their weights through K-split GEMMs with separate normalisation kernels, which
// also round the norm's output where the definition does: the other placement costs more accuracy the wider
// the layer is (measured without any kernel: 2 x the noise floor of a correct bf16 evaluation at d = 1280,
// 3 x at d = 4096).
bool plan_fused(const Ctx* c, int M) {
  (void)M;
  if (c->cfg.dtype != VVS_BF16 || c->cfg.norm_mode == VVS_NORM_SEPARATE) return false;
  const size_t layer_weight_bytes = c->esz * ((size_t)4 * c->d * c->d + (size_t)3 * c->d * c->F);
  return layer_weight_bytes <= ((size_t)48 << 20);
}

// Where the gain of the one launch (vvs_few.hip) ends: 192 rows; with up to 64 (head, prompt) pairs, which leave most CUs idle in the launch of projection and
// attention, 224, and 256 at d 512, whose weights fit the L2s.  us per step, a launch each / one launch (8 layers; XL whole):
//   d 768, 200 rows (48 pairs) 286 / 260, (24) 327 / 258, 256 rows (48) 290 / 296;  d 1280, 220 rows (40) 492 / 452, 210 (60) 479 / 450, 240 (60) 495 / 515, 256 (40) 500 /
//   520;  d 1024, 216 rows (64) 402 / 339, 256 (32) 332 / 359;  d 512, 252 rows (48) 253 / 209, 256 (16) 297 / 202, 240 (64) 241 / 203;  d 1536, 200 rows (48) 500 / 491;
//   XL, 216 rows (80 pairs) 2079 / 2071, 256 (320) 2366 / 2598
// Gate/up tiles of 32 rows x 48 hidden units fill the CUs in more and more rounds as d_ff grows, each pulling its operands anew, so the line falls with
// its square.  12 layers, one launch / a launch each by time (more than 1: the one launch is slower), at the last row-block taken and behind:  d 768, d_ff
// 7680 160 rows 0.93, 192 1.01 to 1.03; 8192 120 rows 1.00, 144 1.01; 9216 128 rows 1.06;  d 640, 10240 64 rows 0.97, 100 1.16;  d 704, 9856 64 rows 0.96, 120 1.12;
// d 512, 12288 64 rows 1.03, 100 1.20;  inside: d 896, 7168 192 rows 0.93, d 1024, 6144 192 rows 0.99 to 1.01.
// Head size 64: its q/k/v tiles are a head's.
int few_rows(const Ctx* c) {
  // (a narrow drafter has one layer to save launches in: 1 prompt x 4 nodes, us, a launch each / one launch, d 64 142 / 150, 128 146 / 152, 192 151 / 154, 256 158 / 155, 512
  // 174 / 166)
  if (!plan_fused(c, c->R) || c->dh != 64 || (c->cfg.draft_input && c->d < 256)) return 0;
  const int blocks = std::max(1, (int)(310000000 / ((long)c->F * c->F)));
  const int most = std::min((long)32 * blocks, (long)(c->H * c->B > 64 ? 192 : c->d <= 512 ? 256 : 224));
  const int tokens = c->cfg.draft_input ? c->Tmax : std::max(c->Tmax, std::min(c->chunk, (int)VVS_MAX_T));   // the longest call of either kind
  return std::min((int)align_up((size_t)c->R * tokens, 32), most);
}

// Wide layers.  us per layer, a launch each / one launch:
//   up to 32 rows:  24 and 32 rows, d 1536 (d_ff 4096) 52.4 / 35.1, 2048 (5504) 59.3 / 45.4, 3072 (8192) 84.9 / 72.0, 4096 (4096) 90.8 / 82.8, (11008) 115 / 102,
//     (12288, 436 MB a layer) 117.5 / 111.8, but (14336, 486 MB) 130 / 133 and (16384) 134 / 136: gate/up tiles in a second round
//   64 rows:   d 1536 58.4 / 40.9, 2048 65.1 / 51.4, 2560 (6912) 81.5 / 78.6, 3072 94.5 / 89.4, 4096 130 / 123;  40 rows, d 2560 77.1 / 77.0, 3072 88.7 / 89.7, 4096 125 / 119
//   96 rows:   d 1536 61.6 / 52.6, 2048 67.7 / 63.6, (8192, 134 MB) 77.8 / 79.0, 2560 89.1 / 104;  128 rows, d 1536 66.7 / 54.5, (8192, 94 MB) 74.1 / 71.1, 2048
//     75.1 / 69.2, (8192) 84.6 / 86.4, 3072 117 / 140
// Few and many hidden units, us per call of 2 to 7 layers, a launch each / one launch:
//   33 to 64 rows, d above 2048, gate/up of two row-blocks to a tile in a second round (d_ff 12800 and more):  d 2176 (13056) 217 / 238, 2560 (12800) 231 / 253, 3072 (13824)
//     268 / 300, 3840 (12800) 306 / 338, 2304 (24576) 284 / 297, 2816 (20480) 316 / 312; one round: 4096 (12288) 318 / 312
//   the same, few hidden units, where normalisation and attention are most of a layer:  3584 (1024) 0.97 to 0.99, 3840 (1536) 0.97 to 0.99 of the one launch's time, 4096
//     (1024) 317 / 326, (1536) 0.94 to 0.95, (2048) 332 / 336; inside: 3840 (1920) 1.22, (2048) 314 / 331, 3328 (832) 1.06, 4096 (3072) 261 / 251
//   up to 32 rows, d 3584 (12544) 254 / 264, 3840 (12800) 271 / 280, (13440) 265 / 274; 3520 (13440) 279 / 263
//   33 to 64 rows, d up to 2048:  1792 (23040) 251 / 249, (25088) 243 / 258;  65 to 128: 960 (9600) 1.03 of its time, (11520) 0.95 to 0.99, (13440) 442 / 510, 1024 (11264) 0.97, 1152
//     (13440) 356 / 398, 768 (6144) 570 / 543, (7680) 589 / 634, 896 (8960) 541 / 570, 1024 (8192) 1.14, (10240) 484 / 494, 1280 (10240) 1.02 (O and down share
//     their operands through LDS where d is a multiple of 128)
int few_wide_rows(const Ctx* c) {
  if (plan_fused(c, c->R) || c->cfg.dtype != VVS_BF16 || c->cfg.draft_input || c->d > 4096) return 0;
  const size_t layer_weight_bytes = c->esz * ((size_t)4 * c->d * c->d + (size_t)3 * c->d * c->F);
  const int d = c->d, F = c->F;
  if (layer_weight_bytes > (size_t)440 << 20 || (d >= 3584 && F > 12288)) return 0;
  int most = 32;
  if (d > 2048) {
    if (F <= 12288 && F > (d > 4032 ? 2048 : d > 3456 ? 1536 : 0)) most = 64;
  } else if (F <= 23040) {
    most = layer_weight_bytes <= (size_t)104 << 20 && (F <= 7168 || (d >= 896 && F < 11264 && F <= (d % 128 ? 10 : 8) * d)) ? 128 : 64;
  }
  return std::min((int)align_up((size_t)c->R * c->Tmax, 32), most);
}

// (More than VVS_MAX_T tokens have no masks.  A device of fewer CUs, a partition of the chip, never has all workgroups running: every launch would wait
// for them in vain, and nothing above was measured there.)
bool layers_in_one_launch(const Ctx* c, int T) {
  return c->cus >= kFewGroups && T <= VVS_MAX_T && c->R * T <= std::max(few_rows(c), few_wide_rows(c));
}

vvs_status plan_sizes(const vvs_config* cfg, Ctx* c, std::string* err) {
  if (!cfg) return fail(err, VVS_EINVAL, "config is NULL");
  const vvs_config& g = *cfg;
  if (g.n_layers < 1 || g.d_model < 4 || g.n_heads < 1 || g.d_ff < 1 || g.vocab < 1 || g.n_prompts < 1 ||
      g.grid_h < 1 || g.grid_w < 1 || g.prefix_len < 1 || g.max_nodes < 0)
    return fail(err, VVS_EINVAL, "config: a dimension is not positive");
  if (g.d_model % g.n_heads) return fail(err, VVS_EINVAL, "config: d_model is not a multiple of n_heads");
  if (g.logit_lo < 0 || g.logit_hi > g.vocab || g.logit_lo >= g.logit_hi)
    return fail(err, VVS_EINVAL, "config: logit slice must satisfy 0 <= lo < hi <= vocab");
  if (g.dtype != VVS_FP32 && g.dtype != VVS_BF16) return fail(err, VVS_EINVAL, "config: unknown dtype");
  if (g.prefix_kind != VVS_PREFIX_CLASS && g.prefix_kind != VVS_PREFIX_DENSE)
    return fail(err, VVS_EINVAL, "config: unknown prefix_kind");
  if (g.prefix_kind == VVS_PREFIX_CLASS && g.n_classes < 1) return fail(err, VVS_EINVAL, "config: n_classes < 1");
  if (g.max_nodes > VVS_MAX_T - 1) return fail(err, VVS_ESIZE, "config: max_nodes exceeds VVS_MAX_T - 1");
  if (g.relax_k < 0 || g.relax_k > 64) return fail(err, VVS_ESIZE, "config: relax_k must be in [0, 64]");
  if (!(g.relax_delta >= 0.f)) return fail(err, VVS_EINVAL, "config: relax_delta < 0");
  if (!(g.rms_eps > 0.f) || !(g.rope_base > 1.f)) return fail(err, VVS_EINVAL, "config: rms_eps / rope_base");
  if (g.feature_slots < 0 || g.feature_slots > VVS_MAX_FEATURE_SLOTS)
    return fail(err, VVS_ESIZE, "config: feature_slots must be in [0, VVS_MAX_FEATURE_SLOTS]");
  if (g.feature_pre_norm != 0 && g.feature_pre_norm != 1) return fail(err, VVS_EINVAL, "config: feature_pre_norm must be 0 or 1");
  if (g.draft_input != 0 && g.draft_input != 1) return fail(err, VVS_EINVAL, "config: draft_input must be 0 or 1");
  if (g.norm_mode != VVS_NORM_AUTO && g.norm_mode != VVS_NORM_SEPARATE) return fail(err, VVS_EINVAL, "config: unknown norm_mode");
  int dh = g.d_model / g.n_heads;
  if (dh % 4) return fail(err, VVS_ESIZE, "config: head size must be a multiple of 4 (2D rotary pairs)");
  if (g.d_model % 8 || g.d_ff % 8) return fail(err, VVS_ESIZE, "config: d_model and d_ff must be multiples of 8");
  if (g.d_model > 16384) return fail(err, VVS_ESIZE, "config: d_model above 16384 is not supported");
  if (dh > 256) return fail(err, VVS_ESIZE, "config: head size above 256 is not supported");
  int veff = g.logit_hi - g.logit_lo;
  if (g.dtype == VVS_BF16) {
    if (g.d_model % 64 || g.d_ff % 64 || veff % 64)
      return fail(err, VVS_ESIZE, "config: bf16 needs d_model, d_ff and the logit slice width to be multiples of 64");
    if (dh != 64 && dh != 128) return fail(err, VVS_ESIZE, "config: bf16 needs head size 64 or 128");
    if (dh == 128 && g.max_nodes > 31) return fail(err, VVS_ESIZE, "config: bf16 with head size 128 supports max_nodes <= 31");
  }
  c->cfg = g;
  c->B = g.n_prompts; c->R = 2 * g.n_prompts; c->d = g.d_model; c->H = g.n_heads; c->dh = dh; c->F = g.d_ff;
  c->L = g.n_layers; c->V = g.vocab; c->lo = g.logit_lo; c->veff = veff; c->P = g.prefix_len;
  c->G = g.grid_h * g.grid_w; c->Tmax = g.max_nodes + 1;
  // Prefill runs in chunks of this many tokens per row.  bf16: as many as give about 4096 GEMM rows (at least 64, at most 512
  // tokens), so that a prefix is one pass over the weights and the projections run in their many-row shapes: beyond 4096
  // rows they gain nothing more and the workspace only grows.  fp32: 64, the width of the plain attention kernel's masks.
  // Never more than the longest prefill there is (the prefix and all image tokens but one).
  c->chunk = g.dtype == VVS_BF16 ? std::min(512, std::max(64, 4096 / c->R / 32 * 32)) : (dh > 64 ? 32 : 64);
  c->chunk = std::min(c->chunk, c->P + c->G - 1);
  // Rows of the activations: the widest verify or drafting call, its tokens padded to the 32 or 64 rows that each row takes in the
  // operand of the fused projection + attention launch, or a prefill chunk; a drafter context never prefills.  Packed operands come
  // in blocks of 32 rows.
  const int call = (int)align_up(c->Tmax, 32);
  c->Mmax = (int)align_up((size_t)c->R * (g.draft_input ? call : std::max(call, c->chunk)), 32);
  c->Mlog = (int)align_up((size_t)c->R * c->Tmax, 32);
  c->S_cap = (int)align_up((size_t)c->P + c->G + VVS_MAX_T, 32);
  c->rope_pos = std::max(g.grid_h + VVS_MAX_T / g.grid_w + 2, g.grid_w);
  c->esz = g.dtype == VVS_BF16 ? 2 : 4;
  // KV cache: K [L][R][H][S_cap][dh], then V [L][R][H][S_cap/32][dh][32]
  c->kv_head_stride = (size_t)c->S_cap * dh;
  c->kv_row_stride = c->kv_head_stride * c->H;
  c->kv_layer_stride = c->kv_row_stride * c->R;
  c->kv_v_off = c->kv_layer_stride * c->L;
  // GEMM partial-sum buffer: worst case over every M this context can be asked for, projection by projection, each with the plan that its
  // launch takes (run_gemm; told apart by their sizes, two with the same columns or contraction would get one plan).  Sums that come whole
  // are written by the projection's own epilogue where it has one.  All limits of a plan lie on multiples of 32 rows, so the largest M of
  // each block of 32 stands for the block.
  size_t go = 0;
  const int d = c->d, F = c->F;
  for (int M = c->Mmax; M >= 32; M -= 32) {                // (downwards: few rows can only need more by many shares of 15 stages and more)
    auto sums = [&](int N, int K) {
      if ((size_t)std::min(8, K / 32 / 15 + 1) * M * N > go) go = std::max(go, (size_t)plan_partial(c, M, N, K).splits * M * N);
    };
    const bool bf16 = g.dtype == VVS_BF16;
    if (!bf16 || (!takes_shared(M, 3 * d, d) && plan_qkv(c, M).splits > 1)) sums(3 * d, d);   // (the shared-operand tiles of the two: whole sums)
    if (!bf16 || !takes_shared(M, 2 * F, d) || gate_up_own(c, M)) {
      const int shares = plan_gate_up(c, M).splits;
      if (!bf16 || shares > 1) go = std::max(go, (size_t)shares * M * 2 * F);
    }
    sums(d, d);                              // O
    sums(d, F);                              // down
    if (g.draft_input) sums(d, 2 * d);       // a drafter's input map
  }
  // workspace carve-up
  Workspace& w = c->w;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, 256); return o; };
  w.state = take(sizeof(int32_t) * 3 * c->B);
  w.ring_state = take(sizeof(int32_t) * 2 * c->R);        // per row: features held, slot of the oldest (zeroed with the state)
  w.outcome = take(sizeof(int32_t) * c->B * kOutcomeInts);
  w.node_result = take(sizeof(int32_t) * c->B * VVS_MAX_T * 2);
  w.tokens = take(sizeof(int32_t) * c->B * VVS_MAX_T);
  w.rope_tab = take(sizeof(float) * 2 * c->rope_pos * (dh / 4));
  w.walk_sync = take(sizeof(uint32_t) * kWalkLine * c->B);      // zeroed with the state
  w.few_gave_up = w.walk_sync + sizeof(uint32_t);               // (a line has room for it behind its counter)
  c->gemm_out_elems = go;
  const int wide = few_wide_rows(c), few = std::max(few_rows(c), wide);
  go = std::max(go, (size_t)kFewWideShares * wide * d);
  w.few_sync = take(few ? sizeof(uint32_t) * kFewLine * (kFewHead + (size_t)few_layer_counters(c->H, few / 32) * c->L + 8) : 0);   // zeroed with the state
  w.x = take(sizeof(float) * (size_t)c->Mmax * d);
  w.h = take(c->esz * (size_t)c->Mmax * d);
  // (a call whose layers are one launch has no partial sums: what its phases hand on lies in their place)
  w.gemm_out = w.few_buf = take(std::max(sizeof(float) * go, wide ? 0 : few_buf_bytes(few, d, F) * c->L));
  if (wide) w.few_buf = take(few_buf_bytes(few, d, F) * c->L);
  w.q = take(c->esz * (size_t)c->Mmax * d);
  w.attn = take(c->esz * (size_t)c->Mmax * d);
  w.act = take(c->esz * (size_t)c->Mmax * F);
  w.hf = take(c->esz * (size_t)c->Mlog * d);
  w.logits = take(sizeof(float) * (size_t)c->Mlog * veff);
  w.probs = take(sizeof(float) * (size_t)c->B * c->Tmax * veff);
  w.pq_work = take(sizeof(float) * (size_t)c->B * c->Tmax * 2 * veff);
  w.ss = take(sizeof(float) * (size_t)c->Mmax * n_slabs(d));     // per-row, per-slab sums of squares of the residual
  w.ss2 = take(sizeof(float) * (size_t)c->Mlog * n_slabs(d));
  w.ring = take(c->esz * (size_t)c->R * std::max(g.feature_slots, 1) * d);
  w.din = take(g.draft_input ? c->esz * (size_t)c->Mmax * 2 * d : 0);                // drafter: [embedding ; feature] rows
  w.total = off;
  // packed weights
  PackedLayout& p = c->p;
  off = 0;
  size_t e = c->esz;
  p.embed = take(e * (size_t)c->V * d);
  p.prefix_embed = take(e * (size_t)(g.n_classes + 1) * d);
  p.gf = take(sizeof(float) * d);
  p.wout = take(e * (size_t)veff * d);
  p.layer0 = off;
  size_t base = off;
  p.g1 = take(sizeof(float) * d) - base;
  p.wqkv = take(e * (size_t)3 * d * d) - base;
  p.wo = take(e * (size_t)d * d) - base;
  p.g2 = take(sizeof(float) * d) - base;
  p.wgu = take(e * (size_t)2 * F * d) - base;
  p.wd = take(e * (size_t)d * F) - base;
  p.layer_stride = off - base;
  off = p.layer0 + p.layer_stride * c->L;
  p.fc = take(g.draft_input ? e * (size_t)2 * d * d : 0);
  p.total = off;
  return VVS_OK;
}

// Validates the topology and fills the kernel-side tables.
vvs_status build_tree(int n_nodes, const int32_t* h_parent, const uint8_t* h_mask, TreeDesc* t, std::string* err) {
  if (n_nodes < 0 || n_nodes > VVS_MAX_T - 1) return fail(err, VVS_ESIZE, "tree: n_nodes out of range");
  const int T = n_nodes + 1;
  std::vector<int> par(T, -1);
  if (h_parent) {
    for (int j = 1; j < T; ++j) {
      int p = h_parent[j - 1];
      if (p < 0 || p > j - 1) return fail(err, VVS_EINVAL, "tree: parent of node j must lie in [0, j-1]");
      par[j] = p;
    }
  } else if (h_mask) {
    // the parent is the closest proper ancestor = the largest index among them
    for (int j = 1; j < T; ++j) {
      int p = -1;
      for (int i = 0; i < j; ++i) if (h_mask[(size_t)j * T + i]) p = i;
      if (p < 0) return fail(err, VVS_EINVAL, "tree mask: a node does not see the root");
      par[j] = p;
    }
  } else {
    for (int j = 1; j < T; ++j) par[j] = j - 1;
  }
  memset(t, 0, sizeof(*t));
  t->T = T;
  bool chain = true;
  for (int j = 0; j < VVS_MAX_T; ++j) { t->parent[j] = -1; t->first_child[j] = -1; t->next_sibling[j] = -1; }
  std::vector<int> last_child(T, -1);
  for (int j = 0; j < T; ++j) {
    uint64_t m = 1ull << j;
    if (j) {
      t->parent[j] = (int8_t)par[j];
      t->depth[j] = (int8_t)(t->depth[par[j]] + 1);
      m |= t->anc[par[j]];
      if (par[j] != j - 1) chain = false;
      if (last_child[par[j]] < 0) t->first_child[par[j]] = (int8_t)j;
      else t->next_sibling[last_child[par[j]]] = (int8_t)j;
      last_child[par[j]] = j;
    }
    t->anc[j] = m;
  }
  t->causal = chain ? 1 : 0;
  if (h_mask) {
    for (int i = 0; i < T; ++i)
      for (int j = 0; j < T; ++j) {
        bool want = (t->anc[i] >> j) & 1ull;
        if ((h_mask[(size_t)i * T + j] != 0) != want)
          return fail(err, VVS_EINVAL, "tree mask is not the ancestor-or-self closure of the parent array");
      }
  }
  return VVS_OK;
}

static void causal_tree(int T, TreeDesc* t) {
  memset(t, 0, sizeof(*t));
  t->T = T;
  t->causal = 1;
  for (int j = 0; j < VVS_MAX_T; ++j) { t->parent[j] = (int8_t)(j - 1); t->first_child[j] = -1; t->next_sibling[j] = -1; }
  for (int j = 0; j < T && j < VVS_MAX_T; ++j) {
    t->depth[j] = (int8_t)j;
    t->anc[j] = (j == 63) ? ~0ull : ((1ull << (j + 1)) - 1);
  }
}

// Such a kernel has to be allowed to, once per device: remembers per (kernel, device) that it has been done.  Contexts may be used on threads of their own.
void allow_dynamic_lds(const void* kernel, size_t bytes) {
  struct Done { const void* fn; int dev; };
  static std::mutex lock;
  static std::vector<Done> done;
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::lock_guard<std::mutex> hold(lock);
  for (const Done& d : done)
    if (d.fn == kernel && d.dev == dev) return;
  // a failure shows up as an invalid-configuration error of the launch that follows
  (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  done.push_back(Done{kernel, dev});
}

static vvs_status hip_fail(Ctx* c, hipError_t e, const char* what) {
  return fail(&c->err, VVS_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

static vvs_status check_launch(Ctx* c, const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(c, e, what);
  return VVS_OK;
}

// Where the forward of T tokens per row that was just launched says that it is not whole (nullptr: it has no waits that could give up)
static const uint32_t* gave_up(const Ctx* c, int T) { return layers_in_one_launch(c, T) ? (const uint32_t*)(c->ws + c->w.few_gave_up) : nullptr; }

}  // namespace vvs

using namespace vvs;

extern "C" {

vvs_status vvs_query_sizes(const vvs_config* cfg, size_t* kv_bytes, size_t* workspace_bytes, size_t* packed_weight_bytes) {
  Ctx c{};
  vvs_status st = plan_sizes(cfg, &c, nullptr);
  if (st != VVS_OK) return st;
  if (kv_bytes) *kv_bytes = 2 * c.kv_v_off * c.esz;
  if (workspace_bytes) *workspace_bytes = c.w.total;
  if (packed_weight_bytes) *packed_weight_bytes = c.p.total;
  return VVS_OK;
}

int32_t vvs_plan_is_fused(const vvs_ctx* ctx, int32_t n_tokens) {
  const Ctx* c = (const Ctx*)ctx;
  return c && n_tokens >= 1 && plan_fused(c, c->R * n_tokens) ? 1 : 0;
}

int32_t vvs_num_weight_tensors(const vvs_config* cfg) { return cfg ? 4 + 9 * cfg->n_layers + (cfg->draft_input ? 1 : 0) : 0; }

vvs_status vvs_check_tree(int32_t n_nodes, const int32_t* h_parent, const uint8_t* h_tree_mask, int32_t* h_depth,
                          int32_t* h_parent_out) {
  TreeDesc t;
  vvs_status st = build_tree(n_nodes, h_parent, h_tree_mask, &t, nullptr);
  if (st != VVS_OK) return st;
  for (int j = 0; j <= n_nodes; ++j) {
    if (h_depth) h_depth[j] = t.depth[j];
    if (h_parent_out && j) h_parent_out[j - 1] = t.parent[j];
  }
  return VVS_OK;
}

vvs_status vvs_create(const vvs_config* cfg, void* d_kv, void* d_workspace, void* d_packed_weights, vvs_ctx** out) {
  if (!out) return fail(nullptr, VVS_EINVAL, "create: out is NULL");
  *out = nullptr;
  if (!d_kv || !d_workspace || !d_packed_weights) return fail(nullptr, VVS_EINVAL, "create: NULL device buffer");
  if (((uintptr_t)d_kv | (uintptr_t)d_workspace | (uintptr_t)d_packed_weights) & 255)
    return fail(nullptr, VVS_EINVAL, "create: device buffers must be 256-byte aligned");
  Ctx* c = new Ctx{};
  vvs_status st = plan_sizes(cfg, c, nullptr);
  if (st != VVS_OK) { delete c; return st; }
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) {
    delete c;
    return fail(nullptr, VVS_EHIP, "create: no HIP device (this library has no CPU path)");
  }
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) { std::string m = std::string("create: ") + hipGetErrorString(e); delete c; return fail(nullptr, VVS_EHIP, m); }
  c->kv = (char*)d_kv; c->ws = (char*)d_workspace; c->pw = (char*)d_packed_weights;
  c->nbr = nullptr;
  c->codebook = nullptr;
  c->code_dim = 0;
  c->wait_polls = kFewPolls;
  // zero the KV cache (padded slots are read, multiplied by zero weights) and the state block
  launch_fill_zero(c->kv, 2 * c->kv_v_off * c->esz, nullptr);
  launch_fill_zero(c->ws, c->w.x, nullptr);
  // rotary table in double -> float: [pos][pair] (cos, sin); theta_i = base^(-2i / (dh/2))
  int np = c->dh / 4;
  std::vector<float> tab((size_t)2 * c->rope_pos * np);
  for (int pos = 0; pos < c->rope_pos; ++pos)
    for (int i = 0; i < np; ++i) {
      double th = pow((double)c->cfg.rope_base, -2.0 * i / (c->dh / 2));
      tab[((size_t)pos * np + i) * 2 + 0] = (float)cos(pos * th);
      tab[((size_t)pos * np + i) * 2 + 1] = (float)sin(pos * th);
    }
  e = hipMemcpy(c->ws + c->w.rope_tab, tab.data(), tab.size() * sizeof(float), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) { std::string m = std::string("create: ") + hipGetErrorString(e); delete c; return fail(nullptr, VVS_EHIP, m); }
  *out = reinterpret_cast<vvs_ctx*>(c);
  return VVS_OK;
}

void vvs_destroy(vvs_ctx* ctx) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return;
  for (auto& t : c->timed) { (void)hipEventDestroy(t.t0); (void)hipEventDestroy(t.t1); }
  delete c;
}

vvs_status vvs_timing_enable(vvs_ctx* ctx, int32_t on) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  c->timing = on != 0;
  if (on) c->n_timed = 0;
  return VVS_OK;
}

vvs_status vvs_timing_read(vvs_ctx* ctx, int32_t kernel_class, int32_t* n_launches, float* total_ms) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (kernel_class < 0 || kernel_class >= VVS_K_CLASSES || !n_launches || !total_ms)
    return fail(&c->err, VVS_EINVAL, "timing_read: bad argument");
  int n = 0;
  float ms = 0.f;
  for (size_t i = 0; i < c->n_timed; ++i) {
    TimedLaunch& t = c->timed[i];
    if (t.cls != kernel_class) continue;
    hipError_t e = hipEventSynchronize(t.t1);
    float one = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&one, t.t0, t.t1);
    if (e != hipSuccess) return hip_fail(c, e, "timing_read");
    ms += one;
    ++n;
  }
  *n_launches = n;
  *total_ms = ms;
  return VVS_OK;
}

vvs_status vvs_set_state(vvs_ctx* ctx, const int32_t* d_state, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_state) return fail(&c->err, VVS_EINVAL, "set_state: NULL");
  if (!c->prefilled) return fail(&c->err, VVS_ESTATE, "set_state: call vvs_prefill first");
  launch_set_state(c, d_state, (hipStream_t)s);
  vvs_status rc = check_launch(c, "set_state");
  if (rc == VVS_OK) c->verify_pending = false;
  return rc;
}

const char* vvs_last_error(const vvs_ctx* ctx) {
  if (!ctx) return g_last_error.c_str();
  return reinterpret_cast<const Ctx*>(ctx)->err.c_str();
}

vvs_status vvs_load_weights(vvs_ctx* ctx, const void* const* d_tensors, int32_t n, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_tensors) return fail(&c->err, VVS_EINVAL, "load_weights: tensor list is NULL");
  if (n != vvs_num_weight_tensors(&c->cfg)) return fail(&c->err, VVS_EINVAL, "load_weights: wrong number of tensors");
  for (int i = 0; i < n; ++i)
    if (!d_tensors[i] && !(i == 1 && c->cfg.prefix_kind == VVS_PREFIX_DENSE))
      return fail(&c->err, VVS_EINVAL, "load_weights: a tensor pointer is NULL");
  launch_pack_weights(c, d_tensors, (hipStream_t)s);
  vvs_status st = check_launch(c, "load_weights");
  if (st == VVS_OK) c->weights_loaded = true;
  return st;
}

vvs_status vvs_set_neighbors(vvs_ctx* ctx, const int32_t* d_nbr) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_nbr) return fail(&c->err, VVS_EINVAL, "set_neighbors: table is NULL");
  if (c->cfg.relax_k < 1) return fail(&c->err, VVS_EINVAL, "set_neighbors: context was created with relax_k = 0");
  c->nbr = d_nbr;
  return VVS_OK;
}

vvs_status vvs_prefill(vvs_ctx* ctx, const void* d_prefix_cond, const void* d_prefix_uncond, int32_t n_forced,
                       const int32_t* d_forced_tokens, const float* d_uniform, int32_t* d_first_token, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (c->cfg.draft_input) return fail(&c->err, VVS_EINVAL, "prefill: this is a drafter context (use vvs_draft)");
  if (!c->weights_loaded) return fail(&c->err, VVS_ESTATE, "prefill: weights not loaded");
  if (!d_prefix_cond || !d_uniform || !d_first_token) return fail(&c->err, VVS_EINVAL, "prefill: NULL argument");
  if (c->cfg.prefix_kind == VVS_PREFIX_DENSE && !d_prefix_uncond)
    return fail(&c->err, VVS_EINVAL, "prefill: dense prefixes need the shared null prefix");
  if (n_forced < 0 || n_forced > c->G - 1) return fail(&c->err, VVS_EINVAL, "prefill: n_forced must be in [0, G-1]");
  if (n_forced > 0 && !d_forced_tokens) return fail(&c->err, VVS_EINVAL, "prefill: forced tokens are NULL");
  hipStream_t st = (hipStream_t)s;
  const int total = c->P + n_forced;
  PosDesc pos{nullptr, nullptr, 0, c->P, c->cfg.grid_w};
  for (int c0 = 0; c0 < total; c0 += c->chunk) {
    int T = std::min(c->chunk, total - c0);
    TreeDesc tree;
    causal_tree(T, &tree);
    pos.kv_base = c0;
    bool last = c0 + T >= total;
    launch_forward(c, tree, pos, T, nullptr, d_prefix_cond, d_prefix_uncond, c0, d_forced_tokens, n_forced, last ? 2 : 0, st);
    if (last) {
      TreeDesc one;
      causal_tree(1, &one);
      launch_accept(c, one, 1, (const float*)(c->ws + c->w.logits), nullptr, nullptr, d_uniform, 1, 0, 0, 0, VVS_STRICT,
                    false, nullptr, nullptr, nullptr, false, gave_up(c, T), st);
      launch_prefill_finish(c, n_forced, d_first_token, st);
      launch_push_prefill_feature(c, T, st);
    }
  }
  vvs_status rc = check_launch(c, "prefill");
  if (rc != VVS_OK) return rc;
  c->prefilled = true;
  c->verify_pending = false;
  c->last_T = 1;
  return VVS_OK;
}

static vvs_status check_verify_args(Ctx* c, const char* who, int32_t n_nodes, const int32_t* d_draft_tokens,
                                    const float* d_draft_probs, const float* d_uniforms, int32_t mode,
                                    int32_t* d_accept_len, int32_t* d_path, int32_t* d_next_token) {
  std::string w(who);
  if (n_nodes < 0) return fail(&c->err, VVS_EINVAL, w + ": n_nodes < 0");
  if (n_nodes > c->cfg.max_nodes) return fail(&c->err, VVS_ESIZE, w + ": n_nodes exceeds max_nodes of the context");
  if (n_nodes > 0 && (!d_draft_tokens || !d_draft_probs)) return fail(&c->err, VVS_EINVAL, w + ": draft tokens / probs are NULL");
  if (!d_uniforms || !d_accept_len || !d_path || !d_next_token) return fail(&c->err, VVS_EINVAL, w + ": NULL argument");
  if (mode != VVS_STRICT && mode != VVS_RELAXED) return fail(&c->err, VVS_EINVAL, w + ": unknown mode");
  if (mode == VVS_RELAXED && c->cfg.relax_k > 0 && !c->nbr)
    return fail(&c->err, VVS_ESTATE, w + ": relaxed mode needs vvs_set_neighbors first");
  return VVS_OK;
}

vvs_status vvs_verify_post(vvs_ctx* ctx, int32_t n_nodes, int32_t n_post, const int32_t* h_parent, const uint8_t* h_tree_mask,
                           const int32_t* d_draft_tokens, const float* d_draft_probs, const float* d_uniforms, int32_t mode,
                           int32_t* d_accept_len, int32_t* d_path, int32_t* d_next_token, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!c->prefilled) return fail(&c->err, VVS_ESTATE, "verify: call vvs_prefill first");
  if (c->verify_pending) return fail(&c->err, VVS_ESTATE, "verify: the previous verify was not committed");
  vvs_status rc = check_verify_args(c, "verify", n_nodes, d_draft_tokens, d_draft_probs, d_uniforms, mode, d_accept_len,
                                    d_path, d_next_token);
  if (rc != VVS_OK) return rc;
  if (n_post < 0 || n_post > n_nodes) return fail(&c->err, VVS_EINVAL, "verify: n_post must be in [0, n_nodes]");
  TreeDesc tree;
  rc = build_tree(n_nodes, h_parent, h_tree_mask, &tree, &c->err);
  if (rc != VVS_OK) return rc;
  for (int j = 1; j <= n_nodes; ++j) {
    if (j <= n_post && tree.parent[j] != j - 1)
      return fail(&c->err, VVS_EINVAL, "verify: the post-verified tokens must form a chain below the root");
    if (j > n_post && tree.parent[j] < n_post)
      return fail(&c->err, VVS_EINVAL, "verify: every candidate must descend from the last post-verified token");
  }
  tree.n_forced = n_post;
  hipStream_t st = (hipStream_t)s;
  const int T = n_nodes + 1;
  const int32_t* state = (const int32_t*)(c->ws + c->w.state);
  PosDesc pos{state, state + c->B, 0, c->P, c->cfg.grid_w};
  launch_build_tokens(c, T, d_draft_tokens, st);
  launch_forward(c, tree, pos, T, (const int32_t*)(c->ws + c->w.tokens), nullptr, nullptr, 0, nullptr, 0, 1, st);
  launch_accept(c, tree, T, (const float*)(c->ws + c->w.logits), d_draft_tokens, d_draft_probs, d_uniforms, 2 * T, 2, 0, 1,
                mode, true, d_accept_len, d_path, d_next_token, true, gave_up(c, T), st);
  rc = check_launch(c, "verify");
  if (rc != VVS_OK) return rc;
  c->verify_pending = true;
  c->last_T = T;
  return VVS_OK;
}

vvs_status vvs_verify(vvs_ctx* ctx, int32_t n_nodes, const int32_t* h_parent, const uint8_t* h_tree_mask,
                      const int32_t* d_draft_tokens, const float* d_draft_probs, const float* d_uniforms, int32_t mode,
                      int32_t* d_accept_len, int32_t* d_path, int32_t* d_next_token, vvs_stream s) {
  return vvs_verify_post(ctx, n_nodes, 0, h_parent, h_tree_mask, d_draft_tokens, d_draft_probs, d_uniforms, mode, d_accept_len,
                         d_path, d_next_token, s);
}

vvs_status vvs_accept_from_logits(vvs_ctx* ctx, int32_t n_nodes, const int32_t* h_parent, const uint8_t* h_tree_mask,
                                  const float* d_raw_logits, const int32_t* d_draft_tokens, const float* d_draft_probs,
                                  const float* d_uniforms, int32_t mode, int32_t* d_accept_len, int32_t* d_path,
                                  int32_t* d_next_token, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_raw_logits) return fail(&c->err, VVS_EINVAL, "accept_from_logits: logits are NULL");
  vvs_status rc = check_verify_args(c, "accept_from_logits", n_nodes, d_draft_tokens, d_draft_probs, d_uniforms, mode,
                                    d_accept_len, d_path, d_next_token);
  if (rc != VVS_OK) return rc;
  TreeDesc tree;
  rc = build_tree(n_nodes, h_parent, h_tree_mask, &tree, &c->err);
  if (rc != VVS_OK) return rc;
  launch_accept(c, tree, n_nodes + 1, d_raw_logits, d_draft_tokens, d_draft_probs, d_uniforms, 2 * (n_nodes + 1), 2, 0, 1,
                mode, false, d_accept_len, d_path, d_next_token, false, nullptr, (hipStream_t)s);
  return check_launch(c, "accept_from_logits");
}

vvs_status vvs_accept_from_logits_noalloc(vvs_ctx* ctx, int32_t n_nodes, const int32_t* h_parent, const uint8_t* h_tree_mask,
                                          const float* d_raw_logits, const int32_t* d_draft_tokens, const float* d_draft_probs,
                                          const float* d_uniforms, int32_t mode, int32_t* d_accept_len, int32_t* d_path,
                                          int32_t* d_next_token, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_raw_logits) return fail(&c->err, VVS_EINVAL, "accept_from_logits_noalloc: logits are NULL");
  vvs_status rc = check_verify_args(c, "accept_from_logits_noalloc", n_nodes, d_draft_tokens, d_draft_probs, d_uniforms, mode,
                                    d_accept_len, d_path, d_next_token);
  if (rc != VVS_OK) return rc;
  TreeDesc tree;
  rc = build_tree(n_nodes, h_parent, h_tree_mask, &tree, &c->err);
  if (rc != VVS_OK) return rc;
  std::string msg;
  rc = launch_accept_noalloc(c, tree, n_nodes + 1, d_raw_logits, d_draft_tokens, d_draft_probs, d_uniforms, mode, d_accept_len, d_path,
                             d_next_token, (hipStream_t)s, &msg);
  if (rc != VVS_OK) return fail(&c->err, rc, msg);
  return check_launch(c, "accept_from_logits_noalloc");
}

vvs_status vvs_kv_commit(vvs_ctx* ctx, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!c->verify_pending) return fail(&c->err, VVS_ESTATE, "kv_commit: no verify to commit");
  launch_commit(c, (hipStream_t)s);
  vvs_status rc = check_launch(c, "kv_commit");
  if (rc != VVS_OK) return rc;
  c->verify_pending = false;
  return VVS_OK;
}

vvs_status vvs_select_unverified(int32_t n_nodes, const int32_t* h_parent, const uint8_t* h_tree_mask, float u, int32_t* h_nodes,
                                 int32_t* n_kept) {
  if (!h_nodes || !n_kept) return VVS_EINVAL;
  if (!(u >= 0.f && u < 1.f)) return VVS_EINVAL;
  TreeDesc t;
  vvs_status st = build_tree(n_nodes, h_parent, h_tree_mask, &t, nullptr);
  if (st != VVS_OK) return st;
  *n_kept = 0;
  // candidate paths = one per leaf, in leaf order; their lengths are the leaves' depths
  std::vector<int> leaves;
  long total = 0;
  for (int j = 1; j <= n_nodes; ++j)
    if (t.first_child[j] < 0) { leaves.push_back(j); total += t.depth[j]; }
  if (leaves.empty()) return VVS_OK;
  const int n_paths = (int)leaves.size();
  const int sel = std::min((int)std::floor((double)u * n_paths), n_paths - 1);
  const int mean_floor = (int)(total / n_paths);                     // floor of the mean path length (Eq. 1)
  const int len = t.depth[leaves[sel]], keep = std::min(len, mean_floor);
  int node = leaves[sel];
  for (int k = len - 1; k >= 0; --k) {                               // walk up; position k of the path is the ancestor at depth k + 1
    if (k < keep) h_nodes[k] = node;
    node = t.parent[node];
  }
  *n_kept = keep;
  return VVS_OK;
}

int32_t vvs_skip_uniform(int32_t step_index, int32_t interval) {
  return interval >= 2 && step_index >= 0 && (step_index + 1) % interval == 0;
}

int32_t vvs_skip_dynamic(float similarity, float threshold, int32_t last_step_verified) {
  return last_step_verified != 0 && similarity >= threshold;
}

vvs_status vvs_set_codebook(vvs_ctx* ctx, const float* d_embed, int32_t dim) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_embed) return fail(&c->err, VVS_EINVAL, "set_codebook: table is NULL");
  if (dim < 1 || dim > 64) return fail(&c->err, VVS_ESIZE, "set_codebook: dim must be in [1, 64]");
  c->codebook = d_embed;
  c->code_dim = dim;
  return VVS_OK;
}

vvs_status vvs_path_similarity(vvs_ctx* ctx, int32_t n_nodes, const int32_t* h_parent, const uint8_t* h_tree_mask,
                               const int32_t* d_draft_tokens, float alpha, int32_t stride, float* d_similarity, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!c->codebook) return fail(&c->err, VVS_ESTATE, "path_similarity: call vvs_set_codebook first");
  if (!d_similarity || (n_nodes > 0 && !d_draft_tokens)) return fail(&c->err, VVS_EINVAL, "path_similarity: NULL argument");
  if (stride < 1) return fail(&c->err, VVS_EINVAL, "path_similarity: stride < 1");
  if (!(alpha > 0.f)) return fail(&c->err, VVS_EINVAL, "path_similarity: alpha must be positive");
  if (n_nodes > c->cfg.max_nodes) return fail(&c->err, VVS_ESIZE, "path_similarity: n_nodes exceeds max_nodes of the context");
  TreeDesc tree;
  vvs_status rc = build_tree(n_nodes, h_parent, h_tree_mask, &tree, &c->err);
  if (rc != VVS_OK) return rc;
  launch_path_similarity(c, tree, n_nodes, d_draft_tokens, alpha, stride, d_similarity, (hipStream_t)s);
  return check_launch(c, "path_similarity");
}

vvs_status vvs_read_features(vvs_ctx* ctx, float* d_features, int32_t* d_count, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_features || !d_count) return fail(&c->err, VVS_EINVAL, "read_features: NULL");
  if (c->cfg.feature_slots < 1) return fail(&c->err, VVS_ESTATE, "read_features: the context was created with feature_slots = 0");
  if (!c->prefilled) return fail(&c->err, VVS_ESTATE, "read_features: call vvs_prefill first");
  launch_read_features(c, d_features, d_count, (hipStream_t)s);
  return check_launch(c, "read_features");
}

vvs_status vvs_draft(vvs_ctx* drafter, vvs_ctx* target, int32_t n_nodes, const int32_t* h_parent, const uint8_t* h_tree_mask,
                     int32_t n_ctx, const int32_t* d_recent_tokens, int32_t n_unverified, const int32_t* d_given_tokens,
                     int32_t* d_draft_tokens, float* d_draft_probs, vvs_stream s) {
  Ctx* dr = reinterpret_cast<Ctx*>(drafter);
  Ctx* tg = reinterpret_cast<Ctx*>(target);
  if (!dr) return VVS_EINVAL;
  if (!tg) return fail(&dr->err, VVS_EINVAL, "draft: target context is NULL");
  if (!dr->cfg.draft_input) return fail(&dr->err, VVS_EINVAL, "draft: the first context was not created with draft_input = 1");
  if (tg->cfg.draft_input) return fail(&dr->err, VVS_EINVAL, "draft: the target is a drafter context");
  if (!dr->weights_loaded) return fail(&dr->err, VVS_ESTATE, "draft: drafter weights not loaded");
  if (!tg->prefilled) return fail(&dr->err, VVS_ESTATE, "draft: call vvs_prefill on the target first");
  const vvs_config &a = dr->cfg, &b = tg->cfg;
  if (a.d_model != b.d_model || a.dtype != b.dtype || a.n_prompts != b.n_prompts || a.vocab != b.vocab || a.logit_lo != b.logit_lo ||
      a.logit_hi != b.logit_hi || a.grid_h != b.grid_h || a.grid_w != b.grid_w)
    return fail(&dr->err, VVS_EINVAL, "draft: drafter and target differ in d_model, dtype, prompts, vocabulary slice or grid");
  if (a.feature_pre_norm != b.feature_pre_norm)
    return fail(&dr->err, VVS_EINVAL, "draft: drafter and target keep different kinds of feature (feature_pre_norm)");
  if (n_nodes < 1) return fail(&dr->err, VVS_EINVAL, "draft: n_nodes < 1");
  if (n_ctx < 1 || n_ctx > b.feature_slots) return fail(&dr->err, VVS_EINVAL, "draft: n_ctx must be in [1, feature_slots of the target]");
  if (n_unverified < 0 || n_unverified > VVS_MAX_FEATURE_SLOTS) return fail(&dr->err, VVS_EINVAL, "draft: n_unverified out of range");
  if (!d_recent_tokens || !d_draft_tokens || !d_draft_probs) return fail(&dr->err, VVS_EINVAL, "draft: NULL argument");
  TreeDesc shape;
  vvs_status rc = build_tree(n_nodes, h_parent, h_tree_mask, &shape, &dr->err);
  if (rc != VVS_OK) return rc;
  // block tokens of the drafter's forwards: the n_ctx pairs (the last is the root), then the nodes that
  // have children, ordered by depth and then id, so that a level only appends tokens
  const int T = n_nodes + 1, k = n_ctx;
  std::vector<int> order;
  int last_level = 0;
  for (int j = 1; j < T; ++j)
    if (shape.first_child[j] >= 0) { order.push_back(j); last_level = std::max(last_level, (int)shape.depth[j]); }
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return shape.depth[x] < shape.depth[y]; });
  if (k + (int)order.size() > dr->Tmax)
    return fail(&dr->err, VVS_ESIZE, "draft: n_ctx + expanded nodes exceeds max_nodes + 1 of the drafter context");
  std::vector<int> slot(T, -1);
  slot[0] = k - 1;
  for (size_t i = 0; i < order.size(); ++i) slot[order[i]] = k + (int)i;
  hipStream_t st = (hipStream_t)s;
  launch_draft_state(dr, tg, k, n_unverified, st);
  launch_draft_zero_leaves(dr, shape, d_draft_probs, st);
  const int32_t* state = (const int32_t*)(dr->ws + dr->w.state);
  PosDesc pos{state, state + dr->B, 0, dr->P, dr->cfg.grid_w};
  DraftLevel lv;
  memset(&lv, 0, sizeof(lv));
  lv.k = k;
  lv.n_nodes = n_nodes;
  lv.all = k + (int)order.size();
  std::vector<int32_t> bp(lv.all > 1 ? lv.all - 1 : 1);
  for (int t = 1; t < lv.all; ++t) {
    if (t < k) { bp[t - 1] = t - 1; continue; }
    const int j = order[t - k];
    lv.node[t] = (int8_t)j;
    lv.parent_slot[t] = (int8_t)slot[shape.parent[j]];
    bp[t - 1] = slot[shape.parent[j]];
  }
  TreeDesc block;
  rc = build_tree(lv.all - 1, bp.data(), nullptr, &block, &dr->err);
  if (rc != VVS_OK) return rc;
  int n_in = 0;
  for (int level = 0; level <= last_level; ++level) {
    // level 0: the pairs; level l: the nodes of depth l that have children (no level up to the last is without)
    lv.first = level ? k + n_in : 0;
    while (n_in < (int)order.size() && shape.depth[order[n_in]] <= level) ++n_in;
    lv.Tq = k + n_in;
    block.T = lv.Tq;
    block.first = lv.first;
    block.all = lv.all;
    lv.n_sel = 0;
    for (int j = 0; j < T; ++j)
      if (shape.first_child[j] >= 0 && shape.depth[j] == level) {
        lv.sel_node[lv.n_sel] = (int8_t)j;
        lv.sel_slot[lv.n_sel] = (int8_t)slot[j];
        ++lv.n_sel;
      }
    launch_draft_input(dr, tg, lv, d_recent_tokens, d_draft_tokens, st);
    launch_forward(dr, block, pos, lv.Tq, nullptr, nullptr, nullptr, 0, nullptr, 0, 1, st, true);
    launch_draft_select(dr, lv, shape, d_given_tokens, d_draft_tokens, d_draft_probs, st);
    lv.Tq_prev = lv.Tq;
    lv.first_prev = lv.first;
  }
  rc = check_launch(dr, "draft");
  if (rc != VVS_OK) return rc;
  dr->last_T = lv.all;
  return VVS_OK;
}

vvs_status vvs_read_state(vvs_ctx* ctx, int32_t* d_state, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_state) return fail(&c->err, VVS_EINVAL, "read_state: NULL");
  launch_read_state(c, d_state, (hipStream_t)s);
  return check_launch(c, "read_state");
}

vvs_status vvs_debug_logits(vvs_ctx* ctx, float* d_raw, float* d_mixed, float* d_probs, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (c->last_T < 1) return fail(&c->err, VVS_ESTATE, "debug_logits: nothing has run yet");
  launch_debug_logits(c, d_raw, d_mixed, d_probs, (hipStream_t)s);
  return check_launch(c, "debug_logits");
}

vvs_status vvs_debug_kv(vvs_ctx* ctx, int32_t layer, int32_t row, int32_t n_slots, float* d_k, float* d_v, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (layer < 0 || layer >= c->L || row < 0 || row >= c->R || n_slots < 0 || n_slots > c->S_cap || !d_k || !d_v)
    return fail(&c->err, VVS_EINVAL, "debug_kv: argument out of range");
  launch_debug_kv(c, layer, row, n_slots, d_k, d_v, (hipStream_t)s);
  return check_launch(c, "debug_kv");
}

vvs_status vvs_debug_copy(vvs_ctx* ctx, void* d_dst, const void* d_src, size_t bytes, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_dst || !d_src || (bytes & 15) || (((uintptr_t)d_dst | (uintptr_t)d_src) & 15))
    return fail(&c->err, VVS_EINVAL, "debug_copy: pointers and size must be multiples of 16");
  launch_copy_bytes(d_dst, d_src, bytes, (hipStream_t)s);
  return check_launch(c, "debug_copy");
}

vvs_status vvs_debug_fill_probe(vvs_ctx* ctx, const void* d_src, size_t region_bytes, size_t wg_stride_bytes, int32_t reps, int32_t mode,
                                int32_t n_workgroups, int32_t waves, uint32_t* d_sink, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (!d_src || !d_sink || ((uintptr_t)d_src & 15) || region_bytes < 8192 || (region_bytes & 8191) || region_bytes > ((size_t)1 << 30) ||
      (wg_stride_bytes & 15) || wg_stride_bytes > ((size_t)1 << 30))
    return fail(&c->err, VVS_EINVAL, "debug_fill_probe: the region must be 16-byte aligned and a multiple of 8192 bytes, region and stride at most 1 GiB");
  if (reps < 1 || reps > (1 << 20) || (mode != 0 && mode != 1) || n_workgroups < 1 || n_workgroups > 65536 || waves < 1 || waves > 16)
    return fail(&c->err, VVS_EINVAL, "debug_fill_probe: reps, mode, workgroups or waves out of range");
  launch_fill_probe(d_src, region_bytes, wg_stride_bytes, reps, mode, n_workgroups, waves, d_sink, (hipStream_t)s);
  return check_launch(c, "debug_fill_probe");
}

vvs_status vvs_debug_wait_limit(vvs_ctx* ctx, int32_t polls) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (polls < 0) return fail(&c->err, VVS_EINVAL, "debug_wait_limit: polls < 0");
  c->wait_polls = polls ? polls : kFewPolls;
  return VVS_OK;
}

size_t vvs_debug_gemm_scratch_bytes(const vvs_ctx* ctx, int32_t m, int32_t n, int32_t k) {
  const Ctx* c = reinterpret_cast<const Ctx*>(ctx);
  if (!c || m < 1 || n < 1 || k < 1) return 0;
  GemmPlan p = plan_partial(c, m, n, k);
  return align_up((size_t)n * k * c->esz, 256) + align_up(align_up((size_t)m, 32) * k * c->esz, 256) +
         align_up((size_t)p.splits * m * n * sizeof(float), 256);
}

vvs_status vvs_debug_gemm(vvs_ctx* ctx, int32_t m, int32_t n, int32_t k, const void* d_a, const void* d_w, void* d_scratch,
                          float* d_c, vvs_stream s) {
  Ctx* c = reinterpret_cast<Ctx*>(ctx);
  if (!c) return VVS_EINVAL;
  if (m < 1 || n < 1 || k < 1 || !d_a || !d_w || !d_scratch || !d_c) return fail(&c->err, VVS_EINVAL, "debug_gemm: bad argument");
  if (c->cfg.dtype == VVS_BF16 && (n % 64 || k % 64)) return fail(&c->err, VVS_ESIZE, "debug_gemm: bf16 needs n, k multiples of 64");
  launch_debug_gemm(c, m, n, k, d_a, d_w, d_scratch, d_c, (hipStream_t)s);
  return check_launch(c, "debug_gemm");
}

}  // extern "C"
