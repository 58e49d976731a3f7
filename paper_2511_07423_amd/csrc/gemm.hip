// Tile planner and launcher of the projection GEMM (kernel: gemm_tile.h).  Host code only.
//
// A tile is 16 MT rows (MT = 1..17) by 256 columns, or by 128 columns (MT = 1..12) for outputs whose width is
// not a multiple of 256 and for small batches; the short ones (128 columns x <= 144 rows, 256 x <= 80) come with
// two MFMA K steps per stage as well.  Why 128 columns: at M = 128 a 256-column tiling gives the 8B gate/up projection
// only 112 blocks and every block pulls its weight stream at the ~24 GB/s one compute unit sustains from HBM;
// 224 blocks of 128 columns stream on twice the compute units.  K may be split into stored slices.
#include "common.h"
#include <algorithm>

static int g_forced = -1;   // tuning hook: forced tile (see gemm_force_variant), -1 = automatic
void gemm_force_variant(int v) { g_forced = v; }
static int g_forced_once = -1;   // test hook: forced GemmArgs::once, -1 = the caller's
void gemm_force_once(int v) { g_forced_once = v; }

static bool tile_fits(const GemmArgs& g, int mt, int nf, int ksub) {
  if (mt < 1 || (nf == 4 ? mt > 17 : mt > 12)) return false;
  if (g.a_paired && ksub != 1) return false;                       // the paired activation array: one K step per stage
  if (ksub == 2 && (nf == 4 ? mt > 5 : mt > 9)) return false;      // three stages of 128-byte rows must fit the LDS
  if (g.K % (32 * ksub) != 0) return false;
  const int bn = 64 * nf;
  if (g.N % bn != 0) return false;
  if (g.epilogue != GEMM_SWIGLU)
    for (int i = 0; i < 3; ++i)
      if (g.w_rows[i] % bn != 0) return false;
  return true;
}

// Whether this launch may store K slices.  Their number is the order of its sums, and the K and V rows that a layer appends round
// to bf16 by it, so a model's outputs move with it (8 layers of the 70B shape, 126 rows over short contexts: logits by about 6e-4 of
// their norm, and single ids, with other slices for QKV, output and down projection).
static bool may_slice(const GemmArgs& g) { return g.epilogue != GEMM_SWIGLU && g.c_parts; }

// Modelled time of one stage (32 ksub of K) of one block, us; from timings on an MI355X.
// Launches that may be sliced: 0.17 us plus 0.086 us per 16-row block and MFMA K step (8B gate/up projection at M = 532 on 256-column
// tiles of 128, 144 and 272 rows); a 128-column tile pays the activation-fragment reads of a 256-column one for half the
// MFMAs: 0.6x, not 0.5x.  A short tile is bound by its weight stream instead: BN rows x 64 bytes per K step at the ~24 GB/s one
// compute unit pulls from HBM.  This fit stays as it is: see may_slice.
// Whole K: tiles with one K step per stage ask for weights by half lines, and short ones wait for that: 70B gate/up projection as one
// tile of 96, 128, 160, 208 rows 1.0, 1.12, 1.19, 1.35 us (0.65 + 0.055 per row block), LM heads of the high part alone 0.85
// at any height, 0.75 in several rounds (two of their blocks share a compute unit; with 0.85 for those too, 545 to 576 rows took 192 x
// 128 instead of 144 x 256: 8B 199 instead of 191 us, 70B 370 instead of 362).  Two K steps per stage: 8B gate/up at 32 .. 144
// rows 0.69 .. 1.02 us, 256 columns (70B) at 32 .. 80 rows 1.37 .. 1.45, the 70B's 96 .. 144 rows on 128 columns (two rounds of
// blocks) 0.87 .. 1.06; LM heads (gemm_k64_whole.hip) 1.13x with several rounds of blocks, or several tiles of rows to read the
// same weights.
static double step_us(const GemmArgs& g, int mt, int nf, int ksub, bool one_tile, bool one_round) {
  const bool lo = g.a_lo != nullptr || g.a_paired;
  if (!may_slice(g) && ksub == 2 && g.K >= 1024) {
    if (lo) return nf == 4 ? 1.35 + 0.02 * mt : 0.6 + 0.048 * mt;
    return (nf == 4 ? 0.9 + 0.05 * mt : 0.43 + 0.035 * mt) * (one_tile && one_round ? 1.0 : 1.13);
  }
  const double mfma = 0.17 + ksub * 0.086 * mt * (nf == 4 ? 1.0 : 0.6) * (lo ? 1.0 : 0.55);   // hi alone: half the MFMAs
  double stream = ksub * 64 * nf * 64 / 24e3;
  if (!may_slice(g) && ksub == 1) {
    if (one_tile) stream = nf / 4.0 * (0.65 + 0.055 * mt);
    if (!lo) stream = std::max(stream, nf == 2 ? 0.425 : one_round ? 0.85 : 0.75);
  }
  return std::max(mfma, stream);
}
static int max_split(const GemmArgs& g, int mt, int nf) {
  if (!may_slice(g)) return 1;
  const long tiles = (long)((g.M + 16 * mt - 1) / (16 * mt)) * (g.N / (64 * nf));
  long split = 256 / tiles;
  const long most = g.K / 32 / 8;               // at least 8 K steps per slice
  split = split < most ? split : most;
  if (split > SY_MAX_K_SLICES) split = SY_MAX_K_SLICES;
  return split < 1 ? 1 : (int)split;
}
// Blocks are equal-sized and one runs per compute unit, so a launch takes ceil(blocks / 256) rounds of
// stages per block x step_us, plus per stored K slice and 2.2 M outputs ~2.4 us to store it and read it back
// (QKV and down projection at M = 532 on 272-row tiles with 5 and 8 slices: 18 - 19 us beyond their K steps).
static double plan_cost(const GemmArgs& g, int mt, int nf, int ksub, int split) {
  const long tiles = (long)((g.M + 16 * mt - 1) / (16 * mt)) * (g.N / (64 * nf));
  const long rounds = (tiles * split + 255) / 256;
  const double steps = (double)(g.K / (32 * ksub)) / split;
  const double merge = split > 1 ? 2.4 * split * ((double)g.M * g.N / 2.2e6) : 0.0;
  return rounds * steps * step_us(g, mt, nf, ksub, g.M <= 16 * mt, rounds == 1) + merge;
}

static void pick(const GemmArgs& g, int* mt_out, int* nf_out, int* ksub_out, int* split_out) {
  if (g_forced >= 0) {
    // forced tile: rows / 16 + 100 for 128 columns + 200 for two K steps per stage
    const int mt = g_forced % 100, nf = (g_forced / 100) % 2 ? 2 : 4, ksub = g_forced >= 200 ? 2 : 1;
    if (tile_fits(g, mt, nf, ksub)) {
      *mt_out = mt;
      *nf_out = nf;
      *ksub_out = ksub;
      *split_out = max_split(g, mt, nf);         // forced tile: as many slices as fit
      return;
    }
  }
  // Tiles below 128 rows only where M itself is smaller: the model's fixed cost per K step was fitted on tall tiles.
  const int need = (g.M + 15) / 16, mt_min = need < 8 ? need : 8;
  int best_mt = -1, best_nf = 4, best_ksub = 1, best_split = 1;
  double best_cost = 0.0;
  for (int nf = 4; nf >= 2; nf -= 2)
    for (int mt = mt_min; mt <= 17; ++mt)
      for (int ksub = 2; ksub >= 1; --ksub) {    // two K steps per stage wherever the tile allows them
        if (!tile_fits(g, mt, nf, ksub)) continue;
        const int most = max_split(g, mt, nf);
        for (int split = 1; split <= most; ++split) {    // fewer slices than fit can win: less to merge
          // pairs, whole K in stages of 64: for the weight stream of one tile of rows; several read the same weights, which makes
          // it a matter of the MFMAs
          if (!may_slice(g) && ksub == 2 && g.K >= 1024 && g.M > 16 * mt && g.a_lo) continue;
          const double c = plan_cost(g, mt, nf, ksub, split);
          if (best_mt < 0 || c < best_cost) {
            best_mt = mt;
            best_nf = nf;
            best_ksub = ksub;
            best_cost = c;
            best_split = split;
          }
        }
      }
  *mt_out = best_mt;
  *nf_out = best_nf;
  *ksub_out = best_ksub;
  *split_out = best_split;
}

void gemm_plan(const GemmArgs& g, int* bm, int* bn, int* split) {
  int mt = -1, nf = 4, ksub = 1;
  pick(g, &mt, &nf, &ksub, split);
  *bm = 16 * mt;
  *bn = 64 * nf;
}

int gemm_plan_bk(const GemmArgs& g) {
  int mt = -1, nf = 4, ksub = 1, split = 1;
  pick(g, &mt, &nf, &ksub, &split);
  return 32 * ksub;
}

int gemm_pick_split(const GemmArgs& g) {
  int mt, nf, ksub, split;
  pick(g, &mt, &nf, &ksub, &split);
  return mt < 0 ? 1 : split;
}

// Up to 16 rows.  Every block of stream.hip reads all activations beside its own weight rows: at 16 rows twice the bytes of
// a residual projection's weights (output + down projection of the 8B shape: 33 us at 8 rows, 40 us at 16), at 32 rows four
// times, where K slices over blocks are the better split.
bool gemm_streams(int M) { return M <= SY_STREAM_ROWS && g_forced < 0; }

hipError_t launch_gemm(const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0) return hipSuccess;
  if (!g.a || !g.w[0] || !g.c || g.N < 128 || g.K < 64 || g.K % 64 != 0 || g.split_k < 1)
    return hipErrorInvalidValue;
  int mt, nf, ksub, split;
  pick(g, &mt, &nf, &ksub, &split);
  if (mt < 0 || g.split_k > g.K / 32 || g.split_k > SY_MAX_K_SLICES) return hipErrorInvalidValue;
  if (g.split_k > 1 && (!g.c_parts || g.epilogue == GEMM_SWIGLU)) return hipErrorInvalidValue;
  if (!g.a_lo && !g.a_paired && g.epilogue != GEMM_STORE_F32) return hipErrorInvalidValue;
  if (g.a_paired && ksub != 1) return hipErrorInvalidValue;
  if (g.c_paired && g.epilogue != GEMM_SWIGLU) return hipErrorInvalidValue;
  if (g.epilogue == GEMM_SWIGLU) {
    if ((!g.c_lo && !g.c_paired) || !g.w[1]) return hipErrorInvalidValue;
  } else {
    long rows = 0;
    for (int i = 0; i < 3; ++i) {
      rows += g.w_rows[i];
      if (g.w_rows[i] % 16 != 0) return hipErrorInvalidValue;   // a copy's 16 tile rows come from one array
    }
    if (rows != g.N) return hipErrorInvalidValue;
  }
  if (ksub == 2) {
    GemmArgs a = g;
    if (g_forced_once >= 0) a.once = g_forced_once != 0;
    return launch_proj_k64(mt, nf, a, s);
  }
  if (nf == 2) return launch_proj_nf2(mt, g, s);
  return mt <= 9 ? launch_proj_nf4_low(mt, g, s) : launch_proj_nf4_high(mt, g, s);
}
