// The launcher of the short tiles with stages of 64 k.  Three kernels:
//   * the high part alone, K at least 16 stages long (LM heads): gemm_k64_whole.hip;
//   * pairs, weights that no cache holds: gemm_k64_once.hip.  Gate/up of the 8B shape at 32 / 64 / 128 rows 50.8 / 56.0 / 70.0 ->
//     49.2 / 54.2 / 66.2 us, of the 70B 203 / 202 / 308 -> 180 / 184 / 255 (above 80 rows on 128 instead of 256 columns); down projection
//     of the 8B at 128 rows 37.1 -> 35.9.  Several tiles of rows, which want the same lines out of one XCD's L2, gain as well: 4096 x
//     4096 in slices at 224 / 560 rows 24.9 / 45.4 -> 23.2 / 43.3, 2048 x 2048 at 192 / 256 11.5 / 12.6 -> 11.2 / 11.9;
//   * the rest, here.
// Pairs are summed in the order of the tiles with one K step per stage, so a product has one set of bits whatever the tile.  The
// kernel for LM heads, which adds two halves of every stage's K at the end, took 49.2 / 54.5 / 66.2 us for gate/up where it kept to
// that order: no less than the tile of gemm_tile.h.
#include "gemm_k64.h"

hipError_t launch_proj_k64_whole(int mt, int nf, GemmArgs g, hipStream_t s);
hipError_t launch_proj_k64_once(int mt, int nf, const GemmArgs& g, hipStream_t s);

hipError_t launch_proj_k64(int mt, int nf, const GemmArgs& g, hipStream_t s) {
  if (g.K % 64 != 0 || g.a_paired || (!g.a_lo && g.epilogue != GEMM_STORE_F32)) return hipErrorInvalidValue;
  if (g.a_lo) return g.once ? launch_proj_k64_once(mt, nf, g, s) : launch_k64_pairs<false>(mt, nf, g, s);
  if (g.split_k == 1 && g.K >= 1024) return launch_proj_k64_whole(mt, nf, g, s);
  return with_short_tile(mt, nf, [&](auto MT, auto NF) {
    constexpr int mt_ = decltype(MT)::value, nf_ = decltype(NF)::value;
    const int m_tiles = (g.M + 16 * mt_ - 1) / (16 * mt_), n_tiles = g.N / (64 * nf_);
    proj_kernel<mt_, nf_, GEMM_STORE_F32, false, 2><<<dim3(8 * ((n_tiles + 7) / 8) * m_tiles, 1, g.split_k), 256, 0, s>>>(g);
    return hipGetLastError();
  });
}
