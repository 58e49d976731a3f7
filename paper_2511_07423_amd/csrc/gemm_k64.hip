// The short tiles with stages of 64 k: 128 columns x 16 .. 144 rows, 256 columns x 16 .. 80 rows.  Three kernels:
//   * K whole and at least 16 stages long: gemm_k64_whole.hip;
//   * K split into slices, weights that no cache holds: gemm_k64_slices.hip;
//   * the rest -- small models, whose launches are over before either pays -- here, the tile of gemm_tile.h (KSUB = 2).  (The tiny
//     decoder, K = 256: three such launches of gemm_k64_whole.hip made a verify of 27 rows 141.4 -> 143.7 us.)
#include "gemm_tile.h"

hipError_t launch_proj_k64_whole(int mt, int nf, GemmArgs g, hipStream_t s);
hipError_t launch_proj_k64_slices(int mt, int nf, const GemmArgs& g, hipStream_t s);

template <int MT, int NF>
static hipError_t launch_k64(const GemmArgs& g, hipStream_t s) {
  const int m_tiles = (g.M + 16 * MT - 1) / (16 * MT), n_tiles = g.N / (64 * NF);
  const dim3 grid(8 * ((n_tiles + 7) / 8) * m_tiles, 1, g.split_k);
  if (!g.a_lo) {
    proj_kernel<MT, NF, GEMM_STORE_F32, false, 2><<<grid, 256, 0, s>>>(g);
    return hipGetLastError();
  }
  switch (g.epilogue) {
    case GEMM_STORE_F32: proj_kernel<MT, NF, GEMM_STORE_F32, true, 2><<<grid, 256, 0, s>>>(g); break;
    case GEMM_ADD_F32: proj_kernel<MT, NF, GEMM_ADD_F32, true, 2><<<grid, 256, 0, s>>>(g); break;
    case GEMM_SWIGLU: proj_kernel<MT, NF, GEMM_SWIGLU, true, 2><<<grid, 256, 0, s>>>(g); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_proj_k64(int mt, int nf, const GemmArgs& g, hipStream_t s) {
  if (g.K % 64 != 0 || g.a_paired || (!g.a_lo && g.epilogue != GEMM_STORE_F32)) return hipErrorInvalidValue;
  if (g.split_k == 1 && g.K >= 1024) return launch_proj_k64_whole(mt, nf, g, s);
  if (g.split_k > 1 && g.once && g.a_lo) return launch_proj_k64_slices(mt, nf, g, s);
  if (nf == 2) {
    switch (mt) {
      case 1: return launch_k64<1, 2>(g, s);
      case 2: return launch_k64<2, 2>(g, s);
      case 3: return launch_k64<3, 2>(g, s);
      case 4: return launch_k64<4, 2>(g, s);
      case 5: return launch_k64<5, 2>(g, s);
      case 6: return launch_k64<6, 2>(g, s);
      case 7: return launch_k64<7, 2>(g, s);
      case 8: return launch_k64<8, 2>(g, s);
      case 9: return launch_k64<9, 2>(g, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (nf == 4) {
    switch (mt) {
      case 1: return launch_k64<1, 4>(g, s);
      case 2: return launch_k64<2, 4>(g, s);
      case 3: return launch_k64<3, 4>(g, s);
      case 4: return launch_k64<4, 4>(g, s);
      case 5: return launch_k64<5, 4>(g, s);
      default: return hipErrorInvalidValue;
    }
  }
  return hipErrorInvalidValue;
}
