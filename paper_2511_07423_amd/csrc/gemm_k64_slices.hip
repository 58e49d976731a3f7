// The short tiles of gemm_k64.hip where K is split into stored slices of 8 to 60 stages and no cache holds the weights: their
// lines are marked as not wanted again (128 rows, down projection of the 8B shape 37.4 -> 36.4 us).  The kernel that takes whole K
// (gemm_k64_whole.hip: 12 wavefronts to start, K halves to add at the end) needs about 1 us longer for those: QKV projection
// in 5 slices at 32 rows 14.3 against 15.2 us, at 128 rows 21.7 against 23.1.
#include "gemm_tile.h"

template <int MT, int NF>
static hipError_t launch_slices(const GemmArgs& g, hipStream_t s) {
  const int m_tiles = (g.M + 16 * MT - 1) / (16 * MT), n_tiles = g.N / (64 * NF);
  const dim3 grid(8 * ((n_tiles + 7) / 8) * m_tiles, 1, g.split_k);
  // (a slice is stored plainly, whatever the epilogue of the whole)
  proj_kernel<MT, NF, GEMM_STORE_F32, true, 2, false, true><<<grid, 256, 0, s>>>(g);
  return hipGetLastError();
}

hipError_t launch_proj_k64_slices(int mt, int nf, const GemmArgs& g, hipStream_t s) {
  if (nf == 2) {
    switch (mt) {
      case 1: return launch_slices<1, 2>(g, s);
      case 2: return launch_slices<2, 2>(g, s);
      case 3: return launch_slices<3, 2>(g, s);
      case 4: return launch_slices<4, 2>(g, s);
      case 5: return launch_slices<5, 2>(g, s);
      case 6: return launch_slices<6, 2>(g, s);
      case 7: return launch_slices<7, 2>(g, s);
      case 8: return launch_slices<8, 2>(g, s);
      case 9: return launch_slices<9, 2>(g, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (nf == 4) {
    switch (mt) {
      case 1: return launch_slices<1, 4>(g, s);
      case 2: return launch_slices<2, 4>(g, s);
      case 3: return launch_slices<3, 4>(g, s);
      case 4: return launch_slices<4, 4>(g, s);
      case 5: return launch_slices<5, 4>(g, s);
      default: return hipErrorInvalidValue;
    }
  }
  return hipErrorInvalidValue;
}
