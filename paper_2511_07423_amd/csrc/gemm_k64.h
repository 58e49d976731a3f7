// The short tiles with stages of 64 k: 128 columns x 16 .. 144 rows (MT = 1 .. 9, NF = 2), 256 columns x 16 .. 80 rows (MT = 1 .. 5,
// NF = 4).  Calls f with the tile's MT and NF as types.
#pragma once
#include "gemm_tile.h"
#include <type_traits>

template <class F>
hipError_t with_short_tile(int mt, int nf, F&& f) {
#define SY_TILE(MT, NF) \
  if (mt == MT && nf == NF) return f(std::integral_constant<int, MT>{}, std::integral_constant<int, NF>{});
  SY_TILE(1, 2) SY_TILE(2, 2) SY_TILE(3, 2) SY_TILE(4, 2) SY_TILE(5, 2) SY_TILE(6, 2) SY_TILE(7, 2) SY_TILE(8, 2) SY_TILE(9, 2)
  SY_TILE(1, 4) SY_TILE(2, 4) SY_TILE(3, 4) SY_TILE(4, 4) SY_TILE(5, 4)
#undef SY_TILE
  return hipErrorInvalidValue;
}

// Activation pairs on the tile of gemm_tile.h (KSUB = 2).
template <bool ONCE>
hipError_t launch_k64_pairs(int mt, int nf, const GemmArgs& g, hipStream_t s) {
  return with_short_tile(mt, nf, [&](auto MT, auto NF) {
    constexpr int mt_ = decltype(MT)::value, nf_ = decltype(NF)::value;
    const int m_tiles = (g.M + 16 * mt_ - 1) / (16 * mt_), n_tiles = g.N / (64 * nf_);
    const dim3 grid(8 * ((n_tiles + 7) / 8) * m_tiles, 1, g.split_k);
    switch (g.epilogue) {
      case GEMM_STORE_F32: proj_kernel<mt_, nf_, GEMM_STORE_F32, true, 2, false, ONCE><<<grid, 256, 0, s>>>(g); break;
      case GEMM_ADD_F32: proj_kernel<mt_, nf_, GEMM_ADD_F32, true, 2, false, ONCE><<<grid, 256, 0, s>>>(g); break;
      case GEMM_SWIGLU: proj_kernel<mt_, nf_, GEMM_SWIGLU, true, 2, false, ONCE><<<grid, 256, 0, s>>>(g); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  });
}
