// The short tiles with stages of 64 k whose weights no cache holds until the next call: their lines are marked as not wanted again
// (which launch takes them, and what it measured: gemm_k64.hip).
#include "gemm_k64.h"

hipError_t launch_proj_k64_once(int mt, int nf, const GemmArgs& g, hipStream_t s) { return launch_k64_pairs<true>(mt, nf, g, s); }
