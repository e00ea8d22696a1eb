// Launches of the small-tile bf16 base products (gemm_ring.hip).
#pragma once

#include "gemm_mfma_kernel.h"

namespace mlora {

// `a` as for k_gemm_mfma (the tile counts and ranges are filled in here); `groups` of four waves per block: 1 or, for one
// operand pair, 2
template <int NSEG>
void launch_ring(gemmk::GemmArgs<NSEG> a, const SegTable& st, bool nn, int groups, int parts, float* scratch, hipStream_t s);

}  // namespace mlora
