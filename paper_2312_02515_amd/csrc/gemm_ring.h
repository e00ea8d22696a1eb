// Launches of the small-tile bf16 base products (gemm_ring.hip).
#pragma once

#include "gemm_mfma_kernel.h"

namespace mlora {

// `a` as for k_gemm_mfma (the tile counts and ranges are filled in here); `groups` of four waves per block: 1 or, for one
// operand pair, 2
template <int NSEG>
void launch_ring(gemmk::GemmArgs<NSEG> a, const SegTable& st, bool nn, int groups, int parts, float* scratch, hipStream_t s);

// fills in the tile counts and ranges; adds the ranges (nothing to do for one)
template <int NSEG>
void ring_tiles(gemmk::GemmArgs<NSEG>* a, const SegTable& st, int parts, float* scratch);
template <int NSEG>
void launch_ring_reduce(const gemmk::GemmArgs<NSEG>& a, hipStream_t s);

// whether an input gradient runs in small tiles (within `limit` bytes of scratch), and the estimate for it in us
bool gemm_small_us(const SegTable& st, int M, int N, int Kd, size_t limit, double* us);
// C = A Bm^T + rows_k(L R_k^T) (an input gradient) where the plan runs it in small tiles: the arguments of the ring kernel
// in `a`, its groups and ranges (within `limit` bytes of scratch)
enum SmallForm { kNotSmall = 0, kSkinny = 1, kRing = 2 };
SmallForm gemm_small_nt(const bf16* A, const bf16* Bm, bf16* C, int M, int N, int Kd, const bf16* L, int ldz, const SegTable& st,
                        const PtrTable& R, size_t limit, gemmk::GemmArgs<1>* a, int* groups, int* parts);

}  // namespace mlora
