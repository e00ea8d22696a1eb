// Host side of the small-tile bf16 base products (gemm_ring_kernel.h): launches.
#include "gemm_ring_kernel.h"
#include "gemm_ring.h"

namespace mlora {
namespace {

template <int G, bool NN, int NSEG>
void launch_tile(const gemmk::GemmArgs<NSEG>& a, hipStream_t s) {
  const int units = a.tiles_m * a.tiles_n;
  hipLaunchKernelGGL((ringk::k_gemm_ring<G, NN, NSEG>), dim3((unsigned)(units * a.parts)), dim3(256 * G), 0, s, a);
  launch_ring_reduce(a, s);
}

}  // namespace

template <int NSEG>
void launch_ring_reduce(const gemmk::GemmArgs<NSEG>& a, hipStream_t s) {
  const int units = a.tiles_m * a.tiles_n;
  if (a.parts == 1) return;
  ringk::RingReduceArgs r;
  r.C = a.C;
  r.part = a.part;
  r.M = a.M;
  r.N = a.N;
  r.tiles_m = a.tiles_m;
  r.tiles_n = a.tiles_n;
  r.parts = a.parts;
  r.K = a.K;
  for (int k = 0; k <= kMaxK; ++k) r.off[k] = a.off[k];
  hipLaunchKernelGGL(ringk::k_ring_reduce, dim3((unsigned)(4 * units)), dim3(256), 0, s, r);
}
template void launch_ring_reduce<1>(const gemmk::GemmArgs<1>&, hipStream_t);

template <int NSEG>
void ring_tiles(gemmk::GemmArgs<NSEG>* a, const SegTable& st, int parts, float* scratch) {
  a->tiles_m = (int)((virtual_rows(st, a->M) + 63) / 64);
  a->tiles_n = (a->N + 63) / 64;
  a->t0 = 0;
  a->parts = parts;
  a->part = scratch;
}
template void ring_tiles<1>(gemmk::GemmArgs<1>*, const SegTable&, int, float*);

template <int NSEG>
void launch_ring(gemmk::GemmArgs<NSEG> a, const SegTable& st, bool nn, int groups, int parts, float* scratch, hipStream_t s) {
  ring_tiles(&a, st, parts, scratch);
  if constexpr (NSEG == 1) {
    if (nn) return groups == 2 ? launch_tile<2, true, 1>(a, s) : launch_tile<1, true, 1>(a, s);
    if (groups == 2) return launch_tile<2, false, 1>(a, s);
  }
  launch_tile<1, false, NSEG>(a, s);
}
template void launch_ring<1>(gemmk::GemmArgs<1>, const SegTable&, bool, int, int, float*, hipStream_t);
template void launch_ring<2>(gemmk::GemmArgs<2>, const SegTable&, bool, int, int, float*, hipStream_t);
template void launch_ring<3>(gemmk::GemmArgs<3>, const SegTable&, bool, int, int, float*, hipStream_t);
template void launch_ring<4>(gemmk::GemmArgs<4>, const SegTable&, bool, int, int, float*, hipStream_t);

}  // namespace mlora
