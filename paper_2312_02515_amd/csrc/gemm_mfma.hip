// Host side of the bf16 MFMA base product with LoRA contraction steps: launch geometry.
// The kernel itself is in gemm_mfma_kernel.h.
//
//   forward  (Eq. "forward"):      Y  = X W   + Z B_k      (W is [h,d], contraction index = rows of W)
//   backward (Eq. "grad_output"):  dX = dY W^T + G A_k^T   (W is [h,d], contraction index = columns of W)
//
// where Z = s_k x_k A_k and G = s_k dy_k B_k^T are the [T, ldz] low-rank intermediates.  The
// base product is launched once over all tasks' rows; the output tile is written once with the
// LoRA term already in it (no full-size intermediate for the LoRA part of dX exists).
#include "gemm_mfma_kernel.h"
#include "gemm_ring.h"
#include "../../include/mlora_testing.h"
#include "mlora_common.h"

namespace mlora {
namespace {

constexpr int BM = 256, BN = gemmk::BN;

}  // namespace

// whole 16-byte chunks in every row
bool gemm_mfma_ok(int M, int N, int Kd) { return M >= 1 && (N % 8) == 0 && (Kd % 8) == 0 && N >= 8 && Kd >= 8; }

namespace {

template <int NSEG>
bool ragged_ranks(const gemmk::GemmArgs<NSEG>& a) {
  for (int g = 0; g < NSEG; ++g)
    for (int k = 0; k < a.K; ++k)
      if (a.rank[g][k] % 8 != 0) return true;
  return false;
}

// whether some contraction ends in a partial tile
template <int NSEG>
bool partial_tiles(const gemmk::GemmArgs<NSEG>& a) {
  for (int g = 0; g < NSEG; ++g)
    if (a.Kd[g] % 64 != 0) return true;
  return false;
}

// tiles [0, tiles) of 256 x 256
template <bool NN, int NSEG>
void launch_whole(const gemmk::GemmArgs<NSEG>& a, int tiles, hipStream_t stream) {
  if constexpr (!NN) {
    if (ragged_ranks(a)) {
      hipLaunchKernelGGL((gemmk::k_gemm_mfma<2, 4, false, NSEG, true>), dim3(tiles), dim3(512), 0, stream, a);
      return;
    }
  }
  // (without the code for partial contraction tiles where there are none: 16448 x 4096 -> 11008 forward, backward and
  // gradients 2406 -> 2396 us, 22548 x 192 -> 8064 490 -> 485.  Ragged ranks, which run one form: 3072 x 4096 -> 4096 with it 235,
  // without 234, 16000 x 5120 -> 13824 3347 and 3349)
  if (partial_tiles(a)) hipLaunchKernelGGL((gemmk::k_gemm_mfma<2, 4, NN, NSEG, false, true>), dim3(tiles), dim3(512), 0, stream, a);
  else hipLaunchKernelGGL((gemmk::k_gemm_mfma<2, 4, NN, NSEG, false, false>), dim3(tiles), dim3(512), 0, stream, a);
}

// tiles [a.t0, total) as halves of 128 x 256, their contraction in a.parts ranges
template <bool NN, int NSEG>
void launch_halves(const gemmk::GemmArgs<NSEG>& a, bool packed, hipStream_t stream) {
  const int units = 2 * (a.tiles_m * a.tiles_n - a.t0);
  const dim3 grid(units * a.parts);
  if (packed) hipLaunchKernelGGL((gemmk::k_gemm_mfma<1, 4, NN, NSEG, true>), grid, dim3(256), 0, stream, a);
  else if (partial_tiles(a)) hipLaunchKernelGGL((gemmk::k_gemm_mfma<1, 4, NN, NSEG, false, true>), grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL((gemmk::k_gemm_mfma<1, 4, NN, NSEG, false, false>), grid, dim3(256), 0, stream, a);
  if (a.parts == 1) return;
  gemmk::ReduceArgs r;
  r.C = a.C;
  r.part = a.part;
  r.M = a.M;
  r.N = a.N;
  r.tiles_m = a.tiles_m;
  r.tiles_n = a.tiles_n;
  r.t0 = a.t0;
  r.parts = a.parts;
  r.packed = packed;
  r.K = a.K;
  for (int k = 0; k <= kMaxK; ++k) r.off[k] = a.off[k];
  hipLaunchKernelGGL(gemmk::k_gemm_reduce, dim3(units * 8), dim3(256), 0, stream, r);
}

// How a product is cut into launches: tiles [0, whole) as 256 x 256 tiles, a multiple of 256 so that
// every round fills the chip, the others as halves of them with the contraction in `parts` ranges.
// A launch takes a round of blocks per 256 blocks; the plan with the smallest estimate wins.  The
// estimates are measured per block and contraction tile of 64 (us): whole tile 10 + 1.3 KT, half tile
// 12 + 0.78 KT, reduction 4 + 1 per 7 MB of partial tiles, taken before the loads were spread over the tile.  Launches of
// the present kernels, forward, N(0,1) data, 32 to 256 tiles deep: whole tiles 15 + 1.37 KT for one round, 1.40 KT a round for two
// and four; half tiles 6 + 0.83 KT for 256 blocks, 4 + 0.70 KT for 176 -- the ratio of the slopes is the same, 1.65.
// Before (whole tiles only) and after:
//   T = 100,   4096 x 4096   (16 tiles)        87 ->  28 us with 7 ranges
//   T = 771,   2048 -> 5632  (88 tiles)        50 ->  38 us as halves
//              its input gradient (32 tiles)  103 ->  42 us as halves, 3 ranges
//   T = 2048,  11008-deep input gradient (128 tiles) 207 -> 165 us as halves
//   T = 2048,  4096 -> 11008 (344 tiles)      191 -> 171 us, one whole round and halves
//   T = 16448, 11008-deep input gradient (1040 tiles) 1227 -> 1090 us, four whole rounds and halves
//   summed input gradient of q, k, v (4096 each): T = 128  250 -> 48 us, T = 512  233 -> 79 us,
//   T = 2048  237 -> 182 us; T = 16448  1447 -> 1354 us
//   T = 3072,  4096 x 4096   (192 tiles): halves would take 125 us instead of 93.
// LoRA: every 64 ranks of a task beyond the first 64 of the tile's first task add 4.7 us to a whole tile (a
// LoRA tile of the pipeline); in a half tile, which holds half as many tasks, each further task adds 1.5 us
// per 32 ranks, and ranks above 64 add 5 us.  Behind full rounds the caches are cold for it: 4 us per 32
// ranks beyond the first 32; and a last round of at most 128 whole tiles takes 0.85 of a full one there.
// Forward, rank 128: 20000 x 2048 x 2048 195 us in whole tiles (201 as two rounds and halves), 12288 x 512
// -> 2048 57 (63), 128 x 256 x 256 22.4 (23.8), but 16 x 1024 x 1024 41 us in whole tiles, 25 as halves.
//
// Small tiles (gemm_ring_kernel.h), 64 x 64 and of one or two groups of four waves, for up to 64 tiles of 256 x 256, or 128
// that are no more than five small ones per CU.
// Estimates (us, measured; n tiles of `steps` contraction and LoRA tiles): one group 5 + m (0.9 + 0.19 steps), m tiles on
// the fullest CU, but 0.25 a step for one that it runs by itself (three fit a CU, so a first, fourth, .. one: with 918
// blocks counted as 3.6 a CU, 3230 x 7248 -> 368 took 54 + 6 us, in half tiles 40 + 6); two groups, for up to 256 tiles,
// 6.3 + 0.4 per two steps; the reduction of ranges as above.  Half or whole tiles -> small tiles, forward and backward
// product, us:
//   128 rows, 256 -> 256, rank 64   15.5, 14.1 ->  6.7,  6.9     1024 x 1024 -> 1024, rank 64   23.7, 22.0 -> 10.2, 10.4
//   220 rows, 1920 -> 2688 (10 tasks)  30.2, 26.6 -> 13.0, 14.9     2048 x 1024 -> 1024   24.8, 23.3 -> 12.9, 12.7
//   1024 x 4096 -> 1024   27.2, 21.7 -> 20.1, 22.6     2048 x 2048 -> 2048   36.0, 33.5 -> 33.3, 32.5
//   beyond: 3000 x 512 -> 2944  22.7 and 31.8 forward; 771 x 2048 -> 5632  34 and 36.  Where the estimates are level the larger
//   tiles stay (771 x 5632 -> 2048: level in a loop, 38 us, and 2 % slower behind other launches).
// The estimate has to be 7 % lower; with more than 64 tiles of 256 x 256, or weights of 32 MiB and more, which small tiles read from
// HBM or the Infinity Cache several times over, 15 %.  Forward calls of 88 sizes from 8 to 700 rows with such weights: none of those
// that the rule takes lost, and with 7 % one, by 8 % (256 x 11008 -> 4096).  Half tiles -> small tiles, us of the call:
//   100 x 4096 -> 4096  31 -> 25     32 x 4096 -> 11008  40 -> 28     100 x 8192 -> 8192  51 -> 42     8 x 2048 -> 8192  28 -> 19
//   30 x 9752 -> 6144 (2 tasks)  72 -> 36     25 x 1824 -> 10296  34 -> 18     50 x 4896 -> 4072 (11 tasks)  50 -> 41
//   2740 x 368 -> 1600 (84 tiles)  24.4 -> 21.6     3191 x 312 -> 1232 (65; now the general kernel, 18.7)  20.0 -> 18.1
//   4291 x 64 -> 1536 (1656 small tiles)  stays: a step 70.8 us, 73.0
constexpr int kSmallTiles = 64, kMostTiles = 128, kMostSmallTiles = 5 * 256;
struct Plan {
  int whole, parts;
  int small;          // groups of four waves per 64 x 64 tile; 0: 256 x 256 tiles and halves
  bool packed;        // halves: rows of several tasks in a piece of 32
  double us;          // small tiles: the estimate
};
constexpr int kMaxParts = 16;
constexpr size_t kSmallWeight = (size_t)32 << 20;
// the fewest us of a product in small tiles, and its plan
double plan_small(const SegTable& st, int M, int N, int KT, int pairs, size_t scratch_limit, Plan* out) {
  const long long n = (virtual_rows(st, M) + 63) / 64 * ((N + 63) / 64);
  // LoRA tiles of a block: two slots of 32 ranks each, for one or two tasks
  int slots = 0, live = 0;
  for (int k = 0; k < st.K; ++k) {
    if (st.off[k + 1] == st.off[k]) continue;
    ++live;
    const int r = (st.rank[k] + 31) / 32;
    slots = r > slots ? r : slots;
  }
  const bool shared = live > 1 && (long long)(st.off[st.K] - st.off[0]) < 64LL * live;   // most tiles hold two tasks
  const int lora = pairs * (shared ? slots : (slots + 1) / 2);
  double best = 0;
  for (int p = 1; p <= kMaxParts && 2 * p <= KT + 1; ++p) {
    const size_t bytes = p > 1 ? (size_t)n * p * 64 * 64 * sizeof(float) : 0;
    if (bytes > scratch_limit) break;
    const int steps = (KT + p - 1) / p + lora;
    const long long m = (n * p + 255) / 256, alone = m % 3 == 1 ? 1 : 0;   // blocks of a CU, those that run by themselves
    const double us = 5.0 + (double)(m - alone) * (0.9 + 0.19 * steps) + (double)alone * (0.9 + 0.25 * steps) +
                      (p > 1 ? 4.0 + (double)bytes / 7e6 : 0.0);
    if (p == 1 || us < best) {
      best = us;
      *out = Plan{0, p, 1, false, us};
    }
    if (p == 1 && n <= 256 && pairs == 1 && 6.3 + 0.4 * ((steps + 1) / 2) < best) {
      best = 6.3 + 0.4 * ((steps + 1) / 2);
      *out = Plan{0, 1, 2, false, best};
    }
  }
  return best;
}
// (`pairs` operand pairs of Kd contraction indices in all; KT contraction tiles)
Plan plan_gemm(const SegTable& st, int M, int N, int KT, int pairs, size_t scratch_limit) {
  const int tiles_m = (int)((virtual_rows(st, M) + BM - 1) / BM), tiles_n = (N + BN - 1) / BN;
  const int total = tiles_m * tiles_n, q = total / 256 * 256, halves = 2 * (total - q);
  // tasks of a tile beyond the first: the most of any tile where a tile's time shows, on average in several
  // rounds
  int live = 0, rmax = 0, most_whole = 0, most_half = 0;
  {
    int tile_w = -1, tile_h = -1, in_w = 0, in_h = 0;
    long long v = (st.off[0] + 31) / 32 * 32;
    for (int k = 0; k < st.K; ++k) {
      rmax = st.rank[k] > rmax ? st.rank[k] : rmax;
      const int len = st.off[k + 1] - st.off[k];
      if (len == 0) continue;
      ++live;
      auto enter = [&](int rows, int& tile, int& in, int& most) {
        const int first = (int)(v / rows), last = (int)((v + len - 1) / rows);
        in = first == tile ? in + 1 : 1;
        most = in > most ? in : most;
        if (last > first) in = 1;
        tile = last;
      };
      enter(BM, tile_w, in_w, most_whole);
      enter(BM / 2, tile_h, in_h, most_half);
      v += (len + 31) / 32 * 32;
    }
  }
  auto others = [&](int tiles, int most) {
    const int n = total > 256 ? (live + tiles - 1) / tiles : most;
    return pairs * (n > 0 ? (n < most ? n : most) - 1 : 0);
  };
  const int r64 = rmax > 0 ? (rmax + 63) / 64 : 1, r32 = rmax > 0 ? (rmax + 31) / 32 : 1;
  const double whole_fixed = 10.0 + 4.7 * (pairs * (r64 - 1) + others(tiles_m, most_whole) * r64);
  const double half_fixed =
      12.0 + pairs * (q > 0 ? 4.0 * (r32 - 1) : (r32 > 2 ? 5.0 : 0.0)) + 1.5 * others(2 * tiles_m, most_half) * r32;
  auto whole_us = [&](int tiles) {
    const int last = tiles % 256;
    const double part = last == 0 ? 0.0 : (tiles > 256 && last <= 128 ? 0.85 : 1.0);
    return (tiles / 256 + part) * (whole_fixed + 1.3 * KT);
  };
  Plan best{total, 1, 0, false, 0};
  double best_us = whole_us(total);
  for (int parts = 1; halves > 0 && parts <= kMaxParts && parts <= KT; ++parts) {
    const size_t bytes = parts > 1 ? (size_t)halves * parts * (BM / 2) * BN * sizeof(float) : 0;
    if (bytes > scratch_limit) break;
    const double us = whole_us(q) + (double)((halves * parts + 255) / 256) * (half_fixed + 0.78 * ((KT + parts - 1) / parts)) +
                      (parts > 1 ? 4.0 + (double)bytes / 7e6 : 0.0);
    if (us < best_us) {
      best_us = us;
      best = Plan{q, parts, 0, false, 0};
    }
  }
  if (packed_rows(st, M)) {
    // half tiles of packed rows: the tasks' LoRA terms one after the other
    const int halves_p = 2 * (int)((M + 255LL) / 256 * tiles_n), in_tile = (int)((long long)live * 128 / M) + 2;
    const double fixed = 12.0 + pairs * 1.5 * ((in_tile < live ? in_tile : live) * r32 - 1);
    for (int parts = 1; parts <= kMaxParts && parts <= KT; ++parts) {
      const size_t bytes = parts > 1 ? (size_t)halves_p * parts * (BM / 2) * BN * sizeof(float) : 0;
      if (bytes > scratch_limit) break;
      const double us = (double)((halves_p * parts + 255) / 256) * (fixed + 0.78 * ((KT + parts - 1) / parts)) +
                        (parts > 1 ? 4.0 + (double)bytes / 7e6 : 0.0);
      if (us < 0.93 * best_us) {
        best_us = us / 0.93;
        best = Plan{0, parts, 0, true, 0};
      }
    }
  }
  Plan small;
  const double margin = total <= kSmallTiles && (size_t)N * KT * 64 * sizeof(bf16) < kSmallWeight ? 0.93 : 0.85;
  if ((total <= kSmallTiles || (total <= kMostTiles && (virtual_rows(st, M) + 63) / 64 * ((N + 63) / 64) <= kMostSmallTiles)) &&
      plan_small(st, M, N, KT, pairs, scratch_limit, &small) < margin * best_us)
    return small;
  return best;
}

// The smallest problems run k_gen_skinny (16 x 64 tiles, operands straight from memory): 128 rows 256 -> 256, rank 64 4.9
// and 5.1 us, in 64 x 64 tiles 6.7 and 6.9; 128 x 1024 -> 256 6.7 and 5.2, 9.4 and 6.6; 1024 x 64 -> 1024 6.4 and 8.6, 6.3 and 9.0.
bool skinny(const SegTable& st, int M, int N, long long Kd) {
  return (virtual_rows(st, M) + BM - 1) / BM * ((N + BN - 1) / BN) <= kSmallTiles && general_skinny(st, M, N, Kd, MLORA_BF16);
}

// Forward products whose features are no multiples of 64 that the general kernel runs: its tiles, of 64 x 64 or 128 x 128, fill the
// chip where those of this file leave CUs idle.  Call, us, the plan above -> the general kernel:
//   between three and four small tiles per CU, seven contraction tiles deep at most (a CU holds five of the general kernel's):
//     641 x 200 -> 4504 16.4 -> 14.7, 1527 x 240 -> 2136 (10 tasks) 18.2 -> 16.2, 700 x 136 -> 4504 15.8 -> 15.1, 1500 x 328 -> 2136
//     18.5 -> 17.6, 700 x 392 -> 4504 19.7 -> 19.5; with 756 tiles (300 x 200 -> 8008) 13.5 and 14.2, beyond 1024 larger tiles.
//   ranks of 16 at most, one or two tiles of 128 x 128 per CU, two to five contraction tiles: of 26 calls none lost.  1826 x 152 -> 2128
//     19.8 -> 12.6, 668 x 120 -> 8648 (10 tasks) 24.3 -> 16.0, 1500 x 136 -> 4504 21.6 -> 16.5, 10829 x 200 -> 328 21.7 -> 18.3,
//     3002 x 256 -> 2248 18.1 -> 17.6; at rank 32 7163 x 272 -> 608 19.2 and 19.5, 17 contraction tiles at rank 64 35.0 and 39.3.
//   ranks of 16 at most, whole tiles whose second round is no more than half full, two to eight contraction tiles: of 19 calls none lost.  1419 x 280 ->
//     10808 48.6 -> 33.0, 13691 x 144 -> 1304 (10 tasks) 49.1 -> 37.7, 3000 x 152 -> 8008 45.9 -> 37.8, 2638 x 392 -> 7440 55.3 -> 45.5,
//     2673 x 384 -> 8416 (10 tasks) 46.8 -> 46.6; with nine tiles 2636 x 536 -> 7840 55.4 and 59.7, 420 tiles of 256 x 256 59.4 and 64.4.
bool general_forward(const SegTable& st, int M, int N, int Kd, const Plan& pl) {
  if ((N % 64 == 0 && Kd % 64 == 0) || pl.parts > 1 || pl.packed) return false;
  const long long v = virtual_rows(st, M);
  if (pl.small > 0) {
    const long long n = (v + 63) / 64 * ((N + 63) / 64);
    return n > 3 * 256 && n <= 4 * 256 && Kd <= 7 * 64;
  }
  int rmax = 0;
  for (int k = 0; k < st.K; ++k) rmax = st.rank[k] > rmax ? st.rank[k] : rmax;
  if (rmax > 16 || Kd <= 64) return false;
  const long long whole = (v + BM - 1) / BM * ((N + BN - 1) / BN), quarters = (v + 127) / 128 * ((N + 127) / 128);
  return (quarters > 256 && quarters <= 512 && Kd <= 5 * 64) || (pl.whole == whole && whole > 256 && whole <= 384 && Kd <= 8 * 64);
}

template <int NSEG>
void fill_common(gemmk::GemmArgs<NSEG>* a, bf16* C, int M, int N, const SegTable& st) {
  a->C = C;
  a->M = M;
  a->N = N;
  a->tiles_n = (N + BN - 1) / BN;
  a->K = st.K;
  for (int k = 0; k <= kMaxK; ++k) a->off[k] = st.off[k];
  a->tiles_m = (int)((virtual_rows(st, M) + BM - 1) / BM);
  a->t0 = 0;
  a->parts = 1;
  a->part = nullptr;
}

template <bool NN, int NSEG>
hipError_t launch(gemmk::GemmArgs<NSEG>& a, float* scratch, size_t scratch_bytes, const SegTable& st,
                  hipStream_t stream) {
  int kt = 0;
  for (int g = 0; g < NSEG; ++g) kt += (a.Kd[g] + 63) / 64;
  const Plan pl = plan_gemm(st, a.M, a.N, kt, NSEG, scratch_bytes);
  a.t0 = pl.whole;
  a.parts = pl.parts;
  a.part = scratch;
  const int slot = profile_begin(kProfileGemm, product_work(a), stream);
  if (pl.small > 0) {
    launch_ring<NSEG>(a, st, NN, pl.small, pl.parts, scratch, stream);
    const hipError_t e = hipGetLastError();
    profile_end(slot, stream);
    return e;
  }
  if (pl.whole > 0) launch_whole<NN, NSEG>(a, pl.whole, stream);
  if (pl.packed) a.tiles_m = (a.M + BM - 1) / BM;
  if (pl.whole < a.tiles_m * a.tiles_n) launch_halves<NN, NSEG>(a, pl.packed, stream);
  const hipError_t err = hipGetLastError();
  profile_end(slot, stream);
  return err;
}

template <int NSEG>
hipError_t launch_sum(const GemmOperands* ops, bf16* C, int M, int N, const SegTable& st, float* scratch, size_t scratch_bytes,
                      hipStream_t stream) {
  gemmk::GemmArgs<NSEG> a;
  fill_common(&a, C, M, N, st);
  for (int g = 0; g < NSEG; ++g) {
    a.A[g] = ops[g].A;
    a.Bm[g] = ops[g].Bm;
    a.L[g] = ops[g].L;
    a.Kd[g] = ops[g].Kd;
    a.ldz[g] = ops[g].ldz;
    for (int k = 0; k < kMaxK; ++k) a.rank[g][k] = (unsigned char)(k < st.K ? ops[g].rank[k] : 0);
    a.R[g] = *ops[g].R;
  }
  return launch<false, NSEG>(a, scratch, scratch_bytes, st, stream);
}

}  // namespace

// C[M,N] = A[M,Kd] * (nn ? Bm[Kd,N] : Bm[N,Kd]^T) + rows_k( L[rows_k, :r_k] * (nn ? R_k[r_k,N] : R_k[N,r_k]^T) )
hipError_t gemm_mfma(const bf16* A, const bf16* Bm, bf16* C, int M, int N, int Kd, bool nn, const bf16* L, int ldz,
                     const SegTable& st, const PtrTable& R, float* scratch, size_t scratch_bytes, hipStream_t stream) {
  if (skinny(st, M, N, Kd) || (nn && general_forward(st, M, N, Kd, plan_gemm(st, M, N, (Kd + 63) / 64, 1, scratch_bytes)))) {
    const GenOperands o{A, Bm, L, Kd, ldz, st.rank, &R};
    return general_gemm(1, &o, MLORA_BF16, C, M, N, nn, st, scratch, scratch_bytes, stream);
  }
  gemmk::GemmArgs<1> a;
  fill_common(&a, C, M, N, st);
  a.A[0] = A;
  a.Bm[0] = Bm;
  a.L[0] = L;
  a.Kd[0] = Kd;
  a.ldz[0] = ldz;
  for (int k = 0; k < kMaxK; ++k) a.rank[0][k] = (unsigned char)(k < st.K ? st.rank[k] : 0);
  a.R[0] = R;
  return nn ? launch<true, 1>(a, scratch, scratch_bytes, st, stream)
            : launch<false, 1>(a, scratch, scratch_bytes, st, stream);
}

bool gemm_small_us(const SegTable& st, int M, int N, int Kd, size_t limit, double* us) {
  if (skinny(st, M, N, Kd)) {
    *us = general_skinny_us(st, M, N, Kd, MLORA_BF16);
    return true;
  }
  const Plan pl = plan_gemm(st, M, N, (Kd + 63) / 64, 1, limit);
  *us = pl.us;
  return pl.small > 0;
}

SmallForm gemm_small_nt(const bf16* A, const bf16* Bm, bf16* C, int M, int N, int Kd, const bf16* L, int ldz, const SegTable& st,
                        const PtrTable& R, size_t limit, gemmk::GemmArgs<1>* a, int* groups, int* parts) {
  if (skinny(st, M, N, Kd)) return kSkinny;
  const Plan pl = plan_gemm(st, M, N, (Kd + 63) / 64, 1, limit);
  if (pl.small == 0) return kNotSmall;
  fill_common(a, C, M, N, st);
  a->A[0] = A;
  a->Bm[0] = Bm;
  a->L[0] = L;
  a->Kd[0] = Kd;
  a->ldz[0] = ldz;
  for (int k = 0; k < kMaxK; ++k) a->rank[0][k] = (unsigned char)(k < st.K ? st.rank[k] : 0);
  a->R[0] = R;
  *groups = pl.small;
  *parts = pl.parts;
  return kRing;
}

GemmForm gemm_form(const SegTable& st, int M, int N, int n, const int* Kd, bool nn, size_t scratch_bytes) {
  const long long mv = virtual_rows(st, M), total = (mv + BM - 1) / BM * ((N + BN - 1) / BN);
  long long kd = 0;
  int kt = 0;
  for (int g = 0; g < n; ++g) {
    kd += Kd[g];
    kt += (Kd[g] + 63) / 64;
  }
  auto tiles = [&](int rows) { return (int)((mv + rows - 1) / rows * ((N + 63) / 64)); };
  if (skinny(st, M, N, kd)) return GemmForm{MLORA_FORM_SKINNY, 1, tiles(16), tiles(16), 16};
  const Plan pl = plan_gemm(st, M, N, kt, n, scratch_bytes);
  if (nn && general_forward(st, M, N, Kd[0], pl)) {
    const int* const rank = st.rank;
    return general_gemm_form(st, M, N, 1, Kd, &rank, true, MLORA_BF16, scratch_bytes);
  }
  if (pl.small > 0) return GemmForm{MLORA_FORM_RING, pl.parts, tiles(64), tiles(64), 64};
  if (pl.packed) return GemmForm{MLORA_FORM_HALVES, pl.parts, 0, (M + BM - 1) / BM * ((N + BN - 1) / BN), BM / 2};
  const int form = pl.whole == total ? MLORA_FORM_WHOLE : (pl.whole == 0 ? MLORA_FORM_HALVES : MLORA_FORM_MIXED);
  return GemmForm{form, pl.parts, pl.whole, (int)total, form == MLORA_FORM_WHOLE ? BM : BM / 2};
}

size_t gemm_partial_bytes(int K, int T, int N, int Kd) {
  const long long mv = most_virtual_rows(K, T), tiles = (mv + BM - 1) / BM * ((N + BN - 1) / BN);
  const int kt = (Kd + 63) / 64, parts = kt < kMaxParts ? kt : kMaxParts;
  return parts > 1 ? (size_t)(2 * (tiles < 255 ? tiles : 255)) * parts * (BM / 2) * BN * sizeof(float) : 0;
}

// C[M,N] = sum_g ( A_g[M,Kd_g] * Bm_g[N,Kd_g]^T + rows_k( L_g[rows_k, :r_gk] * R_gk[N,r_gk]^T ) ), 1 <= n <= 4
hipError_t gemm_mfma_sum_nt(int n, const GemmOperands* ops, bf16* C, int M, int N, const SegTable& st, float* scratch,
                            size_t scratch_bytes, hipStream_t stream) {
  long long kd = 0;
  GenOperands o[MLORA_MAX_GROUP];
  if (n < 1 || n > MLORA_MAX_GROUP) return hipErrorInvalidValue;
  for (int g = 0; g < n; ++g) {
    kd += ops[g].Kd;
    o[g] = GenOperands{ops[g].A, ops[g].Bm, ops[g].L, ops[g].Kd, ops[g].ldz, ops[g].rank, ops[g].R};
  }
  if (skinny(st, M, N, kd))
    return general_gemm(n, o, MLORA_BF16, C, M, N, false, st, scratch, scratch_bytes, stream);
  switch (n) {
    case 1: return launch_sum<1>(ops, C, M, N, st, scratch, scratch_bytes, stream);
    case 2: return launch_sum<2>(ops, C, M, N, st, scratch, scratch_bytes, stream);
    case 3: return launch_sum<3>(ops, C, M, N, st, scratch, scratch_bytes, stream);
    case 4: return launch_sum<4>(ops, C, M, N, st, scratch, scratch_bytes, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace mlora
