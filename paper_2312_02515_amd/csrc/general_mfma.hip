// General kernels: every shape, segment layout, rank and alignment, in fp32 or bf16 storage, on the
// matrix pipes with fp32 accumulation.  They carry the fp32 mode and every bf16 problem whose
// sizes or addresses the direct-to-LDS kernels (gemm_mfma_kernel.h, lowrank_mfma.hip) do not take.
//
// Steps (section 3.3.1 of the mLoRA paper, with the scaling s_k folded into the low-rank
// intermediates):
//   forward :  Z = s_k x_k A_k            (k_gen_rows)
//              Y = X W + Z B_k            (k_gen_gemm, W [h,d] read along its rows)
//   backward:  G = s_k dy_k B_k^T         (k_gen_rows)
//              dB_k = Z^T dy_k            (k_gen_grad)
//              dX = dY W^T + G A_k^T      (k_gen_gemm, W [h,d] as the transposed operand)
//              dA_k = x_k^T G             (k_gen_grad)
//
// fp32 products run on v_mfma_f32_32x32x2_f32 / 16x16x4_f32 (IEEE fp32 multiply-adds), bf16 ones on
// the bf16 MFMAs; any assignment of contraction indices to MFMA slots is correct as long as both
// operands use the same one, which is what lets a lane feed its four MFMAs from one 16-byte piece.
#include <type_traits>

#include "gemm_ring.h"
#include "gemm_ring_kernel.h"
#include "mfma_staging.h"
#include "../../include/mlora_testing.h"
#include "mlora_common.h"
#include "row_axis.h"

namespace mlora {
namespace {

using namespace stage;
using namespace rowaxis;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

// 16 bytes at an address that is only a multiple of the element size (global memory takes them at
// any alignment; a misaligned piece costs a second cache line)
template <typename T> struct Piece16;
template <> struct Piece16<float> {
  typedef unsigned type __attribute__((ext_vector_type(4), aligned(4)));
};
template <> struct Piece16<bf16> {
  typedef unsigned type __attribute__((ext_vector_type(4), aligned(2)));
};
template <typename T> constexpr int kV = 16 / (int)sizeof(T);   // elements per 16-byte piece

// Elements i .. i + V - 1 of a row of n elements.  A piece that crosses the row's end is loaded so
// that it ends there; tail_shift() moves it into place and fills with zeros (rows shorter than one
// piece are put together element by element, already in place).
template <typename T>
__device__ __forceinline__ u32x4 load_piece(const T* row, int i, int n) {
  constexpr int V = kV<T>;
  if (n >= V) {
    const int s = i < n - V ? i : n - V;
    return *reinterpret_cast<const typename Piece16<T>::type*>(row + s);
  }
  union {
    u32x4 v;
    T e[V];
  } u;
  u.v = u32x4{0, 0, 0, 0};
#pragma unroll
  for (int e = 0; e < V; ++e)
    if (i + e < n) u.e[e] = row[i + e];
  return u.v;
}
template <typename T>
__device__ __forceinline__ u32x4 tail_shift(u32x4 v, int i, int n) {
  constexpr int V = kV<T>;
  if (n < V) return v;
  const int d = i - (n - V);
  if (d <= 0) return v;
  if (d >= V) return u32x4{0, 0, 0, 0};
  const int bits = d * 8 * (int)sizeof(T);
  const unsigned __int128 x = __builtin_bit_cast(unsigned __int128, v) >> bits;
  return __builtin_bit_cast(u32x4, x);
}

// acc += a x b over one 16-byte piece per lane of each operand (32 rows x 32 columns)
__device__ __forceinline__ void mma32(f32x16& acc, u32x4 a, u32x4 b, bf16) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
__device__ __forceinline__ void mma32(f32x16& acc, u32x4 a, u32x4 b, float) {
  const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[e], y[e], acc, 0, 0, 0);
}
// ... for FM x FN such accumulators; fp32: one contraction pair after the other, so that an accumulator
// comes up again only FM x FN MFMAs later
template <int FM, int FN>
__device__ __forceinline__ void mma_tile(f32x16 (&acc)[FM][FN], const u32x4 (&a)[FM], const u32x4 (&b)[FN], bf16) {
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) mma32(acc[i][j], a[i], b[j], bf16{});
}
template <int FM, int FN>
__device__ __forceinline__ void mma_tile(f32x16 (&acc)[FM][FN], const u32x4 (&a)[FM], const u32x4 (&b)[FN], float) {
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(f32x4, a[i])[e], __builtin_bit_cast(f32x4, b[j])[e],
                                                         acc[i][j], 0, 0, 0);
}
// the same on 16 rows x 16 columns
__device__ __forceinline__ void mma16(f32x4& acc, u32x4 a, u32x4 b, bf16) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
__device__ __forceinline__ void mma16(f32x4& acc, u32x4 a, u32x4 b, float) {
  const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
  for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[e], y[e], acc, 0, 0, 0);
}

// Scheduling of straight-line code of n MFMAs: behind each a memory instruction and two of vector
// arithmetic, as long as there are any
template <int n>
__device__ __forceinline__ void interleave() {
#pragma unroll
  for (int m = 0; m < n; ++m) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // an MFMA
    __builtin_amdgcn_sched_group_barrier(0x320, 1, 0);   // a load, an LDS read or write
    __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);   // vector arithmetic
  }
}

// ------------------------------------------------------------------------------------------
// C[M,N] = sum_g ( A_g[M,Kd_g] * op(W_g) + rows_k( L_g[rows_k, :r_gk] * R_gk ) )
//   NN = true : W_g [Kd_g, N], R_gk [r_gk, N]      NN = false: W_g [N, Kd_g], R_gk [N, r_gk]
// ------------------------------------------------------------------------------------------
template <int NSEG>
struct GenGemmArgs {
  void* C;
  float* part;                           // fp32 partial tiles when parts > 1
  int M, N, tiles_m, tiles_n, parts;
  int units;                             // tiles of the launch (times parts: its blocks)
  int t0;                                // quarters: the first 128 x 128 tile (of tiles_m x tiles_n) cut into them
  int K;
  int off[kMaxK + 1];
  const void* A[NSEG];
  const void* W[NSEG];
  const void* L[NSEG];
  int Kd[NSEG];
  int ldz[NSEG];
  unsigned char rank[NSEG][kMaxK];
  PtrTable R[NSEG];
};

// Block id -> (tile, part).  Consecutive ids go round-robin over the 8 XCDs; each XCD takes a
// contiguous eighth of the order (8 row tiles x all column tiles at a time, column by column), so
// that the blocks it runs together share operand strips in its L2.  `unit` numbers the partial tiles.
struct BlockTile {
  int tm, tn, part, unit;
};
template <bool QUARTERS, typename Args>
__device__ __forceinline__ BlockTile tile_of_unit(const Args& a, int u) {
  const int t = QUARTERS ? a.t0 + u / 4 : u;
  constexpr int GM = 8;
  const int gsize = GM * a.tiles_n;
  const int group = t / gsize, first = group * GM;
  const int gm = (a.tiles_m - first) < GM ? (a.tiles_m - first) : GM;
  const int in_g = t - group * gsize;
  const int tm = first + in_g % gm, tn = in_g / gm;
  return QUARTERS ? BlockTile{2 * tm + u % 4 / 2, 2 * tn + u % 2, 0, u} : BlockTile{tm, tn, 0, u};
}
template <bool QUARTERS, typename Args>
__device__ __forceinline__ BlockTile block_tile(const Args& a, int bid) {
  const int per = a.units * a.parts / 8;
  const int t = bid < per * 8 ? (bid % 8) * per + bid / 8 : bid;
  BlockTile b = tile_of_unit<QUARTERS>(a, t / a.parts);
  b.part = t % a.parts;
  return b;
}

// Output column behind column n of the grid's tiles (-1: none).  NN: the weight's rows are loaded in pieces of V
// columns; the piece that crosses the right edge is loaded so that it ends there and is not shifted into
// place, so its V columns are the output's last V.  Those that belong to the piece before it are not stored: that
// piece may lie in a tile whose contraction is cut into other ranges.  (Shifted
// into place tile by tile, the blocks at the right edge took up to twice as long and every launch waited for
// them: forward, fp32 3000 x 4001 -> 4001 956 us against 728, 913 x 1000 -> 1500 67 against 44, bf16 156
// against 127 for 2048 x 4100 -> 4100.)
template <typename T, bool NN>
__device__ __forceinline__ int real_column(int n, int N) {
  constexpr int V = kV<T>;
  const int piece = n / V * V;
  if (NN && N >= V && piece < N && piece + V > N) return N - V + n % V >= piece ? N - V + n % V : -1;
  return n < N ? n : -1;
}

// C element store of one 32 x 32 accumulator: lane holds column `col` (-1: none) and rows 8 g + 4 lhi + e
template <typename T>
__device__ __forceinline__ void store_frag(const f32x16& acc, T* C, int N, const RowPiece& p, int col, int lhi) {
  if (col >= 0) {
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int o = 8 * g + 4 * lhi + e;
        if (o < p.n) C[(size_t)(p.row + o) * N + col] = from_f32<T>(acc[4 * g + e]);
      }
  }
}

// Tile BM x BN, 4 waves as 2 x 2, contraction tiles of 128 bytes per row (64 bf16 or 32 fp32).
// Operands go through registers into two LDS stages: the pieces of tile kt+2 are requested while
// tile kt is multiplied and written to LDS a tile later, so a load has one whole tile of MFMAs to
// land, and tails, short rows and odd strides are handled between the load and the LDS write.
// K-contiguous tiles keep 16-byte piece c of row r at c ^ ((r >> 1) & 7) (conflict-free b128 reads);
// the NN weight tile keeps its rows as they are in memory (bf16: pieces permuted for the
// transposing reads; fp32: read element by element, 32 columns of a row at a time).
// The LoRA term is added from registers at the end, 32-row piece by piece: L and R_k come straight
// from memory (r_k <= 128 contraction indices against thousands).
// With parts > 1 a tile's contraction is cut into `parts` ranges, one block each; the partial tiles
// go to memory in fp32 and k_gen_reduce adds them in order.
// A tile's LDS writes and the next loads are issued between its MFMA groups, whose fragments are read
// one group ahead; tiles that need no masks load without bounds arithmetic.
// Bound by the fp32 matrix rate in fp32 (153 TFLOP/s for a large product on this card).  Median and least of
// 20 traced passes: T = 2048, 4096 x 4096 561 and 513 us forward, 551 and 503 us backward layout (1714 and
// 1686 us on the vector ALUs; an untraced forward and backward pass takes 1060 us, of which the low-rank
// launches are 57); T = 1024 300 and 287, 293 and 280 us.  bf16, T = 2048, 4100 x 4100, whole tiles and quarters: 113 and
// 119 us, bound by LDS traffic and the wait for each tile's loads.
// QUARTERS: tiles of 64 x 64 that are quarters of 128 x 128 tiles.
// PACKED (64 x 64): many tasks of few rows, whose pieces of 32 rows would hold few rows each: pieces hold rows of several
// tasks, and the LoRA term is added task by task, to the task's own rows only (a select, no product with zeros).
template <int BM, int BN> constexpr int kGemmLds = 2 * (BM + BN) * 128;
template <typename T, int BM, int BN, bool NN, int NSEG, bool QUARTERS, bool PACKED>
__device__ __forceinline__ void gemm_body(const GenGemmArgs<NSEG>& a, int bid, char* sm) {
  constexpr int V = kV<T>, BK = 8 * V;
  constexpr int WM = BM / 2, WN = BN / 2, FM = WM / 32, FN = WN / 32;
  constexpr int NA = BM / 32, NB = BN / 32;          // pieces per thread and tile of each operand
  constexpr int ABYTES = BM * 128, BBYTES = BN * 128;
  constexpr int CPR = BN / V;                        // pieces per row of the NN weight tile
  constexpr bool B16 = sizeof(T) == 2;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l32 = lane & 31, lhi = lane >> 5;
  const BlockTile bt = block_tile<QUARTERS>(a, bid);
  const int part = bt.part, col0 = bt.tn * BN, N = a.N;
  if (QUARTERS && col0 >= N) return;                 // a quarter beyond the right edge

  RowPiece pc[NA];
  if constexpr (PACKED) {
#pragma unroll
    for (int f = 0; f < NA; ++f) pc[f] = packed_piece(a.M, (unsigned)bt.tm * BM + 32 * f);
  } else {
    const RowAxis axis = row_axis(a);
#pragma unroll
    for (int f = 0; f < NA; ++f) pc[f] = find_piece(a, axis, (unsigned)bt.tm * BM + 32 * f);
  }

  if (QUARTERS && pc[0].n == 0) return;              // ... or below the last row

  f32x16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // this part's share of the contraction tiles of all operand pairs
  int total_kt = 0;
#pragma unroll
  for (int g = 0; g < NSEG; ++g) total_kt += (a.Kd[g] + BK - 1) / BK;
  // (below 2^32: a contraction has up to 2^22 indices, so 16 parts of 4 operand pairs of 2^17 tiles make 2^23)
  int p0 = (int)((unsigned)total_kt * (unsigned)part / (unsigned)a.parts);
  int p1 = (int)((unsigned)total_kt * (unsigned)(part + 1) / (unsigned)a.parts);

  const int ar = tid >> 3, ac = tid & 7;             // K-contiguous: row (of 32) and piece of this thread
  const bool narrow = NN && N < V;                   // no whole piece in a row of W
  // fragment addresses
  const int fsw = (l32 >> 1) & 7;
  const int a_off = (wm * WM + l32) * 128, b_off = (wn * WN + l32) * 128;
  const int L16 = lane & 15, blk = lane >> 4, kq = L16 >> 2;
  const int tr_k = 8 * (blk >> 1) + kq, tr_n = 16 * (blk & 1) + 4 * (L16 & 3);

  for (int g = 0; g < NSEG; ++g) {
    const int Kd = a.Kd[g];
    const int KT = (Kd + BK - 1) / BK;
    const int t0 = p0 > 0 ? p0 : 0, t1 = p1 < KT ? p1 : KT;
    p0 -= KT;
    p1 -= KT;
    if (t0 >= t1) continue;
    const T* A = static_cast<const T*>(a.A[g]);
    const T* W = static_cast<const T*>(a.W[g]);
    // rows of this thread's pieces, as byte offsets from the block's first row (a block spans at most
    // BM rows of up to 16 MiB: below 2^32)
    const int row0 = pc[0].row;
    const char* abase = reinterpret_cast<const char*>(A + (size_t)row0 * Kd);
    unsigned aoff[NA], boff[NB];
#pragma unroll
    for (int it = 0; it < NA; ++it) {
      const int last = pc[it].n > 0 ? pc[it].n - 1 : 0;
      aoff[it] = (unsigned)(((size_t)(pc[it].row - row0 + (ar < last ? ar : last)) * Kd + ac * V) * sizeof(T));
    }
    const char* bbase;
    if constexpr (NN) {
      bbase = reinterpret_cast<const char*>(W);
#pragma unroll
      for (int it = 0; it < NB; ++it) {
        const int idx = tid + 256 * it;
        int n = col0 + (idx % CPR) * V;
        n = n <= N - V || narrow ? n : N - V;        // (see real_column)
        boff[it] = (unsigned)(((size_t)(idx / CPR) * N + n) * sizeof(T));
      }
    } else {
      bbase = reinterpret_cast<const char*>(W + (size_t)col0 * Kd);
#pragma unroll
      for (int it = 0; it < NB; ++it) {
        const int n = col0 + ar + 32 * it;
        boff[it] = (unsigned)(((size_t)((n < N ? n : N - 1) - col0) * Kd + ac * V) * sizeof(T));
      }
    }
    const size_t bstep = (NN ? (size_t)BK * N : (size_t)BK) * sizeof(T);
    // tiles before `whole` need no masks
    const int whole = narrow ? 0 : Kd / BK;
    typedef typename Piece16<T>::type Piece;
    u32x4 ra[NA], rb[NB];
    auto load = [&](int kt) {
      const int k0 = kt * BK;
      const char* at = abase + (size_t)k0 * sizeof(T);
      const char* bt = bbase + (size_t)kt * bstep;
      if (kt < whole) {
#pragma unroll
        for (int it = 0; it < NA; ++it) ra[it] = *reinterpret_cast<const Piece*>(at + aoff[it]);
#pragma unroll
        for (int it = 0; it < NB; ++it) rb[it] = *reinterpret_cast<const Piece*>(bt + boff[it]);
        return;
      }
#pragma unroll
      for (int it = 0; it < NA; ++it)
        ra[it] = load_piece<T>(reinterpret_cast<const T*>(abase + aoff[it]) - ac * V, k0 + ac * V, Kd);
#pragma unroll
      for (int it = 0; it < NB; ++it) {
        if constexpr (NN) {
          const int idx = tid + 256 * it;
          int k = k0 + idx / CPR;
          k = k < Kd ? k : Kd - 1;
          if (narrow) rb[it] = load_piece<T>(W + (size_t)k * N, col0 + (idx % CPR) * V, N);
          else rb[it] = *reinterpret_cast<const Piece*>(bbase + (ptrdiff_t)(k - idx / CPR) * N * (ptrdiff_t)sizeof(T) + boff[it]);
        } else {
          rb[it] = load_piece<T>(reinterpret_cast<const T*>(bbase + boff[it]) - ac * V, k0 + ac * V, Kd);
        }
      }
    };
    auto write = [&](char* st) {
      const int sw = (ac ^ ((ar >> 1) & 7)) << 4;
#pragma unroll
      for (int it = 0; it < NA; ++it) *reinterpret_cast<u32x4*>(st + (ar + 32 * it) * 128 + sw) = ra[it];
      char* sb = st + ABYTES;
#pragma unroll
      for (int it = 0; it < NB; ++it) {
        if constexpr (NN) {
          const int idx = tid + 256 * it;
          const int k = idx / CPR, c = idx % CPR;
          const int cs = !B16 ? c : (CPR == 16 ? c ^ ((k & 3) << 2) : c ^ (((k >> 1) & 1) << 2));
          *reinterpret_cast<u32x4*>(sb + (k * CPR + cs) * 16) = rb[it];
        } else {
          *reinterpret_cast<u32x4*>(sb + (ar + 32 * it) * 128 + sw) = rb[it];
        }
      }
    };
    auto put = [&](int kt, char* st) {
      if (kt >= whole) {
        const int k0 = kt * BK;
#pragma unroll
        for (int it = 0; it < NA; ++it) ra[it] = tail_shift<T>(ra[it], k0 + ac * V, Kd);
#pragma unroll
        for (int it = 0; it < NB; ++it) {
          if constexpr (NN) {
            const int idx = tid + 256 * it;
            if (k0 + idx / CPR >= Kd) rb[it] = u32x4{0, 0, 0, 0};
          } else {
            rb[it] = tail_shift<T>(rb[it], k0 + ac * V, Kd);
          }
        }
      }
      write(st);
    };
    // fragments of group ks (a quarter) of the tile in st
    auto read = [&](const char* st, int ks, u32x4 (&af)[FM], u32x4 (&bfr)[FN]) {
      const char* sb = st + ABYTES;
      const int coff = ((2 * ks + lhi) ^ fsw) << 4;
#pragma unroll
      for (int i = 0; i < FM; ++i) af[i] = *reinterpret_cast<const u32x4*>(st + a_off + i * 4096 + coff);
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        if constexpr (!NN) {
          bfr[j] = *reinterpret_cast<const u32x4*>(sb + b_off + j * 4096 + coff);
        } else if constexpr (B16) {
          const int n = wn * WN + 32 * j + tr_n, kk = 16 * ks + tr_k;
          const int c = CPR == 16 ? (n >> 3) ^ (kq << 2) : (n >> 3) ^ (((kk >> 1) & 1) << 2);
          const char* q = sb + (kk * CPR + c) * 16 + (n & 7) * 2;
          bfr[j] = __builtin_bit_cast(u32x4, lds_read_tr_pair(q, q + 4 * CPR * 16));
        } else {
          const float* q = reinterpret_cast<const float*>(sb) + (2 * ks + lhi) * 4 * BN + wn * WN + 32 * j + l32;
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = q[e * BN];
          bfr[j] = __builtin_bit_cast(u32x4, v);
        }
      }
    };
    auto multiply = [&](const u32x4 (&af)[FM], const u32x4 (&bfr)[FN]) { mma_tile<FM, FN>(acc, af, bfr, T{}); };
    __syncthreads();   // the previous operand pair's last tile has been read
    load(t0);
    put(t0, sm);
    if (t0 + 1 < t1) load(t0 + 1);
    __syncthreads();
    int kt = t0;
    // fp32, tiles whose successors need no masks: straight-line code, one memory instruction and two
    // others behind each MFMA (64 cycles).  bf16 MFMAs are too short for that: 4 % slower there.
    auto load_whole = [&](int kt) {
      const char* at = abase + (size_t)kt * (BK * sizeof(T));
      const char* bt = bbase + (size_t)kt * bstep;
#pragma unroll
      for (int it = 0; it < NA; ++it) ra[it] = *reinterpret_cast<const Piece*>(at + aoff[it]);
#pragma unroll
      for (int it = 0; it < NB; ++it) rb[it] = *reinterpret_cast<const Piece*>(bt + boff[it]);
    };
    const int steady = B16 && BM == 128 ? 0 : (whole < t1 ? whole : t1);
    u32x4 af[2][FM], bfr[2][FN];
    if constexpr (!B16) {
      if (kt + 2 < steady) read(sm, 0, af[0], bfr[0]);
      for (; kt + 2 < steady; ++kt) {
        const int s = (kt - t0) & 1;
        const char* st = sm + s * (ABYTES + BBYTES);
        char* const next = sm + (s ^ 1) * (ABYTES + BBYTES);
        read(st, 1, af[1], bfr[1]);
        multiply(af[0], bfr[0]);
        write(next);
        read(st, 2, af[0], bfr[0]);
        multiply(af[1], bfr[1]);
        load_whole(kt + 2);
        read(st, 3, af[1], bfr[1]);
        multiply(af[0], bfr[0]);
        interleave<12 * FM * FN>();
        // the tile's last fragments are in registers and the next tile is written: the barrier stands in
        // front of the last group, whose MFMAs cover the first fragment reads of the next tile
        __syncthreads();
        read(next, 0, af[0], bfr[0]);
        multiply(af[1], bfr[1]);
        interleave<4 * FM * FN>();
      }
    }
    __syncthreads();
    // bf16 in 64 x 64 tiles: the loop below without its masks and their branches (913 x 1500 x 1000, backward layout
    // 14.2 -> 13.6 us; 128 x 128 tiles 2-4 % slower with a loop more)
    if constexpr (B16 && BM == 64) {
      for (; kt + 2 < steady; ++kt) {
        const int s = (kt - t0) & 1;
        const char* st = sm + s * (ABYTES + BBYTES);
        read(st, 0, af[0], bfr[0]);
        read(st, 1, af[1], bfr[1]);
        multiply(af[0], bfr[0]);
        write(sm + (s ^ 1) * (ABYTES + BBYTES));
        read(st, 2, af[0], bfr[0]);
        multiply(af[1], bfr[1]);
        load_whole(kt + 2);
        read(st, 3, af[1], bfr[1]);
        multiply(af[0], bfr[0]);
        multiply(af[1], bfr[1]);
        __syncthreads();
      }
    }
    for (; kt < t1; ++kt) {
      const int s = (kt - t0) & 1;
      const char* st = sm + s * (ABYTES + BBYTES);
      read(st, 0, af[0], bfr[0]);
      read(st, 1, af[1], bfr[1]);
      multiply(af[0], bfr[0]);
      if (kt + 1 < t1) put(kt + 1, sm + (s ^ 1) * (ABYTES + BBYTES));
      read(st, 2, af[0], bfr[0]);
      multiply(af[1], bfr[1]);
      if (kt + 2 < t1) load(kt + 2);
      read(st, 3, af[1], bfr[1]);
      multiply(af[0], bfr[0]);
      multiply(af[1], bfr[1]);
      __syncthreads();
    }
  }

  // LoRA term: with the last part
  if (part == a.parts - 1) {
    for (int g = 0; g < NSEG; ++g) {
      const T* L = static_cast<const T*>(a.L[g]);
      const int ldz = a.ldz[g];
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        RowPiece p = pc[i];
        if (wm == 1) p = pc[NA / 2 + i];
        const int task = __builtin_amdgcn_readfirstlane(p.task);
        const T* lrow = L + (size_t)(p.row + (l32 < p.n ? l32 : p.n - 1)) * ldz;
        if constexpr (PACKED) {
          // task by task: the others' rows are computed from whatever L holds there and left out
          const TaskWalk walk = task_walk(a);
          const int row = __builtin_amdgcn_readfirstlane(p.row), end = row + __builtin_amdgcn_readfirstlane(p.n);
          for (int k = first_task(a, row); k < a.K && row < end; ++k) {
            const int b = task_begin(walk, k, a.off[kMaxK]);
            if (b >= end) break;
            const int lo = b - row, hi = task_begin(walk, k + 1, a.off[kMaxK]) - row;
            if (hi <= lo) continue;
            const int r = a.rank[g][k];
            const T* R = static_cast<const T*>(a.R[g].p[k]);
            f32x16 sum[FN];
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
              for (int e = 0; e < 16; ++e) sum[j][e] = 0.f;
#pragma unroll 2
            for (int q0 = 0; q0 < r; q0 += 2 * V) {
              const int q = q0 + lhi * V;
              const u32x4 lf = *reinterpret_cast<const typename Piece16<T>::type*>(lrow + q);
#pragma unroll
              for (int j = 0; j < FN; ++j) {
                int n = real_column<T, NN>(col0 + wn * WN + 32 * j + l32, N);
                n = n >= 0 ? n : N - 1;
                union {
                  u32x4 v;
                  T e[V];
                } rf;
#pragma unroll
                for (int e = 0; e < V; ++e)
                  rf.e[e] = q + e < r ? (NN ? R[(size_t)(q + e) * N + n] : R[(size_t)n * r + q + e]) : T(0.f);
                mma32(sum[j], lf, rf.v, T{});
              }
            }
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
              for (int e = 0; e < 16; ++e) {
                const int o = 8 * (e / 4) + 4 * lhi + e % 4;
                acc[i][j][e] += o >= lo && o < hi ? sum[j][e] : 0.f;
              }
          }
          continue;
        }
        if (task < 0) continue;
        const int r = a.rank[g][task];
        const T* R = static_cast<const T*>(a.R[g].p[task]);
        for (int q0 = 0; q0 < r; q0 += 2 * V) {
          const int q = q0 + lhi * V;                // q + V <= ldz: ldz is a multiple of 16
          const u32x4 lf = *reinterpret_cast<const typename Piece16<T>::type*>(lrow + q);
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            int n = real_column<T, NN>(col0 + wn * WN + 32 * j + l32, N);
            n = n >= 0 ? n : N - 1;
            union {
              u32x4 v;
              T e[V];
            } rf;
#pragma unroll
            for (int e = 0; e < V; ++e)
              rf.e[e] = q + e < r ? (NN ? R[(size_t)(q + e) * N + n] : R[(size_t)n * r + q + e]) : T(0.f);
            mma32(acc[i][j], lf, rf.v, T{});
          }
        }
      }
    }
  }

  if (a.parts > 1) {
    float* dst = a.part + ((size_t)part * a.units + bt.unit) * (BM * BN);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *reinterpret_cast<f32x4*>(dst + ((wave * FM + i) * FN + j) * 1024 + g * 256 + lane * 4) =
              f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
    return;
  }
  T* C = static_cast<T*>(a.C);
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    RowPiece p = pc[i];
    if (wm == 1) p = pc[NA / 2 + i];
#pragma unroll
    for (int j = 0; j < FN; ++j) store_frag<T>(acc[i][j], C, N, p, real_column<T, NN>(col0 + wn * WN + 32 * j + l32, N), lhi);
  }
}

template <typename T, int BM, int BN, bool NN, int NSEG, bool QUARTERS, bool PACKED>
__global__ __launch_bounds__(256) void k_gen_gemm(const GenGemmArgs<NSEG> a) {
  __shared__ __attribute__((aligned(1024))) char sm[kGemmLds<BM, BN>];
  gemm_body<T, BM, BN, NN, NSEG, QUARTERS, PACKED>(a, blockIdx.x, sm);
}

// Adds the parts of k_gen_gemm in order; block = fragment (i, j) of each of a tile's four waves.
struct GenReduceArgs {
  void* C;
  const float* part;
  int M, N, tiles_m, tiles_n, parts, units, t0;
  int packed;                            // as the product's PACKED
  int K;
  int off[kMaxK + 1];
};
template <typename T, int BM, int BN, bool NN, bool QUARTERS>
__global__ __launch_bounds__(256) void k_gen_reduce(const GenReduceArgs a) {
  constexpr int WM = BM / 2, WN = BN / 2, FM = WM / 32, FN = WN / 32;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int j = blockIdx.x % FN, i = blockIdx.x / FN % FM, tile = blockIdx.x / (FM * FN);
  const BlockTile bt = tile_of_unit<QUARTERS>(a, tile);
  if (QUARTERS && bt.tn * BN >= a.N) return;
  const unsigned v0 = (unsigned)bt.tm * BM + wm * WM + 32 * i;
  const RowPiece p = a.packed ? packed_piece(a.M, v0) : find_piece(a, row_axis(a), v0);
  if (p.n <= 0) return;
  const float* src = a.part + (size_t)tile * (BM * BN) + ((wave * FM + i) * FN + j) * 1024 + lane * 4;
  const size_t step = (size_t)a.units * (BM * BN);
  f32x16 acc;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll 2
  for (int s = 0; s < a.parts; ++s)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(src + s * step + g * 256);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[4 * g + e] += v[e];
    }
  store_frag<T>(acc, static_cast<T*>(a.C), a.N, p, real_column<T, NN>(bt.tn * BN + wn * WN + 32 * j + (lane & 31), a.N), lane >> 5);
}

// ------------------------------------------------------------------------------------------
// Out[i, 0:ldz] = s_k * In[i, :] * M_k for the rows i of task k; columns >= r_k are zero.
//   KMAJOR = true : M_k = A_k [inner, r_k]      KMAJOR = false: M_k = B_k^T, B_k [r_k, inner]
// Block: 16 RM rows of one task; its NW waves split the contraction (each takes every NW-th run of
// U x 64 bytes per row, no barrier in the loop) and add their sums through LDS in a fixed order.
// Lanes load MFMA operands straight from memory: a row's 64-byte run is shared by four lanes.  Each
// block runs the body for its own task's rank (VW groups of 16 columns), so that the deepest run a
// wave keeps in flight does not depend on the largest rank of the call.
// A_k's columns are contiguous where the MFMA wants contraction indices: lane i of 16 carries
// columns VW i .. VW i + VW - 1, one for each group, loads them as one piece per contraction index
// and regroups them in registers; a lane whose columns would cross the rank takes the last VW
// columns instead (the same sums a second time).
// ------------------------------------------------------------------------------------------
struct GenRowsArgs {
  const void* In;
  void* Out;
  int inner, ldz, K, b0;                 // b0: first block of this launch
  // parts > 1: the contraction is cut into ranges, one block each; range s writes its fp32 sums of row i at part +
  // (s * rows + i - off[0]) * ldz, rows = off[K] - off[0], and k_gen_rows_reduce adds them in order
  int parts;
  float* part;
  int off[kMaxK + 1];
  unsigned char rank[kMaxK];
  float s[kMaxK];
  PtrTable M;
};

// Adds a stretch of contraction to a wave's accumulators (16 RM rows x 16 VW columns): rows x[i] of
// `inner` elements times the columns col0 .. of the small operand,
//   KMAJOR = true : M [inner, stride], `ncols` columns in all      KMAJOR = false: M [ncols, stride]
// Each of the NW waves takes every NW-th run of U groups.
template <int VW>
__device__ __forceinline__ int first_column(int i16, int col0, int ncols) {   // k-major: first column of lane i16
  const int q = col0 + VW * i16;
  return q < ncols - VW ? q : ncols - VW;
}
template <typename T, int VW, int RM, int NW, bool KMAJOR>
__device__ __forceinline__ void accumulate_rows(f32x4 (&acc)[RM][VW], const T* const (&x)[RM], int inner, const T* M, size_t stride,
                                                int col0, int ncols, int wave, int lane) {
  constexpr int V = kV<T>, STEP = 4 * V;             // contraction indices per MFMA group (64 bytes)
  constexpr int U = VW <= 2 ? 4 : (VW == 4 ? 2 : 1);
  typedef T Cols __attribute__((ext_vector_type(VW), aligned(sizeof(T))));
  const int l16 = lane & 15, kg = lane >> 4;
  const int q0 = first_column<VW>(l16, col0, ncols);

  // operand pieces of contraction indices k0 + kg V ..; `tail`: some lie beyond `inner`
  struct Small {
    u32x4 v[VW];
  };
  auto small = [&](int k0, bool tail) {
    const int kk = k0 + kg * V;
    Small o;
    if constexpr (KMAJOR) {
      union {
        u32x4 v[VW];
        T e[VW][V];
      } u;
      const T* p = M + (size_t)kk * stride + q0;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        Cols c;
        if (!tail || kk + e < inner) {
          c = *reinterpret_cast<const Cols*>(p + (size_t)e * stride);
        } else {
#pragma unroll
          for (int f = 0; f < VW; ++f) c[f] = T(0.f);
        }
#pragma unroll
        for (int f = 0; f < VW; ++f) u.e[f][e] = c[f];
      }
#pragma unroll
      for (int f = 0; f < VW; ++f) o.v[f] = u.v[f];
    } else {
#pragma unroll
      for (int f = 0; f < VW; ++f) {
        const int q = col0 + 16 * f + l16;
        o.v[f] = load_piece<T>(M + (size_t)(q < ncols ? q : ncols - 1) * stride, kk, tail ? inner : kk + V);
        if (tail) o.v[f] = tail_shift<T>(o.v[f], kk, inner);
      }
    }
    return o;
  };
  auto big = [&](int k0, int i, bool tail) {
    const int kk = k0 + kg * V;
    u32x4 v = load_piece<T>(x[i], kk, tail ? inner : kk + V);
    if (tail) v = tail_shift<T>(v, kk, inner);
    return v;
  };

  const int full = inner / (U * STEP);               // runs that need no masks
  for (int run = wave; run < full; run += NW) {
    const int k0 = run * U * STEP;
    u32x4 xf[U][RM];
    Small sf[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < RM; ++i) xf[u][i] = big(k0 + u * STEP, i, false);
      sf[u] = small(k0 + u * STEP, false);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int j = 0; j < VW; ++j)
#pragma unroll
        for (int i = 0; i < RM; ++i) mma16(acc[i][j], xf[u][i], sf[u].v[j], T{});
  }
  // what is left of the contraction, in single groups
  for (int k0 = full * U * STEP + wave * STEP; k0 < inner; k0 += NW * STEP) {
    u32x4 xf[RM];
#pragma unroll
    for (int i = 0; i < RM; ++i) xf[i] = big(k0, i, true);
    const Small sv = small(k0, true);
#pragma unroll
    for (int j = 0; j < VW; ++j)
#pragma unroll
      for (int i = 0; i < RM; ++i) mma16(acc[i][j], xf[i], sv.v[j], T{});
  }
}

// The waves' sums through LDS: the upper half of the waves hands its sums to the lower half, which adds
// them and hands on its own; element t of the block's sum is then the NW / 2 slots red[w * FR + t] in
// wave order.  acc[i][j]: lane holds operand column l16 of group j and rows 16 i + 4 kg + e; t holds
// group (i, j) in its upper bits, then the row of 16 and the operand column.
template <int VW, int RM, int NW>
__device__ __forceinline__ void share_sums(const f32x4 (&acc)[RM][VW], float* red, int wave, int lane) {
  constexpr int H = NW / 2, FR = RM * VW * 256;
  const int l16 = lane & 15, kg = lane >> 4;
  auto slot = [&](int w, int i, int j, int e) -> float& { return red[w * FR + (i * VW + j) * 256 + (4 * kg + e) * 16 + l16]; };
  if (wave >= H) {
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int j = 0; j < VW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) slot(wave - H, i, j, e) = acc[i][j][e];
  }
  __syncthreads();
  if (wave < H) {
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int j = 0; j < VW; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) slot(wave, i, j, e) = acc[i][j][e] + slot(wave, i, j, e);
  }
  __syncthreads();
}
template <int FR, int H>
__device__ __forceinline__ float shared_sum(const float* red, int t) {
  float sum = red[t];
#pragma unroll
  for (int w = 1; w < H; ++w) sum += red[w * FR + t];
  return sum;
}

template <typename T, int VW, int RM, int NW, bool KMAJOR, bool RANGES>
__device__ __forceinline__ void rows_body(const GenRowsArgs& a, int k, int lo, int hi, int sp, float* red) {
  const int r = a.rank[k];
  // this block's range, in whole runs of 64 contraction indices
  int c0 = 0, inner = a.inner;
  if constexpr (RANGES) {
    const unsigned runs = (unsigned)(a.inner + 63) / 64;
    c0 = (int)(runs * (unsigned)sp / (unsigned)a.parts) * 64;
    const int c1 = (int)(runs * (unsigned)(sp + 1) / (unsigned)a.parts) * 64;
    inner = (c1 < a.inner ? c1 : a.inner) - c0;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const T* x[RM];
#pragma unroll
  for (int i = 0; i < RM; ++i) {
    const int row = lo + 16 * i + (lane & 15);
    x[i] = static_cast<const T*>(a.In) + (size_t)(row < hi ? row : hi - 1) * a.inner + c0;
  }
  f32x4 acc[RM][VW];
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < VW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  accumulate_rows<T, VW, RM, NW, KMAJOR>(acc, x, inner, static_cast<const T*>(a.M.p[k]) + (KMAJOR ? (size_t)c0 * r : (size_t)c0),
                                         KMAJOR ? r : a.inner, 0, r, wave, lane);
  share_sums<VW, RM, NW>(acc, red, wave, lane);
  constexpr int FR = RM * VW * 256;
  if constexpr (RANGES) {
    float* part = a.part + ((size_t)sp * (a.off[a.K] - a.off[0]) + lo - a.off[0]) * a.ldz;
    for (int t = tid; t < FR; t += NW * 64) {
      const float sum = shared_sum<FR, NW / 2>(red, t);
      const int ij = t >> 8, i = ij / VW, j = ij % VW, i16 = t & 15;
      const int o = 16 * i + ((t >> 4) & 15), q = KMAJOR ? first_column<VW>(i16, 0, r) + j : 16 * j + i16;
      if (lo + o < hi && q < r) part[(size_t)o * a.ldz + q] = sum;
    }
    return;
  }
  const float s = a.s[k];
  T* Out = static_cast<T*>(a.Out);
  for (int t = tid; t < FR; t += NW * 64) {
    const float sum = shared_sum<FR, NW / 2>(red, t);
    const int ij = t >> 8, i = ij / VW, j = ij % VW, i16 = t & 15;
    const int row = lo + 16 * i + ((t >> 4) & 15), q = KMAJOR ? first_column<VW>(i16, 0, r) + j : 16 * j + i16;
    if (row < hi && q < r) Out[(size_t)row * a.ldz + q] = from_f32<T>(sum * s);
  }
  const int pad = a.ldz - r;
  if (pad > 0)
    for (int t = tid; t < (hi - lo) * pad; t += NW * 64) Out[(size_t)(lo + t / pad) * a.ldz + r + t % pad] = T(0.f);
}

// RANGES: whether the contraction is cut (the code for it costs the others 0.2 to 0.3 us of a launch of 4.1)
template <typename T, int RM, int NW, bool KMAJOR, bool RANGES>
__global__ __launch_bounds__(NW * 64, 4) void k_gen_rows(const GenRowsArgs a) {
  extern __shared__ float red[];         // NW / 2 x RM x (groups of the largest rank) KiB
  int lo = 0, hi = 0;
  int block = blockIdx.x, sp = 0;
  if constexpr (RANGES) {
    sp = block % a.parts;
    block /= a.parts;
  }
  const int k = rows_block<16 * RM>(a, a.b0 + block, &lo, &hi);
  if (k < 0) return;
  const int r = a.rank[k];
  if (r <= 16) rows_body<T, 1, RM, NW, KMAJOR, RANGES>(a, k, lo, hi, sp, red);
  else if (r <= 32) rows_body<T, 2, RM, NW, KMAJOR, RANGES>(a, k, lo, hi, sp, red);
  else if (r <= 64) rows_body<T, 4, RM, NW, KMAJOR, RANGES>(a, k, lo, hi, sp, red);
  else if constexpr (RM == 1) rows_body<T, 8, RM, NW, KMAJOR, RANGES>(a, k, lo, hi, sp, red);   // (two row groups: ranks up to 64)
}

// Adds the contraction ranges of k_gen_rows in order, scales and rounds.  One thread per four columns of a row.
template <typename T>
__global__ __launch_bounds__(256) void k_gen_rows_reduce(const GenRowsArgs a) {
  const int rows = a.off[a.K] - a.off[0], per = a.ldz / 4;
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= (long long)rows * per) return;
  const int i = (int)(t / per), q = (int)(t % per) * 4;
  const int k = task_of_row(a, a.off[0] + i);
  const int r = a.rank[k];
  const float s = a.s[k];
  f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
  if (q < r) {
    const float* p = a.part + (size_t)i * a.ldz + q;
    const size_t step = (size_t)rows * a.ldz;
#pragma unroll 4
    for (int u = 0; u < a.parts; ++u) sum += *reinterpret_cast<const f32x4*>(p + u * step);
  }
  T* out = static_cast<T*>(a.Out) + (size_t)(a.off[0] + i) * a.ldz + q;
#pragma unroll
  for (int e = 0; e < 4; ++e) out[e] = from_f32<T>(q + e < r ? sum[e] * s : 0.f);
}

// ------------------------------------------------------------------------------------------
// The base product of k_gen_gemm for small problems: block = 16 rows x 64 columns, its 8 waves split the
// contraction as in k_gen_rows (LoRA term: a second stretch of it), operands straight from memory.
// ------------------------------------------------------------------------------------------
constexpr int kSkinnySums = 4 * 4 * 256;
template <typename T, bool NN, int NSEG>
__device__ __forceinline__ void skinny_body(const GenGemmArgs<NSEG>& a, int bid, float* red) {
  constexpr int NW = 8, VW = 4;
  const int tm = bid % a.tiles_m, tn = bid / a.tiles_m;
  const int N = a.N, col0 = tn * 16 * VW;
  RowPiece p = find_piece(a, row_axis(a), 16u * tm);
  if (p.n <= 0) return;
  p.n = p.n < 16 ? p.n : 16;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15;
  const size_t row = p.row + (l16 < p.n ? l16 : p.n - 1);
  const int task = __builtin_amdgcn_readfirstlane(p.task);
  f32x4 acc[1][VW];
#pragma unroll
  for (int j = 0; j < VW; ++j) acc[0][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int g = 0; g < NSEG; ++g) {
    const int Kd = a.Kd[g];
    if (Kd == 0) continue;
    const T* const x[1] = {static_cast<const T*>(a.A[g]) + row * Kd};
    accumulate_rows<T, VW, 1, NW, NN>(acc, x, Kd, static_cast<const T*>(a.W[g]), NN ? N : Kd, col0, N, wave, lane);
    if (task >= 0) {
      const int r = a.rank[g][task];
      const T* const l[1] = {static_cast<const T*>(a.L[g]) + row * a.ldz[g]};
      accumulate_rows<T, VW, 1, NW, NN>(acc, l, r, static_cast<const T*>(a.R[g].p[task]), NN ? N : r, col0, N, wave, lane);
    }
  }
  share_sums<VW, 1, NW>(acc, red, wave, lane);
  T* C = static_cast<T*>(a.C);
  for (int t = tid; t < VW * 256; t += NW * 64) {
    const float sum = shared_sum<VW * 256, NW / 2>(red, t);
    const int j = t >> 8, i16 = t & 15, o = (t >> 4) & 15;
    const int col = NN ? first_column<VW>(i16, col0, N) + j : col0 + 16 * j + i16;
    if (o < p.n && col < N) C[(size_t)(p.row + o) * N + col] = from_f32<T>(sum);
  }
}
template <typename T, bool NN, int NSEG>
__global__ __launch_bounds__(512, 4) void k_gen_skinny(const GenGemmArgs<NSEG> a) {
  __shared__ float red[kSkinnySums];
  skinny_body<T, NN, NSEG>(a, blockIdx.x, red);
}

// ------------------------------------------------------------------------------------------
// Gradients, contraction over a task's tokens:
//   WIDE_FIRST = true : out_k[c, q] (+)= sum_t Big[t, c] * Small[t, q]   (dA_k = x_k^T G)
//   WIDE_FIRST = false: out_k[q, c] (+)= sum_t Small[t, q] * Big[t, c]   (dB_k = Z^T dy_k)
// A wave owns 64 columns of Big as four MFMA fragments of 16: lane i of 16 carries columns
// 4 i .. 4 i + 3, one for each fragment, so that it loads (and, for dB, stores) them as one piece.
// splits > 1: a task's tokens are cut into ranges of whole MFMA groups, one block each, whose sums go
// to part + range * part_step ([sum of r_k][wide]) for grad_reduce to add in order.  fp32, T = 2048, 4 tasks, 4096
// columns, rank 16: dB and dA in one launch 18 us + 5 us of reduction for 67 MB, against 131 us each with
// a serial sum per output element.  Small calls are bound by latency: a run of groups is requested at once, the
// last one with masks and without the groups behind the last token (one launch, 64 tokens x 256 columns x 2 tasks 4.9 us
// instead of 10.4 with a wait per group, 125 x 1000 x 8 7.6 instead of 19.3; bf16 300 x (1000 + 1500) x 3 6.4 instead of
// 16.6, 1333 tokens 9.5 instead of 19.9).  Where a task has no more tokens than a group there is nothing to overlap:
// fp32, 64 tasks of one token, 16 + 16 columns, rank 128 9.9 us, a wait per group 9.2, all groups of the run 12.7;
// rank 64 6.6, 6.3, 8.0.
// ------------------------------------------------------------------------------------------
struct GenGradArgs {
  const void* Big;
  const void* Small;
  int wide, ldz, K, accumulate, chunks, splits;
  size_t part_step;
  float* part;
  int off[kMaxK + 1];
  unsigned char rank[kMaxK];
  OutTable out;
};

template <typename T, int NQ, bool WIDE_FIRST>
__device__ __forceinline__ void grad_body(const GenGradArgs& a, int c0, int sp, int k) {
  constexpr int GT = sizeof(T) == 2 ? 32 : 4;        // tokens per MFMA
  constexpr int TE = GT / 4;                         // ... of which a lane carries TE
  const int wide = a.wide;
  int lo = a.off[k], hi = a.off[k + 1];
  if (a.splits > 1) {
    const int len = ((hi - lo + a.splits - 1) / a.splits + 31) / 32 * 32;
    lo = lo + sp * len < hi ? lo + sp * len : hi;
    hi = lo + len < hi ? lo + len : hi;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int l16 = lane & 15, kg = lane >> 4;
  if (c0 >= wide) return;
  const int r = a.rank[k];
  // lane i's four columns start here: a piece that crosses the end is loaded so that it ends there and is not
  // shifted; its columns below c0 + 4 i belong to other lanes and are not stored
  auto first_col = [&](int i) {
    const int c = c0 + 4 * i;
    return wide < 4 || c < wide - 4 ? c : wide - 4;
  };
  const int cb = first_col(l16);
  const T* Big = static_cast<const T*>(a.Big);
  const T* Small = static_cast<const T*>(a.Small);

  f32x4 acc[4][NQ];
#pragma unroll
  for (int f = 0; f < 4; ++f)
#pragma unroll
    for (int j = 0; j < NQ; ++j) acc[f][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  typedef T Vec4 __attribute__((ext_vector_type(4), aligned(sizeof(T))));
  const T zero = T(0.f);
  // A group of GT tokens: what a lane carries of it.  Loading knows no branches, so that the loads of all of
  // a run's groups are in flight together (with one per piece at the right edge, each group waited for its own:
  // fp32, 64 tokens of 256 columns 10.4 us).
  struct Group {
    Vec4 b[TE];
    T s[NQ][TE];
  };
  auto load = [&](Group& g, int t0) {
#pragma unroll
    for (int e = 0; e < TE; ++e) {
      int t = t0 + kg * TE + e;
      t = t < hi ? t : hi - 1;
      g.b[e] = *reinterpret_cast<const Vec4*>(Big + (size_t)t * wide + cb);
      const T* srow = Small + (size_t)t * a.ldz;
#pragma unroll
      for (int j = 0; j < NQ; ++j) g.s[j][e] = srow[(16 * j < a.ldz ? 16 * j : 0) + l16];
    }
  };
  auto load_narrow = [&](Group& g, int t0) {         // rows of fewer than four columns
#pragma unroll
    for (int e = 0; e < TE; ++e) {
      int t = t0 + kg * TE + e;
      t = t < hi ? t : hi - 1;
#pragma unroll
      for (int f = 0; f < 4; ++f) g.b[e][f] = cb + f < wide ? Big[(size_t)t * wide + cb + f] : zero;
      const T* srow = Small + (size_t)t * a.ldz;
#pragma unroll
      for (int j = 0; j < NQ; ++j) g.s[j][e] = srow[(16 * j < a.ldz ? 16 * j : 0) + l16];
    }
  };
  auto multiply = [&](Group& g, int t0, bool tail) {
    if (tail) {
#pragma unroll
      for (int e = 0; e < TE; ++e) {
        if (t0 + kg * TE + e < hi) continue;
#pragma unroll
        for (int f = 0; f < 4; ++f) g.b[e][f] = zero;
#pragma unroll
        for (int j = 0; j < NQ; ++j) g.s[j][e] = zero;
      }
    }
#pragma unroll
    for (int j = 0; j < NQ; ++j)
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        if constexpr (sizeof(T) == 2) {
          bf16x8 b8, s8;
#pragma unroll
          for (int e = 0; e < TE; ++e) {
            b8[e] = g.b[e][f];
            s8[e] = g.s[j][e];
          }
          acc[f][j] = WIDE_FIRST ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(b8, s8, acc[f][j], 0, 0, 0)
                                 : __builtin_amdgcn_mfma_f32_16x16x32_bf16(s8, b8, acc[f][j], 0, 0, 0);
        } else {
          acc[f][j] = WIDE_FIRST ? __builtin_amdgcn_mfma_f32_16x16x4f32(g.b[0][f], g.s[j][0], acc[f][j], 0, 0, 0)
                                 : __builtin_amdgcn_mfma_f32_16x16x4f32(g.s[j][0], g.b[0][f], acc[f][j], 0, 0, 0);
        }
      }
  };
  constexpr int U = sizeof(T) == 4 ? (NQ <= 2 ? 8 : 4) : (NQ <= 2 ? 2 : 1);   // groups of a run
  auto run = [&](int t, bool tail) {
    Group g[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (!tail || u == 0 || t + u * GT < hi) load(g[u], t + u * GT);
    __builtin_amdgcn_sched_barrier(0);               // (the loads stay in front)
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (!tail || u == 0 || t + u * GT < hi) multiply(g[u], t + u * GT, tail);
  };
  int t = lo;
  if (wide >= 4) {
    for (; t + U * GT <= hi; t += U * GT) run(t, false);
    if (t < hi) run(t, true);
  } else {
    for (; t < hi; t += GT) {
      Group g;
      load_narrow(g, t);
      multiply(g, t, true);
    }
  }

  float* o = a.out.p[k];
  int accumulate = a.accumulate;
  if (a.splits > 1) {
    int rbase = 0;
    for (int kk = 0; kk < k; ++kk) rbase += a.rank[kk];
    o = a.part + sp * a.part_step + (size_t)rbase * wide;
    accumulate = 0;
  }
  // columns cb + f of a lane, f from `skip` on
  auto put = [&](float* dst, float v) { *dst = accumulate ? *dst + v : v; };
#pragma unroll
  for (int j = 0; j < NQ; ++j) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // WIDE_FIRST: lane holds q = 16 j + l16 and the columns carried by lane i = 4 kg + e
      const int i = WIDE_FIRST ? 4 * kg + e : l16;
      const int c = first_col(i), skip = c0 + 4 * i - c, q = WIDE_FIRST ? 16 * j + l16 : 16 * j + 4 * kg + e;
      if (q >= r) continue;
      const unsigned n = wide >= 4 ? 4 : (wide > c ? wide - c : 0);   // (from four columns on c + 3 < wide)
#pragma unroll
      for (int f = 0; f < 4; ++f)
        if ((unsigned)(f - skip) < n) put(WIDE_FIRST ? o + (size_t)(c + f) * r + q : o + (size_t)q * wide + c + f, acc[f][j][e]);
    }
  }
}

// the body for the task's own rank, of NQ groups of 16 columns at most; a chunk is the four columns of 64 of four waves
template <typename T, int NQ, bool WIDE_FIRST>
__device__ __forceinline__ void gen_grad_body(const GenGradArgs& a, int bid) {
  const int ch = bid % a.chunks, sp = bid / a.chunks % a.splits, k = bid / (a.chunks * a.splits);
  const int r = a.rank[k], c0 = (ch * 4 + (__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & 3)) * 64;
  if (NQ == 1 || r <= 16) grad_body<T, 1, WIDE_FIRST>(a, c0, sp, k);
  else if (NQ == 2 || r <= 32) grad_body<T, 2, WIDE_FIRST>(a, c0, sp, k);
  else if (NQ == 4 || r <= 64) grad_body<T, 4, WIDE_FIRST>(a, c0, sp, k);
  else grad_body<T, 8, WIDE_FIRST>(a, c0, sp, k);
}
// block `bid` of four waves: dB (the first blocks_b blocks) or dA
template <typename T, int NQ>
__device__ __forceinline__ void gen_grads_body(const GenGradArgs& b, const GenGradArgs& a, int blocks_b, int blocks, int bid) {
  if (bid < blocks_b) gen_grad_body<T, NQ, false>(b, bid);
  else if (bid < blocks) gen_grad_body<T, NQ, true>(a, bid - blocks_b);
}

// dB (the first blocks_b blocks) and dA of one call
template <typename T, int NQ>
__global__ __launch_bounds__(256) void k_gen_grad(const GenGradArgs b, const GenGradArgs a, int blocks_b) {
  gen_grads_body<T, NQ>(b, a, blocks_b, gridDim.x, blockIdx.x);
}

// ... of two projections that share their input
struct TwoGrads {
  GenGradArgs b[2], a[2];
  int blocks_b[2], blocks[2];
};
template <typename T, int NQ>
__global__ __launch_bounds__(256) void k_gen_grad_two(const TwoGrads p) {
  const int second = (int)blockIdx.x >= p.blocks[0] ? 1 : 0;
  gen_grads_body<T, NQ>(p.b[second], p.a[second], p.blocks_b[second], p.blocks[second], (int)blockIdx.x - (second ? p.blocks[0] : 0));
}

// Both gradients (the first blocks, which take longest) and the input gradient's product in one launch: neither reads what the other
// writes, each leaves most of the chip idle in a small call, and a launch costs 4 us.  Backward calls, two launches and the ranges'
// reduction -> one, us: bf16 913 x 1000 -> 1500 (3 tasks) 28.9 -> 22.9, 1024 -> 1536 21.9 -> 16.4, 1000 x 3000 -> 1000 33.0 -> 26.0,
// 400 x 64 -> 64 13.6 -> 11.1; fp32 128 x 256 -> 256 14.4 -> 11.2, 500 x 700 -> 1000 34.2 -> 27.1, 1000 x 300 -> 1500 44.1 -> 37.3.
struct BackArgs {
  GenGradArgs b, a;
  int blocks_b, blocks;
  int lead;              // blocks of the launch that hold gradients
};
// A block of gradients is four waves, the others of a larger block leave: gradients wait for loads and fp32 MFMAs, and two to a
// CU took up to twice as long while most CUs had nothing to do (fp32 512 x 500 -> 500, one task in 8 ranges, a step 33 us -> 28; 4
// tasks in one 48 -> 36).  Only where the blocks of the two-group ring, one to a CU, would be more than the CUs that way, a block holds
// two (908 x 768 -> 2624, 12 tasks, a step 48.2 -> 45.4).
template <typename T, int NQ>
__global__ __launch_bounds__(512, NQ == 4 ? 2 : 4) void k_gen_back_skinny(const GenGemmArgs<1> g, const BackArgs p) {
  __shared__ float red[kSkinnySums];
  const int bid = blockIdx.x;
  if (bid >= p.lead) skinny_body<T, false, 1>(g, bid - p.lead, red);
  else if (threadIdx.x < 256) gen_grads_body<T, NQ>(p.b, p.a, p.blocks_b, p.blocks, bid);
}
template <typename T, int NQ>
__global__ __launch_bounds__(256) void k_gen_back_64(const GenGemmArgs<1> g, const BackArgs p) {
  __shared__ __attribute__((aligned(1024))) char sm[kGemmLds<64, 64>];
  const int bid = blockIdx.x;
  if (bid >= p.lead) gemm_body<T, 64, 64, false, 1, false, false>(g, bid - p.lead, sm);
  else gen_grads_body<T, NQ>(p.b, p.a, p.blocks_b, p.blocks, bid);
}
template <int G, int NQ>
__global__ __launch_bounds__(256 * G, G == 1 ? 3 : 2) void k_gen_back_ring(const gemmk::GemmArgs<1> g, const BackArgs p) {
  __shared__ __attribute__((aligned(1024))) char sm[ringk::kRingLds<G>];
  const int bid = blockIdx.x;
  if (bid >= p.lead) return ringk::ring_body<G, false, 1>(g, bid - p.lead, sm);
  const int half = G == 1 ? 0 : (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const bool two = G == 2 && p.lead < p.blocks;      // neighbours: mostly of one task, which take as long
  if (two || half == 0) gen_grads_body<bf16, NQ>(p.b, p.a, p.blocks_b, p.blocks, two ? 2 * bid + half : bid);
}

int row_blocks(const SegTable& st, int tm) {
  int blocks = 0;
  for (int k = 0; k < st.K; ++k) blocks += (st.off[k + 1] - st.off[k] + tm - 1) / tm;
  return blocks;
}

// 32 rows per block halve the fetches of the small operand once that still leaves two blocks
// for every CU (ranks above 64 leave no registers for it)
bool two_row_groups(const CallCtx& c) { return c.ldz <= 64 && row_blocks(c.st, 32) >= 512; }

// Contraction ranges of one low-rank product: a block reads 16 rows and its task's whole operand, and a CU draws
// about 30 GB/s that way, so few blocks of long contractions take long while the other CUs idle.  From 320 KB a block on, as
// many ranges as give every CU a block, of at least 64 KB each.  One launch -> ranges and their reduction, us:
//   fp32  91 x 3840 (25 tasks), rank 64  45.7 -> 14.3;  687 x 2480, rank 58  33.0 -> 15.4, its s dy B^T, 1320 deep 14.4 -> 12.1
//         2048 x 4096, rank 16 (128 blocks)  14.7, 17.1 -> 14.7, 15.4
//   bf16  112 x 4960 (15 tasks), rank 87  30.1 -> 11.1;  212 x 10674, rank 64  24.5 -> 11.4
//         61 x 13770, rank 72, s dy B^T  64.8 -> 15.9;  106 x 3120 (4 tasks), rank 39  11.3 -> 9.0
int gen_rows_parts(const CallCtx& c, int inner, size_t limit) {
  if (c.K == 0 || two_row_groups(c)) return 1;
  const int blocks = row_blocks(c.st, 16);
  int rmax = 0;
  for (int k = 0; k < c.K; ++k) rmax = c.st.rank[k] > rmax ? c.st.rank[k] : rmax;
  const long long bytes = (long long)(16 + (rmax + 15) / 16 * 16) * inner * (c.dtype == MLORA_F32 ? 4 : 2);
  if (blocks == 0 || bytes < 320 << 10) return 1;
  const size_t one = (size_t)(c.st.off[c.K] - c.st.off[0]) * c.ldz * sizeof(float);
  int p = 256 / blocks;
  p = p < 16 ? p : 16;
  p = p < bytes >> 16 ? p : (int)(bytes >> 16);
  while (p > 1 && p * one > limit) --p;
  return p > 1 ? p : 1;
}

// algorithmic work of the launches below, as the timing of launches counts it (rows and gradients: bytes)
template <typename T>
double rows_work(const CallCtx& c, int inner) {
  double b = (double)(c.st.off[c.K] - c.st.off[0]) * ((double)inner + c.ldz);
  for (int k = 0; k < c.K; ++k) b += (double)c.st.rank[k] * inner;
  return b * sizeof(T);
}
double grads_work(const CallCtx& c, bool both) {
  const double wide = (double)c.d + (both ? c.h : 0), el = c.dtype == MLORA_F32 ? 4.0 : 2.0;
  double b = (double)(c.st.off[c.K] - c.st.off[0]) * (wide + (both ? 2.0 : 1.0) * c.ldz) * el;
  for (int k = 0; k < c.K; ++k) b += (double)c.st.rank[k] * wide * 4.0;
  return b;
}
double grads_flops(const CallCtx& c) {
  double f = 0;
  for (int k = 0; k < c.K; ++k) f += 2.0 * (c.st.off[k + 1] - c.st.off[k]) * (double)c.st.rank[k] * ((double)c.h + c.d);
  return f;
}

template <typename T, bool KMAJOR>
hipError_t rows_t(const CallCtx& c, const void* In, int inner, void* Out, const PtrTable& M, float* scratch) {
  if (c.K == 0 || c.T == 0 || row_blocks(c.st, 16) == 0) return hipSuccess;
  GenRowsArgs a;
  a.In = In;
  a.Out = Out;
  a.inner = inner;
  a.ldz = c.ldz;
  a.K = c.K;
  for (int k = 0; k <= kMaxK; ++k) a.off[k] = c.st.off[k];
  for (int k = 0; k < kMaxK; ++k) {
    a.rank[k] = (unsigned char)c.st.rank[k];
    a.s[k] = c.st.s[k];
  }
  a.M = M;
  a.parts = gen_rows_parts(c, inner, c.scratch_bytes);
  a.part = scratch;
  const bool two = two_row_groups(c);
  const int blocks = row_blocks(c.st, two ? 32 : 16);
  const int groups = c.ldz <= 16 ? 1 : (c.ldz <= 32 ? 2 : (c.ldz <= 64 ? 4 : 8));
  const unsigned lds = 4 * (two ? 2 : 1) * groups * 1024;
  constexpr int most = 1 << 22;          // a launch holds fewer than 2^32 threads
  const Profiled timed(kProfileRows, rows_work<T>(c, inner), c.stream);
  for (a.b0 = 0; a.b0 < blocks; a.b0 += most) {
    const dim3 grid((unsigned)(blocks - a.b0 < most ? blocks - a.b0 : most) * (unsigned)a.parts);
    if (two) hipLaunchKernelGGL((k_gen_rows<T, 2, 8, KMAJOR, false>), grid, dim3(512), lds, c.stream, a);
    else if (a.parts > 1) hipLaunchKernelGGL((k_gen_rows<T, 1, 8, KMAJOR, true>), grid, dim3(512), lds, c.stream, a);
    else hipLaunchKernelGGL((k_gen_rows<T, 1, 8, KMAJOR, false>), grid, dim3(512), lds, c.stream, a);
  }
  if (a.parts > 1) {
    const long long n = (long long)(c.st.off[c.K] - c.st.off[0]) * (c.ldz / 4);
    hipLaunchKernelGGL((k_gen_rows_reduce<T>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c.stream, a);
  }
  return hipGetLastError();
}

// Tile size and contraction parts of one base product.  Small problems (rows of up to 4 KB, up to 640 KB
// of them over all blocks of 16 rows) run k_gen_skinny: with 64 x 64 tiles the few blocks walk the
// contraction one tile after the other.  us, 64 x 64 tiles -> skinny: fp32 128 rows 256 x 256 10 -> 5,
// 1024 x 1024 20 -> 15, 500 rows 512 x 512 16 -> 9; beyond the line: 128 rows, 4096 deep 31 -> 60,
// 1000 rows 1024 x 1024 33 -> 43.  Beyond a round of blocks (1024; 1536 with ranks above 32, whose LoRA term
// the tiles add last: 700 x 2000 fp32, 4 deep, rank 128 21.5 us against 18.4) only outputs of one column
// block do: whole calls, tiles against skinny, 4000 x 2000 outputs 4 deep 11.4 against 22.8 us, 1500 x 2000, 32 deep 7.4
// against 10.3, 16000 x 100, 100 deep 12.4 against 16.6, but 40000 x 50, 50 deep, rank 64 55 against 41.
// 128 x 128 tiles once they give every CU a block; below that 64 x 64, the contraction cut into `parts`
// ranges where that is faster.  (From 193 to 255 tiles of 128 x 128 that line is too high for deep contractions: 64 x 64
// against 128 x 128, 2050 deep, fp32 216-316 against 212-301 us, bf16 64-90 against 58-76; 1100 deep fp32 level, bf16 up to 9 %; 500
// deep level to 3 % for 64 x 64.)  A launch costs a CU the tiles of its fullest share, so of the 128 x 128 tiles
// only whole rounds of 256 need be run as such: the others may run as quarters of 64 x 64, in ranges.  Both
// choices go by an estimate from measured times per contraction tile (constants below).  Forward, us:
//   fp32  2048 x 2048 -> 2176 (272 tiles)  248 in whole tiles, 151 as one round and quarters in 8 ranges
//         2048 x 4100 -> 4100 (528)        740 and 533 (4 ranges);   8000 x 1501 -> 701 (378)  188 and 161
//         2048 x 2048 -> 4096 (512: two rounds) 253; quarters alone take 283
//         1280 x 2048 -> 2048 (160: all 64 x 64) 110 in one range (two, 100 us, would be more than kMostUnits partial
//         tiles); 1024 x 2048 -> 2048 79 in one, 82 in two
//   bf16  2048 x 4100 -> 4100              128 and 104;   2048 x 2048 -> 2176  40 and 42
struct GemmPlan {
  bool skinny, small;
  int tiles_m, tiles_n, parts;           // of 16 x 64, 64 x 64 (small) or 128 x 128
  int whole;                             // 128 x 128: tiles [0, whole) as such, the others in quarters (small: 0)
  bool packed;                           // rows of several tasks in a piece
  double us;                             // the estimate
};
constexpr int kMaxParts = 16, kMostUnits = 1024, kTilesPerPart = 4;   // (contraction tiles of 128 bytes per row)
// us per contraction tile: a block alone on its CU, and the share of one among several; and per 16 ranks of the
// LoRA term of a 64 x 64 tile, forward and backward layout
struct StepTimes {
  double large_alone, large, small_alone, small, lora_nn, lora_nt;
};
constexpr StepTimes kSteps[2] = {{1.97, 1.97, 0.70, 0.58, 0.45, 0.9}, {0.80, 0.60, 0.36, 0.27, 0.3, 0.7}};   // fp32, bf16
// launches of n blocks of a form: 256 of them are a round
double rounds_us(long long n, double alone, double among) { return n <= 256 ? alone : (double)((n + 255) / 256) * among; }
// `units` 64 x 64 tiles of kt contraction tiles with `lora` us of LoRA term in the last range and `per_7mb` us of
// reduction for 7 MB of partial tiles: fewest us, the ranges for it, at least kTilesPerPart deep.  An XCD deals its
// blocks to its 32 CUs in turn, so with 2, 4, 8 or 16 ranges the tiles' last ranges, which hold the LoRA terms, share a
// half .. a sixteenth of the CUs: each further one on a CU adds 0.8 of the term.
double small_tiles_us(long long units, long long kt, const StepTimes& t, double lora, double per_7mb, size_t scratch_limit,
                      int* parts) {
  double best = 0;
  *parts = 0;
  for (int p = 1; p <= kMaxParts && (p == 1 || (kt / p >= kTilesPerPart && units * p <= kMostUnits)); ++p) {
    const size_t bytes = p > 1 ? (size_t)units * p * 64 * 64 * sizeof(float) : 0;
    if (bytes > scratch_limit) break;
    const long long on_one_cu = (units * (p & -p) + 255) / 256;   // (p & -p: the power of two in p)
    const double us = 6 + (double)((kt + p - 1) / p) * rounds_us(units * p, t.small_alone, t.small) +
                      lora * (1 + 0.8 * (double)(on_one_cu - 1)) + (p > 1 ? 4 + per_7mb * (double)bytes / 7e6 : 0);
    if (*parts == 0 || us < best) {
      best = us;
      *parts = p;
    }
  }
  return best;
}
// steps of 16 of the largest rank
int rank_steps(const int* rank, int K) {
  int rmax = 0;
  for (int k = 0; k < K; ++k) rmax = rank[k] > rmax ? rank[k] : rmax;
  return (rmax + 15) / 16;
}
long long contraction_tiles(long long Kd, int dtype) { return (Kd + (dtype == MLORA_F32 ? 31 : 63)) / (dtype == MLORA_F32 ? 32 : 64); }
}  // namespace
bool general_skinny(const SegTable& st, int M, int N, long long Kd, int dtype) {
  int rmax = 0;
  for (int k = 0; k < st.K; ++k) rmax = st.rank[k] > rmax ? st.rank[k] : rmax;
  const long long most_units = rmax > 32 ? 1536 : 1024;
  const long long units = (virtual_rows(st, M) + 15) / 16 * ((N + 63) / 64), row_bytes = Kd * (dtype == MLORA_F32 ? 4 : 2);
  return N >= 4 && row_bytes <= 4096 && units * row_bytes <= 640 << 10 && (units <= most_units || N <= 64);
}
namespace {
// (`steps16` steps of 16 ranks over all operand pairs)
GemmPlan plan_gemm(const SegTable& st, int M, int N, long long Kd_total, int steps16, bool nn, int dtype, size_t scratch_limit) {
  if (general_skinny(st, M, N, Kd_total, dtype))
    return GemmPlan{true, true, (int)((virtual_rows(st, M) + 15) / 16), (N + 63) / 64, 1, 0, false, general_skinny_us(st, M, N, Kd_total, dtype)};
  GemmPlan p;
  p.skinny = false;
  p.packed = false;
  const long long mv = virtual_rows(st, M);
  const long long t128 = ((mv + 127) / 128) * ((N + 127) / 128);
  p.small = t128 < 256;
  const int b = p.small ? 64 : 128;
  p.tiles_m = (int)((mv + b - 1) / b);
  p.tiles_n = (N + b - 1) / b;
  const long long tiles = (long long)p.tiles_m * p.tiles_n, kt = contraction_tiles(Kd_total, dtype);
  const StepTimes& t = kSteps[dtype == MLORA_F32 ? 0 : 1];
  p.parts = 1;
  p.whole = p.small ? 0 : (int)tiles;
  double us = 6 + (double)kt * rounds_us(tiles, t.large_alone, t.large);
  if (p.small) {
    // The LoRA term and 1.25 us: without the one and with 1, high ranks were cut into too many ranges.  Backward, product
    // and reduction, us with ranges of 4 contraction tiles and more whatever the rank, of 16 and more, and as chosen here:
    //   fp32  500 rows, 2000 deep, 700 columns, rank 128  48, 40, 34;   500 x 1000 x 1000, rank 128  37, 30, 30
    //   bf16  300 x 1500 x 1500, rank 128  30.6, 20.2, 20.4;   150 rows, 3000 deep, 300 columns, rank 2  12.6, 17.0, 12.9
    // (1292 products of 60 to 1500 rows: 1 % less in sum than with the first rule, none more than 6 % behind it).
    us = small_tiles_us(tiles, kt, t, steps16 * (nn ? t.lora_nn : t.lora_nt), 1.25, scratch_limit, &p.parts);
  } else if (tiles % 256 != 0) {
    const long long q = tiles / 256 * 256;
    int parts;
    // (The round of 128 x 128 tiles that the quarters replace has a LoRA term too; with it and 1.5 us the choice
    // takes 6-10 % longer: forward, fp32 2540 x 300 -> 2037, rank 128 46.8 and 59.9, bf16 3436 x 1500 -> 2549, rank 8
    // 55 and 61.)
    const double rest = small_tiles_us(4 * (tiles - q), kt, t, 0, 1, scratch_limit, &parts);
    if ((double)kt * rounds_us(q, t.large_alone, t.large) + rest < (double)kt * rounds_us(tiles, t.large_alone, t.large)) {
      p.whole = (int)q;
      p.parts = parts;
      us = 6 + (double)kt * rounds_us(q, t.large_alone, t.large) + rest;
    }
  }
  if (packed_rows(st, M) && ((M + 127LL) / 128) * ((N + 127) / 128) < 256) {
    // 64 x 64 tiles of packed rows: the LoRA terms of a piece's tasks one after the other.  Padded -> packed, us:
    // fp32 364 rows of 47 tasks, 2896 -> 384 49 -> 40, 2896 -> 3968 334 -> 122, the summed input gradient of both
    // 364 -> 167; but 41 rows of 33 tasks, 2816 -> 384 32 -> 51, which the estimate leaves padded.
    long long live = 0;
    for (int k = 0; k < st.K; ++k) live += st.off[k + 1] > st.off[k];
    const double in_piece = (double)live * 32 / M + 1;
    const int tm = (M + 63) / 64, tn = (N + 63) / 64;
    int parts;
    const double packed_us = small_tiles_us((long long)tm * tn, kt, t, steps16 * (nn ? t.lora_nn : t.lora_nt) * (in_piece < live ? in_piece : (double)live),
                                            1.25, scratch_limit, &parts);
    if (packed_us < 0.93 * us) return GemmPlan{false, true, tm, tn, parts, 0, true, packed_us};
  }
  p.us = us;
  return p;
}

template <typename T, bool NN, int NSEG>
hipError_t launch_gemm(GenGemmArgs<NSEG>& a, const GemmPlan& pl, float* scratch, hipStream_t s) {
  a.tiles_m = pl.tiles_m;
  a.tiles_n = pl.tiles_n;
  a.part = scratch;
  a.parts = 1;
  a.t0 = a.units = pl.whole;
  const int tiles = pl.tiles_m * pl.tiles_n;
  const Profiled timed(kProfileGemm, product_work(a), s);
  if (pl.skinny) {
    hipLaunchKernelGGL((k_gen_skinny<T, NN, NSEG>), dim3((unsigned)tiles), dim3(512), 0, s, a);
    return hipGetLastError();
  }
  if (pl.whole > 0) hipLaunchKernelGGL((k_gen_gemm<T, 128, 128, NN, NSEG, false, false>), dim3((unsigned)pl.whole), dim3(256), 0, s, a);
  if (pl.whole == tiles) return hipGetLastError();
  a.parts = pl.parts;
  a.units = pl.small ? tiles : 4 * (tiles - pl.whole);
  const dim3 grid((unsigned)(a.units * pl.parts));
  if (pl.packed) hipLaunchKernelGGL((k_gen_gemm<T, 64, 64, NN, NSEG, false, true>), grid, dim3(256), 0, s, a);
  else if (pl.small) hipLaunchKernelGGL((k_gen_gemm<T, 64, 64, NN, NSEG, false, false>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_gen_gemm<T, 64, 64, NN, NSEG, true, false>), grid, dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || pl.parts == 1) return e;
  GenReduceArgs r;
  r.C = a.C;
  r.part = scratch;
  r.M = a.M;
  r.N = a.N;
  r.tiles_m = a.tiles_m;
  r.tiles_n = a.tiles_n;
  r.parts = a.parts;
  r.units = a.units;
  r.t0 = a.t0;
  r.packed = pl.packed;
  r.K = a.K;
  for (int k = 0; k <= kMaxK; ++k) r.off[k] = a.off[k];
  if (pl.small) hipLaunchKernelGGL((k_gen_reduce<T, 64, 64, NN, false>), dim3((unsigned)a.units), dim3(256), 0, s, r);
  else hipLaunchKernelGGL((k_gen_reduce<T, 64, 64, NN, true>), dim3((unsigned)a.units), dim3(256), 0, s, r);
  return hipGetLastError();
}

// adds the ranges of a product in 64 x 64 tiles, backward layout
void launch_reduce64(const GenGemmArgs<1>& a, bool f32, hipStream_t s) {
  GenReduceArgs r;
  r.C = a.C;
  r.part = a.part;
  r.M = a.M;
  r.N = a.N;
  r.tiles_m = a.tiles_m;
  r.tiles_n = a.tiles_n;
  r.parts = a.parts;
  r.units = a.units;
  r.t0 = 0;
  r.packed = 0;
  r.K = a.K;
  for (int k = 0; k <= kMaxK; ++k) r.off[k] = a.off[k];
  if (f32) hipLaunchKernelGGL((k_gen_reduce<float, 64, 64, false, false>), dim3((unsigned)a.units), dim3(256), 0, s, r);
  else hipLaunchKernelGGL((k_gen_reduce<bf16, 64, 64, false, false>), dim3((unsigned)a.units), dim3(256), 0, s, r);
}

template <int NSEG>
hipError_t gemm_n(int n, const GenOperands* ops, int dtype, void* C, int M, int N, bool nn, const SegTable& st, float* scratch,
                  size_t scratch_bytes, hipStream_t s) {
  GenGemmArgs<NSEG> a;
  a.C = C;
  a.M = M;
  a.N = N;
  a.K = st.K;
  for (int k = 0; k <= kMaxK; ++k) a.off[k] = st.off[k];
  long long kd = 0;
  int steps16 = 0;
  for (int g = 0; g < NSEG; ++g) {
    const GenOperands& o = ops[g < n ? g : 0];
    a.A[g] = o.A;
    a.W[g] = o.W;
    a.L[g] = o.L;
    a.Kd[g] = g < n ? o.Kd : 0;
    a.ldz[g] = o.ldz;
    for (int k = 0; k < kMaxK; ++k) a.rank[g][k] = (unsigned char)(g < n && k < st.K ? o.rank[k] : 0);
    a.R[g] = *o.R;
    kd += a.Kd[g];
    if (g < n) steps16 += rank_steps(o.rank, st.K);
  }
  const GemmPlan pl = plan_gemm(st, M, N, kd, steps16, nn, dtype, scratch_bytes);
  const bool f32 = dtype == MLORA_F32;
  if (!nn) return f32 ? launch_gemm<float, false, NSEG>(a, pl, scratch, s) : launch_gemm<bf16, false, NSEG>(a, pl, scratch, s);
  if constexpr (NSEG == 1)
    return f32 ? launch_gemm<float, true, 1>(a, pl, scratch, s) : launch_gemm<bf16, true, 1>(a, pl, scratch, s);
  return hipErrorInvalidValue;   // only input gradients are summed over projections
}

// Token ranges per task of up to `longest` tokens: about four blocks per CU, at least `least` tokens each
int gen_grad_ranges(const SegTable& st, int wide_b, int wide_a, int longest, int least) {
  const int blocks = st.K * ((wide_b + 255) / 256 + (wide_a + 255) / 256);
  int s = (1024 + blocks - 1) / blocks;
  s = s < 16 ? s : 16;
  s = s < longest / least ? s : longest / least;
  return s > 1 ? s : 1;
}
constexpr int kLeastTokens = 64;
// ... as far as the scratch goes
int gen_grad_splits(const SegTable& st, int wide_b, int wide_a, size_t scratch_limit, int least = kLeastTokens) {
  int s = gen_grad_ranges(st, wide_b, wide_a, longest_task(st), least);
  while (s > 1 && grad_sum_bytes(st, s, wide_b, wide_a) > scratch_limit) --s;
  return s;
}

// the most plan_gemm cuts off for up to T rows
size_t gemm_part_bytes(int K, int T, int N, int Kd, int dtype) {
  const long long rows = most_virtual_rows(K, T), units = 4 * ((rows + 127) / 128) * ((N + 127) / 128);
  const long long deep = contraction_tiles(Kd, dtype) / kTilesPerPart, parts = deep < kMaxParts ? deep : kMaxParts;
  const long long blocks = units * parts < kMostUnits ? units * parts : kMostUnits;
  return parts > 1 ? (size_t)blocks * 64 * 64 * sizeof(float) : 0;
}

template <typename T>
void launch_grads(const GenGradArgs& b, const GenGradArgs& a, int blocks_b, int blocks, int ldz, hipStream_t s) {
  const dim3 grid((unsigned)blocks);
  if (ldz <= 16) hipLaunchKernelGGL((k_gen_grad<T, 1>), grid, dim3(256), 0, s, b, a, blocks_b);
  else if (ldz <= 32) hipLaunchKernelGGL((k_gen_grad<T, 2>), grid, dim3(256), 0, s, b, a, blocks_b);
  else if (ldz <= 64) hipLaunchKernelGGL((k_gen_grad<T, 4>), grid, dim3(256), 0, s, b, a, blocks_b);
  else hipLaunchKernelGGL((k_gen_grad<T, 8>), grid, dim3(256), 0, s, b, a, blocks_b);
}

}  // namespace

size_t general_grad_bytes(const SegTable& st, int T, int h, int d) {
  const int s = st.K > 0 ? gen_grad_ranges(st, d, h, T, kLeastTokens) : 1;
  return s > 1 ? grad_sum_bytes(st, s, d, h) : 0;
}
size_t general_dx_bytes(int K, int T, int h, int d, int dtype) { return gemm_part_bytes(K, T, h, d, dtype); }
size_t general_scratch_bytes(const SegTable& st, int T, int h, int d, int dtype) {
  size_t b = 0;
  auto most = [&](size_t v) { b = v > b ? v : b; };
  most(general_grad_bytes(st, T, h, d));
  most(gemm_part_bytes(st.K, T, d, h, dtype));
  most(gemm_part_bytes(st.K, T, h, d, dtype));
  return b;
}

GemmForm general_gemm_form(const SegTable& st, int M, int N, int n, const int* Kd, const int* const* rank, bool nn, int dtype,
                           size_t scratch_bytes) {
  long long kd = 0;
  int steps = 0;
  for (int g = 0; g < n; ++g) {
    kd += Kd[g];
    steps += rank_steps(rank[g], st.K);
  }
  const GemmPlan pl = plan_gemm(st, M, N, kd, steps, nn, dtype, scratch_bytes);
  const int form = pl.skinny ? MLORA_FORM_SKINNY : (pl.small ? MLORA_FORM_64 : MLORA_FORM_128), tiles = pl.tiles_m * pl.tiles_n;
  const bool quarters = form == MLORA_FORM_128 && pl.whole < tiles;
  return GemmForm{form, pl.parts, form == MLORA_FORM_128 ? pl.whole : tiles, tiles, pl.skinny ? 16 : (pl.small || quarters ? 64 : 128)};
}
// Estimate for s x A (us): blocks of 16 rows, the share of the fullest CU, at what a CU draws; `block_bytes`: what a block reads
double general_rows_us(const CallCtx& c, int inner, double* block_bytes) {
  const int parts = gen_rows_parts(c, inner, c.scratch_bytes);
  const double blocks = (double)row_blocks(c.st, 16) * parts;
  int rmax = 0;
  for (int k = 0; k < c.K; ++k) rmax = c.st.rank[k] > rmax ? c.st.rank[k] : rmax;
  const double bytes = (16.0 + (rmax + 15) / 16 * 16) * inner * (c.dtype == MLORA_F32 ? 4 : 2) / parts;
  *block_bytes = bytes;
  return 4.0 + (blocks <= 256 ? 1.0 : blocks / 256) * bytes / 30e3 + (parts > 1 ? 4.5 : 0.0);
}
RowsForm general_rows_form(const CallCtx& c, int inner) {
  return RowsForm{two_row_groups(c) ? 32 : 16, gen_rows_parts(c, inner, c.scratch_bytes)};
}
namespace {
// Token ranges of a small call's gradients (up to kMostShared activation elements, ranks up to 64), of at least `least` tokens, as an
// estimate in us has it: the longest range of any task, at so much per token (below: fp32 and bf16, ranks up to 16, 32 and 64);
// the blocks; the reduction, 3 and 14 per million elements and 0.3 per MB of sums (fp32 2.5 and 0.2 per MB).  Beside a product of `product` us what takes
// longer, and half of the ranges' time for the CUs that they take from it.  236 calls of 128 to 8000 tokens with dX beside them: the choice
// takes 0.6 % more than the best number of ranges in the mean, 8 % at most; always one 29 %, always as many as 64 tokens allow
// 3 %.  Forward, backward and gradients, one range -> several, us: fp32 256 x 256 -> 64 (one task) 19.5 -> 16.9, 1024 39 -> 19.5, but
// 128 x 1000 -> 1500 43.7 -> 45.3; bf16 1024 x 500 -> 500 29.2 -> 23.4, but 512 x 1000 -> 1500 33.7 -> 36.4, 1801 x 666 -> 87 (16 tasks, rank
// 64) 43.0 -> 53.5; by themselves 1716 x 2054 -> 115 (13 tasks, rank 32) 60.9 -> 70.1.
constexpr double kTokenUs[2][3] = {{0.026, 0.041, 0.07}, {0.0125, 0.0185, 0.033}};
int best_grad_ranges(const CallCtx& c, double product, int least) {
  const int most = gen_grad_splits(c.st, c.d, c.h, c.scratch_bytes, least);
  const bool f32 = c.dtype == MLORA_F32;
  size_t rtotal = 0;
  for (int k = 0; k < c.K; ++k) rtotal += c.st.rank[k];
  const double elements = (double)rtotal * (c.h + c.d), blocks = (double)c.K * ((c.h + 255) / 256 + (c.d + 255) / 256);
  int best = 1;
  double best_us = 0;
  for (int s = 1; s <= most; ++s) {
    double g = 0;
    for (int k = 0; k < c.K; ++k) {
      const int len = c.st.off[k + 1] - c.st.off[k], range = ((len + s - 1) / s + 31) / 32 * 32, r = c.st.rank[k];
      const double us = 3.0 + kTokenUs[f32 ? 0 : 1][r <= 16 ? 0 : (r <= 32 ? 1 : 2)] * (range < len ? range : len);
      g = us > g ? us : g;
    }
    const double us = (product > g ? product : g) + (product > 0 ? 0.5 * g : 0.0) + 0.5 * s * blocks / 64 +
                      (s == 1 ? 0.0 : (f32 ? 2.5 + 0.8e-6 * s * elements : 3.0 + (14e-6 + 1.2e-6 * s) * elements));
    if (s == 1 || us < best_us) {
      best_us = us;
      best = s;
    }
  }
  return best;
}
}  // namespace
int general_grad_ranges(const CallCtx& c) {
  if (c.K == 0) return 1;
  return c.ldz <= 64 && (long long)c.T * (c.h + c.d) <= kMostShared ? best_grad_ranges(c, 0.0, kLeastTokens)
                                                                    : gen_grad_splits(c.st, c.d, c.h, c.scratch_bytes);
}
// 16 x 64 tiles: the waves of a block share out rows of the contraction, a round of 256 blocks takes as long as its bytes
double general_skinny_us(const SegTable& st, int M, int N, long long Kd, int dtype) {
  const long long units = (virtual_rows(st, M) + 15) / 16 * ((N + 63) / 64);
  return 4.0 + 0.00235 * (double)(Kd * (dtype == MLORA_F32 ? 4 : 2)) * (double)((units + 255) / 256);
}

hipError_t general_Z(const CallCtx& c, const void* X, void* Z, float* scratch) {
  return c.dtype == MLORA_F32 ? rows_t<float, true>(c, X, c.h, Z, c.A, scratch) : rows_t<bf16, true>(c, X, c.h, Z, c.A, scratch);
}

hipError_t general_G(const CallCtx& c, const void* dY, void* G, float* scratch) {
  return c.dtype == MLORA_F32 ? rows_t<float, false>(c, dY, c.d, G, c.B, scratch) : rows_t<bf16, false>(c, dY, c.d, G, c.B, scratch);
}

hipError_t general_gemm(int n, const GenOperands* ops, int dtype, void* C, int M, int N, bool nn, const SegTable& st,
                        float* scratch, size_t scratch_bytes, hipStream_t stream) {
  if (M <= 0) return hipSuccess;
  if (n < 1 || n > MLORA_MAX_GROUP) return hipErrorInvalidValue;
  return n == 1 ? gemm_n<1>(n, ops, dtype, C, M, N, nn, st, scratch, scratch_bytes, stream)
                : gemm_n<MLORA_MAX_GROUP>(n, ops, dtype, C, M, N, nn, st, scratch, scratch_bytes, stream);
}

namespace {
// both gradients' arguments; returns the blocks of dB and of both
struct GradPlan {
  GenGradArgs b, a;
  int blocks_b, blocks, splits;
};
void plan_grads(const CallCtx& c, const void* dY, const void* Z, const OutTable& dB, const void* X, const void* G, const OutTable* dA,
                int accumulate, int ranges, float* scratch, GradPlan* p) {
  const int wide_b = c.d, wide_a = dA != nullptr ? c.h : 0;
  p->splits = ranges;
  size_t rtotal = 0;
  for (int k = 0; k < c.K; ++k) rtotal += c.st.rank[k];
  auto fill = [&](GenGradArgs& g, const void* big, int wide, const void* small, const OutTable& out, float* part) {
    g.Big = big;
    g.Small = small;
    g.wide = wide;
    g.ldz = c.ldz;
    g.K = c.K;
    g.accumulate = accumulate;
    g.chunks = (wide + 255) / 256;
    g.splits = p->splits;
    g.part_step = rtotal * ((size_t)wide_b + wide_a);
    g.part = part;
    for (int k = 0; k <= kMaxK; ++k) g.off[k] = c.st.off[k];
    for (int k = 0; k < kMaxK; ++k) g.rank[k] = (unsigned char)c.st.rank[k];
    g.out = out;
    return c.K * g.chunks * p->splits;
  };
  p->blocks_b = fill(p->b, dY, wide_b, Z, dB, scratch);
  p->blocks = p->blocks_b + (dA != nullptr ? fill(p->a, X, wide_a, G, *dA, scratch + rtotal * wide_b) : (p->a = p->b, 0));
}

template <typename T, int NQ>
void launch_back(const GenGemmArgs<1>& g, bool skinny, const BackArgs& p, hipStream_t s) {
  const dim3 grid((unsigned)(p.blocks + g.tiles_m * g.tiles_n * g.parts));
  if (skinny) hipLaunchKernelGGL((k_gen_back_skinny<T, NQ>), grid, dim3(512), 0, s, g, p);
  else hipLaunchKernelGGL((k_gen_back_64<T, NQ>), grid, dim3(256), 0, s, g, p);
}
template <int NQ>
void launch_back_ring(const gemmk::GemmArgs<1>& g, int groups, BackArgs p, hipStream_t s) {
  const int products = g.tiles_m * g.tiles_n * g.parts;
  if (groups == 2 && p.blocks + products > 256) p.lead = (p.blocks + 1) / 2;
  const dim3 grid((unsigned)(p.lead + products));
  if (groups == 2) hipLaunchKernelGGL((k_gen_back_ring<2, NQ>), grid, dim3(512), 0, s, g, p);
  else hipLaunchKernelGGL((k_gen_back_ring<1, NQ>), grid, dim3(256), 0, s, g, p);
}
}  // namespace

hipError_t general_grads(const CallCtx& c, const void* dY, const void* Z, const OutTable& dB, const void* X, const void* G,
                         const OutTable* dA, int accumulate, int ranges, float* scratch) {
  if (c.K == 0) return hipSuccess;
  GradPlan p;
  // (planned for both outputs, so that the scratch suffices for either)
  plan_grads(c, dY, Z, dB, X, G, dA, accumulate, ranges > 0 ? ranges : general_grad_ranges(c), scratch, &p);
  const Profiled timed(kProfileGrad, grads_work(c, dA != nullptr), c.stream);
  if (c.dtype == MLORA_F32) launch_grads<float>(p.b, p.a, p.blocks_b, p.blocks, c.ldz, c.stream);
  else launch_grads<bf16>(p.b, p.a, p.blocks_b, p.blocks, c.ldz, c.stream);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.splits == 1) return e;
  return grad_reduce(c.st, scratch, p.splits, c.d, dB, dA != nullptr ? c.h : 0, dA != nullptr ? *dA : dB, accumulate, c.stream);
}

namespace {
// whether dX runs in a form that gradients share a launch with, and the estimate for it
bool small_product(const CallCtx& c, bool aligned, size_t limit, double* us) {
  if (aligned) return gemm_small_us(c.st, c.T, c.h, c.d, limit, us);
  const GemmPlan pl = plan_gemm(c.st, c.T, c.h, c.d, rank_steps(c.st.rank, c.K), false, c.dtype, limit);
  *us = pl.us;
  return pl.small && !pl.packed;
}
}  // namespace

namespace {
template <typename T>
void launch_two(const TwoGrads& p, int ldz, hipStream_t s) {
  const dim3 grid((unsigned)(p.blocks[0] + p.blocks[1]));
  if (ldz <= 16) hipLaunchKernelGGL((k_gen_grad_two<T, 1>), grid, dim3(256), 0, s, p);
  else if (ldz <= 32) hipLaunchKernelGGL((k_gen_grad_two<T, 2>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((k_gen_grad_two<T, 4>), grid, dim3(256), 0, s, p);
}
}  // namespace

// The gradients of a group's projections, two to a launch where their sums fit the scratch together: a group's dX is a product of its
// own, and the ranges that suit a shared launch are long ones.  A launch each in ranges of 64 tokens -> as here, a step, us:
// bf16 500 x 701 -> 3 x 701 110 -> 109, 1000 x 500 -> 2 x 300 (4 tasks, rank 40) 60 -> 52; fp32 300 x 2001 -> 2001, 501 142 -> 138; a
// launch each in the long ranges 120, 64, 149.
hipError_t general_grads_group(int n, const GradItem* items, int accumulate, float* scratch, size_t scratch_bytes) {
  for (int i = 0; i < n; ++i) {
    const GradItem& x = items[i];
    const CallCtx& c = *x.c;
    auto sums = [](const GradItem& g) { return g.ranges > 1 ? grad_sum_bytes(g.c->st, g.ranges, g.c->d, g.c->h) : 0; };
    const size_t first = sums(x);
    hipError_t e;
    if (i + 1 == n || c.ldz > 64 || items[i + 1].c->ldz > 64 || first + sums(items[i + 1]) > scratch_bytes) {
      e = general_grads(c, x.dY, x.Z, *x.dB, x.X, x.G, x.dA, accumulate, x.ranges, scratch);
      if (e != hipSuccess) return e;
      continue;
    }
    const GradItem& y = items[++i];
    TwoGrads p;
    int ldz = 0;
    for (int q = 0; q < 2; ++q) {
      const GradItem& g = q ? y : x;
      GradPlan gp;
      plan_grads(*g.c, g.dY, g.Z, *g.dB, g.X, g.G, g.dA, accumulate, g.ranges, scratch + (q ? first / sizeof(float) : 0), &gp);
      p.b[q] = gp.b;
      p.a[q] = gp.a;
      p.blocks_b[q] = gp.blocks_b;
      p.blocks[q] = gp.blocks;
      ldz = g.c->ldz > ldz ? g.c->ldz : ldz;
    }
    const Profiled timed(kProfileGrad, grads_work(*x.c, x.dA != nullptr) + grads_work(*y.c, y.dA != nullptr), c.stream);
    if (c.dtype == MLORA_F32) launch_two<float>(p, ldz, c.stream);
    else launch_two<bf16>(p, ldz, c.stream);
    e = hipGetLastError();
    for (int q = 0; q < 2 && e == hipSuccess; ++q) {
      const GradItem& g = q ? y : x;
      if (g.ranges > 1)
        e = grad_reduce(g.c->st, scratch + (q ? first / sizeof(float) : 0), g.ranges, g.c->d, *g.dB, g.dA != nullptr ? g.c->h : 0,
                        g.dA != nullptr ? *g.dA : *g.dB, accumulate, c.stream);
    }
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Calls whose gradients and dX leave most CUs idle each: up to 4 Mi activation elements, ranks up to 64 (higher ones take all
// registers), and up to 32 where the aligned gradients could run, which are faster above (2000 x 256 -> 256, 16 tasks, rank 64
// 18 against 24 us); and dX in small tiles.
// The sizes and the problem's own addresses decide, so that a group's gradients, and those of a call whose dX overlaps what they
// read, have the bits of the shared launch.  (Without dX they run by themselves, in ranges of their own.)
BackPlan plan_back(const CallCtx& c, bool aligned) {
  const BackPlan apart{false, 0, c.scratch_bytes};
  const bool fast = c.dtype == MLORA_BF16 && c.h % 64 == 0 && c.d % 64 == 0;
  if (c.K == 0 || c.T == 0 || (long long)c.T * (c.h + c.d) > kMostShared || c.ldz > (fast ? 32 : 64)) return apart;
  double product;
  if (!small_product(c, aligned, c.scratch_bytes, &product)) return apart;
  const int ranges = best_grad_ranges(c, product, c.dtype == MLORA_F32 ? kLeastTokens : 2 * kLeastTokens);
  if (ranges == 1) return BackPlan{true, 1, c.scratch_bytes};
  const size_t left = c.scratch_bytes - grad_sum_bytes(c.st, ranges, c.d, c.h);
  return small_product(c, aligned, left, &product) ? BackPlan{true, ranges, left} : apart;
}

hipError_t general_back(const CallCtx& c, const BackPlan& bp, bool aligned, const void* X, const void* W, const void* dY, const void* Z, const void* G,
                        void* dX, const OutTable& dA, const OutTable& dB, int accumulate, float* scratch) {
  GradPlan gp;
  plan_grads(c, dY, Z, dB, X, G, &dA, accumulate, bp.ranges, scratch, &gp);
  const size_t left = bp.left;
  float* const partial = scratch + (c.scratch_bytes - left) / sizeof(float);   // behind the gradients' sums
  const BackArgs p{gp.b, gp.a, gp.blocks_b, gp.blocks, gp.blocks};
  const int nq = c.ldz <= 16 ? 1 : (c.ldz <= 32 ? 2 : 4);
  hipError_t e;
  gemmk::GemmArgs<1> r;
  int groups = 0, parts = 1;
  const SmallForm form = aligned ? gemm_small_nt((const bf16*)dY, (const bf16*)W, (bf16*)dX, c.T, c.h, c.d, (const bf16*)G, c.ldz,
                                                 c.st, c.A, left, &r, &groups, &parts)
                                 : kNotSmall;
  if (form == kRing) {
    ring_tiles(&r, c.st, parts, partial);
    const Profiled timed(kProfileGemm, product_work(r) + grads_flops(c), c.stream);
    if (nq == 1) launch_back_ring<1>(r, groups, p, c.stream);
    else if (nq == 2) launch_back_ring<2>(r, groups, p, c.stream);
    else launch_back_ring<4>(r, groups, p, c.stream);
    e = hipGetLastError();
    if (e == hipSuccess && parts > 1) {
      launch_ring_reduce(r, c.stream);
      e = hipGetLastError();
    }
  } else {
    const GemmPlan pl = plan_gemm(c.st, c.T, c.h, c.d, rank_steps(c.st.rank, c.K), false, c.dtype, left);
    if (aligned ? form != kSkinny || !pl.skinny : !pl.small || pl.packed) return hipErrorNotSupported;
    GenGemmArgs<1> g;
    g.C = dX;
    g.M = c.T;
    g.N = c.h;
    g.K = c.K;
    for (int k = 0; k <= kMaxK; ++k) g.off[k] = c.st.off[k];
    g.A[0] = dY;
    g.W[0] = W;
    g.L[0] = G;
    g.Kd[0] = c.d;
    g.ldz[0] = c.ldz;
    for (int k = 0; k < kMaxK; ++k) g.rank[0][k] = (unsigned char)c.st.rank[k];
    g.R[0] = c.A;
    g.tiles_m = pl.tiles_m;
    g.tiles_n = pl.tiles_n;
    g.units = pl.tiles_m * pl.tiles_n;
    g.parts = pl.parts;
    g.part = partial;
    g.t0 = 0;
    const bool f32 = c.dtype == MLORA_F32;
    const Profiled timed(kProfileGemm, product_work(g) + grads_flops(c), c.stream);
    if (nq == 1) f32 ? launch_back<float, 1>(g, pl.skinny, p, c.stream) : launch_back<bf16, 1>(g, pl.skinny, p, c.stream);
    else if (nq == 2) f32 ? launch_back<float, 2>(g, pl.skinny, p, c.stream) : launch_back<bf16, 2>(g, pl.skinny, p, c.stream);
    else f32 ? launch_back<float, 4>(g, pl.skinny, p, c.stream) : launch_back<bf16, 4>(g, pl.skinny, p, c.stream);
    e = hipGetLastError();
    if (e == hipSuccess && g.parts > 1) {
      launch_reduce64(g, f32, c.stream);
      e = hipGetLastError();
    }
  }
  if (e != hipSuccess || gp.splits == 1) return e;
  return grad_reduce(c.st, scratch, gp.splits, c.d, dB, c.h, dA, accumulate, c.stream);
}

}  // namespace mlora
