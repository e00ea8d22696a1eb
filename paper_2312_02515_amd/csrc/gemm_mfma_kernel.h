// bf16 MFMA GEMM kernel with the LoRA term folded in as extra contraction steps (gfx950),
// on v_mfma_f32_16x16x32_bf16.
//
//   C[M,N] = A[M,Kd] * op(Bm) + rows_k( L[rows_k, :r_k] * R_k )
//     NN = true  (forward,  Eq. "forward"):      Bm = W [Kd,N] (contraction index = rows of W),  R_k = B_k [r_k, N]
//     NN = false (backward, Eq. "grad_output"):  Bm = W [N,Kd] (contraction index = columns),     R_k = A_k [N, r_k]
//
// Why this MFMA shape: under this operator's data the board runs at its power cap, so what a
// kernel sustains is set by energy per flop.  A 16x16x32 MFMA sums 32 products into each
// accumulator element, a 32x32x16 MFMA 16: half the accumulator traffic per flop.  A loop of
// MFMAs plus the LDS fragment reads of this tile shape sustains about 10 % more with the
// 16x16x32 shape on the same data.
//
// Tile 256 x 256 x 64, WAVES_M x WAVES_N waves (2 x 4: wave tile WM x WN = 128 x 64), fp32
// accumulators in AccVGPRs, LDS tiles filled by direct global->LDS loads (16 B per lane) into
// three stages for A and two for Bm.  A wave-wide direct load fills 1 KiB of contiguous LDS, so the bank-conflict
// swizzle is applied by choosing which global 16-byte chunk each lane fetches:
//   * K-contiguous tiles (A, and Bm when !NN): 256 rows x 128 B; chunk c of row r sits at chunk
//     position c ^ ((r >> 1) & 7); a fragment (16 rows x 32 contraction indices) is one
//     ds_read_b128 per lane: lane l reads chunk 4 q + l / 16 of row l % 16 (q = which half of the tile).
//   * Bm when NN: 64 contraction rows x 512 B; chunk c of row k sits at
//     c ^ (((k & 3) << 2) | (((k >> 3) & 1) << 1)); read with two ds_read_b64_tr_b16 per lane,
//     which hand it eight consecutive contraction indices of one output column -- no transposed
//     copy of W is ever made.
// The weight fragment is the MFMA's first operand, so a lane ends up with four consecutive
// output columns of one row; the output tile goes through LDS once more so that it leaves the CU
// as full row segments.
//
// Schedule.  A contraction tile is four sub-steps: (first 32 contraction indices, upper half of
// the wave's rows), (same, lower half), (last 32, upper), (last 32, lower); a sub-step runs
// 4 x WN/16 MFMAs on 4 row fragments and WN/16 weight fragments.  Row fragments are read one
// sub-step ahead of their use (two register sets); a weight fragment serves both sub-steps of
// its half tile and is re-read in place right behind its last MFMA, a sub-step before its next
// use.  At most one memory instruction rides behind each MFMA:
//   sub-steps 0..2 of tile kt: MFMAs | LDS reads of the next sub-step's fragments | the direct loads
//               of A's tile kt+2 (three in sub-step 0, one in sub-step 1)
//   s_waitcnt vmcnt(4), lgkmcnt(0); barrier  (tile kt+1 visible -- the 4 loads still in flight are
//                                             A's of tile kt+2; every wave holds its last fragments
//                                             of tile kt in registers: kt's stages are free)
//   sub-step 3: MFMAs | LDS reads of tile kt+1's first fragments | the direct loads of Bm's tile kt+2
// Where the loads ride matters: a wave-wide load of 16 B per lane occupies the CU's address path for 16
// cycles (measured: 62 B per clock and CU), so the 64 loads of a tile need 1024 of the 2048 cycles that its
// MFMAs take.  All of them behind the barrier, in sub-step 3 (512 cycles of MFMAs), made every wave stand in
// that queue; spread over the tile, 16384 x 5120 x 5120 takes 562 / 551 us forward / backward instead of
// 579 / 574, 32768 rows 1131 / 1125 instead of 1180 / 1177, and half tiles 2048 x 11008 -> 4096 137 instead of 150.
// One shape loses, and on zeros only, where no power cap holds the loop: a contraction 13824 deep into 5120 columns, us
// per launch of 32768 rows, loads behind the barrier -> spread: zeros 2596 -> 2764 forward, 2600 -> 2810 backward; N(0,1) data 3214
// -> 3090 and 3170 -> 3100 (every other shape measured, 4096 to 16384 deep, gains 5-25 % on zeros and 1-13 % on data).  It
// is not A's lead: all four of A's loads in sub-step 0 leave it where it is, and so does one of them behind the
// barrier (2790-2820 both ways); two behind it bring zeros to 2670 and 2490 and cost most shapes 2-8 % on data.
// A keeps more than one tile of lead because its rows come from HBM, once per launch: with two stages
// and one tile of lead the blocks that share a row strip stalled together on every cold line (the time lost grew
// linearly with the rate at which A is read from HBM, at every shape measured).  Bm, the weight,
// is read from the Infinity Cache and keeps one tile of lead; 3 + 2 stages of 32 KiB are all of
// the CU's 160 KiB of LDS, which is why the block's piece table lives in a register.
//
// Rows: the grid tiles a virtual row axis on which every row range of the call (the rows before
// the first task, each task's rows, the rows after the last task) is padded to a multiple of 32.
// A 32-row fragment pair therefore never holds rows of two tasks, and a task's LoRA tile runs its
// MFMAs only on that task's rows: no row ever meets another task's adapter (not even multiplied
// by zero, which would turn an Inf or NaN of a diverged adapter into NaN in its neighbours'
// rows).  Padding rows re-read the range's last row and are not stored.
#pragma once

#include <type_traits>

#include "mfma_staging.h"
#include "mlora_common.h"
#include "row_axis.h"

namespace mlora {
namespace gemmk {

using namespace stage;
using namespace rowaxis;

constexpr int BN = 256;   // columns of a tile; its rows: 128 x WAVES_M
typedef __attribute__((ext_vector_type(4))) float f32x4;

// Kernel arguments (passed by value, read with scalar loads).  The contraction may run over
// NSEG operand pairs in turn, all accumulating into the same output tile:
//   C = sum_g ( A_g[M,Kd_g] * op(Bm_g) + rows_k( L_g[rows_k, :r_gk] * R_gk ) )
// NSEG = 1 is the plain operator; NSEG > 1 is the input gradient of several projections that
// share their input (dX = sum_p dY_p W_p^T + ...), kept in fp32 until the single store.
template <int NSEG>
struct GemmArgs {
  bf16* C;
  int M, N, tiles_m, tiles_n;            // tiles_m counts 256-row tiles of the virtual row axis
  int t0, parts;                         // HALF: first tile of the launch, contraction ranges per tile
  float* part;                           // HALF: partial tiles in fp32 when parts > 1
  int K;                                 // tasks
  int off[kMaxK + 1];                    // split positions (rows of C)
  const bf16* A[NSEG];                   // [M, Kd_g]
  const bf16* Bm[NSEG];                  // NN: [Kd_g, N]; NT: [N, Kd_g]
  const bf16* L[NSEG];                   // [M, ldz_g] low-rank intermediate (Z or G)
  int Kd[NSEG];
  int ldz[NSEG];
  unsigned char rank[NSEG][kMaxK];       // r_gk <= 128
  PtrTable R[NSEG];                      // NN: B_k [r, N]; NT: A_k [N, r]
};

// 16 zero bytes in device memory: where the lanes of a LoRA tile point whose row, column or rank
// index lies outside the task (a direct-to-LDS load cannot be masked)
static __device__ uint4 g_zero_chunk;


// r_gk: a dword read (a byte at a run-time index would be a vector load)
template <int NSEG>
__device__ __forceinline__ int rank_of(const GemmArgs<NSEG>& a, int sg, int k) {
  static_assert(offsetof(GemmArgs<NSEG>, rank) % 4 == 0, "read as dwords");
  return (int)(reinterpret_cast<const unsigned*>(a.rank[sg])[k >> 2] >> (8 * (k & 3))) & 255;
}

// The LoRA term's contraction tiles.  A slot is 32 ranks of one (operand pair, task of the block); a LoRA tile holds two
// slots, one in each half of its 64 contraction indices, and a piece of rows takes part in the halves of its own task
// only.  Lane t of the table keeps tile t's two slots (the most is 4 pairs x 8 pieces x 4 slots = 64 tiles): 16 bits
// each, task in 7 (127: none), pair in 2, first rank / 32 in 2.
struct LoraTiles {
  unsigned tab;
  int n;
};
struct LoraSlot {
  int sg, k, q0;
};
constexpr unsigned kNoSlot = 127;
__device__ __forceinline__ LoraSlot lora_slot(const LoraTiles& t, int tile, int half) {
  const unsigned v = (unsigned)__builtin_amdgcn_readlane((int)t.tab, __builtin_amdgcn_readfirstlane(tile)) >> (16 * half);
  return LoraSlot{(int)(v >> 7 & 3), (int)(v & 127), (int)(v >> 9 & 3) * 32};
}
// `task(f)`: task of the block's piece f (-1: none); the pieces of a task are consecutive
template <int NFR, int NSEG, typename F>
__device__ __forceinline__ LoraTiles lora_tiles(const GemmArgs<NSEG>& a, F task) {
  const int lane = threadIdx.x & 63;
  LoraTiles t{kNoSlot | kNoSlot << 16, 0};
  int e = 0;
  for (int sg = 0; sg < NSEG; ++sg)
    for (int f = 0; f < NFR; ++f) {
      const int k = task(f);
      if (k < 0 || (f > 0 && task(f - 1) == k)) continue;
      const int r = rank_of(a, sg, k);
      for (int q = 0; 32 * q < r; ++q, ++e) {
        const unsigned v = (unsigned)k | (unsigned)sg << 7 | (unsigned)q << 9;
        if (lane == e >> 1) t.tab = e & 1 ? (t.tab & 0xffffu) | v << 16 : (t.tab & 0xffff0000u) | v;
      }
    }
  t.n = (e + 1) / 2;
  return t;
}

// c += a x b on a 16 x 16 x 32 bf16 MFMA, accumulating in place in AccVGPRs.  Written as inline
// assembly with the accumulator as a tied operand: with the builtin the register allocator is
// free to give the result another register than the input, and in a loop of 128 MFMAs on 32
// accumulators it then rotates the accumulators through the register file with one copy per
// MFMA.  Every accumulator is used again at the earliest 16 MFMAs later and read by other
// instructions only after the main loop's final barrier, so no wait states are owed here.
__device__ __forceinline__ void mfma_16x16x32(f32x4& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// WAVES_M = 1 (HALF): 128 x 256 tiles of 4 waves for grids that leave the chip idle: the halves of the
// tiles that do not fill a round of 256 blocks, their contraction cut into ranges where even those
// are too few (fp32 partial tiles, added in order by k_gemm_reduce).  Such blocks are short, and what
// they spend outside the contraction loop counts: the loop is not unrolled (47 KB of code, fetched
// once, cost 10 us of a block's time) and the LoRA term is added from registers instead of by LoRA
// tiles in the pipeline (T = 100, 4096 x 4096, 8 ranges: 33 us -> 22 us).
// RAG (backward layout, whole tiles; the registers of a half tile take any rank): some rank is no
// multiple of 8, so A_k's rows [N, r] are no whole 16-byte chunks; such a task's LoRA tile is put
// together in registers, element by element (at most two of a block's contraction tiles per task).
// B_k [r, N] has whole chunks for any rank.  12 tasks of 256 tokens, 4096 x 4096, ranks 1 to 128: 99 us,
// as long as the forward product, against 244 us in the general kernel.
// RAG of half tiles stands for PACKED: many tasks of few rows, whose pieces of 32 rows would hold few rows each.  Pieces
// then hold rows of several tasks, and the LoRA term is added task by task, to the task's own rows only (a select, no
// product with zeros).  855 rows of 42 tasks, 10880 -> 1728, rank 64 83 -> 70 us.
// TAIL: whether a contraction may end in a partial tile (the code for it costs the others 1-2 us of 34 in half tiles, up to
// 1 % in whole ones).
template <int WAVES_M, int WAVES_N, bool NN, int NSEG, bool RAG, bool TAIL = true>
__global__ __launch_bounds__(WAVES_M* WAVES_N * 64) void k_gemm_mfma(const GemmArgs<NSEG> ga) {
  constexpr int BK = 64;
  constexpr int BM = 128 * WAVES_M;
  constexpr bool HALF = WAVES_M == 1;
  bf16* __restrict__ C = ga.C;
  const int M = ga.M, N = ga.N, tiles_m = ga.tiles_m, tiles_n = ga.tiles_n;
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr int FM = WM / 16, FN = WN / 16;    // 16-row fragments, 16-column weight fragments of the wave tile
  constexpr int HM = FM / 2;                   // row fragments per sub-step
  constexpr int NMF = HM * FN;                 // MFMAs per sub-step
  constexpr int ROWB = BK * 2, CPR = BK / 8, RW = 256 / ROWB, RPI = 1024 / ROWB;
  constexpr int ABYTES = BM * ROWB, BBYTES = BN * ROWB;   // the NN weight tile (BK x 512 B) has BBYTES too
  constexpr int LPA = ABYTES / 1024 / NW;      // wave-wide loads per wave and tile: A side,
  constexpr int LPB = BBYTES / 1024 / NW;      // Bm side
  constexpr int PER_TILE = LPA + LPB;
  static_assert(WM == 128, "the sub-steps halve a 128-row wave tile");
  constexpr bool PACKED = HALF && RAG;
  static_assert(!RAG || HALF || !NN, "B_k takes any rank");

  // Three stages for the A side, two for the Bm side: all 160 KiB of the CU's LDS.  The rows of
  // A come from HBM (every element once per launch, cold), the weight from the Infinity Cache; a
  // cold line takes longer than the one contraction tile a two-stage ring gives it, and every
  // block that shares the strip waits for it together.  With the third stage the A loads run two
  // tiles ahead of their use, the Bm loads one.
  __shared__ __attribute__((aligned(1024))) char sA0[ABYTES];
  __shared__ __attribute__((aligned(1024))) char sA1[ABYTES];
  __shared__ __attribute__((aligned(1024))) char sA2[ABYTES];
  __shared__ __attribute__((aligned(1024))) char sB0[BBYTES];
  __shared__ __attribute__((aligned(1024))) char sB1[BBYTES];
  // A half tile takes half as long, so its weight loads need two tiles of lead as well; 3 + 3 stages of
  // 16 and 32 KiB fit.
  __shared__ __attribute__((aligned(1024))) char sB2[HALF ? BBYTES : 16];
  char* const sA[3] = {sA0, sA1, sA2};
  char* const sB[3] = {sB0, sB1, sB2};

  // block -> tile.  Tiles are taken in a grouped order (8 row tiles x all column tiles per group,
  // column by column), cut into chunks of 32: a chunk is an 8 x 4 patch of output tiles sharing
  // 8 row strips of A and 4 strips of Bm.  Consecutive block ids go round-robin over the 8 XCDs
  // and an XCD runs 32 blocks at a time, so block b = 8 l + x (XCD x) takes tile l % 32 of chunk
  // 8 (l / 32) + x: the blocks resident on one XCD share their strips in that XCD's L2 (hit rate
  // 79 %, the share an 8 x 4 patch allows), and the eight XCDs work on eight neighbouring chunks,
  // i.e. on one or two row groups of A at a time.  (Giving each XCD a contiguous eighth of the
  // order instead, eight row groups at a time: level on benchmark-like data, 2-10 % slower when
  // the weight is 141 MB, because every XCD then walks all of it on its own.)  Other patch shapes: 4 x 8
  // misses more where the column tiles are no multiple of 8, 16 x 2 is 9 % slower.
  // The tiles beyond the last full round of 256 are taken in block order.
  const int total = tiles_m * tiles_n;
  const int bid = blockIdx.x;
  int t = bid, part = 0, half = 0;
  if constexpr (HALF) {
    // the upper and the lower half of the tiles from t0 on, range by range of the contraction; an
    // XCD takes a contiguous eighth of that order
    const int units = 2 * (total - ga.t0), per = units * ga.parts / 8;
    const int u = bid < 8 * per ? (bid % 8) * per + bid / 8 : bid;
    part = u / units;
    t = ga.t0 + (u % units) / 2;
    half = u % 2;
  } else if (bid < (total / 256) * 256) {
    const int xcd = bid % 8, local = bid / 8;
    t = 256 * (local / 32) + 32 * xcd + (local % 32);
  }
  constexpr int GM = 8;
  const int gsize = GM * tiles_n;
  const int group = t / gsize;
  const int first_m = group * GM;
  const int gm = (tiles_m - first_m) < GM ? (tiles_m - first_m) : GM;
  const int in_g = t - group * gsize;
  const int tm256 = first_m + in_g % gm, tn = in_g / gm;
  const int tm = HALF ? 2 * tm256 + half : tm256;
  const int col0 = tn * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  // ---- the block's 8 pieces of 32 virtual rows: first real row, number of real rows (0 = beyond
  // the last row: such a piece re-reads row M-1 and stores nothing) and task (-1 = rows of no
  // task).  Range s of the call is [b_s, b_{s+1}) with b_0 = 0, b_{1+k} = off[k], b_{K+2} = M;
  // task k owns range 1 + k.
  // The table lives in one vector register (the stages leave no LDS for it): every wave works it
  // out for itself, lane 8 c + f holding column c (0: first row, 1: rows, 2: task) of piece f.
  // Every use looks up a wave-uniform piece, so an entry is read with v_readlane.
  constexpr int NFR = BM / 32;
  int v_tab = 0;
  if constexpr (PACKED) {
    const RowPiece p = packed_piece(M, (unsigned)(tm * BM + 32 * (lane & (NFR - 1))));
    const int col = lane / NFR;
    v_tab = col == 0 ? p.row : (col == 1 ? p.n : p.task);
  } else if (__builtin_expect(ga.K <= kFewTasks, 1)) {
    const int v0 = tm * BM + 32 * (lane & (NFR - 1));
    int vstart = 0, prev = 0, frow = M - 1, fn = 0, ftask = -1;
    for (int r = 0; r < ga.K + 2; ++r) {
      const int b1 = r <= ga.K ? ga.off[r] : M;
      const int len = b1 - prev, vlen = (len + 31) & ~31;
      if (v0 >= vstart && v0 < vstart + vlen) {
        const int o = v0 - vstart;
        frow = prev + o;
        fn = (len - o) < 32 ? (len - o) : 32;
        ftask = (r >= 1 && r <= ga.K) ? r - 1 : -1;
      }
      vstart += vlen;
      prev = b1;
    }
    const int col = lane / NFR;
    v_tab = col == 0 ? frow : (col == 1 ? fn : ftask);
  } else {
    const RowAxis axis = row_axis(ga);
    const int col = lane / NFR;
    for (int f = 0; f < NFR; ++f) {
      const RowPiece p = find_piece(ga, axis, (unsigned)(tm * BM + 32 * f));
      if ((lane & (NFR - 1)) == f) v_tab = col == 0 ? p.row : (col == 1 ? p.n : p.task);
    }
  }
  auto tab = [&](int c, int f) { return __builtin_amdgcn_readlane(v_tab, __builtin_amdgcn_readfirstlane(NFR * c + f)); };
  auto frag_row = [&](int f) { return tab(0, f); };
  auto frag_n = [&](int f) { return tab(1, f); };
  auto frag_task = [&](int f) { return tab(2, f); };
  const int row0 = frag_row(0);  // the block's lowest real row
  if constexpr (HALF) {
    if (frag_n(0) == 0) return;  // the last row tile's lower half may be empty
  }
  // real row behind row rl (0..255) of the block's tile; the 8 rows of one wave-wide load lie in
  // one piece, so f is wave-uniform there
  auto real_row = [&](int rl) {
    const int f = rl >> 5, o = rl & 31;
    const int n = frag_n(f);
    return frag_row(f) + (o < n ? o : (n > 0 ? n - 1 : 0));
  };

  // ---- direct-to-LDS loads: wave-uniform base of the tile's rows (advanced per contraction
  // tile with scalar arithmetic) plus a constant 32-bit per-lane byte offset; both are set per
  // operand pair by set_operands()
  const char* abase = nullptr;
  const char* bbase = nullptr;
  unsigned aoff[LPA], boff[LPB];
  size_t bstep = 0;  // bytes per contraction tile of Bm
  auto nn_swz = [](int kr) { return ((kr & 3) << 2) | (((kr >> 3) & 1) << 1); };
  auto set_operands = [&](const bf16* A, const bf16* Bm, int Kd) {
    abase = reinterpret_cast<const char*>(A + (size_t)row0 * Kd);
    bbase = NN ? reinterpret_cast<const char*>(Bm + col0) : reinterpret_cast<const char*>(Bm + (size_t)col0 * Kd);
#pragma unroll
    for (int it = 0; it < LPA; ++it) {
      const int rl = RPI * (wave + NW * it) + lane / CPR;
      const int c = (lane % CPR) ^ ((rl / RW) % CPR);
      const int gr = real_row(rl);
      aoff[it] = (unsigned)(((size_t)(gr - row0) * Kd + c * 8) * 2);
    }
#pragma unroll
    for (int it = 0; it < LPB; ++it) {
      const int w = wave + NW * it;
      if (NN) {
        const int kr = 2 * w + (lane >> 5);
        const int c = (lane & 31) ^ nn_swz(kr);
        int n = col0 + c * 8;
        n = n < N ? n : N - 8;
        boff[it] = (unsigned)(((size_t)kr * N + (n - col0)) * 2);
      } else {
        const int rl = RPI * w + lane / CPR;
        const int c = (lane % CPR) ^ ((rl / RW) % CPR);
        int gn = col0 + rl;
        gn = gn < N ? gn : N - 1;
        boff[it] = (unsigned)(((size_t)(gn - col0) * Kd + c * 8) * 2);
      }
    }
    bstep = (NN ? (size_t)BK * N : (size_t)BK) * 2;
  };

  // fragment addressing: lane l = 16 kg + r16 holds contraction indices 8 kg .. 8 kg + 7 (of the
  // 32 of a half tile) of row / column r16 of the fragment
  const int r16 = lane & 15, kg = lane >> 4;
  const int fsw = (r16 >> 1) & 7;
  const int a_row_off = (wm * WM + r16) * ROWB;
  const int b_row_off = (wn * WN + r16) * ROWB;
  const int kq = r16 >> 2;
  const int nn_k = 8 * kg + kq;                   // first of the lane's two 4-row pieces of the W tile
  const int nn_n = wn * WN + 4 * (r16 & 3);

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  bf16x8 af[2][HM], bfr[FN];

  // weight fragment j of half q of the tile in sb
  auto read_b = [&](const char* sb, int q, int j) {
    if (NN) {
      const int k = 32 * q + nn_k;
      const int n = nn_n + 16 * j;
      const int phys = (n >> 3) ^ ((kq << 2) | ((kg & 1) << 1));
      const char* p0 = sb + k * 512 + phys * 16 + (n & 7) * 2;
      bfr[j] = lds_read_tr_pair(p0, p0 + 4 * 512);
    } else {
      bfr[j] = *(const bf16x8*)(sb + b_row_off + j * 16 * ROWB + (((4 * q + kg) ^ fsw) << 4));
    }
  };
  // row fragment i (0..HM-1) of half h of the wave's rows, half q of the tile in sa
  auto read_a = [&](const char* sa, int q, int h, int i, bf16x8 (&af)[HM]) {
    af[i] = *(const bf16x8*)(sa + a_row_off + (h * HM + i) * 16 * ROWB + (((4 * q + kg) ^ fsw) << 4));
  };

  // ---- LoRA contraction tiles.  After the last operand pair's base tiles the same pipeline runs the tiles of `lora`: the
  // A side is the tasks' slices of L (Z or G; zeros for the other pieces), the B side the same ranks of R_k (B_k
  // or A_k), fetched into the same LDS layouts by the same direct loads two tiles ahead, so the LoRA term
  // costs ceil(r_k / 32) more half tiles on the same accumulators and no exposed load latency.
  LoraTiles lora{0, 0};
  // what the load slots of a tile fetch: base tile kt of the current operand pair, or a LoRA tile.
  // `left`: contraction indices of the tile, fewer than 64 in the last one of features that are no multiple of 64
  struct LoadCtx {
    bool lora;
    const char* atile;
    const char* btile;
    int lt;              // which LoRA tile
    int left, Kd;
  };
  auto base_ctx = [&](int kt) {
    return LoadCtx{false, abase + (size_t)kt * (BK * 2), bbase + (size_t)kt * bstep, 0, BK, 0};
  };
  const char* const zeros = reinterpret_cast<const char*>(&g_zero_chunk);
  // wave-wide load number idx (0..LPA-1: A side, LPA..PER_TILE-1: Bm side) of a base tile that needs no masks
  auto issue_one = [&](const LoadCtx& lc, int idx, char* sa, char* sb) {
    if (idx < LPA)
      load_lds_16B_sbase(lc.atile, aoff[idx], sa + (wave + NW * idx) * 1024);
    else
      load_lds_16B_sbase(lc.btile, boff[idx - LPA], sb + (wave + NW * (idx - LPA)) * 1024);
  };
  // One side of a partial or LoRA tile.  The loops are rolled: this code stands in every launch's path, where it is
  // fetched cold, and runs a few times at most.
  auto masked = [](const LoadCtx& lc) { return (!HALF && lc.lora) || (TAIL && lc.left < BK); };
  // (the chunk a lane fetches: the same in every load of a wave, the rows of two loads are a multiple of 16 apart)
  const int kchunk = (lane % CPR) ^ ((RPI * wave + lane / CPR) / RW % CPR);
  static_assert(RPI * NW % (RW * CPR) == 0, "chunk of a lane");
  auto issue_masked_a = [&](const LoadCtx& lc, char* sa) {
    const int h = kchunk >> 2;                     // (LoRA: the half of the tile, i.e. the slot)
    const char* base = lc.atile;
    int ld = lc.Kd, q = kchunk * 8, end = lc.left, task = -1;
    if (!HALF && lc.lora) {
      const LoraSlot s0 = lora_slot(lora, lc.lt, 0), s1 = lora_slot(lora, lc.lt, 1);
      const int l0 = ga.ldz[s0.sg], l1 = ga.ldz[s1.sg];
      const bf16 *p0 = ga.L[s0.sg], *p1 = ga.L[s1.sg];
      base = reinterpret_cast<const char*>(h ? p1 : p0);
      ld = end = h ? l1 : l0;
      q = (h ? s1.q0 : s0.q0) + (kchunk & 3) * 8;
      task = h ? s1.k : s0.k;
    }
#pragma clang loop unroll(disable)
    for (int it = 0; it < LPA; ++it) {
      const int w = wave + NW * it;
      const int rl = RPI * w + lane / CPR;
      // (a LoRA tile: the rows of its tasks)
      const bool in = q < end && (HALF || !lc.lora || frag_task(rl >> 5) == task);
      const int row = !HALF && lc.lora ? real_row(rl) : real_row(rl) - row0;
      load_lds_16B(in ? base + ((size_t)row * ld + q) * 2 : zeros, sa + w * 1024);
    }
  };
  auto issue_masked_b = [&](const LoadCtx& lc, char* sb) {
    const char *p0 = lc.btile, *p1 = lc.btile;
    int r0 = lc.left, r1 = lc.left, q0 = 0, q1 = 32;   // contraction indices that exist, first of each half
    if (!HALF && lc.lora) {
      const LoraSlot s0 = lora_slot(lora, lc.lt, 0), s1 = lora_slot(lora, lc.lt, 1);
      r0 = rank_of(ga, s0.sg, s0.k & 63);
      p0 = static_cast<const char*>(ga.R[s0.sg].p[s0.k & 63]) + (size_t)col0 * 2 * (NN ? 1 : r0);
      q0 = s0.q0;
      r1 = rank_of(ga, s1.sg, s1.k & 63);
      p1 = static_cast<const char*>(ga.R[s1.sg].p[s1.k & 63]) + (size_t)col0 * 2 * (NN ? 1 : r1);
      q1 = s1.q0;
      if (s1.k == (int)kNoSlot) r1 = 0;
    }
    // (NT: a lane's half is that of its chunk; NN: a load's rows lie in one half)
    const int ch = kchunk >> 2, cr = ch ? r1 : r0, cq = (ch ? q1 : q0) + (kchunk & 3) * 8;
    const char* const cp = ch ? p1 : p0;
#pragma clang loop unroll(disable)
    for (int it = 0; it < LPB; ++it) {
      const int w = wave + NW * it;
      const char* p = zeros;
      if (NN) {
        const int kr = 2 * w + (lane >> 5), n = ((lane & 31) ^ nn_swz(kr)) * 8;
        const bool hi = w >= 16;
        const int q = (hi ? q1 - 32 : q0) + kr;
        if (q < (hi ? r1 : r0) && col0 + n < N) p = (hi ? p1 : p0) + ((size_t)q * N + n) * 2;
      } else {
        const int rl = RPI * w + lane / CPR;
        if constexpr (RAG && !HALF) {
          if (lc.lora && ((r0 | r1) & 7) != 0) {
            const bf16* row = reinterpret_cast<const bf16*>(cp) + (size_t)rl * cr;
            bf16x8 v;
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = (col0 + rl < N && cq + e < cr) ? row[cq + e] : (bf16)0.f;
            *(bf16x8*)(sb + w * 1024 + lane * 16) = v;
            continue;
          }
        }
        if (col0 + rl < N && cq < cr) p = cp + ((size_t)rl * (!HALF && lc.lora ? cr : lc.Kd) + cq) * 2;
      }
      load_lds_16B(p, sb + w * 1024);
    }
  };

  // Which of the wave's WM / 32 pieces take part in each half of a tile: all of them in a base tile, the pieces of
  // the half's task in a LoRA tile (the others' MFMAs are skipped, and those of an empty slot).
  struct FragOn {
    bool on[2][WM / 32];
  };
  auto frags_of = [&](int lt, bool base) {
    FragOn f;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int k = base ? 0 : lora_slot(lora, lt, q).k;
#pragma unroll
      for (int i = 0; i < WM / 32; ++i) f.on[q][i] = base || frag_task(wm * (WM / 32) + i) == k;
    }
    return f;
  };

  // Sub-step S (0..3) of a tile: the MFMAs of (half q = S / 2 of the contraction tile, half
  // h = S % 2 of the wave's rows), weight fragment by weight fragment (MFMA number m uses weight
  // fragment m / HM and row fragment m % HM of set h).  Row fragments are double-buffered: the HM
  // fragments of the next sub-step are read behind the first HM MFMAs.  Weight fragments are
  // not: they serve both sub-steps of a half tile, and in the second of them (h = 1) fragment j
  // is re-read for the next half tile right behind its last MFMA (slot HM j + HM - 1), a whole
  // sub-step before its next use -- 16 registers instead of 32.  The reads come from (rsa, rsb)
  // (if rd); `load(n)` is called in the n-th slot behind the first HM that carries no read, and issues the
  // direct load that rides there, if any.  rd is std::true_type / std::false_type in
  // the steady-state loop, so that it compiles to straight-line code, and a plain bool in the few
  // tiles around it; `fo` is std::true_type there (base tiles: every piece) and a FragOn in
  // the tiles that may be LoRA tiles.
  auto substep = [&](auto S_, auto rd, const char* rsa, const char* rsb, auto load, const auto& fo) {
    constexpr int S = decltype(S_)::value;
    constexpr int q = S / 2, h = S % 2;
    constexpr int NS_ = (S + 1) % 4;                 // the sub-step whose row fragments are read now
    constexpr int nq = NS_ / 2, nh = NS_ % 2;
    int slot = 0;
#pragma unroll
    for (int m = 0; m < NMF; ++m) {
      const int j = m / HM, i = m % HM;
      bool on = true;
      if constexpr (!std::is_same_v<std::decay_t<decltype(fo)>, std::true_type>) on = fo.on[q][(h * HM + i) / 2];
      if (on) mfma_16x16x32(acc[h * HM + i][j], bfr[j], af[h][i]);
      if (rd && m < HM) read_a(rsa, nq, nh, m, af[nh]);
      if (rd && h == 1 && i == HM - 1) read_b(rsb, nq, j);
      if (m >= HM && !(h == 1 && i == HM - 1)) load(slot++);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  constexpr std::integral_constant<int, 0> S0{};
  constexpr std::integral_constant<int, 1> S1{};
  constexpr std::integral_constant<int, 2> S2{};
  constexpr std::integral_constant<int, 3> S3{};
  const LoadCtx none{false, nullptr, nullptr, 0, BK, 0};

  // A tile whose operands sit in (ca, cb): sub-steps 0..2 with the late loads of `lcl` into lsl (if ldl; whole
  // tiles: the A side of tile v + 2, half tiles: its Bm side), barrier, sub-step 3 with the reads of the next
  // tile's first fragments from (na, nb) (if rd) and the early loads of `lce` (if lde; whole tiles: the Bm side
  // of tile v + 2 into cb, half tiles: the A side of tile v + 3 into ca).
  // `behind`: whether loads of tile v + 2 follow those of tile v + 1 that the barrier waits for -- vector
  // loads return in order, so the wait leaves exactly the younger ones in flight.
  // Loads per sub-step: a wave-wide load keeps the CU's one address path busy for 16 cycles.
  constexpr int EARLY = HALF ? LPA : LPB, LATE = HALF ? LPB : LPA;
  constexpr int E_GAP = 2, L0 = LATE < 3 ? LATE : 3, L0_GAP = 4, L1 = LATE - L0 < 3 ? LATE - L0 : 3, L1_GAP = 3, L2 = LATE - L0 - L1;
  static_assert((EARLY - 1) * E_GAP < (FN - 1) * (HM - 1) && (L0 - 1) * L0_GAP < (FN - 1) * HM &&
                    (L1 == 0 || (L1 - 1) * L1_GAP < (FN - 1) * (HM - 1)) && (L2 == 0 || (L2 - 1) * L1_GAP < (FN - 1) * HM),
                "load slots");
  auto tile = [&](char* ca, char* cb, const char* na, const char* nb, auto rd, auto ldl, const LoadCtx& lcl, char* lsl,
                  auto lde, const LoadCtx& lce, auto behind, const auto& fo, char* lsa = nullptr) {
    // load `first` + n / gap of the side in every gap-th slot
    auto late = [&](int slot, int first, int count, int gap) {
      if (!ldl || slot % gap != 0 || slot / gap >= count || masked(lcl)) return;
      if constexpr (HALF)
        issue_one(lcl, LPA + first + slot / gap, nullptr, lsl);
      else
        issue_one(lcl, first + slot / gap, lsl, nullptr);
    };
    auto early = [&](int slot) {
      if (!lde || slot % E_GAP != 0 || slot / E_GAP >= EARLY || masked(lce)) return;
      if constexpr (HALF)
        issue_one(lce, slot / E_GAP, ca, nullptr);
      else
        issue_one(lce, LPA + slot / E_GAP, nullptr, cb);
    };
    if (ldl && masked(lcl)) {
      issue_masked_a(lcl, HALF ? lsa : lsl);
      if constexpr (HALF) issue_masked_b(lcl, lsl);
    }
    substep(S0, yes, ca, cb, [&](int slot) { late(slot, 0, L0, L0_GAP); }, fo);
    substep(S1, yes, ca, cb, [&](int slot) { late(slot, L0, L1, L1_GAP); }, fo);
    substep(S2, yes, ca, cb, [&](int slot) { late(slot, L0 + L1, L2, L1_GAP); }, fo);
    // the next tile has landed (this wave's part), every fragment of this tile is in registers
    // (the weight fragments of this half tile stay in use until sub-step 3 re-reads them)
    if (behind)
      wait_vmcnt<HALF ? PER_TILE : LPA>();
    else
      wait_vmcnt<0>();
    wait_lds();
    __builtin_amdgcn_s_barrier();
    if constexpr (!HALF) {
      if (lde && masked(lce)) issue_masked_b(lce, cb);
    }
    substep(S3, rd, na, nb, early, fo);
  };

  // ---- main contraction loop.  Tile v of a pass uses A stage v % 3 and Bm stage v % 2; the steady
  // state is unrolled by six so that stage addresses are constants.  Operand pairs run one after
  // the other.  When a pair's last tile has passed its barrier every wave holds that tile's last
  // fragments in registers, so all stages are free for the next pair's first tiles.
  int h0 = 0, h1 = 0;   // HALF: this block's range of the base tiles of all operand pairs
  if constexpr (HALF) {
    int total_kt = 0;
    for (int sg = 0; sg < NSEG; ++sg) total_kt += (ga.Kd[sg] + BK - 1) / BK;
    // (below 2^32: a contraction has up to 2^22 indices, so 16 ranges of 4 operand pairs of 2^16 tiles make 2^22)
    h0 = (int)((unsigned)total_kt * (unsigned)part / (unsigned)ga.parts);
    h1 = (int)((unsigned)total_kt * (unsigned)(part + 1) / (unsigned)ga.parts);
  }
  for (int sg = 0; sg < NSEG; ++sg) {
    const int last = TAIL ? ga.Kd[sg] % BK : 0;   // contraction indices of a last, partial tile (0: none)
    int KT = ga.Kd[sg] / BK, k0 = 0;         // whole base tiles of this pass
    int base_tiles = KT + (last != 0);
    if constexpr (HALF) {
      const int all = base_tiles, lo = h0 > 0 ? h0 : 0, hi = h1 < all ? h1 : all;
      h0 -= all;
      h1 -= all;
      if (lo >= hi) continue;
      k0 = lo;
      KT = (hi < KT ? hi : KT) - lo;
      base_tiles = hi - lo;
    }
    set_operands(ga.A[sg], ga.Bm[sg], ga.Kd[sg]);
    abase += (size_t)k0 * (BK * 2);
    bbase += (size_t)k0 * bstep;
    int VT = base_tiles;                     // tiles of this pass: base tiles, then (whole tiles, last pair) LoRA tiles
    auto ctx_of = [&](int v) {
      LoadCtx lc = base_ctx(v);
      lc.Kd = ga.Kd[sg];
      if (!HALF && v >= base_tiles) lc = LoadCtx{true, nullptr, nullptr, v - base_tiles, BK, 0};
      else if (v >= KT) lc.left = last;
      return lc;
    };
    auto issue_a = [&](const LoadCtx& lc, char* sa) {
      if (masked(lc)) return issue_masked_a(lc, sa);
#pragma unroll
      for (int idx = 0; idx < LPA; ++idx) issue_one(lc, idx, sa, nullptr);
    };
    auto issue_b = [&](const LoadCtx& lc, char* sb) {
      if (masked(lc)) return issue_masked_b(lc, sb);
#pragma unroll
      for (int idx = 0; idx < LPB; ++idx) issue_one(lc, LPA + idx, nullptr, sb);
    };
    auto stage_a = [&](int u) { return u % 3 == 0 ? sA0 : (u % 3 == 1 ? sA1 : sA2); };
    auto stage_b = [&](int u) {
      if constexpr (HALF) return u % 3 == 0 ? sB0 : (u % 3 == 1 ? sB1 : sB2);
      else return u % 2 == 0 ? sB0 : sB1;
    };
    // whole tiles: tiles 0 and 1.  HALF: also the A side of tile 2.  The first reads need tile 0
    // (the table of the LoRA tiles is made while tile 0, a base tile, is on its way: in front of it, every block paid for the table before
    // its first load.  Call, us: 13358 x 384 -> 3392 159.6 -> 157.7 and 180.7 -> 178.2 (6 and 40 tasks), 22548 x 192 -> 8064 forward
    // 184.8 -> 179.6, 8192 x 4096 -> 4096 437.9 -> 435.5)
#pragma unroll(HALF ? 3 : 1)
    for (int t = 0; t < (HALF ? 3 : 2); ++t) {
      if constexpr (!HALF) {
        if (t == 1 && sg == NSEG - 1) {
          lora = lora_tiles<NFR>(ga, [&](int f) { return frag_task(f); });
          VT += lora.n;
        }
      }
      if (t >= VT) break;
      const LoadCtx lc = ctx_of(t);
      issue_a(lc, stage_a(t));
      if (t < 2) issue_b(lc, stage_b(t));
    }
    // (RAG: a LoRA tile's weight side is stored from registers, so that fewer than PER_TILE loads may stand behind tile 0)
    if (VT > 2 && HALF) wait_vmcnt<PER_TILE + LPA>();
    else if (VT > 1 && !(RAG && !HALF && base_tiles == 1)) wait_vmcnt<PER_TILE>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int j = 0; j < FN; ++j) read_b(sB[0], 0, j);
#pragma unroll
    for (int i = 0; i < HM; ++i) read_a(sA[0], 0, 0, i, af[0]);
    __builtin_amdgcn_sched_barrier(0);
    int v = 0;
    // (A half tile's short contraction is not worth fetching six copies of the loop's code.)
    for (; !HALF && v + 7 < KT; v += 6) {
      tile(sA[0], sB[0], sA[1], sB[1], yes, yes, base_ctx(v + 2), sA[2], yes, base_ctx(v + 2), yes, yes);
      tile(sA[1], sB[1], sA[2], sB[0], yes, yes, base_ctx(v + 3), sA[0], yes, base_ctx(v + 3), yes, yes);
      tile(sA[2], sB[0], sA[0], sB[1], yes, yes, base_ctx(v + 4), sA[1], yes, base_ctx(v + 4), yes, yes);
      tile(sA[0], sB[1], sA[1], sB[0], yes, yes, base_ctx(v + 5), sA[2], yes, base_ctx(v + 5), yes, yes);
      tile(sA[1], sB[0], sA[2], sB[1], yes, yes, base_ctx(v + 6), sA[0], yes, base_ctx(v + 6), yes, yes);
      tile(sA[2], sB[1], sA[0], sB[0], yes, yes, base_ctx(v + 7), sA[1], yes, base_ctx(v + 7), yes, yes);
    }
    for (; v + 3 < KT; ++v)
      tile(stage_a(v), stage_b(v), stage_a(v + 1), stage_b(v + 1), yes, yes, base_ctx(v + 2), HALF ? stage_b(v + 2) : stage_a(v + 2), yes,
           base_ctx(HALF ? v + 3 : v + 2), yes, yes);
    // the last base tiles and the LoRA tiles
    auto frags_at = [&](int u) {
      return u < base_tiles ? frags_of(0, true) : frags_of(u - base_tiles, false);
    };
    for (; v < VT; ++v) {
      const LoadCtx lc = v + 2 < VT ? ctx_of(v + 2) : none;
      if constexpr (HALF)
        // (a partial tile's A side comes late, with its weight)
        tile(stage_a(v), stage_b(v), stage_a(v + 1), stage_b(v + 1), v + 1 < VT, v + 2 < VT, lc, stage_b(v + 2), no, none, v + 2 < VT, yes,
             stage_a(v + 2));
      else
        tile(stage_a(v), stage_b(v), stage_a(v + 1), stage_b(v + 1), v + 1 < VT, v + 2 < VT, lc, stage_a(v + 2), v + 2 < VT, lc,
             v + 2 < VT, frags_at(v));
    }
  }  // operand pairs

  // the accumulators were last written by MFMAs in inline assembly: wait states before other
  // instructions read them
  asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
  // ---- HALF: the LoRA term, from registers, with the last range.  Fragments straight from memory (a few
  // KB per block that the caches hold): lane 16 kg + r16 loads 8 ranks of row r16 of L, and of output
  // column r16 of R_k, which is kept while the pieces belong to the same task.
  if constexpr (PACKED) {
    const TaskWalk walk = task_walk(ga);
    const int end = row0 + BM < M ? row0 + BM : M, first = part == ga.parts - 1 ? first_task(ga, row0) : ga.K;
    for (int sg = 0; sg < NSEG; ++sg) {
      const bf16* L = ga.L[sg];
      const int ldz = ga.ldz[sg];
      for (int k = first; k < ga.K; ++k) {
        const int lo = task_begin(walk, k, ga.off[kMaxK]), hi = task_begin(walk, k + 1, ga.off[kMaxK]);
        if (lo >= end) break;
        if (hi <= lo) continue;
        const int r = rank_of(ga, sg, k);
        const bf16* Rk = static_cast<const bf16*>(ga.R[sg].p[k]);
        for (int q0 = 0; q0 < r; q0 += 32) {
          const int q = q0 + 8 * kg;
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            int n = col0 + wn * WN + 16 * j + r16;
            n = n < N ? n : N - 1;
            if (!NN && r % 8 == 0) {
              bfr[j] = *(const bf16x8*)(q < r ? Rk + (size_t)n * r + q : reinterpret_cast<const bf16*>(zeros));
              continue;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) bfr[j][e] = q + e < r ? Rk[NN ? (size_t)(q + e) * N + n : (size_t)n * r + q + e] : (bf16)0.f;
          }
#pragma unroll
          for (int i = 0; i < FM; ++i) {
            const int first_row = row0 + 16 * i, row = first_row + r16;
            if (hi <= first_row || lo >= first_row + 16 || first_row >= M) continue;
            const bf16x8 lf = *(const bf16x8*)(q < ldz ? L + (size_t)(row < M ? row : M - 1) * ldz + q : reinterpret_cast<const bf16*>(zeros));
#pragma unroll
            for (int j = 0; j < FN; ++j) {
              const f32x4 t = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], lf, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[i][j][e] += row >= lo && row < hi ? t[e] : 0.f;
            }
          }
        }
      }
    }
  } else if constexpr (HALF) {
    for (int sg = 0; part == ga.parts - 1 && sg < NSEG; ++sg) {
      const bf16* L = ga.L[sg];
      const int ldz = ga.ldz[sg];
      for (int q0 = 0; q0 < ldz; q0 += 32) {
        int held = -1;
#pragma unroll
        for (int f = 0; f < NFR; ++f) {
          const int k = frag_task(f);
          if (k < 0) continue;
          const int r = ga.rank[sg][k];
          if (q0 >= r) continue;
          const int q = q0 + 8 * kg;
          if (k != held) {
            held = k;
            const bf16* Rk = static_cast<const bf16*>(ga.R[sg].p[k]);
#pragma unroll
            for (int j = 0; j < FN; ++j) {
              int n = col0 + wn * WN + 16 * j + r16;
              n = n < N ? n : N - 1;
              // A_k's whole 16-byte chunks in one piece (128 rows of 4 tasks, 256 x 256, rank 128: the input
              // gradient 26 us, element by element 75)
              if (!NN && r % 8 == 0) {
                bfr[j] = *(const bf16x8*)(q < r ? Rk + (size_t)n * r + q : reinterpret_cast<const bf16*>(zeros));
                continue;
              }
#pragma unroll
              for (int e = 0; e < 8; ++e)
                bfr[j][e] = q + e < r ? Rk[NN ? (size_t)(q + e) * N + n : (size_t)n * r + q + e] : (bf16)0.f;
            }
          }
          const int n = frag_n(f);
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int o = 16 * i + r16;
            bf16x8 lf;
            if (q < ldz) {
              lf = *(const bf16x8*)(L + (size_t)(frag_row(f) + (o < n ? o : n - 1)) * ldz + q);
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e) lf[e] = (bf16)0.f;
            }
#pragma unroll
            for (int j = 0; j < FN; ++j) acc[2 * f + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[j], lf, acc[2 * f + i][j], 0, 0, 0);
          }
        }
      }
    }
  }
  if constexpr (HALF) {
    if (ga.parts > 1) {
      // fp32 partial tile, one KiB per fragment in lane order (k_gemm_reduce reads it back the same way)
      float* dst = ga.part + ((size_t)part * 2 * (total - ga.t0) + 2 * (t - ga.t0) + half) * (BM * BN) + lane * 4;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        if (frag_n(i / 2) == 0) break;   // pieces beyond the last row come last
#pragma unroll
        for (int j = 0; j < FN; ++j) *(f32x4*)(dst + ((i * WAVES_N + wave) * FN + j) * 256) = acc[i][j];
      }
      return;
    }
  }
  // ---- output: through LDS, so that the tile leaves as 16 B per lane in full row segments of
  // the wave's sub-tile.  Each wave owns WM x WN x 2 bytes of the stage arrays (row stride WN x 2
  // bytes, chunk c of row m at c ^ swizzle(m)); nothing is shared between waves after the barrier.
  constexpr int OCH = WN / 8;                 // 16-byte chunks per output row of the wave's sub-tile
  constexpr int OROWB = WN * 2;               // bytes per such row
  constexpr int ORPI = 64 / OCH;              // rows per wave-wide store
  constexpr int WBYTES = WM * OROWB;          // bytes per wave
  constexpr int WPA = ABYTES / WBYTES;        // waves per A stage
  static_assert(ABYTES % WBYTES == 0 && (HALF ? NW == 3 * WPA + 1 : NW == 4 * WPA && ABYTES == BBYTES),
                "sub-tiles must fit the stage arrays");
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  auto oswz = [](int m) { return OCH == 8 ? ((m >> 1) & 7) : (m & (OCH - 1)); };
  __syncthreads();
  char* ep = sA0;
  if (wave / WPA == 1) ep = sA1;
  if (wave / WPA == 2) ep = HALF ? sA2 : sB0;
  if (wave / WPA == 3) ep = HALF ? sB0 : sB1;
  ep += (wave % WPA) * WBYTES;
  // lane 16 kg + r16 holds row 16 i + r16, columns 16 j + 4 kg + 0..3 of the wave's sub-tile
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = static_cast<bf16>(acc[i][j][e]);
      const int m = 16 * i + r16, c = 2 * j + (kg >> 1);
      *(bf16x4*)(ep + m * OROWB + ((c ^ oswz(m)) << 4) + 8 * (kg & 1)) = o;
    }
#pragma unroll
  for (int it = 0; it < WM / ORPI; ++it) {
    const int r = ORPI * it + lane / OCH, cp = lane % OCH;
    const int c = cp ^ oswz(r);
    const uint4 v = *(const uint4*)(ep + r * OROWB + cp * 16);
    // the row's piece of the block (WM is a multiple of 32; the rows of one store share a piece)
    const int f = (wm * WM + ORPI * it) >> 5, o = r & 31;
    const int grow = frag_row(f) + o, gcol = col0 + wn * WN + c * 8;
    // non-temporal: the output is not read again by this launch, so it should not displace the
    // operand strips in the L2 / Infinity Cache (measured +0.7 % on the whole forward + backward)
    if (o < frag_n(f) && gcol < N)
      __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), (u32x4*)(C + (size_t)grow * N + gcol));
  }
}

// Adds the contraction ranges of k_gemm_mfma<1, 4, ..> in order and writes the rows: block = 16 rows
// (fragment row i) of one half tile, a wave its 64 columns.
struct ReduceArgs {
  bf16* C;
  const float* part;
  int M, N, tiles_m, tiles_n, t0, parts, packed, K;
  int off[kMaxK + 1];
};
static __global__ __launch_bounds__(256) void k_gemm_reduce(const ReduceArgs a) {
  constexpr int GM = 8, FM = 8, FN = 4;
  const int i = blockIdx.x % FM, u = blockIdx.x / FM;
  const int t = a.t0 + u / 2;
  const int gsize = GM * a.tiles_n, group = t / gsize, first_m = group * GM;
  const int gm = (a.tiles_m - first_m) < GM ? (a.tiles_m - first_m) : GM;
  const int in_g = t - group * gsize;
  const int tm = 2 * (first_m + in_g % gm) + u % 2, tn = in_g / gm;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, kg = lane >> 4;
  const int v0 = tm * 128 + 16 * i;      // the fragment's first virtual row
  // (16 rows: the upper or lower half of a piece)
  RowPiece p;
  if (a.packed) {
    p = packed_piece(a.M, (unsigned)v0);
  } else {
    p = find_piece(a, row_axis(a), (unsigned)v0);
  }
  const int row = p.row, n = p.n;
  const int units = 2 * (a.tiles_m * a.tiles_n - a.t0);
  const float* src = a.part + (size_t)u * (128 * BN) + ((i * 4 + wave) * FN) * 256 + lane * 4;
  const size_t step = (size_t)units * (128 * BN);
  if (n <= 0) return;
  f32x4 acc[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s_ = 0; s_ < a.parts; ++s_)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[j] += *(const f32x4*)(src + s_ * step + j * 256);
  if (r16 >= n) return;
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int col = tn * BN + wave * 64 + 16 * j + 4 * kg;
    if (col < a.N) {
      bf16x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = static_cast<bf16>(acc[j][e]);
      *(bf16x4*)(a.C + (size_t)(row + r16) * a.N + col) = o;
    }
  }
}

}  // namespace gemmk
}  // namespace mlora
