// bf16 base products in small tiles (gfx950): the same operator as gemm_mfma_kernel.h,
//
//   C[M,N] = sum_g ( A_g[M,Kd_g] * op(Bm_g) + rows_k( L_g[rows_k, :r_gk] * R_gk ) ),
//
// for problems that leave most CUs without a 128 x 256 or 256 x 256 tile, and for features that are
// multiples of 8 but not of 64.
//
// Such calls are bound by latency, not by a rate: what a block does before, between and behind its MFMAs counts.
// A block of one or two groups of 4 waves owns a 64 x 64 tile; the waves of a group split each contraction tile, and two
// groups take every other one.  Contraction tiles of 64 come by direct global->LDS loads into a ring of three stages (NS) per
// group, NS - 1 tiles ahead of their use, with one barrier per tile; the loop is rolled (its code is fetched cold by
// every launch).  The LoRA term is more contraction tiles from the same ring, of two slots of 32 ranks each, so that no
// load of it is waited for at the end.
//
// Features that are no multiple of 64: the last contraction tile's chunks beyond the features come from 16 zero
// bytes (a direct load cannot be masked); chunks of 8 are whole, so stores are too.
#pragma once

#include "gemm_mfma_kernel.h"

namespace mlora {
namespace ringk {

using namespace stage;
using namespace rowaxis;
using gemmk::f32x4;
using gemmk::GemmArgs;

// Block id -> (tile, range).  Consecutive ids go round-robin over the 8 XCDs; each XCD takes a contiguous
// eighth of the order (8 row tiles x all column tiles at a time, column by column), so that the blocks it runs
// together share operand strips in its L2.
struct Tile {
  int tm, tn;
};
__device__ __forceinline__ Tile tile_of(int t, int tiles_m, int tiles_n) {
  constexpr int GM = 8;
  const int gsize = GM * tiles_n, group = t / gsize, first = group * GM;
  const int gm = (tiles_m - first) < GM ? (tiles_m - first) : GM;
  const int in_g = t - group * gsize;
  return Tile{first + in_g % gm, in_g / gm};
}

constexpr int NS = 3;
template <int G> constexpr int kRingLds = G * NS * 2 * 64 * 128;
template <int G, bool NN, int NSEG>
__device__ __forceinline__ void ring_body(const GemmArgs<NSEG>& ga, int bid, char* sm) {
  constexpr int BK = 64, BM = 64, BN = 64, NFR = 2;
  constexpr int ABYTES = BM * 128, SBYTES = 2 * ABYTES;
  constexpr int LP = 2, PER_TILE = 2 * LP;             // wave-wide loads of 1 KiB per wave and tile: A, Bm
  static_assert((NS - 2) * PER_TILE < 64 && NS >= 3, "vmcnt range");
  static_assert(G == 1 || G == 2, "groups of four waves");
  static_assert(G * NS * SBYTES >= (G == 1 ? 48 : 64) * 1024, "the waves' sums fit the rings");

  const int N = ga.N;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3), grp = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 8);
  char* const ring = sm + grp * (NS * SBYTES);
  const int units = ga.tiles_m * ga.tiles_n, per = units * ga.parts / 8;
  const int u = bid < 8 * per ? (bid % 8) * per + bid / 8 : bid;
  const int unit = u / ga.parts, part = u % ga.parts;
  const Tile bt = tile_of(unit, ga.tiles_m, ga.tiles_n);
  const int col0 = bt.tn * BN;

  // the block's pieces of 32 virtual rows
  RowPiece pc[NFR];
  {
    const RowAxis axis = row_axis(ga);
#pragma unroll
    for (int f = 0; f < NFR; ++f) pc[f] = find_piece(ga, axis, (unsigned)(bt.tm * BM + 32 * f));
  }
  if (pc[0].n == 0) return;
  const int row0 = pc[0].row;

  // this range's share of the contraction tiles of all operand pairs
  int h0 = 0, h1 = 0;
  {
    int total_kt = 0;
#pragma unroll
    for (int sg = 0; sg < NSEG; ++sg) total_kt += (ga.Kd[sg] + BK - 1) / BK;
    // (below 2^32: a contraction has up to 2^22 indices, so 16 ranges of 4 operand pairs of 2^16 tiles make 2^22)
    h0 = (int)((unsigned)total_kt * (unsigned)part / (unsigned)ga.parts);
    h1 = (int)((unsigned)total_kt * (unsigned)(part + 1) / (unsigned)ga.parts);
  }
  // LoRA tiles, with the last range
  gemmk::LoraTiles lora{0, 0};
  bool ragged = false;                 // whether some A_k's rows are no whole chunks
  if (part == ga.parts - 1) {
    lora = gemmk::lora_tiles<NFR>(ga, [&](int f) { return pc[f].task; });
    if constexpr (!NN) {
#pragma unroll
      for (int sg = 0; sg < NSEG; ++sg)
#pragma unroll
        for (int f = 0; f < NFR; ++f) ragged = ragged || (pc[f].task >= 0 && gemmk::rank_of(ga, sg, pc[f].task) % 8 != 0);
    }
  }

  // what this lane fetches: row and 16-byte chunk of each wave-wide load, which covers 8 rows of 128 bytes.  Load `it` of
  // wave w takes rows 8 w + 32 it ..: rows of one piece.  K-contiguous tiles (A, and Bm when !NN) keep chunk c of
  // row r at c ^ ((r >> 1) & 7); Bm when NN keeps its contraction rows as they are in memory, the
  // chunks permuted for the transposing reads
  const int lrow = 8 * wave + (lane >> 3), lchunk = lane & 7;
  const int kchunk = lchunk ^ ((lrow >> 1) & 7);
  auto nn_swz = [](int k) { return ((k >> 1) & 1) << 2; };
  int arow[LP];                        // real row - row0
#pragma unroll
  for (int it = 0; it < LP; ++it) {
    const int n = pc[it].n;
    arow[it] = pc[it].row - row0 + (lrow < n ? lrow : (n > 0 ? n - 1 : 0));
  }
  const char* const zeros = reinterpret_cast<const char*>(&gemmk::g_zero_chunk);

  // Wave w multiplies the whole tile by contraction indices 16 w .. 16 w + 15 of every contraction tile: a 2 x 2
  // arrangement of the waves would read every fragment twice.  32 x 32 x 16 fragments: lane 32 lhi + l32 holds
  // contraction indices 8 lhi .. + 7 of row / column l32.
  const int l32 = lane & 31, lhi = lane >> 5;
  const int foff = l32 * 128 + (((2 * wave + lhi) ^ ((l32 >> 1) & 7)) << 4);
  const int L16 = lane & 15, blk = lane >> 4;
  const int tr_k = 16 * wave + 8 * (blk >> 1) + (L16 >> 2), tr_n = 16 * (blk & 1) + 4 * (L16 & 3);

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  bf16x8 af[2], bf[2];
  auto read = [&](const char* st) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      af[j] = *(const bf16x8*)(st + j * 4096 + foff);
      if constexpr (NN) {
        const int n = 32 * j + tr_n;
        const char* p0 = st + ABYTES + tr_k * 128 + (((n >> 3) ^ nn_swz(tr_k)) << 4) + (n & 7) * 2;
        bf[j] = lds_read_tr_pair(p0, p0 + 4 * 128);   // (four rows on, the swizzle is the same)
      } else {
        bf[j] = *(const bf16x8*)(st + ABYTES + j * 4096 + foff);
      }
    }
  };
  auto multiply = [&](bool on0, bool on1) {
    if (on0) {
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[0], af[0], acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[1], af[0], acc[0][1], 0, 0, 0);
    }
    if (on1) {
      acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[0], af[1], acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[1], af[1], acc[1][1], 0, 0, 0);
    }
  };

  for (int sg = 0; sg < NSEG; ++sg) {
    const int Kd = ga.Kd[sg], KT = (Kd + BK - 1) / BK;
    const int lo = h0 > 0 ? h0 : 0, hi = h1 < KT ? h1 : KT;
    h0 -= KT;
    h1 -= KT;
    const int n_base = hi > lo ? hi - lo : 0, VT = n_base + (sg == NSEG - 1 ? lora.n : 0);
    if (VT == 0) continue;
    const char* abase = reinterpret_cast<const char*>(ga.A[sg] + (size_t)row0 * Kd);
    const char* bbase = reinterpret_cast<const char*>(NN ? ga.Bm[sg] + col0 : ga.Bm[sg] + (size_t)col0 * Kd);
    const size_t bstep = (NN ? (size_t)BK * N : (size_t)BK) * 2;
    unsigned aoff[LP], boff[LP];
#pragma unroll
    for (int it = 0; it < LP; ++it) {
      aoff[it] = (unsigned)(((size_t)arow[it] * Kd + kchunk * 8) * 2);
      const int rl = lrow + 32 * it;
      if constexpr (NN) {
        const int c = (lchunk ^ nn_swz(rl)) * 8, n = col0 + c < N ? c : N - 8 - col0;
        boff[it] = (unsigned)(((size_t)rl * N + n) * 2);
      } else {
        const int gn = col0 + rl < N ? rl : N - 1 - col0;
        boff[it] = (unsigned)(((size_t)gn * Kd + kchunk * 8) * 2);
      }
    }
    const int full = Kd / BK - lo;     // (this range's tiles before it need no masks)
    auto issue = [&](int v, char* st) {
      char* const da = st + wave * 1024;
      char* const db = da + ABYTES;
      if (v < n_base) {
        const char* at = abase + (size_t)(lo + v) * (BK * 2);
        const char* bt_ = bbase + (size_t)(lo + v) * bstep;
        if (v < full) {
#pragma unroll
          for (int it = 0; it < LP; ++it) load_lds_16B_sbase(at, aoff[it], da + it * 4096);
#pragma unroll
          for (int it = 0; it < LP; ++it) load_lds_16B_sbase(bt_, boff[it], db + it * 4096);
          return;
        }
        const int left = Kd - (lo + v) * BK;           // contraction indices of this tile: a multiple of 8
        const bool in = kchunk * 8 < left;
#pragma unroll
        for (int it = 0; it < LP; ++it) load_lds_16B(in ? at + aoff[it] : zeros, da + it * 4096);
#pragma unroll
        for (int it = 0; it < LP; ++it)
          load_lds_16B((NN ? lrow + 32 * it < left : in) ? bt_ + boff[it] : zeros, db + it * 4096);
        return;
      }
      const gemmk::LoraSlot s0 = gemmk::lora_slot(lora, v - n_base, 0), s1 = gemmk::lora_slot(lora, v - n_base, 1);
      const int r0 = gemmk::rank_of(ga, s0.sg, s0.k & 63), r1 = s1.k == (int)gemmk::kNoSlot ? 0 : gemmk::rank_of(ga, s1.sg, s1.k);
      const bf16* const R0 = static_cast<const bf16*>(ga.R[s0.sg].p[s0.k & 63]);
      const bf16* const R1 = static_cast<const bf16*>(ga.R[s1.sg].p[s1.k & 63]);
      // K-contiguous: a lane's chunk lies in one half of the tile, i.e. one slot
      const int h = kchunk >> 2, q = (h ? s1.q0 : s0.q0) + (kchunk & 3) * 8, r = h ? r1 : r0, ldz = h ? ga.ldz[s1.sg] : ga.ldz[s0.sg];
      const bf16* const L = h ? ga.L[s1.sg] : ga.L[s0.sg];
      const int task = h ? s1.k : s0.k;
#pragma unroll
      for (int it = 0; it < LP; ++it)
        load_lds_16B(pc[it].task == task && q < ldz ? reinterpret_cast<const char*>(L + (size_t)(row0 + arow[it]) * ldz + q) : zeros,
                     da + it * 4096);
#pragma unroll
      for (int it = 0; it < LP; ++it) {
        const int rl = lrow + 32 * it;
        if constexpr (NN) {
          // (load `it` holds the ranks of slot `it`)
          const int qn = (it ? s1.q0 : s0.q0) + lrow, n = col0 + (lchunk ^ nn_swz(rl)) * 8;
          load_lds_16B(qn < (it ? r1 : r0) && n < N ? reinterpret_cast<const char*>((it ? R1 : R0) + (size_t)qn * N + n) : zeros, db + it * 4096);
        } else {
          const int n = col0 + rl;
          const bf16* const Rk = h ? R1 : R0;
          if (((r0 | r1) & 7) != 0) {
            // A_k's rows are no whole chunks: put together in registers
            bf16x8 v8;
#pragma unroll
            for (int e = 0; e < 8; ++e) v8[e] = n < N && q + e < r ? Rk[(size_t)n * r + q + e] : (bf16)0.f;
            *(bf16x8*)(db + it * 4096 + lane * 16) = v8;
          } else {
            load_lds_16B(n < N && q < r ? reinterpret_cast<const char*>(Rk + (size_t)n * r + q) : zeros, db + it * 4096);
          }
        }
      }
    };
    // Tile v of group g is tile G v + g of the pass.  Of these, `count` exist and the loads of `counted` can be counted (the
    // ragged LoRA tiles issue fewer)
    const int count = (VT - grp + G - 1) / G, counted = ragged ? (n_base - grp + G - 1) / G : count, steps = (VT + G - 1) / G;
    // (the previous operand pair's last tile has been read before its stage is filled again)
    if (NSEG > 1) {
      wait_lds();
      __builtin_amdgcn_s_barrier();
    }
#pragma unroll 1
    for (int s = 0; s < NS - 1 && s < count; ++s) issue(G * s + grp, ring + s * SBYTES);   // (one copy of the code)
    // One barrier per tile: tile v has landed (this wave's part; the NS - 2 younger tiles may be in flight), every wave has
    // read tile v - 1, whose stage is filled next, while the fragments of tile v are on their way to the registers.
    int s = 0, v = 0;
    auto advance = [&]() {
      if (v + NS - 2 < counted) wait_vmcnt<(NS - 2) * PER_TILE>();
      else wait_vmcnt<0>();
      wait_lds();
      __builtin_amdgcn_s_barrier();
      read(ring + s * SBYTES);
      const int fill = s == 0 ? NS - 1 : s - 1;
      if (v + NS - 1 < count) issue(G * (v + NS - 1) + grp, ring + fill * SBYTES);
      s = s + 1 == NS ? 0 : s + 1;
    };
#pragma unroll 1
    for (; v < n_base / G; ++v) {
      advance();
      multiply(true, true);
    }
#pragma unroll 1
    for (; v < steps; ++v) {
      advance();
      const int t = G * v + grp;
      bool on0 = t < n_base, on1 = on0;
      if (!on0 && t < VT) {
        // (this wave's 16 contraction indices lie in one slot)
        const gemmk::LoraSlot l = gemmk::lora_slot(lora, t - n_base, wave >> 1);
        on0 = pc[0].task == l.k;
        on1 = pc[1].task == l.k;
      }
      multiply(on0, on1);
    }
  }

  // The waves' sums: wave 2 i + j adds up quadrant (i, j), in wave order.  Slot (q, w) of 4 KiB holds wave w's sums
  // of quadrant q (w counted without the owner).
  wait_lds();
  __builtin_amdgcn_s_barrier();
  if constexpr (G == 2) {
    // the second group's sums go to the first
    char* const mine = sm + wave * 16384 + lane * 16;
    if (grp == 1) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          *(f32x4*)(mine + (4 * q + g) * 1024) = f32x4{acc[q / 2][q % 2][4 * g], acc[q / 2][q % 2][4 * g + 1], acc[q / 2][q % 2][4 * g + 2], acc[q / 2][q % 2][4 * g + 3]};
    }
    __syncthreads();
    if (grp == 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 x = *(const f32x4*)(mine + (4 * q + g) * 1024);
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[q / 2][q % 2][4 * g + e] += x[e];
        }
    }
    wait_lds();
    __syncthreads();
    if (grp == 1) return;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (q == wave) continue;
    char* dst = sm + (3 * q + (wave > q ? wave - 1 : wave)) * 4096 + lane * 16;
#pragma unroll
    for (int g = 0; g < 4; ++g) *(f32x4*)(dst + g * 1024) = f32x4{acc[q / 2][q % 2][4 * g], acc[q / 2][q % 2][4 * g + 1], acc[q / 2][q % 2][4 * g + 2], acc[q / 2][q % 2][4 * g + 3]};
  }
  __syncthreads();
  f32x4 sum[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    f32x4 own;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float a0 = acc[0][0][4 * g + e], a1 = acc[0][1][4 * g + e], a2 = acc[1][0][4 * g + e], a3 = acc[1][1][4 * g + e];
      own[e] = wave == 0 ? a0 : (wave == 1 ? a1 : (wave == 2 ? a2 : a3));
    }
    const char* src = sm + 3 * wave * 4096 + g * 1024 + lane * 16;
    f32x4 x[3];
#pragma unroll
    for (int w = 0; w < 3; ++w) x[w] = *(const f32x4*)(src + w * 4096);
    // (waves 0 .. 3 in order)
    const f32x4 w0 = wave == 0 ? own : x[0], w1 = wave == 1 ? own : (wave == 0 ? x[0] : x[1]);
    const f32x4 w2 = wave == 2 ? own : (wave == 3 ? x[2] : x[1]), w3 = wave == 3 ? own : x[2];
    sum[g] = ((w0 + w1) + w2) + w3;
  }
  // lane holds row l32 and columns 8 g + 4 lhi + 0..3 of quadrant (wave / 2, wave % 2)
  if (ga.parts > 1) {
    float* dst = ga.part + (((size_t)part * units + unit) * 4 + wave) * 1024 + lane * 4;
#pragma unroll
    for (int g = 0; g < 4; ++g) *(f32x4*)(dst + g * 256) = sum[g];
    return;
  }
  // output through LDS, so that it leaves in whole row segments: 64 columns of a row, chunk c of row m at c ^ (m & 7)
  __syncthreads();
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = static_cast<bf16>(sum[g][e]);
    const int m = 32 * (wave >> 1) + l32, c = 4 * (wave & 1) + g;
    *(bf16x4*)(sm + m * 128 + ((c ^ (m & 7)) << 4) + 8 * lhi) = o;
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int o = tid >> 3, m = 32 * it + o, c = tid & 7, col = col0 + c * 8;
    const uint4 v = *(const uint4*)(sm + m * 128 + ((c ^ (m & 7)) << 4));
    if (o < pc[it].n && col < N) *(uint4*)(ga.C + (size_t)(pc[it].row + o) * N + col) = v;
  }
}

template <int G, bool NN, int NSEG>
__global__ __launch_bounds__(256 * G, G == 1 ? 3 : 2) void k_gemm_ring(const GemmArgs<NSEG> ga) {
  __shared__ __attribute__((aligned(1024))) char sm[kRingLds<G>];
  ring_body<G, NN, NSEG>(ga, blockIdx.x, sm);
}

// Adds the contraction ranges in order and writes the rows: block = a quarter of each quadrant of a tile, a wave one of
// them (32 rows x 8 columns).
struct RingReduceArgs {
  bf16* C;
  const float* part;
  int M, N, tiles_m, tiles_n, parts, K;
  int off[kMaxK + 1];
};
static __global__ __launch_bounds__(256) void k_ring_reduce(const RingReduceArgs a) {
  const int lane = threadIdx.x & 63, l32 = lane & 31, lhi = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int unit = blockIdx.x / 4, g = blockIdx.x % 4;
  const Tile bt = tile_of(unit, a.tiles_m, a.tiles_n);
  const RowPiece p = find_piece(a, row_axis(a), (unsigned)(bt.tm * 64 + (wave >> 1) * 32));
  if (p.n <= 0) return;
  const float* src = a.part + ((size_t)unit * 4 + wave) * 1024 + g * 256 + lane * 4;
  const size_t step = (size_t)a.tiles_m * a.tiles_n * 4096;
  f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = 0; s < a.parts; ++s) sum += *(const f32x4*)(src + s * step);
  const int col = bt.tn * 64 + (wave & 1) * 32 + 8 * g + 4 * lhi;
  if (l32 >= p.n || col >= a.N) return;
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = static_cast<bf16>(sum[e]);
  *(bf16x4*)(a.C + (size_t)(p.row + l32) * a.N + col) = o;
}

}  // namespace ringk
}  // namespace mlora
