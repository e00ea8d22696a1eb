// bf16 MFMA kernels for the low-rank products of the BatchLoRA operator (gfx950).
// Each one streams a full activation tensor once, so HBM bandwidth bounds them;
// MFMA keeps the arithmetic (up to 128 flop per byte at rank 64) off the critical path.
//
//   lowrank_rows   Z = s_k x_k A_k          (forward workflow, section 3.3.1; A_k is [h, r_k])
//                  G = s_k dy_k B_k^T       (first factor of Eq. "grad_lora" / "grad_output"; B_k is [r_k, d])
//   grad           dA_k = x_k^T G           (Eq. "grad_lora", left)
//                  dB_k = Z^T dy_k          (Eq. "grad_lora", right)
//
// One launch covers all tasks: a block finds its task from the split positions.
// Tiles are staged with direct global->LDS loads (16 B per lane) into a ring of three stages, two tiles in
// flight per block (some gradients: two stages and one tile), and two blocks per CU where they fit (an HBM-bound
// stream needs tens of KiB in flight per CU); operands whose contraction index is not contiguous in memory (A_k, and
// everything in the two gradient products, where the contraction runs over
// tokens) are read from LDS with the transposing ds_read_b64_tr_b16.
#include "mfma_staging.h"
#include "mlora_common.h"
#include "row_axis.h"

namespace mlora {
namespace {

using namespace stage;
using namespace rowaxis;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// Bank-conflict swizzle of a small tile stored with the contraction index as its rows
// ([64 k][w] bf16) and read with transposing LDS reads, which touch 4 consecutive rows x 64 B per
// 16 lanes: with rows of 128 or 256 B those rows would share banks, so the 64-byte segments of
// row k are permuted by XOR with seg_swizzle(k, w).  A direct-to-LDS load fills LDS contiguously,
// so the permutation is applied by choosing which global chunk each lane fetches, and undone in
// the read address (column n -> n ^ (seg_swizzle << 5)).
__device__ __forceinline__ int seg_swizzle(int k, int w) {
  return w == 128 ? (k & 3) : (w == 64 ? ((k >> 1) & 1) : 0);
}
// element offset inside the tile that LDS chunk position `chunk` (16 B units) must be filled with
__device__ __forceinline__ int swizzled_source(int chunk, int w) {
  const int cpr = w / 8;
  const int row = chunk / cpr, pc = chunk % cpr;
  const int seg = (pc >> 2) ^ seg_swizzle(row, w);
  return row * w + (((seg << 2) | (pc & 3)) << 3);
}

// A_k's tile (64 contraction indices x r, contiguous in memory) for ranks that are no multiple of 8:
// its rows are no whole 16-byte chunks, so it is filled in memory order (chunks beyond it re-fetch
// the first one) and never swizzled.
__device__ __forceinline__ int ragged_source(int chunk, int r) {
  if (r % 8 == 0) return swizzled_source(chunk, r);
  return 8 * chunk < 64 * r ? 8 * chunk : 0;
}
// MFMA operand of column n, contraction indices 8 (lane / 32) .. + 7 of step ks, from a tile with
// rows of r elements that are no multiple of 8 bytes (r % 4 != 0): element by element
__device__ __forceinline__ bf16x8 ragged_column(const char* ss, int ks, int j, int r, int lane, int zero_off) {
  asm volatile("" : "+v"(lane));   // addresses worked out here: hoisted out of the tile loop they fill the register file
  const int n = 32 * j + (lane & 31), k0 = 16 * ks + 8 * (lane >> 5);
  bf16x8 v;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = *(const bf16*)(ss + (n < r ? ((k0 + e) * r + n) * 2 : zero_off));
  return v;
}

// ------------------------------------------------------------------------------------------
// Arguments of the two kernels, passed by value.  NP > 1 serves projections that share their
// input: the big operand (X) is streamed once and multiplied with every projection's small
// operand; each projection has its own ranks, scalings, pointers and output.
// ------------------------------------------------------------------------------------------
template <int NP>
struct RowsArgs {
  const bf16* In;                       // [T, inner]
  int inner;
  int K;
  int off[kMaxK + 1];
  bf16* Out[NP];                        // [T, ldz_p]
  int ldz[NP];
  unsigned char rank[NP][kMaxK];
  float s[NP][kMaxK];
  PtrTable M[NP];
  // splits > 1 (NP == 1 only): the contraction is cut into `splits` ranges, one block each; range s
  // writes its fp32 sums of row i at part + (s * rows + i - off[0]) * ldz, rows = off[K] - off[0], and
  // k_rows_reduce adds the ranges in order
  int splits;
  float* part;
};

template <int NP>
struct GradArgs {
  const bf16* Big;                      // [T, wide]
  int wide, T;
  int K;
  int off[kMaxK + 1];
  const bf16* Small[NP];                // [T, ldz_p]
  int ldz[NP];
  unsigned char rank[NP][kMaxK];
  OutTable out[NP];
  int accumulate, chunks;
  // splits > 1 (NP == 1 only): a task's tokens are cut into `splits` ranges, one block each;
  // block (task k, range s) overwrites its partial sums at part + s * part_step + rbase_k * wide
  // (same element order as the output), and k_grad_reduce adds the ranges in order
  int splits;
  size_t part_step;
  float* part;
};

// ------------------------------------------------------------------------------------------
// Out_p[i, 0:ldz_p] = s_pk * In[i, :] * M_pk   for the rows i of task k; columns >= r_pk are zero.
//   SMALL_KMAJOR = true : M_k = A_k  [inner, r_k]  (rows of A_k are contraction indices)
//   SMALL_KMAJOR = false: M_k = B_k^T, B_k [r_k, inner]
// Block: TM rows of one task (TM = 32, 64 or 128), one wave per 32 rows, contraction tiles of 64.
// NQ = 32-column groups of the widest Out_p.
// RAG: some rank is no multiple of 8 (k-major operand; B_k's rows are whole chunks for any rank).
// ------------------------------------------------------------------------------------------
template <bool SMALL_KMAJOR, int NQ, int NS, int TM, int NP, bool RAG>
__global__ __launch_bounds__(TM * 2) void k_lowrank_mfma(const RowsArgs<NP> ra) {
  constexpr int NWV = TM / 32;                     // waves per block
  constexpr int SPW = (4 * NQ + NWV - 1) / NWV;    // 1 KiB pieces of one small operand per wave
  constexpr int SBYTES = NQ * 32 * 128;
  // a small-operand tile is followed by 64 zero bytes: where lanes beyond the tile's columns point
  constexpr int SREG = SBYTES + 1024;              // per projection; keeps every 1 KiB load slot aligned
  __shared__ __attribute__((aligned(1024))) char sX0[TM * 128];
  __shared__ __attribute__((aligned(1024))) char sX1[TM * 128];
  __shared__ __attribute__((aligned(1024))) char sX2[TM * 128];
  __shared__ __attribute__((aligned(1024))) char sX3[NS > 3 ? TM * 128 : 16];
  __shared__ __attribute__((aligned(1024))) char sS0[NP * SREG];
  __shared__ __attribute__((aligned(1024))) char sS1[NP * SREG];
  __shared__ __attribute__((aligned(1024))) char sS2[NP * SREG];
  __shared__ __attribute__((aligned(1024))) char sS3[NS > 3 ? NP * SREG : 64];
  static_assert(NS == 3 || NS == 4, "ring depth");
  static_assert(SMALL_KMAJOR || NP == 1, "shared-input form exists for the k-major operand only");
  char* const sX[4] = {sX0, sX1, sX2, sX3};
  char* const sS[4] = {sS0, sS1, sS2, sS3};

  const bf16* __restrict__ In = ra.In;
  const int inner = ra.inner;
  const int sp = NP == 1 ? blockIdx.x % ra.splits : 0;
  int lo = 0, hi = 0;
  const int k = rows_block<TM>(ra, NP == 1 ? blockIdx.x / ra.splits : blockIdx.x, &lo, &hi);
  if (k < 0) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (tid < 16) {
#pragma unroll
    for (int s_ = 0; s_ < NS; ++s_)
#pragma unroll
      for (int p = 0; p < NP; ++p) reinterpret_cast<int*>(sS[s_] + p * SREG + SBYTES)[tid] = 0;
  }

  const bf16* xptr[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int rl = 8 * (wave + NWV * it) + (lane >> 3);
    const int c = (lane & 7) ^ ((rl >> 1) & 7);
    int row = lo + rl;
    row = row < hi ? row : hi - 1;
    xptr[it] = In + (size_t)row * inner + c * 8;
  }
  int r[NP];
  size_t sstep[NP];
  const bf16* sptr[NP][SPW];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    r[p] = ra.rank[p][k];
    const bf16* Mk = static_cast<const bf16*>(ra.M[p].p[k]);
    const int pieces = (r[p] + 7) / 8;  // 1 KiB pieces of the small operand's tile
#pragma unroll
    for (int it = 0; it < SPW; ++it) {
      // pieces beyond the operand's rank re-fetch piece 0 into their own (never read) slot, so
      // that every wave issues the same number of loads per tile
      const int piece = (wave + NWV * it) < pieces ? (wave + NWV * it) : 0;
      if (SMALL_KMAJOR) {
        sptr[p][it] = Mk + (RAG ? ragged_source(piece * 64 + lane, r[p]) : swizzled_source(piece * 64 + lane, r[p]));
      } else {
        int q = 8 * piece + (lane >> 3);
        const int c = (lane & 7) ^ ((q >> 1) & 7);
        q = q < r[p] ? q : r[p] - 1;
        sptr[p][it] = Mk + (size_t)q * inner + c * 8;
      }
    }
    sstep[p] = SMALL_KMAJOR ? (size_t)64 * r[p] : (size_t)64;
  }

  auto issue = [&](int kt, char* sx, char* ss) {
#pragma unroll
    for (int it = 0; it < 4; ++it) load_lds_16B(xptr[it] + (size_t)kt * 64, sx + (wave + NWV * it) * 1024);
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int it = 0; it < SPW; ++it)
        load_lds_16B(sptr[p][it] + (size_t)kt * sstep[p], ss + p * SREG + (wave + NWV * it) * 1024);
  };
  // loads per wave per tile; the same for every wave because NWV divides 4 NQ
  static_assert((4 * NQ) % NWV == 0, "small-operand pieces must split evenly over the waves");
  constexpr int PER_TILE = 4 + NP * SPW;
  static_assert((NS - 2) * PER_TILE < 64, "vmcnt range");

  const int l32 = lane & 31, lhi = lane >> 5;
  const int fsw = (l32 >> 1) & 7;
  const int L16 = lane & 15, blk = lane >> 4, kq = L16 >> 2;
  const int tr_k = 8 * (blk >> 1) + kq;
  const int tr_n = 16 * (blk & 1) + 4 * (L16 & 3);

  f32x16 acc[NP][NQ];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int j = 0; j < NQ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[p][j][e] = 0.f;

  auto compute = [&](const char* sx, const char* ssall) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int coff = ((2 * ks + lhi) ^ fsw) << 4;
      const bf16x8 xf = *(const bf16x8*)(sx + (32 * wave + l32) * 128 + coff);
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const char* ss = ssall + p * SREG;
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
          if (32 * j < r[p]) {
            bf16x8 sf;
            if (SMALL_KMAJOR && RAG && r[p] % 4 != 0) {
              sf = ragged_column(ss, ks, j, r[p], lane, SBYTES);
            } else if (SMALL_KMAJOR) {
              const int n = 32 * j + tr_n;
              const int kk = 16 * ks + tr_k;
              const int ns = n ^ (seg_swizzle(kk, r[p]) << 5);
              const char* p0 = ss + ((n < r[p]) ? (kk * r[p] + ns) * 2 : SBYTES);
              const char* p1 = ss + ((n < r[p]) ? ((kk + 4) * r[p] + ns) * 2 : SBYTES);
              sf = join(lds_read_tr(p0), lds_read_tr(p1));
            } else {
              sf = *(const bf16x8*)(ss + (32 * j + l32) * 128 + coff);
            }
            acc[p][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sf, xf, acc[p][j], 0, 0, 0);
          }
        }
      }
    }
  };

  // NS-stage ring, one barrier per tile: before tile kt is read, this wave's loads of tile kt
  // have landed (the loads of the NS-2 younger tiles may stay in flight); the barrier then makes
  // every wave's part of tile kt visible and tells that all waves are done with tile kt-1,
  // whose stage is refilled next.
  int KT = inner / 64;
  if (NP == 1 && ra.splits > 1) {
    // (below 2^32: 16 ranges of a contraction of up to 2^22 indices, 2^16 tiles)
    const int k0 = (int)((unsigned)KT * (unsigned)sp / (unsigned)ra.splits), k1 = (int)((unsigned)KT * (unsigned)(sp + 1) / (unsigned)ra.splits);
#pragma unroll
    for (int it = 0; it < 4; ++it) xptr[it] += (size_t)k0 * 64;
#pragma unroll
    for (int it = 0; it < SPW; ++it) sptr[0][it] += (size_t)k0 * sstep[0];
    KT = k1 - k0;
  }
  __syncthreads();  // the zero pads
#pragma unroll
  for (int s_ = 0; s_ < NS - 1; ++s_)
    if (s_ < KT) issue(s_, sX[s_], sS[s_]);
  for (int kt0 = 0; kt0 < KT; kt0 += NS) {
#pragma unroll
    for (int s_ = 0; s_ < NS; ++s_) {
      const int kt = kt0 + s_;
      if (kt < KT) {
        if (kt + NS - 2 < KT)
          wait_vmcnt<(NS - 2) * PER_TILE>();
        else
          wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        if (kt + NS - 1 < KT) issue(kt + NS - 1, sX[(s_ + NS - 1) % NS], sS[(s_ + NS - 1) % NS]);
        compute(sX[s_], sS[s_]);
      }
    }
  }

  // lane holds row m = 32*wave + l32 and columns q = 32j + 8g + 4*lhi + 0..3
  const int row = lo + 32 * wave + l32;
  if (NP == 1 && ra.splits > 1) {
    if (row < hi) {
      const int ldz = ra.ldz[0];
      float* part = ra.part + ((size_t)sp * (ra.off[ra.K] - ra.off[0]) + row - ra.off[0]) * ldz;
#pragma unroll
      for (int j = 0; j < NQ; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int q = 32 * j + 8 * g + 4 * lhi;
          if (q < r[0])
            *(f32x4*)(part + q) = f32x4{acc[0][j][4 * g], acc[0][j][4 * g + 1], acc[0][j][4 * g + 2], acc[0][j][4 * g + 3]};
        }
    }
    return;
  }
  if (row < hi) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const float s = ra.s[p][k];
      const int ldz = ra.ldz[p];
      bf16* __restrict__ Out = ra.Out[p];
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int q = 32 * j + 8 * g + 4 * lhi;
          if (q < ldz) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = static_cast<bf16>((q + e < r[p]) ? acc[p][j][4 * g + e] * s : 0.f);
            *(bf16x4*)(Out + (size_t)row * ldz + q) = o;
          }
        }
      }
    }
  }
}

// Adds the contraction ranges of k_lowrank_mfma in order, scales and rounds.  One thread per four
// columns of a row.
__global__ __launch_bounds__(256) void k_rows_reduce(const RowsArgs<1> ra) {
  const int ldz = ra.ldz[0], rows = ra.off[ra.K] - ra.off[0], per = ldz / 4;
  const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
  if (t >= (long long)rows * per) return;
  const int i = (int)(t / per), q = (int)(t % per) * 4;
  const int k = task_of_row(ra, ra.off[0] + i);
  const int r = ra.rank[0][k];
  const float s = ra.s[0][k];
  f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
  if (q < r) {
    const float* p = ra.part + (size_t)i * ldz + q;
    const size_t step = (size_t)rows * ldz;
#pragma unroll 4
    for (int s_ = 0; s_ < ra.splits; ++s_) sum += *(const f32x4*)(p + s_ * step);
  }
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = static_cast<bf16>(q + e < r ? sum[e] * s : 0.f);
  *(bf16x4*)(ra.Out[0] + (size_t)(ra.off[0] + i) * ldz + q) = o;
}

// ------------------------------------------------------------------------------------------
// The same product for calls with few rows (the 32-row tiling still leaves the chip short of
// waves): a block owns 32 rows and its 4 waves split the contraction -- wave w takes the tiles
// kt = w, w + 4, ... through a ring of its own (no barrier in the loop: a wave reads only what
// its own loads wrote), then waves 1..3 hand their partial sums to wave 0 through LDS, which adds
// them in that order (deterministic) and writes the rows.  Ranks up to 64.
// ------------------------------------------------------------------------------------------
template <bool SMALL_KMAJOR, int NQ, int NS, bool RAG>
__global__ __launch_bounds__(256) void k_lowrank_mfma_splitk(const RowsArgs<1> ra) {
  constexpr int TM = 32, NSPLIT = 4;
  constexpr int SBYTES = NQ * 32 * 128;
  constexpr int SREG = SBYTES + 1024;
  constexpr int XB = TM * 128;
  static_assert(NQ <= 2, "LDS holds four rings only up to rank 64");
  __shared__ __attribute__((aligned(1024))) char sXall[NSPLIT * NS * XB];
  __shared__ __attribute__((aligned(1024))) char sSall[NSPLIT * NS * SREG];
  static_assert(3 * NQ * 16 * 256 <= NSPLIT * NS * SREG, "partial sums fit the small-operand rings");

  const bf16* __restrict__ In = ra.In;
  const int inner = ra.inner;
  int lo = 0, hi = 0;
  const int k = rows_block<TM>(ra, blockIdx.x, &lo, &hi);
  if (k < 0) return;
  const int r = ra.rank[0][k];
  const bf16* Mk = static_cast<const bf16*>(ra.M[0].p[k]);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  char* const sXw = sXall + wave * NS * XB;
  char* const sSw = sSall + wave * NS * SREG;
  if (lane < 16) {
#pragma unroll
    for (int s_ = 0; s_ < NS; ++s_) reinterpret_cast<int*>(sSw + s_ * SREG + SBYTES)[lane] = 0;
  }

  const bf16* xptr[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int rl = 8 * it + (lane >> 3);
    const int c = (lane & 7) ^ ((rl >> 1) & 7);
    int row = lo + rl;
    row = row < hi ? row : hi - 1;
    xptr[it] = In + (size_t)row * inner + c * 8;
  }
  const int pieces = (r + 7) / 8;
  const bf16* sptr[4 * NQ];
#pragma unroll
  for (int it = 0; it < 4 * NQ; ++it) {
    const int piece = it < pieces ? it : 0;
    if (SMALL_KMAJOR) {
      sptr[it] = Mk + (RAG ? ragged_source(piece * 64 + lane, r) : swizzled_source(piece * 64 + lane, r));
    } else {
      int q = 8 * piece + (lane >> 3);
      const int c = (lane & 7) ^ ((q >> 1) & 7);
      q = q < r ? q : r - 1;
      sptr[it] = Mk + (size_t)q * inner + c * 8;
    }
  }
  const size_t sstep = SMALL_KMAJOR ? (size_t)64 * r : (size_t)64;
  constexpr int PER_TILE = 4 + 4 * NQ;

  auto issue = [&](int kt, int stage) {
    char* sx = sXw + stage * XB;
    char* ss = sSw + stage * SREG;
#pragma unroll
    for (int it = 0; it < 4; ++it) load_lds_16B(xptr[it] + (size_t)kt * 64, sx + it * 1024);
#pragma unroll
    for (int it = 0; it < 4 * NQ; ++it) load_lds_16B(sptr[it] + (size_t)kt * sstep, ss + it * 1024);
  };

  const int l32 = lane & 31, lhi = lane >> 5;
  const int fsw = (l32 >> 1) & 7;
  const int L16 = lane & 15, blk = lane >> 4, kq = L16 >> 2;
  const int tr_k = 8 * (blk >> 1) + kq;
  const int tr_n = 16 * (blk & 1) + 4 * (L16 & 3);

  f32x16 acc[NQ];
#pragma unroll
  for (int j = 0; j < NQ; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

  auto compute = [&](int stage) {
    const char* sx = sXw + stage * XB;
    const char* ss = sSw + stage * SREG;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int coff = ((2 * ks + lhi) ^ fsw) << 4;
      const bf16x8 xf = *(const bf16x8*)(sx + l32 * 128 + coff);
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        if (32 * j < r) {
          bf16x8 sf;
          if (SMALL_KMAJOR && RAG && r % 4 != 0) {
            sf = ragged_column(ss, ks, j, r, lane, SBYTES);
          } else if (SMALL_KMAJOR) {
            const int n = 32 * j + tr_n;
            const int kk = 16 * ks + tr_k;
            const int ns = n ^ (seg_swizzle(kk, r) << 5);
            const char* p0 = ss + ((n < r) ? (kk * r + ns) * 2 : SBYTES);
            const char* p1 = ss + ((n < r) ? ((kk + 4) * r + ns) * 2 : SBYTES);
            sf = join(lds_read_tr(p0), lds_read_tr(p1));
          } else {
            sf = *(const bf16x8*)(ss + (32 * j + l32) * 128 + coff);
          }
          acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sf, xf, acc[j], 0, 0, 0);
        }
      }
    }
  };

  // this wave's tiles: kt = wave + 4 i, i < n
  const int KT = inner / 64;
  const int n = (KT - wave + NSPLIT - 1) / NSPLIT;
#pragma unroll
  for (int s_ = 0; s_ < NS - 1; ++s_)
    if (s_ < n) issue(wave + NSPLIT * s_, s_);
  for (int i0 = 0; i0 < n; i0 += NS) {
#pragma unroll
    for (int s_ = 0; s_ < NS; ++s_) {
      const int i = i0 + s_;
      if (i < n) {
        if (i + NS - 2 < n)
          wait_vmcnt<(NS - 2) * PER_TILE>();
        else
          wait_vmcnt<0>();
        // the stage of tile i-1 is refilled: its fragment reads have returned
        wait_lds();
        if (i + NS - 1 < n) issue(wave + NSPLIT * (i + NS - 1), (s_ + NS - 1) % NS);
        compute(s_);
      }
    }
  }

  // partial sums of waves 1..3 -> LDS (the rings are idle after the barrier), wave 0 adds them
  __syncthreads();
  float* red = reinterpret_cast<float*>(sSall);
  if (wave > 0) {
#pragma unroll
    for (int j = 0; j < NQ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) red[(((wave - 1) * NQ + j) * 16 + e) * 64 + lane] = acc[j][e];
  }
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int w = 0; w < NSPLIT - 1; ++w)
#pragma unroll
    for (int j = 0; j < NQ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[j][e] += red[((w * NQ + j) * 16 + e) * 64 + lane];

  const float s = ra.s[0][k];
  const int ldz = ra.ldz[0];
  bf16* __restrict__ Out = ra.Out[0];
  const int row = lo + l32;
  if (row < hi) {
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int q = 32 * j + 8 * g + 4 * lhi;
        if (q < ldz) {
          bf16x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = static_cast<bf16>((q + e < r) ? acc[j][4 * g + e] * s : 0.f);
          *(bf16x4*)(Out + (size_t)row * ldz + q) = o;
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// Gradient products whose contraction runs over the tokens of one task:
//   WIDE_FIRST = true : out_pk[c, q] (+)= sum_t Big[t, c] * Small_p[t, q]   (dA_k = x_k^T G,  out row stride r_k)
//   WIDE_FIRST = false: out_k[q, j]  (+)= sum_t Small[t, q] * Big[t, j]     (dB_k = Z^T dy_k, out row stride wide)
// Big is [T, wide] (X or dY), Small_p is [T, ldz_p] (G or Z, zero in columns >= r_pk).
// Block: one task, 128 columns of Big, all its tokens in tiles of 64; 4 waves x 32 columns.
// The whole reduction of an output element happens inside one block: deterministic, no atomics.
// ------------------------------------------------------------------------------------------
// LDS of one ring stage: 64 tokens x 128 columns of Big; 64 tokens x ldz of every Small_p, ldz <= 32 NQ, in
// NQ x 4 KiB each.  Lanes whose column lies beyond the tile sum what is not stored: they read another column or, with
// `pads`, the 64 zero bytes behind the tile.  The pads take a barrier before the first load, but the long tasks of one
// block per CU are faster with them (dB and dA, rank 128, 32768 x 4096, one task 142 us against 153, 16384 x 1024 -> 4096, 4
// tasks 63 against 68); short tasks and the smaller ranks are not (4 us launches 0.2 us longer).  The
// stages are separate arrays of the kernels (as members of one struct they cost the shared-input
// launch 10 us of 178).
constexpr int kBigStage = 64 * 128 * 2;
constexpr bool grad_pads(int nq, int np, int stages) { return nq == 4 && np == 1 && stages == 3; }
template <int NQ, int NP, int NS> constexpr int kSmallStage = NQ * 32 * 128 + (grad_pads(NQ, NP, NS) ? 1024 : 0);
// Three stages (two tiles in flight) where two blocks of them share a CU, and where a CU has no second block to
// run; two where that is what makes room for the second block (160 KiB of LDS).  us with three and with two stages: ranks above
// 64, dB and dA, 16384 x 4096 (32 tasks) 123 and 90, 8192 x 4096 (16) 63 and 45, 512 x 4096 (12) 25 and 20, but at
// most 256 blocks: 1024 x 64 (4 tasks) 10.4 and 11.9, 2048 x 1024 (16) 12.1 and 13.2, 16384 x 4096 (4) 73.8 and 75.1;
// dA of three projections that share X, ranks up to 64, 32768 x 5120 168 and 133.  Where two blocks of three
// stages fit, two stages lose: 16384 x 4096, ranks up to 64, 53 and 59.
template <int NQ, int NP>
constexpr int grad_stages() {
  constexpr int stage = kBigStage + NP * kSmallStage<NQ, NP, 2>, half = 80 * 1024;
  return 3 * stage > half && 2 * stage <= half ? 2 : 3;
}
#define MLORA_GRAD_STAGES(NQ, NP, NS)                                                                          \
  constexpr int kSmall = NP * kSmallStage<NQ, NP, NS>;                                                          \
  __shared__ __attribute__((aligned(1024))) char sB0[kBigStage], sB1[kBigStage], sS0[kSmall], sS1[kSmall],       \
      sB2[NS == 3 ? kBigStage : 1], sS2[NS == 3 ? kSmall : 1];                                                   \
  char* const sB[3] = {sB0, sB1, sB2};                                                                          \
  char* const sS[3] = {sS0, sS1, sS2}

template <bool WIDE_FIRST, int NQ, int NP, int NS>
__device__ __forceinline__ void grad_body(const GradArgs<NP>& ga, int bid, char* const (&sB)[3], char* const (&sS)[3]) {
  constexpr int WC = 128;
  constexpr int SREG = kSmallStage<NQ, NP, NS>, SBYTES = NQ * 32 * 128;
  constexpr bool PADS = grad_pads(NQ, NP, NS);
  static_assert(WIDE_FIRST || NP == 1, "shared-input form exists for dA only");

  const bf16* __restrict__ Big = ga.Big;
  const int wide = ga.wide;
  const int ch = bid % ga.chunks;
  const int sp = (bid / ga.chunks) % ga.splits;
  const int k = bid / (ga.chunks * ga.splits);
  const int col0 = ch * WC;
  int lo = ga.off[k], hi = ga.off[k + 1];
  if (ga.splits > 1) {
    // token range of this block: whole 64-token tiles, possibly empty (then zeros are written)
    const int len = ((hi - lo + ga.splits - 1) / ga.splits + 63) / 64 * 64;
    lo = lo + sp * len < hi ? lo + sp * len : hi;
    hi = lo + len < hi ? lo + len : hi;
  }
  const int tk = hi - lo;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

  if (PADS && tid < 16) {
#pragma unroll
    for (int s_ = 0; s_ < NS; ++s_) reinterpret_cast<int*>(sS[s_] + SBYTES)[tid] = 0;
  }

  // Big tile: 64 token rows x 256 B; wave instruction w covers rows 4w..4w+3
  int brow[4], bcol[4];
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int rl = 4 * (wave + 4 * it) + (lane >> 4);
    const int c = (lane & 15) ^ ((rl & 3) << 2);
    int col = col0 + c * 8;
    col = col < wide ? col : wide - 8;
    brow[it] = rl;
    bcol[it] = col;
  }
  // Small tiles: 64 tokens x ldz_p, contiguous in memory; piece = 1 KiB = 64 chunks of 16 B
  int ldz[NP], rank[NP];
  int srow[NP][NQ], scol[NP][NQ];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    ldz[p] = ga.ldz[p];
    rank[p] = ga.rank[p][k];
    const int cpr = ldz[p] / 8;  // chunks per token row = 1 KiB pieces per tile
#pragma unroll
    for (int it = 0; it < NQ; ++it) {
      // pieces beyond the tile re-fetch piece 0 into their own (never read) slot, so that every
      // wave issues the same number of loads per tile
      const int piece = (wave + 4 * it) < cpr ? (wave + 4 * it) : 0;
      const int src = swizzled_source(piece * 64 + lane, ldz[p]);
      srow[p][it] = src / ldz[p];
      scol[p][it] = src % ldz[p];
    }
  }
  constexpr int PER_TILE = 4 + NP * NQ;
  static_assert((NS - 2) * PER_TILE < 64, "vmcnt range");

  auto issue = [&](int kt, char* sb, char* ss) {
    const int t0 = lo + kt * 64;
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      // rows past the block's token range re-read its last row (they meet zeros of the masked
      // small operand): a block touches no row of another task, whatever that row holds
      int tok = t0 + brow[it];
      tok = tok < hi ? tok : hi - 1;
      load_lds_16B(Big + (size_t)tok * wide + bcol[it], sb + (wave + 4 * it) * 1024);
    }
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int it = 0; it < NQ; ++it) {
        int tok = t0 + srow[p][it];
        tok = tok < hi ? tok : hi - 1;
        load_lds_16B(ga.Small[p] + (size_t)tok * ldz[p] + scol[p][it], ss + p * SREG + (wave + 4 * it) * 1024);
      }
  };

  const int l32 = lane & 31, lhi = lane >> 5;
  const int L16 = lane & 15, blk = lane >> 4, kq = L16 >> 2;
  const int tr_k = 8 * (blk >> 1) + kq;
  const int tr_n = 16 * (blk & 1) + 4 * (L16 & 3);
  const int wide_n = 32 * wave + tr_n;
  const int wide_off = (((wide_n >> 3) ^ (kq << 2)) << 4) + (wide_n & 7) * 2;

  f32x16 acc[NP][NQ];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int j = 0; j < NQ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[p][j][e] = 0.f;

  // `valid` = number of tokens of this tile that belong to the task (64 except in the last tile)
  auto compute = [&](const char* sb, const char* ssall, int valid) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int kk = 16 * ks + tr_k;
      const bf16x8 wf = join(lds_read_tr(sb + kk * 256 + wide_off), lds_read_tr(sb + (kk + 4) * 256 + wide_off));
#pragma unroll
      for (int p = 0; p < NP; ++p) {
        const char* ss = ssall + p * SREG;
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
          if (32 * j < rank[p]) {
            const bool in = 32 * j + tr_n < ldz[p];
            const int n = in || PADS ? 32 * j + tr_n : 0;
            const int ns = n ^ (seg_swizzle(kk, ldz[p]) << 5);
            const char* p0 = ss + (in || !PADS ? (kk * ldz[p] + ns) * 2 : SBYTES);
            const char* p1 = ss + (in || !PADS ? ((kk + 4) * ldz[p] + ns) * 2 : SBYTES);
            short4v s0 = lds_read_tr(p0), s1 = lds_read_tr(p1);
            if (valid < 64) {
              // the lane's 8 contraction indices are tokens 16ks + 8*lhi + 0..7 of the tile
              const int tbase = 16 * ks + 8 * lhi;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                if (tbase + e >= valid) s0[e] = 0;
                if (tbase + 4 + e >= valid) s1[e] = 0;
              }
            }
            const bf16x8 sf = join(s0, s1);
            if (WIDE_FIRST)
              acc[p][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, sf, acc[p][j], 0, 0, 0);
            else
              acc[p][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sf, wf, acc[p][j], 0, 0, 0);
          }
        }
      }
    }
  };

  const int KT = (tk + 63) / 64;
  if (PADS) __syncthreads();
#pragma unroll
  for (int s_ = 0; s_ < NS - 1; ++s_)
    if (s_ < KT) issue(s_, sB[s_], sS[s_]);
  for (int kt0 = 0; kt0 < KT; kt0 += NS) {
#pragma unroll
    for (int s_ = 0; s_ < NS; ++s_) {
      const int kt = kt0 + s_;
      if (kt < KT) {
        if (kt + NS - 2 < KT)
          wait_vmcnt<(NS - 2) * PER_TILE>();
        else
          wait_vmcnt<0>();
        __builtin_amdgcn_s_barrier();
        if (kt + NS - 1 < KT) issue(kt + NS - 1, sB[(s_ + NS - 1) % NS], sS[(s_ + NS - 1) % NS]);
        const int left = tk - kt * 64;
        compute(sB[s_], sS[s_], left < 64 ? left : 64);
      }
    }
  }

  int accumulate = ga.accumulate;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    float* o = ga.out[p].p[k];
    const int r = ga.rank[p][k];
    if (NP == 1 && ga.splits > 1) {
      int rbase = 0;
      for (int kk = 0; kk < k; ++kk) rbase += ga.rank[0][kk];
      o = ga.part + sp * ga.part_step + (size_t)rbase * wide;
      accumulate = 0;
    }
    if (WIDE_FIRST) {
      // D[i = column c of Big][j = q]: lane holds q = 32j + l32 and c = col0 + 32*wave + 8g + 4*lhi + e
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        const int q = 32 * j + l32;
        if (q < r) {
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int c = col0 + 32 * wave + 8 * g + 4 * lhi + e;
              if (c < wide) {
                float* dst = o + (size_t)c * r + q;
                *dst = accumulate ? *dst + acc[p][j][4 * g + e] : acc[p][j][4 * g + e];
              }
            }
        }
      }
    } else {
      // D[i = q][j = column of Big]: lane holds column col0 + 32*wave + l32 and q = 32j + 8g + 4*lhi + e
      const int col = col0 + 32 * wave + l32;
      if (col < wide) {
#pragma unroll
        for (int j = 0; j < NQ; ++j)
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int q = 32 * j + 8 * g + 4 * lhi + e;
              if (q < r) {
                float* dst = o + (size_t)q * wide + col;
                *dst = accumulate ? *dst + acc[p][j][4 * g + e] : acc[p][j][4 * g + e];
              }
            }
      }
    }
  }
}

// dA of projections that share their input
template <int NQ, int NP>
__global__ __launch_bounds__(256) void k_grad_mfma(const GradArgs<NP> ga) {
  constexpr int NS = grad_stages<NQ, NP>();
  MLORA_GRAD_STAGES(NQ, NP, NS);
  grad_body<true, NQ, NP, NS>(ga, blockIdx.x, sB, sS);
}
// dB (the first blocks_b blocks: dY has just been read for G) and dA of one call
template <int NQ, int NS>
__global__ __launch_bounds__(256) void k_grad_pair(const GradArgs<1> b, const GradArgs<1> a, int blocks_b) {
  MLORA_GRAD_STAGES(NQ, 1, NS);
  if ((int)blockIdx.x < blocks_b) grad_body<false, NQ, 1, NS>(b, blockIdx.x, sB, sS);
  else grad_body<true, NQ, 1, NS>(a, blockIdx.x - blocks_b, sB, sS);
}

// Adds the token ranges' partial sums in range order (deterministic) into the tasks' outputs.  One
// thread per output element; a range holds the tasks' dB, then their dA (part_step elements in all).
struct ReduceArgs {
  const float* part;
  size_t part_step;
  int splits, wide_b, wide_a, rtotal, K, accumulate;
  unsigned char rank[kMaxK];
  OutTable out_b, out_a;
};
__global__ __launch_bounds__(256) void k_grad_reduce(const ReduceArgs a) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= a.part_step) return;
  float sum = 0.f;
#pragma unroll 4
  for (int s_ = 0; s_ < a.splits; ++s_) sum += a.part[s_ * a.part_step + e];
  const size_t nb = (size_t)a.rtotal * a.wide_b;
  const bool is_b = e < nb;
  const size_t g = is_b ? e : e - nb;
  const int wide = is_b ? a.wide_b : a.wide_a;
  // which task: element g lies in [rbase_k * wide, (rbase_k + r_k) * wide)
  size_t base = 0;
  int k = 0;
  for (; k < a.K; ++k) {
    const size_t n = (size_t)a.rank[k] * wide;
    if (g < base + n) break;
    base += n;
  }
  float* dst = (is_b ? a.out_b.p[k] : a.out_a.p[k]) + (g - base);
  *dst = a.accumulate ? *dst + sum : sum;
}

// Ring depth: three stages (two tiles in flight) keep a block at 75 KiB of LDS for ranks up to 64,
// so two blocks share a CU; measured 8 % faster than four stages with one block per CU.
constexpr int kRing = 3;

int nq_of(int ldz) { return ldz <= 32 ? 1 : (ldz <= 64 ? 2 : 4); }

int row_blocks(const SegTable& st, int tm) {
  int blocks = 0;
  for (int k = 0; k < st.K; ++k) blocks += (st.off[k + 1] - st.off[k] + tm - 1) / tm;
  return blocks;
}

// the largest row tile that still gives every CU (256) a block: at equal block counts the
// larger tile is faster (fewer fetches of the small operand per row)
int pick_row_tile(const SegTable& st) {
  int tm = 128;
  if (row_blocks(st, tm) < 256) tm = 64;
  if (tm == 64 && row_blocks(st, tm) < 256) tm = 32;
  return tm;
}

// Row tile and contraction ranges of one launch.  Ranges (fp32 sums in scratch, one more launch to add
// them) where the rows alone leave the chip short of loads in flight; powers of two, so that an XCD
// sees the same ranges of the small operand in every row block.  Measured, us, all launches of the
// product, one range -> as chosen here:
//   ranks above 64 (four column groups: the four-wave form of few rows does not fit the LDS):
//     3072 x 4096 (12 tasks)  s x A 85 -> 25, s dy B^T 56 -> 22;  8192 x 4096  62 -> 33, 56 -> 33
//     short tasks, both products, blocks of 128 rows -> of 32: 2048 x 2048 (64 tasks) 53 -> 41, 3000 x 3072 (60) 67 ->
//     48, 1000 x 4096 (40) 54 -> 41; with 1024 blocks at most 47, 54, 48; where the number of ranges stays the same
//     (200 x 2048, 10 tasks) 32.5 and 33.3
//   ranks up to 64:
//     16448 x 11008  119 -> 90,  16448 x 4096  44 -> 38-40,  12288 x 4096  31 -> 26
//     8192 x 4096, a forward and backward pass 474 -> 466 with two such products
//     2048 x 11008, operands from HBM  30 -> 22 (from the Infinity Cache 21 -> 19)
//   left alone: 32768 rows (64 against 70 with two ranges), fewer than 4096 rows of 4096 features (the
//   four-wave form takes less than two launches: 771 x 2048  9 against 12), and shallow contractions, whose
//   sums and their reduction weigh more than what the ranges bring.  Time of a forward call with 64 outputs
//   with one range over its time with ranges, rank 64, 16384 rows: 512 deep 0.84, 1024 0.86, 3072 0.98-1.0,
//   4096 1.02, 8192 0.96 (12288 rows: 0.88, 0.96, 1.01, 1.17, 1.10); rank 8, 16384 rows: 4096 and 5120 deep
//   0.92-0.96, 8192 1.02; rank 128: 512 deep 0.85-0.95, 1024 1.01-1.17 up to 12288 rows and 0.95 with 16384,
//   2048 1.05-1.4.  And tasks that leave a quarter of their blocks of 128 rows empty: 64 tasks of 64 rows, 4096
//   deep, rank 8  14.6 against 19.2 us.
struct RowsPlan {
  int tm, splits;
};
RowsPlan plan_rows(const SegTable& st, int inner, int ldz, size_t limit) {
  const RowsPlan plain{pick_row_tile(st), 1};
  const int KT = inner / 64, b128 = row_blocks(st, 128), b32 = row_blocks(st, 32);
  if (b128 == 0 || b128 >= 256) return plain;
  const long long rows = st.off[st.K] - st.off[0];
  RowsPlan pl = plain;
  if (nq_of(ldz) == 4) {
    if (KT < 16 || (KT < 32 && b128 >= 128)) return plain;
    auto ranges = [&](int blocks, int most) {
      int n = 1;
      while (2 * n * blocks <= most && 8 * n <= KT && n < 16) n *= 2;
      return n;
    };
    pl = RowsPlan{128, ranges(b128, 256)};
    // short tasks, whose 128-row blocks are mostly empty, in blocks of one wave where that makes room for
    // more ranges
    if (2 * rows <= 128LL * b128 && b32 <= 256 && ranges(b32, 512) > pl.splits) pl = RowsPlan{32, ranges(b32, 512)};
  } else if (b32 >= 128 && KT >= 64 && !(nq_of(ldz) == 1 && KT < 128 && b128 >= 128) && 4 * rows >= 3 * 128LL * b128) {
    pl = RowsPlan{128, KT >= 128 ? 8 : 4};
  } else if (b32 >= 32 && KT >= 128) {
    pl = RowsPlan{64, 8};
  } else if (b32 < 32 && KT > 64) {
    pl = RowsPlan{32, KT >= 128 ? 16 : 8};
  }
  const size_t one = (size_t)rows * ldz * sizeof(float);
  while (pl.splits > 1 && (one * pl.splits > limit || 4 * pl.splits > KT)) pl.splits /= 2;
  return pl.splits > 1 ? pl : plain;
}

// few rows: four waves per 32-row block, each on a quarter of the contraction
bool four_wave_form(int tm, int nq, int inner, int blocks) { return tm == 32 && nq <= 2 && inner >= 1024 && blocks <= 1024; }

// Algorithmic bytes of one launch: the tasks' rows of the big operand read once, the outputs
// written once, the small operands read once.
template <int NP>
double rows_bytes(const RowsArgs<NP>& a) {
  const double rows = a.K > 0 ? a.off[a.K] - a.off[0] : 0;
  double b = rows * a.inner * 2.0;
  for (int p = 0; p < NP; ++p) {
    b += rows * a.ldz[p] * 2.0;
    for (int k = 0; k < a.K; ++k) b += (double)a.rank[p][k] * a.inner * 2.0;
  }
  return b;
}

template <int NP>
double grad_bytes(const GradArgs<NP>& a) {
  const double rows = a.K > 0 ? a.off[a.K] - a.off[0] : 0;
  double b = rows * a.wide * 2.0;
  for (int p = 0; p < NP; ++p) {
    b += rows * a.ldz[p] * 2.0;
    for (int k = 0; k < a.K; ++k) b += (double)a.rank[p][k] * a.wide * 4.0;
  }
  return b;
}

// whether a k-major small operand needs the ragged form
template <int NP>
bool ragged_ranks(const RowsArgs<NP>& a) {
  for (int p = 0; p < NP; ++p)
    for (int k = 0; k < a.K; ++k)
      if (a.rank[p][k] % 8 != 0) return true;
  return false;
}

template <bool KMAJOR, int NQ, int TM, int NP>
hipError_t launch_rows_one(const RowsArgs<NP>& a, int blocks, hipStream_t s) {
  if constexpr (NP * NQ <= 8) {
    const int slot = profile_begin(kProfileRows, rows_bytes(a), s);
    bool rag = false;
    if constexpr (KMAJOR) {
      rag = ragged_ranks(a);
      if (rag) hipLaunchKernelGGL((k_lowrank_mfma<true, NQ, kRing, TM, NP, true>), dim3(blocks), dim3(TM * 2), 0, s, a);
    }
    if (!rag) hipLaunchKernelGGL((k_lowrank_mfma<KMAJOR, NQ, kRing, TM, NP, false>), dim3(blocks), dim3(TM * 2), 0, s, a);
    const hipError_t e = hipGetLastError();
    profile_end(slot, s);
    return e;
  } else {
    return hipErrorInvalidValue;
  }
}

template <bool KMAJOR, int NQ, int NP>
hipError_t launch_rows_tm(const RowsArgs<NP>& a, int tm, int blocks, hipStream_t s) {
  if (tm == 128) return launch_rows_one<KMAJOR, NQ, 128, NP>(a, blocks, s);
  if (tm == 64) return launch_rows_one<KMAJOR, NQ, 64, NP>(a, blocks, s);
  return launch_rows_one<KMAJOR, NQ, 32, NP>(a, blocks, s);
}

template <bool KMAJOR, int NQ>
hipError_t launch_rows_splitk(const RowsArgs<1>& a, int blocks, hipStream_t s) {
  const int slot = profile_begin(kProfileRows, rows_bytes(a), s);
  bool rag = false;
  if constexpr (KMAJOR) {
    rag = ragged_ranks(a);
    if (rag) hipLaunchKernelGGL((k_lowrank_mfma_splitk<true, NQ, kRing, true>), dim3(blocks), dim3(256), 0, s, a);
  }
  if (!rag) hipLaunchKernelGGL((k_lowrank_mfma_splitk<KMAJOR, NQ, kRing, false>), dim3(blocks), dim3(256), 0, s, a);
  const hipError_t e = hipGetLastError();
  profile_end(slot, s);
  return e;
}

template <bool KMAJOR, int NP>
hipError_t launch_rows(const RowsArgs<NP>& a, int nq, int tm, int blocks, hipStream_t s) {
  if constexpr (NP == 1) {
    if (a.splits > 1) {
      hipError_t e = nq == 1 ? launch_rows_tm<KMAJOR, 1, 1>(a, tm, blocks, s)
                             : (nq == 2 ? launch_rows_tm<KMAJOR, 2, 1>(a, tm, blocks, s) : launch_rows_tm<KMAJOR, 4, 1>(a, tm, blocks, s));
      if (e != hipSuccess) return e;
      const long long n = (long long)(a.off[a.K] - a.off[0]) * (a.ldz[0] / 4);
      const int slot = profile_begin(kProfileRows, 0.0, s);   // its time counts, it adds no algorithmic bytes
      hipLaunchKernelGGL(k_rows_reduce, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
      e = hipGetLastError();
      profile_end(slot, s);
      return e;
    }
    if (four_wave_form(tm, nq, a.inner, blocks)) {
      return nq == 1 ? launch_rows_splitk<KMAJOR, 1>(a, blocks, s) : launch_rows_splitk<KMAJOR, 2>(a, blocks, s);
    }
  }
  if (nq == 1) return launch_rows_tm<KMAJOR, 1, NP>(a, tm, blocks, s);
  if (nq == 2) return launch_rows_tm<KMAJOR, 2, NP>(a, tm, blocks, s);
  return launch_rows_tm<KMAJOR, 4, NP>(a, tm, blocks, s);
}

template <int NQ, int NP>
hipError_t launch_grad_one(const GradArgs<NP>& a, int blocks, hipStream_t s) {
  if constexpr (NP * NQ <= 8) {
    const int slot = profile_begin(kProfileGrad, grad_bytes(a), s);
    hipLaunchKernelGGL((k_grad_mfma<NQ, NP>), dim3(blocks), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    profile_end(slot, s);
    return e;
  } else {
    return hipErrorInvalidValue;
  }
}

template <int NP>
hipError_t launch_grad(const GradArgs<NP>& a, int nq, int blocks, hipStream_t s) {
  if (nq == 1) return launch_grad_one<1, NP>(a, blocks, s);
  if (nq == 2) return launch_grad_one<2, NP>(a, blocks, s);
  return launch_grad_one<4, NP>(a, blocks, s);
}

template <int NP>
hipError_t rows_group(const LowrankGroupItem* it, const SegTable& st, const bf16* In, int inner, int nq, hipStream_t s) {
  RowsArgs<NP> a;
  a.In = In;
  a.inner = inner;
  a.K = st.K;
  for (int k = 0; k <= kMaxK; ++k) a.off[k] = st.off[k];
  for (int p = 0; p < NP; ++p) {
    a.Out[p] = it[p].rows_out;
    a.ldz[p] = it[p].ldz;
    for (int k = 0; k < kMaxK; ++k) {
      a.rank[p][k] = (unsigned char)(k < st.K ? it[p].rank[k] : 0);
      a.s[p][k] = k < st.K ? it[p].s[k] : 0.f;
    }
    a.M[p] = *it[p].M;
  }
  a.splits = 1;
  a.part = nullptr;
  const int tm = pick_row_tile(st);
  const int blocks = row_blocks(st, tm);
  if (blocks == 0) return hipSuccess;
  return launch_rows<true, NP>(a, nq, tm, blocks, s);
}

template <int NP>
hipError_t grad_group(const LowrankGroupItem* it, const SegTable& st, const bf16* Big, int wide, int T, int nq,
                      int accumulate, hipStream_t s) {
  GradArgs<NP> a;
  a.Big = Big;
  a.wide = wide;
  a.T = T;
  a.K = st.K;
  for (int k = 0; k <= kMaxK; ++k) a.off[k] = st.off[k];
  for (int p = 0; p < NP; ++p) {
    a.Small[p] = it[p].grad_small;
    a.ldz[p] = it[p].ldz;
    for (int k = 0; k < kMaxK; ++k) a.rank[p][k] = (unsigned char)(k < st.K ? it[p].rank[k] : 0);
    a.out[p] = *it[p].grad_out;
  }
  a.accumulate = accumulate;
  a.chunks = (wide + 127) / 128;
  a.splits = 1;
  a.part_step = 0;
  a.part = nullptr;
  return launch_grad<NP>(a, nq, st.K * a.chunks, s);
}

}  // namespace

// plan_rows cuts fewer than 256 blocks of 128 rows into at most KT / 4 ranges: up to 8, up to 16 of fewer than 32 blocks of
// 32 rows, or (ranks above 64) up to 16 as long as there are no more than 256 blocks of 128 rows or 512 of 32, which is half
// as many rows
size_t rows_partial_bytes(int T, int inner, int ldz) {
  const bool four = nq_of(ldz) == 4;
  const int KT = inner / 64;
  auto sums = [&](long long rows, int most) {
    const int splits = KT / 4 < most ? KT / 4 : most;
    return splits > 1 ? (rows < T ? rows : (long long)T) * splits : 0;
  };
  constexpr long long block_rows = 256 * 128;
  const long long many = sums(block_rows, four ? 16 : 8), few = four ? 0 : sums(31 * 32, 16);
  const long long most = four && many > block_rows ? block_rows : (many > few ? many : few);
  return align_up((size_t)most * ldz * sizeof(float), 256);
}

RowsForm rows_form(const SegTable& st, int inner, int ldz, size_t limit) {
  const RowsPlan pl = plan_rows(st, inner, ldz, limit);
  return RowsForm{pl.tm, pl.splits};
}

// A_k's tile of a rank above 64 that is no multiple of 4 is read element by element (2.7 us a contraction tile): where
// the rows fill few blocks, the general kernel, which puts such columns together in registers, is faster: 219 x 1920 (10
// tasks, ranks up to 114) 27.3 -> 9.2 us, 4458 x 640 (43 tasks, up to 123) 27.4 -> 9.8, 6251 x 448 (2 tasks, up to 96) 13.7 ->
// 5.8.  Blocks that read more than 512 KB, and a single or few contraction tiles, stay (3072 x 4096, 12 tasks, up to 128: 21.8).
bool general_rows_pay(const CallCtx& c) {
  if (nq_of(c.ldz) != 4 || c.h < 256) return false;
  bool odd = false;
  for (int k = 0; k < c.K; ++k) odd = odd || c.st.rank[k] % 4 != 0;
  if (!odd) return false;
  const RowsPlan pl = plan_rows(c.st, c.h, c.ldz, c.scratch_bytes);
  if (pl.tm == 32 && pl.splits > 1) return false;   // (short tasks in blocks of one wave and ranges)
  const double blocks = (double)row_blocks(c.st, pl.tm) * pl.splits, rounds = blocks <= 256 ? 1.0 : blocks / 256;
  const double us = 4.0 + rounds * 2.7 * (c.h / 64) / pl.splits + (pl.splits > 1 ? 4.5 : 0.0);
  double bytes;
  return general_rows_us(c, c.h, &bytes) < 0.7 * us && bytes <= 512 << 10;
}

// Z = s x A (a_major = true, M = A_k) or G = s dy B^T (a_major = false, M = B_k).
hipError_t lowrank_rows_mfma(const CallCtx& c, const bf16* In, int inner, bf16* Out, const PtrTable& M,
                             bool a_major, float* partial, size_t limit) {
  const RowsPlan pl = plan_rows(c.st, inner, c.ldz, limit);
  const int tm = pl.tm, blocks = row_blocks(c.st, tm) * pl.splits;
  if (blocks == 0) return hipSuccess;
  RowsArgs<1> a;
  a.splits = pl.splits;
  a.part = partial;
  a.In = In;
  a.inner = inner;
  a.K = c.st.K;
  for (int k = 0; k <= kMaxK; ++k) a.off[k] = c.st.off[k];
  a.Out[0] = Out;
  a.ldz[0] = c.ldz;
  for (int k = 0; k < kMaxK; ++k) {
    a.rank[0][k] = (unsigned char)c.st.rank[k];
    a.s[0][k] = c.st.s[k];
  }
  a.M[0] = M;
  const int nq = nq_of(c.ldz);
  return a_major ? launch_rows<true, 1>(a, nq, tm, blocks, c.stream) : launch_rows<false, 1>(a, nq, tm, blocks, c.stream);
}

// Token ranges per task of up to `longest` tokens for the gradient kernels, one number for dB and dA: as many
// as give every CU a block (at most 16, at least 256 tokens each).  More cost their reduction more than they
// bring: 6000 tokens of 4 tasks, 4096 x 4096, rank 64, forward + backward 423 us with two blocks per CU, 411
// us with one.  Ranks above 64: no more than 256 in all, each with a CU to itself (65536 tokens of one task, 1024 ->
// 4096, rank 128, backward 843 us with 280 blocks of three stages, 753 with 240).  Up to 512 blocks, two on a CU with two
// stages, would suit few long tasks and hurt others, sums included, rank 128 unless stated: 16384 x 5120 (2 tasks) 129 -> 88 us,
// 32768 x 1024 -> 4096 (4) 129 -> 95, 8192 x 5120 (2, rank 72) 62 -> 43, but 8192 x 1024 (12) 21 -> 40, 4096 x 1024 -> 4096 (4) 24
// -> 33, 8192 x 4096 (4, rank 72) 36 -> 42: that takes a rule of its own.
int grad_ranges(const SegTable& st, int wide_b, int wide_a, int longest) {
  const int blocks = st.K * ((wide_b + 127) / 128 + (wide_a + 127) / 128);
  int rmax = 0;
  for (int k = 0; k < st.K; ++k) rmax = st.rank[k] > rmax ? st.rank[k] : rmax;
  int s = (256 + (rmax > 64 ? 0 : blocks - 1)) / blocks;
  s = s < 16 ? s : 16;
  s = s < longest / 256 ? s : longest / 256;
  return s > 1 ? s : 1;
}
// ... as far as their partial sums stay within `limit` bytes
int grad_splits(const SegTable& st, int wide_b, int wide_a, size_t limit) {
  int s = grad_ranges(st, wide_b, wide_a, longest_task(st));
  while (s > 1 && grad_sum_bytes(st, s, wide_b, wide_a) > limit) --s;
  return s;
}

size_t grad_partial_bytes(const SegTable& st, int T, int wide_b, int wide_a) {
  const int s = grad_ranges(st, wide_b, wide_a, T);
  return s > 1 ? grad_sum_bytes(st, s, wide_b, wide_a) : 0;
}

// What the size queries reserve for one gradient of `wide` columns whatever the launch plan: sums of the
// ranges that would give every CU two blocks.
size_t grad_reserve_bytes(const SegTable& st, int wide) {
  const int blocks = st.K * ((wide + 127) / 128);
  if (st.K == 0 || blocks >= 384) return 0;
  const int longest = longest_task(st);
  int s = (512 + blocks - 1) / blocks;
  s = s < 16 ? s : 16;
  s = s < longest / 256 ? s : longest / 256;
  return s > 1 ? grad_sum_bytes(st, s, wide, 0) : 0;
}

// dB_k = Z^T dy_k and, unless dA is NULL, dA_k = x_k^T G, in one launch (and one that adds the token
// ranges where there are several): two launches each before, which cost few tokens 10 us of 108
// (771 tokens, 2048 -> 5632) and 8192 tokens of 4096 features 40 us instead of 33.
hipError_t grads_mfma(const CallCtx& c, const bf16* dY, const bf16* Z, const OutTable& dB, const bf16* X, const bf16* G,
                      const OutTable* dA, int accumulate, float* partial, size_t limit) {
  if (c.K == 0) return hipSuccess;
  const int wide_b = c.d, wide_a = dA != nullptr ? c.h : 0;
  // (planned for both outputs: dB's bits are the same whether or not a group computes dA elsewhere)
  const int splits = grad_splits(c.st, wide_b, c.h, limit);
  size_t rtotal = 0;
  for (int k = 0; k < c.K; ++k) rtotal += c.st.rank[k];
  GradArgs<1> b, a;
  auto fill = [&](GradArgs<1>& g, const bf16* big, int wide, const bf16* small, const OutTable& out, float* part) {
    g.Big = big;
    g.wide = wide;
    g.T = c.T;
    g.K = c.st.K;
    for (int k = 0; k <= kMaxK; ++k) g.off[k] = c.st.off[k];
    g.Small[0] = small;
    g.ldz[0] = c.ldz;
    for (int k = 0; k < kMaxK; ++k) g.rank[0][k] = (unsigned char)c.st.rank[k];
    g.out[0] = out;
    g.accumulate = accumulate;
    g.chunks = (wide + 127) / 128;
    g.splits = splits;
    g.part_step = rtotal * ((size_t)wide_b + wide_a);
    g.part = part;
    return c.K * g.chunks * splits;
  };
  const int blocks_b = fill(b, dY, wide_b, Z, dB, partial);
  const int blocks_a = dA != nullptr ? fill(a, X, wide_a, G, *dA, partial + rtotal * wide_b) : (a = b, 0);
  const int nq = nq_of(c.ldz);
  const int slot = profile_begin(kProfileGrad, grad_bytes(b) + (dA != nullptr ? grad_bytes(a) : 0.0), c.stream);
  const dim3 grid((unsigned)(blocks_b + blocks_a));
  if (nq == 1) hipLaunchKernelGGL((k_grad_pair<1, grad_stages<1, 1>()>), grid, dim3(256), 0, c.stream, b, a, blocks_b);
  else if (nq == 2) hipLaunchKernelGGL((k_grad_pair<2, grad_stages<2, 1>()>), grid, dim3(256), 0, c.stream, b, a, blocks_b);
  else if (grid.x > 256) hipLaunchKernelGGL((k_grad_pair<4, grad_stages<4, 1>()>), grid, dim3(256), 0, c.stream, b, a, blocks_b);
  else hipLaunchKernelGGL((k_grad_pair<4, 3>), grid, dim3(256), 0, c.stream, b, a, blocks_b);   // (see grad_stages)
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && splits > 1)
    e = grad_reduce(c.st, partial, splits, wide_b, dB, wide_a, dA != nullptr ? *dA : dB, accumulate, c.stream);
  profile_end(slot, c.stream);
  return e;
}

hipError_t grad_reduce(const SegTable& st, const float* partial, int splits, int wide_b, const OutTable& dB, int wide_a,
                       const OutTable& dA, int accumulate, hipStream_t stream) {
  ReduceArgs r;
  r.part = partial;
  r.splits = splits;
  r.rtotal = 0;
  for (int k = 0; k < st.K; ++k) r.rtotal += st.rank[k];
  r.wide_b = wide_b;
  r.wide_a = wide_a;
  r.part_step = (size_t)r.rtotal * ((size_t)wide_b + wide_a);
  r.K = st.K;
  r.accumulate = accumulate;
  for (int k = 0; k < kMaxK; ++k) r.rank[k] = (unsigned char)st.rank[k];
  r.out_b = dB;
  r.out_a = dA;
  hipLaunchKernelGGL(k_grad_reduce, dim3((unsigned)((r.part_step + 255) / 256)), dim3(256), 0, stream, r);
  return hipGetLastError();
}

// Whether np projections whose widest low-rank row stride is max_ldz fit the shared-input kernels
// (accumulators: np x ceil(max_ldz / 32) MFMA column groups, at most 8).
bool lowrank_group_ok(int np, int max_ldz) { return np >= 2 && np <= 4 && np * nq_of(max_ldz) <= 8; }

// Below these sizes the shared pass leaves the chip idle, while a launch per projection has as many blocks
// as projections, and deep contractions in ranges.  Whole group calls, time with a launch each over time
// with one pass:
//   rows, P = 3, 1024 | 4096 features, tokens   2048         8192         12288        16384
//     ranks up to 32                           0.97 | 0.91  1.00 | 0.99  1.10 | 1.02  1.08 | 1.03
//     ranks up to 64                           0.93 | 0.83  0.95 | 0.95  0.90 | 0.92  1.06 | 1.01
//   (32768 tokens of 5120: the pass 120 us, a launch 64 each); P = 4, 512 features 1.04-1.13 from 2048 to
//   16384 tokens, but 0.88-0.92 at 12288 tokens of rank 64
//   gradients, 4096 features: 4 tasks 0.94-1.0 up to 24576 tokens, 1 task 0.83-0.91, 16 tasks 1.0
// The pass is taken only where a launch of the projection's own would add in the same order, so that a
// group's Z and Y have the bits of the single calls.
bool group_rows_pay(const SegTable& st, int h, int ldz, size_t limit) {
  const RowsPlan pl = plan_rows(st, h, ldz, limit);
  if (pl.splits > 1 || four_wave_form(pl.tm, nq_of(ldz), h, row_blocks(st, pl.tm))) return false;
  return h <= 512 || row_blocks(st, 128) >= 128;
}
bool group_grads_pay(const SegTable& st, int h) { return st.K * ((h + 127) / 128) >= 256; }

// Z_p = s_pk x_k A_pk for np projections in one pass over X.
hipError_t lowrank_rows_mfma_group(int np, const LowrankGroupItem* items, const SegTable& st, const bf16* X, int h,
                                   hipStream_t stream) {
  int mx = 0;
  for (int p = 0; p < np; ++p) mx = items[p].ldz > mx ? items[p].ldz : mx;
  if (!lowrank_group_ok(np, mx)) return hipErrorInvalidValue;
  const int nq = nq_of(mx);
  if (np == 2) return rows_group<2>(items, st, X, h, nq, stream);
  if (np == 3) return rows_group<3>(items, st, X, h, nq, stream);
  return rows_group<4>(items, st, X, h, nq, stream);
}

// dA_pk = x_k^T G_p for np projections in one pass over X.
hipError_t grad_mfma_group(int np, const LowrankGroupItem* items, const SegTable& st, const bf16* X, int h, int T,
                           int accumulate, hipStream_t stream) {
  if (st.K == 0) return hipSuccess;
  int mx = 0;
  for (int p = 0; p < np; ++p) mx = items[p].ldz > mx ? items[p].ldz : mx;
  if (!lowrank_group_ok(np, mx)) return hipErrorInvalidValue;
  const int nq = nq_of(mx);
  if (np == 2) return grad_group<2>(items, st, X, h, T, nq, accumulate, stream);
  if (np == 3) return grad_group<3>(items, st, X, h, T, nq, accumulate, stream);
  return grad_group<4>(items, st, X, h, T, nq, accumulate, stream);
}

}  // namespace mlora
