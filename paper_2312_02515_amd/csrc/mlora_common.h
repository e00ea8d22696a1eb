// Shared declarations of the HIP side of libmlora (gfx950 only).
// Notation follows section 3.3.1 of the mLoRA paper: X [T,h], W [h,d], A_k [h,r_k],
// B_k [r_k,d]; task k owns rows [off[k], off[k+1]) of X, Y, dY and dX.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/mlora.h"

namespace mlora {

constexpr int kMaxK = MLORA_MAX_ADAPTERS;
constexpr int kMaxRank = MLORA_MAX_RANK;

typedef __bf16 bf16;

// Split positions, ranks and scalings of one call, passed to kernels by value
// (they land in the kernel-argument segment and are read with scalar loads).
struct SegTable {
  int K;
  int off[kMaxK + 1];
  int rank[kMaxK];
  float s[kMaxK];
};

struct PtrTable {
  const void* p[kMaxK];
};

struct OutTable {
  float* p[kMaxK];
};

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(bf16 v) { return static_cast<float>(v); }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
// fp32 -> bf16, round to nearest even, NaN/Inf propagate
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float v) { return static_cast<bf16>(v); }

// Row stride (in elements) of the saved intermediate Z and of G: the largest rank
// rounded up to a multiple of 16, so that rank-padded MFMA steps read zeros.
inline int lowrank_ld(const mlora_problem* p) {
  int rmax = 0;
  for (int k = 0; k < p->K; ++k) rmax = p->ranks[k] > rmax ? p->ranks[k] : rmax;
  return (rmax + 15) / 16 * 16;
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Rows of the virtual axis that the base products tile: every row range of the call (before the first
// task, each task, after the last) rounded up to whole 32-row pieces; and the most of T rows in K + 2 ranges.
inline long long virtual_rows(const SegTable& st, int M) {
  long long mv = 0;
  int prev = 0;
  for (int r = 0; r < st.K + 2; ++r) {
    const int b1 = r <= st.K ? st.off[r] : M;
    mv += (b1 - prev + 31) / 32 * 32;
    prev = b1;
  }
  return mv;
}
// Whether the pieces of 32 rows are packed instead: rows of several tasks in one piece, whose LoRA terms are added
// task by task and row by row.  Taken where the padding makes a quarter more rows (tasks of few rows).
inline bool packed_rows(const SegTable& st, int M) { return 4 * virtual_rows(st, M) > 5LL * M && M > 32; }
inline long long most_virtual_rows(int K, int T) {
  const long long padded = (long long)T + 31LL * (K + 2), apart = 32LL * T;
  return padded < apart ? padded : apart;
}

// tokens of the longest task
inline int longest_task(const SegTable& st) {
  int n = 0;
  for (int k = 0; k < st.K; ++k) n = st.off[k + 1] - st.off[k] > n ? st.off[k + 1] - st.off[k] : n;
  return n;
}
// partial sums of the gradients over `ranges` token ranges
inline size_t grad_sum_bytes(const SegTable& st, int ranges, int wide_b, int wide_a) {
  size_t rtotal = 0;
  for (int k = 0; k < st.K; ++k) rtotal += st.rank[k];
  return align_up((size_t)ranges * rtotal * ((size_t)wide_b + wide_a) * sizeof(float), 256);
}

// How a base product is cut up: MLORA_FORM_* (mlora_testing.h), contraction ranges per tile, and of the tiles of
// that form how many run as such
struct GemmForm {
  int form, parts;
  int whole, tiles;
  int rows;           // rows of the smallest tiles
};
// ... and a low-rank product: rows per block, contraction ranges
struct RowsForm {
  int rows, parts;
};

// Everything the launchers need, filled once per call from the validated problem.
struct CallCtx {
  int T, h, d, K, ldz;
  int dtype;
  SegTable st;
  PtrTable A, B;
  size_t scratch_bytes;   // behind the low-rank intermediates in the workspace
  hipStream_t stream;
};

// ---- launchers (each returns a hipError_t; all work goes to c.stream) ----
// general_mfma.hip : any shape, rank and alignment, fp32 or bf16 storage
// Launches that cut a contraction into ranges are planned within the `scratch_bytes` (`limit`) bytes at
// `scratch` (`partial`) that they are given; 0 = none does.  The size functions give the most that T
// rows or fewer use, whatever their split positions.
size_t general_scratch_bytes(const SegTable& st, int T, int h, int d, int dtype);
size_t general_grad_bytes(const SegTable& st, int T, int h, int d);     // the gradients' share of it
size_t general_dx_bytes(int K, int T, int h, int d, int dtype);         // the input gradient's
hipError_t general_Z(const CallCtx& c, const void* X, void* Z, float* scratch);      // Z = s x A
hipError_t general_G(const CallCtx& c, const void* dY, void* G, float* scratch);     // G = s dy B^T
// One operand pair of a base product: A [M, Kd], W [Kd, N] (nn) or [N, Kd], L [M, ldz] with
// R_k [rank[k], N] (nn) or [N, rank[k]].
struct GenOperands {
  const void* A;
  const void* W;
  const void* L;
  int Kd, ldz;
  const int* rank;     // K entries
  const PtrTable* R;
};
// whether the product runs in 16 x 64 tiles there (`Kd` over all operand pairs)
bool general_skinny(const SegTable& st, int M, int N, long long Kd, int dtype);
// (the form of a sum over n operand pairs of Kd[g] contraction indices and rank[g][k])
GemmForm general_gemm_form(const SegTable& st, int M, int N, int n, const int* Kd, const int* const* rank, bool nn, int dtype,
                           size_t scratch_bytes);
double general_rows_us(const CallCtx& c, int inner, double* block_bytes);
RowsForm general_rows_form(const CallCtx& c, int inner);
int general_grad_ranges(const CallCtx& c);
double general_skinny_us(const SegTable& st, int M, int N, long long Kd, int dtype);
// C = sum over the n <= MLORA_MAX_GROUP operand pairs of A op(W) + rows_k(L R_k)
hipError_t general_gemm(int n, const GenOperands* ops, int dtype, void* C, int M, int N, bool nn, const SegTable& st,
                        float* scratch, size_t scratch_bytes, hipStream_t stream);
// dB_k = Z^T dy_k and, unless dA is NULL, dA_k = x_k^T G, in `ranges` token ranges (0: as many as suit the launch alone)
hipError_t general_grads(const CallCtx& c, const void* dY, const void* Z, const OutTable& dB, const void* X, const void* G,
                         const OutTable* dA, int accumulate, int ranges, float* scratch);

// ... of a group's projections (same tasks and X), in `ranges` >= 1
struct GradItem {
  const CallCtx* c;
  const void *dY, *Z, *X, *G;
  const OutTable *dB, *dA;
  int ranges;
};
hipError_t general_grads_group(int n, const GradItem* items, int accumulate, float* scratch, size_t scratch_bytes);

// Small backward calls: dX (as in general_gemm, one operand pair; `aligned`: in the forms of gemm_mfma), dA_k and dB_k in
// one launch, and one each for ranges to add.
constexpr long long kMostShared = 4 << 20;   // activation elements (X and dY) of such a call
struct BackPlan {
  bool shared;        // whether a call of these sizes runs so
  int ranges;         // token ranges of the gradients (0: not shared)
  size_t left;        // scratch for the product's ranges, behind the gradients' sums
};
BackPlan plan_back(const CallCtx& c, bool aligned);
// hipErrorNotSupported, with nothing launched: buffers whose alignment takes dX to another form than the plan's
hipError_t general_back(const CallCtx& c, const BackPlan& bp, bool aligned, const void* X, const void* W, const void* dY, const void* Z, const void* G,
                        void* dX, const OutTable& dA, const OutTable& dB, int accumulate, float* scratch);

// gemm_mfma.hip : bf16 MFMA GEMM with the LoRA term as extra contraction steps
bool gemm_mfma_ok(int M, int N, int Kd);
hipError_t gemm_mfma(const bf16* A, const bf16* Bm, bf16* C, int M, int N, int Kd, bool nn, const bf16* L, int ldz,
                     const SegTable& st, const PtrTable& R, float* scratch, size_t scratch_bytes, hipStream_t stream);
size_t gemm_partial_bytes(int K, int T, int N, int Kd);
GemmForm gemm_form(const SegTable& st, int M, int N, int n, const int* Kd, bool nn, size_t scratch_bytes);

// One operand pair of a summed contraction (the input gradient of projections that share X):
// A [M, Kd], Bm [N, Kd], L [M, ldz] with R_k [N, rank[k]].
struct GemmOperands {
  const bf16* A;
  const bf16* Bm;
  const bf16* L;
  int Kd, ldz;
  const int* rank;     // K entries
  const PtrTable* R;
};
hipError_t gemm_mfma_sum_nt(int n, const GemmOperands* ops, bf16* C, int M, int N, const SegTable& st, float* scratch,
                            size_t scratch_bytes, hipStream_t stream);

// profile.hip : optional HIP-event timing of the MFMA kernels' launches, by kind
enum { kProfileGemm = 0, kProfileRows = 1, kProfileGrad = 2, kProfileKinds = 3 };
int profile_enable(int enable);
int profile_begin(int kind, double units, hipStream_t stream);
void profile_end(int slot, hipStream_t stream);
// flops of a product with its LoRA terms, from a kernel's arguments
template <typename Args>
double product_work(const Args& a) {
  double f = 0;
  for (int g = 0; g < (int)(sizeof(a.Kd) / sizeof(a.Kd[0])); ++g) {
    f += 2.0 * a.M * (double)a.N * a.Kd[g];
    for (int k = 0; k < a.K; ++k) f += 2.0 * (a.off[k + 1] - a.off[k]) * (double)a.rank[g][k] * a.N;
  }
  return f;
}
struct Profiled {      // the launches of a scope
  const int slot;
  const hipStream_t stream;
  Profiled(int kind, double units, hipStream_t s) : slot(profile_begin(kind, units, s)), stream(s) {}
  ~Profiled() { profile_end(slot, stream); }
  Profiled(const Profiled&) = delete;
  Profiled& operator=(const Profiled&) = delete;
};
hipError_t profile_read(double* ms, double* units, int* launches);

// w8_kernels.hip : column-wise absmax code of the frozen weight and its decoder
hipError_t w8_quantize(const void* W, int dtype, int h, int d, int8_t* Wq, float* c, hipStream_t stream);
hipError_t w8_dequantize(const int8_t* Wq, const float* c, int dtype, int h, int d, void* Wh, hipStream_t stream);

// lowrank_mfma.hip : bf16 MFMA kernels for Z, G (row-local) and dA_k, dB_k (reduce over a task's tokens)
size_t rows_partial_bytes(int T, int inner, int ldz);
RowsForm rows_form(const SegTable& st, int inner, int ldz, size_t limit);
// whether Z = s x A is faster in the general kernel
bool general_rows_pay(const CallCtx& c);
int grad_splits(const SegTable& st, int wide_b, int wide_a, size_t limit);
hipError_t lowrank_rows_mfma(const CallCtx& c, const bf16* In, int inner, bf16* Out, const PtrTable& M, bool a_major,
                             float* partial, size_t limit);
// Gradients dB (wide_b = d columns) and dA (wide_a = h columns) of one call.
size_t grad_partial_bytes(const SegTable& st, int T, int wide_b, int wide_a);
size_t grad_reserve_bytes(const SegTable& st, int wide);
hipError_t grads_mfma(const CallCtx& c, const bf16* dY, const bf16* Z, const OutTable& dB, const bf16* X, const bf16* G,
                      const OutTable* dA, int accumulate, float* partial, size_t limit);
// adds `splits` ranges of partial sums ([range][sum of ranks][wide_b], then [sum of ranks][wide_a]) in
// order into the tasks' outputs
hipError_t grad_reduce(const SegTable& st, const float* partial, int splits, int wide_b, const OutTable& dB, int wide_a,
                       const OutTable& dA, int accumulate, hipStream_t stream);

// One projection of a group that shares its input, for the two shared-input kernels:
// rows: Z_p = s_pk x_k A_pk (M = A_pk, output rows_out [T, ldz]); grad: dA_pk = x_k^T G_p
// (grad_small = G_p [T, ldz], output table grad_out).
struct LowrankGroupItem {
  int ldz;
  const int* rank;      // K entries
  const float* s;       // K entries
  const PtrTable* M;
  bf16* rows_out;
  const bf16* grad_small;
  const OutTable* grad_out;
};
bool lowrank_group_ok(int np, int max_ldz);
// whether one pass over X for all projections beats a launch per projection at these sizes
bool group_rows_pay(const SegTable& st, int h, int ldz, size_t limit);   // (asked for every projection)
bool group_grads_pay(const SegTable& st, int h);
hipError_t lowrank_rows_mfma_group(int np, const LowrankGroupItem* items, const SegTable& st, const bf16* X, int h,
                                   hipStream_t stream);
hipError_t grad_mfma_group(int np, const LowrankGroupItem* items, const SegTable& st, const bf16* X, int h, int T,
                           int accumulate, hipStream_t stream);

}  // namespace mlora
