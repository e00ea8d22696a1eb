// 8-bit frozen base weight (the single-GPU setup of section 4.1 keeps the pre-trained weights
// in 8 bits): column-wise absmax code of W [h, d],
//     c_j = max_i |W[i, j]| / 127,   Wq[i, j] = rint(W[i, j] / c_j),   W^[i, j] = Wq[i, j] c_j.
// Streaming kernels: the coder (run once when a model is loaded) and the decoder that the
// w8 entry points run in front of the base products (1 byte read and one element written per
// weight: 1 % of the product it feeds at 32768 tokens, a seventh at 2048).  Decoding inside the product was
// not tried: every row tile would decode the weight again, in the inner loop and without the direct
// global-to-LDS loads.
#include "mlora_common.h"

namespace mlora {
namespace {

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef unsigned u32x4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));

// The code is an integer decided by floating point: the maximum is exact, both divisions are IEEE
// fp32 divisions and rintf rounds halves to even, so the result is defined bit for bit and does not
// depend on how the rows are split over blocks.
//
// Coder in three launches, each a stream over W in pieces of VEC columns (16 bytes where alignment
// allows) by blocks of 64 column threads x 4 row threads: column maxima of `rows` rows each into
// `part` ([row range][d] fp32), their maxima and c_j, then the codes.  Bound by W's bytes (read twice,
// the second time largely from the Infinity Cache) and in the third by the divisions.  One block per 64
// columns walking all rows twice kept 172 of 256 CUs busy with four waves each and took 568 us for
// a 4096 x 11008 bf16 weight; the three launches take 15 + 4 + 24 us (the last 32 us with a division
// per element).
template <typename T, int VEC>
__device__ __forceinline__ void load_cols(const T* p, float (&v)[VEC]) {
  if constexpr (VEC == 1) {
    v[0] = to_f32(*p);
  } else {
    union {
      u32x4v q;
      T e[VEC];
    } u;
    u.q = *reinterpret_cast<const u32x4v*>(p);
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] = to_f32(u.e[e]);
  }
}

template <typename T, int VEC>
__global__ __launch_bounds__(256) void k_w8_colmax(const T* __restrict__ W, int h, int d, int rows, float* __restrict__ part) {
  __shared__ float s_max[4][64 * VEC];
  const int cl = threadIdx.x & 63, rg = threadIdx.x >> 6;
  const int col = (blockIdx.x * 64 + cl) * VEC;
  const int lo = blockIdx.y * rows, hi = lo + rows < h ? lo + rows : h;
  float amax[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) amax[e] = 0.f;
  if (col < d) {
#pragma unroll 8
    for (int i = lo + rg; i < hi; i += 4) {
      float v[VEC];
      load_cols<T, VEC>(W + (size_t)i * d + col, v);
#pragma unroll
      for (int e = 0; e < VEC; ++e) amax[e] = fmaxf(amax[e], fabsf(v[e]));
    }
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) s_max[rg][cl * VEC + e] = amax[e];
  __syncthreads();
  for (int t = threadIdx.x; t < 64 * VEC; t += 256) {
    const int j = blockIdx.x * 64 * VEC + t;
    if (j < d) part[(size_t)blockIdx.y * d + j] = fmaxf(fmaxf(s_max[0][t], s_max[1][t]), fmaxf(s_max[2][t], s_max[3][t]));
  }
}

__global__ __launch_bounds__(256) void k_w8_scale(const float* __restrict__ part, int ranges, int d, float* __restrict__ c) {
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= d) return;
  float amax = 0.f;
#pragma unroll 8
  for (int s = 0; s < ranges; ++s) amax = fmaxf(amax, part[(size_t)s * d + j]);
  c[j] = amax / 127.0f;
}

// v / c, correctly rounded, for c in [2^-100, 2^100] and |v| <= 127 c, with y = fl(1 / c): Markstein's
// step -- the remainder of the approximate quotient is exact in an fma, and correcting by it times the
// correctly rounded reciprocal rounds correctly.  (Where |v| is so small that the remainder is not
// exact the quotient is far below 1/2, and its code is 0 either way.)
__device__ __forceinline__ float quotient(float v, float c, float y) {
  const float q = v * y;
  return fmaf(fmaf(-q, c, v), y, q);
}

template <typename T, int VEC>
__global__ __launch_bounds__(256) void k_w8_code(const T* __restrict__ W, int h, int d, int rows, const float* __restrict__ c,
                                                 int8_t* __restrict__ Wq) {
  const int cl = threadIdx.x & 63, rg = threadIdx.x >> 6;
  const int col = (blockIdx.x * 64 + cl) * VEC;
  const int lo = blockIdx.y * rows, hi = lo + rows < h ? lo + rows : h;
  if (col >= d) return;
  float cj[VEC], yj[VEC];
  bool fast = true;
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    cj[e] = c[col + e];
    yj[e] = 1.0f / cj[e];
    fast = fast && cj[e] >= 0x1p-100f && cj[e] <= 0x1p100f;
  }
#pragma unroll 4
  for (int i = lo + rg; i < hi; i += 4) {
    float v[VEC];
    load_cols<T, VEC>(W + (size_t)i * d + col, v);
    union {
      int8_t e[VEC];
      unsigned w[VEC < 4 ? 1 : VEC / 4];
    } o;
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      float q = 0.f;
      if (fast) {
        q = rintf(quotient(v[e], cj[e], yj[e]));
        q = fminf(fmaxf(q, -127.f), 127.f);
      } else if (cj[e] > 0.f) {
        q = rintf(v[e] / cj[e]);
        q = fminf(fmaxf(q, -127.f), 127.f);
      }
      o.e[e] = (int8_t)(int)q;
    }
    int8_t* dst = Wq + (size_t)i * d + col;
    if constexpr (VEC == 1) {
      *dst = o.e[0];
    } else {
#pragma unroll
      for (int e = 0; e < VEC / 4; ++e) reinterpret_cast<unsigned*>(dst)[e] = o.w[e];
    }
  }
}

// The same in one launch, for weights of few rows: no room for the maxima of several row ranges.
template <typename T>
__global__ __launch_bounds__(256) void k_w8_quantize(const T* __restrict__ W, int h, int d,
                                                     int8_t* __restrict__ Wq, float* __restrict__ c) {
  __shared__ float s_max[4][64];
  const int cl = threadIdx.x & 63, rg = threadIdx.x >> 6;
  const int col = blockIdx.x * 64 + cl;
  float amax = 0.f;
  if (col < d) {
    for (int i = rg; i < h; i += 4) amax = fmaxf(amax, fabsf(to_f32(W[(size_t)i * d + col])));
  }
  s_max[rg][cl] = amax;
  __syncthreads();
  amax = fmaxf(fmaxf(s_max[0][cl], s_max[1][cl]), fmaxf(s_max[2][cl], s_max[3][cl]));
  const float cj = amax / 127.0f;
  if (col >= d) return;
  if (rg == 0) c[col] = cj;
  for (int i = rg; i < h; i += 4) {
    float q = 0.f;
    if (cj > 0.f) {
      q = rintf(to_f32(W[(size_t)i * d + col]) / cj);
      q = fminf(fmaxf(q, -127.f), 127.f);
    }
    Wq[(size_t)i * d + col] = (int8_t)(int)q;
  }
}

typedef int8_t i8x8 __attribute__((ext_vector_type(8)));
// W^ = fl32(Wq * c_j), rounded to the storage type.
// Vector form (d a multiple of 16, 16-byte aligned buffers): a lane owns 8 consecutive columns,
// keeps their scales in registers and walks down the rows (blockIdx.y, stride gridDim.y); a wave
// reads 512 B and writes 1 or 2 KiB of contiguous memory per row.  Bound by its bytes (4.7 TB/s, two thirds of
// them written).  4096 x 11008 from cold caches: 29 us to bf16, 61 to fp32; with 16 columns a lane, whose 16-byte
// stores left gaps that the next ones filled, 33 and 79.  Eight waves per CU instead of 16: 42 us, 32 level.
template <typename T>
__global__ __launch_bounds__(64) void k_w8_dequantize_cols8(const int8_t* __restrict__ Wq, const float* __restrict__ c,
                                                            int h, int d, T* __restrict__ Wh) {
  const int j0 = (blockIdx.x * 64 + threadIdx.x) * 8;
  if (j0 >= d) return;
  float cs[8];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const f32x4v cg = *reinterpret_cast<const f32x4v*>(c + j0 + 4 * g);
#pragma unroll
    for (int e = 0; e < 4; ++e) cs[4 * g + e] = cg[e];
  }
#pragma unroll 8
  for (int i = blockIdx.y; i < h; i += gridDim.y) {
    const size_t o = (size_t)i * d + j0;
    const i8x8 q = __builtin_nontemporal_load(reinterpret_cast<const i8x8*>(Wq + o));
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)q[e] * cs[e];
    T* out = Wh + o;
    if constexpr (sizeof(T) == 2) {
      bf16x8v w;
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] = from_f32<bf16>(v[e]);
      *reinterpret_cast<bf16x8v*>(out) = w;
    } else {
#pragma unroll
      for (int g = 0; g < 2; ++g) *reinterpret_cast<f32x4v*>(out + 4 * g) = f32x4v{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
    }
  }
}

// Any d, any alignment: one element per thread.
template <typename T>
__global__ __launch_bounds__(256) void k_w8_dequantize_any(const int8_t* __restrict__ Wq, const float* __restrict__ c,
                                                           size_t n, int d, T* __restrict__ Wh) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += stride)
    Wh[t] = from_f32<T>((float)Wq[t] * c[t % (size_t)d]);
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

namespace {

template <typename T, int VEC>
void quantize_split(const T* W, int h, int d, int ranges, float* part, int8_t* Wq, float* c, hipStream_t stream) {
  const int rows = (h + ranges - 1) / ranges;
  const dim3 grid((unsigned)((d + 64 * VEC - 1) / (64 * VEC)), (unsigned)ranges), block(256);
  hipLaunchKernelGGL((k_w8_colmax<T, VEC>), grid, block, 0, stream, W, h, d, rows, part);
  hipLaunchKernelGGL(k_w8_scale, dim3((unsigned)((d + 255) / 256)), block, 0, stream, part, ranges, d, c);
  hipLaunchKernelGGL((k_w8_code<T, VEC>), grid, block, 0, stream, W, h, d, rows, c, Wq);
}

template <typename T>
hipError_t quantize_t(const T* W, int h, int d, int8_t* Wq, float* c, hipStream_t stream) {
  // The maxima of the row ranges live in the code buffer until the codes overwrite them: `ranges`
  // rows of d fp32 in h * d bytes (and up to 3 bytes to align them).  Up to 64 ranges of at least 32
  // rows: enough blocks for the chip from about 16 columns' worth of column blocks on.
  const int ranges = h / 32 < 64 ? h / 32 : 64;
  constexpr int VEC = 16 / (int)sizeof(T);
  // (Few rows: one launch at about 0.075 us a row takes less than three, 15 us whatever the weight up to
  // 256 x 32768: 64 x 11008 10.7 against 15.4 us, 160 x 4096 14.0 against 15.1, 192 x 4096 16.5 against 15.1,
  // 4096 x 11008 691 against 49; where the columns alone are more than a round of blocks earlier: 131072
  // columns, 64 rows 12.1 against 15.1, 96 rows 20.0 against 15.5.)
  if (ranges < 2 || h < 80 || (h <= 160 && d <= 1 << 16)) {
    hipLaunchKernelGGL(k_w8_quantize<T>, dim3((unsigned)((d + 63) / 64)), dim3(256), 0, stream, W, h, d, Wq, c);
    return hipGetLastError();
  }
  float* part = reinterpret_cast<float*>((reinterpret_cast<uintptr_t>(Wq) + 3) & ~(uintptr_t)3);
  if (d % VEC == 0 && aligned16(W) && (reinterpret_cast<uintptr_t>(Wq) & 3) == 0)
    quantize_split<T, VEC>(W, h, d, ranges, part, Wq, c, stream);
  else
    quantize_split<T, 1>(W, h, d, ranges, part, Wq, c, stream);
  return hipGetLastError();
}

}  // namespace

hipError_t w8_quantize(const void* W, int dtype, int h, int d, int8_t* Wq, float* c, hipStream_t stream) {
  return dtype == MLORA_F32 ? quantize_t((const float*)W, h, d, Wq, c, stream)
                            : quantize_t((const bf16*)W, h, d, Wq, c, stream);
}

hipError_t w8_dequantize(const int8_t* Wq, const float* c, int dtype, int h, int d, void* Wh, hipStream_t stream) {
  const size_t n = (size_t)h * (size_t)d;
  if (d % 16 == 0 && aligned16(Wq) && aligned16(c) && aligned16(Wh)) {
    const int gx = (d / 8 + 63) / 64;
    int gy = (256 * 16 + gx - 1) / gx;          // about 16 waves per CU over the whole grid
    gy = gy < h ? gy : h;
    const dim3 grid((unsigned)gx, (unsigned)gy), block(64);
    if (dtype == MLORA_F32)
      hipLaunchKernelGGL(k_w8_dequantize_cols8<float>, grid, block, 0, stream, Wq, c, h, d, (float*)Wh);
    else
      hipLaunchKernelGGL(k_w8_dequantize_cols8<bf16>, grid, block, 0, stream, Wq, c, h, d, (bf16*)Wh);
    return hipGetLastError();
  }
  size_t blocks = (n + 255) / 256;
  if (blocks > 256 * 64) blocks = 256 * 64;   // grid-stride beyond 64 blocks per CU
  const dim3 grid((unsigned)blocks), block(256);
  if (dtype == MLORA_F32)
    hipLaunchKernelGGL(k_w8_dequantize_any<float>, grid, block, 0, stream, Wq, c, n, d, (float*)Wh);
  else
    hipLaunchKernelGGL(k_w8_dequantize_any<bf16>, grid, block, 0, stream, Wq, c, n, d, (bf16*)Wh);
  return hipGetLastError();
}

}  // namespace mlora
