// Device-side helpers for gfx950 (CDNA4, wave64): vector types, bf16/fp32
// conversion, 16-byte vector loads/stores and the bf16 matrix-core op.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nt {

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;

// Workgroups of a launch, in rows of at most kGridX: a launch whose grid x times
// the block size reaches 2^32 is refused, or runs with that product modulo 2^32.
// kGridX is a multiple of 8, so workgroup id still runs on XCD id % 8.  The last
// of several rows may hold ids past the launch's own: the kernel returns on them.
// The row length is the constant and not gridDim.x, which every workgroup would
// load before its first table entry.
constexpr int64_t kGridX = 1 << 21;
inline dim3 folded_grid(int64_t blocks) {
  return dim3((unsigned)(blocks < kGridX ? blocks : kGridX), (unsigned)((blocks + kGridX - 1) / kGridX));
}
__device__ __forceinline__ uint32_t block_id() { return blockIdx.y * (uint32_t)kGridX + blockIdx.x; }

// D(16x16, f32) += A(16x32, bf16) * B(32x16, bf16).  Lane l supplies A row
// l%16 and B column l%16, each with eight k values selected by l/16; the k
// order is the same for A and B, so any consistent k permutation gives the
// same product.  Lane l receives D rows 4*(l/16) + i, i = 0..3, column l%16.
__device__ __forceinline__ f32x4 mfma16(const bf16x8& a, const bf16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---- pair-tiled operand layout -----------------------------------------------
// One channel plane of sample i (an N x N matrix, rows r, columns k) is cut
// into 16 x 32 tiles, row tiles outer, each tile stored in the lane order of a
// matrix-core fragment: element (r, k) of a tile sits at ((k/8)*16 + r%16)*8
// + k%8, so lane l of a wave reads the 8 consecutive k of tile row l%16 and
// k-group l/16 as one 16-byte piece and the whole wave reads 1 KB contiguously.
// Planes occupy round_up(N,16) x round_up(N,32) elements; nkt = round_up(N,32)/32.
__host__ __device__ __forceinline__ int32_t tiled_offset(int32_t r, int32_t k, int32_t nkt) {
  return (((r >> 4) * nkt + (k >> 5)) << 9) + ((((k & 31) >> 3) << 4) + (r & 15)) * 8 + (k & 7);
}

// ---- 16-byte vectors of a storage type, converted to/from fp32 ------------
template <typename T> struct Vec;

template <> struct Vec<float> {
  static constexpr int N = 4;
  float v[4];
  __device__ __forceinline__ void load(const float* p) {
    const float4 t = *reinterpret_cast<const float4*>(p);
    v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
  }
  __device__ __forceinline__ void store(float* p) const {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  }
};

template <> struct Vec<bf16> {
  static constexpr int N = 8;
  float v[8];
  __device__ __forceinline__ void load(const bf16* p) {
    const uint4 t = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[2 * j] = __uint_as_float(w[j] << 16);
      v[2 * j + 1] = __uint_as_float(w[j] & 0xffff0000u);
    }
  }
  __device__ __forceinline__ void store(bf16* p) const {
    bf16x8 t;
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = (bf16)v[j];
    *reinterpret_cast<bf16x8*>(p) = t;
  }
};

// Non-temporal 16- and 8-byte stores (streaming hint: the lines are not kept
// in the caches on the way out).
typedef uint32_t u32x4_nt __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_nt __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_nt(bf16* p, const bf16x8& v) {
  __builtin_nontemporal_store(__builtin_bit_cast(u32x4_nt, v), reinterpret_cast<u32x4_nt*>(p));
}
__device__ __forceinline__ void store_nt(bf16* p, const bf16x4& v) {
  __builtin_nontemporal_store(__builtin_bit_cast(u32x2_nt, v), reinterpret_cast<u32x2_nt*>(p));
}

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16 x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_f32(float x);
template <> __device__ __forceinline__ float from_f32<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float x) { return (bf16)x; }

// GELU, x Phi(x), in its error-function form: with h = erfc(|x| / sqrt 2) / 2
// it is max(x, 0) - |x| h for either sign.  erfc(z) = exp(-z^2) t P(t) with
// t = 1 / (1 + 0.3 z), the form of Hastings (Approximations for Digital
// Computers, 1955; Abramowitz and Stegun 7.1.26), and P a degree-8 fit made for
// this kernel, of erfcx(z) / t to equal relative error (2.1e-8).  In fp32 the largest absolute error over |x| < 12 is 2.4e-7
// (0.5 x (1 + erff) has 4.5e-7, and loses the whole value where 1 + erf
// cancels).  About 17 instructions without a branch; erff evaluates two
// polynomials and an exponential under masks.
__device__ __forceinline__ float gelu(float x) {
  const float a = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(fmaf(0.21213203435596426f, a, 1.f));
  float q = -6.462623179e-02f;
  q = fmaf(q, t, 2.421491444e-01f);
  q = fmaf(q, t, -2.548829019e-01f);
  q = fmaf(q, t, 2.724800110e-01f);
  q = fmaf(q, t, -4.641081393e-02f);
  q = fmaf(q, t, 1.070898473e-01f);
  q = fmaf(q, t, 7.426083088e-02f);
  q = fmaf(q, t, 8.534543961e-02f);
  q = fmaf(q, t, 8.459468186e-02f);
  const float h = q * t * __builtin_amdgcn_exp2f(x * x * -0.72134752044448170f);
  return fmaxf(x, 0.f) - fminf(a, 64.f) * h;      // h is 0 long before 64, also at infinity
}

// Sum over the four lanes l, l^16, l^32, l^48 (the k-groups holding one row
// of a matrix-core fragment): two lane-row swaps, no LDS round trip.  Every
// lane adds the same two values in either order, so all four get identical
// bits.
__device__ __forceinline__ float sum_over_kgroups(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Reductions within aligned groups of `width` lanes (width a power of two <= 64).
template <int width>
__device__ __forceinline__ float group_sum(float x) {
#pragma unroll
  for (int m = width / 2; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
  return x;
}
template <int width>
__device__ __forceinline__ float group_max(float x) {
#pragma unroll
  for (int m = width / 2; m >= 1; m >>= 1) x = fmaxf(x, __shfl_xor(x, m, 64));
  return x;
}

}  // namespace nt
