// Large-K projection (the packed-token encoder path, Sec. 3.3: V' = V W^T + b
// on packed rows, with the pre-normalisation of the encoder layer): a tiled
// bf16 GEMM on the matrix cores for K a multiple of 32, computed transposed as
// D^T = W X^T so that a lane ends up with four consecutive output channels of
// one row.
//
// A workgroup owns a TM-row x TN-channel output tile; its WN x WM waves each
// compute TN / WN channels x TM / WM rows.  With KS = 2 a second set of waves
// takes every other 64 k and the two sums are added through LDS at the end: a
// tile alone on its CU then needs half the steps, each bound by its own
// latency.  Operand tiles of 64 k (whole
// 128-byte lines per row: the texture-address unit, which the copies and not
// the products keep busiest, works by the line) are copied global -> LDS with
// global_load_lds into a ring of ST stages, ST - 1 steps ahead, so one barrier
// per step covers both "the copy has landed" and "the slot is free again".
// Each 128-byte row of a staged tile holds its eight 16-byte pieces in the
// order piece ^ (row & 7): the 16 rows of a fragment read then fall on
// different bank groups.  With a LayerNorm the rows are first normalised
// (two-pass statistics in fp32, result rounded to bf16 as the product consumes
// it) into the caller's workspace by a one-wave-per-row pass, and the product
// reads that copy: one extra write and read of the rows instead of every
// channel tile re-reducing them.
#include <algorithm>

#include "nt_device.h"
#include "nt_internal.h"

namespace nt {
namespace {

constexpr int kGBK = 64;                  // k per stage

typedef uint32_t g_u32x4 __attribute__((ext_vector_type(4)));
// N fragments of one 32-wide half step, 16 staged rows (2 KB) apart, from the
// byte address a.  The caller waits for them (lds_wait): as plain loads the
// compiler would make them wait for the copies still in flight into the other
// stages.
template <int N>
__device__ __forceinline__ void lds_frags(uint32_t a, g_u32x4 (&r)[N]) {
  static_assert(N == 2 || N == 4 || N == 8, "2, 4 or 8 fragments");
  if constexpr (N == 2) {
    asm volatile("ds_read_b128 %0, %2\n"
                 "ds_read_b128 %1, %2 offset:2048\n"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0]), "=&v"(r[1])
                 : "v"(a)
                 : "memory");
  } else if constexpr (N == 4) {
    asm volatile("ds_read_b128 %0, %4\n"
                 "ds_read_b128 %1, %4 offset:2048\n"
                 "ds_read_b128 %2, %4 offset:4096\n"
                 "ds_read_b128 %3, %4 offset:6144\n"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
                 : "v"(a)
                 : "memory");
  } else {
    asm volatile("ds_read_b128 %0, %8\n"
                 "ds_read_b128 %1, %8 offset:2048\n"
                 "ds_read_b128 %2, %8 offset:4096\n"
                 "ds_read_b128 %3, %8 offset:6144\n"
                 "ds_read_b128 %4, %8 offset:8192\n"
                 "ds_read_b128 %5, %8 offset:10240\n"
                 "ds_read_b128 %6, %8 offset:12288\n"
                 "ds_read_b128 %7, %8 offset:14336\n"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
                 : "v"(a)
                 : "memory");
  }
}
// Both operands of a half step in one block, with one wait (8 weight and 4 row
// fragments, the large tile).
__device__ __forceinline__ void lds_frags_8_4(uint32_t aw, uint32_t ax, g_u32x4 (&w)[8], g_u32x4 (&x)[4]) {
  asm volatile("ds_read_b128 %0, %12\n"
               "ds_read_b128 %1, %12 offset:2048\n"
               "ds_read_b128 %2, %12 offset:4096\n"
               "ds_read_b128 %3, %12 offset:6144\n"
               "ds_read_b128 %4, %12 offset:8192\n"
               "ds_read_b128 %5, %12 offset:10240\n"
               "ds_read_b128 %6, %12 offset:12288\n"
               "ds_read_b128 %7, %12 offset:14336\n"
               "ds_read_b128 %8, %13\n"
               "ds_read_b128 %9, %13 offset:2048\n"
               "ds_read_b128 %10, %13 offset:4096\n"
               "ds_read_b128 %11, %13 offset:6144\n"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7]),
                 "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3])
               : "v"(aw), "v"(ax)
               : "memory");
}

// at most N copies of this wave outstanding (the other counters free)
template <int N>
__device__ __forceinline__ void wait_copies() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4 << 14));
}

template <int TN, int TM, int WN, int WM, int ST, int KS>
constexpr size_t gemm_smem() {
  constexpr int EC = TN / WN < 64 ? TN / WN : 64;
  const size_t ring = (size_t)ST * KS * (TN + TM) * kGBK * 2, epi = (size_t)WN * TM * (EC + 4) * 4;
  return ring > epi ? ring : epi;
}

template <int TN, int TM, int WN, int WM, int ST, int KS>
__global__ void __launch_bounds__(64 * WN * WM * KS, TN == 256 ? 2 : 0) gemm_kernel(GemmArgs p) {
  constexpr int NW = WN * WM, FN = TN / WN / 16, FM = TM / WM / 16;   // waves; weight and row fragments of a wave
  constexpr int COPIES = (TN + TM) / 8 / NW;                          // copy instructions per wave and stage (8 rows each)
  constexpr int STAGE = (TN + TM) * kGBK;                             // elements of one wave set
  constexpr int EC = TN / WN < 64 ? TN / WN : 64;                     // channels per epilogue round
  static_assert((TN + TM) / 8 % NW == 0 && TN / 8 % NW == 0, "whole copies per wave");
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16* ring = reinterpret_cast<bf16*>(smem);

  // ---- tile of this workgroup: XCD x = id % 8 takes row tiles x, x + 8, ...
  // and walks their channel tiles in order, so a row tile is read into one L2
  const int id = blockIdx.x;
  const int xcd = id % kXcds, kq = id / kXcds;
  const int rt = __builtin_amdgcn_readfirstlane(kq / p.ntn) * kXcds + xcd;
  const int nt = __builtin_amdgcn_readfirstlane(kq % p.ntn);
  if (rt >= p.ntm) return;
  const int m0 = rt * TM, n0 = nt * TN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int ks = wave / NW, wv = wave % NW;               // wave set, wave within it
  const int wc = wv % WN, wr = wv / WN;
  const int nk64 = (p.K + kGBK - 1) / kGBK, nk = (nk64 + KS - 1) / KS;   // 64 k each; steps

  // ---- stage copies: instruction c copies 8 rows of the W tile (c < TN / 8)
  // or of the X tile; lane l -> row 8 c' + l / 8, the piece whose place is
  // l % 8.  Rows past the matrix repeat its last row (their outputs are never
  // stored); in a last stage of 32 k the upper pieces repeat the lower ones
  // (not multiplied).
  const int piece = (lane & 7) ^ ((lane >> 3) & 7);
  const bf16* src[COPIES];
#pragma unroll
  for (int u = 0; u < COPIES; ++u) {
    const int c = wv + NW * u;
    const bool isx = c >= TN / 8;
    const int row = (isx ? c - TN / 8 : c) * 8 + (lane >> 3);
    src[u] = (isx ? p.x + (int64_t)min(m0 + row, p.rows - 1) * p.ldx : p.w + (int64_t)min(n0 + row, p.N - 1) * p.K) + piece * 8;
  }
  auto copy_stage = [&](int kt, int slot) {
    bf16* st = ring + (slot * KS + ks) * STAGE;
    const int k = min(kt * KS + ks, nk64 - 1) * kGBK;       // the set without a last 64 k repeats it (not multiplied)
    const int back = k + 32 < p.K ? 0 : (piece >= 4 ? 32 : 0);
#pragma unroll
    for (int u = 0; u < COPIES; ++u)
      __builtin_amdgcn_global_load_lds((const void*)(src[u] + k - back),
                                       (__attribute__((address_space(3))) void*)(st + (wv + NW * u) * 512), 16, 0, 0);
  };
  for (int s = 0; s < ST - 1; ++s)
    if (s < nk) copy_stage(s, s);

  f32x4 acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // this lane's byte offset inside a 16-row fragment block: row l16, piece g
  // (k half 0) or 4 + g at its swizzled place
  const uint32_t lofs0 = (uint32_t)(l16 * kGBK * 2 + ((g ^ (l16 & 7)) << 4));
  const uint32_t lofs1 = (uint32_t)(l16 * kGBK * 2 + (((4 + g) ^ (l16 & 7)) << 4));
  const uint32_t ring0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) bf16*)ring;
  int slot = 0;
  for (int kt = 0; kt < nk; ++kt) {
    // stage kt has landed for this wave (later stages may still be in flight)
    const int later = min(ST - 2, nk - 1 - kt);
    static_assert(ST >= 2 && ST <= 8 && (ST - 2) * COPIES < 64, "two to eight stages, within the counter's range");
    switch (later) {
      case 1: wait_copies<(ST > 2 ? 1 : 0) * COPIES>(); break;
      case 2: wait_copies<(ST > 3 ? 2 : 0) * COPIES>(); break;
      case 3: wait_copies<(ST > 4 ? 3 : 0) * COPIES>(); break;
      case 4: wait_copies<(ST > 5 ? 4 : 0) * COPIES>(); break;
      case 5: wait_copies<(ST > 6 ? 5 : 0) * COPIES>(); break;
      case 6: wait_copies<(ST > 7 ? 6 : 0) * COPIES>(); break;
      default: wait_copies<0>();
    }
    // stage kt complete everywhere and slot kt - 1 free (every wave's reads of
    // it ended in an LDS wait).  The plain barrier: __syncthreads would also
    // wait for the copies still in flight, leaving no lookahead.
    __builtin_amdgcn_s_barrier();
    if (kt + ST - 1 < nk) copy_stage(kt + ST - 1, slot == 0 ? ST - 1 : slot - 1);
    const uint32_t st = ring0 + (slot * KS + ks) * (STAGE * 2);
    slot = slot == ST - 1 ? 0 : slot + 1;
    const uint32_t aw = st + wc * (TN / WN) * kGBK * 2, ax = st + (TN + wr * (TM / WM)) * kGBK * 2;
    const int kb = (kt * KS + ks) * kGBK, halves = kb + 32 < p.K ? 2 : kb < p.K ? 1 : 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (h >= halves) break;
      g_u32x4 rw[FN], rx[FM];
      if constexpr (FN == 8 && FM == 4) {
        lds_frags_8_4(aw + (h ? lofs1 : lofs0), ax + (h ? lofs1 : lofs0), rw, rx);
      } else {
        lds_frags<FN>(aw + (h ? lofs1 : lofs0), rw);
        lds_frags<FM>(ax + (h ? lofs1 : lofs0), rx);
      }
#pragma unroll
      for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j)
          acc[i][j] = mfma16(__builtin_bit_cast(bf16x8, rw[i]), __builtin_bit_cast(bf16x8, rx[j]), acc[i][j]);
    }
  }

  // ---- epilogue, rounds of EC channels per wave through LDS: acc[i][j][ii]
  // is channel n0 + wc TN/WN + 16 i + 4 g + ii of row m0 + wr TM/WM + 16 j + l16
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();                                // the ring is free for the epilogue stage
  if constexpr (KS == 2) {                        // the second set's sums, in the lanes' order
    f32x4* hand = reinterpret_cast<f32x4*>(smem) + wv * (FN * FM * 64) + lane;
    if (ks == 1) {
#pragma unroll
      for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) hand[(i * FM + j) * 64] = acc[i][j];
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
      for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] += hand[(i * FM + j) * 64];
    }
    __syncthreads();
    if (ks == 1) return;
  }
  constexpr int ES = EC + 4, PR = EC / 8, RP = 64 / PR;   // stage row stride; pieces per row; rows per pass
  float* es = reinterpret_cast<float*>(smem) + wv * (TM / WM) * ES;
#pragma unroll
  for (int round = 0; round < TN / WN / EC; ++round) {
#pragma unroll
    for (int i = 0; i < EC / 16; ++i)
#pragma unroll
      for (int j = 0; j < FM; ++j) {
        const int ii = round * (EC / 16) + i;
        *reinterpret_cast<float4*>(&es[(j * 16 + l16) * ES + i * 16 + 4 * g]) =
            make_float4(acc[ii][j][0], acc[ii][j][1], acc[ii][j][2], acc[ii][j][3]);
      }
    // the wave's own stage: its LDS writes complete before its reads
    const int cc = lane % PR, n = n0 + wc * (TN / WN) + round * EC + cc * 8;
    float bv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) bv[e] = (p.bias && n + e < p.N) ? p.bias[n + e] : 0.f;
#pragma unroll
    for (int q = 0; q < TM / WM / RP; ++q) {
      const int rl = q * RP + lane / PR, m = m0 + wr * (TM / WM) + rl;
      if (m >= p.rows || n >= p.N) continue;      // N % 8 == 0: a piece is all in or all out
      const float4 a0 = *reinterpret_cast<const float4*>(&es[rl * ES + cc * 8]);
      const float4 a1 = *reinterpret_cast<const float4*>(&es[rl * ES + cc * 8 + 4]);
      float v[8] = {a0.x + bv[0], a0.y + bv[1], a0.z + bv[2], a0.w + bv[3], a1.x + bv[4], a1.y + bv[5], a1.z + bv[6], a1.w + bv[7]};
      if (p.epi == NT_EPI_GELU) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = gelu(v[e]);
      } else if (p.epi == NT_EPI_RESIDUAL) {
        const uint4 rr = *reinterpret_cast<const uint4*>(p.res + (int64_t)m * p.ld_res + n);
        const uint32_t w4[4] = {rr.x, rr.y, rr.z, rr.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[2 * e] += __uint_as_float(w4[e] << 16);
          v[2 * e + 1] += __uint_as_float(w4[e] & 0xffff0000u);
        }
      }
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (bf16)v[e];
      *reinterpret_cast<bf16x8*>(p.y + (int64_t)m * p.ldy + n) = o;
    }
  }
}

template <int TN, int TM, int WN, int WM, int ST, int KS = 1>
hipError_t launch_tile(GemmArgs p, hipStream_t s) {
  p.ntm = (p.rows + TM - 1) / TM;
  p.ntn = (p.N + TN - 1) / TN;
  constexpr size_t smem = gemm_smem<TN, TM, WN, WM, ST, KS>();
  const hipError_t e = hipFuncSetAttribute((const void*)gemm_kernel<TN, TM, WN, WM, ST, KS>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  const int grid = (p.ntm + kXcds - 1) / kXcds * kXcds * p.ntn;
  gemm_kernel<TN, TM, WN, WM, ST, KS><<<dim3((unsigned)grid), dim3(64 * WN * WM * KS), smem, s>>>(p);
  return hipGetLastError();
}

// LayerNorm of every row into xn [rows, K] (row stride K), one wave per row:
// lane c of the row holds 16-byte pieces c, c + 64, ... in registers.
template <int CPL>
__global__ void __launch_bounds__(256) layernorm_rows_kernel(const bf16* x, int64_t ldx, int rows, int K,
                                                             const float* gamma, const float* beta, float eps,
                                                             bf16* xn) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int nc = K / 8;
  const bf16* xr = x + (int64_t)row * ldx;
  float v[CPL][8];
#pragma unroll
  for (int u = 0; u < CPL; ++u) {
    const int c = lane + 64 * u;
    const uint4 r = c < nc ? *reinterpret_cast<const uint4*>(xr + c * 8) : make_uint4(0u, 0u, 0u, 0u);
    const uint32_t w4[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[u][2 * e] = __uint_as_float(w4[e] << 16);
      v[u][2 * e + 1] = __uint_as_float(w4[e] & 0xffff0000u);
    }
  }
  float s1 = 0.f;
#pragma unroll
  for (int u = 0; u < CPL; ++u)
#pragma unroll
    for (int e = 0; e < 8; ++e) s1 += v[u][e];
  const float mean = group_sum<64>(s1) / (float)K;
  float s2 = 0.f;
#pragma unroll
  for (int u = 0; u < CPL; ++u) {
    if (lane + 64 * u >= nc) break;
#pragma unroll
    for (int e = 0; e < 8; ++e) { const float d = v[u][e] - mean; s2 += d * d; }
  }
  const float rstd = rsqrtf(group_sum<64>(s2) / (float)K + eps);
#pragma unroll
  for (int u = 0; u < CPL; ++u) {
    const int c = lane + 64 * u;
    if (c >= nc) break;
    const float4 g0 = *reinterpret_cast<const float4*>(gamma + c * 8), g1 = *reinterpret_cast<const float4*>(gamma + c * 8 + 4);
    const float4 b0 = beta ? *reinterpret_cast<const float4*>(beta + c * 8) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 b1 = beta ? *reinterpret_cast<const float4*>(beta + c * 8 + 4) : make_float4(0.f, 0.f, 0.f, 0.f);
    const float gg[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
    const float bb[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16)((v[u][e] - mean) * rstd * gg[e] + bb[e]);
    *reinterpret_cast<bf16x8*>(xn + (int64_t)row * K + c * 8) = o;
  }
}

}  // namespace

bool gemm_fits(int K) { return K % 32 == 0 && K >= 128 && K <= 64 * 8 * 8; }

hipError_t launch_gemm(GemmArgs p, hipStream_t s) {
  if (p.rows == 0) return hipSuccess;
  if (p.gamma) {
    if (!p.ln_ws) return hipErrorInvalidValue;
    hipError_t e;
    bf16* xn = p.ln_ws;
    const dim3 grid((unsigned)((p.rows + 3) / 4));
    const int cpl = (p.K / 8 + 63) / 64;          // 16-byte pieces per lane
    if (cpl <= 2) layernorm_rows_kernel<2><<<grid, dim3(256), 0, s>>>(p.x, p.ldx, p.rows, p.K, p.gamma, p.beta, p.eps, xn);
    else if (cpl <= 4) layernorm_rows_kernel<4><<<grid, dim3(256), 0, s>>>(p.x, p.ldx, p.rows, p.K, p.gamma, p.beta, p.eps, xn);
    else layernorm_rows_kernel<8><<<grid, dim3(256), 0, s>>>(p.x, p.ldx, p.rows, p.K, p.gamma, p.beta, p.eps, xn);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    p.x = xn;
    p.ldx = p.K;
    p.gamma = p.beta = nullptr;
  }
  // The tile size with the least time by rounds over the CUs: XCD x holds row
  // tiles x, x + 8, ..., its 32 CUs run 2, 2 or 1 workgroups of the 64-, 128- and
  // 256-wide tiles, and a round of them takes 8.2, 16 and 25 us at K = 768 (at
  // every K from 384 to 3072 about as 1 to 2 to 3).  64-wide tiles that leave
  // every CU at most one workgroup split K (3072 x 768 at 1019 rows: 24.6 us
  // without).
  const auto per_xcd = [&](int t) { return ((p.rows + t - 1) / t + kXcds - 1) / kXcds * (int64_t)((p.N + t - 1) / t); };
  const int cus = compute_units() / kXcds;
  const auto rounds = [&](int t, int per_cu) { return (per_xcd(t) + cus * per_cu - 1) / (cus * per_cu); };
  const int64_t c64 = rounds(64, 2), c128 = 2 * rounds(128, 2), c256 = 3 * rounds(256, 1);
  if (c256 <= c128 && c256 <= c64) return launch_tile<256, 256, 2, 4, 2>(p, s);
  if (c128 <= c64) return launch_tile<128, 128, 2, 2, 2>(p, s);
  if (per_xcd(64) > cus) return launch_tile<64, 64, 2, 2, 4>(p, s);
  return launch_tile<64, 64, 2, 2, 4, 2>(p, s);
}

}  // namespace nt
