// Backward of row / column attention with pair bias (the starting- and
// ending-node attention of the Pairformer cited in Sec. 4.3) for a training
// step (Sec. 3.4).  Per sample i, pair row r and head h (axis 1: the same on
// the sample's transpose), with S = scale Q K^T + B and P = softmax_k(S):
//   lse_j = log sum_k exp S_jk,  D_j = sum_k P_jk (dO_j . V_k)  (= dO_j . O_j),
//   dS_jk = P_jk (dO_j . V_k - D_j),
//   dQ_j = scale sum_k dS_jk K_k,  dK_k = scale sum_j dS_jk Q_j,
//   dV_k = sum_j P_jk dO_j,        dB_jk = sum_r dS_jk   (the bias is shared by all rows).
//
// Every product runs on the matrix cores with fp32 accumulation.  Q K^T and
// dO V^T have bf16 operands as they are.  P and dS stay fp32: as operands of
// dQ, dK and dV each is split into three bf16 parts (the upper, middle and
// lower 8 bits of its significand, exact), one product per part, so no bit
// of them is dropped.  Softmax arithmetic is fp32 on the vector units.
//
// attn_bwd_rows_kernel: one workgroup per (pair row, head); the row's q, k, v
// and dO are copied into LDS.  Phase A: a wave per 16-query tile, first the
// softmax statistics over all keys, then dQ; phase B: a wave per 16-key tile,
// dK and dV.  lse and D go to the workspace for the bias gradient.
// attn_bwd_bias_kernel: a workgroup per (sample, head, 64 queries, 64 keys)
// walks all pair rows and keeps its sums of dS in registers (no atomics).
//
// The vector units bound the rows kernel: per score it spends about 16 vector
// instructions on the 3-way splits and one exponential in each of three
// passes (statistics, dQ, dK/dV), against 30 products per 512 scores.  At
// B=8, N 66..317, 4 heads: 560 us; one thread per query or key with fp32 FMAs
// took 12.2 ms (and the bias gradient 5.8 ms, now 232 us).
#include <algorithm>

#include "nt_device.h"
#include "nt_internal.h"

namespace nt {
namespace {

constexpr int kD = 32;                 // head_dim
constexpr float kLog2e = 1.4426950408889634f;

struct AttnBwdArgs {
  int axis, H;
  const bf16* q;
  const bf16* k;
  const bf16* v;
  int64_t ld_qkv;
  const bf16* bias;                    // NULL: no bias
  int64_t ld_bias, ld_bias_head;
  const bf16* dout;
  int64_t ld_dout;
  float scale;
  bf16* dq;
  bf16* dk;
  bf16* dv;
  int64_t ld_dqkv;
  float* dbias;
  int64_t ld_dbias, ld_dbias_head;
  float* lse;                          // workspace: [H][sum N^2], element cu + r n + j of row r, query j
  float* dsum;                         // workspace: D, same layout
  int64_t cells;                       // sum N^2
  const int32_t* work;                 // (sample, row) pairs; -1 = idle
  uint32_t row_blocks;                 // workgroups of the rows kernel: work positions x heads
  const int32_t* cu_seqlens;
  const int32_t* cu_pairs;
  // bias images (IMG instances): tile (a, b) of head h at
  // (h * img_tiles + bias_tiles[i] + a * kti + b) * 64 + lane, kti = round_up(n, 64) / 16
  const uint2* img_q;                  // lane l16 + 16 g: bias(16 a + l16, 16 b + 4 g + e)
  const uint2* img_k;                  // lane l16 + 16 g: bias(16 b + 4 g + e, 16 a + l16)
  int64_t img_tiles;
  const int32_t* bias_tiles;
  const int32_t* cu_bgrad;             // [batch + 1] prefix of the bias-gradient blocks of one head
  int batch;
};

// a value that is the same in all lanes, as a scalar
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ float exp_native(float x) { return __builtin_amdgcn_exp2f(x * kLog2e); }

__device__ __forceinline__ uint32_t lds_addr(const bf16* ptr) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) bf16*)ptr;
}
__device__ __forceinline__ bf16x8 pack_u2(uint2 lo, uint2 hi) {
  const uint32_t w[4] = {lo.x, lo.y, hi.x, hi.y};
  return __builtin_bit_cast(bf16x8, w);
}

// LDS image of 16 rows x 32 dims (1 KB): the 16-byte piece (row, dims 8 d ..
// 8 d + 7) sits in slot 16 d + (row ^ 8 (d & 1)).  Read as a matrix-core
// fragment (lane l16 + 16 g: row l16, dims 8 g ..) it is a permutation of the
// whole 1 KB; the XOR puts the two pieces of a transposed read on different
// banks.
__device__ __forceinline__ int frag_offset(int l16, int g) { return (g * 16 + (l16 ^ ((g & 1) << 3))) * 8; }
__device__ __forceinline__ bf16x8 frag(const bf16* T, int tile, int fo) {
  return *reinterpret_cast<const bf16x8*>(T + tile * 512 + fo);
}
// Transposed fragments: ds_read_b64_tr_b16 hands lane 4q+m of each 16-lane
// group element m of the 8-byte pieces addressed by lanes q, q+4, q+8, q+12;
// pointing lane i at row 4 g + i/4, dims 4 (i%4) gives lane l16 rows 4 g ..
// 4 g + 3 of dim l16.  Dims 16..31 are 512 bytes further on, the next tile
// 1024 bytes.
__device__ __forceinline__ uint32_t tr_offset(int l16, int g) {
  const int row = 4 * g + (l16 >> 2), d = (l16 & 3) >> 1;
  return (uint32_t)((d * 16 + (row ^ (d << 3))) * 16 + (l16 & 1) * 8);
}
// tiles t, t + 1 of T: f[0] dims 0-15, f[1] dims 16-31 (k slots: rows 4 g .. of tile t, then of t + 1)
__device__ __forceinline__ void tr_frags(const bf16* T, int tile, uint32_t to, bf16x8 (&f)[2]) {
  const uint32_t a = lds_addr(T + tile * 512) + to;
  uint2 r[4];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %4\n"
      "ds_read_b64_tr_b16 %1, %4 offset:1024\n"
      "ds_read_b64_tr_b16 %2, %4 offset:512\n"
      "ds_read_b64_tr_b16 %3, %4 offset:1536\n"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
      : "v"(a)
      : "memory");
  f[0] = pack_u2(r[0], r[1]);
  f[1] = pack_u2(r[2], r[3]);
}

// x = part[0] + part[1] + part[2] for eight fp32 values (finite): the parts
// are the upper, middle and lower 8 bits of the significand.
__device__ __forceinline__ void split3(const float (&x)[8], bf16x8 (&part)[3]) {
  uint32_t w[3][4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t h[2], m[2], l[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      h[u] = __float_as_uint(x[2 * e + u]);
      const float r = x[2 * e + u] - __uint_as_float(h[u] & 0xffff0000u);
      m[u] = __float_as_uint(r);
      l[u] = __float_as_uint(r - __uint_as_float(m[u] & 0xffff0000u));
    }
    w[0][e] = __builtin_amdgcn_perm(h[1], h[0], 0x07060302u);
    w[1][e] = __builtin_amdgcn_perm(m[1], m[0], 0x07060302u);
    w[2][e] = __builtin_amdgcn_perm(l[1], l[0], 0x07060302u);
  }
#pragma unroll
  for (int t = 0; t < 3; ++t) part[t] = __builtin_bit_cast(bf16x8, w[t]);
}

// head-h bias of (query j, key k) of a sample (axis 1: of cell (k, j))
__device__ __forceinline__ float bias_at(const AttnBwdArgs& p, int64_t cu, int n, int j, int k, int h) {
  if (!p.bias) return 0.f;
  const int64_t cell = cu + (p.axis == 0 ? (int64_t)j * n + k : (int64_t)k * n + j);
  return (float)p.bias[cell * p.ld_bias + (int64_t)h * p.ld_bias_head];
}

// maximum over the four lanes l16 + 16 g (g = 0..3)
__device__ __forceinline__ float max_over_kgroups(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// 16 rows x 32 dims of a gradient: lane (l16, g) holds dims 4 g .. 4 g + 3
// (acc[0]) and 16 + 4 g .. (acc[1]) of row l16.  Lane rows g, g ^ 1 trade
// halves so that every lane stores 16 bytes.
__device__ __forceinline__ void store_rows(bf16* row, bool valid, int g, const f32x4 (&acc)[2], float mul) {
  uint32_t w[2][2];
#pragma unroll
  for (int dt = 0; dt < 2; ++dt) {
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16)(acc[dt][e] * mul);
    const uint2 u = __builtin_bit_cast(uint2, o);
    w[dt][0] = u.x;
    w[dt][1] = u.y;
  }
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const auto sw = __builtin_amdgcn_permlane16_swap(w[0][e], w[1][e], false, false);
    w[0][e] = sw[0];
    w[1][e] = sw[1];
  }
  if (valid) {
    const int d0 = (g & 1) ? 16 + 4 * (g - 1) : 4 * g;
    *reinterpret_cast<uint4*>(row + d0) = make_uint4(w[0][0], w[0][1], w[1][0], w[1][1]);
  }
}

template <int NW, bool IMG>
__global__ void __launch_bounds__(64 * NW, 4) attn_bwd_rows_kernel(AttnBwdArgs p, int nt_max) {
  extern __shared__ __attribute__((aligned(16))) bf16 lds[];
  // workgroup 8 (H k + h) + x runs on XCD x: the heads of a pair row, which
  // share cache lines, run on one XCD one after the other
  const uint32_t id = block_id();
  if (id >= p.row_blocks) return;
  const int x = id % kXcds, t0 = id / kXcds;
  // everything derived from the block index is the same in all lanes: kept in scalars
  const int h = uni(t0 % p.H), pos = uni(t0 / p.H) * kXcds + x;
  const int i = uni(p.work[2 * pos]), r = uni(p.work[2 * pos + 1]);
  if (i < 0) return;
  const int n = uni(p.cu_seqlens[i + 1] - p.cu_seqlens[i]);
  const int64_t cu = uni(p.cu_pairs[i]);
  const int nt = (n + 15) >> 4, nt2 = (nt + 1) & ~1;      // 16-row tiles, padded to whole 32-row steps
  bf16* Qs = lds;
  bf16* Ks = Qs + nt_max * 512;
  bf16* Vs = Ks + nt_max * 512;
  bf16* Gs = Vs + nt_max * 512;
  float* lse_s = reinterpret_cast<float*>(Gs + nt_max * 512);
  float* d_s = lse_s + nt_max * 16;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  // element t of this row: packed row base + t * step
  const int64_t base = p.axis == 0 ? cu + (int64_t)r * n : cu + r;
  const int64_t step = p.axis == 0 ? 1 : n;

  // ---- copy the row's four operands; tiles up to nt2, rows past N repeat row N - 1
  {
    const int hD = h * kD, row16 = l16 ^ ((g & 1) << 3);
    for (int t = wave; t < nt2 * 4; t += NW) {
      const int tile = t >> 2, which = t & 3;
      const int64_t row = base + (int64_t)min(tile * 16 + row16, n - 1) * step;
      const bf16* src = (which == 0 ? p.q : which == 1 ? p.k : which == 2 ? p.v : p.dout) +
                        row * (which == 3 ? p.ld_dout : p.ld_qkv) + hD + g * 8;
      bf16* dst = lds + (which * nt_max + tile) * 512;
      __builtin_amdgcn_global_load_lds((const void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();

  const int fo = frag_offset(l16, g);
  const uint32_t to = tr_offset(l16, g);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const int kti = ((n + 63) >> 6) * 4;
  const int64_t img0 = IMG ? ((int64_t)h * p.img_tiles + uni(p.bias_tiles[i])) * 64 : 0;

  // bias of the two tiles (a, b), (a, b + 1): values of lane (l16, g), -inf
  // outside the sample.  BYQ: query 16 a + l16, keys 16 b + 4 g + e; else
  // key 16 a + l16, queries 16 b + 4 g + e.
  auto bias8 = [&](bool byq, int a, int b, float (&out)[8]) {
    if constexpr (IMG) {
      const uint2* img = (byq ? p.img_q : p.img_k) + img0 + ((int64_t)a * kti + b) * 64;
      const uint2 u[2] = {img[(uint32_t)lane], img[(uint32_t)lane + 64]};
#pragma unroll
      for (int w = 0; w < 2; ++w) {
        out[4 * w] = __uint_as_float(u[w].x << 16);
        out[4 * w + 1] = __uint_as_float(u[w].x & 0xffff0000u);
        out[4 * w + 2] = __uint_as_float(u[w].y << 16);
        out[4 * w + 3] = __uint_as_float(u[w].y & 0xffff0000u);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int ai = 16 * a + l16, bi = 16 * (b + (e >> 2)) + 4 * g + (e & 3);
        out[e] = -INFINITY;
        if (ai < n && bi < n) out[e] = byq ? bias_at(p, cu, n, ai, bi, h) : bias_at(p, cu, n, bi, ai, h);
      }
    }
  };

  // ---- phase A: statistics and dQ, a wave per 16 queries
  for (int qt = wave; qt < nt; qt += NW) {
    const bf16x8 qf = frag(Qs, qt, fo), gf = frag(Gs, qt, fo);
    const int j = qt * 16 + l16;
    // every lane runs its own maximum over its keys (4 g + e of each tile)
    float m = -INFINITY, l = 0.f, acc = 0.f;
    for (int kt = 0; kt < nt2; kt += 2) {
      const f32x4 s0 = mfma16(frag(Ks, kt, fo), qf, zero), s1 = mfma16(frag(Ks, kt + 1, fo), qf, zero);
      const f32x4 d0 = mfma16(frag(Vs, kt, fo), gf, zero), d1 = mfma16(frag(Vs, kt + 1, fo), gf, zero);
      float b[8];
      bias8(true, qt, kt, b);
      float sv[8], mx = m;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sv[e] = fmaf(e < 4 ? s0[e & 3] : s1[e & 3], p.scale, b[e]);
        mx = fmaxf(mx, sv[e]);
      }
      const float ms = mx == -INFINITY ? 0.f : mx;       // nothing but masked keys so far: every weight 0
      const float c = exp_native(m - ms);
      l *= c;
      acc *= c;
      m = mx;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float w = exp_native(sv[e] - ms);
        l += w;
        acc = fmaf(w, e < 4 ? d0[e & 3] : d1[e & 3], acc);
      }
    }
    const float mm = max_over_kgroups(m);
    const float c = m == -INFINITY ? 0.f : exp_native(m - mm);
    l = sum_over_kgroups(l * c);
    acc = sum_over_kgroups(acc * c);
    const float ls = mm + __logf(l), ds = acc / l;
    if (g == 0) {
      const bool ok = j < n;
      lse_s[j] = ok ? ls : 0.f;                          // queries past N weigh nothing in phase B
      d_s[j] = ok ? ds : 0.f;
      if (ok) {
        const int64_t at = (int64_t)h * p.cells + cu + (int64_t)r * n + j;
        p.lse[at] = ls;
        p.dsum[at] = ds;
      }
    }
    // dQ^T += K^T dS^T
    f32x4 dq[2] = {zero, zero};
    for (int kt = 0; kt < nt2; kt += 2) {
      const f32x4 s0 = mfma16(frag(Ks, kt, fo), qf, zero), s1 = mfma16(frag(Ks, kt + 1, fo), qf, zero);
      const f32x4 d0 = mfma16(frag(Vs, kt, fo), gf, zero), d1 = mfma16(frag(Vs, kt + 1, fo), gf, zero);
      float b[8], dsv[8];
      bias8(true, qt, kt, b);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float pr = exp_native(fmaf(e < 4 ? s0[e & 3] : s1[e & 3], p.scale, b[e]) - ls);
        dsv[e] = pr * ((e < 4 ? d0[e & 3] : d1[e & 3]) - ds);
      }
      bf16x8 part[3], kf[2];
      split3(dsv, part);
      tr_frags(Ks, kt, to, kf);
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        dq[0] = mfma16(kf[0], part[t], dq[0]);
        dq[1] = mfma16(kf[1], part[t], dq[1]);
      }
    }
    store_rows(p.dq + (base + (int64_t)j * step) * p.ld_dqkv + h * kD, j < n, g, dq, p.scale);
  }
  if (nt2 > nt && threadIdx.x < 16) {                     // the padded tile's statistics
    lse_s[nt * 16 + threadIdx.x] = 0.f;
    d_s[nt * 16 + threadIdx.x] = 0.f;
  }
  __syncthreads();

  // ---- phase B: dK and dV, a wave per 16 keys
  for (int kt = wave; kt < nt; kt += NW) {
    const bf16x8 kf = frag(Ks, kt, fo), vf = frag(Vs, kt, fo);
    f32x4 dk[2] = {zero, zero}, dv[2] = {zero, zero};
    for (int qt = 0; qt < nt2; qt += 2) {
      const f32x4 s0 = mfma16(frag(Qs, qt, fo), kf, zero), s1 = mfma16(frag(Qs, qt + 1, fo), kf, zero);
      const f32x4 d0 = mfma16(frag(Gs, qt, fo), vf, zero), d1 = mfma16(frag(Gs, qt + 1, fo), vf, zero);
      float b[8], pr[8], dsv[8];
      bias8(false, kt, qt, b);
      const float4 la = *reinterpret_cast<const float4*>(lse_s + qt * 16 + 4 * g);
      const float4 lb = *reinterpret_cast<const float4*>(lse_s + qt * 16 + 16 + 4 * g);
      const float4 da = *reinterpret_cast<const float4*>(d_s + qt * 16 + 4 * g);
      const float4 db = *reinterpret_cast<const float4*>(d_s + qt * 16 + 16 + 4 * g);
      const float ls[8] = {la.x, la.y, la.z, la.w, lb.x, lb.y, lb.z, lb.w};
      const float dd[8] = {da.x, da.y, da.z, da.w, db.x, db.y, db.z, db.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        pr[e] = exp_native(fmaf(e < 4 ? s0[e & 3] : s1[e & 3], p.scale, b[e]) - ls[e]);
        dsv[e] = pr[e] * ((e < 4 ? d0[e & 3] : d1[e & 3]) - dd[e]);
      }
      bf16x8 part[3], tf[2];
      split3(dsv, part);
      tr_frags(Qs, qt, to, tf);
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        dk[0] = mfma16(tf[0], part[t], dk[0]);
        dk[1] = mfma16(tf[1], part[t], dk[1]);
      }
      split3(pr, part);
      tr_frags(Gs, qt, to, tf);
#pragma unroll
      for (int t = 0; t < 3; ++t) {
        dv[0] = mfma16(tf[0], part[t], dv[0]);
        dv[1] = mfma16(tf[1], part[t], dv[1]);
      }
    }
    const int key = kt * 16 + l16;
    const int64_t at = (base + (int64_t)key * step) * p.ld_dqkv + h * kD;
    store_rows(p.dk + at, key < n, g, dk, p.scale);
    store_rows(p.dv + at, key < n, g, dv, 1.f);
  }
}

// Bias gradient: workgroup = (sample, head, 64 queries, 64 keys), 8 waves of
// 16 x 32 sums each.  It walks all pair rows; a row's 64 q, dO, k and v rows
// (16 KB) and softmax statistics are copied into one of kBiasStages LDS
// stages, kBiasStages - 1 rows ahead, with one barrier per row.  The blocks of
// all samples are cut into eight equal stretches, one per XCD, head after head,
// so the rows that the workgroups of an XCD walk together come from its own
// L2, and a batch launches the blocks that it has (the longest sample's number
// for every sample took 239 us instead of 224 at B=8, N 66..317, 4 heads, and
// passed a launch's limit on batches of one long and thousands of short ones).
// The texture-address unit bounds it (each copy instruction gathers 16 rows of
// 64 bytes), so operands are shared by 64 x 64 blocks: a wave loading
// its own 16 x 64 block straight into registers took 761 us at B=8,
// N 66..317, 4 heads (2.5 KB per 256 scores instead of 1 KB, and every row's
// latency exposed).  With room for partial sums a workgroup walks
// kBiasChunk rows only and bias_grad_sum_kernel adds the chunks in order:
// walking all N rows, the workgroups of an XCD drift apart and each fetches
// its rows past the L2 again (12 M misses, 358 us at the same sizes).
constexpr int kBiasBlk = 64, kBiasStages = 3, kBiasChunk = 64;
constexpr int kBiasStageBytes = 16 * 1024 + 512;          // 4 tiles each of q, dO, k, v; 64 lse, 64 D

__device__ __forceinline__ void wait_vm(int left) {
  // at most `left` vector-memory operations outstanding (the other counters free)
  switch (left) {
    case 0: __builtin_amdgcn_s_waitcnt(0x0F70); break;
    case 2: __builtin_amdgcn_s_waitcnt(0x0F72); break;
    case 3: __builtin_amdgcn_s_waitcnt(0x0F73); break;
  }
}

__global__ void __launch_bounds__(512, 4) attn_bwd_bias_kernel(AttnBwdArgs p, int chunk, float* partial) {
  __shared__ __attribute__((aligned(16))) unsigned char stages[kBiasStages * kBiasStageBytes];
  // item x S + k of head h runs on XCD x: equal stretches of the samples' (row
  // chunk, query block, key block) lists, numbered for one chunk per 64 rows
  const int total = p.cu_bgrad[p.batch], per = (total + kXcds - 1) / kXcds;
  const uint32_t id = block_id(), t0 = id / kXcds;
  const int h = uni(t0 / per), slot = uni(t0 - h * per), item = (int)(id % kXcds) * per + slot;
  if (h >= p.H || item >= total) return;
  int lo = 0, hi = p.batch - 1;                           // sample: largest i with cu_bgrad[i] <= item
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (p.cu_bgrad[mid] <= item) lo = mid; else hi = mid - 1;
  }
  const int i = uni(lo);
  const int n = uni(p.cu_seqlens[i + 1] - p.cu_seqlens[i]);
  const int nq = (n + kBiasBlk - 1) / kBiasBlk;
  const int li = uni(item - p.cu_bgrad[i]), rc = uni(li / (nq * nq));
  if (rc * chunk >= n) return;                            // chunks of more than 64 rows: fewer of them
  const int qk = li - rc * nq * nq, qb = uni(qk / nq);
  const int j0 = qb * kBiasBlk, k0 = (qk - qb * nq) * kBiasBlk;
  const int r_first = rc * chunk, r_end = min(n, r_first + chunk);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int64_t cu = uni(p.cu_pairs[i]);
  const int64_t step = p.axis == 0 ? 1 : n, rstep = p.axis == 0 ? n : 1;

  // copies of this wave: tiles 2 w, 2 w + 1 of [q 0-3 | dO 4-7 | k 8-11 | v 12-15],
  // rows past N repeat row N - 1 (their sums are not stored); waves 0 and 1
  // also copy the 64 queries' lse and D
  const int which = wave >> 1;
  const int64_t ld = which == 1 ? p.ld_dout : p.ld_qkv;
  const bf16* src = (which == 0 ? p.q : which == 1 ? p.dout : which == 2 ? p.k : p.v) + h * kD + g * 8;
  const int first = (which < 2 ? j0 : k0) + (wave & 1) * 32 + (l16 ^ ((g & 1) << 3));
  const bf16* s0 = src + (cu + (int64_t)min(first, n - 1) * step) * ld;
  const bf16* s1 = src + (cu + (int64_t)min(first + 16, n - 1) * step) * ld;
  const int64_t rld = rstep * ld;
  const float* stat = (wave == 0 ? p.lse : p.dsum) + (int64_t)h * p.cells + cu + min(j0 + lane, n - 1);
  auto copy_row = [&](int r, int stage) {
    unsigned char* st = stages + stage * kBiasStageBytes;
    unsigned char* dst = st + wave * 2048;
    __builtin_amdgcn_global_load_lds((const void*)(s0 + r * rld), (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
    __builtin_amdgcn_global_load_lds((const void*)(s1 + r * rld), (__attribute__((address_space(3))) void*)(dst + 1024), 16, 0, 0);
    if (wave < 2)
      __builtin_amdgcn_global_load_lds((const void*)(stat + (int64_t)r * n),
                                       (__attribute__((address_space(3))) void*)(st + 16384 + wave * 256), 4, 0, 0);
  };

  // this wave's sums: queries j0 + 16 qw + l16, keys k0 + 32 kw + 16 t + 4 g + e
  const int qw = wave >> 1, kw = wave & 1;
  const int j = j0 + 16 * qw + l16, kk = k0 + 32 * kw + 4 * g;
  float b[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) b[t][e] = j < n && kk + 16 * t + e < n ? bias_at(p, cu, n, j, kk + 16 * t + e, h) : 0.f;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 acc[2] = {zero, zero};
  const uint32_t lds0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)stages;
  const uint32_t fo = frag_offset(l16, g) * 2;
  const uint32_t aq = lds0 + qw * 1024 + fo, ak = lds0 + 8192 + kw * 2048 + fo, as = lds0 + 16384 + (16 * qw + l16) * 4;

  // the first kBiasStages - 1 rows in flight; copies past the last row repeat
  // it, so every wave always has the same number outstanding
  __builtin_amdgcn_s_waitcnt(0x0F70);                     // the bias loads: only copies are counted below
#pragma unroll
  for (int r = 0; r < kBiasStages - 1; ++r) copy_row(min(r_first + r, r_end - 1), r);
  int stage = 0;
  for (int r = r_first; r < r_end; ++r) {
    // this wave's copies of row r have landed (those of row r + 1 may be in
    // flight); past the barrier everyone's have, and row r - 1's stage is free
    static_assert(kBiasStages == 3, "one later row in flight");
    wait_vm(wave < 2 ? 3 : 2);
    __builtin_amdgcn_s_barrier();
    const int next = stage == 0 ? kBiasStages - 1 : stage - 1;
    copy_row(min(r + kBiasStages - 1, r_end - 1), next);
    uint4 f[6];
    float ls, ds;
    const uint32_t so = stage * kBiasStageBytes;
    asm volatile(
        "ds_read_b128 %0, %8\n"
        "ds_read_b128 %1, %9\n"
        "ds_read_b128 %2, %8 offset:4096\n"
        "ds_read_b128 %3, %9 offset:4096\n"
        "ds_read_b128 %4, %9 offset:1024\n"
        "ds_read_b128 %5, %9 offset:5120\n"
        "ds_read_b32 %6, %10\n"
        "ds_read_b32 %7, %10 offset:256\n"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(ls), "=&v"(ds)
        : "v"(aq + so), "v"(ak + so), "v"(as + so)
        : "memory");
    const bf16x8 qf = __builtin_bit_cast(bf16x8, f[0]), gf = __builtin_bit_cast(bf16x8, f[2]);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const f32x4 s = mfma16(__builtin_bit_cast(bf16x8, f[t ? 4 : 1]), qf, zero);
      const f32x4 d = mfma16(__builtin_bit_cast(bf16x8, f[t ? 5 : 3]), gf, zero);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc[t][e] = fmaf(exp_native(fmaf(s[e], p.scale, b[t][e]) - ls), d[e] - ds, acc[t][e]);
    }
    stage = stage == kBiasStages - 1 ? 0 : stage + 1;
  }
  __builtin_amdgcn_s_waitcnt(0);                          // no copy into LDS outlives the workgroup
  if (j >= n) return;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = kk + 16 * t + e;
      if (k >= n) continue;
      const int64_t cell = cu + (p.axis == 0 ? (int64_t)j * n + k : (int64_t)k * n + j);
      if (partial) partial[((int64_t)rc * p.H + h) * p.cells + cell] = acc[t][e];
      else p.dbias[cell * p.ld_dbias + (int64_t)h * p.ld_dbias_head] = acc[t][e];
    }
}

// Sums the row chunks' partials of every cell and head in chunk order.
__global__ void __launch_bounds__(256) bias_grad_sum_kernel(AttnBwdArgs p, int chunk, const float* partial) {
  const int64_t cell = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (cell >= p.cells) return;
  int lo = 0, hi = p.batch - 1;                           // sample: largest i with cu_pairs[i] <= cell
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (p.cu_pairs[mid] <= cell) lo = mid; else hi = mid - 1;
  }
  const int n = p.cu_seqlens[lo + 1] - p.cu_seqlens[lo], nc = (n + chunk - 1) / chunk, h = blockIdx.y;
  float s = 0.f;
  for (int c = 0; c < nc; ++c) s += partial[((int64_t)c * p.H + h) * p.cells + cell];
  p.dbias[cell * p.ld_dbias + (int64_t)h * p.ld_dbias_head] = s;
}

template <int NW>
hipError_t launch_rows(const AttnBwdArgs& a, int nt_max, size_t smem, hipStream_t s) {
  const void* fn = a.img_q ? (const void*)attn_bwd_rows_kernel<NW, true> : (const void*)attn_bwd_rows_kernel<NW, false>;
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  const dim3 grid = folded_grid(a.row_blocks);
  if (a.img_q) attn_bwd_rows_kernel<NW, true><<<grid, dim3(64 * NW), smem, s>>>(a, nt_max);
  else attn_bwd_rows_kernel<NW, false><<<grid, dim3(64 * NW), smem, s>>>(a, nt_max);
  return hipGetLastError();
}

// bytes of the softmax statistics, rounded up so that the bias images behind
// them are aligned
size_t stats_bytes(const nt_layout& L, int H) { return 2 * (size_t)L.sum_n2 * (size_t)H * sizeof(float); }
size_t images_offset(const nt_layout& L, int H) { return (stats_bytes(L, H) + 255) / 256 * 256; }
int bias_chunks(const nt_layout& L) { return (L.max_len + kBiasChunk - 1) / kBiasChunk; }

}  // namespace

size_t attention_backward_min_workspace_bytes(const nt_layout& L, int H) { return stats_bytes(L, H); }

size_t attention_backward_workspace_bytes(const nt_layout& L, int H) {
  if (L.sum_n2 == 0) return 0;
  return images_offset(L, H) + 2 * bias_image_bytes(L, H) + (size_t)bias_chunks(L) * H * L.sum_n2 * sizeof(float);
}

hipError_t launch_attention_backward(const nt_layout& L, int axis, int H, const void* q, const void* k,
                                     const void* v, int64_t ld_qkv, const void* bias, int64_t ld_bias,
                                     int64_t ld_bias_head, const void* dout,
                                     int64_t ld_dout, float scale, void* dq, void* dk, void* dv, int64_t ld_dqkv,
                                     float* dbias, int64_t ld_dbias, int64_t ld_dbias_head, void* workspace,
                                     size_t workspace_bytes, hipStream_t s) {
  if (L.attn_items() == 0) return hipSuccess;
  float* lse = static_cast<float*>(workspace);
  AttnBwdArgs a{axis, H, (const bf16*)q, (const bf16*)k, (const bf16*)v, ld_qkv, (const bf16*)bias, ld_bias,
                ld_bias_head, (const bf16*)dout, ld_dout, scale, (bf16*)dq, (bf16*)dk,
                (bf16*)dv, ld_dqkv, dbias, ld_dbias, ld_dbias_head, lse, lse + L.sum_n2 * H, L.sum_n2, L.d_attn_work,
                (uint32_t)(L.attn_items() * H), L.d_cu_seqlens, L.d_cu_pairs, nullptr, nullptr, L.bias_tiles_total(), L.d_bias_tiles,
                L.d_cu_bgrad, L.batch};
  // A workspace of the full size also holds two bias images, so that both
  // phases read the bias as whole 512-byte tiles, and the bias gradient's
  // partial sums; with one of the minimum size (statistics only) every score
  // gathers its own two bytes and a workgroup walks all pair rows.
  const bool full = workspace_bytes >= attention_backward_workspace_bytes(L, H);
  if (bias && full) {
    char* img = static_cast<char*>(workspace) + images_offset(L, H);
    a.img_q = reinterpret_cast<const uint2*>(img);
    a.img_k = reinterpret_cast<const uint2*>(img + bias_image_bytes(L, H));
    hipError_t e = launch_bias_image(L, axis, H, bias, ld_bias, ld_bias_head, 1.f, kMaxBf16, (void*)a.img_q, s);
    // by keys: the image of the transposed bias
    if (e == hipSuccess) e = launch_bias_image(L, 1 - axis, H, bias, ld_bias, ld_bias_head, 1.f, kMaxBf16, (void*)a.img_k, s);
    if (e != hipSuccess) return e;
  }
  const int nt_max = (L.max_len + 31) / 32 * 2;
  const size_t smem = (size_t)nt_max * (4 * 1024 + 2 * 16 * sizeof(float));
  // Waves per workgroup: as many as keep four waves on each SIMD with the
  // workgroups that fit a CU's 160 KB of LDS, and no more than the tiles.
  hipError_t e = nt_max <= 8 ? launch_rows<4>(a, nt_max, smem, s)
                 : smem <= 80 * 1024 ? launch_rows<8>(a, nt_max, smem, s)
                                     : launch_rows<16>(a, nt_max, smem, s);
  if (e != hipSuccess || !dbias) return e;
  const int chunk = full ? kBiasChunk : kAttnLongLen, nc = (L.max_len + chunk - 1) / chunk;
  float* partial = nc > 1 ? reinterpret_cast<float*>(static_cast<char*>(workspace) + images_offset(L, H) + 2 * bias_image_bytes(L, H))
                          : nullptr;
  static_assert(kBiasBlk == kBgradBlock && kBiasChunk == kBgradBlock, "cu_bgrad counts blocks of 64 queries, keys and rows");
  const int64_t blocks = (int64_t)(L.cu_bgrad.back() + kXcds - 1) / kXcds * kXcds * H;
  attn_bwd_bias_kernel<<<folded_grid(blocks), dim3(512), 0, s>>>(a, chunk, partial);
  e = hipGetLastError();
  if (e != hipSuccess || !partial) return e;
  bias_grad_sum_kernel<<<dim3((unsigned)((L.sum_n2 + 255) / 256), (unsigned)H), dim3(256), 0, s>>>(a, chunk, partial);
  return hipGetLastError();
}

}  // namespace nt
