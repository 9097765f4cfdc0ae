// Segmented softmax attention over packed buffers, one launch for the batch.
//
// A segment is one pair row (axis 0: cells (i, r, *)), one pair column
// (axis 1: cells (i, *, r)) or one sample's tokens (axis 2).  The workgroup
// for (segment, head) stages the segment's keys and transposed values in LDS
// once; each wave then runs 16-query tiles through an online softmax over
// 64-key chunks on matrix cores:
//   S^T = K Q^T       lane (g, q) holds scores of keys 16t + 4g + i for query q,
//                     so the running max/sum of a query live in one lane column
//   O^T += V^T P^T    P is taken from the S^T registers as the B operand
//                     (keys {4g..4g+3} of two 16-key tiles), no shuffles.
#include <algorithm>
#include <type_traits>

#include <mutex>

#include "nt_device.h"
#include "nt_internal.h"

namespace nt {
namespace {

constexpr float kLog2e = 1.4426950408889634f;

struct AttnArgs {
  int axis, H;
  const bf16* q;
  const bf16* k;
  const bf16* v;
  int64_t ld_qkv;
  const bf16* bias;
  int64_t ld_bias, ld_bias_head;  // element (cell c, head h) at c * ld_bias + h * ld_bias_head
  float scale_log2;      // softmax scale * log2(e)
  bf16* o;
  int64_t ld_o;
  const int32_t* work;   // (sample, row) or (sample, query block) pairs
  const int32_t* cu_seqlens;
  const int32_t* cu_pairs;
  int vstride;           // LDS row stride of V^T (elements)
  const bf16* gate;      // NULL, or o = sigmoid(gate) * attention (gate row stride ld_gate)
  int64_t ld_gate;
};

struct Seg {
  int n;                 // keys in the segment
  int64_t base, step;    // packed row of element t: base + t * step
  int q_begin, q_end;
  int64_t cu;            // pair offset of the sample (bias addressing)
  int sample;
};

template <typename A>
__device__ __forceinline__ bool segment_of(const A& p, Seg& s) {
  const int i = p.work[2 * blockIdx.x], r = p.work[2 * blockIdx.x + 1];
  if (i < 0) return false;
  s.sample = i;
  if (p.axis == 2) {
    s.n = p.cu_seqlens[i + 1] - p.cu_seqlens[i];
    s.base = p.cu_seqlens[i];
    s.step = 1;
    s.q_begin = r * kSeqQBlock;
    s.q_end = min(s.n, s.q_begin + kSeqQBlock);
    s.cu = 0;
  } else {
    s.n = p.cu_seqlens[i + 1] - p.cu_seqlens[i];
    s.cu = p.cu_pairs[i];
    s.base = p.axis == 0 ? s.cu + (int64_t)r * s.n : s.cu + r;
    s.step = p.axis == 0 ? 1 : s.n;
    s.q_begin = 0;
    s.q_end = s.n;
  }
  return true;
}

template <int D>
__global__ void __launch_bounds__(256) attention_mfma_kernel(AttnArgs p) {
  extern __shared__ __attribute__((aligned(16))) bf16 lds[];
  constexpr int KS = D + 8;                    // LDS stride of K rows (bf16)
  constexpr int DV = D / 8;                    // 16-byte vectors per head row
  Seg sg;
  if (!segment_of(p, sg)) return;
  const int h = blockIdx.y;
  const int n = sg.n;
  const int npad = (n + 63) & ~63;
  bf16* Ks = lds;                              // [npad][KS]
  bf16* Vt = lds + (size_t)npad * KS;          // [D][vstride]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;

  // ---- stage keys (row-major) and values (transposed) of this head -------
  for (int c = tid; c < npad * DV; c += 256) {
    const int key = c / DV, dc = (c % DV) * 8;
    uint4 kk = make_uint4(0, 0, 0, 0), vv = make_uint4(0, 0, 0, 0);
    if (key < n) {
      const int64_t row = sg.base + (int64_t)key * sg.step;
      kk = *reinterpret_cast<const uint4*>(p.k + row * p.ld_qkv + h * D + dc);
      vv = *reinterpret_cast<const uint4*>(p.v + row * p.ld_qkv + h * D + dc);
    }
    *reinterpret_cast<uint4*>(&Ks[key * KS + dc]) = kk;
    const bf16x8 vb = *reinterpret_cast<const bf16x8*>(&vv);
#pragma unroll
    for (int j = 0; j < 8; ++j) Vt[(dc + j) * p.vstride + key] = vb[j];
  }
  __syncthreads();

  for (int qt = sg.q_begin / 16 + wave; qt * 16 < sg.q_end; qt += 4) {
    const int qi = qt * 16 + l16;
    const bool qvalid = qi < sg.q_end;
    const int64_t qrow = sg.base + (int64_t)qi * sg.step;
    bf16x8 qf[D / 32];
#pragma unroll
    for (int dd = 0; dd < D / 32; ++dd) {
      if (qvalid) qf[dd] = *reinterpret_cast<const bf16x8*>(p.q + qrow * p.ld_qkv + h * D + dd * 32 + g * 8);
      else qf[dd] = bf16x8{};
    }
    float m_run = -INFINITY, l_run = 0.f;
    f32x4 O[D / 16];
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16* brow = nullptr;                // bias row of this query (axis 0)
    if (p.bias && qvalid)
      brow = p.bias + (int64_t)h * p.ld_bias_head + (sg.cu + (p.axis == 0 ? (int64_t)qi * n : qi)) * p.ld_bias;
    const int64_t bstep = (p.axis == 0 ? 1 : n) * p.ld_bias;

    for (int kc = 0; kc < npad; kc += 64) {
      f32x4 s[4];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) {
        s[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dd = 0; dd < D / 32; ++dd) {
          const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Ks[(kc + kt * 16 + l16) * KS + dd * 32 + g * 8]);
          s[kt] = mfma16(kf, qf[dd], s[kt]);
        }
      }
      float x[4][4];
      float mloc = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int key = kc + kt * 16 + 4 * g + i;
          float t = s[kt][i] * p.scale_log2;
          if (brow && key < n) t += (float)brow[(int64_t)key * bstep] * kLog2e;
          t = key < n ? t : -INFINITY;
          x[kt][i] = t;
          mloc = fmaxf(mloc, t);
        }
      mloc = fmaxf(mloc, __shfl_xor(mloc, 16, 64));
      mloc = fmaxf(mloc, __shfl_xor(mloc, 32, 64));
      const float m_new = fmaxf(m_run, mloc);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) O[dt] *= alpha;
      bf16x8 pf[2];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float e = __builtin_amdgcn_exp2f(x[kt][i] - m_new);
          l_run += e;
          pf[kt >> 1][(kt & 1) * 4 + i] = (bf16)e;
        }
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt)
#pragma unroll
        for (int pp = 0; pp < 2; ++pp) {
          const bf16* vr = &Vt[(dt * 16 + l16) * p.vstride + kc + pp * 32 + 4 * g];
          const bf16x4 lo = *reinterpret_cast<const bf16x4*>(vr);
          const bf16x4 hi = *reinterpret_cast<const bf16x4*>(vr + 16);
          const bf16x8 vf = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          O[dt] = mfma16(vf, pf[pp], O[dt]);
        }
    }
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    if (qvalid) {
      const float inv = 1.f / l_run;
      bf16* orow = p.o + qrow * p.ld_o + h * D;
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) {
        bf16x4 ov;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float val = O[dt][i] * inv;
          if (p.gate) {
            const float gl = (float)p.gate[qrow * p.ld_gate + h * D + dt * 16 + 4 * g + i];
            val *= __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-gl * kLog2e));
          }
          ov[i] = (bf16)val;
        }
        *reinterpret_cast<bf16x4*>(orow + dt * 16 + 4 * g) = ov;
      }
    }
  }
}

// ---------------------------------------------------------------- pair attention arguments
struct PairAttnArgs {
  int axis;
  const bf16* q;
  const bf16* k;
  const bf16* v;
  int64_t ld_qkv;
  const bf16* bias;
  int64_t ld_bias, ld_bias_head;
  float scale_log2;
  bf16* o;
  int64_t ld_o;
  const int32_t* work;   // axis 3: quads (sample, first 16-query tile, 0, tile count); row kernel: (sample, row) pairs
  const int32_t* cu_seqlens;
  const int32_t* cu_pairs;
  int H;                 // heads (interleaved in the grid)
  const uint2* bias_img; // bias image (see bias_image_kernel) or NULL for no bias
  int64_t img_head;      // uint2 entries per head of the image
  const int32_t* bias_tiles;
  int batch;             // samples (persistent instance: rows are found from cu_short and cu_cost)
  const int32_t* cu_short;   // persistent instance: prefix of the short samples' rows and of their cost
  const int64_t* cu_cost;
  int64_t total_cost;
  const bf16* gate;      // gated output: o = sigmoid(gate) * attention, gate [rows, >= H*D] (GATE instances)
  int64_t ld_gate;
};

// Pair bias image: for head h, sample i, 16-query tile qt and 16-key tile kt
// (kt < round_up(N_i,64)/16), lane l = l16 + 16 g of tile
// ((h * T + bias_tiles[i] + qt * KT_i + kt) holds the four values
// bias(j, k) * mul, j = 16 qt + l16, k = 16 kt + 4 g .. +3, each rounded to
// bf16 -- exactly the register image the attention lanes keep.  Finite values
// stay within +-limit, so a finite mask is still finite where it is multiplied
// (by mul here or in fp32 later); infinities and NaN pass.  A wave looks at its
// values one by one only if one is past `far`: checking each took 15.0 us
// instead of 14.1 at 12 heads, N 32..512, B = 8.  Keys past N hold
// -inf (for queries inside N), so the scores they seed are masked without
// further work; queries past N hold 0.
// bias(j, k) is the head-h bias of cell(j, k) for axis 0 and of cell(k, j)
// for axis 1, read at cell * ld_bias + h * ld_bias_head; the sample is found by
// bisection.
struct BiasImgArgs {
  int axis, batch;
  const bf16* bias;
  int64_t ld_bias, ld_bias_head;
  float mul, limit;
  float far;              // values up to this size are within the limit once multiplied
  uint2* img;
  int64_t tiles;          // tiles per head
  const int32_t* bias_tiles;
  const int32_t* cu_seqlens;
  const int32_t* cu_pairs;
};

// One wave per U (1 or 4) key tiles of a query tile (the tile count of a sample
// is a multiple of four).  Where the keys of a query are adjacent (axes 0 and 3,
// unit cell stride) a lane reads its four values at once, at whatever 2-byte
// boundary they start: 12 heads of N 32..512, B = 8 took 27 us value by value.
template <int U>
__global__ void __launch_bounds__(256) bias_image_kernel(BiasImgArgs p) {
  const int64_t tile = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * U;
  if (tile >= p.tiles) return;
  const int h = blockIdx.y, lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  int lo = 0, hi = p.batch - 1;                 // sample: largest i with bias_tiles[i] <= tile
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (p.bias_tiles[mid] <= tile) lo = mid; else hi = mid - 1;
  }
  const int i = __builtin_amdgcn_readfirstlane(lo);
  const int n = p.cu_seqlens[i + 1] - p.cu_seqlens[i];
  const int kti = ((n + 63) >> 6) * 4;
  const int t = (int)(tile - p.bias_tiles[i]);
  const int j = (t / kti) * 16 + l16, kt0 = (t % kti) * 16 + 4 * g;
  const bf16* bh = p.bias + (int64_t)h * p.ld_bias_head + (int64_t)p.cu_pairs[i] * p.ld_bias;
  const bool adjacent = p.axis != 1 && p.ld_bias == 1;
  bf16x4 raw[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int k0 = kt0 + 16 * u;
    raw[u] = bf16x4{};
    if (adjacent && j < n && k0 + 4 <= n) {
      __builtin_memcpy(&raw[u], bh + (int64_t)j * n + k0, 8);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = k0 + e;
        if (j < n && k < n) raw[u][e] = bh[(p.axis != 1 ? (int64_t)j * n + k : (int64_t)k * n + j) * p.ld_bias];
      }
    }
  }
  f32x4 b[U];
  bool far = false;                             // some value may pass the limit
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float v = (float)raw[u][e];
      far |= fabsf(v) > p.far;
      b[u][e] = v * p.mul;
    }
  if (__builtin_expect(__any(far), 0)) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if ((__builtin_bit_cast(uint16_t, (bf16)raw[u][e]) & 0x7f80) != 0x7f80) b[u][e] = fminf(fmaxf(b[u][e], -p.limit), p.limit);
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    bf16x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (bf16)(j >= n ? 0.f : kt0 + 16 * u + e < n ? b[u][e] : -INFINITY);
    *reinterpret_cast<bf16x4*>(&p.img[(int64_t)h * p.tiles * 64 + (tile + u) * 64 + lane]) = o;
  }
}

// ---------------------------------------------------------------- shared pieces
// Value rows of 32 dims (64 bytes) staged row-major, the 16-byte piece at
// column c of key row kv holding dim group c ^ ((kv >> 2) & 3) (so the four
// key groups of a transposed read fall on different banks).  Fragments for
// O^T += V^T P^T: lane (dim 16 dt + l16, k-group g) needs keys 32 kb +
// {4g..4g+3, 16+4g..16+4g+3}.  ds_read_b64_tr_b16 hands lane 4q+m of each
// 16-lane group element m of the 8-byte pieces addressed by lanes q, q+4,
// q+8, q+12; pointing lane i at key base + i/4, dims 16 dt + 4 (i%4)
// therefore delivers 4 consecutive keys of dim l16.  Key blocks are 2 KB
// apart and keys kk, kk + 16 share (kk >> 2) & 3 = g, so every read of a lane
// uses the same swizzled column.  The reads of one or two key blocks are
// issued together from inline assembly with their own wait: the compiler
// cannot tell them apart from global->LDS copies in flight into other
// buffers and would otherwise wait for those first.
struct VtLane {
  uint32_t a0, a1;       // byte offsets in a value buffer, key block 0: dims 4q.., 16 + 4q..
};
__device__ __forceinline__ VtLane vt_lane(int l16, int g) {
  const int kk = 4 * g + (l16 >> 2), q = l16 & 3;
  return VtLane{(uint32_t)((kk * 32 + ((q >> 1) ^ g) * 8 + (q & 1) * 4) * 2),
                (uint32_t)((kk * 32 + (((q >> 1) + 2) ^ g) * 8 + (q & 1) * 4) * 2)};
}
__device__ __forceinline__ uint32_t lds_addr(const bf16* ptr) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) bf16*)ptr;
}
// bf16 ones as an MFMA operand, materialised where it is used: kept live
// across the row loop it is one of the first values the register allocator
// spills, and its reload waits for every copy in flight.
__device__ __forceinline__ bf16x8 ones_bf16x8() {
  uint32_t w;
  asm volatile("v_mov_b32 %0, 0x3f803f80" : "=v"(w));
  const uint32_t q[4] = {w, w, w, w};
  return __builtin_bit_cast(bf16x8, q);
}
// an opaque copy of a lane-dependent value: what is derived from it is
// recomputed at each use instead of being hoisted out of the row loop and
// kept live (or spilled) across it
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ bf16x8 pack_u2(uint2 lo, uint2 hi) {
  const uint32_t w[4] = {lo.x, lo.y, hi.x, hi.y};
  return __builtin_bit_cast(bf16x8, w);
}
// one key block: f[0] dims 0-15, f[1] dims 16-31
__device__ __forceinline__ void vt_frags1(const bf16* Vr, int kb, const VtLane& vl, bf16x8 (&f)[2]) {
  const uint32_t base = lds_addr(Vr + kb * 32 * 32), a0 = base + vl.a0, a1 = base + vl.a1;
  uint2 r[4];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %4\n"
      "ds_read_b64_tr_b16 %1, %4 offset:1024\n"
      "ds_read_b64_tr_b16 %2, %5\n"
      "ds_read_b64_tr_b16 %3, %5 offset:1024\n"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
      : "v"(a0), "v"(a1)
      : "memory");
  f[0] = pack_u2(r[0], r[1]);
  f[1] = pack_u2(r[2], r[3]);
}
// two key blocks kb, kb + 1: f[0..1] as above for kb, f[2..3] for kb + 1
__device__ __forceinline__ void vt_frags2(const bf16* Vr, int kb, const VtLane& vl, bf16x8 (&f)[4]) {
  const uint32_t base = lds_addr(Vr + kb * 32 * 32), a0 = base + vl.a0, a1 = base + vl.a1;
  uint2 r[8];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n"
      "ds_read_b64_tr_b16 %1, %8 offset:1024\n"
      "ds_read_b64_tr_b16 %2, %9\n"
      "ds_read_b64_tr_b16 %3, %9 offset:1024\n"
      "ds_read_b64_tr_b16 %4, %8 offset:2048\n"
      "ds_read_b64_tr_b16 %5, %8 offset:3072\n"
      "ds_read_b64_tr_b16 %6, %9 offset:2048\n"
      "ds_read_b64_tr_b16 %7, %9 offset:3072\n"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3]), "=&v"(r[4]), "=&v"(r[5]), "=&v"(r[6]), "=&v"(r[7])
      : "v"(a0), "v"(a1)
      : "memory");
  f[0] = pack_u2(r[0], r[1]);
  f[1] = pack_u2(r[2], r[3]);
  f[2] = pack_u2(r[4], r[5]);
  f[3] = pack_u2(r[6], r[7]);
}
// Values of a pair row staged in LDS, 1 KB per 16 keys: the 16-byte piece
// (key, dims 8 d ..) sits in slot 16 d + (key ^ 8 (d & 1)), so that the pieces
// of a transposed read fall on different banks.  Lane i of a 16-lane group
// points at key 4 g + i/4, dims 4 (i%4) and receives keys 4 g .. 4 g + 3 of dim
// l16 (see vt_lane); dims 16..31 are 512 bytes further on, the next 16 keys
// 1024.  f[0] dims 0-15, f[1] dims 16-31 of 32 keys.
__device__ __forceinline__ uint32_t row_tr_offset(int l16, int g) {
  const int row = 4 * g + (l16 >> 2), d = (l16 & 3) >> 1;
  return (uint32_t)((d * 16 + (row ^ (d << 3))) * 16 + (l16 & 1) * 8);
}
__device__ __forceinline__ void row_tr_frags(uint32_t a, bf16x8 (&f)[2]) {
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
// maximum over the four lanes l16 + 16 g holding one query: the swaps pair
// lane l with l ^ 16, then with l ^ 32, and leave both values in place
__device__ __forceinline__ float query_max(float v) {
  const auto s16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(s16[0]), __uint_as_float(s16[1]));
  const auto s32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(s32[0]), __uint_as_float(s32[1]));
}

// Scores against the reference maximum m: the weight is 2^((S - m) c).  With
// nm = -fl(m c) it takes one fused multiply-add per score, and the rounding
// error of m c, up to 2^-24 of it, scales every weight of the chunk alike: no
// more than the fp32 score's own error, but a power of two that overflows or
// vanishes, and differs between chunks, once |m| is that of a finite mask
// (-1e9 and beyond).  Past kFarMax, and where m is still -inf because every key
// so far is masked, the difference is taken first (against 0 for -inf); a
// chunk's keys pay for it only then.
constexpr float kFarMax = 4096.f;
// factor of the accumulators when the maximum moves from m to m_new
__device__ __forceinline__ float rescale(float m, float m_new, float c) {
  return m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f((m - m_new) * c);
}
// scale log2(e) S + log2(e) bias: the score in log2 units, in fp32
__device__ __forceinline__ f32x4 log2_scores(f32x4 S, float scale_log2, f32x4 bias) {
#pragma unroll
  for (int e = 0; e < 4; ++e) S[e] = fmaf(S[e], scale_log2, bias[e] * kLog2e);
  return S;
}

// ---------------------------------------------------------------- pair attention, head_dim 32
// Pair attention for head_dim 32 and the samples up to kAttnShortLen, organised
// so that the exponentials are nearly the only vector work.  Persistent: one
// workgroup of 16 waves per CU (all queries of a row, so a row's keys and values
// are copied once per CU; 64 KB of LDS, four waves per SIMD) runs a stretch of
// pair rows of one head, an equal share of the rows' cost; longer samples are
// skipped, their rows are attention_row_kernel's.
//   * the bias of (query, key) does not depend on the pair row, so each lane
//     keeps the bias of its query for its 4-key groups of every key tile in
//     registers while the rows belong to one sample, read from the bias
//     image.  Divided by the softmax scale there (one bf16 rounding) it seeds
//     the score accumulators: the matrix cores produce bias/scale + q.k
//     directly.  EXACT instances read the bias itself and form the score in
//     log2 units in fp32 (see attention_row_kernel);
//   * keys and values of a row are copied straight into LDS (keys as fragment
//     images: 64 lanes x 16 bytes, read as one contiguous 1 KB per wave) in
//     two buffers, the next row's copies in flight while the current row
//     runs: one barrier per row;
//   * the softmax denominator comes from one more matrix-core product with a
//     ones operand, on the same bf16 probabilities as the numerator (EXACT:
//     from the fp32 weights, added per lane).
// Scores are kept transposed (S^T = K Q^T), so a lane holds 16 keys of one
// query per 64-key chunk and the running max is mostly lane-local.
template <int NMAX, int NW, bool GATE, bool EXACT>
__global__ void __launch_bounds__(64 * NW, 4) attention_pair_kernel(PairAttnArgs p) {
  constexpr int D = 32;
  constexpr int KT16 = NMAX / 16;               // key tiles
  static_assert(NW * 16 >= NMAX && NMAX <= 256, "a workgroup covers all queries of a row");
  extern __shared__ __attribute__((aligned(16))) bf16 lds[];
  bf16* Kb0 = lds;                                         // key images: tile of 16 keys -> 512 elements
  bf16* Kb1 = Kb0 + NMAX * D;
  bf16* Vb0 = Kb1 + NMAX * D;                              // values, row-major [key][D]
  bf16* Vb1 = Vb0 + NMAX * D;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;

  // ---- rows of this workgroup, [row, row_end) of one head (one workgroup per
  // CU): the rows of all short samples are cut into 8 M slices of equal cost
  // (attn_row_cost, crossing sample boundaries).  XCD x takes the x-th M of
  // them for every head, its workgroup k head k % H and slice k / H, so the
  // heads of a row run on one XCD together.  Rows are counted by rows[], where
  // longer samples have none.  The cuts are rounded once, to the nearest row:
  // cutting the XCDs' shares first and those into slices gave one workgroup 28
  // rows where 27 suffice (B=8, N 208..222).
  const int32_t* rows = p.cu_short;
  const int x = blockIdx.x % kXcds, k = blockIdx.x / kXcds;
  const int h = __builtin_amdgcn_readfirstlane(k % p.H), m = __builtin_amdgcn_readfirstlane(k / p.H);
  const int M = __builtin_amdgcn_readfirstlane((int)(gridDim.x / kXcds) / p.H);   // the grid is a multiple of 8 H
  const int slice = x * M + m;
  // total_cost q / (8 M), in 32 bits where they suffice (a 64-bit division costs about a microsecond)
  auto cost_at = [&](int q) -> int64_t {
    if (p.total_cost * (kXcds * M) < (int64_t(1) << 32)) return (uint32_t)p.total_cost * (uint32_t)q / (uint32_t)(kXcds * M);
    return p.total_cost * q / (kXcds * M);
  };
  // The table entries of the sample at cost t, found by the lanes together: 64
  // entries a step, one step for batches up to 63, and both ends of the slice
  // side by side.  A dependent load is most of a microsecond of a small call: with
  // two bisections the launch took 124 us instead of 122 at B=8, N 208..222, and
  // 112 instead of 110 on the four-block stack's samples.
  struct Window { int lo; int64_t cost; int rows, pairs, tiles; };
  auto window = [&](int64_t t) {
    int lo = 0;
    for (int cnt = p.batch; cnt > 63;) {        // the sample is one of cnt from lo on
      const int step = (cnt + 63) / 64;
      const bool le = lane * step < cnt && p.cu_cost[lo + lane * step] <= t;
      const int j = __popcll(__ballot(le)) - 1;
      lo += j * step;
      cnt = min(step, cnt - j * step);
    }
    const int at = min(lo + lane, p.batch);
    return Window{lo, p.cu_cost[at], rows[at], p.cu_pairs[at], p.bias_tiles[at]};
  };
  // the row boundary nearest to cost t: index r0 of sample i, which has n0 rows
  // counted from first, its cells from cu0 and its image tiles from bt0
  int i, n0, first, r0, cu0, bt0;
  auto row_at = [&](int64_t t, const Window& w) {
    const int j = __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < 63 && w.lo + lane < p.batch && w.cost <= t)) - 1);
    i = w.lo + j;
    first = __builtin_amdgcn_readlane(w.rows, j);
    n0 = __builtin_amdgcn_readlane(w.rows, j + 1) - first;
    cu0 = __builtin_amdgcn_readlane(w.pairs, j);
    bt0 = __builtin_amdgcn_readlane(w.tiles, j);
    // within one sample, whose cost fits 32 bits
    const int c = (int)((uint32_t)t - (uint32_t)__builtin_amdgcn_readlane((int)w.cost, j)) - kAttnSampleCost;
    const uint32_t u = (uint32_t)attn_row_cost(n0);
    r0 = min(n0, (int)(((uint32_t)max(c, 0) + u / 2u) / u));
  };
  const int64_t ta = cost_at(slice), tb = cost_at(slice + 1);
  const Window wa = window(ta), wb = window(tb);
  row_at(tb, wb);
  const int64_t row_end = first + r0;
  row_at(ta, wa);
  int64_t row = first + r0;
  if (row >= row_end) return;
  if (r0 == n0) {                               // the first row of the next non-empty sample
    do ++i; while (rows[i + 1] <= row);
    n0 = rows[i + 1] - (int)row;
    cu0 = p.cu_pairs[i];
    bt0 = p.bias_tiles[i];
    r0 = 0;
  }
  i = __builtin_amdgcn_readfirstlane(i);
  const int jw = 16 * wave + l16;               // this lane's query

  // ---- per-row staging: straight global -> LDS copies ---------------------
  // Each wave copies its key tiles (wave, wave + NW, ...; 16 keys each) with
  // global_load_lds, lane l's 16 bytes landing at byte 16 l of the tile:
  //   keys as fragment images: lane l = (key l%16, dims 8 (l/16) ..),
  //   values row-major [key][32]: lane l = (key l/4, dims 8 (l%4) ..).
  // Every tile below the 64-key padded length is written (the last chunk
  // reads up to there): keys past N repeat key N-1, so the padding holds
  // finite values whose probabilities are masked to zero.
  // this head's queries, keys, values, outputs (and gates): the head offset
  // as a scalar, so the bases stay in scalar registers (global pointers)
  const int hD = __builtin_amdgcn_readfirstlane(h * D);
  const bf16* kbase = p.k + hD;
  const bf16* vbase = p.v + hD;
  const bf16* qbase = p.q + hD;
  bf16* obase = p.o + hD;
  const bf16* gbase = GATE ? p.gate + hD : nullptr;
  auto dma_kv = [&](int sn, int64_t scu, int r, bf16* Kb, bf16* Vr) {
    const int snpad = (sn + 63) & ~63;
    const int64_t ssr = p.axis == 0 ? sn : 1, sst = p.axis == 1 ? sn : 1;
    const int ln = opaque(lane);
#pragma unroll
    for (int kt = wave; kt < KT16; kt += NW) {
      if (kt * 16 >= snpad) break;
      // values: the 16-byte chunk at column c of key row kv holds dim group
      // c ^ ((kv >> 2) & 3), so the four key groups of a transpose read fall
      // on different banks
      const int kv = kt * 16 + (ln >> 2);
      const int key_k = min(kt * 16 + (ln & 15), sn - 1), key_v = min(kv, sn - 1);
      const int dgv = (ln & 3) ^ ((kv >> 2) & 3);
      const bf16* sk = kbase + (scu + (int64_t)r * ssr + (int64_t)key_k * sst) * p.ld_qkv + (ln >> 4) * 8;
      const bf16* sv = vbase + (scu + (int64_t)r * ssr + (int64_t)key_v * sst) * p.ld_qkv + dgv * 8;
      __builtin_amdgcn_global_load_lds((const void*)sk, (__attribute__((address_space(3))) void*)(Kb + kt * 512), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void*)sv, (__attribute__((address_space(3))) void*)(Vr + kt * 512), 16, 0, 0);
    }
  };
  // query fragment of this lane for row r of a sample with sn elements at
  // pair offset scu (zero past N)
  auto load_q = [&](int sn, int64_t scu, int r) -> bf16x8 {
    if (jw >= sn) return bf16x8{};
    const int64_t ssr = p.axis == 0 ? sn : 1, sst = p.axis == 1 ? sn : 1;
    return *reinterpret_cast<const bf16x8*>(qbase + (scu + (int64_t)r * ssr + (int64_t)jw * sst) * p.ld_qkv + g * 8);
  };
  const VtLane vl = vt_lane(l16, g);
  auto v_frags1 = [&](const bf16* Vr, int kb, bf16x8 (&f)[2]) { vt_frags1(Vr, kb, vl, f); };
  auto v_frags2 = [&](const bf16* Vr, int kb, bf16x8 (&f)[4]) { vt_frags2(Vr, kb, vl, f); };

  // ---- per-sample state ------------------------------------------------------
  int n = 0;
  int64_t cu = 0, sr = 0, st = 0;               // cell(r, t) = cu + r*sr + t*st
  bool wave_has_queries = false, qvalid = false;
  // lane's bias: query 16*wave + l16, keys 16*kt + 4g .. +3 of every key
  // tile, read from the bias image (one contiguous 512 bytes per wave and tile)
  uint2 bias_r[KT16];
  auto set_sample = [&](int tiles, int sn, int64_t scu) {
    n = sn;
    cu = scu;
    sr = p.axis == 0 ? n : 1;
    st = p.axis == 1 ? n : 1;
    wave_has_queries = 16 * wave < n;
    qvalid = jw < n;
    const int kti = ((n + 63) & ~63) / 16;
    const uint2* img = p.bias_img && wave_has_queries
                           ? p.bias_img + h * p.img_head + (tiles + (int64_t)wave * kti) * 64 + lane
                           : nullptr;
#pragma unroll
    for (int kt = 0; kt < KT16; ++kt) {
      bias_r[kt] = img && kt < kti ? img[kt * 64] : make_uint2(0u, 0u);
    }
  };
  set_sample(__builtin_amdgcn_readfirstlane(bt0), __builtin_amdgcn_readfirstlane(n0), __builtin_amdgcn_readfirstlane(cu0));
  int r = __builtin_amdgcn_readfirstlane(r0);
  bf16x8 qf = load_q(n, cu, r);
  dma_kv(n, cu, r, Kb0, Vb0);
  __builtin_amdgcn_s_waitcnt(0);                // this wave's copies have landed
  __syncthreads();

  const float c = p.scale_log2;                 // scale * log2(e)
  bool odd = false;
  for (; row < row_end; ++row) {
    const bf16* Kb = odd ? Kb1 : Kb0;
    const bf16* Vb = odd ? Vb1 : Vb0;
    const bool more = row + 1 < row_end;
    // the next row: same sample, or the first row of the next non-empty one
    // (sample extents are read only when the sample changes: a global load
    // here would make the wave wait for every copy and store in flight)
    int i2 = i, r2 = r + 1, n2 = n, bt2 = 0;
    int64_t cu2 = cu;
    if (more && r2 >= n) {
      i2 = i + 1;
      while (rows[i2 + 1] <= row + 1) ++i2;
      r2 = 0;
      n2 = rows[i2 + 1] - rows[i2];
      cu2 = p.cu_pairs[i2];
      bt2 = p.bias_tiles[i2];
    }
    i2 = __builtin_amdgcn_readfirstlane(i2);
    r2 = __builtin_amdgcn_readfirstlane(r2);
    n2 = __builtin_amdgcn_readfirstlane(n2);
    bt2 = __builtin_amdgcn_readfirstlane(bt2);
    cu2 = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(cu2 >> 32)) << 32) |
                    (uint32_t)__builtin_amdgcn_readfirstlane((int)cu2));
    // gate of this lane's outputs (GATE): issued before the next row's
    // copies, so waiting for it leaves those in flight; the query index is
    // clamped into the row, so the load is unconditional
    uint2 gt[2];
    if constexpr (GATE) {
      if (wave_has_queries) {
        const bf16* gr = gbase + (cu + (int64_t)r * sr + (int64_t)min(jw, n - 1) * st) * p.ld_gate + 4 * g;
        gt[0] = *reinterpret_cast<const uint2*>(gr);
        gt[1] = *reinterpret_cast<const uint2*>(gr + 16);
      }
    }
    bf16x8 qn = qf;
    if (more) {
      dma_kv(n2, cu2, r2, odd ? Kb0 : Kb1, odd ? Vb0 : Vb1);
      qn = load_q(n2, cu2, r2);
    }
    // keep the bias packed: converting it once outside the row loop would
    // double its registers
#pragma unroll
    for (int kt = 0; kt < KT16; ++kt) asm volatile("" : "+v"(bias_r[kt].x), "+v"(bias_r[kt].y));
    float m_s = -INFINITY;                        // running max of bias/scale + q.k (EXACT: of the log2 score)
    bool far = false;                             // some lane's m_s is -inf or beyond kFarMax
    float l_s = 0.f;                              // EXACT: this lane's part of the row sum
    f32x4 O[3];                                   // dims 0-15, 16-31, row sum
#pragma unroll
    for (int u = 0; u < 3; ++u) O[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (wave_has_queries) {
      // Keys in super-chunks of 128 (8 key tiles), the last one cut to the
      // 2, 4 or 6 tiles that hold keys: all score products of a super-chunk
      // are issued together, one maximum per query, then the exponentials
      // and the value products.  Tiles read stay below the staged length.
      auto super_chunk = [&](auto sc_c, auto nt_c) {
        constexpr int SC = decltype(sc_c)::value, NT = decltype(nt_c)::value;
        constexpr int T0 = SC * 8;                // first key tile
        const int kc = SC * 128;
        f32x4 S[NT];
#pragma unroll
        for (int kt = 0; kt < NT; ++kt) {
          const uint2 bb = bias_r[T0 + kt];
          const f32x4 b4 = {__uint_as_float(bb.x << 16), __uint_as_float(bb.x & 0xffff0000u),
                            __uint_as_float(bb.y << 16), __uint_as_float(bb.y & 0xffff0000u)};
          const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Kb[(T0 + kt) * 512 + lane * 8]);
          S[kt] = mfma16(kf, qf, EXACT ? f32x4{0.f, 0.f, 0.f, 0.f} : b4);
          if constexpr (EXACT) S[kt] = log2_scores(S[kt], c, b4);
          // at most four key fragments in flight (registers)
          if (kt % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        if (!p.bias_img && kc + NT * 16 > n) {    // keys past N (with a bias the image masks them)
#pragma unroll
          for (int kt = 0; kt < NT; ++kt)
#pragma unroll
            for (int ii = 0; ii < 4; ++ii)
              if (kc + kt * 16 + 4 * g + ii >= n) S[kt][ii] = -INFINITY;
        }
        float mloc = S[0][0];
#pragma unroll
        for (int kt = 0; kt < NT; ++kt)
#pragma unroll
          for (int ii = 0; ii < 4; ++ii) mloc = fmaxf(mloc, S[kt][ii]);
        mloc = query_max(mloc);
        // the reference max moves only when some query's max grew by more
        // than 8 (log2 units): probabilities then stay below 2^8, and most
        // super-chunks skip rescaling the accumulators
        if constexpr (SC == 0) {                  // the row's first: nothing to rescale
          m_s = mloc;
          far = __any(fabsf(m_s) > kFarMax);
        } else if (__any((EXACT ? mloc - m_s : (mloc - m_s) * c) > 8.f)) {
          const float m_new = fmaxf(m_s, mloc);
          const float alpha = rescale(m_s, m_new, EXACT ? 1.f : c);
          m_s = m_new;
          far = __any(fabsf(m_s) > kFarMax);
          l_s *= alpha;
#pragma unroll
          for (int u = 0; u < (EXACT ? 2 : 3); ++u) O[u] *= alpha;
        }
        float nm = EXACT ? (m_s == -INFINITY ? 0.f : -m_s) : -m_s * c;
        if (!EXACT && far) {
          nm = m_s == -INFINITY ? 0.f : m_s;
#pragma unroll
          for (int kt = 0; kt < NT; ++kt) S[kt] -= nm;
          nm = 0.f;
        }
        bf16x8 P[NT / 2];
#pragma unroll
        for (int kt = 0; kt < NT; ++kt)
#pragma unroll
          for (int ii = 0; ii < 4; ++ii) {
            const float w = __builtin_amdgcn_exp2f(EXACT ? S[kt][ii] + nm : fmaf(S[kt][ii], c, nm));
            if constexpr (EXACT) l_s += w;
            P[kt >> 1][(kt & 1) * 4 + ii] = (bf16)w;
          }
        const bf16x8 ones = ones_bf16x8();
#pragma unroll
        for (int pp = 0; pp + 1 < NT / 2; pp += 2) {
          bf16x8 vf[4];
          v_frags2(Vb, SC * 4 + pp, vf);
          O[0] = mfma16(vf[0], P[pp], O[0]);
          O[1] = mfma16(vf[1], P[pp], O[1]);
          if constexpr (!EXACT) O[2] = mfma16(ones, P[pp], O[2]);
          O[0] = mfma16(vf[2], P[pp + 1], O[0]);
          O[1] = mfma16(vf[3], P[pp + 1], O[1]);
          if constexpr (!EXACT) O[2] = mfma16(ones, P[pp + 1], O[2]);
        }
        if constexpr ((NT / 2) % 2 == 1) {
          bf16x8 vf[2];
          v_frags1(Vb, SC * 4 + NT / 2 - 1, vf);
          O[0] = mfma16(vf[0], P[NT / 2 - 1], O[0]);
          O[1] = mfma16(vf[1], P[NT / 2 - 1], O[1]);
          if constexpr (!EXACT) O[2] = mfma16(ones, P[NT / 2 - 1], O[2]);
        }
      };
      // keys left at super-chunk SC: more than 96 take all 8 tiles (the
      // staged length, a multiple of 64, then reaches 128 past kc)
      auto run_sc = [&](auto sc_c) {
        constexpr int SC = decltype(sc_c)::value;
        const int rem = n - SC * 128;
        if (rem <= 0) return;
        if (rem > 96) super_chunk(sc_c, std::integral_constant<int, 8>{});
        else if (rem > 64) super_chunk(sc_c, std::integral_constant<int, 6>{});
        else if (rem > 32) super_chunk(sc_c, std::integral_constant<int, 4>{});
        else super_chunk(sc_c, std::integral_constant<int, 2>{});
      };
      run_sc(std::integral_constant<int, 0>{});
      run_sc(std::integral_constant<int, 1>{});
    }
    if (wave_has_queries) {
      // lane (l16, g) holds dims 4g .. 4g+3 and 16 + 4g .. +3 of its query;
      // the rows g, g ^ 1 trade halves so that an even row holds dims
      // 4g .. 4g+7 and an odd one 16 + 4(g-1) .. +7: one 16-byte store per
      // lane instead of two 8-byte ones (each store instruction gathers 16
      // cells and holds the texture-address unit the copies also need)
      const float inv = 1.f / (EXACT ? sum_over_kgroups(l_s) : O[2][0]);
      uint32_t ow[2][2];
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        float gs[4] = {1.f, 1.f, 1.f, 1.f};
        if constexpr (GATE) {
          const float gl[4] = {__uint_as_float(gt[dt].x << 16), __uint_as_float(gt[dt].x & 0xffff0000u),
                               __uint_as_float(gt[dt].y << 16), __uint_as_float(gt[dt].y & 0xffff0000u)};
#pragma unroll
          for (int ii = 0; ii < 4; ++ii) gs[ii] = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-gl[ii] * kLog2e));
        }
        bf16x4 ov;
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) ov[ii] = (bf16)(O[dt][ii] * inv * gs[ii]);
        const uint2 u = __builtin_bit_cast(uint2, ov);
        ow[dt][0] = u.x;
        ow[dt][1] = u.y;
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        // odd rows of the first operand trade with even rows of the second
        const auto sw = __builtin_amdgcn_permlane16_swap(ow[0][e], ow[1][e], false, false);
        ow[0][e] = sw[0];
        ow[1][e] = sw[1];
      }
      if (qvalid) {
        bf16* orow = obase + (cu + (int64_t)r * sr + (int64_t)jw * st) * p.ld_o;
        const int go = opaque(g), d0 = (go & 1) ? 16 + 4 * (go - 1) : 4 * go;
        *reinterpret_cast<uint4*>(orow + d0) = make_uint4(ow[0][0], ow[0][1], ow[1][0], ow[1][1]);
      }
    }
    // bias of the next sample, landed before the back edge, so the loop head has
    // no load pending and waits for none of the next row's copies
    if (i2 != i) set_sample(bt2, n2, cu2);
    __builtin_amdgcn_s_waitcnt(0);              // copies for the next row have landed
    __syncthreads();
    i = i2;
    r = r2;
    qf = qn;
    odd = !odd;
  }
}

// ---------------------------------------------------------------- pair attention, a workgroup per pair row
// Pair attention for head_dim 32 (axes 0 and 1) and samples longer than
// kAttnShortLen: a workgroup of W waves copies the keys and values of one pair
// row of one head into LDS (128 bytes per key), and its waves take the row's
// 16-query tiles in turn, all keys of the row per tile.  Single attention with
// pair bias (axis 3) is the same with a sample's tokens as the row and up to
// 128 of its queries per workgroup.  The copy is the only
// barrier.  The bias of a tile is read in 64-key chunks from the bias image
// (bf16, lane order, 512 bytes per 16 x 16 tile), one chunk ahead and across
// tiles, so any row length that the LDS holds runs the same loop: registers
// for the whole row's bias, as attention_pair_kernel keeps them, would take
// the occupancy.  On shorter samples that kernel is the faster one (172 us
// here against 136 there at B=8, N 208..224, 4 heads: a row's copy has no
// other row's work to hide behind in its own workgroup).
//
// Scores are kept transposed (S^T = K Q^T + bias / scale).  The running
// maximum is moved, and the accumulators rescaled, only where a score exceeds
// it by more than 8 in log2 units, so most chunks need no exchange between
// lanes.  A chunk whose keys are all masked (-inf) leaves a maximum of -inf
// and weights of 0.
//
// EXACT instances read the bias itself and form scale S + bias in log2 units
// in fp32 (any scale, and no rounding of bias / scale), and the denominator is
// the sum of the fp32 weights: two more vector instructions per score, two
// matrix-core products less per chunk.
// WIDE instances take 64-bit offsets within a tile of 16 rows.
template <int W, bool GATE, bool BIAS, bool EXACT, bool WIDE>
__global__ void __launch_bounds__(64 * W, 4) attention_row_kernel(PairAttnArgs p) {
  constexpr int D = 32;
  extern __shared__ __attribute__((aligned(16))) bf16 lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
  // workgroup 8 (H k + h) + x runs on XCD x: the heads of a pair row, which
  // share cache lines, follow each other on one XCD
  const int x = blockIdx.x % kXcds, t0 = blockIdx.x / kXcds;
  const int h = uni(t0 % p.H), pos = uni(t0 / p.H) * kXcds + x;
  // axes 0 and 1: (sample, pair row); axis 3: (sample, first query tile, -, tiles)
  const bool single = p.axis == 3;
  const int32_t* item = p.work + (single ? 4 : 2) * pos;
  const int i = uni(item[0]), r = uni(item[1]);
  if (i < 0) return;
  const int n = uni(p.cu_seqlens[i + 1] - p.cu_seqlens[i]);
  const int q_first = single ? r : 0, q_end = single ? r + uni(item[3]) : (n + 15) >> 4;
  const int nch = (n + 63) >> 6, nt = 4 * nch;          // 64-key chunks, key tiles
  const int64_t cu = uni(p.cu_pairs[i]);
  const int64_t base = single ? uni(p.cu_seqlens[i]) : p.axis == 0 ? cu + (int64_t)r * n : cu + r;
  const int64_t st = p.axis == 1 ? n : 1;
  // rows of tile `tile` (16 elements of the pair row): a uniform 64-bit base
  // and a 32-bit byte offset per lane (16 rows span less than 4 GB, else WIDE);
  // rows (and whole tiles) past N repeat rows below N
  auto at = [&](const bf16* b, int tile, int row_in_tile, int64_t ld, int dim) {
    tile = min(tile, (n - 1) >> 4);
    const int rl = min(row_in_tile, n - 1 - 16 * tile);
    const char* u = reinterpret_cast<const char*>(b + (int64_t)(16 * tile) * st * ld);
    if constexpr (WIDE) return u + ((int64_t)rl * st * ld + dim) * 2;
    return u + ((uint32_t)rl * (uint32_t)(st * ld) + (uint32_t)dim) * 2u;
  };
  const int64_t qoff = base * p.ld_qkv + h * D;

  // ---- keys and values: [keys | values][tile] of 1 KB
  {
    const int row16 = l16 ^ ((g & 1) << 3);
    for (int tile = wave; tile < nt; tile += W) {
      __builtin_amdgcn_global_load_lds((const void*)at(p.k + qoff, tile, row16, p.ld_qkv, g * 8),
                                       (__attribute__((address_space(3))) void*)(lds + tile * 512), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void*)at(p.v + qoff, tile, row16, p.ld_qkv, g * 8),
                                       (__attribute__((address_space(3))) void*)(lds + (nt + tile) * 512), 16, 0, 0);
    }
  }
  const uint2* img = BIAS ? p.bias_img + (int64_t)h * p.img_head + (int64_t)uni(p.bias_tiles[i]) * 64 : nullptr;
  auto load_bias = [&](int qt, int c, uint2 (&b)[4]) {
    if constexpr (BIAS) {
      const uint2* u = img + (int64_t)(qt * nt + 4 * c) * 64;
#pragma unroll
      for (int t = 0; t < 4; ++t) b[t] = u[(uint32_t)(t * 64 + lane)];
    }
  };
  auto load_q = [&](int qt) { return *reinterpret_cast<const bf16x8*>(at(p.q + qoff, qt, l16, p.ld_qkv, g * 8)); };
  // the (query tile, chunk) steps of this wave, in order
  int c = 0, qt = q_first + wave;
  uint2 b0[4], b1[4];
  bf16x8 qf = bf16x8{}, qn = bf16x8{};
  if (qt < q_end) {
    load_bias(qt, 0, b0);
    qn = load_q(qt);
  }
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (qt >= q_end) return;

  const uint32_t lds0 = lds_addr(lds), fo = (uint32_t)((g * 16 + (l16 ^ ((g & 1) << 3))) * 16), to = row_tr_offset(l16, g);
  const float sc = p.scale_log2, slack = EXACT ? 8.f : 8.f / sc;
  const bf16x8 ones = ones_bf16x8();
  float m_s = -INFINITY, nm = 0.f;                      // running maximum of bias/scale + q.k, and -m_s sc (0 where far)
  bool far = true;                                      // some lane's m_s is -inf or beyond kFarMax
  float l_s = 0.f;                                      // EXACT: this lane's part of the row sum
  f32x4 O[3];                                           // dims 0-15, 16-31, row sum
  // one step with the bias in b; the next step's bias is read into bn.
  // Returns false after the last step.
  auto step = [&](const uint2 (&b)[4], uint2 (&bn)[4]) -> bool {
    const bool last = c + 1 == nch;
    const int qtn = last && qt + W < q_end ? qt + W : qt;    // after the last tile: a read that nothing uses
    load_bias(qtn, last ? 0 : c + 1, bn);
    if (c == 0) {
      qf = qn;
      m_s = -INFINITY;
      nm = 0.f;
      far = true;
      l_s = 0.f;
#pragma unroll
      for (int u = 0; u < 3; ++u) O[u] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    uint2 gt[2];
    if (last) {
      qn = load_q(qtn);
      if constexpr (GATE) {
        const char* gr = at(p.gate + base * p.ld_gate + h * D, qt, l16, p.ld_gate, 4 * g);
        gt[0] = *reinterpret_cast<const uint2*>(gr);
        gt[1] = *reinterpret_cast<const uint2*>(gr + 32);
      }
    }
    const uint32_t kt0 = (uint32_t)(4 * c * 1024);
    const unsigned char* ks = reinterpret_cast<const unsigned char*>(lds) + kt0 + fo;
    f32x4 S[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      f32x4 b4 = {0.f, 0.f, 0.f, 0.f};
      if constexpr (BIAS)
        b4 = f32x4{__uint_as_float(b[t].x << 16), __uint_as_float(b[t].x & 0xffff0000u),
                   __uint_as_float(b[t].y << 16), __uint_as_float(b[t].y & 0xffff0000u)};
      S[t] = mfma16(*reinterpret_cast<const bf16x8*>(ks + t * 1024), qf, EXACT ? f32x4{0.f, 0.f, 0.f, 0.f} : b4);
      if constexpr (EXACT && BIAS) S[t] = log2_scores(S[t], sc, b4);
      else if constexpr (EXACT) S[t] *= sc;
    }
    if constexpr (!BIAS) {                              // keys past N (the image masks them)
      if (64 * c + 64 > n) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (64 * c + 16 * t + 4 * g + e >= n) S[t][e] = -INFINITY;
      }
    }
    float mx = S[0][0];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) mx = fmaxf(mx, S[t][e]);
    if (__any(mx > m_s + slack)) {
      const float m_new = fmaxf(m_s, query_max(mx));
      const float alpha = rescale(m_s, m_new, EXACT ? 1.f : sc);
      m_s = m_new;
      far = __any(fabsf(m_s) > kFarMax);
      nm = EXACT ? (m_s == -INFINITY ? 0.f : -m_s) : far ? 0.f : -m_s * sc;
      l_s *= alpha;
#pragma unroll
      for (int u = 0; u < (EXACT ? 2 : 3); ++u) O[u] *= alpha;
    }
    if (!EXACT && far) {
      const float ms = m_s == -INFINITY ? 0.f : m_s;
#pragma unroll
      for (int t = 0; t < 4; ++t) S[t] -= ms;
    }
    bf16x8 P[2];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float w = __builtin_amdgcn_exp2f(EXACT ? S[t][e] + nm : fmaf(S[t][e], sc, nm));
        if constexpr (EXACT) l_s += w;
        P[t >> 1][(t & 1) * 4 + e] = (bf16)w;
      }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      bf16x8 vf[2];
      row_tr_frags(lds0 + kt0 + (uint32_t)(nt * 1024 + u * 2048) + to, vf);
      O[0] = mfma16(vf[0], P[u], O[0]);
      O[1] = mfma16(vf[1], P[u], O[1]);
      if constexpr (!EXACT) O[2] = mfma16(ones, P[u], O[2]);
    }
    if (last) {
      // lane (l16, g) holds dims 4g .. 4g+3 and 16 + 4g .. +3 of its query;
      // the rows g, g ^ 1 trade halves so that every lane stores 16 bytes
      const float inv = 1.f / (EXACT ? sum_over_kgroups(l_s) : O[2][0]);
      uint32_t ow[2][2];
#pragma unroll
      for (int dt = 0; dt < 2; ++dt) {
        float gs[4] = {1.f, 1.f, 1.f, 1.f};
        if constexpr (GATE) {
          const float gl[4] = {__uint_as_float(gt[dt].x << 16), __uint_as_float(gt[dt].x & 0xffff0000u),
                               __uint_as_float(gt[dt].y << 16), __uint_as_float(gt[dt].y & 0xffff0000u)};
#pragma unroll
          for (int e = 0; e < 4; ++e) gs[e] = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-gl[e] * kLog2e));
        }
        bf16x4 ov;
#pragma unroll
        for (int e = 0; e < 4; ++e) ov[e] = (bf16)(O[dt][e] * inv * gs[e]);
        const uint2 u = __builtin_bit_cast(uint2, ov);
        ow[dt][0] = u.x;
        ow[dt][1] = u.y;
      }
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const auto sw = __builtin_amdgcn_permlane16_swap(ow[0][e], ow[1][e], false, false);
        ow[0][e] = sw[0];
        ow[1][e] = sw[1];
      }
      if (qt * 16 + l16 < n) {
        const int d0 = (g & 1) ? 16 + 4 * (g - 1) : 4 * g;
        *reinterpret_cast<uint4*>(const_cast<char*>(at(p.o + base * p.ld_o + h * D, qt, l16, p.ld_o, d0))) =
            make_uint4(ow[0][0], ow[0][1], ow[1][0], ow[1][1]);
      }
      if (qt + W >= q_end) return false;
      qt = qtn;
      c = 0;
      return true;
    }
    ++c;
    return true;
  };
  while (step(b0, b1) && step(b1, b0)) {}
}

// ---------------------------------------------------------------- 1-D attention, head_dim 32 / 64
// Variable-length attention over each sample's tokens (Sec. 3.3 "Attention
// through packed blocks"), head_dim D in {32, 64}, at most NMAX keys per
// sample.  Queries of sample i are rows cu_q[i] .. cu_q[i+1] and its keys and
// values rows cu_kv[i] .. cu_kv[i+1]: self-attention passes the same offsets
// twice; cross-attention passes the key structure separately, and the output
// takes the query structure (a query whose sample has no keys gets the empty
// sum, 0).  A workgroup of 8 waves takes (sample, block of up to 128 queries,
// head): all keys and values of the sample are copied global -> LDS once
// (32-dim halves: keys as fragment images, values row-major with the swizzle
// of the value reads), then each wave runs its 16 queries over 128-key
// super-chunks -- score products, one maximum per query, the exponentials and
// the value products -- with the lazily rescaled running maximum of the pair
// kernel.  Keys past the key count repeat the last key in LDS and get
// probability zero.
struct SeqAttnArgs {
  const bf16* q;
  int64_t ld_q;
  const bf16* k;
  const bf16* v;
  int64_t ld_kv;
  float scale_log2;
  bf16* o;
  int64_t ld_o;
  const int32_t* work;   // quads (sample, first 16-query tile, 0, tile count) over the query layout
  const int32_t* cu_q;   // query offsets
  const int32_t* cu_kv;  // key / value offsets (= cu_q for self-attention)
  int H;
};

template <int NMAX, int D>
__global__ void __launch_bounds__(512, NMAX <= 256 ? 4 : 2) attention_seq_kernel(SeqAttnArgs p) {
  static_assert(D == 32 || D == 64, "head_dim 32 or 64");
  constexpr int HV = D / 32;                      // 32-dim halves
  constexpr int KT16 = NMAX / 16;
  extern __shared__ __attribute__((aligned(16))) bf16 lds[];
  const int x = blockIdx.x % kXcds, t = blockIdx.x / kXcds;
  const int h = t % p.H, pos = (t / p.H) * kXcds + x;
  const int4 w4 = reinterpret_cast<const int4*>(p.work)[pos];
  const int i = w4.x;
  if (i < 0) return;
  const int qt0 = w4.y, nqt = w4.w;
  const int64_t qbase = p.cu_q[i];
  const int n = p.cu_q[i + 1] - (int)qbase;       // queries of the sample
  const int64_t kbase = p.cu_kv[i];
  const int m = p.cu_kv[i + 1] - (int)kbase;      // keys of the sample
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int j0 = qt0 * 16;
  const int jw = j0 + 16 * wave + l16;            // this lane's query
  const bool wave_has_queries = wave < nqt && j0 + 16 * wave < n;
  const bool qvalid = jw < n;
  if (m == 0) {
    // no keys: the empty sum
    if (wave_has_queries && qvalid) {
      bf16* orow = p.o + (qbase + jw) * p.ld_o + h * D;
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) *reinterpret_cast<bf16x4*>(orow + dt * 16 + 4 * g) = bf16x4{};
    }
    return;
  }
  const int npad = (m + 63) & ~63;
  bf16* Kh[2] = {lds, lds + NMAX * 32};           // key images per 32-dim half: tile of 16 keys -> 512 elements
  bf16* Vh[2] = {lds + HV * NMAX * 32, lds + (HV + 1) * NMAX * 32};   // values, row-major [key][32] per half

  // ---- stage keys and values of the whole sample (tiles below npad)
  for (int kt = wave; kt < KT16; kt += 8) {
    if (kt * 16 >= npad) break;
    const int key_k = min(kt * 16 + l16, m - 1);
    const int kv = kt * 16 + (lane >> 2), key_v = min(kv, m - 1);
    const int dgv = (lane & 3) ^ ((kv >> 2) & 3);
    const bf16* sk = p.k + (kbase + key_k) * p.ld_kv + h * D + g * 8;
    const bf16* sv = p.v + (kbase + key_v) * p.ld_kv + h * D + dgv * 8;
#pragma unroll
    for (int hv = 0; hv < HV; ++hv) {
      __builtin_amdgcn_global_load_lds((const void*)(sk + 32 * hv), (__attribute__((address_space(3))) void*)(Kh[hv] + kt * 512), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const void*)(sv + 32 * hv), (__attribute__((address_space(3))) void*)(Vh[hv] + kt * 512), 16, 0, 0);
    }
  }
  bf16x8 qf[HV];
#pragma unroll
  for (int hv = 0; hv < HV; ++hv) qf[hv] = bf16x8{};
  if (qvalid) {
    const bf16* qr = p.q + (qbase + jw) * p.ld_q + h * D + g * 8;
#pragma unroll
    for (int hv = 0; hv < HV; ++hv) qf[hv] = *reinterpret_cast<const bf16x8*>(qr + 32 * hv);
  }
  __builtin_amdgcn_s_waitcnt(0);                  // this wave's copies have landed
  __syncthreads();
  if (!wave_has_queries) return;

  const VtLane vl = vt_lane(l16, g);
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16)1.f;
  const float c = p.scale_log2;
  float m_s = -INFINITY;
  constexpr int NO = D / 16;                      // output accumulators; O[NO] is the row sum
  f32x4 O[NO + 1];
#pragma unroll
  for (int u = 0; u <= NO; ++u) O[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto super_chunk = [&](auto sc_c, auto nt_c) {
    constexpr int SC = decltype(sc_c)::value, NT = decltype(nt_c)::value;
    constexpr int T0 = SC * 8;
    const int kc = SC * 128;
    f32x4 S[NT];
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) {
      S[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int hv = 0; hv < HV; ++hv) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Kh[hv][(T0 + kt) * 512 + lane * 8]);
        S[kt] = mfma16(kf, qf[hv], S[kt]);
      }
      if (kt % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // bounded key fragments in flight
    }
    if (kc + NT * 16 > m) {
#pragma unroll
      for (int kt = 0; kt < NT; ++kt)
#pragma unroll
        for (int ii = 0; ii < 4; ++ii)
          if (kc + kt * 16 + 4 * g + ii >= m) S[kt][ii] = -INFINITY;
    }
    float mloc = S[0][0];
#pragma unroll
    for (int kt = 0; kt < NT; ++kt)
#pragma unroll
      for (int ii = 0; ii < 4; ++ii) mloc = fmaxf(mloc, S[kt][ii]);
    mloc = query_max(mloc);
    if (__any((mloc - m_s) * c > 8.f)) {
      const float m_new = fmaxf(m_s, mloc);
      const float alpha = __builtin_amdgcn_exp2f((m_s - m_new) * c);
      m_s = m_new;
#pragma unroll
      for (int u = 0; u <= NO; ++u) O[u] *= alpha;
    }
    const float nm = -m_s * c;
    bf16x8 P[NT / 2];
#pragma unroll
    for (int kt = 0; kt < NT; ++kt)
#pragma unroll
      for (int ii = 0; ii < 4; ++ii)
        P[kt >> 1][(kt & 1) * 4 + ii] = (bf16)__builtin_amdgcn_exp2f(fmaf(S[kt][ii], c, nm));
#pragma unroll
    for (int pp = 0; pp + 1 < NT / 2; pp += 2) {
      bf16x8 vf[HV][4];
#pragma unroll
      for (int hv = 0; hv < HV; ++hv) vt_frags2(Vh[hv], SC * 4 + pp, vl, vf[hv]);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
#pragma unroll
        for (int hv = 0; hv < HV; ++hv) {
          O[2 * hv] = mfma16(vf[hv][2 * u], P[pp + u], O[2 * hv]);
          O[2 * hv + 1] = mfma16(vf[hv][2 * u + 1], P[pp + u], O[2 * hv + 1]);
        }
        O[NO] = mfma16(ones, P[pp + u], O[NO]);
      }
    }
    if constexpr ((NT / 2) % 2 == 1) {
      bf16x8 vf[HV][2];
#pragma unroll
      for (int hv = 0; hv < HV; ++hv) vt_frags1(Vh[hv], SC * 4 + NT / 2 - 1, vl, vf[hv]);
#pragma unroll
      for (int hv = 0; hv < HV; ++hv) {
        O[2 * hv] = mfma16(vf[hv][0], P[NT / 2 - 1], O[2 * hv]);
        O[2 * hv + 1] = mfma16(vf[hv][1], P[NT / 2 - 1], O[2 * hv + 1]);
      }
      O[NO] = mfma16(ones, P[NT / 2 - 1], O[NO]);
    }
  };
  auto run_sc = [&](auto sc_c) {
    constexpr int SC = decltype(sc_c)::value;
    const int rem = m - SC * 128;
    if (rem <= 0) return;
    if (rem > 96) super_chunk(sc_c, std::integral_constant<int, 8>{});
    else if (rem > 64) super_chunk(sc_c, std::integral_constant<int, 6>{});
    else if (rem > 32) super_chunk(sc_c, std::integral_constant<int, 4>{});
    else super_chunk(sc_c, std::integral_constant<int, 2>{});
  };
  run_sc(std::integral_constant<int, 0>{});
  run_sc(std::integral_constant<int, 1>{});
  if constexpr (NMAX > 256) {
    run_sc(std::integral_constant<int, 2>{});
    run_sc(std::integral_constant<int, 3>{});
  }
  if (qvalid) {
    const float inv = 1.f / O[NO][0];
    bf16* orow = p.o + (qbase + jw) * p.ld_o + h * D;
#pragma unroll
    for (int dt = 0; dt < NO; ++dt) {
      bf16x4 ov;
#pragma unroll
      for (int ii = 0; ii < 4; ++ii) ov[ii] = (bf16)(O[dt][ii] * inv);
      *reinterpret_cast<bf16x4*>(orow + dt * 16 + 4 * g) = ov;
    }
  }
}

// ---------------------------------------------------------------- fp32 path
struct AttnF32Args {
  int axis, H;
  const float* q;
  const float* k;
  const float* v;
  int64_t ld_qkv;
  const float* bias;
  int64_t ld_bias, ld_bias_head;
  float scale;
  float* o;
  int64_t ld_o;
  const int32_t* work;
  const int32_t* cu_seqlens;
  const int32_t* cu_pairs;
  const int32_t* cu_kv;  // axis 2: key / value offsets (= cu_seqlens for self-attention)
  int64_t ld_q;          // row stride of q (ld_qkv is that of k and v)
  const float* gate;     // NULL, or o = sigmoid(gate) * attention
  int64_t ld_gate;
};

// Exact two-pass softmax per query in fp32: one thread per query.  On axis 2
// the keys of sample i are rows cu_kv[i] .. cu_kv[i+1]; a query with no keys
// gets the empty sum, 0.
template <int D>
__global__ void __launch_bounds__(256) attention_f32_kernel(AttnF32Args p) {
  Seg sg;
  if (!segment_of(p, sg)) return;
  const int h = blockIdx.y;
  int n = sg.n;                                   // keys
  int64_t kbase = sg.base;
  if (p.axis == 2) {
    kbase = p.cu_kv[sg.sample];
    n = p.cu_kv[sg.sample + 1] - (int)kbase;
  }
  for (int qi = sg.q_begin + (int)threadIdx.x; qi < sg.q_end; qi += 256) {
    const int64_t qrow = sg.base + (int64_t)qi * sg.step;
    if (n == 0) {
#pragma unroll
      for (int d = 0; d < D; ++d) p.o[qrow * p.ld_o + h * D + d] = 0.f;
      continue;
    }
    float qv[D];
#pragma unroll
    for (int d = 0; d < D; ++d) qv[d] = p.q[qrow * p.ld_q + h * D + d];
    const float* brow = p.bias ? p.bias + (int64_t)h * p.ld_bias_head + (sg.cu + (p.axis == 0 ? (int64_t)qi * n : qi)) * p.ld_bias
                               : nullptr;
    auto logit = [&](int key) {
      const int64_t krow = kbase + (int64_t)key * sg.step;
      float s = 0.f;
#pragma unroll
      for (int d = 0; d < D; ++d) s = fmaf(qv[d], p.k[krow * p.ld_qkv + h * D + d], s);
      s *= p.scale;
      if (brow) s += brow[(p.axis == 0 ? (int64_t)key : (int64_t)key * n) * p.ld_bias];
      return s;
    };
    float mx = -INFINITY;
    for (int key = 0; key < n; ++key) mx = fmaxf(mx, logit(key));
    float sum = 0.f, acc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) acc[d] = 0.f;
    for (int key = 0; key < n; ++key) {
      const float e = expf(logit(key) - mx);
      sum += e;
      const int64_t krow = kbase + (int64_t)key * sg.step;
#pragma unroll
      for (int d = 0; d < D; ++d) acc[d] = fmaf(e, p.v[krow * p.ld_qkv + h * D + d], acc[d]);
    }
#pragma unroll
    for (int d = 0; d < D; ++d) {
      float val = acc[d] / sum;
      if (p.gate) val /= 1.f + expf(-p.gate[qrow * p.ld_gate + h * D + d]);
      p.o[qrow * p.ld_o + h * D + d] = val;
    }
  }
}

}  // namespace

// ---------------------------------------------------------------- allocation-free scratch
// Scratch of nt_pair_row_attention_noalloc: one array per device, resolved to
// its device address once per device on first use.  Host code never passes
// the array's name to a kernel, only the resolved address.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

hipError_t noalloc_scratch(void** ptr) {
  static std::mutex mu;
  static void* addr[64] = {nullptr};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return hipSuccess;
}

size_t bias_image_bytes(const nt_layout& L, int H) { return (size_t)H * (size_t)L.bias_tiles_total() * 512; }

hipError_t launch_bias_image(const nt_layout& L, int axis, int H, const void* bias, int64_t ld_bias,
                             int64_t ld_bias_head, float mul, float limit, void* img, hipStream_t s) {
  const int64_t tiles = L.bias_tiles_total();
  if (tiles == 0) return hipSuccess;
  BiasImgArgs b{axis, L.batch, (const bf16*)bias, ld_bias, ld_bias_head, mul, limit, 0.999f * limit / mul, (uint2*)img, tiles,
                L.d_bias_tiles, L.d_cu_seqlens, L.d_cu_pairs};
  // A tile per wave where all of them are in flight at once (256 CUs, 32 waves
  // each): 832 tiles took 3.8 us against 4.7 with four per wave, 7168 tiles 5.0
  // against 5.6, 32400 tiles (12 heads, N 32..512, B = 8) 20.1 against 14.8.
  if (tiles * H <= 8192) bias_image_kernel<1><<<dim3((unsigned)((tiles + 3) / 4), (unsigned)H), dim3(256), 0, s>>>(b);
  else bias_image_kernel<4><<<dim3((unsigned)((tiles + 15) / 16), (unsigned)H), dim3(256), 0, s>>>(b);
  return hipGetLastError();
}

size_t attention_full_workspace_bytes(const nt_layout& L, int axis, int H, int D, nt_dtype dtype, bool has_bias) {
  // only the d = 32 pair kernels read the bias through an image
  return !has_bias || dtype != NT_BF16 || D != 32 || axis == 2 ? 0 : bias_image_bytes(L, H);
}

size_t attention_workspace_bytes(const nt_layout& L, int axis, int H, int D, nt_dtype dtype, bool has_bias) {
  // past kAttnLongLen the image is optional: without it the per-row kernel gathers the bias
  return L.max_len > kAttnLongLen ? 0 : attention_full_workspace_bytes(L, axis, H, D, dtype, has_bias);
}

namespace {
// Work items per launch of a kernel with an item and a head per workgroup: no
// more than kGridX workgroups, a multiple of 8 so that XCDs keep their items.
// The tokens of 720000 samples at 12 heads are 8.6 million workgroups; folding
// them into a second grid dimension instead costs every launch (1-D attention
// of 64 samples, 12 heads x 64: 70.7 -> 71.5 us).
int64_t launch_items(int H) { return std::max<int64_t>(8, kGridX / H / 8 * 8); }

// 1-D attention on bf16 rows, head_dim 32 or 64: queries by Lq's offsets,
// keys and values by cu_kv (device) whose longest segment is kv_max_len
// (<= kAttnLongLen).
hipError_t launch_seq_attention(const nt_layout& Lq, const int32_t* cu_kv, int kv_max_len, int H, int D,
                                const void* q, int64_t ld_q, const void* k, const void* v, int64_t ld_kv,
                                float scale, void* o, int64_t ld_o, hipStream_t s) {
  if (Lq.sattn_items() == 0) return hipSuccess;
  if (D != 32 && D != 64) return hipErrorInvalidValue;
  const bool shortk = kv_max_len <= kAttnShortLen;
  const int nmax = shortk ? kAttnShortLen : kAttnLongLen;
  SeqAttnArgs a{(const bf16*)q, ld_q, (const bf16*)k, (const bf16*)v, ld_kv, scale * kLog2e, (bf16*)o, ld_o,
                Lq.d_sattn_work, Lq.d_cu_seqlens, cu_kv, H};
  const size_t smem = sizeof(bf16) * 2 * (size_t)(D / 32) * (size_t)nmax * 32;
  const dim3 block(512);
  const void* fn = D == 64 ? (shortk ? (const void*)attention_seq_kernel<kAttnShortLen, 64>
                                     : (const void*)attention_seq_kernel<kAttnLongLen, 64>)
                           : (shortk ? (const void*)attention_seq_kernel<kAttnShortLen, 32>
                                     : (const void*)attention_seq_kernel<kAttnLongLen, 32>);
  hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  const int64_t most = launch_items(H);
  for (int64_t first = 0; e == hipSuccess && first < Lq.sattn_items(); first += most) {
    const dim3 grid((unsigned)(std::min(most, Lq.sattn_items() - first) * H));
    a.work = Lq.d_sattn_work + 4 * first;
    if (D == 64) {
      if (shortk) attention_seq_kernel<kAttnShortLen, 64><<<grid, block, smem, s>>>(a);
      else attention_seq_kernel<kAttnLongLen, 64><<<grid, block, smem, s>>>(a);
    } else {
      if (shortk) attention_seq_kernel<kAttnShortLen, 32><<<grid, block, smem, s>>>(a);
      else attention_seq_kernel<kAttnLongLen, 32><<<grid, block, smem, s>>>(a);
    }
    e = hipGetLastError();
  }
  return e;
}
}  // namespace

hipError_t launch_cross_attention(const nt_layout& Lq, const nt_layout& Lkv, int H, int D, const void* q,
                                  int64_t ld_q, const void* k, const void* v, int64_t ld_kv, float scale, void* o,
                                  int64_t ld_o, nt_dtype dtype, hipStream_t s) {
  if (Lq.sum_n == 0) return hipSuccess;
  if (dtype == NT_BF16) {
    if (Lkv.max_len > kAttnLongLen) return hipErrorInvalidValue;
    return launch_seq_attention(Lq, Lkv.d_cu_seqlens, Lkv.max_len, H, D, q, ld_q, k, v, ld_kv, scale, o, ld_o, s);
  }
  // fp32: the exact kernel, one workgroup per (sample, query block)
  if (Lq.seq_items() == 0) return hipSuccess;
  AttnF32Args a{2, H, (const float*)q, (const float*)k, (const float*)v, ld_kv, nullptr, 1, 1, scale, (float*)o,
                ld_o, Lq.d_seq_work, Lq.d_cu_seqlens, Lq.d_cu_pairs, Lkv.d_cu_seqlens, ld_q, nullptr, 0};
  const dim3 grid((unsigned)Lq.seq_items(), (unsigned)H), block(256);
  switch (D) {
    case 8: attention_f32_kernel<8><<<grid, block, 0, s>>>(a); break;
    case 16: attention_f32_kernel<16><<<grid, block, 0, s>>>(a); break;
    case 32: attention_f32_kernel<32><<<grid, block, 0, s>>>(a); break;
    case 64: attention_f32_kernel<64><<<grid, block, 0, s>>>(a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

namespace {
template <int W, bool GATE, bool BIAS, bool EXACT, bool WIDE>
hipError_t launch_row_instance(const PairAttnArgs& a, dim3 grid, size_t smem, hipStream_t s) {
  const hipError_t e = hipFuncSetAttribute((const void*)attention_row_kernel<W, GATE, BIAS, EXACT, WIDE>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  attention_row_kernel<W, GATE, BIAS, EXACT, WIDE><<<grid, dim3(64 * W), smem, s>>>(a);
  return hipGetLastError();
}

template <int W, bool EXACT, bool WIDE>
hipError_t launch_attention_rows(PairAttnArgs a, int64_t items, int max_keys, hipStream_t s) {
  const size_t smem = (size_t)max_keys * 128;
  const int64_t most = launch_items(a.H);
  hipError_t e = hipSuccess;
  for (; e == hipSuccess && items > 0; items -= most, a.work += (a.axis == 3 ? 4 : 2) * most) {
    const dim3 grid((unsigned)(std::min(most, items) * a.H));
    if (!a.bias_img)
      e = a.gate ? launch_row_instance<W, true, false, EXACT, WIDE>(a, grid, smem, s)
                 : launch_row_instance<W, false, false, EXACT, WIDE>(a, grid, smem, s);
    else
      e = a.gate ? launch_row_instance<W, true, true, EXACT, WIDE>(a, grid, smem, s)
                 : launch_row_instance<W, false, true, EXACT, WIDE>(a, grid, smem, s);
  }
  return e;
}

// The row kernel's instances: exact (see the dispatch below) and wide (64-bit
// offsets, always exact).  8 waves where two workgroups share a CU's 160 KB of
// LDS and for single attention's blocks of 128 queries, else 16: four waves per
// SIMD either way.
hipError_t launch_attention_rows(const PairAttnArgs& a, bool exact, bool wide, int64_t items, int max_keys,
                                 hipStream_t s) {
  if (wide) return launch_attention_rows<16, true, true>(a, items, max_keys, s);
  if (a.axis == 3 || max_keys <= 640)
    return exact ? launch_attention_rows<8, true, false>(a, items, max_keys, s)
                 : launch_attention_rows<8, false, false>(a, items, max_keys, s);
  return launch_attention_rows<16, true, false>(a, items, max_keys, s);   // past kAttnLongLen: exact
}

template <bool GATE, bool EXACT>
hipError_t launch_pair_instance(const PairAttnArgs& a, dim3 grid, hipStream_t s) {
  const size_t smem = sizeof(bf16) * 4 * (size_t)kAttnShortLen * 32;
  const hipError_t e = hipFuncSetAttribute((const void*)attention_pair_kernel<kAttnShortLen, 16, GATE, EXACT>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  attention_pair_kernel<kAttnShortLen, 16, GATE, EXACT><<<grid, dim3(1024), smem, s>>>(a);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_attention(const nt_layout& L, int axis, int H, int D, const void* q, const void* k,
                            const void* v, int64_t ld_qkv, const void* bias, int64_t ld_bias, int64_t ld_bias_head,
                            float scale, void* o, int64_t ld_o, nt_dtype dtype, void* workspace, hipStream_t s,
                            const void* gate, int64_t ld_gate) {
  const int32_t* work = axis == 2 ? L.d_seq_work : L.d_attn_work;
  const int64_t items = axis == 2 ? L.seq_items() : L.attn_items();
  if (items == 0) return hipSuccess;
  const dim3 grid((unsigned)items, (unsigned)H), block(256);
  if (dtype == NT_F32) {
    AttnF32Args a{axis, H, (const float*)q, (const float*)k, (const float*)v, ld_qkv, (const float*)bias,
                  ld_bias, ld_bias_head, scale, (float*)o, ld_o, work, L.d_cu_seqlens, L.d_cu_pairs,
                  L.d_cu_seqlens, ld_qkv, (const float*)gate, ld_gate};
    switch (D) {
      case 8: attention_f32_kernel<8><<<grid, block, 0, s>>>(a); break;
      case 16: attention_f32_kernel<16><<<grid, block, 0, s>>>(a); break;
      case 32: attention_f32_kernel<32><<<grid, block, 0, s>>>(a); break;
      case 64: attention_f32_kernel<64><<<grid, block, 0, s>>>(a); break;
      default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  // Samples longer than kAttnShortLen go to the row kernel, the others to the
  // persistent one; the row kernel reads the bias from the image in the
  // workspace, and without one the per-row kernel below takes a batch that has
  // longer samples.  The line is where one workgroup of
  // 16 waves stops covering a row's queries: splitting the keys of longer rows
  // between wave pairs of a persistent instance took 412 us on the four-block
  // stack (N 48..420), its rows past 256 on the row kernel 221 us and the rest
  // on the persistent one 118 us; with the line at 320 or 400 the row kernel
  // and that instance took 416 and 406 us together.
  const bool longer = L.max_len > kAttnShortLen;
  // 16 rows of a tile, 2 bytes an element, past 4 GB
  const int64_t ld_max = std::max(std::max(ld_qkv, ld_o), gate ? ld_gate : 0);
  const bool wide = 32 * ld_max * (axis == 1 ? L.max_len : 1) >= (int64_t(1) << 32);
  // EXACT instances for batches with samples past kAttnLongLen, whose bias and
  // softmax denominator stay fp32, and for scales that are zero, negative or too
  // small to divide the bias by (the others take the maximum before the scale);
  // the wide ones are always exact.
  const bool exact = wide || L.max_len > kAttnLongLen || !(scale >= 1e-6f);
  if (D == 32 && (axis == 3 || (axis <= 1 && (!longer || !bias || workspace)))) {
    const int64_t tiles = L.bias_tiles_total();
    const uint2* img = nullptr;
    if (bias && tiles > 0) {
      // The caller's workspace receives the bias image.  A finite value stays
      // finite where it is divided by the scale, or multiplied by log2(e) in fp32.
      const float mul = exact ? 1.f : 1.f / scale, limit = exact ? 2.33e38f : kMaxBf16;
      const hipError_t e = launch_bias_image(L, axis, H, bias, ld_bias, ld_bias_head, mul, limit, workspace, s);
      if (e != hipSuccess) return e;
      img = (const uint2*)workspace;
    }
    PairAttnArgs a{axis, (const bf16*)q, (const bf16*)k, (const bf16*)v, ld_qkv, (const bf16*)bias, ld_bias,
                   ld_bias_head, scale * kLog2e, (bf16*)o, ld_o, L.d_sattn_work, L.d_cu_seqlens, L.d_cu_pairs, H,
                   img, tiles * 64, L.d_bias_tiles, L.batch, L.d_cu_short,
                   reinterpret_cast<const int64_t*>(L.d_cu_short_cost), L.short_cost(), (const bf16*)gate, ld_gate};
    const int keys = (L.max_len + 63) & ~63;
    if (axis == 3) {
      // the 1-D attention's (sample, 128-query block) items
      return L.sattn_items() == 0 ? hipSuccess : launch_attention_rows(a, exact, wide, L.sattn_items(), keys, s);
    }
    if (longer) {
      PairAttnArgs al = a;
      al.work = L.d_lattn_work;
      const hipError_t e = launch_attention_rows(al, exact, wide, L.lattn_items(), keys, s);
      if (e != hipSuccess) return e;
    }
    if (L.short_rows() == 0) return hipSuccess;
    // persistent: one workgroup of 16 waves per CU (all queries of a row); per
    // XCD a multiple of H workgroups, at least H, so every head gets an equal
    // share of each XCD's rows
    const dim3 gridp((unsigned)(std::max(H, compute_units() / kXcds / H * H) * kXcds));
    if (exact)
      return gate ? launch_pair_instance<true, true>(a, gridp, s) : launch_pair_instance<false, true>(a, gridp, s);
    return gate ? launch_pair_instance<true, false>(a, gridp, s) : launch_pair_instance<false, false>(a, gridp, s);
  }
  const int npad = (L.max_len + 63) & ~63;
  if (axis == 2 && L.max_len <= kAttnLongLen)
    return launch_seq_attention(L, L.d_cu_seqlens, L.max_len, H, D, q, ld_qkv, k, v, ld_qkv, scale, o, ld_o, s);
  const int vstride = (npad + 127) / 128 * 128 + 4;
  AttnArgs a{axis, H, (const bf16*)q, (const bf16*)k, (const bf16*)v, ld_qkv, (const bf16*)bias, ld_bias,
             ld_bias_head, scale * kLog2e, (bf16*)o, ld_o, work, L.d_cu_seqlens, L.d_cu_pairs, vstride,
             (const bf16*)gate, ld_gate};
  const size_t smem = sizeof(bf16) * ((size_t)npad * (D + 8) + (size_t)D * vstride);
  if (D == 32) {
    if (smem > 65536) hipFuncSetAttribute((const void*)attention_mfma_kernel<32>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attention_mfma_kernel<32><<<grid, block, smem, s>>>(a);
  } else if (D == 64) {
    if (smem > 65536) hipFuncSetAttribute((const void*)attention_mfma_kernel<64>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attention_mfma_kernel<64><<<grid, block, smem, s>>>(a);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace nt
