// Device half of libq4nx for gfx950: the Q4NX dequantization kernel
// (Sec. 3.1.1), the fused dequant mat-vec of the decode phase (FusedDQP,
// Sec. 3.2.1, Eq. 14/15) and the fused dequant matrix product of the prefill
// phase (Sec. 3.1.2), with their C-ABI launchers -- for Q4NX blocks and for
// the MXFP4 variant of the block (FP4 E2M1 codes, one E8M0 scale per group).
//
// Common lane mapping inside a 32 x 256 block: a 16-byte load by lane l at
// byte 1024t + 16l of the block holds the 32 codes of one quantization group,
// row r = 8t + l/8, group c = l%8 (columns 32c..32c+31).  So a wave reads a
// whole block with four fully coalesced 1 KiB loads, and the scale/offset of
// the lane's group sits at index 8r + c = 64t + l of the block's tables.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <string>
#include <vector>

#include "q4nx_device.h"
#include "q4nx_internal.h"
#include "q4nx_xlane.h"

namespace q4nx {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------------------
// device helpers
// ---------------------------------------------------------------------------

// Hides the known bits of a value from the optimizer, so that byte extraction
// of a masked word maps onto v_cvt_f32_ubyte{0..3} (one op per code) instead
// of a per-code AND followed by a convert.
__device__ __forceinline__ uint32_t opaque(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

__device__ __forceinline__ float bf16_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  bf16x2 p = __builtin_convertvector((float __attribute__((ext_vector_type(2)))){a, b}, bf16x2);
  return __builtin_bit_cast(uint32_t, p);
}

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float a) {
  return (uint16_t)(pack_bf16x2(a, 0.0f) & 0xFFFFu);
}

// Streaming loads of the packed weights (read once per call).
__device__ __forceinline__ u32x4 load_codes(const uint8_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ uint32_t load_u16(const uint8_t* p) {
  return (uint32_t)__builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(p));
}

// A byte holding a 4-bit code q, read as an FP8 E4M3 value, is exactly
// q * 2^-9 (codes 0..7 are the subnormals m * 2^-9, codes 8..15 the first
// normal binade (8 + m) * 2^-9), so one gfx950 conversion turns two code bytes
// into two exact bf16 values; the conversion's scale operand 2^9 makes them q.
template <bool HI_WORD>
__device__ __forceinline__ bf16x2 codes2_bf16(uint32_t bytes) {
  return __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(bytes, 512.0f, HI_WORD);
}

// sum_i q_i * x_i over one group of 32 codes (one 16-byte word), with x given
// as 16 bf16 pairs in the order the nibble split produces: for each 8-column
// run u, (x0,x2), (x4,x6), (x1,x3), (x5,x7).  Products of two bf16 values are
// exact; v_dot2 adds two of them to the float32 accumulator.
__device__ __forceinline__ float group_dot_bf16(u32x4 q, const uint32_t (&xp)[16]) {
  float a = 0.0f, b = 0.0f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint32_t lo = opaque(q[u] & 0x0F0F0F0Fu);          // columns 8u + 0, 2, 4, 6
    const uint32_t hi = opaque((q[u] >> 4) & 0x0F0F0F0Fu);   // columns 8u + 1, 3, 5, 7
    a = __builtin_amdgcn_fdot2_f32_bf16(codes2_bf16<false>(lo), __builtin_bit_cast(bf16x2, xp[4 * u + 0]), a, false);
    a = __builtin_amdgcn_fdot2_f32_bf16(codes2_bf16<true>(lo), __builtin_bit_cast(bf16x2, xp[4 * u + 1]), a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(codes2_bf16<false>(hi), __builtin_bit_cast(bf16x2, xp[4 * u + 2]), b, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(codes2_bf16<true>(hi), __builtin_bit_cast(bf16x2, xp[4 * u + 3]), b, false);
  }
  return a + b;
}

// Two code bytes as two float32 values q * 2^-9 (exact) in one conversion.
template <bool HI_WORD>
__device__ __forceinline__ f32x2 codes2_f32(uint32_t bytes) {
  return __builtin_amdgcn_cvt_pk_f32_fp8(bytes, HI_WORD);
}

// Eq. 3 from a scaled code: (q 2^-9) * (d 2^9) is the exact product d*q (both
// scalings are exact powers of two inside the value domain), so one FMA gives
// RN(d*q + m) -- the same bits as the plain definition.
__device__ __forceinline__ float eq3(float q_scaled, float d_times_512, float m) {
  return fmaf(q_scaled, d_times_512, m);
}

// Dequantizes 8 consecutive weights (one 32-bit word of codes) of a group to
// bf16 pairs in column order; d512 = d * 2^9 (see eq3).
__device__ __forceinline__ u32x4 dequant8_bf16(uint32_t codes, float d512, float m) {
  const uint32_t lo = opaque(codes & 0x0F0F0F0Fu);          // columns 0, 2, 4, 6
  const uint32_t hi = opaque((codes >> 4) & 0x0F0F0F0Fu);   // columns 1, 3, 5, 7
  const f32x2 a = codes2_f32<false>(lo), b = codes2_f32<true>(lo);
  const f32x2 e = codes2_f32<false>(hi), g = codes2_f32<true>(hi);
  u32x4 o;
  o[0] = pack_bf16x2(eq3(a[0], d512, m), eq3(e[0], d512, m));
  o[1] = pack_bf16x2(eq3(a[1], d512, m), eq3(e[1], d512, m));
  o[2] = pack_bf16x2(eq3(b[0], d512, m), eq3(g[0], d512, m));
  o[3] = pack_bf16x2(eq3(b[1], d512, m), eq3(g[1], d512, m));
  return o;
}

// ---- MXFP4 variant of the block --------------------------------------------
// Codes are FP4 E2M1 values and each group has one E8M0 scale byte e,
// X = 2^(e-127) (OCP MX v1.0).  gfx950 converts one code byte (low nibble =
// the even column) into two bf16 or float32 values times a float32 scale in
// one instruction; an FP4 value times a power of two in [2^-100, 2^100] is
// exact in both types.  Shifted into the float32 exponent field, e is X
// itself (e = 0, what a load past the end of a tile returns, gives +0).
__device__ __forceinline__ float e8m0_f32(uint32_t e) { return __uint_as_float(e << 23); }

__device__ __forceinline__ uint32_t load_u8(const uint8_t* p) { return (uint32_t)__builtin_nontemporal_load(p); }

template <int BYTE>
__device__ __forceinline__ uint32_t fp4x2_bf16(uint32_t codes, float scale) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(codes, scale, BYTE));
}

// 8 weights (one 32-bit word of codes) times X, as bf16 pairs in column order.
__device__ __forceinline__ u32x4 mx8_bf16(uint32_t codes, float X) {
  u32x4 o;
  o[0] = fp4x2_bf16<0>(codes, X);
  o[1] = fp4x2_bf16<1>(codes, X);
  o[2] = fp4x2_bf16<2>(codes, X);
  o[3] = fp4x2_bf16<3>(codes, X);
  return o;
}

// sum_i fp4(q_i) * x_i over one group (one 16-byte word of codes), x given as
// 16 bf16 pairs in natural column order.  The products are exact; v_dot2 adds
// two of them to the float32 accumulator.
__device__ __forceinline__ float group_dot_mx(u32x4 q, const uint32_t (&xp)[16]) {
  float a = 0.0f, b = 0.0f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint32_t w = q[u];
    a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, fp4x2_bf16<0>(w, 1.0f)),
                                        __builtin_bit_cast(bf16x2, xp[4 * u + 0]), a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, fp4x2_bf16<1>(w, 1.0f)),
                                        __builtin_bit_cast(bf16x2, xp[4 * u + 1]), b, false);
    a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, fp4x2_bf16<2>(w, 1.0f)),
                                        __builtin_bit_cast(bf16x2, xp[4 * u + 2]), a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, fp4x2_bf16<3>(w, 1.0f)),
                                        __builtin_bit_cast(bf16x2, xp[4 * u + 3]), b, false);
  }
  return a + b;
}

// Weight operand of the matrix kernels: a Q4NX blob, an MXFP4-variant blob or
// a plain bf16 matrix [N][K].
enum WFmt : int { kWBf16 = 0, kWQ4NX = 1, kWMX = 2 };
template <int F>
constexpr int wblock_bytes() {
  return F == kWMX ? kMxBlockBytes : kBlockBytes;
}

// ---------------------------------------------------------------------------
// q4nx_dequant / q4nx_mx_dequant: every weight, written row-major [N][K]
// ---------------------------------------------------------------------------
// One workgroup of 256 threads per block.  Every store is 16 bytes per lane and
// every store instruction writes whole lines: bf16, 32 lanes per block row, lane
// j the columns 8j..8j+7 (one 32-bit word of codes, in group j/4; 512 bytes a
// row), eight rows per pass and four passes; float32, 64 lanes per row, lane j
// the columns 4j..4j+3 (a 16-bit half of a word, in group j/8; 1024 bytes a
// row), four rows per pass and eight passes.  (A lane per group, 64 bytes of
// output per lane, writes a quarter of every line per instruction and ran at
// a fifth of this speed; float32 as two 16-byte halves of 32 bytes per lane
// wrote half of every line: 21504 x 5376 in 142 us.)
template <int F, bool BF16>
__global__ __launch_bounds__(256) void dequant_kernel(const uint8_t* __restrict__ blob, int64_t N, int64_t K,
                                                      int64_t KB, int64_t nblocks, void* __restrict__ W) {
  constexpr int kBytes = wblock_bytes<F>();
  constexpr int kCols = BF16 ? 8 : 4, kLanes = kBlockCols / kCols, kRows = 256 / kLanes;  // per lane, row and pass
  const int lr = threadIdx.x / kLanes, j = threadIdx.x % kLanes;
  for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
    const int64_t i = b / KB, jb = b - i * KB;
    const int64_t k = jb * kBlockCols + kCols * j;
    if (k >= K) continue;  // K is a multiple of 32: whole groups lie past K
    const uint8_t* blk = blob + b * kBytes;
#pragma unroll
    for (int pass = 0; pass < kBlockRows / kRows; ++pass) {
      const int r = kRows * pass + lr;
      const int64_t n = i * kBlockRows + r;
      if (n >= N) break;
      uint32_t codes;
      if constexpr (BF16) codes = *reinterpret_cast<const uint32_t*>(blk + 128 * r + 4 * j);
      else codes = *reinterpret_cast<const uint16_t*>(blk + 128 * r + 2 * j);
      const int gi = kGroupsPerRow * r + j * kCols / kGroup;
      if constexpr (F == kWMX) {
        const float X = e8m0_f32(blk[kCodeBytes + gi]);
        if constexpr (BF16) {
          *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(W) + n * K + k) = mx8_bf16(codes, X);
        } else {
          const f32x2 a = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, X, 0);
          const f32x2 c = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(codes, X, 1);
          *reinterpret_cast<f32x4*>(static_cast<float*>(W) + n * K + k) = (f32x4){a[0], a[1], c[0], c[1]};
        }
      } else {
        const float d512 = bf16_to_f32(*reinterpret_cast<const uint16_t*>(blk + kCodeBytes + 2 * gi)) * 512.0f;
        const float m = bf16_to_f32(*reinterpret_cast<const uint16_t*>(blk + kCodeBytes + kScaleBytes + 2 * gi));
        if constexpr (BF16) {
          *reinterpret_cast<u32x4*>(static_cast<uint16_t*>(W) + n * K + k) = dequant8_bf16(codes, d512, m);
        } else {
          const f32x2 e = codes2_f32<false>(codes & 0x0F0Fu);         // columns 0, 2
          const f32x2 o = codes2_f32<false>((codes >> 4) & 0x0F0Fu);  // columns 1, 3
          *reinterpret_cast<f32x4*>(static_cast<float*>(W) + n * K + k) =
              (f32x4){eq3(e[0], d512, m), eq3(o[0], d512, m), eq3(e[1], d512, m), eq3(o[1], d512, m)};
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// q4nx_quantize: float32 weights -> packed blob (the offline conversion)
// ---------------------------------------------------------------------------
// Per group of 32 consecutive input columns (Q4_1-style, Sec. 3.1.1):
//   w -> 0 if NaN, else clamped to [-2^100, 2^100] (keeps d and m in the
//   format's value domain); lo, hi = min, max (a zero minimum is +0);
//   d = RNE_bf16(RN(RN(hi - lo) / 15)), m = RNE_bf16(lo), magnitudes below
//   2^-100 flushed to a zero of the same sign;
//   q = the code whose Eq. 3 value is nearest to w (float64 differences),
//   the smaller code on a tie.
// The Eq. 3 levels L_q = fma(q, d, m) are non-decreasing in q, so the exact
// search (quant_code, for the groups the quotient below cannot decide) finds
// the nearest level with two binary searches instead of a scan: c = the number
// of levels below w; the candidates are level c (the first >= w) and the
// first code whose level equals level c-1.
constexpr float kQuantClamp = 1.2676506002282294e30f;  // 2^100

__device__ __forceinline__ uint32_t bf16_rne_flushed(float v) {
  uint32_t b = pack_bf16x2(v, 0.0f) & 0xFFFFu;
  if ((b & 0x7FFFu) < (27u << 7)) b &= 0x8000u;  // |v| < 2^-100 -> signed zero
  return b;
}

// Number of codes q in 0..15 whose level fma(q, d, m) is below v.
__device__ __forceinline__ int levels_below(float v, float d, float m) {
  int c = 0;
#pragma unroll
  for (int s = 8; s >= 1; s >>= 1)
    if (fmaf((float)(c + s - 1), d, m) < v) c += s;
  if (c == 15 && fmaf(15.0f, d, m) < v) c = 16;
  return c;
}

// The exact code of one (clamped) weight; see above.
__device__ __forceinline__ int quant_code(float w, float d, float m) {
  const int cnt = levels_below(w, d, m);
  if (cnt == 0) return 0;
  const float l_lo = fmaf((float)(cnt - 1), d, m);
  // The first code with that level: cnt - 1 unless the level below is the
  // same value (a d small next to m), then the binary search.
  const int q_lo = (cnt == 1 || fmaf((float)(cnt - 2), d, m) < l_lo) ? cnt - 1 : levels_below(l_lo, d, m);
  if (cnt == 16) return q_lo;
  const float l_hi = fmaf((float)cnt, d, m);
  const double dist_hi = (double)l_hi - (double)w;
  const double dist_lo = (double)w - (double)l_lo;
  return dist_hi < dist_lo ? cnt : q_lo;
}

// The 32 float32 weights of each lane's group (row 8t + lane/8 of the block,
// group lane%8) for the wave that holds row octet t: every load instruction
// takes one whole row of the block (1 KiB contiguous), and the lanes pick
// their groups out of the wave's own LDS slot (128 bytes per group and 16 of
// padding, conflict-free).  Reading a group per lane straight from memory, 16
// bytes at a stride of 128, runs the address unit at a quarter of its rate.
// Rows past N and columns past K repeat the last; their groups are not used.
constexpr int kQuantGroupBytes = 144;
constexpr int kQuantSlotBytes = 64 * kQuantGroupBytes;

__device__ __forceinline__ void load_groups(const float* __restrict__ W, int64_t N, int64_t K, int64_t n0, int64_t kc,
                                            int lane, uint8_t* slot, float (&w)[32]) {
  const int64_t k = min(kc + 4 * lane, K - 4);
  f32x4 v[8];
#pragma unroll
  for (int j = 0; j < 8; ++j)
    v[j] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(W + min(n0 + j, N - 1) * K + k));
#pragma unroll
  for (int j = 0; j < 8; ++j)
    *reinterpret_cast<f32x4*>(slot + (8 * j + (lane >> 3)) * kQuantGroupBytes + 16 * (lane & 7)) = v[j];
  // A wave's LDS instructions are carried out in order.
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(slot + lane * kQuantGroupBytes + 16 * j);
    w[4 * j + 0] = x[0];
    w[4 * j + 1] = x[1];
    w[4 * j + 2] = x[2];
    w[4 * j + 3] = x[3];
  }
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// Almost every code follows from t = (w - m) / d in float32: with e bounding
// the error of t and of the levels in units of d, the code is t rounded and
// clamped to 0..15 (the levels do not decrease) unless t lies within e of a
// half-integer.  The terms of e, with R = |m| / d and u = 2^-24: w - m and the
// product are rounded and 1/d is good to 1 ulp (below 4u of |t| <= 16: 64u;
// beyond 16 the code is 15 or 0 with room to spare); a level RN(d q + m) is
// off by at most u (15 + R).  e = u (128 + R) leaves a factor of about two on
// the first.  A lane with a t that close to a half-integer (one group in two
// thousand for weights around zero) compares the two levels around the t it
// has: up to R = kQuantMaxR = 2^22, e is at most about 1/4, so the nearest
// level is one of the two, and d is more than an ulp of any level, so the
// levels are distinct.  A group with a NaN or a value to be clamped is taken
// into the domain and goes through once more.  A larger R (32 weights within
// a few ulps of each other) takes the exact search, eight weights at a time
// from the LDS slot (all 32 unrolled, it held 232 registers and halved the
// rate of the whole kernel).
// The exact search for every weight (35 operations) was bound by the VALU:
// 21504 x 5376 in 130-158 us; this takes 87 us (6.1 TB/s), 90 with every R
// above 2^17, 94 with a NaN in every group (250 us where those took the exact
// search, one weight at a time), and 200 us with every R above 2^22.
constexpr float kQuantMaxR = 4194304.0f, kQuantU = 5.9604644775390625e-08f;

__global__ __launch_bounds__(256) void quantize_kernel(const float* __restrict__ W, int64_t N, int64_t K, int64_t KB,
                                                       int64_t nblocks, uint8_t* __restrict__ blob) {
  __shared__ __attribute__((aligned(16))) uint8_t slots[4][kQuantSlotBytes];
  const int t = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = 8 * t + (lane >> 3), c = lane & 7;
  for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
    const int64_t i = b / KB, j = b - i * KB;
    uint8_t* blk = blob + b * kBlockBytes;
    u32x4 codes = (u32x4){0u, 0u, 0u, 0u};
    uint32_t sb = 0, mb = 0;
    float w[32];
    load_groups(W, N, K, i * kBlockRows + 8 * t, j * kBlockCols, lane, slots[t], w);
    if (i * kBlockRows + r < N && j * kBlockCols + kGroup * c < K) {
      bool search;
#pragma unroll 1
      for (;;) {
        float lo = w[0], hi = w[0];
#pragma unroll
        for (int e = 1; e < 32; ++e) {
          lo = fminf(lo, w[e]);
          hi = fmaxf(hi, w[e]);
        }
        lo = lo + 0.0f;  // a zero minimum is +0
        sb = bf16_rne_flushed((hi - lo) / 15.0f);
        mb = bf16_rne_flushed(lo);
        const float d = bf16_to_f32(sb), m = bf16_to_f32(mb);
        const float inv = d == 0.0f ? 0.0f : __builtin_amdgcn_rcpf(d);  // d = 0: every code is 0
        const float R = fabsf(m) * inv, near = 0.5f - kQuantU * (128.0f + R);
        bool outside = !(lo >= -kQuantClamp && hi <= kQuantClamp);  // (a NaN shows up below)
        search = !(R <= kQuantMaxR);
        if (__builtin_expect(__ballot(!search) == 0, 0)) {  // the whole wave: no codes to be had here
#pragma unroll
          for (int e = 0; e < 32; ++e) outside |= w[e] != w[e];
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            uint32_t ev = 0, od = 0;  // codes of the even and odd columns, a byte each
            bool sure = true;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float x = (w[8 * u + e] - m) * inv;
              const float q = rintf(x);
              sure &= fabsf(x - q) <= near;  // false for a NaN
              uint32_t& dst = (e & 1) ? od : ev;
              dst = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(q, 0.0f, 15.0f), e >> 1, dst);
            }
            if (!sure) {
              ev = od = 0;
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                const float v = w[8 * u + e];
                outside |= v != v;
                const float q = __builtin_amdgcn_fmed3f(floorf((v - m) * inv), 0.0f, 14.0f);
                const double below = (double)v - (double)fmaf(q, d, m), above = (double)fmaf(q + 1.0f, d, m) - (double)v;
                uint32_t& dst = (e & 1) ? od : ev;
                dst = __builtin_amdgcn_cvt_pk_u8_f32(above < below ? q + 1.0f : q, e >> 1, dst);
              }
            }
            codes[u] = ev | (od << 4);
          }
        }
        if (!outside) break;
        // Into the domain, and once more.
#pragma unroll
        for (int e = 0; e < 32; ++e)
          w[e] = w[e] != w[e] ? 0.0f : __builtin_amdgcn_fmed3f(w[e], -kQuantClamp, kQuantClamp);
      }
      if (search) {
        const float* g = reinterpret_cast<const float*>(slots[t] + lane * kQuantGroupBytes);
        const auto clamped = [&](int e) {
          const float x = g[e];
          return x != x ? 0.0f : fminf(fmaxf(x, -kQuantClamp), kQuantClamp);
        };
        const float de = bf16_to_f32(sb), me = bf16_to_f32(mb);
#pragma unroll 1
        for (int u = 0; u < 4; ++u) {
          uint32_t word = 0;
#pragma unroll
          for (int e = 0; e < 8; ++e) word |= (uint32_t)quant_code(clamped(8 * u + e), de, me) << (4 * e);
          codes[0] = u == 0 ? word : codes[0];
          codes[1] = u == 1 ? word : codes[1];
          codes[2] = u == 2 ? word : codes[2];
          codes[3] = u == 3 ? word : codes[3];
        }
      }
    }
    *reinterpret_cast<u32x4*>(blk + 1024 * t + 16 * lane) = codes;
    *reinterpret_cast<uint16_t*>(blk + kCodeBytes + 2 * (64 * t + lane)) = (uint16_t)sb;
    *reinterpret_cast<uint16_t*>(blk + kCodeBytes + kScaleBytes + 2 * (64 * t + lane)) = (uint16_t)mb;
  }
}

// q4nx_mx_quantize: float32 weights -> MXFP4-variant blob, with the loads and
// the lane mapping of quantize_kernel.  Per group (OCP MX v1.0 conversion):
// inputs taken into the domain as above; amax = max |w|; shared exponent
// e = floor(log2 amax) - 2 (2 = the largest FP4 exponent), clamped to
// [-100, 100], 0 for an all-zero group; each element w / 2^e rounded to the
// nearest FP4 magnitude -- the midpoints of {0, .5, 1, 1.5, 2, 3, 4, 6} go to
// the even mantissa -- saturating at 6, with the sign of w (-0 is code 0):
// gfx950's conversion of two float32 values over a power of two.  The group
// maximum is read from the bit patterns, so that denormal inputs give the same
// exponent whatever the denormal mode.  Seven comparisons a weight against
// the midpoints and a group per lane from memory: 21504 x 5376 in 106 us.
__global__ __launch_bounds__(256) void mx_quantize_kernel(const float* __restrict__ W, int64_t N, int64_t K,
                                                          int64_t KB, int64_t nblocks, uint8_t* __restrict__ blob) {
  __shared__ __attribute__((aligned(16))) uint8_t slots[4][kQuantSlotBytes];
  const int t = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = 8 * t + (lane >> 3), c = lane & 7;
  for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
    const int64_t i = b / KB, j = b - i * KB;
    uint8_t* blk = blob + b * kMxBlockBytes;
    u32x4 codes = (u32x4){0u, 0u, 0u, 0u};
    uint32_t eb = kMxPadScale;  // padding: code 0 with scale 1
    float w[32];
    load_groups(W, N, K, i * kBlockRows + 8 * t, j * kBlockCols, lane, slots[t], w);
    if (i * kBlockRows + r < N && j * kBlockCols + kGroup * c < K) {
      uint32_t amax = 0;  // bits of max |w|
#pragma unroll
      for (int e = 0; e < 32; ++e) {
        const uint32_t bits = __float_as_uint(w[e]), mag = bits & 0x7FFFFFFFu;
        // NaN (and -0) -> +0
        w[e] = mag - 1u < 0x7F800000u ? w[e] : 0.0f;
        amax = max(amax, __float_as_uint(w[e]) & 0x7FFFFFFFu);
      }
      if (amax > __float_as_uint(kQuantClamp)) {
#pragma unroll
        for (int e = 0; e < 32; ++e) w[e] = fminf(fmaxf(w[e], -kQuantClamp), kQuantClamp);
        amax = __float_as_uint(kQuantClamp);
      }
      const int ex = amax == 0 ? 0 : max(-100, min(100, (int)(amax >> 23) - 127 - 2));
      eb = (uint32_t)(ex + 127);
      const float X = e8m0_f32(eb);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        uint32_t q = 0;
        q = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q, w[8 * u + 0], w[8 * u + 1], X, 0);
        q = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q, w[8 * u + 2], w[8 * u + 3], X, 1);
        q = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q, w[8 * u + 4], w[8 * u + 5], X, 2);
        q = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(q, w[8 * u + 6], w[8 * u + 7], X, 3);
        codes[u] = q;
      }
    }
    *reinterpret_cast<u32x4*>(blk + 1024 * t + 16 * lane) = codes;
    blk[kCodeBytes + 64 * t + lane] = (uint8_t)eb;
  }
}

// ---------------------------------------------------------------------------
// q4nx_gemv / q4nx_gemv_batched: FusedDQP
// ---------------------------------------------------------------------------
// A workgroup owns a row group of R = 8*tq consecutive rows (tq = 4: a whole
// 32-row strip; 2: half a strip; 1: a quarter) and all of K.  Its W waves
// split the strip's blocks round-robin (block j goes to wave j % W); each
// wave accumulates, per lane, the rows 8t + l/8 (t = t0..t0+tq-1) of group
// l%8 as
//     acc += d_g * (sum_{k in g} q_k x_k) + m_g * S_g ,  S_g = sum_{k in g} x_k
// (Eq. 3 folded into Eq. 15), so the per-weight work is the exact code ->
// bf16 conversion and one v_dot2 per two weights.  A wave loads each block's
// x (512 bytes) together with the block's weights, in the same register slot,
// and stages it in its own LDS slot as bf16 pairs in the order the nibble
// split produces, forming the group sums with lane shuffles; groups are
// padded to 20 dwords so the eight groups a wave reads at once fall in
// distinct banks.  No wave waits for x beyond its own block, and there is no
// workgroup-wide staging phase or barrier before the first block.  At the end a 3-step
// butterfly adds the 8 groups of a row and the W waves' partial sums are added
// in wave order through LDS.  No workgroup talks to another, so there is no
// cross-XCD traffic and no device-wide fence.  The summation order is fixed
// for a given launch (results are reproducible call to call); it depends on
// the wave count W, which is chosen for the launch as a whole.
// Each wave prefetches its next block while computing the current one.
// For the MXFP4 variant the per-group term is X_g * (sum_{k in g} fp4(q_k) x_k)
// (no offset), with x staged in natural column order.
constexpr int kGemvMaxWaves = 16;
// A strip's weights are read 88 blocks at a time through one buffer
// descriptor (every Gemma3 K in one piece).
constexpr int kGemvChunkBlocks = 88;
constexpr int kGroupPadDw = 20;  // dwords per staged group (16 bf16 pairs + 4 pad: conflict-free reads)
constexpr int kRedFloats = kGemvMaxWaves * 32;
// Blocks in flight per wave (register slots), by row octets per wave.
constexpr int kGemvDepth4 = 1, kGemvDepth2 = 3, kGemvDepth1 = 4;
// Workgroups per CU of the streaming form (gemv_stream_kernel), LDS permitting.
constexpr int kGemvStreamPerCu = 4;

struct GemvJob {
  const uint8_t* blob;
  const uint16_t* x;
  void* y;
  int N, K;
  int nrg;       // row groups of 8 * tq rows
  int nwg;       // workgroups of this job (each loops over row groups)
  int wg_begin;  // first workgroup of this job in the launch
  int pad;
};

// The launch's first job travels as scalar kernel arguments, which gfx950
// preloads into registers (the build's -amdgpu-kernarg-preload-count), so a
// workgroup of it starts its first loads without a memory round trip for its
// arguments; the workgroups of a batch's other jobs look theirs up in memory.
struct GemvRest {
  GemvJob job[Q4NX_MAX_BATCH - 1];
};
constexpr int kGemvBf16Out = 1, kGemvJobsShift = 1;  // flags: y is bf16, number of jobs

// J holds the first job on entry.  The index first, then each field by itself:
// selecting whole structures moves them to scratch memory, at 2.5 times the
// cost of a launch.
__device__ __forceinline__ void gemv_pick(GemvJob& J, int flags, const GemvRest& rest) {
  const int wg = blockIdx.x;
  if (wg < J.nwg) return;
  int j = 0;
#pragma unroll
  for (int t = 1; t < Q4NX_MAX_BATCH - 1; ++t)
    if (t + 1 < (flags >> kGemvJobsShift) && wg >= rest.job[t].wg_begin) j = t;
  J.blob = rest.job[j].blob;
  J.x = rest.job[j].x;
  J.y = rest.job[j].y;
  J.N = rest.job[j].N;
  J.K = rest.job[j].K;
  J.nrg = rest.job[j].nrg;
  J.nwg = rest.job[j].nwg;
  J.wg_begin = rest.job[j].wg_begin;
}

// Registers of one in-flight block: TQ row octets of codes, scales, offsets
// (E8M0 scale bytes and no offsets for the MXFP4 variant).
template <int TQ>
struct GemvSlot {
  u32x4 q[TQ];
  uint32_t s[TQ], m[TQ];
  uint32_t xv[2];  // gemv_kernel: this lane's 4 bf16 of x for the block
};

// Buffer descriptor over one chunk of one strip (at most 88 blocks <= 440 KiB,
// so every offset fits the 32-bit descriptor range); raw, stride 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t chunk_rsrc(const uint8_t* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base), (short)0, bytes, 0x00020000);
}

// Cache policy of the weight loads: non-temporal (read once per call).
constexpr int kNtLoad = 2;

// Loads row octets t0..t0+TQ-1 of block `jj` of the chunk.  Every lane loads
// (all addresses lie inside the chunk); the caller skips blocks past the end
// with a wave-uniform branch.
template <int TQ, int F>
__device__ __forceinline__ void gemv_load(__amdgpu_buffer_rsrc_t rs, int jj, int t0, int lane, GemvSlot<TQ>& R) {
  const int boff = jj * wblock_bytes<F>();
#pragma unroll
  for (int t = 0; t < TQ; ++t) {
    const int tt = t0 + t;
    R.q[t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, 16 * lane, boff + 1024 * tt, kNtLoad));
    if constexpr (F == kWMX) {
      R.s[t] = __builtin_amdgcn_raw_buffer_load_b8(rs, lane, boff + kCodeBytes + 64 * tt, kNtLoad);
    } else {
      R.s[t] = __builtin_amdgcn_raw_buffer_load_b16(rs, 2 * lane, boff + kCodeBytes + 128 * tt, kNtLoad);
      R.m[t] = __builtin_amdgcn_raw_buffer_load_b16(rs, 2 * lane, boff + kCodeBytes + kScaleBytes + 128 * tt, kNtLoad);
    }
  }
}

// x for one block, per wave: lane l = c + 8r (group c, r = 0..7) reads
// columns 32c + 4r .. 32c + 4r + 3 of the block (8 bytes; 512 contiguous
// bytes per wave), in the same ring slot as the block's weights.  The
// descriptor covers the chunk's columns inside K, so columns past K read 0.
__device__ __forceinline__ void gemv_load_x(__amdgpu_buffer_rsrc_t xr, int jj, int lane, uint32_t (&xv)[2]) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 v = __builtin_bit_cast(
      u32x2, __builtin_amdgcn_raw_buffer_load_b64(xr, 2 * (kBlockCols * jj + 32 * (lane & 7) + 4 * (lane >> 3)), 0, 0));
  xv[0] = v[0];
  xv[1] = v[1];
}

// Stages one block's x in the wave's own LDS slot and returns the group sum
// S_g of this lane's group.  Q4NX: lane c + 8r writes the bf16 pairs of its 4
// columns, (x0,x2),(x1,x3) for even r, (x4,x6),(x5,x7) for odd r, so that each
// 8-column run u of a group holds (x0,x2),(x1,x3),(x4,x6),(x5,x7) at dwords
// 4u..4u+3 (slot of group c at dword c * kGroupPadDw).  S_g is formed in the
// same order as the workgroup-wide staging: per 8-column run
// ((x0+x1) + (x2+x3)) + (x4+x5) + (x6+x7), then (run0 + run1) + (run2 + run3).
// MXFP4 variant: the pairs in natural order, no sum.  The wave reads the slot
// right after writing it: a wave's LDS instructions are carried out in order,
// and the fence keeps the compiler from moving the reads above the writes.
template <int F>
__device__ __forceinline__ float gemv_stage_x(const uint32_t (&xv)[2], uint32_t* __restrict__ xw, int lane) {
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  const int c = lane & 7, r = lane >> 3;
  uint32_t* dst = xw + c * kGroupPadDw + 2 * r;
  if constexpr (F == kWMX) {
    *reinterpret_cast<u32x2*>(dst) = (u32x2){xv[0], xv[1]};
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    return 0.0f;
  }
  const uint32_t pa = (xv[0] & 0xFFFFu) | (xv[1] << 16);           // (x0,x2) or (x4,x6)
  const uint32_t pb = (xv[0] >> 16) | (xv[1] & 0xFFFF0000u);       // (x1,x3) or (x5,x7)
  *reinterpret_cast<u32x2*>(dst) = (u32x2){pa, pb};
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  const float s01 = __uint_as_float(xv[0] << 16) + __uint_as_float(xv[0] & 0xFFFF0000u);
  const float s23 = __uint_as_float(xv[1] << 16) + __uint_as_float(xv[1] & 0xFFFF0000u);
  const float o01 = xor_lane<8>(s01), o23 = xor_lane<8>(s23);  // the odd lane's (x4+x5), (x6+x7)
  float sm = 0.0f;
  sm += s01;
  sm += s23;
  sm += o01;
  sm += o23;                       // the run's sum, on the even lanes
  sm += xor_lane<16>(sm);
  sm += xor_lane<32>(sm);
  const float se = xor_lane<8>(sm);
  return (r & 1) ? se : sm;
}

// One block's contribution to the lane's row sums: Eq. 15 with Eq. 3 folded
// in, x from the wave's slot (see gemv_stage_x).  Groups past K (block
// padding) contribute nothing whatever the padding holds.
template <int TQ, int F>
__device__ __forceinline__ void gemv_compute(const GemvSlot<TQ>& R, bool gvalid, const uint32_t* __restrict__ xg,
                                               float S, float (&acc)[4]) {
  uint32_t xp[16];
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const u32x4 xv = *reinterpret_cast<const u32x4*>(xg + 4 * v);
    if constexpr (F == kWMX) {
      xp[4 * v + 0] = xv[0];
      xp[4 * v + 1] = xv[1];
      xp[4 * v + 2] = xv[2];
      xp[4 * v + 3] = xv[3];
    } else {  // slot order (x0,x2),(x1,x3),(x4,x6),(x5,x7) -> the nibble split's order
      xp[4 * v + 0] = xv[0];
      xp[4 * v + 1] = xv[2];
      xp[4 * v + 2] = xv[1];
      xp[4 * v + 3] = xv[3];
    }
  }
  if constexpr (F == kWMX) {
#pragma unroll
    for (int t = 0; t < TQ; ++t) {
      const float dot = group_dot_mx(R.q[t], xp);
      acc[t] = fmaf(gvalid ? e8m0_f32(R.s[t]) : 0.0f, dot, acc[t]);
    }
    return;
  }
#pragma unroll
  for (int t = 0; t < TQ; ++t) {
    const float dot = group_dot_bf16(R.q[t], xp);
    const float d = gvalid ? bf16_to_f32(R.s[t]) : 0.0f;
    const float m = gvalid ? bf16_to_f32(R.m[t]) : 0.0f;
    acc[t] = fmaf(d, dot, acc[t]);
    acc[t] = fmaf(m, S, acc[t]);
  }
}

template <int TQ, int D, int F>
__global__ __launch_bounds__(64 * kGemvMaxWaves) void gemv_kernel(
    const uint8_t* blob0, const uint16_t* x0, void* y0, int N0, int K0, int nrg0, int nwg0, int waves, int flags,
    const GemvRest rest) {
  constexpr int kBytes = wblock_bytes<F>();
  // red: the waves' row sums; xw: each wave's x slot (one block of x).
  __shared__ float red[kRedFloats];
  __shared__ __attribute__((aligned(16))) uint32_t xw_all[kGemvMaxWaves][kGroupsPerRow * kGroupPadDw];

  GemvJob J = {blob0, x0, y0, N0, K0, nrg0, nwg0, 0, 0};
  gemv_pick(J, flags, rest);
  const int wg = blockIdx.x, KB = (J.K + kBlockCols - 1) / kBlockCols;
  const bool y_bf16 = flags & kGemvBf16Out;

  // The wave index is uniform across a wave; saying so keeps every block
  // offset and branch derived from it in scalar registers.
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 7;
  const int W = waves;
  const bool wave_on = w < W;  // wave-uniform
  constexpr int CB = kGemvChunkBlocks;
  const int nchunks = (KB + CB - 1) / CB;
  uint32_t* const xw = xw_all[wave_on ? w : 0];

  for (int rg = wg - J.wg_begin; rg < J.nrg; rg += J.nwg) {
    const int row0 = rg * 8 * TQ;
    const int strip = row0 >> 5, t0 = (row0 & 31) >> 3;
    const uint8_t* sblob = J.blob + (size_t)strip * KB * kBytes;
    float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};

    for (int ch = 0; ch < nchunks; ++ch) {
      const int jc0 = ch * CB;
      const int nb = min(CB, KB - jc0);
      const __amdgpu_buffer_rsrc_t rs = chunk_rsrc(sblob + (size_t)jc0 * kBytes, nb * kBytes);
      const int kvalid = J.K - jc0 * kBlockCols;  // columns of this chunk inside K
      const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<uint16_t*>(J.x + (size_t)jc0 * kBlockCols), (short)0, 2 * min(kvalid, nb * kBlockCols),
          0x00020000);
      if (!wave_on) continue;
      // Ring of D register slots: block w + iW lives in slot i % D and the
      // slot is refilled with block w + (i + D)W right after it is consumed;
      // each slot carries the block's x with its weights, so a wave starts
      // on its first block as soon as that block has arrived.
      GemvSlot<TQ> buf[D];
#pragma unroll
      for (int d = 0; d < D; ++d)
        if (w + d * W < nb) {
          gemv_load_x(xr, w + d * W, lane, buf[d].xv);
          gemv_load<TQ, F>(rs, w + d * W, t0, lane, buf[d]);
        }
      for (int i0 = 0; w + i0 * W < nb; i0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
          const int jj = w + (i0 + d) * W;
          if (jj < nb) {
            const float S = gemv_stage_x<F>(buf[d].xv, xw, lane);
            gemv_compute<TQ, F>(buf[d], jj * kBlockCols + kGroup * c < kvalid, xw + c * kGroupPadDw, S, acc);
            if (jj + D * W < nb) {
              gemv_load_x(xr, jj + D * W, lane, buf[d].xv);
              gemv_load<TQ, F>(rs, jj + D * W, t0, lane, buf[d]);
            }
          }
        }
      }
    }

    // Add the 8 groups of each row: lanes 8r'..8r'+7 hold row octet t, row r'.
#pragma unroll
    for (int t = 0; t < TQ; ++t) {
      acc[t] += xor_lane<1>(acc[t]);
      acc[t] += xor_lane<2>(acc[t]);
      acc[t] += xor_lane<4>(acc[t]);
    }
    // Lane with c == t (t < TQ) holds row 8t + l/8 of the row group.
    if (wave_on && c < TQ) {
      const float v = (c == 0) ? acc[0] : (c == 1) ? acc[1] : (c == 2) ? acc[2] : acc[3];
      red[w * 32 + 8 * c + (lane >> 3)] = v;
    }
    __syncthreads();
    if (threadIdx.x < 8 * TQ) {
      float sum = 0.0f;
      for (int q = 0; q < W; ++q) sum += red[q * 32 + threadIdx.x];
      const int64_t n = (int64_t)row0 + threadIdx.x;
      if (n < J.N) {
        if (y_bf16)
          static_cast<uint16_t*>(J.y)[n] = f32_to_bf16_bits(sum);
        else
          static_cast<float*>(J.y)[n] = sum;
      }
    }
    __syncthreads();  // red[] is rewritten by the next row group
  }
}

// Persistent streaming form of gemv_kernel, for launches whose K fits one
// chunk (every Gemma3 K).  A job's row groups are dealt to a bounded number
// of workgroups, rg = r0, r0 + nwg, ...; each wave streams its blocks of all
// its row groups (w, w + W, ... of each), each block with its x, through one
// ring of D register slots that runs on across row groups, so the next row
// group's loads are in flight while the current one's rows are added up and
// stored.  The arithmetic and the order of every sum are those of
// gemv_kernel (same waves per row group), hence the same bits.  Every wave
// meets the same barriers: two per row group.
template <int TQ, int D, int F>
__global__ __launch_bounds__(64 * kGemvMaxWaves) void gemv_stream_kernel(
    const uint8_t* blob0, const uint16_t* x0, void* y0, int N0, int K0, int nrg0, int nwg0, int waves, int flags,
    const GemvRest rest) {
  constexpr int kBytes = wblock_bytes<F>();
  __shared__ float red[kRedFloats];
  __shared__ __attribute__((aligned(16))) uint32_t xw_all[kGemvMaxWaves][kGroupsPerRow * kGroupPadDw];

  GemvJob J = {blob0, x0, y0, N0, K0, nrg0, nwg0, 0, 0};
  gemv_pick(J, flags, rest);
  const int wg = blockIdx.x, KB = (J.K + kBlockCols - 1) / kBlockCols;
  const bool y_bf16 = flags & kGemvBf16Out;

  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 7;
  const int W = waves, nb = KB;
  const bool wave_on = w < W;  // wave-uniform
  const int r0 = wg - J.wg_begin;
  // Row groups of this workgroup (one each unless there are more than the grid holds).
  const int nrg = r0 >= J.nrg ? 0 : J.nwg == J.nrg ? 1 : (J.nrg - 1 - r0) / J.nwg + 1;
  if (nrg == 0) return;                                           // the whole workgroup
  const int nbw = wave_on ? (nb - w + W - 1) / W : 0;              // this wave's blocks per row group
  const int Q = nbw * nrg;
  const int kvalid = J.K;
  const int sbytes = nb * kBytes;  // bytes of one strip
  uint32_t* const xw = xw_all[wave_on ? w : 0];
  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(J.x), (short)0, 2 * J.K, 0x00020000);

  // Load cursor: row group lk of this workgroup, this wave's block ljq of it.
  int lk = 0, ljq = 0;
  auto load_next = [&](GemvSlot<TQ>& R, int& jj) {
    const int row0 = (r0 + lk * J.nwg) * 8 * TQ;
    jj = w + ljq * W;
    gemv_load_x(xr, jj, lane, R.xv);
    gemv_load<TQ, F>(chunk_rsrc(J.blob + (size_t)(row0 >> 5) * sbytes, sbytes), jj, (row0 & 31) >> 3, lane, R);
    if (++ljq == nbw) {
      ljq = 0;
      ++lk;
    }
  };

  GemvSlot<TQ> buf[D];
  int jjs[D];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    jjs[d] = 0;
    if (d < Q) load_next(buf[d], jjs[d]);
  }

  // Row group k of this workgroup is complete in every wave: add the 8 groups
  // of each row, then the W waves' sums in wave order, and store.
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  auto finish = [&](int k) {
#pragma unroll
    for (int t = 0; t < TQ; ++t) {
      acc[t] += xor_lane<1>(acc[t]);
      acc[t] += xor_lane<2>(acc[t]);
      acc[t] += xor_lane<4>(acc[t]);
    }
    if (wave_on && c < TQ) {
      const float v = (c == 0) ? acc[0] : (c == 1) ? acc[1] : (c == 2) ? acc[2] : acc[3];
      red[w * 32 + 8 * c + (lane >> 3)] = v;
    }
    __syncthreads();
    if (threadIdx.x < 8 * TQ) {
      float sum = 0.0f;
      for (int q = 0; q < W; ++q) sum += red[q * 32 + threadIdx.x];
      const int64_t n = (int64_t)(r0 + k * J.nwg) * 8 * TQ + threadIdx.x;
      if (n < J.N) {
        if (y_bf16)
          static_cast<uint16_t*>(J.y)[n] = f32_to_bf16_bits(sum);
        else
          static_cast<float*>(J.y)[n] = sum;
      }
    }
    __syncthreads();  // red[] is rewritten for the next row group
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = 0.0f;
  };

  if (Q == 0) {  // a wave without blocks still meets every barrier
    for (int k = 0; k < nrg; ++k) finish(k);
    return;
  }
  // Ring of D slots: block q of the wave's stream lives in slot q % D and the
  // slot is refilled with block q + D right after it is consumed.
  int ck = 0, cjq = 0;
  for (int q0 = 0; q0 < Q; q0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int q = q0 + d;
      if (q < Q) {
        const int jj = jjs[d];
        const float S = gemv_stage_x<F>(buf[d].xv, xw, lane);
        gemv_compute<TQ, F>(buf[d], jj * kBlockCols + kGroup * c < kvalid, xw + c * kGroupPadDw, S, acc);
        if (q + D < Q) load_next(buf[d], jjs[d]);
        if (++cjq == nbw) {
          finish(ck);
          cjq = 0;
          ++ck;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// q4nx_gemm: fused dequant + bf16 MFMA matrix product
// ---------------------------------------------------------------------------
// Every kernel below walks K in steps of 64 (two quantization groups) and
// feeds v_mfma_f32_32x32x16_bf16 from LDS: the X tile as loaded (bf16) and
// the W tile dequantized with Eq. 3 in float32 and rounded to bf16 (the
// paper's prefill dequantizes to bf16 before the MM).  LDS rows are padded to
// 72 elements (144 B) so that the 16-byte fragment reads of 8 consecutive
// rows, and the 16-byte tile writes, hit distinct banks.  Each output is the
// float32 sum of its MFMA chain over K in increasing order, so these kernels
// and all their tile shapes give the same bits.  (Where gemm_ks_kernel, below,
// takes a product, it sums in another fixed order.)  MXFP4-variant weights take the
// same path with the Eq. 3 step replaced by the exact FP4 x scale conversion.
constexpr int kBK = 64;
constexpr int kLdsStride = kBK + 8;  // bf16 elements per LDS row

// Tile order.  Workgroups are dispatched round-robin over the 8 XCDs, each
// with its own L2.  Workgroup w runs on XCD w % 8, so XCD x is given the
// contiguous range of logical tiles [x*T/8, (x+1)*T/8); logical tiles are
// ordered in groups of kGroupM tile rows, column by column, so the tiles an
// XCD runs at the same time share a few X row blocks and W column blocks in
// its L2 instead of streaming the whole operands from the memory-side cache.
constexpr int kXcds = 8;
constexpr int kGroupM = 4;

__device__ __forceinline__ void gemm_tile_of(int wg, int ntiles, int tiles_n, int& bm, int& bn) {
  const int x = wg % kXcds, l = wg / kXcds;
  const int base = ntiles / kXcds, rem = ntiles % kXcds;
  const int t = x * base + min(x, rem) + l;
  const int tiles_m = ntiles / tiles_n;
  const int group = t / (kGroupM * tiles_n);
  const int rows = min(kGroupM, tiles_m - group * kGroupM);  // tile rows in this (last) group
  const int r = t - group * kGroupM * tiles_n;
  bm = group * kGroupM + r % rows;
  bn = r / rows;
}


// Output of one wave's TI x TJ accumulator blocks when its whole 32TI x 32TJ
// sub-tile lies inside the matrix.  base (uniform over the wave) is the
// sub-tile's first element, ldy
// the row stride in elements (float32, or bf16 when bf16 != 0).  In the MFMA
// layout, element e of lane l is column l%32 and row 8(e/4) + 4(l/32) + e%4
// of its block: only the lane's own part of an address varies across the
// wave, so every element is one buffer store whose block and row offset is a
// scalar -- no per-element 64-bit address arithmetic and no bounds tests,
// which made the plain per-element stores several times longer than the
// memory needs to take them.
// Offsets inside a wave's sub-tile are 32-bit: its extent is below 2^31 bytes
// for every row stride below 2^21 elements (at most 256 rows of 4 bytes).
// Wider rows take the checked per-element stores, which address in 64 bits.
constexpr int kFastStoreMaxLdy = 1 << 21;

template <int TI, int TJ>
__device__ __forceinline__ void store_wave_tile(const f32x16 (&acc)[TI][TJ], void* base, int ldy, int bf16) {
  // The lane index is recomputed here rather than kept live across the K loop.
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const unsigned esz = bf16 ? 2u : 4u, rb = (unsigned)ldy * esz;
  // base is the same in every lane; saying so keeps the descriptor scalar
  // (otherwise each store may become a loop over distinct descriptors).
  const uint64_t bp = reinterpret_cast<uint64_t>(base);
  // (readfirstlane yields an int: each half goes through uint32_t so that the
  // low word is not sign-extended into the high one.)
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(bp >> 32));
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)bp);
  void* const ub = reinterpret_cast<void*>(((uint64_t)hi << 32) | (uint64_t)lo);
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      ub, (short)0, (int)((32 * TI - 1) * rb + 32 * TJ * esz), 0x00020000);
  const int vo = (int)(4u * (unsigned)(lane >> 5) * rb + (unsigned)(lane & 31) * esz);
  if (bf16) {
#pragma unroll
    for (int a = 0; a < TI; ++a)
#pragma unroll
      for (int b = 0; b < TJ; ++b)
#pragma unroll
        for (int e = 0; e < 16; e += 2) {  // rows r and r + 1
          const uint32_t v = pack_bf16x2(acc[a][b][e], acc[a][b][e + 1]);
          const int so = (int)((unsigned)(32 * a + 8 * (e >> 2) + (e & 3)) * rb + 64u * b);
          __builtin_amdgcn_raw_buffer_store_b16((unsigned short)v, rs, vo, so, 0);
          __builtin_amdgcn_raw_buffer_store_b16((unsigned short)(v >> 16), rs, vo, so + (int)rb, 0);
        }
  } else {
#pragma unroll
    for (int a = 0; a < TI; ++a)
#pragma unroll
      for (int b = 0; b < TJ; ++b)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int so = (int)((unsigned)(32 * a + 8 * (e >> 2) + (e & 3)) * rb + 128u * b);
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[a][b][e]), rs, vo, so, 0);
        }
  }
}

// ---- 256 x 256 tile, one wave per SIMD ------------------------------------
// Four waves in a 2 x 2 grid, each owning a 128 x 128 sub-tile: 16 MFMA
// accumulators (256 accumulation registers, which live in the AGPR half of the
// register file), so each 16-deep K slice costs 16 MFMAs against 8 fragment
// reads -- half the LDS read traffic per MFMA of a 128 x 64 wave tile.  With
// a single wave per SIMD nothing hides a stall, so the instruction order is
// fixed by hand: a K step is four blocks of 16 MFMA slots, each slot one MFMA
// plus a fixed share of the other work, fenced so the compiler keeps it there:
//   slots  0-15  MFMAs of K slice 0 | fragment reads of slice 1 | part of
//                the next step's tiles written to the other LDS stage (X, or
//                bf16 W) | weight group 0 of the next step dequantized (a
//                quarter of 8 columns per slot)
//   slots 16-31  slice 1 | reads of slice 2 | more of the tiles | weight
//                group 1 dequantized
//   slots 32-47  slice 2 | reads of slice 3 | the rest of a bf16 W tile
//   barrier      (the other stage is complete; this stage's reads are done)
//   slots 48-63  slice 3 | reads of slice 0 of the next step
// with the global loads of step + 3 issued as their registers free up (the
// exact placement is given at the step function below).  The raw operands of
// a step are loaded into registers two steps ahead.  X and
// W are read through buffer descriptors limited to the tile's rows and strips;
// in the last step of a K that is not a multiple of 64 the columns past K are
// given an offset past the descriptor's end, which reads as zero -- code 0,
// scale 0 and offset 0 give w = +0 (code 0 with E8M0 byte 0 as well) -- so no
// mask is needed anywhere else.  X
// rows past M and W strips past the matrix are clamped to the last valid one;
// their outputs are never stored.
constexpr int kWideThreads = 256;
constexpr int kMaxSplit = 4;  // K segments of a split-K launch, at most
constexpr int kWideLdsBytes = 2 * 2 * 256 * kLdsStride * 2;  // two stages of X and W
constexpr int64_t kWideMaxK = int64_t(1) << 22;               // 256 rows x K x 2 B < 2^31

// Raw operands of one K step held by one thread.  X (and bf16 W): rows
// tid/8 + 32i, columns 8(tid%8)..+7 of the step.  Packed W: codes, scale and
// offset (no offset for the MXFP4 variant) of group (row tid/2 + 128g, half
// tid%2 of the step).
template <int WF>
struct WideRegs {
  u32x4 x[8];
  u32x4 q[2];
  uint32_t s[2], m[2];
};
template <>
struct WideRegs<kWBf16> {
  u32x4 x[8];
  u32x4 w[8];
};

// Dequantization of one packed weight group (16 code bytes, its scale s and
// offset m as loaded) in 16 pieces: piece p handles a quarter of the 8
// columns 8(p/4)..+7 (Eq. 3, as in dequant8_bf16; for the MXFP4 variant one
// FP4 x scale conversion of a code byte, as in mx8_bf16), and the last
// quarter stores the 8 bf16 weights at dst + 8(p/4).  The hand-scheduled
// GEMM kernels spread the pieces over their MFMA slots, one per slot.
template <int WF>
struct GroupDequant {
  uint32_t lo = 0, hi = 0;
  float d = 0.0f, m = 0.0f;
  f32x2 a, e, b, g;
  u32x4 o;
  __device__ __forceinline__ void piece(const u32x4& q, uint32_t s, uint32_t mo, int p, uint16_t* dst) {
    const int u = p >> 2, qt = p & 3;
    if constexpr (WF == kWMX) {
      if (p == 0) d = e8m0_f32(s);
      const uint32_t w = q[u];
      if (qt == 0) o[0] = fp4x2_bf16<0>(w, d);
      else if (qt == 1) o[1] = fp4x2_bf16<1>(w, d);
      else if (qt == 2) o[2] = fp4x2_bf16<2>(w, d);
      else {
        o[3] = fp4x2_bf16<3>(w, d);
        *reinterpret_cast<u32x4*>(dst + 8 * u) = o;
      }
    } else {
      if (qt == 0) {
        if (u == 0) {
          d = bf16_to_f32(s) * 512.0f;
          m = bf16_to_f32(mo);
        }
        lo = opaque(q[u] & 0x0F0F0F0Fu);
        hi = opaque((q[u] >> 4) & 0x0F0F0F0Fu);
        a = codes2_f32<false>(lo);
      } else if (qt == 1) {
        e = codes2_f32<false>(hi);
        o[0] = pack_bf16x2(eq3(a[0], d, m), eq3(e[0], d, m));
        o[1] = pack_bf16x2(eq3(a[1], d, m), eq3(e[1], d, m));
      } else if (qt == 2) {
        b = codes2_f32<true>(lo);
        g = codes2_f32<true>(hi);
        o[2] = pack_bf16x2(eq3(b[0], d, m), eq3(g[0], d, m));
      } else {
        o[3] = pack_bf16x2(eq3(b[1], d, m), eq3(g[1], d, m));
        *reinterpret_cast<u32x4*>(dst + 8 * u) = o;
      }
    }
  }
};

// WF: W is a packed Q4NX or MXFP4-variant matrix (dequantized on the fly), or
// bf16 [N][K], whose tile is staged exactly like the X tile.
// Split K: workgroup (x, y) computes tile x over K steps [y*ksteps,
// min((y+1)*ksteps, all steps)) and, when `part` is given, writes its float32
// partial product to part + y*M*ldy (row stride ldy) instead of Y.
template <bool KTAIL, int WF>
__global__ __launch_bounds__(kWideThreads) void gemm256_kernel(const uint16_t* __restrict__ X,
                                                               const uint8_t* __restrict__ wsrc,
                                                               void* __restrict__ Y, int M, int N, int K, int ldy,
                                                               int KB, int NS, int tiles_n, int y_bf16, int ksteps,
                                                               float* __restrict__ part) {
  constexpr int TI = 4, TJ = 4;
  extern __shared__ __attribute__((aligned(16))) uint16_t gl[];
  uint16_t* const xs0 = gl;                          // [2][256][72]
  uint16_t* const ws0 = gl + 2 * 256 * kLdsStride;   // [2][256][72]

  int bm, bn;
  gemm_tile_of(blockIdx.x, gridDim.x, tiles_n, bm, bn);
  const int m0 = bm * 256, n0 = bn * 256;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  const int rows_x = min(256, M - m0);
  const __amdgpu_buffer_rsrc_t rsx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(X + (size_t)m0 * K), (short)0, rows_x * K * 2, 0x00020000);
  constexpr bool WQ4 = WF != kWBf16;  // packed weights
  constexpr int kBB = wblock_bytes<WF>();
  const int s0 = n0 >> 5, nst = min(8, NS - s0), rows_w = min(256, N - n0);
  const __amdgpu_buffer_rsrc_t rsw =
      WQ4 ? __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wsrc + (size_t)s0 * KB * kBB), (short)0,
                                              nst * KB * kBB, 0x00020000)
          : __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wsrc + (size_t)n0 * K * 2), (short)0,
                                              rows_w * K * 2, 0x00020000);
  constexpr int kPastEnd = 0x7FFFFFF0;  // beyond every descriptor: loads return 0
  // Global loads per thread and K step.
  constexpr int kLoads = WF == kWQ4NX ? 14 : WF == kWMX ? 12 : 16;

  const int c8 = tid & 7, half = tid & 1;
  int vx[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) vx[i] = (min((tid >> 3) + 32 * i, rows_x - 1) * K + 8 * c8) * 2;
  int vq[2], vs[2], vw[8];
  if constexpr (WQ4) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const int r = (tid >> 1) + 128 * g;
      const int st = min(r >> 5, nst - 1), rr = r & 31;
      vq[g] = st * KB * kBB + 128 * rr + 16 * half;
      vs[g] = st * KB * kBB + kCodeBytes + (WF == kWMX ? 1 : 2) * (8 * rr + half);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) vw[i] = (min((tid >> 3) + 32 * i, rows_w - 1) * K + 8 * c8) * 2;
  }
  // K steps of this workgroup's segment: sb .. sb + nsteps - 1.
  const int sb = blockIdx.y * ksteps;
  const int nsteps = min((K + kBK - 1) / kBK, sb + ksteps) - sb;

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TJ; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.0f;

  // Global loads of step t of the segment (clamped to its last step) into R,
  // one of the kLoads loads per call, so that they can be spread over MFMA
  // slots.
  auto load1 = [&](WideRegs<WF>& R, int t, int i) {
    const int k0 = (sb + min(t, nsteps - 1)) * kBK;
    const int sq = (k0 >> 8) * kBB + 16 * ((k0 & 255) >> 5);
    const int ss = (k0 >> 8) * kBB + (WF == kWMX ? 1 : 2) * ((k0 & 255) >> 5);
    const bool okx = !KTAIL || k0 + 8 * c8 < K;
    const bool okw = !KTAIL || k0 + kGroup * half < K;
    if (i < 8) {
      if (!KTAIL)
        R.x[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsx, vx[i], 2 * k0, 0));
      else
        R.x[i] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsx, okx ? vx[i] + 2 * k0 : kPastEnd, 0, 0));
      return;
    }
    if constexpr (!WQ4) {
      if (!KTAIL)
        R.w[i - 8] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsw, vw[i - 8], 2 * k0, 0));
      else
        R.w[i - 8] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsw, okx ? vw[i - 8] + 2 * k0 : kPastEnd, 0, 0));
    } else if (i < 10) {
      const int g = i - 8;
      R.q[g] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsw, okw ? vq[g] + sq : kPastEnd, 0, kNtLoad));
    } else if (i < 12) {
      const int g = i - 10;
      if constexpr (WF == kWMX)
        R.s[g] = __builtin_amdgcn_raw_buffer_load_b8(rsw, okw ? vs[g] + ss : kPastEnd, 0, kNtLoad);
      else
        R.s[g] = __builtin_amdgcn_raw_buffer_load_b16(rsw, okw ? vs[g] + ss : kPastEnd, 0, kNtLoad);
    } else {
      const int g = i - 12;
      R.m[g] = __builtin_amdgcn_raw_buffer_load_b16(rsw, okw ? vs[g] + ss + kScaleBytes : kPastEnd, 0, kNtLoad);
    }
  };
  auto xs_row = [&](int st) { return xs0 + st * 256 * kLdsStride + (tid >> 3) * kLdsStride + 8 * c8; };
  auto ws_row = [&](int st, int g) {
    return ws0 + st * 256 * kLdsStride + ((tid >> 1) + 128 * g) * kLdsStride + kGroup * half;
  };
  // Fragment i of K slice kq, in first-use order A0, B0, B1, B2, B3, A1, A2, A3.
  const int fa = (128 * wm + (lane & 31)) * kLdsStride + 8 * (lane >> 5);
  const int fb = (128 * wn + (lane & 31)) * kLdsStride + 8 * (lane >> 5);
  auto read1 = [&](int st, int kq, bf16x8 (&A)[TI], bf16x8 (&B)[TJ], int i) {
    const uint16_t* xs = xs0 + st * 256 * kLdsStride + fa + 16 * kq;
    const uint16_t* ws = ws0 + st * 256 * kLdsStride + fb + 16 * kq;
    if (i == 0) A[0] = *reinterpret_cast<const bf16x8*>(xs);
    else if (i <= 4) B[i - 1] = *reinterpret_cast<const bf16x8*>(ws + 32 * (i - 1) * kLdsStride);
    else A[i - 4] = *reinterpret_cast<const bf16x8*>(xs + 32 * (i - 4) * kLdsStride);
  };
  auto mma1 = [&](const bf16x8 (&A)[TI], const bf16x8 (&B)[TJ], int i) {
    acc[i >> 2][i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[i >> 2], B[i & 3], acc[i >> 2][i & 3], 0, 0, 0);
  };
  // Weight group g of the next step dequantized piece by piece.
  GroupDequant<WF> gdq;
  auto wpiece = [&](const WideRegs<WF>& R, int st, int g, int p) {
    if constexpr (WQ4) gdq.piece(R.q[g], R.s[g], WF == kWMX ? 0u : R.m[g], p, ws_row(st, g));
  };
  // bf16 W: chunk i of the thread's W rows, staged like X.
  auto wchunk = [&](const WideRegs<WF>& R, int st, int i) {
    if constexpr (!WQ4)
      *reinterpret_cast<u32x4*>(xs_row(st) + 2 * 256 * kLdsStride + 32 * i * kLdsStride) = R.w[i];
  };

  // One K step: MFMAs of step s from stage s&1 while step s+1 (held in Rs) is
  // written to the other stage and step s+3 is loaded into Rs.
  //
  // Placement of the LDS accesses.  A slot is one MFMA, 32 clocks, in which
  // the CU's LDS serves about six 1 KiB wave reads or two and a half wave
  // writes (measured on MI355X: ~190 and ~78 bytes per clock), and every
  // slice reads its 8 fragments of the next slice.  The writes of the
  // other stage must land before the barrier, so they are spread over the
  // slices before it instead of being packed into one:
  //   bf16 W (16 writes: x0..x7, w0..w7), odd slots from 1: slice 0 x0..x5,
  //     slice 1 x6 x7 w0..w3, slice 2 w4..w7 -- at most 14 accesses in a
  //     slice; fragment reads on the even slots (slice 2: slots 0, 2, 4, 6,
  //     8-11, well before the barrier);
  //   packed W: reads on the even slots of slices 0-1, X at slots 1, 5, 9, 13
  //     (x0..x3 in slice 0, x4..x7 in slice 1) between the dequantized W
  //     writes at slots 3, 7, 11, 15.  (With a K tail the X writes stay at
  //     slots 8-15 of slice 0: the interleaved form costs that instantiation
  //     a register spill.)
  // The order of the MFMAs, hence every result bit, does not depend on this.
  constexpr bool kSpreadPacked = WQ4 && !KTAIL;
  auto stage_write = [&](WideRegs<WF>& Rs, uint16_t* xsn, int nxt, int slice, int i) {
    if (!(i & 1)) return;
    const int o = i >> 1;
    if constexpr (!WQ4) {
      if (slice < 2 ? o >= 6 : o >= 4) return;
      const int k = slice * 6 + o;
      if (k < 8)
        *reinterpret_cast<u32x4*>(xsn + 32 * k * kLdsStride) = Rs.x[k];
      else
        wchunk(Rs, nxt, k - 8);
    } else if constexpr (kSpreadPacked) {
      if (slice < 2 && (o & 1) == 0) {
        const int k = 4 * slice + (o >> 1);
        *reinterpret_cast<u32x4*>(xsn + 32 * k * kLdsStride) = Rs.x[k];
      }
    }
  };
  const auto read_slot = [](int slice, int i) {
    if (!WQ4 || kSpreadPacked) {
      if (slice < 2) return (i & 1) ? -1 : i >> 1;
      if (!WQ4) return i < 8 ? ((i & 1) ? -1 : i >> 1) : (i < 12 ? i - 4 : -1);
    }
    return i < 8 ? i : -1;
  };
  // Global loads of step s + 3 go out as soon as their registers are free:
  // one slot after the write that empties them (bf16 W, and X of packed W),
  // and a packed W group in the slice after the one that dequantizes it.  So
  // they spread over slices 0-2 instead of forming one burst in slice 2, and
  // leave up to two slices earlier.  (With a K tail, packed W keeps the
  // original order: all loads in slice 2, load i at slot i.)
  auto early_load = [&](WideRegs<WF>& Rs, int s, int slice, int i) {
    if constexpr (!WQ4) {
      // load k one slot after write k (odd slot 2o+1 of its slice; the
      // per-slice write counts of stage_write)
      if ((i & 1) || i == 0) return;
      constexpr int c[3] = {6, 6, 4};
      const int o = (i >> 1) - 1;
      if (o >= c[slice]) return;
      const int k = (slice > 0 ? c[0] : 0) + (slice > 1 ? c[1] : 0) + o;
      load1(Rs, s + 3, k);
    } else if constexpr (kSpreadPacked) {
      if (slice < 2 && (i & 3) == 2) load1(Rs, s + 3, 4 * slice + (i >> 2));  // x after its write at i - 1
      // W group 0 after slice 0's dequant, group 1 after slice 1's
      if (slice == 1 && (i & 1) && i < 7) {
        const int j = i >> 1;  // 0 q, 1 s, 2 m
        const int idx = 8 + 2 * j;
        if (idx < kLoads) load1(Rs, s + 3, idx);
      }
      if (slice == 2 && !(i & 1) && i < 6) {
        const int j = i >> 1;
        const int idx = 9 + 2 * j;
        if (idx < kLoads) load1(Rs, s + 3, idx);
      }
    }
  };
  bf16x8 A0[TI], B0[TJ], A1[TI], B1[TJ];
  auto step = [&](int s, WideRegs<WF>& Rs) {
    const int cur = s & 1, nxt = cur ^ 1;
    uint16_t* xsn = xs_row(nxt);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      mma1(A0, B0, i);
      if (read_slot(0, i) >= 0) read1(cur, 1, A1, B1, read_slot(0, i));
      if constexpr (WQ4 && !kSpreadPacked) {
        if (i >= 8) *reinterpret_cast<u32x4*>(xsn + 32 * (i - 8) * kLdsStride) = Rs.x[i - 8];
      } else {
        stage_write(Rs, xsn, nxt, 0, i);
      }
      wpiece(Rs, nxt, 0, i);
      early_load(Rs, s, 0, i);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      mma1(A1, B1, i);
      if (read_slot(1, i) >= 0) read1(cur, 2, A0, B0, read_slot(1, i));
      stage_write(Rs, xsn, nxt, 1, i);
      wpiece(Rs, nxt, 1, i);
      early_load(Rs, s, 1, i);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      mma1(A0, B0, i);
      if (read_slot(2, i) >= 0) read1(cur, 3, A1, B1, read_slot(2, i));
      stage_write(Rs, xsn, nxt, 2, i);
      if constexpr (WQ4 && !kSpreadPacked) {
        if (i < kLoads) load1(Rs, s + 3, i);
      } else {
        early_load(Rs, s, 2, i);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      mma1(A1, B1, i);
      if (i < 8) read1(nxt, 0, A0, B0, i);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  WideRegs<WF> R0, R1;
#pragma unroll
  for (int i = 0; i < kLoads; ++i) load1(R0, 0, i);
#pragma unroll
  for (int i = 0; i < kLoads; ++i) load1(R1, 1, i);
  {
    uint16_t* xs = xs_row(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4*>(xs + 32 * i * kLdsStride) = R0.x[i];
    if constexpr (WF == kWMX) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const float X = e8m0_f32(R0.s[g]);
#pragma unroll
        for (int u = 0; u < 4; ++u) *reinterpret_cast<u32x4*>(ws_row(0, g) + 8 * u) = mx8_bf16(R0.q[g][u], X);
      }
    } else if constexpr (WQ4) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const float d512 = bf16_to_f32(R0.s[g]) * 512.0f, m = bf16_to_f32(R0.m[g]);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          *reinterpret_cast<u32x4*>(ws_row(0, g) + 8 * u) = dequant8_bf16(R0.q[g][u], d512, m);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) wchunk(R0, 0, i);
    }
  }
#pragma unroll
  for (int i = 0; i < kLoads; ++i) load1(R0, 2, i);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; ++i) read1(0, 0, A0, B0, i);
  int s = 0;
  for (; s + 1 < nsteps; s += 2) {  // two steps per trip, so the register sets stay static
    step(s, R1);
    step(s + 1, R0);
  }
  if (s < nsteps) step(s, R1);

  // Accumulator element e of lane l: column l%32, row 8(e/4) + 4(l/32) + e%4.
  // (One output pointer and one format flag, chosen before the loop: three
  // store paths inside it make the compiler hoist per-element addresses and
  // spill.)
  const bool full = m0 + 256 <= M && n0 + 256 <= N;
  // (The slab offset is formed in unsigned 32-bit pieces: a 64-bit copy of
  // ldy shared with the element addresses below turns each of them into a
  // full 64 x 64-bit multiply.)
  void* const Yo = part ? static_cast<void*>(part + (size_t)(blockIdx.y * (unsigned)M) * (unsigned)ldy) : Y;
  const int obf16 = part ? 0 : y_bf16;
  if (full && ldy < kFastStoreMaxLdy) {
    store_wave_tile(acc,
                    static_cast<char*>(Yo) + ((size_t)(unsigned)(m0 + 128 * wm) * (unsigned)ldy +
                                              (unsigned)(n0 + 128 * wn)) * (obf16 ? 2u : 4u),
                    ldy, obf16);
    return;
  }
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TJ; ++b) {
      const int col = n0 + 128 * wn + 32 * b + (lane & 31);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = m0 + 128 * wm + 32 * a + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (full || (row < M && col < N)) {
          if (obf16)
            static_cast<uint16_t*>(Yo)[(size_t)row * ldy + col] = f32_to_bf16_bits(acc[a][b][e]);
          else
            static_cast<float*>(Yo)[(size_t)row * ldy + col] = acc[a][b][e];
        }
      }
    }
}

// ---- tiles of 64 TI x 64 TJ, one wave per SIMD ------------------------------
// The 256 x 256 kernel's scheme for any tile of 64 TI x 64 TJ with K a
// multiple of 64: four waves in a 2 x 2 grid, each owning a 32 TI x 32 TJ
// sub-tile, and a K step of four slices of P = TI TJ MFMA slots with the other
// work spread evenly over them: the TI + TJ fragment reads of the next slice,
// the stage writes of the next step's X (and bf16 W) over the 3P slots before
// the barrier, its weight groups dequantized piece by piece, and each global
// load of step s + 1 + D one slot after the write that frees its registers (D
// register sets: 2, or 4 where a step is short).  The MFMA chain of every
// output is the same as in the other kernels, hence the same bits.
// Why a family of tiles: a launch costs whole rounds of tiles, so the tile
// that fills the CUs once decides most products of a few hundred rows.
// Measured on MI355X against the tiles there were before (256 x 256,
// 256 x 128, 128 x 128 and 128 x 64), us: 300 rows of Gemma3-27B gate/up 254 ->
// 166 (320 x 192; MXFP4 weights 220 -> 147), 512 rows of 4B gate/up 73 -> 64
// (256 x 192), 128 rows 41 -> 28 (128 x 128, a wave per SIMD instead of two
// on the compiler's schedule), 512 rows of 4B q/k/v 37 -> 26 (64 x 128).  Tiles of 64 x 64, 128 x 64, 128 x 192
// and 192 x 192 were nowhere ahead by more than 2% and are not built.
template <int TI, int TJ, int WF>
struct TileRegs {
  u32x4 x[2 * TI];
  u32x4 q[(TJ + 1) / 2];
  uint32_t s[(TJ + 1) / 2], m[(TJ + 1) / 2];
};
template <int TI, int TJ>
struct TileRegs<TI, TJ, kWBf16> {
  u32x4 x[2 * TI];
  u32x4 w[2 * TJ];
};

template <int TI, int TJ>
constexpr int tile_lds_bytes() {
  return 2 * (64 * TI + 64 * TJ) * kLdsStride * 2;
}

template <int TI, int TJ, int D, int WF>
__global__ __launch_bounds__(kWideThreads, (tile_lds_bytes<TI, TJ>() <= 80 * 1024 ? 2 : 1)) void gemm_tile_kernel(
    const uint16_t* __restrict__ X, const uint8_t* __restrict__ wsrc, void* __restrict__ Y, int M, int N, int K,
    int ldy, int KB, int NS, int tiles_n, int y_bf16) {
  constexpr int BM = 64 * TI, BN = 64 * TJ, P = TI * TJ, S = 3 * P;  // MFMAs per slice; slots before the barrier
  constexpr bool WQ4 = WF != kWBf16;
  constexpr int kBB = wblock_bytes<WF>();
  constexpr int kG = (TJ + 1) / 2;  // packed weight groups per thread and step
  constexpr int kXW = 2 * TI, kWW = 2 * TJ;
  extern __shared__ __attribute__((aligned(16))) uint16_t gl[];
  uint16_t* const xs0 = gl;                        // [2][BM][72]
  uint16_t* const ws0 = gl + 2 * BM * kLdsStride;  // [2][BN][72]

  int bm, bn;
  gemm_tile_of(blockIdx.x, gridDim.x, tiles_n, bm, bn);
  const int m0 = bm * BM, n0 = bn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  const int rows_x = min(BM, M - m0);
  const __amdgpu_buffer_rsrc_t rsx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(X + (size_t)m0 * K), (short)0, rows_x * K * 2, 0x00020000);
  const int s0 = n0 >> 5, nst = min(2 * TJ, NS - s0), rows_w = min(BN, N - n0);
  const __amdgpu_buffer_rsrc_t rsw =
      WQ4 ? __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wsrc + (size_t)s0 * KB * kBB), (short)0,
                                              nst * KB * kBB, 0x00020000)
          : __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wsrc + (size_t)n0 * K * 2), (short)0,
                                              rows_w * K * 2, 0x00020000);

  const int c8 = tid & 7, hh = tid & 1;
  int vx[kXW];
#pragma unroll
  for (int i = 0; i < kXW; ++i) vx[i] = (min((tid >> 3) + 32 * i, rows_x - 1) * K + 8 * c8) * 2;
  // Group g of a thread: row tid/2 + 128g of the tile, half tid%2 of the step.
  // With an odd TJ the second half of the threads repeats the first half's
  // last group (the same values to the same place).
  int vq[kG], vs[kG], gr[kG], vw[kWW];
  if constexpr (WQ4) {
#pragma unroll
    for (int g = 0; g < kG; ++g) {
      const int row = (tid >> 1) + 128 * g;
      gr[g] = row < BN ? row : row - 64;
      const int st = min(gr[g] >> 5, nst - 1), rr = gr[g] & 31;
      vq[g] = st * KB * kBB + 128 * rr + 16 * hh;
      vs[g] = st * KB * kBB + kCodeBytes + (WF == kWMX ? 1 : 2) * (8 * rr + hh);
    }
  } else {
#pragma unroll
    for (int i = 0; i < kWW; ++i) vw[i] = (min((tid >> 3) + 32 * i, rows_w - 1) * K + 8 * c8) * 2;
  }
  const int nsteps = K / kBK;

  f32x16 acc[TI][TJ];
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TJ; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.0f;

  using Regs = TileRegs<TI, TJ, WF>;
  auto load_x = [&](Regs& R, int t, int i) {
    R.x[i] = __builtin_bit_cast(
        u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsx, vx[i], 2 * kBK * min(t, nsteps - 1), 0));
  };
  auto load_w = [&](Regs& R, int t, int i) {
    const int k0 = min(t, nsteps - 1) * kBK;
    if constexpr (!WQ4) {
      R.w[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsw, vw[i], 2 * k0, 0));
    } else {
      const int c = (k0 & 255) >> 5, sb = (k0 >> 8) * kBB;
      R.q[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsw, vq[i] + sb + 16 * c, 0, kNtLoad));
      if constexpr (WF == kWMX) {
        R.s[i] = __builtin_amdgcn_raw_buffer_load_b8(rsw, vs[i] + sb + c, 0, kNtLoad);
      } else {
        R.s[i] = __builtin_amdgcn_raw_buffer_load_b16(rsw, vs[i] + sb + 2 * c, 0, kNtLoad);
        R.m[i] = __builtin_amdgcn_raw_buffer_load_b16(rsw, vs[i] + sb + 2 * c + kScaleBytes, 0, kNtLoad);
      }
    }
  };
  auto write_x = [&](const Regs& R, int st, int k) {
    *reinterpret_cast<u32x4*>(xs0 + st * BM * kLdsStride + ((tid >> 3) + 32 * k) * kLdsStride + 8 * c8) = R.x[k];
  };
  auto write_w = [&](const Regs& R, int st, int k) {
    if constexpr (!WQ4)
      *reinterpret_cast<u32x4*>(ws0 + st * BN * kLdsStride + ((tid >> 3) + 32 * k) * kLdsStride + 8 * c8) = R.w[k];
  };
  GroupDequant<WF> gdq;
  auto wpiece = [&](const Regs& R, int st, int p) {
    if constexpr (WQ4) {
      const int g = p >> 4;
      gdq.piece(R.q[g], R.s[g], WF == kWMX ? 0u : R.m[g], p & 15,
                ws0 + st * BN * kLdsStride + gr[g] * kLdsStride + kGroup * hh);
    }
  };
  const int fa = (32 * TI * wm + (lane & 31)) * kLdsStride + 8 * (lane >> 5);
  const int fb = (32 * TJ * wn + (lane & 31)) * kLdsStride + 8 * (lane >> 5);
  // Fragment i of K slice kq, in first-use order A0, B0 .. , A1 ..
  auto read1 = [&](int st, int kq, bf16x8 (&A)[TI], bf16x8 (&B)[TJ], int i) {
    const uint16_t* xs = xs0 + st * BM * kLdsStride + fa + 16 * kq;
    const uint16_t* ws = ws0 + st * BN * kLdsStride + fb + 16 * kq;
    if (i == 0) A[0] = *reinterpret_cast<const bf16x8*>(xs);
    else if (i <= TJ) B[i - 1] = *reinterpret_cast<const bf16x8*>(ws + 32 * (i - 1) * kLdsStride);
    else A[i - TJ] = *reinterpret_cast<const bf16x8*>(xs + 32 * (i - TJ) * kLdsStride);
  };
  auto mma1 = [&](const bf16x8 (&A)[TI], const bf16x8 (&B)[TJ], int i) {
    acc[i / TJ][i % TJ] =
        __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[i / TJ], B[i % TJ], acc[i / TJ][i % TJ], 0, 0, 0);
  };
  // Slots of the stage writes of step s + 1 among the S slots before the
  // barrier, evenly spaced, and of the loads that reuse their registers, one
  // slot later.
  constexpr int kPieces = WQ4 ? 16 * kG : 0;
  constexpr int kPSlots = kPieces <= 2 * P ? 2 * P : S;
  constexpr int kWrites = kXW + (WQ4 ? 0 : kWW);
  const auto wslot = [](int k) { return ((2 * k + 1) * S) / (2 * kWrites); };
  const auto pslot = [](int p) { return (p * kPSlots) / (kPieces ? kPieces : 1); };
  auto side = [&](Regs& Rs, int nxt, int s, int g) {
    if constexpr (WQ4) {
#pragma unroll
      for (int p = 0; p < kPieces; ++p)
        if (pslot(p) == g) wpiece(Rs, nxt, p);
    }
#pragma unroll
    for (int k = 0; k < kWrites; ++k) {
      if (wslot(k) == g) {
        if (k < kXW) write_x(Rs, nxt, k);
        else write_w(Rs, nxt, k - kXW);
      }
      if (wslot(k) + 1 == g) {
        if (k < kXW) load_x(Rs, s + 1 + D, k);
        else load_w(Rs, s + 1 + D, k - kXW);
      }
    }
    if constexpr (WQ4) {
#pragma unroll
      for (int w = 0; w < kG; ++w)
        if (pslot(16 * w + 15) + 1 == g) load_w(Rs, s + 1 + D, w);
    }
  };
  bf16x8 A0[TI], B0[TJ], A1[TI], B1[TJ];
  auto slice = [&](int sl, const bf16x8 (&A)[TI], const bf16x8 (&B)[TJ], bf16x8 (&An)[TI], bf16x8 (&Bn)[TJ], int rst,
                   int rkq, Regs& Rs, int nxt, int s) {
#pragma unroll
    for (int i = 0; i < P; ++i) {
      mma1(A, B, i);
#pragma unroll
      for (int f = 0; f < TI + TJ; ++f)
        if (f * P / (TI + TJ) == i) read1(rst, rkq, An, Bn, f);
      side(Rs, nxt, s, sl * P + i);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto step = [&](int s, int cur, Regs& Rs) {
    const int nxt = cur ^ 1;
    slice(0, A0, B0, A1, B1, cur, 1, Rs, nxt, s);
    slice(1, A1, B1, A0, B0, cur, 2, Rs, nxt, s);
    slice(2, A0, B0, A1, B1, cur, 3, Rs, nxt, s);
    __syncthreads();
    slice(3, A1, B1, A0, B0, nxt, 0, Rs, nxt, s);
  };

  // Register set t % D holds the operands of step t; step 0 goes to LDS at once.
  Regs R[D];
#pragma unroll
  for (int t = 0; t < D; ++t) {
#pragma unroll
    for (int i = 0; i < kXW; ++i) load_x(R[t], t, i);
#pragma unroll
    for (int i = 0; i < (WQ4 ? kG : kWW); ++i) load_w(R[t], t, i);
  }
#pragma unroll
  for (int i = 0; i < kXW; ++i) write_x(R[0], 0, i);
  if constexpr (WQ4) {
#pragma unroll
    for (int p = 0; p < kPieces; ++p) wpiece(R[0], 0, p);
  } else {
#pragma unroll
    for (int i = 0; i < kWW; ++i) write_w(R[0], 0, i);
  }
#pragma unroll
  for (int i = 0; i < kXW; ++i) load_x(R[0], D, i);
#pragma unroll
  for (int i = 0; i < (WQ4 ? kG : kWW); ++i) load_w(R[0], D, i);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < TI + TJ; ++i) read1(0, 0, A0, B0, i);
  // D steps per trip, so the register sets stay static (D is even, so the
  // stages do too).
  int s = 0;
  for (; s + D <= nsteps; s += D) {
#pragma unroll
    for (int p = 0; p < D; ++p) step(s + p, p & 1, R[(p + 1) % D]);
  }
#pragma unroll
  for (int p = 0; p < D - 1; ++p)
    if (s + p < nsteps) step(s + p, p & 1, R[(p + 1) % D]);

  const bool full = m0 + BM <= M && n0 + BN <= N;
  if (full && ldy < kFastStoreMaxLdy) {
    store_wave_tile(acc,
                    static_cast<char*>(Y) + ((size_t)(unsigned)(m0 + 32 * TI * wm) * (unsigned)ldy +
                                             (unsigned)(n0 + 32 * TJ * wn)) * (y_bf16 ? 2u : 4u),
                    ldy, y_bf16);
    return;
  }
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TJ; ++b) {
      const int col = n0 + 32 * TJ * wn + 32 * b + (lane & 31);
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = m0 + 32 * TI * wm + 32 * a + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (full || (row < M && col < N)) {
          if (y_bf16)
            static_cast<uint16_t*>(Y)[(size_t)row * ldy + col] = f32_to_bf16_bits(acc[a][b][e]);
          else
            static_cast<float*>(Y)[(size_t)row * ldy + col] = acc[a][b][e];
        }
      }
    }
}

// Sum of the split-K partial products part[0..ks-1][M][N] (row stride N), in
// segment order, to Y (row stride ldy) in float32 or bf16.  Thread t handles
// four consecutive columns of one row.  With vec (N and ldy multiples of 4,
// Y 16-byte aligned) a full quad is read as one 16-byte load per segment --
// every segment's load issued before the adds -- and written as one store;
// the order of the adds, hence every bit, is that of the scalar path.
__global__ __launch_bounds__(256) void splitk_sum_kernel(const float* __restrict__ part, int ks, int M, int N,
                                                         void* __restrict__ Y, int64_t ldy, int y_bf16, int vec) {
  const int q = (N + 3) >> 2;  // column quads per row
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (id >= (int64_t)M * q) return;
  const int row = (int)(id / q), col = (int)(id - (int64_t)row * q) * 4;
  const int64_t MN = (int64_t)M * N;
  const float* p = part + (int64_t)row * N + col;
  if (vec && col + 3 < N) {
    f32x4 seg[kMaxSplit];
#pragma unroll
    for (int s = 0; s < kMaxSplit; ++s)
      if (s < ks) seg[s] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p + s * MN));
    f32x4 v = seg[0];
#pragma unroll
    for (int s = 1; s < kMaxSplit; ++s)
      if (s < ks) v += seg[s];
    if (y_bf16) {
      typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
      *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(Y) + row * ldy + col) =
          (u32x2){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    } else {
      *reinterpret_cast<f32x4*>(static_cast<float*>(Y) + row * ldy + col) = v;
    }
    return;
  }
  float v[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = col + j < N ? p[j] : 0.0f;
  for (int s = 1; s < ks; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (col + j < N) v[j] += p[s * MN + j];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (col + j >= N) break;
    if (y_bf16)
      static_cast<uint16_t*>(Y)[row * ldy + col + j] = f32_to_bf16_bits(v[j]);
    else
      static_cast<float*>(Y)[row * ldy + col + j] = v[j];
  }
}

// ---- general tiles, two waves per SIMD --------------------------------------
// Workgroup tile BM (tokens) x BN (outputs) for the K the hand-scheduled tiles
// do not serve: not a multiple of 64, or past their range.  WAVES_M x WAVES_N waves; each owns a (BM/WAVES_M) x
// (BN/WAVES_N) sub-tile.  LDS holds two stages of the X tile and of the
// dequantized W tile; a K step runs the MFMAs of step k from one stage while
// the same waves dequantize step k+1 into the other, with the raw global data
// of step k+1 loaded into registers two steps earlier.  One workgroup barrier
// per K step.
template <int BM, int BN, int WAVES_M, int WAVES_N>
struct GemmCfg {
  static constexpr int kThreads = 64 * WAVES_M * WAVES_N;
  static constexpr int kWTM = BM / WAVES_M, kWTN = BN / WAVES_N;
  static constexpr int kTI = kWTM / 32, kTJ = kWTN / 32;
  static constexpr int kXChunks = BM * (kBK / 8) / kThreads;   // 16-byte X chunks per thread per step
  // Weight groups per step and per thread (threads past the step's groups --
  // whole waves, since BN * 2 is a multiple of 64 -- dequantize none).
  static constexpr int kStepGroups = BN * (kBK / kGroup);
  static constexpr int kWGroups = (kStepGroups + kThreads - 1) / kThreads;
  static constexpr int kWChunks = BN * (kBK / 8) / kThreads;   // 16-byte chunks of a bf16 W tile
  static constexpr int kLdsElems = 2 * (BM + BN) * kLdsStride;
  static_assert(kXChunks >= 1 && kWGroups >= 1, "tile too small for the thread count");
  static_assert(kTI >= 1 && kTJ >= 1, "wave tile below 32 x 32");
};

// Raw global data of one K step held by one thread: its X chunks and either
// the codes / scale / offset of its weight groups or its bf16 W chunks.
template <int XC, int WG, int WC>
struct GemmRegs {
  u32x4 x[XC];
  u32x4 q[WG];
  uint32_t s[WG], m[WG];
  u32x4 w[WC];
};

// WF: W is a packed Q4NX or MXFP4-variant matrix (blob), or bf16 [N][K].
template <int BM, int BN, int WAVES_M, int WAVES_N, int WF>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_kernel(
    const uint16_t* __restrict__ X, const uint8_t* __restrict__ blob, void* __restrict__ Y, int M, int N, int K,
    int ldy, int KB, int NS, int tiles_n, int y_bf16) {
  constexpr bool WQ4 = WF != kWBf16;  // packed weights
  using C = GemmCfg<BM, BN, WAVES_M, WAVES_N>;
  using Regs = GemmRegs<C::kXChunks, WQ4 ? C::kWGroups : 1, WQ4 ? 1 : C::kWChunks>;
  const uint16_t* const Wb = reinterpret_cast<const uint16_t*>(blob);
  extern __shared__ __attribute__((aligned(16))) uint16_t gl[];
  uint16_t* xs0 = gl;                              // [2][BM][72]
  uint16_t* ws0 = gl + 2 * BM * kLdsStride;        // [2][BN][72]

  int bm, bn;
  gemm_tile_of(blockIdx.x, gridDim.x, tiles_n, bm, bn);
  const int m0 = bm * BM, n0 = bn * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  f32x16 acc[C::kTI][C::kTJ];
#pragma unroll
  for (int a = 0; a < C::kTI; ++a)
#pragma unroll
    for (int b = 0; b < C::kTJ; ++b)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.0f;

  // Global loads of step k0 into registers.  Row and column indices are
  // clamped so every address is inside the operands; the values that belong
  // outside the matrices are zeroed only when the step is stored, so nothing
  // here waits for the loads to return.
  auto load_step = [&](Regs& R, int k0) {
#pragma unroll
    for (int i = 0; i < C::kXChunks; ++i) {
      const int ch = tid + i * C::kThreads;       // chunk: row ch/8, columns 8(ch%8)..+7
      const int r = ch >> 3, kk = k0 + 8 * (ch & 7);
      R.x[i] = *reinterpret_cast<const u32x4*>(X + (size_t)min(m0 + r, M - 1) * K + min(kk, K - 8));
    }
    if constexpr (!WQ4) {
#pragma unroll
      for (int i = 0; i < C::kWChunks; ++i) {
        const int ch = tid + i * C::kThreads;     // chunk: W row ch/8, columns 8(ch%8)..+7
        const int r = ch >> 3, kk = k0 + 8 * (ch & 7);
        R.w[i] = *reinterpret_cast<const u32x4*>(Wb + (size_t)min(n0 + r, N - 1) * K + min(kk, K - 8));
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < C::kWGroups; ++i) {
      const int gi = tid + i * C::kThreads;       // group: row gi/2, half gi%2 of the K step
      if (C::kStepGroups % C::kThreads != 0 && gi >= C::kStepGroups) break;  // wave-uniform
      const int r = gi >> 1, gk = min(k0 + kGroup * (gi & 1), K - kGroup);
      const int gn = n0 + r, rr = gn & 31;
      const int j = gk >> 8, c = (gk & 255) >> 5;
      const uint8_t* blk = blob + ((size_t)min(gn >> 5, NS - 1) * KB + j) * wblock_bytes<WF>();
      R.q[i] = load_codes(blk + 128 * rr + 16 * c);
      if constexpr (WF == kWMX) {
        R.s[i] = load_u8(blk + kCodeBytes + 8 * rr + c);
      } else {
        R.s[i] = load_u16(blk + kCodeBytes + 2 * (8 * rr + c));
        R.m[i] = load_u16(blk + kCodeBytes + kScaleBytes + 2 * (8 * rr + c));
      }
    }
  };

  // Zero what lies outside the matrices, dequantize the weight groups (Eq. 3
  // in float32, rounded to bf16) and write X and W of step k0 to LDS stage st.
  auto store_step = [&](const Regs& R, int st, int k0) {
    uint16_t* xs = xs0 + st * BM * kLdsStride;
    uint16_t* ws = ws0 + st * BN * kLdsStride;
#pragma unroll
    for (int i = 0; i < C::kXChunks; ++i) {
      const int ch = tid + i * C::kThreads;
      const bool ok = m0 + (ch >> 3) < M && k0 + 8 * (ch & 7) < K;
      *reinterpret_cast<u32x4*>(xs + (ch >> 3) * kLdsStride + 8 * (ch & 7)) = ok ? R.x[i] : (u32x4){0u, 0u, 0u, 0u};
    }
    if constexpr (!WQ4) {
#pragma unroll
      for (int i = 0; i < C::kWChunks; ++i) {
        const int ch = tid + i * C::kThreads;
        const bool ok = n0 + (ch >> 3) < N && k0 + 8 * (ch & 7) < K;
        *reinterpret_cast<u32x4*>(ws + (ch >> 3) * kLdsStride + 8 * (ch & 7)) = ok ? R.w[i] : (u32x4){0u, 0u, 0u, 0u};
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < C::kWGroups; ++i) {
      const int gi = tid + i * C::kThreads;
      if (C::kStepGroups % C::kThreads != 0 && gi >= C::kStepGroups) break;  // wave-uniform
      const bool ok = ((n0 + (gi >> 1)) >> 5) < NS && k0 + kGroup * (gi & 1) < K;
      const u32x4 q = ok ? R.q[i] : (u32x4){0u, 0u, 0u, 0u};
      if constexpr (WF == kWMX) {
        const float Xs = ok ? e8m0_f32(R.s[i]) : 0.0f;
        u32x4* wd = reinterpret_cast<u32x4*>(ws + (gi >> 1) * kLdsStride + kGroup * (gi & 1));
#pragma unroll
        for (int v = 0; v < 4; ++v) wd[v] = mx8_bf16(q[v], Xs);
        continue;
      }
      const float d512 = ok ? bf16_to_f32(R.s[i]) * 512.0f : 0.0f, m = ok ? bf16_to_f32(R.m[i]) : 0.0f;
      u32x4* wd = reinterpret_cast<u32x4*>(ws + (gi >> 1) * kLdsStride + kGroup * (gi & 1));
#pragma unroll
      for (int v = 0; v < 4; ++v) wd[v] = dequant8_bf16(q[v], d512, m);
    }
  };

  // The MFMAs of one K step from LDS stage st.
  auto mma_step = [&](int st) {
    const uint16_t* xs = xs0 + st * BM * kLdsStride;
    const uint16_t* ws = ws0 + st * BN * kLdsStride;
#pragma unroll
    for (int kq = 0; kq < kBK / 16; ++kq) {
      const int kk = kq * 16 + 8 * (lane >> 5);
      bf16x8 af[C::kTI], bfr[C::kTJ];
#pragma unroll
      for (int a = 0; a < C::kTI; ++a)
        af[a] = *reinterpret_cast<const bf16x8*>(xs + (C::kWTM * wm + 32 * a + (lane & 31)) * kLdsStride + kk);
#pragma unroll
      for (int b = 0; b < C::kTJ; ++b)
        bfr[b] = *reinterpret_cast<const bf16x8*>(ws + (C::kWTN * wn + 32 * b + (lane & 31)) * kLdsStride + kk);
#pragma unroll
      for (int a = 0; a < C::kTI; ++a)
#pragma unroll
        for (int b = 0; b < C::kTJ; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[a], bfr[b], acc[a][b], 0, 0, 0);
    }
  };

  const int nsteps = (K + kBK - 1) / kBK;
  Regs R0, R1;
  load_step(R0, 0);
  store_step(R0, 0, 0);
  load_step(R0, kBK);
  load_step(R1, 2 * kBK);
  __syncthreads();
  int ks = 0;
  // Steady state, two steps per trip so the register sets stay static.
  for (; ks + 2 < nsteps; ks += 2) {
    mma_step(0);
    store_step(R0, 1, (ks + 1) * kBK);
    // Unconditional (addresses are clamped; data past the last step is never
    // stored), so the wait-count bookkeeping sees the same load order on every
    // trip and waits only for the register set being consumed.
    load_step(R0, (ks + 3) * kBK);
    __syncthreads();
    mma_step(1);
    store_step(R1, 0, (ks + 2) * kBK);
    load_step(R1, (ks + 4) * kBK);
    __syncthreads();
  }
  // Tail: one or two steps left; step ks+1 (if any) is in R0.
  if (ks + 1 < nsteps) {
    mma_step(ks & 1);
    store_step(R0, (ks + 1) & 1, (ks + 1) * kBK);
    __syncthreads();
    ++ks;
  }
  mma_step(ks & 1);

  if (m0 + BM <= M && n0 + BN <= N && ldy < kFastStoreMaxLdy) {
    store_wave_tile(acc,
                    static_cast<char*>(Y) + ((size_t)(unsigned)(m0 + C::kWTM * wm) * (unsigned)ldy +
                                             (unsigned)(n0 + C::kWTN * wn)) * (y_bf16 ? 2u : 4u),
                    ldy, y_bf16);
    return;
  }
  // Accumulator element e of lane l: column l%32, row 8(e/4) + 4(l/32) + e%4.
#pragma unroll
  for (int a = 0; a < C::kTI; ++a)
#pragma unroll
    for (int b = 0; b < C::kTJ; ++b) {
      const int col = n0 + C::kWTN * wn + 32 * b + (lane & 31);
      if (col >= N) continue;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = m0 + C::kWTM * wm + 32 * a + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
        if (row < M) {
          if (y_bf16)
            static_cast<uint16_t*>(Y)[(size_t)row * ldy + col] = f32_to_bf16_bits(acc[a][b][e]);
          else
            static_cast<float*>(Y)[(size_t)row * ldy + col] = acc[a][b][e];
        }
      }
    }
}

// ---- few rows: K split over the waves of a workgroup -------------------------
// For products with too few tiles of the kernels above to fill the CUs: short
// prompts, batches of decoding users, the last chunk of a prompt.  There the
// latency of the operand loads bounds gemm_kernel (one K step of a
// 128 x 64 tile took 0.7 us with 8 us of matrix work in 256 of them).  A
// workgroup owns 16 MT rows x 16 NT outputs and all of K; its W waves deal the
// 128-column units of K out among themselves (unit u to wave u % W), each wave
// computing the whole tile over its units without a barrier, and the W partial
// tiles are added in wave order through LDS at the end.  Splitting K rather
// than the tile over the waves keeps every X fragment and every dequantized
// weight in one wave, so nothing is read or converted twice, and all of a CU's
// waves have loads in flight.
// A unit of W (half a block) and of X go through the wave's own LDS slot:
// loaded with whole 64-byte (codes) and 256-byte (X) row pieces, written with
// padded rows (272 bytes for X, 80 for codes), and read back in
// the operand layout of v_mfma_f32_16x16x32_bf16: lane l holds row l % 16 and
// group l / 16 of the unit, whose 8-column runs are the fragments of four
// MFMAs.  (Loading the fragments straight from memory, 16 bytes per row and
// lane, took 20 instead of 16 us on a 32-row tile: the address unit handles
// such a load at a quarter of the rate.)  A wave's LDS instructions are
// carried out in order, so one slot per wave is enough.
// Measured on MI355X, Q4NX weights (plans of gemm_kernel -> this one, us):
// Gemma3-1B at 16 rows q/k/v 14.7 -> 4.2, o 13.4 -> 4.0, gate/up 16.4 -> 7.1,
// down 67.5 -> 9.0; 4B at 77 rows 29.0 -> 9.7, 23.9 -> 6.9, 41.5 -> 30.9,
// 100 -> 18.4.  Whole calls through q4nx_gemm_ex: eight 1B layers at 16 rows
// 869 -> 181 us (then bound by the caller), four 4B layers at 77 rows 816 ->
// 220 us, two at 512 rows 541 -> 301 us.
// What bounds it: one wave per SIMD does a unit's LDS writes, fragment reads,
// dequantization and MFMAs one after another.  Of a wave's cycles at 4B and 77
// rows (counters; q/k/v, o and down, gate/up): VALU 28, 38 and 33%, MFMA 11, 12
// and 19%, LDS instructions 11, 12 and 9% (28 to 31% of the LDS cycles are bank
// conflicts), waiting for memory or LDS data 27, 25 and 18%, for the LDS queue 3
// to 5%.
// Tiles of 80 and 96 columns: an X fragment read and an X row staged serve more
// outputs, and products of many columns take one round of tiles where 64 columns
// needed two.  4B gate/up at 77 rows 31.1 -> 21.5 us, 27B gate/up at 77 rows 96
// -> 77, 27B o at 300 rows 31.8 -> 29.7 (MXFP4 28.0 -> 25.3).  (128 columns
// spill or were slower.)  bf16 weights run the same tiles, X in two passes where
// the LDS does not hold both operands' rows, and one unit of W ahead where the
// registers do not hold two: as 64 x 64 tiles instead, and the smaller ones
// spilling at two waves per SIMD, 77 x 20480 x 2560 took 47.6 us (now 29.4),
// 223 x 5376 x 4096 41.7 (26.7), 226 x 2560 x 10240 94.8 (40.5).
// The order of every sum is fixed by M, N and K, and is the same for the three
// weight operands, so they agree bit for bit on the same bf16 weights.
constexpr int kKsUnit = 128;              // columns of K per unit
constexpr int kKsRow = 2 * kKsUnit + 16;  // LDS bytes per staged bf16 row
constexpr int kKsCodeRow = 80;            // LDS bytes per staged row of codes

// One unit of W as loaded.  Packed: codes of 16 rows per load (4 lanes per
// row), scale and offset of row l % 16, group l / 16.  bf16: 4 rows per load.
template <int NT, int WF>
struct KsUnit {
  u32x4 q[NT];
  uint32_t s[NT], m[NT];
};
template <int NT>
struct KsUnit<NT, kWBf16> {
  u32x4 q[4 * NT];
};

// Blocks of 16 rows of X staged at a time.  The LDS holds nine blocks of bf16
// rows per wave, so beside NT blocks of bf16 W the X of the larger tiles goes
// through in passes (each output still takes its products in the same order).
template <int MT, int NT, int WF>
constexpr int ks_x_blocks() {
  if (WF != kWBf16) return MT;
  const int passes = (MT + 8 - NT) / (9 - NT);
  return (MT + passes - 1) / passes;
}
template <int MT, int NT, int WF>
constexpr int ks_wave_lds() {
  return 16 * ks_x_blocks<MT, NT, WF>() * kKsRow + 16 * NT * (WF == kWBf16 ? kKsRow : kKsCodeRow);
}
template <int MT, int NT, int W, int WF>
constexpr int ks_lds_bytes() {
  return W * std::max(ks_wave_lds<MT, NT, WF>(), MT * NT * 1024);
}

// A tile of which the LDS holds one takes the whole register file (one wave per SIMD).
template <int MT, int NT, int W, int WF>
__global__ __launch_bounds__(64 * W, (ks_lds_bytes<MT, NT, W, WF>() > 80 * 1024 ? 1 : 2)) void gemm_ks_kernel(
    const uint16_t* __restrict__ X, const uint8_t* __restrict__ wsrc, void* __restrict__ Y, int M, int N, int K,
    int ldy, int KB, int NS, int tiles_n, int y_bf16) {
  constexpr int kBB = wblock_bytes<WF>();
  constexpr int kXI = 4 * MT;                 // X loads (4 rows each) per unit
  constexpr uint32_t kPastEnd = 0x7FFFFFF0u;  // beyond every descriptor: loads return 0
  extern __shared__ __attribute__((aligned(16))) uint16_t gl[];

  int bm, bn;
  gemm_tile_of(blockIdx.x, gridDim.x, tiles_n, bm, bn);
  const int m0 = bm * 16 * MT, n0 = bn * 16 * NT;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, h = lane >> 4;
  uint8_t* const xs = reinterpret_cast<uint8_t*>(gl) + wave * ks_wave_lds<MT, NT, WF>();
  constexpr int kXB = ks_x_blocks<MT, NT, WF>();
  uint8_t* const ws = xs + 16 * kXB * kKsRow;

  const int rows_x = min(16 * MT, M - m0);
  const __amdgpu_buffer_rsrc_t rsx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(X + (size_t)m0 * K), (short)0, rows_x * K * 2, 0x00020000);
  // Packed W: the strips that hold rows n0 .. n0 + 16 NT - 1 (n0 may lie in the middle of one).
  const int s0 = n0 >> 5, r0 = n0 & 31, nst = min((r0 + 16 * NT + 31) >> 5, NS - s0), rows_w = min(16 * NT, N - n0);
  const __amdgpu_buffer_rsrc_t rsw =
      WF != kWBf16 ? __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wsrc + (size_t)s0 * KB * kBB), (short)0,
                                                       nst * KB * kBB, 0x00020000)
                   : __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(wsrc + (size_t)n0 * K * 2), (short)0,
                                                       rows_w * K * 2, 0x00020000);
  // Rows past M and strips past the matrix read 0 (their outputs are never stored).
  uint32_t vx[kXI];
#pragma unroll
  for (int i = 0; i < kXI; ++i) {
    const int row = h + 4 * i;
    vx[i] = row < rows_x ? (uint32_t)(row * K + 8 * c) * 2 : kPastEnd;
  }
  constexpr int kVW = WF == kWBf16 ? 4 * NT : NT;
  uint32_t vw[kVW], vs[NT];
  if constexpr (WF != kWBf16) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int rq = r0 + 16 * t + (lane >> 2), rs = r0 + 16 * t + c;  // rows from strip s0's first
      vw[t] = (rq >> 5) < nst ? (uint32_t)((rq >> 5) * KB * kBB + 128 * (rq & 31) + 16 * (lane & 3)) : kPastEnd;
      vs[t] = (rs >> 5) < nst
                  ? (uint32_t)((rs >> 5) * KB * kBB + kCodeBytes + (WF == kWMX ? 1 : 2) * (8 * (rs & 31) + h))
                  : kPastEnd;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4 * NT; ++i) {
      const int row = h + 4 * i;
      vw[i] = row < rows_w ? (uint32_t)(row * K + 8 * c) * 2 : kPastEnd;
    }
  }
  // Units of this wave: wave + W i for i < nu.
  const int units = (K + kKsUnit - 1) / kKsUnit;
  const int nu = wave < units ? (units - wave + W - 1) / W : 0;

  // Loads of the wave's i-th unit.  Columns past K, and units past the wave's
  // last, read 0 (with the scalar offset inside the descriptor).
  // (X: registers j0 .. j1 - 1.)
  auto load_x = [&](u32x4 (&R)[kXI], int i, int j0, int j1) {
    const int k0 = (wave + W * i) * kKsUnit;
    const bool on = i < nu;  // uniform over the wave
    const uint32_t past = on && k0 + 8 * c < K ? 0 : kPastEnd;
    const int so = on ? 2 * k0 : 0;
#pragma unroll
    for (int j = j0; j < j1; ++j)
      R[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsx, vx[j] | past, so, 0));
  };
  auto load_w = [&](KsUnit<NT, WF>& R, int i) {
    const int u = wave + W * i, k0 = u * kKsUnit;
    const bool on = i < nu;
    if constexpr (WF == kWBf16) {
      const uint32_t past = on && k0 + 8 * c < K ? 0 : kPastEnd;
      const int so = on ? 2 * k0 : 0;
#pragma unroll
      for (int j = 0; j < 4 * NT; ++j)
        R.q[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsw, vw[j] | past, so, 0));
    } else {
      const uint32_t past = on ? 0 : kPastEnd;
      const int so = on ? (u >> 1) * kBB : 0, hb = u & 1;  // block, half of it
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        R.q[t] = __builtin_bit_cast(u32x4,
                                    __builtin_amdgcn_raw_buffer_load_b128(rsw, (vw[t] + 64 * hb) | past, so, kNtLoad));
        if constexpr (WF == kWMX) {
          R.s[t] = __builtin_amdgcn_raw_buffer_load_b8(rsw, (vs[t] + 4 * hb) | past, so, kNtLoad);
        } else {
          R.s[t] = __builtin_amdgcn_raw_buffer_load_b16(rsw, (vs[t] + 8 * hb) | past, so, kNtLoad);
          R.m[t] = __builtin_amdgcn_raw_buffer_load_b16(rsw, (vs[t] + kScaleBytes + 8 * hb) | past, so, kNtLoad);
        }
      }
    }
  };

  f32x4 acc[MT][NT];
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[a][b] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};

  // Two units of W ahead; one where two bf16 ones do not fit the registers.
  constexpr int kAhead = WF == kWBf16 && MT * NT >= 30 ? 1 : 2;
  u32x4 Xr[kXI];
  KsUnit<NT, WF> W0, W1;
  load_w(W0, 0);
  load_x(Xr, 0, 0, kXI);
  if constexpr (kAhead == 2) load_w(W1, 1);
  // One unit: its X and W registers go to LDS and are reloaded at once, then
  // the MFMAs from LDS.
  auto unit = [&](KsUnit<NT, WF>& Wr, int i) {
#pragma unroll
    for (int j = 0; j < 4 * kXB; ++j) *reinterpret_cast<u32x4*>(xs + (h + 4 * j) * kKsRow + 16 * c) = Xr[j];
    float d[NT], mo[NT];
    if constexpr (WF == kWBf16) {
#pragma unroll
      for (int j = 0; j < 4 * NT; ++j) *reinterpret_cast<u32x4*>(ws + (h + 4 * j) * kKsRow + 16 * c) = Wr.q[j];
    } else {
      // A group past K is scale and offset 0 whatever the padding holds.
      const bool in_k = (wave + W * i) * kKsUnit + kGroup * h < K;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        *reinterpret_cast<u32x4*>(ws + (16 * t + (lane >> 2)) * kKsCodeRow + 16 * (lane & 3)) = Wr.q[t];
        if constexpr (WF == kWMX) {
          d[t] = in_k ? e8m0_f32(Wr.s[t]) : 0.0f;
        } else {
          d[t] = in_k ? bf16_to_f32(Wr.s[t]) * 512.0f : 0.0f;
          mo[t] = in_k ? bf16_to_f32(Wr.m[t]) : 0.0f;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_sched_barrier(0);
    load_x(Xr, i + 1, 0, 4 * kXB);
    load_w(Wr, i + kAhead);
    u32x4 q[NT];
    if constexpr (WF != kWBf16) {
#pragma unroll
      for (int t = 0; t < NT; ++t) q[t] = *reinterpret_cast<const u32x4*>(ws + (16 * t + c) * kKsCodeRow + 16 * h);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      bf16x8 A[kXB];
#pragma unroll
      for (int a = 0; a < kXB; ++a)
        A[a] = *reinterpret_cast<const bf16x8*>(xs + (16 * a + c) * kKsRow + 64 * h + 16 * u);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        u32x4 b;
        if constexpr (WF == kWQ4NX) b = dequant8_bf16(q[t][u], d[t], mo[t]);
        else if constexpr (WF == kWMX) b = mx8_bf16(q[t][u], d[t]);
        else b = *reinterpret_cast<const u32x4*>(ws + (16 * t + c) * kKsRow + 64 * h + 16 * u);
#pragma unroll
        for (int a = 0; a < kXB; ++a)
          acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[a], __builtin_bit_cast(bf16x8, b), acc[a][t], 0, 0, 0);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    if constexpr (kXB < MT) {  // bf16 W: the other rows of X
      static_assert(MT <= 2 * kXB, "two passes");
      constexpr int kRest = MT - kXB;
#pragma unroll
      for (int j = 0; j < 4 * kRest; ++j)
        *reinterpret_cast<u32x4*>(xs + (h + 4 * j) * kKsRow + 16 * c) = Xr[4 * kXB + j];
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      __builtin_amdgcn_sched_barrier(0);
      load_x(Xr, i + 1, 4 * kXB, kXI);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        bf16x8 A[kRest];
#pragma unroll
        for (int a = 0; a < kRest; ++a)
          A[a] = *reinterpret_cast<const bf16x8*>(xs + (16 * a + c) * kKsRow + 64 * h + 16 * u);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const bf16x8 b = *reinterpret_cast<const bf16x8*>(ws + (16 * t + c) * kKsRow + 64 * h + 16 * u);
#pragma unroll
          for (int a = 0; a < kRest; ++a)
            acc[kXB + a][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[a], b, acc[kXB + a][t], 0, 0, 0);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    }
  };
  int i = 0;
  if constexpr (kAhead == 2) {
    for (; i + 1 < nu; i += 2) {
      unit(W0, i);
      unit(W1, i + 1);
    }
    if (i < nu) unit(W0, i);
  } else {
    for (; i < nu; ++i) unit(W0, i);
  }

  // Add the waves' partial tiles in wave order.  Element e of lane l of block
  // (a, t) is row 16a + 4h + e, column 16t + c.
  f32x4* const red = reinterpret_cast<f32x4*>(gl);
  __syncthreads();
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int t = 0; t < NT; ++t) red[((wave * MT + a) * NT + t) * 64 + lane] = acc[a][t];
  __syncthreads();
  for (int sl = wave; sl < MT * NT; sl += W) {
    f32x4 v = red[sl * 64 + lane];
#pragma unroll
    for (int p = 1; p < W; ++p) v += red[(p * MT * NT + sl) * 64 + lane];
    const int col = n0 + 16 * (sl % NT) + c, row = m0 + 16 * (sl / NT) + 4 * h;
    if (col >= N) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (row + e < M) {
        if (y_bf16)
          static_cast<uint16_t*>(Y)[(size_t)(row + e) * ldy + col] = f32_to_bf16_bits(v[e]);
        else
          static_cast<float*>(Y)[(size_t)(row + e) * ldy + col] = v[e];
      }
  }
}

// ---- launch planning ----------------------------------------------------------
// Tile shapes of the plan: 0 = 256 x 256, 1 = 256 x 128, 2 = 128 x 128, 3 =
// 128 x 64, as gemm_kernel (256 x 256: gemm256_kernel) computes them;
// where K allows, gemm_tile_kernel takes a region over (see kPlanWide).  The
// round costs below were measured with gemm_kernel.
struct GemmTile {
  int bm, bn;
  float round_cost;  // time of one full round (a tile on every CU), relative to shape 0
};
// Round costs measured on MI355X for the Gemma3 prefill projections (K = 5376).
constexpr GemmTile kGemmTiles[4] = {{256, 256, 1.0f}, {256, 128, 0.68f}, {128, 128, 0.52f}, {128, 64, 0.38f}};

// A rectangle of the output computed by one launch (ks > 1: by ks K segments
// of the 256 x 256 kernel and a second launch that adds their partials).
struct GemmRegion {
  int tile;
  int64_t m0, n0, M, N;
  int ks;
};

// Split K.  With a caller workspace, a 256 x 256 launch may run every tile as
// ks K segments on ks workgroups that write float32 partial products, which a
// second launch adds in segment order (deterministic).  It pays where a long
// K meets few tiles (Gemma3 down projections).  Split plans are costed in the
// planner's unit, a round of 256 x 256 tiles at the full K, through a time
// model fitted on MI355X: such a round over K columns takes about
// 40 + 0.0226 K us, and the sum streams its operands at about 5 TB/s after a
// ~5 us launch.
constexpr double kRoundFixedUs = 40.0, kRoundPerKUs = 0.0226;
constexpr double kSumLaunchUs = 5.0, kSumBytesPerUs = 5.0e6;
// (The round costs and this model were fitted to kernels that compute few of
// these tiles now.  They decide whether K is split, whether the weights are
// dequantized first (timed again on the present kernels: below) and the
// workspace a call asks for; other tiles compete by the times further down.)
constexpr int kMinSegmentSteps = 8;

static double round_us(int64_t K) { return kRoundFixedUs + kRoundPerKUs * (double)K; }

// K steps per segment when K is split into ks non-empty segments of at least
// kMinSegmentSteps steps each; 0 if it cannot be.
static int split_steps(int64_t K, int ks) {
  if (ks < 2 || K >= kWideMaxK) return 0;
  const int64_t nsteps = ceil_div(K, kBK), per = ceil_div(nsteps, ks);
  return (per >= kMinSegmentSteps && (ks - 1) * per < nsteps) ? (int)per : 0;
}

static int device_cus() { return current_device_cus(); }

// Chooses one launch, or two launches over a split of the rows or columns,
// minimising the estimated time: sum over launches of (rounds of tiles on the
// CUs) x (round cost of the tile shape), plus a small cost per extra launch.
// A launch whose last round is only partly filled still pays a whole round,
// so a shape with 336 256x256 tiles on 256 CUs is better done as one full
// round of 256 x 256 tiles and the rest in smaller tiles.  With split_ok, the
// whole product or the second region may also be split along K.
static int gemm_plan(int64_t M, int64_t N, int64_t K, int cus, bool split_ok, GemmRegion (&plan)[2],
                     double* est_us = nullptr) {
  const auto rounds = [&](int t, int64_t m, int64_t n) {
    return (double)ceil_div(ceil_div(m, kGemmTiles[t].bm) * ceil_div(n, kGemmTiles[t].bn), cus);
  };
  // Cost of an (m x n) region as ks K segments of 256 x 256 tiles plus the sum.
  const auto split_cost = [&](int64_t m, int64_t n, int ks) {
    const int per = split_steps(K, ks);
    if (!split_ok || per == 0) return 1e300;
    const double r = (double)ceil_div(ceil_div(m, 256) * ceil_div(n, 256) * ks, cus);
    const double sum_us = kSumLaunchUs + (4.0 * ks + 4.0) * (double)m * (double)n / kSumBytesPerUs;
    return (r * round_us((int64_t)per * kBK) + sum_us) / round_us(K);
  };
  double best = 1e300;
  int count = 0;
  for (int ks = 2; ks <= kMaxSplit; ++ks) {
    const double c = split_cost(M, N, ks);
    if (c < best) {
      best = c;
      plan[0] = {0, 0, 0, M, N, ks};
      count = 1;
    }
  }
  for (int a = 0; a < 4; ++a) {
    const double c1 = rounds(a, M, N) * kGemmTiles[a].round_cost;
    if (c1 < best) {
      best = c1;
      plan[0] = {a, 0, 0, M, N, 1};
      count = 1;
    }
    const int64_t tm = ceil_div(M, kGemmTiles[a].bm), tn = ceil_div(N, kGemmTiles[a].bn);
    const int64_t full = (tm * tn) / cus;  // whole rounds of shape a
    if (full < 1) continue;
    for (int dir = 0; dir < 2; ++dir) {
      // Largest leading block of rows (dir 0) or columns (dir 1) whose tiles
      // fit in the whole rounds; the rest goes to a smaller shape.
      const int64_t split = dir == 0 ? (full * cus / tn) * kGemmTiles[a].bm : (full * cus / tm) * kGemmTiles[a].bn;
      if (split <= 0 || split >= (dir == 0 ? M : N)) continue;
      const int64_t ma = dir == 0 ? split : M, na = dir == 0 ? N : split;
      const int64_t mb = dir == 0 ? M - split : M, nb = dir == 0 ? N : N - split;
      for (int b = a + 1; b < 4; ++b) {
        const double c2 = rounds(a, ma, na) * kGemmTiles[a].round_cost +
                          rounds(b, mb, nb) * kGemmTiles[b].round_cost + 0.02 + 0.001 * dir;
        if (c2 < best) {
          best = c2;
          plan[0] = {a, 0, 0, ma, na, 1};
          plan[1] = {b, dir == 0 ? split : 0, dir == 0 ? 0 : split, mb, nb, 1};
          count = 2;
        }
      }
      for (int ks = 2; ks <= kMaxSplit; ++ks) {
        const double c2 = rounds(a, ma, na) * kGemmTiles[a].round_cost + split_cost(mb, nb, ks) + 0.02 + 0.001 * dir;
        if (c2 < best) {
          best = c2;
          plan[0] = {a, 0, 0, ma, na, 1};
          plan[1] = {0, dir == 0 ? split : 0, dir == 0 ? 0 : split, mb, nb, ks};
          count = 2;
        }
      }
    }
  }
  if (est_us) *est_us = best * round_us(K);
  return count;
}

// Workspace bytes a plan needs: the regions run one after the other on one
// stream, so they share it.
static size_t plan_work_bytes(const GemmRegion* plan, int count) {
  size_t b = 0;
  for (int i = 0; i < count; ++i)
    if (plan[i].ks > 1) b = std::max(b, (size_t)plan[i].ks * (size_t)plan[i].M * (size_t)plan[i].N * sizeof(float));
  return b;
}

// Dequantize, then multiply.  The fused kernel dequantizes every weight once
// per row of output tiles (16 times at M = 4096).  With a workspace that holds
// W in bf16, a Q4NX product can dequantize each weight once instead (the
// dequant kernel streams at ~5.5 TB/s) and run the same plan on the bf16
// weights: the same bf16 values, the same MFMA chains and partial sums, so
// the same bits.  The fused kernel's extra work is Eq. 3 inside the K loop, so
// the two-phase route is taken when the dequantization pass is estimated below
// a share of the planned K-loop time: every Gemma3 27B product at M = 4096, the
// 4B gate/up and down products at M = 2048, not the 4B q/k/v and o products.
// (The MXFP4 variant's conversion is cheap enough that the fused kernel runs at
// the bf16 speed.)  Measured on MI355X both ways over the eleven stacked Gemma3
// products at M = 512 to 4096, 88 products: where it is taken the fused launches
// take up to 1.15 times as long (us: 4096 x 43008 x 5376 1552 against 1793, 2048 x
// 20480 x 2560 217 against 229, 2048 x 2560 x 10240 118 against 129), where it is
// not the two phases take up to 1.36 times as long (4096 x 1536 x 1152 23.2
// against 26.4, 1024 x 8192 x 5376 96 against 103); the wrong one is taken three
// times, for 3 to 4% (1536 x 20480 x 2560 172 against 165, 1280 x 8192 x 5376 117
// against 113, 1536 x 5376 x 21504 337 against 329).
constexpr double kDequantLaunchUs = 3.0, kDequantBytesPerUs = 5.5e6;
constexpr double kFusedExtraWide = 0.20, kFusedExtraSmall = 0.14;

// ---- the launches of a product ------------------------------------------------
// gemm_plan above decides how much workspace a product asks for and whether a
// part of it is split along K; what runs is the cheapest of that plan, one or
// two launches of gemm_tile_kernel, and one of gemm_ks_kernel, by the times
// below.  They were fitted on MI355X to launches over K = 1152 .. 21504 and 40
// to 640 tiles and predict those within about a tenth (several full rounds of
// 256 x 256 tiles with Q4NX weights take 1.2 times as long as with bf16 ones, where
// the table has 1.1).  Which of the three runs depends on M, N, K, the device
// and whether there is a workspace alone, so the three weight operands always
// take the same sums; the tiles, which do not change a bit, are chosen for the
// operand.

// A full round of gemm_tile_kernel's tiles over K columns takes fixed_us +
// slope K (slope_us: Q4NX weights dequantized in the K loop; bf16_us: the
// other operands); with a part u of the CUs at work the slope falls by
// `relief` (1 - u): the larger tiles are bound by what the whole chip shares.
struct WideTile {
  int ti, tj;
  float fixed_us, slope_us, bf16_us, relief;
};
constexpr WideTile kWideTiles[] = {{1, 2, 4.5f, 0.0067f, 0.0060f, 0.15f}, {2, 2, 5.0f, 0.0091f, 0.0082f, 0.20f},
                                   {3, 2, 6.4f, 0.0128f, 0.0113f, 0.25f}, {4, 2, 8.0f, 0.0152f, 0.0135f, 0.50f},
                                   {2, 4, 8.0f, 0.0171f, 0.0148f, 0.50f}, {5, 2, 8.5f, 0.0185f, 0.0165f, 0.50f},
                                   {4, 3, 9.0f, 0.0225f, 0.0182f, 0.50f}, {3, 4, 9.0f, 0.0240f, 0.0211f, 0.50f},
                                   {5, 3, 10.0f, 0.0295f, 0.0237f, 0.50f}, {4, 4, 9.5f, 0.0265f, 0.0242f, 0.50f}};
constexpr int kWideConfigs = (int)(sizeof(kWideTiles) / sizeof(kWideTiles[0]));
constexpr int kWideSquare = kWideConfigs - 1;  // 256 x 256
constexpr int kPlanWide[4] = {kWideSquare, 3, 1, 0};  // what computes a region of a plan, by its tile
constexpr int64_t kSquareLongK = 4096;
// Up to 448 columns of K the general kernel computes the 128 and 256 column
// tiles of two to four row blocks: gemm_tile_kernel's one wave per SIMD has too
// few steps to earn its longer start and end.  Measured on MI355X, gemm_tile_kernel
// against the general kernel (us, Q4NX and bf16 weights): 480 x 13328 x 64 12.6
// and 12.1 against 8.1 and 9.0, 272 x 9908 x 64 7.3 and 6.8 against 6.1 and 5.4,
// 741 x 7685 x 256 12.7 and 11.9 against 11.0 and 11.3, 1569 x 1451 x 384 10.1 and 9.1
// against 9.2 and 8.2, 1835 x 1257 x 448 10.8 and 9.5 against 10.2 and 8.9; level at K =
// 704 (384 x 5631).  The 64 x 128 tile and the larger ones stay ahead (339 x 4798
// x 128 5.6 against 6.1, 1266 x 8017 x 192 17.4 against 25.6).
constexpr int64_t kTileShortK = 512;
static int short_k_tile(int wide_tile, int64_t K) {  // tile of kGemmTiles, or -1: gemm_tile_kernel's own
  if (K >= kTileShortK || wide_tile < 1 || wide_tile > 3) return -1;
  return wide_tile == 1 ? 2 : 1;
}
// K that gemm_tile_kernel takes: whole steps, and 320 rows of X below 2^31 bytes.
static bool wide_ok(int64_t K) { return K % kBK == 0 && K < kWideMaxK / 2; }
constexpr double kExtraLaunchUs = 2.0;

static double wide_us(const WideTile& t, double tiles, double K, int cus, bool dequant) {
  const double full = std::floor(tiles / cus), u = tiles / cus - full;
  const double k_us = (dequant ? t.slope_us : t.bf16_us) * K;
  double us = full * (t.fixed_us + k_us);
  if (u > 0.0) us += t.fixed_us + k_us * (1.0 - t.relief * (1.0 - u));
  return us;
}

// Tiles of gemm_ks_kernel (16 mt rows x 16 nt outputs, K over `waves` waves):
// a tile takes fixed_us + unit_us per 128-column unit on a CU, a launch
// kKsLaunchUs more; with bf16 weights `bf16` times that (four times the bytes
// of W per tile, and X staged in two passes beside the larger tiles).
struct KsTile {
  int mt, nt, waves;
  float fixed_us, unit_us, bf16;
};
constexpr KsTile kKsTiles[] = {
    {1, 1, 8, 1.0f, 0.09f, 0.90f}, {1, 2, 4, 1.0f, 0.15f, 0.95f}, {2, 2, 4, 0.9f, 0.18f, 0.95f},
    {3, 2, 4, 1.6f, 0.24f, 0.95f}, {2, 4, 4, 1.8f, 0.31f, 1.03f}, {3, 4, 4, 3.4f, 0.36f, 1.05f},
    {4, 4, 4, 4.4f, 0.40f, 1.08f}, {5, 4, 4, 4.8f, 0.50f, 1.10f}, {6, 4, 4, 5.1f, 0.57f, 1.10f},
    {8, 4, 4, 6.6f, 0.675f, 1.20f}, {4, 5, 4, 6.0f, 0.49f, 1.15f}, {5, 5, 4, 7.0f, 0.55f, 1.30f},
    {4, 6, 4, 6.0f, 0.58f, 1.15f}, {5, 6, 4, 6.5f, 0.65f, 1.15f}, {6, 6, 4, 7.2f, 0.70f, 1.35f}};
constexpr int kKsConfigs = (int)(sizeof(kKsTiles) / sizeof(kKsTiles[0]));
constexpr double kKsLaunchUs = 3.2;
constexpr int64_t kKsMaxTiles = 16384;  // beyond it the chip is full many times over
// bf16 weights take about kOtherBf16 of the Q4NX times in the other launches,
// and no launch reads them faster than kBf16ReadBytesPerUs.  The few-rows tile
// that is the fastest for Q4NX weights runs for all operands (one order of the
// sums) unless Q4NX and bf16 together would lose more than the tables' error.
// Measured on MI355X, the few-rows tile against the other launches (Q4NX, bf16
// us): refused at 705 x 2944 x 2304 (24.7 and 27.2 against 25.5 and 19.7), 261 x
// 13309 x 2208 (46 and 56 against 38 and 38) and 391 x 12099 x 6560 (116 and
// 141 against 112 and 102); taken at 303 x 5419 x 4096 (29.8 and 36.6 against
// 31.5 and 31.1) and 77 x 20480 x 2560 (21.3 and 29.4 against 28.2 and 33.1).
constexpr double kOtherBf16 = 0.8, kBf16ReadBytesPerUs = 4.0e6, kKsMaxLoss = 1.18;

// What a full round of the plan's tiles (kGemmTiles) takes: those the general
// kernel still computes (K with a tail, or past the wide kernels' range) and
// 256 x 256 ones.  (round_us overestimates small launches; it only ranks the
// plan's own choices.)
constexpr double kTileFixedUs = 16.0, kTilePerKUs = 0.0237;
constexpr double kTileCost[4] = {0.88, 0.65, 0.50, 0.38};

struct WideRegion {
  int tile;  // of kWideTiles
  int64_t m0, n0, M, N;
};

// One launch of gemm_tile_kernel, or two over a split of the rows or columns
// (whole rounds of a large tile, then the rest), and their estimated time.
static int wide_plan(int64_t M, int64_t N, int64_t K, int cus, bool dequant, WideRegion (&plan)[2], double* est_us) {
  const auto tiles = [](const WideTile& t, int64_t m, int64_t n) {
    return (double)ceil_div(m, 64 * t.ti) * (double)ceil_div(n, 64 * t.tj);
  };
  double best = 1e300;
  int count = 0;
  for (int a = 0; a < kWideConfigs; ++a) {
    const double c = wide_us(kWideTiles[a], tiles(kWideTiles[a], M, N), (double)K, cus, dequant);
    if (c < best) {
      best = c;
      plan[0] = {a, 0, 0, M, N};
      count = 1;
    }
  }
  for (int a : {kWideSquare, 6, 3}) {  // 256 x 256, 256 x 192, 256 x 128
    const WideTile& t = kWideTiles[a];
    const int64_t tm = ceil_div(M, 64 * t.ti), tn = ceil_div(N, 64 * t.tj), full = tm * tn / cus;
    if (full < 1) continue;
    for (int dir = 0; dir < 2; ++dir) {
      // Largest leading block of rows (dir 0) or columns (dir 1) whose tiles
      // fit in the whole rounds.
      const int64_t split = dir == 0 ? (full * cus / tn) * 64 * t.ti : (full * cus / tm) * 64 * t.tj;
      if (split <= 0 || split >= (dir == 0 ? M : N)) continue;
      const int64_t ma = dir == 0 ? split : M, na = dir == 0 ? N : split;
      const int64_t mb = dir == 0 ? M - split : M, nb = dir == 0 ? N : N - split;
      const double ca = wide_us(t, tiles(t, ma, na), (double)K, cus, dequant) + kExtraLaunchUs;
      for (int b = 0; b < kWideConfigs; ++b) {
        const double c = ca + wide_us(kWideTiles[b], tiles(kWideTiles[b], mb, nb), (double)K, cus, dequant);
        if (c < best) {
          best = c;
          plan[0] = {a, 0, 0, ma, na};
          plan[1] = {b, dir == 0 ? split : 0, dir == 0 ? 0 : split, mb, nb};
          count = 2;
        }
      }
    }
  }
  *est_us = best;
  return count;
}

static double plan_us(const GemmRegion* plan, int count, int64_t K, int cus) {
  double us = 0.0;
  for (int i = 0; i < count; ++i) {
    const GemmRegion& r = plan[i];
    const GemmTile& t = kGemmTiles[r.tile];
    const double tiles = (double)ceil_div(r.M, t.bm) * (double)ceil_div(r.N, t.bn) * r.ks;
    if (r.ks == 1 && wide_ok(K)) {
      const WideTile& w = kWideTiles[kPlanWide[r.tile]];
      us += wide_us(w, (double)ceil_div(r.M, 64 * w.ti) * (double)ceil_div(r.N, 64 * w.tj), (double)K, cus, true);
    } else if (wide_ok(K)) {
      us += wide_us(kWideTiles[kWideSquare], tiles, (double)K / r.ks, cus, true);
    } else {
      us += std::ceil(tiles / cus) * kTileCost[r.tile] * (kTileFixedUs + kTilePerKUs * (double)K / r.ks);
    }
    if (r.ks > 1)
      us += kSumLaunchUs + (4.0 * r.ks + 4.0) * (double)r.M * (double)r.N / kSumBytesPerUs;
    if (i > 0) us += kExtraLaunchUs;
  }
  return us;
}

// The fastest gemm_ks_kernel tile for a product that takes `other` us
// otherwise, or -1 if none is faster or bf16 weights lose too much.
static int ks_choose(int64_t M, int64_t N, int64_t K, int cus, double other) {
  double best = other;
  int pick = -1;
  const double units = (double)ceil_div(K, kKsUnit);
  for (int i = 0; i < kKsConfigs; ++i) {
    const KsTile& t = kKsTiles[i];
    const int64_t tiles = ceil_div(M, 16 * t.mt) * ceil_div(N, 16 * t.nt);
    if (tiles > kKsMaxTiles) continue;
    // A CU with one tile more than the others takes that much longer, and of
    // the small tiles, two of which share a CU, nearly so: 1.25 rounds of them
    // measured 1.72-1.93 times one, 1.5 rounds 1.78-1.88, 2.5 rounds 2.75-2.9.
    const double full = (double)(tiles / cus), u = (double)tiles / cus - full;
    double load = full + (u > 0.0 ? t.mt * t.nt >= 16 ? 1.0 : 0.75 + 0.25 * u : 0.0);
    load = std::max(1.0, load);
    const double c = kKsLaunchUs + load * (t.fixed_us + units * t.unit_us);
    if (c < best) {
      best = c;
      pick = i;
    }
  }
  if (pick < 0) return -1;
  const double read = 2.0 * (double)N * (double)K / kBf16ReadBytesPerUs;
  const double bf16 = std::max(kKsTiles[pick].bf16 * best, read), other_bf16 = std::max(kOtherBf16 * other, read);
  if (best + bf16 > kKsMaxLoss * (other + other_bf16)) return -1;
  return pick;
}

struct GemmChoice {
  GemmRegion plan[2];
  int count;
  WideRegion wide[2];
  int wide_count;     // launches of gemm_tile_kernel instead of the plan (0: the plan)
  int ks;             // index into kKsTiles: one launch of gemm_ks_kernel instead of either; -1: not
  bool two_phase;
  size_t w_bytes;     // bf16 W at the start of the workspace (two-phase only)
  size_t part_bytes;  // split-K partial products after it
};

// (The workspace a call asks for is that of the plan, also where another launch
// leaves it unused: whether there is one is part of the choice, so reporting 0
// there would move a caller who then passes none to other sums.)
static GemmChoice gemm_choose(int wf, int64_t M, int64_t N, int64_t K, bool have_work) {
  GemmChoice c{};
  double est_us = 0.0;
  const int cus = device_cus();
  c.count = gemm_plan(M, N, K, cus, have_work, c.plan, &est_us);
  c.part_bytes = plan_work_bytes(c.plan, c.count);
  const double deq_us = kDequantLaunchUs + (kBlockBytes / (double)(kBlockRows * kBlockCols) + 2.0) * (double)N *
                                               (double)K / kDequantBytesPerUs;
  const double kloop_us = est_us * kRoundPerKUs * (double)K / round_us(K);
  const double extra = c.plan[0].tile == 0 ? kFusedExtraWide : kFusedExtraSmall;
  c.two_phase = have_work && wf == kWQ4NX && deq_us < extra * kloop_us;
  c.w_bytes = c.two_phase ? (size_t)ceil_div(N * K * 2, 256) * 256 : 0;
  double best = plan_us(c.plan, c.count, K, cus), wide = 0.0;
  // One chain over all of K does not take the place of a split one, although it
  // may be a few percent faster (699 -> 681 us on one product): its float32
  // sums are longer, and the error against 64 bits went from 3.4e-7 to 6.2e-7.
  // (gemm_ks_kernel's four sums are shorter than the segments'.)
  bool split = false;
  for (int i = 0; i < c.count; ++i) split = split || c.plan[i].ks > 1;
  if (wide_ok(K) && !split) {
    const int n = wide_plan(M, N, K, cus, true, c.wide, &wide);
    if (wide <= best) {
      best = wide;
      c.wide_count = n;
    }
  }
  c.ks = K < kWideMaxK ? ks_choose(M, N, K, cus, best) : -1;
  if (c.ks < 0 && c.wide_count > 0 && (wf != kWQ4NX || c.two_phase))
    c.wide_count = wide_plan(M, N, K, cus, false, c.wide, &wide);
  return c;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int WF>
static q4nx_status launch_gemm(int64_t M, int64_t N, int64_t K, const uint16_t* X, const void* blob, void* Y,
                               int64_t ldy, int y_bf16, hipStream_t stream) {
  using Cfg = GemmCfg<BM, BN, WAVES_M, WAVES_N>;
  const int64_t tiles_n = ceil_div(N, BN), tiles_m = ceil_div(M, BM);
  const size_t lds = sizeof(uint16_t) * Cfg::kLdsElems;
  auto kern = gemm_kernel<BM, BN, WAVES_M, WAVES_N, WF>;
  static LdsReservation lds_res;  // LDS above 64 KiB, requested once per device
  if (!lds_res.ensure(reinterpret_cast<const void*>(kern), (int)lds))
    return fail(Q4NX_ERR_HIP, "q4nx_gemm: cannot reserve LDS");
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_n * tiles_m)), dim3(Cfg::kThreads), lds, stream, X,
                     static_cast<const uint8_t*>(blob), Y, (int)M, (int)N, (int)K, (int)ldy,
                     (int)ceil_div(K, kBlockCols), (int)ceil_div(N, kBlockRows), (int)tiles_n, y_bf16);
  return Q4NX_OK;
}

template <bool KTAIL, int WF>
static q4nx_status launch_gemm256(int64_t M, int64_t N, int64_t K, const uint16_t* X, const void* blob, void* Y,
                                  int64_t ldy, int y_bf16, hipStream_t stream, int ks = 1, float* part = nullptr) {
  auto kern = gemm256_kernel<KTAIL, WF>;
  static LdsReservation lds_res;
  if (!lds_res.ensure(reinterpret_cast<const void*>(kern), kWideLdsBytes))
    return fail(Q4NX_ERR_HIP, "q4nx_gemm: cannot reserve LDS");
  const int64_t tiles_n = ceil_div(N, 256), tiles_m = ceil_div(M, 256);
  const int ksteps = ks > 1 ? split_steps(K, ks) : (int)ceil_div(K, kBK);
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_n * tiles_m), (unsigned)ks), dim3(kWideThreads), kWideLdsBytes,
                     stream, X, static_cast<const uint8_t*>(blob), Y, (int)M, (int)N, (int)K, (int)ldy,
                     (int)ceil_div(K, kBlockCols), (int)ceil_div(N, kBlockRows), (int)tiles_n, y_bf16, ksteps,
                     ks > 1 ? part : nullptr);
  return Q4NX_OK;
}

template <int TI, int TJ, int WF>
static q4nx_status launch_tile(int64_t M, int64_t N, int64_t K, const uint16_t* X, const void* w, void* Y, int64_t ldy,
                               int y_bf16, hipStream_t stream) {
  constexpr int D = TI * TJ <= 2 ? 4 : 2;
  auto kern = gemm_tile_kernel<TI, TJ, D, WF>;
  constexpr int lds = tile_lds_bytes<TI, TJ>();
  static LdsReservation lds_res;
  if (!lds_res.ensure(reinterpret_cast<const void*>(kern), lds))
    return fail(Q4NX_ERR_HIP, "q4nx_gemm: cannot reserve LDS");
  const int64_t tiles_n = ceil_div(N, 64 * TJ), tiles_m = ceil_div(M, 64 * TI);
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_n * tiles_m)), dim3(kWideThreads), lds, stream, X,
                     static_cast<const uint8_t*>(w), Y, (int)M, (int)N, (int)K, (int)ldy,
                     (int)ceil_div(K, kBlockCols), (int)ceil_div(N, kBlockRows), (int)tiles_n, y_bf16);
  return Q4NX_OK;
}

// X rows m0.., W rows n0.. (strips n0/32.. of a packed matrix) and Y at
// (m0, n0) of a region of the product, in the given weight format.
template <int WF>
static void region_operands(int64_t m0, int64_t n0, int64_t N, int64_t K, int y_bf16, const uint16_t*& X,
                            const void*& w, void*& Y) {
  X += m0 * K;
  w = static_cast<const uint8_t*>(w) +
      (WF != kWBf16 ? (n0 / kBlockRows) * ceil_div(K, kBlockCols) * wblock_bytes<WF>() : 2 * n0 * K);
  Y = static_cast<uint8_t*>(Y) + (m0 * N + n0) * (y_bf16 ? 2 : 4);
}

// The product by the general kernel with a tile of kGemmTiles (256 x 256:
// gemm256_kernel's K tail form, up to its range).
template <int WF>
static q4nx_status launch_general(int tile, int64_t M, int64_t N, int64_t K, const uint16_t* X, const void* w, void* Y,
                                  int64_t ldy, int y_bf16, hipStream_t stream) {
  switch (tile) {
    case 0:
      if (K >= kWideMaxK) return launch_gemm<256, 256, 2, 4, WF>(M, N, K, X, w, Y, ldy, y_bf16, stream);
      return launch_gemm256<true, WF>(M, N, K, X, w, Y, ldy, y_bf16, stream);
    case 1:
      // Q4NX weights as 16 waves of 32 x 64 (four per SIMD), which hide the
      // dequantization in the tile loads better than 8 waves of 64 x 64
      // (1999 x 2500 x 2016 40.3 -> 37.0 us, 261 x 13309 x 2208 40.3 -> 38.0, 741 x
      // 7685 x 256 12.2 -> 11.1); bf16 and MXFP4-variant weights run 8, ahead for
      // bf16 on 2040 x 3999 x 2592 (52.0 against 54.0) and 1 to 13% behind on the
      // five other products timed.  Same MFMA chains, same bits.
      if constexpr (WF == kWQ4NX) return launch_gemm<256, 128, 8, 2, WF>(M, N, K, X, w, Y, ldy, y_bf16, stream);
      else return launch_gemm<256, 128, 4, 2, WF>(M, N, K, X, w, Y, ldy, y_bf16, stream);
    case 2: return launch_gemm<128, 128, 2, 4, WF>(M, N, K, X, w, Y, ldy, y_bf16, stream);
    default: return launch_gemm<128, 64, 2, 2, WF>(M, N, K, X, w, Y, ldy, y_bf16, stream);
  }
}

template <int WF>
static q4nx_status launch_wide(const WideRegion& r, int64_t N, int64_t K, const uint16_t* X, const void* w, void* Y,
                               int y_bf16, hipStream_t stream) {
  region_operands<WF>(r.m0, r.n0, N, K, y_bf16, X, w, Y);
  if (const int t = short_k_tile(r.tile, K); t >= 0)
    return launch_general<WF>(t, r.M, r.N, K, X, w, Y, N, y_bf16, stream);
  switch (r.tile) {
    case 0: return launch_tile<1, 2, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
    case 1: return launch_tile<2, 2, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
    case 2: return launch_tile<3, 2, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
    case 3: return launch_tile<4, 2, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
    case 4: return launch_tile<2, 4, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
    case 5: return launch_tile<5, 2, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
    case 6: return launch_tile<4, 3, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
    case 7: return launch_tile<3, 4, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
    case 8: return launch_tile<5, 3, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
    default:
      // Over a long K gemm256_kernel's own placement of the same work is ahead
      // (bf16 weights, 27B gate/up's 160 x 16 tiles at K = 5376: 1427 against
      // 1486 us), over a short one the even spacing (1B gate/up at 1024 rows,
      // K = 1152: 44.1 against 40.9 us; level at K = 2560).
      if (K >= kSquareLongK) return launch_gemm256<false, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
      return launch_tile<4, 4, WF>(r.M, r.N, K, X, w, Y, N, y_bf16, stream);
  }
}

template <int MT, int NT, int W, int WF>
static q4nx_status launch_ks(int64_t M, int64_t N, int64_t K, const uint16_t* X, const void* w, void* Y, int y_bf16,
                             hipStream_t stream) {
  auto kern = gemm_ks_kernel<MT, NT, W, WF>;
  constexpr int lds = ks_lds_bytes<MT, NT, W, WF>();
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  static LdsReservation lds_res;
  if (!lds_res.ensure(reinterpret_cast<const void*>(kern), lds))
    return fail(Q4NX_ERR_HIP, "q4nx_gemm: cannot reserve LDS");
  const int64_t tiles_n = ceil_div(N, 16 * NT), tiles_m = ceil_div(M, 16 * MT);
  hipLaunchKernelGGL(kern, dim3((unsigned)(tiles_n * tiles_m)), dim3(64 * W), lds, stream, X,
                     static_cast<const uint8_t*>(w), Y, (int)M, (int)N, (int)K, (int)N,
                     (int)ceil_div(K, kBlockCols), (int)ceil_div(N, kBlockRows), (int)tiles_n, y_bf16);
  return Q4NX_OK;
}

// The product by gemm_ks_kernel with tile `cfg` of kKsTiles (the same for every operand).
template <int WF, int I = 0>
static q4nx_status launch_ks_config(int cfg, int64_t M, int64_t N, int64_t K, const uint16_t* X, const void* w,
                                    void* Y, int y_bf16, hipStream_t stream) {
  if constexpr (I + 1 < kKsConfigs)
    if (cfg != I) return launch_ks_config<WF, I + 1>(cfg, M, N, K, X, w, Y, y_bf16, stream);
  constexpr KsTile t = kKsTiles[I];
  return launch_ks<t.mt, t.nt, t.waves, WF>(M, N, K, X, w, Y, y_bf16, stream);
}

// One region of a plan, an ordinary smaller problem.
template <int WF>
static q4nx_status launch_region(const GemmRegion& r, int64_t N, int64_t K, const uint16_t* Xr, const void* Wr,
                                 void* Yr, int y_bf16, hipStream_t stream, float* work) {
  if (r.ks == 1 && wide_ok(K))
    return launch_wide<WF>({kPlanWide[r.tile], r.m0, r.n0, r.M, r.N}, N, K, Xr, Wr, Yr, y_bf16, stream);
  region_operands<WF>(r.m0, r.n0, N, K, y_bf16, Xr, Wr, Yr);
  if (r.ks > 1) {
    // Partials [ks][r.M][r.N] in the workspace, then their sum into Y.
    const q4nx_status st = K % kBK != 0
                               ? launch_gemm256<true, WF>(r.M, r.N, K, Xr, Wr, Yr, r.N, y_bf16, stream, r.ks, work)
                               : launch_gemm256<false, WF>(r.M, r.N, K, Xr, Wr, Yr, r.N, y_bf16, stream, r.ks, work);
    if (st != Q4NX_OK) return st;
    const int64_t threads = r.M * ceil_div(r.N, 4);
    const int vec = r.N % 4 == 0 && N % 4 == 0 && aligned(Yr, 16);
    hipLaunchKernelGGL(splitk_sum_kernel, dim3((unsigned)ceil_div(threads, 256)), dim3(256), 0, stream, work, r.ks,
                       (int)r.M, (int)r.N, Yr, N, y_bf16, vec);
    return Q4NX_OK;
  }
  return launch_general<WF>(r.tile, r.M, r.N, K, Xr, Wr, Yr, N, y_bf16, stream);
}

// The launches of gemm_tile_kernel, or the plan's.
template <int WF>
static q4nx_status launch_planned(const GemmChoice& c, int64_t N, int64_t K, const uint16_t* X, const void* w, void* Y,
                                  int y_bf16, hipStream_t stream, float* part) {
  q4nx_status st = Q4NX_OK;
  for (int i = 0; i < c.wide_count && st == Q4NX_OK; ++i)
    st = launch_wide<WF>(c.wide[i], N, K, X, w, Y, y_bf16, stream);
  if (c.wide_count == 0)
    for (int i = 0; i < c.count && st == Q4NX_OK; ++i)
      st = launch_region<WF>(c.plan[i], N, K, X, w, Y, y_bf16, stream, part);
  return st;
}

static q4nx_status check_launch(const char* fn);

// Validation shared by the matrix-product entry points, then the planned
// launches (split along K only when a workspace is given).
template <int WF>
static q4nx_status gemm_entry(int64_t M, int64_t N, int64_t K, const uint16_t* d_X, const void* d_W, void* d_Y,
                              q4nx_dtype y_dtype, void* d_work, size_t work_bytes, hipStream_t stream,
                              const char* fn) {
  clear_error();
  if (q4nx_status st = check_shape(N, K, fn)) return st;
  if (M <= 0 || M > Q4NX_MAX_DIM) return fail(Q4NX_ERR_SHAPE, std::string(fn) + ": M must lie in 1..2^30");
  if (!d_X || !d_W || !d_Y) return fail(Q4NX_ERR_INVALID_ARG, std::string(fn) + ": NULL pointer");
  if (y_dtype != Q4NX_F32 && y_dtype != Q4NX_BF16)
    return fail(Q4NX_ERR_INVALID_ARG, std::string(fn) + ": unknown y_dtype");
  if (!aligned(d_X, 16) || !aligned(d_W, 16) || !aligned(d_Y, 16))
    return fail(Q4NX_ERR_ALIGNMENT, std::string(fn) + (WF != kWBf16 ? ": X, blob and Y need 16-byte alignment"
                                                                    : ": X, W and Y need 16-byte alignment"));
  if (M * N > (int64_t(1) << 40)) return fail(Q4NX_ERR_SHAPE, std::string(fn) + ": problem too large for one launch");
  if (d_work && !aligned(d_work, 16)) return fail(Q4NX_ERR_ALIGNMENT, std::string(fn) + ": work needs 16-byte alignment");
  const GemmChoice c = gemm_choose(WF, M, N, K, d_work != nullptr);
  if (c.w_bytes + c.part_bytes > work_bytes)
    return fail(Q4NX_ERR_BUFFER_TOO_SMALL, std::string(fn) + ": work_bytes < q4nx_gemm_workspace_size(...)");
  const int y_bf16 = y_dtype == Q4NX_BF16;
  float* part = reinterpret_cast<float*>(static_cast<uint8_t*>(d_work) + c.w_bytes);
  q4nx_status st = Q4NX_OK;
  if (c.ks >= 0) {
    st = launch_ks_config<WF>(c.ks, M, N, K, d_X, d_W, d_Y, y_bf16, stream);
  } else if (c.two_phase) {
    const int64_t KB = ceil_div(K, kBlockCols), nblocks = ceil_div(N, kBlockRows) * KB;
    hipLaunchKernelGGL((dequant_kernel<kWQ4NX, true>), dim3((unsigned)std::min<int64_t>(nblocks, int64_t(1) << 20)),
                       dim3(256), 0, stream, static_cast<const uint8_t*>(d_W), N, K, KB, nblocks, d_work);
    st = launch_planned<kWBf16>(c, N, K, d_X, d_work, d_Y, y_bf16, stream, part);
  } else {
    st = launch_planned<WF>(c, N, K, d_X, d_W, d_Y, y_bf16, stream, part);
  }
  if (st != Q4NX_OK) return st;
  return check_launch(fn);
}

static q4nx_status check_launch(const char* fn) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(Q4NX_ERR_HIP, std::string(fn) + ": " + hipGetErrorString(e));
  return Q4NX_OK;
}

// The kernels that a choice runs, as launch_wide and launch_region pick them.
static std::string launches_text(const GemmChoice& c, int wf, int64_t K) {
  const auto size = [](int m, int n) { return std::to_string(m) + "x" + std::to_string(n); };
  const auto wide = [&](int tile) {
    const WideTile& t = kWideTiles[tile];
    if (const int g = short_k_tile(tile, K); g >= 0) return "general " + size(kGemmTiles[g].bm, kGemmTiles[g].bn);
    return (tile == kWideSquare && K >= kSquareLongK ? "gemm256 " : "tile ") + size(64 * t.ti, 64 * t.tj);
  };
  if (c.ks >= 0) return "ks " + size(16 * kKsTiles[c.ks].mt, 16 * kKsTiles[c.ks].nt);
  std::string s = wf == kWQ4NX && c.two_phase ? "dequant" : "";
  const auto add = [&](const std::string& l) { s += (s.empty() ? "" : " + ") + l; };
  for (int i = 0; i < c.wide_count; ++i) add(wide(c.wide[i].tile));
  for (int i = 0; c.wide_count == 0 && i < c.count; ++i) {
    const GemmRegion& r = c.plan[i];
    if (r.ks > 1) add("split" + std::to_string(r.ks) + " 256x256");
    else if (wide_ok(K)) add(wide(kPlanWide[r.tile]));
    else add((r.tile == 0 && K < kWideMaxK ? "gemm256 " : "general ") + size(kGemmTiles[r.tile].bm, kGemmTiles[r.tile].bn));
  }
  return s;
}

// Row-group size: whole strips when there are enough of them to keep at least
// ~160 CUs streaming (one CU sustains ~55 GB/s of the ~7 TB/s), else halves or
// quarters of strips.  `strips` is the number of strips of the whole launch.
static int gemv_tq(int64_t strips) {
  if (strips >= 160) return 4;
  if (strips * 2 >= 160) return 2;
  return 1;
}

// Waves per workgroup (they split K).  A power of two, so that workgroups tile
// the 16 waves a CU holds at this kernel's register budget; fewer waves per
// row group when the launch has many row groups (longer streams per wave),
// more when it has few (more parallelism per strip).  Capped so every wave
// owns at least one block of every job.  Measured on MI355X over the Gemma3
// 1B/4B/27B projection shapes.
static int gemv_waves(int64_t row_groups, int min_kb) {
  int w = row_groups >= 4096 ? 2 : row_groups >= 512 ? 4 : row_groups >= 128 ? 8 : 16;
  while (w > 1 && w > min_kb) w >>= 1;
  return w;
}

template <int F>
static q4nx_status gemv_launch(const q4nx_gemv_desc* descs, int count, q4nx_dtype y_dtype, hipStream_t stream,
                               const char* fn) {
  clear_error();
  if (!descs || count < 1 || count > Q4NX_MAX_BATCH)
    return fail(Q4NX_ERR_INVALID_ARG, std::string(fn) + ": need 1..8 descriptors");
  if (y_dtype != Q4NX_F32 && y_dtype != Q4NX_BF16)
    return fail(Q4NX_ERR_INVALID_ARG, std::string(fn) + ": unknown y_dtype");
  int64_t strips = 0;
  for (int i = 0; i < count; ++i) {
    const q4nx_gemv_desc& d = descs[i];
    if (q4nx_status st = check_shape(d.N, d.K, fn)) return st;
    if (!d.blob || !d.x || !d.y) return fail(Q4NX_ERR_INVALID_ARG, std::string(fn) + ": NULL pointer");
    if (!aligned(d.blob, 16) || !aligned(d.x, 16) || !aligned(d.y, 4))
      return fail(Q4NX_ERR_ALIGNMENT, std::string(fn) + ": blob/x need 16-byte, y 4-byte alignment");
    strips += ceil_div(d.N, kBlockRows);
  }
  int min_kb = 1 << 30, max_kb = 0;
  for (int i = 0; i < count; ++i) {
    min_kb = std::min<int>(min_kb, (int)ceil_div(descs[i].K, kBlockCols));
    max_kb = std::max<int>(max_kb, (int)ceil_div(descs[i].K, kBlockCols));
  }
  // Launches of 80-159 strips take the streaming form with half-strip row
  // groups, 8 waves each.  Measured on MI355X in whole Gemma3 decode steps:
  // the 4B step 3% faster (its q/k/v, o and down launches); with quarter-strip
  // groups at 160-256 strips the 27B step was 2% slower (although each of
  // those launch types alone, repeated, ran 2-5% faster), so those launches
  // keep gemv_kernel.
  const bool streaming = max_kb <= kGemvChunkBlocks && strips >= 80 && strips < 160;
  const int tq = streaming ? 2 : gemv_tq(strips);
  int waves = streaming ? 8 : gemv_waves(strips * (4 / tq), min_kb);
  while (waves > 1 && waves > min_kb) waves >>= 1;
  GemvJob jobs[Q4NX_MAX_BATCH] = {};
  int64_t wg = 0;
  for (int i = 0; i < count; ++i) {
    const q4nx_gemv_desc& d = descs[i];
    GemvJob& J = jobs[i];
    J.blob = static_cast<const uint8_t*>(d.blob);
    J.x = d.x;
    J.y = d.y;
    J.N = (int)d.N;
    J.K = (int)d.K;
    J.nrg = (int)ceil_div(d.N, kBlockRows) * (4 / tq);
    // One workgroup per row group (the hardware keeps every CU fed as
    // workgroups retire); the loop over row groups only engages past 2^20.
    J.nwg = std::min(J.nrg, 1 << 20);
    J.wg_begin = (int)wg;
    wg += J.nwg;
  }
  const int flags = (y_dtype == Q4NX_BF16 ? kGemvBf16Out : 0) | count << kGemvJobsShift;
  // LDS of both kernels (static): the row sums and one x slot per wave.
  constexpr int64_t lds = sizeof(float) * (kRedFloats + kGemvMaxWaves * kGroupsPerRow * kGroupPadDw);
  const dim3 block(64 * waves);
  if (streaming) {
    // Streaming form: a bounded grid (workgroups per CU as the LDS allows, at
    // most kGemvStreamPerCu), dealt to the jobs in proportion to their row
    // groups; each workgroup walks its job's row groups r0, r0 + nwg, ...
    const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(kGemvStreamPerCu, (160 * 1024) / lds));
    const int64_t total_rg = strips * (4 / tq), budget = (int64_t)device_cus() * per_cu;
    int64_t sw = 0;
    for (int i = 0; i < count; ++i) {
      GemvJob& J = jobs[i];
      J.nwg = (int)std::max<int64_t>(1, std::min<int64_t>(J.nrg, (budget * J.nrg + total_rg - 1) / total_rg));
      J.wg_begin = (int)sw;
      sw += J.nwg;
    }
    wg = sw;
  }
  GemvRest rest;
  std::copy(jobs + 1, jobs + Q4NX_MAX_BATCH, rest.job);
  const GemvJob& J = jobs[0];
  const auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)wg), block, 0, stream, J.blob, J.x, J.y, J.N, J.K, J.nrg, J.nwg, waves,
                       flags, rest);
  };
  if (streaming) launch(gemv_stream_kernel<2, kGemvDepth2, F>);
  else if (tq == 4) launch(gemv_kernel<4, kGemvDepth4, F>);  // x is staged per wave in static LDS
  else if (tq == 2) launch(gemv_kernel<2, kGemvDepth2, F>);
  else launch(gemv_kernel<1, kGemvDepth1, F>);
  return check_launch(fn);
}

template <int F>
static q4nx_status dequant_entry(const void* d_blob, int64_t N, int64_t K, void* d_W, q4nx_dtype w_dtype,
                                 hipStream_t stream, const char* fn) {
  clear_error();
  if (q4nx_status st = check_shape(N, K, fn)) return st;
  if (!d_blob || !d_W) return fail(Q4NX_ERR_INVALID_ARG, std::string(fn) + ": NULL pointer");
  if (w_dtype != Q4NX_F32 && w_dtype != Q4NX_BF16)
    return fail(Q4NX_ERR_INVALID_ARG, std::string(fn) + ": unknown w_dtype");
  if (!aligned(d_blob, 16) || !aligned(d_W, 16))
    return fail(Q4NX_ERR_ALIGNMENT, std::string(fn) + ": blob and W need 16-byte alignment");
  const int64_t KB = ceil_div(K, kBlockCols);
  const int64_t nblocks = ceil_div(N, kBlockRows) * KB;
  const int64_t grid = std::min<int64_t>(nblocks, int64_t(1) << 20);
  const uint8_t* blob = static_cast<const uint8_t*>(d_blob);
  if (w_dtype == Q4NX_BF16)
    hipLaunchKernelGGL((dequant_kernel<F, true>), dim3((unsigned)grid), dim3(256), 0, stream, blob, N, K, KB, nblocks,
                       d_W);
  else
    hipLaunchKernelGGL((dequant_kernel<F, false>), dim3((unsigned)grid), dim3(256), 0, stream, blob, N, K, KB,
                       nblocks, d_W);
  return check_launch(fn);
}

// Measurement aid: read a buffer once with the GEMV's load pattern (16-byte
// non-temporal loads, a workgroup per contiguous slice, through a buffer
// descriptor limited to the slice, so no load needs a bounds test) and fold it
// into one value per wave (lane shuffles, no LDS and no barrier), so that
// nothing is dead code and the kernel has no tail beyond the loads.  Gives the
// read bandwidth, and the per-launch floor, of a plain streaming kernel.
constexpr int kStreamWgs = 2048;
__global__ __launch_bounds__(256) void stream_read_kernel(const uint8_t* __restrict__ src, int64_t n16,
                                                          float* __restrict__ sink) {
  const int64_t per = (n16 + gridDim.x - 1) / gridDim.x;
  const int64_t b = (int64_t)blockIdx.x * per, e = min(n16, b + per);
  const int cnt = (int)max<int64_t>(0, e - b);  // 16-byte pieces of this slice
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(src) + (e > b ? b * 16 : 0), (short)0, cnt * 16, 0x00020000);
  uint32_t acc = 0;
  for (int i = threadIdx.x; i < cnt; i += 4 * 256) {
    u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (i + u * 256) * 16, 0, kNtLoad));
#pragma unroll
    for (int u = 0; u < 4; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  acc ^= (uint32_t)xor_lane_bits<32>((int)acc);
  acc ^= (uint32_t)xor_lane_bits<16>((int)acc);
  acc ^= (uint32_t)xor_lane_bits<8>((int)acc);
  acc ^= (uint32_t)xor_lane_bits<4>((int)acc);
  acc ^= (uint32_t)xor_lane_bits<2>((int)acc);
  acc ^= (uint32_t)xor_lane_bits<1>((int)acc);
  if ((threadIdx.x & 63) == 0) sink[blockIdx.x * 4 + (threadIdx.x >> 6)] = __uint_as_float(acc & 0x3FFFFFFFu);
}

}  // namespace q4nx

using namespace q4nx;

extern "C" {

q4nx_status q4nx_dequant(const void* d_blob, int64_t N, int64_t K, void* d_W, q4nx_dtype w_dtype,
                         hipStream_t stream) {
  return dequant_entry<kWQ4NX>(d_blob, N, K, d_W, w_dtype, stream, "q4nx_dequant");
}

q4nx_status q4nx_mx_dequant(const void* d_blob, int64_t N, int64_t K, void* d_W, q4nx_dtype w_dtype,
                            hipStream_t stream) {
  return dequant_entry<kWMX>(d_blob, N, K, d_W, w_dtype, stream, "q4nx_mx_dequant");
}

q4nx_status q4nx_quantize(const float* d_W, int64_t N, int64_t K, void* d_blob, hipStream_t stream) {
  clear_error();
  if (q4nx_status st = check_shape(N, K, "q4nx_quantize")) return st;
  if (!d_W || !d_blob) return fail(Q4NX_ERR_INVALID_ARG, "q4nx_quantize: NULL pointer");
  if (!aligned(d_W, 16) || !aligned(d_blob, 16))
    return fail(Q4NX_ERR_ALIGNMENT, "q4nx_quantize: W and blob need 16-byte alignment");
  const int64_t KB = ceil_div(K, kBlockCols);
  const int64_t nblocks = ceil_div(N, kBlockRows) * KB;
  const int64_t grid = std::min<int64_t>(nblocks, int64_t(1) << 20);
  hipLaunchKernelGGL(quantize_kernel, dim3((unsigned)grid), dim3(256), 0, stream, d_W, N, K, KB, nblocks,
                     static_cast<uint8_t*>(d_blob));
  return check_launch("q4nx_quantize");
}

q4nx_status q4nx_mx_quantize(const float* d_W, int64_t N, int64_t K, void* d_blob, hipStream_t stream) {
  clear_error();
  if (q4nx_status st = check_shape(N, K, "q4nx_mx_quantize")) return st;
  if (!d_W || !d_blob) return fail(Q4NX_ERR_INVALID_ARG, "q4nx_mx_quantize: NULL pointer");
  if (!aligned(d_W, 16) || !aligned(d_blob, 16))
    return fail(Q4NX_ERR_ALIGNMENT, "q4nx_mx_quantize: W and blob need 16-byte alignment");
  const int64_t KB = ceil_div(K, kBlockCols);
  const int64_t nblocks = ceil_div(N, kBlockRows) * KB;
  const int64_t grid = std::min<int64_t>(nblocks, int64_t(1) << 20);
  hipLaunchKernelGGL(mx_quantize_kernel, dim3((unsigned)grid), dim3(256), 0, stream, d_W, N, K, KB, nblocks,
                     static_cast<uint8_t*>(d_blob));
  return check_launch("q4nx_mx_quantize");
}

q4nx_status q4nx_stream_read(const void* d_src, size_t bytes, float* d_sink, hipStream_t stream) {
  clear_error();
  if (!d_src || !d_sink) return fail(Q4NX_ERR_INVALID_ARG, "q4nx_stream_read: NULL pointer");
  if (bytes == 0 || bytes % 16 != 0 || bytes / kStreamWgs >= (size_t(1) << 31))
    return fail(Q4NX_ERR_SHAPE, "q4nx_stream_read: bytes must be a positive multiple of 16, below 2^42");
  if (!aligned(d_src, 16) || !aligned(d_sink, 4)) return fail(Q4NX_ERR_ALIGNMENT, "q4nx_stream_read: src needs 16-byte alignment");
  hipLaunchKernelGGL(stream_read_kernel, dim3(kStreamWgs), dim3(256), 0, stream, static_cast<const uint8_t*>(d_src),
                     (int64_t)(bytes / 16), d_sink);
  return check_launch("q4nx_stream_read");
}

q4nx_status q4nx_gemv(const void* d_blob, const uint16_t* d_x, void* d_y, q4nx_dtype y_dtype, int64_t N,
                      int64_t K, hipStream_t stream) {
  q4nx_gemv_desc d = {d_blob, d_x, d_y, N, K};
  return gemv_launch<kWQ4NX>(&d, 1, y_dtype, stream, "q4nx_gemv");
}

q4nx_status q4nx_gemv_batched(const q4nx_gemv_desc* descs, int32_t count, q4nx_dtype y_dtype,
                              hipStream_t stream) {
  return gemv_launch<kWQ4NX>(descs, count, y_dtype, stream, "q4nx_gemv_batched");
}

q4nx_status q4nx_mx_gemv(const void* d_blob, const uint16_t* d_x, void* d_y, q4nx_dtype y_dtype, int64_t N,
                         int64_t K, hipStream_t stream) {
  q4nx_gemv_desc d = {d_blob, d_x, d_y, N, K};
  return gemv_launch<kWMX>(&d, 1, y_dtype, stream, "q4nx_mx_gemv");
}

q4nx_status q4nx_mx_gemv_batched(const q4nx_gemv_desc* descs, int32_t count, q4nx_dtype y_dtype,
                                 hipStream_t stream) {
  return gemv_launch<kWMX>(descs, count, y_dtype, stream, "q4nx_mx_gemv_batched");
}

q4nx_status q4nx_gemm(int64_t M, int64_t N, int64_t K, const uint16_t* d_X, const void* d_blob, void* d_Y,
                      q4nx_dtype y_dtype, hipStream_t stream) {
  return gemm_entry<kWQ4NX>(M, N, K, d_X, d_blob, d_Y, y_dtype, nullptr, 0, stream, "q4nx_gemm");
}

q4nx_status q4nx_mx_gemm(int64_t M, int64_t N, int64_t K, const uint16_t* d_X, const void* d_blob, void* d_Y,
                         q4nx_dtype y_dtype, hipStream_t stream) {
  return gemm_entry<kWMX>(M, N, K, d_X, d_blob, d_Y, y_dtype, nullptr, 0, stream, "q4nx_mx_gemm");
}

q4nx_status q4nx_gemm_bf16(int64_t M, int64_t N, int64_t K, const uint16_t* d_X, const uint16_t* d_W, void* d_Y,
                           q4nx_dtype y_dtype, hipStream_t stream) {
  return gemm_entry<kWBf16>(M, N, K, d_X, d_W, d_Y, y_dtype, nullptr, 0, stream, "q4nx_gemm_bf16");
}

int q4nx_internal_gemm_launches(int w_format, int64_t M, int64_t N, int64_t K, int have_work, char* text, int size) {
  if (!text || size <= 0 || M <= 0 || M > Q4NX_MAX_DIM || check_shape(N, K, "q4nx_internal_gemm_launches") != Q4NX_OK ||
      M * N > (int64_t(1) << 40) || w_format < Q4NX_WEIGHTS_Q4NX || w_format > Q4NX_WEIGHTS_BF16)
    return -1;
  const int wf = w_format == Q4NX_WEIGHTS_Q4NX ? kWQ4NX : w_format == Q4NX_WEIGHTS_MXFP4 ? kWMX : kWBf16;
  const std::string s = launches_text(gemm_choose(wf, M, N, K, have_work != 0), wf, K);
  if ((int)s.size() >= size) return -1;
  std::copy(s.c_str(), s.c_str() + s.size() + 1, text);
  return (int)s.size();
}

size_t q4nx_gemm_workspace_size(q4nx_weights w_format, int64_t M, int64_t N, int64_t K) {
  if (M <= 0 || N <= 0 || K <= 0 || K % kGroup != 0 || M > Q4NX_MAX_DIM || N > Q4NX_MAX_DIM || K > Q4NX_MAX_DIM ||
      M * N > (int64_t(1) << 40))
    return 0;
  int wf;
  switch (w_format) {
    case Q4NX_WEIGHTS_Q4NX: wf = kWQ4NX; break;
    case Q4NX_WEIGHTS_MXFP4: wf = kWMX; break;
    case Q4NX_WEIGHTS_BF16: wf = kWBf16; break;
    default: return 0;
  }
  const GemmChoice c = gemm_choose(wf, M, N, K, true);
  return c.w_bytes + c.part_bytes;
}

q4nx_status q4nx_gemm_ex(q4nx_weights w_format, int64_t M, int64_t N, int64_t K, const uint16_t* d_X,
                         const void* d_W, void* d_Y, q4nx_dtype y_dtype, void* d_work, size_t work_bytes,
                         hipStream_t stream) {
  switch (w_format) {
    case Q4NX_WEIGHTS_Q4NX:
      return gemm_entry<kWQ4NX>(M, N, K, d_X, d_W, d_Y, y_dtype, d_work, work_bytes, stream, "q4nx_gemm_ex");
    case Q4NX_WEIGHTS_MXFP4:
      return gemm_entry<kWMX>(M, N, K, d_X, d_W, d_Y, y_dtype, d_work, work_bytes, stream, "q4nx_gemm_ex");
    case Q4NX_WEIGHTS_BF16:
      return gemm_entry<kWBf16>(M, N, K, d_X, d_W, d_Y, y_dtype, d_work, work_bytes, stream, "q4nx_gemm_ex");
    default:
      clear_error();
      return fail(Q4NX_ERR_INVALID_ARG, "q4nx_gemm_ex: unknown w_format");
  }
}

}  // extern "C"
