// FlowKV decode attention for gfx950: the attention of one decode position
// over the KV cache (the causal-attention equation of the decoding section),
// computed with FlowKV's chunk sweep (Eq. 6-12 with a query chunk of 1), with
// its sliding-window variant.
//
// The sweep is split in two launches.  Phase 1 gives every (KV group, chunk of
// 16 to 512 positions) to one workgroup, which computes for the H/G query heads
// of the group the chunk's own running state: the max score m_c (Eq. 7), the
// denominator l_c = sum exp(s - m_c) (Eq. 8, 10) and the weighted values
// Y_c = sum exp(s - m_c) v (Eq. 11), into the caller's workspace.  Phase 2
// merges the chunks of each head with the correction factor of Eq. 9 taken
// relative to the largest chunk max, which is what the left-to-right
// recurrence reaches after the last chunk, then divides (Eq. 12).  Reading the cache is the whole cost: each K and V
// row is read once, by one workgroup, with full 128-byte rows per load.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <string>
#include <type_traits>

#include "q4nx_device.h"
#include "q4nx_internal.h"
#include "q4nx_xlane.h"

namespace q4nx {

typedef __bf16 bf16x2f __attribute__((ext_vector_type(2)));

constexpr int kMinChunk = 16;      // smallest chunk: sizes the workspace
// Positions a wave takes at a time: 4 KiB of K (and of V), at least 16
// positions.  (8 KiB at d = 64 and 128 kept the workgroups of short ranges to
// half and their waves to twice the serial work: 8 heads in one group at
// d = 64 over 100 positions 13.5 us, now 7.7; 4 KiB at d = 256 would halve the
// loads in flight of the ranges that stream.)
constexpr int sub_positions(int d) { return d >= 128 ? 16 : 2048 / d; }
constexpr int kFkvThreads = 256;   // merge workgroups
constexpr int kMergeRegs = 8;      // chunks per slice the one-pass merge holds in registers

// a.lo * b.lo + a.hi * b.hi + c for two bf16 pairs (exact products, float32 sum).
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2f, a), __builtin_bit_cast(bf16x2f, b), c, false);
}

// K and V are read once per call: non-temporal.  (Default loads took 8% longer
// over the 4B layer stack at 32K and 9% over the 27B one at 16K, and were at
// most 2% ahead where a whole model's cache stays on the chip.)
__device__ __forceinline__ uint4 load_stream(const uint4* p) {
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const u4 v = __builtin_nontemporal_load(reinterpret_cast<const u4*>(p));
  return make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ float bf16lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf16hi(uint32_t v) { return __uint_as_float(v & 0xFFFF0000u); }

// Wave-wide reductions in a fixed order (deterministic): exchanges with lane
// l ^ 32, then ^ 16, ..., ^ 1.
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, xor_lane<32>(v));
  v = fmaxf(v, xor_lane<16>(v));
  v = fmaxf(v, xor_lane<8>(v));
  v = fmaxf(v, xor_lane<4>(v));
  v = fmaxf(v, xor_lane<2>(v));
  return fmaxf(v, xor_lane<1>(v));
}
// Sum over the lanes l ^ m for m = R, 2R, ..., 32 (R a power of two, 8 to
// 32), in that order.
template <int R>
__device__ __forceinline__ float sum_lanes_from(float v) {
  if constexpr (R <= 8) v += xor_lane<8>(v);
  if constexpr (R <= 16) v += xor_lane<16>(v);
  return v + xor_lane<32>(v);
}

// The 8 lanes u of a position each hold a part of H * A values (H heads, A
// groups of positions); their sums are formed and shared out over the lanes:
// the low bits of u pick the head, the next ones the group, and lanes that are
// left over hold the same sums.  Lanes 1, 2 and 4 apart are added in turn (M),
// each step halving the values that a lane still holds.
template <int M, int H, int A, int NR>
__device__ __forceinline__ void scatter_sum(const float* v, float* out, int u) {
  const bool up = u & M;
  if constexpr (M == 8) {
#pragma unroll
    for (int i = 0; i < NR; ++i) out[i] = v[i];
  } else if constexpr (H > 1) {
    float w[H / 2 * A];
#pragma unroll
    for (int h = 0; h < H / 2; ++h)
#pragma unroll
      for (int a = 0; a < A; ++a) {
        const float x0 = v[2 * h * A + a], x1 = v[(2 * h + 1) * A + a];
        w[h * A + a] = (up ? x1 : x0) + xor_lane<M>(up ? x0 : x1);
      }
    scatter_sum<2 * M, H / 2, A, NR>(w, out, u);
  } else if constexpr (A > 1) {
    float w[A / 2];
#pragma unroll
    for (int a = 0; a < A / 2; ++a) {
      const float x0 = v[2 * a], x1 = v[2 * a + 1];
      w[a] = (up ? x1 : x0) + xor_lane<M>(up ? x0 : x1);
    }
    scatter_sum<2 * M, 1, A / 2, NR>(w, out, u);
  } else {
    const float w = v[0] + xor_lane<M>(v[0]);
    scatter_sum<2 * M, 1, 1, NR>(&w, out, u);
  }
}

// Phase 1.  grid (chunks, G), W waves: workgroup (c, g) covers `chunk`
// positions from j0 + c chunk, each wave a contiguous part of them, for the HG
// query heads of group g.  Partial of (head, chunk) at
// work[(head * nchunks + chunk) * (D + 4)]: m_c, l_c, -, -, Y_c[D].
//
// A wave walks its part in sub-chunks of SP positions (sub_positions below)
// with FlowKV's running state (Eq. 7-11), no barrier and no workgroup-wide
// phase: K of the next sub-chunk is requested as soon as the scores are out of
// its registers, V as soon as the weighted sums are, so the wave always has
// loads in flight; the waves' states are merged at the end, through LDS.
// Short ranges (the sliding-window layers) are bound by latency and take one
// sub-chunk per wave: one round trip for q, K and V together, and none of the
// six barriers of a workgroup that forms one softmax.
//
// Lane roles: scores use 8 lanes per position (lane u of the 8 takes dims
// 64i + 8u .. +7 of 64-dim piece i).  scatter_sum leaves each lane the scores
// of one head and of its share of the positions 8a + lane/8, so that every
// exponential is taken once and a lane keeps the running maximum of one head.
// (With the sums left in all 8 lanes, each of them took the exponentials of
// every head: 16 heads in 2 groups at d = 256 over 9000 positions ran 27.5 us
// where a workgroup that forms one softmax took 20.3; now 16.4.)  Weighted
// values use R = D / 8 lanes per row (16 bytes, 8 dims, each), P = 64 / R rows
// per load.  The probabilities, and the correction of the heads' sums, change
// lanes through the wave's own LDS slot.
template <int W, int D, int HG>
__global__ __launch_bounds__(64 * W, HG >= 8 && D >= 256 ? 1 : 2) void flowkv_chunk_kernel(const uint16_t* __restrict__ q,
                                                                const uint16_t* __restrict__ K,
                                                                const uint16_t* __restrict__ V, int64_t L, int j0,
                                                                int j1, int chunk, float scale,
                                                                float* __restrict__ work) {
  constexpr int kPart = D + 4;
  constexpr int SP = sub_positions(D);
  constexpr int NP = D / 64, NG = SP / 8;   // 64-dim pieces of a row, groups of 8 positions
  constexpr int R = D / 8, P = 64 / R, NV = SP / P;
  constexpr bool kQRegs = HG <= 4;          // the query in registers (64 of them at most), else in LDS
  // Scores per lane after scatter_sum: head u % HG, and kSplit further bits of
  // u as the low bits of the group.
  constexpr int kHBits = HG == 8 ? 3 : HG == 4 ? 2 : HG == 2 ? 1 : 0;
  constexpr int kSplit = std::min(3 - kHBits, NG == 2 ? 1 : 2);
  constexpr int NR = NG >> kSplit;
  static_assert(NG == 2 || NG == 4, "groups of a sub-chunk");
  __shared__ __attribute__((aligned(16))) uint32_t qs[kQRegs ? 1 : HG][D / 2];
  __shared__ __attribute__((aligned(16))) float fs[W][SP][HG];  // a sub-chunk's exp(s - m)
  __shared__ __attribute__((aligned(16))) float cs[W][HG];      // its correction exp(m_left - m)
  __shared__ float ms[W][HG], ls[W][HG];
  __shared__ __attribute__((aligned(16))) float ys[W > 1 ? W : 1][W > 1 ? HG : 1][D];

  const int c = blockIdx.x, g = blockIdx.y, nchunks = gridDim.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int u = lane & 7, kw = lane >> 3;
  const int rs = lane / R, db = lane % R;
  const int per = chunk / W;                                // a multiple of SP
  const int k0 = j0 + c * chunk + wave * per;               // this wave's positions: k0 .. k0 + n - 1
  const int n = max(0, min(j1 - k0, per));
  const uint16_t* Kg = K + ((size_t)g * L + min(k0, j1 - 1)) * D;
  const uint16_t* Vg = V + ((size_t)g * L + min(k0, j1 - 1)) * D;
  const int last = max(n - 1, 0);

  // Positions past the range read the last one; their scores are -inf.
  uint4 kr[NG][NP], vr[NV];
  const auto load_k = [&](int p0) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < NG; ++a) {
      const uint4* row = reinterpret_cast<const uint4*>(Kg + (size_t)min(p0 + 8 * a + kw, last) * D);
#pragma unroll
      for (int i = 0; i < NP; ++i) kr[a][i] = load_stream(row + 8 * i + u);
    }
  };
  const auto load_v = [&](int p0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < NV; ++j)
      vr[j] = load_stream(reinterpret_cast<const uint4*>(Vg + (size_t)min(p0 + P * j + rs, last) * D) + db);
  };

  uint4 qr[kQRegs ? HG : 1][kQRegs ? NP : 1];
  if constexpr (kQRegs) {
#pragma unroll
    for (int h = 0; h < HG; ++h)
#pragma unroll
      for (int i = 0; i < NP; ++i) qr[h][i] = reinterpret_cast<const uint4*>(q + (size_t)(g * HG + h) * D)[8 * i + u];
  }
  load_k(0);
  load_v(0);
  if constexpr (!kQRegs) {
    for (int e = tid; e < HG * D / 8; e += 64 * W)
      reinterpret_cast<uint4*>(&qs[0][0])[e] = reinterpret_cast<const uint4*>(q + (size_t)g * HG * D)[e];
    __syncthreads();
  }

  const int hu = u & (HG - 1);                             // the lane's head
  const int pu = 8 * ((u >> kHBits) & ((1 << kSplit) - 1)) + kw;  // and its positions: pu + 8 (a << kSplit)
  float m = -INFINITY, l = 0.0f;            // running state of the lane's head, l over the lane's own positions
  float y[HG][8];                           // every head, over the lane's own rows
#pragma unroll
  for (int h = 0; h < HG; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) y[h][e] = 0.0f;
  for (int p0 = 0; p0 < n; p0 += SP) {
    // Scores (Eq. 6).
    float v[HG][NG];
#pragma unroll
    for (int h = 0; h < HG; ++h) {
#pragma unroll
      for (int a = 0; a < NG; ++a) v[h][a] = 0.0f;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        uint4 qv;
        if constexpr (kQRegs) qv = qr[h][i];
        else qv = *reinterpret_cast<const uint4*>(&qs[h][32 * i + 4 * u]);
#pragma unroll
        for (int a = 0; a < NG; ++a) {
          v[h][a] = dot2(kr[a][i].x, qv.x, v[h][a]);
          v[h][a] = dot2(kr[a][i].y, qv.y, v[h][a]);
          v[h][a] = dot2(kr[a][i].z, qv.z, v[h][a]);
          v[h][a] = dot2(kr[a][i].w, qv.w, v[h][a]);
        }
      }
    }
    float s[NR];
    scatter_sum<1, HG, NG, NR>(&v[0][0], s, u);
    if (p0 + SP < n) load_k(p0 + SP);
    // Running maximum (Eq. 7), exponentials (Eq. 8), correction (Eq. 9, 10).
    float mx = m;
#pragma unroll
    for (int a = 0; a < NR; ++a) {
      s[a] = p0 + pu + 8 * (a << kSplit) < n ? s[a] * scale : -INFINITY;
      mx = fmaxf(mx, s[a]);
    }
    if constexpr (kSplit > 0) mx = fmaxf(mx, xor_lane<(1 << kHBits)>(mx));
    if constexpr (kSplit > 1) mx = fmaxf(mx, xor_lane<(2 << kHBits)>(mx));
    mx = fmaxf(mx, xor_lane<8>(mx));
    mx = fmaxf(mx, xor_lane<16>(mx));
    mx = fmaxf(mx, xor_lane<32>(mx));
    const float base = mx == -INFINITY ? 0.0f : mx;  // no finite score yet: exp(-inf) = 0
    const float corr = expf(m - base);
    m = mx;
    l *= corr;
    if (HG > 1 && lane < HG) cs[wave][lane] = corr;
#pragma unroll
    for (int a = 0; a < NR; ++a) {
      const float f = expf(s[a] - base);
      l += f;
      fs[wave][pu + 8 * (a << kSplit)][hu] = f;
    }
    // (A wave's LDS instructions are carried out in order; the fences keep the
    // compiler from moving the accesses across.)
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    // Rows past the range are copies of the last one with weight 0, which
    // times an infinity would be NaN.
    if (p0 + SP > n) {
#pragma unroll
      for (int j = 0; j < NV; ++j)
        if (p0 + P * j + rs >= n) vr[j] = make_uint4(0, 0, 0, 0);
    }
    // Weighted values (Eq. 11).
#pragma unroll
    for (int h = 0; h < HG; ++h) {
      const float ch = HG > 1 ? cs[wave][h] : corr;
#pragma unroll
      for (int e = 0; e < 8; ++e) y[h][e] *= ch;
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const float* f = fs[wave][P * j + rs];
      const float w[8] = {bf16lo(vr[j].x), bf16hi(vr[j].x), bf16lo(vr[j].y), bf16hi(vr[j].y),
                          bf16lo(vr[j].z), bf16hi(vr[j].z), bf16lo(vr[j].w), bf16hi(vr[j].w)};
#pragma unroll
      for (int h = 0; h < HG; ++h)
#pragma unroll
        for (int e = 0; e < 8; ++e) y[h][e] = fmaf(f[h], w[e], y[h][e]);
    }
    if (p0 + SP < n) load_v(p0 + SP);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }

  // Sum over the lanes: l over the lanes of a head (those that share out its
  // positions), y over the rows of a load (lanes rs).
  if constexpr (kSplit > 0) l += xor_lane<(1 << kHBits)>(l);
  if constexpr (kSplit > 1) l += xor_lane<(2 << kHBits)>(l);
  l = sum_lanes_from<8>(l);
#pragma unroll
  for (int h = 0; h < HG; ++h)
#pragma unroll
    for (int e = 0; e < 8; ++e) y[h][e] = sum_lanes_from<R>(y[h][e]);
  if constexpr (W == 1) {
#pragma unroll
    for (int h = 0; h < HG; ++h) {
      float* part = work + ((size_t)(g * HG + h) * nchunks + c) * kPart;
      if (rs == 0) {
        reinterpret_cast<float4*>(part + 4 + 8 * db)[0] = make_float4(y[h][0], y[h][1], y[h][2], y[h][3]);
        reinterpret_cast<float4*>(part + 4 + 8 * db)[1] = make_float4(y[h][4], y[h][5], y[h][6], y[h][7]);
      }
    }
    if (lane < HG) {
      float* part = work + ((size_t)(g * HG + lane) * nchunks + c) * kPart;
      part[0] = m;
      part[1] = l;
    }
  } else {
#pragma unroll
    for (int h = 0; h < HG; ++h) {
      if (rs == 0) {
        reinterpret_cast<float4*>(&ys[wave][h][8 * db])[0] = make_float4(y[h][0], y[h][1], y[h][2], y[h][3]);
        reinterpret_cast<float4*>(&ys[wave][h][8 * db])[1] = make_float4(y[h][4], y[h][5], y[h][6], y[h][7]);
      }
    }
    if (lane < HG) {
      ms[wave][lane] = m;
      ls[wave][lane] = l;
    }
    __syncthreads();
    // The waves' states merged in wave order (a wave without a finite score
    // has weight 0).
    for (int e = tid; e < HG * D; e += 64 * W) {
      const int h = e / D, dd = e % D;
      float mx = ms[0][h];
#pragma unroll
      for (int w = 1; w < W; ++w) mx = fmaxf(mx, ms[w][h]);
      const float base = mx == -INFINITY ? 0.0f : mx;
      float yt = 0.0f, lt = 0.0f;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const float a = expf(ms[w][h] - base);
        yt = fmaf(a, ys[w][h][dd], yt);
        lt = fmaf(a, ls[w][h], lt);
      }
      float* part = work + ((size_t)(g * HG + h) * nchunks + c) * kPart;
      part[4 + dd] = yt;
      if (dd == 0) {
        part[0] = mx;
        part[1] = lt;
      }
    }
  }
}

// Phase 2.  grid (H, D / DW), 256 threads: workgroup (h, b) produces dims
// b*DW .. b*DW + DW-1 of head h, with S = 256 / DW slices of DW threads; slice
// s takes chunks s, s + S, ...  With M the largest chunk max, Eq. 9's
// correction of chunk c relative to M is exp(m_c - M); the head's output is
// sum_c exp(m_c - M) Y_c / sum_c exp(m_c - M) l_c (Eq. 10-12), summed over
// the chunks in increasing order within a slice and then over the slices
// (every workgroup of a head forms the same denominator in the same order).
// Splitting the dims keeps many chunks from serialising on a few workgroups
// when there are few heads (Gemma3 1B: 4 heads, 512 chunks at 32K).
template <int D, int DW, bool REGS>
__global__ __launch_bounds__(kFkvThreads) void flowkv_merge_kernel(const float* __restrict__ work, int nchunks,
                                                                   void* __restrict__ out, int out_bf16) {
  constexpr int kPart = D + 4, S = kFkvThreads / DW;
  __shared__ float mx[kFkvThreads / 64];
  __shared__ float ls[S], yls[S][DW];
  const int h = blockIdx.x, tid = threadIdx.x, dd = tid % DW, sl = tid / DW;
  const int dim = blockIdx.y * DW + dd;
  const float* part = work + (size_t)h * nchunks * kPart;
  // REGS (at most kMergeRegs chunks per slice): each thread reads its chunks'
  // (m_c, l_c, Y_c[dim]) once, in one round trip, and the block max comes
  // from those; otherwise the max and the sums read the partials in two
  // passes.  Either way M is the same maximum and the sums run over the same
  // chunks in the same order, so the bits do not depend on the path.
  constexpr bool in_regs = REGS;
  float pm[kMergeRegs], pl[kMergeRegs], py[kMergeRegs];
  float mloc = -INFINITY;
  if (in_regs) {
#pragma unroll
    for (int k = 0; k < kMergeRegs; ++k) {
      const int c = sl + k * S;
      pm[k] = -INFINITY;
      pl[k] = py[k] = 0.0f;
      if (c < nchunks) {
        const float* pc = part + (size_t)c * kPart;
        pm[k] = pc[0];
        pl[k] = pc[1];
        py[k] = pc[4 + dim];
      }
    }
#pragma unroll
    for (int k = 0; k < kMergeRegs; ++k) mloc = fmaxf(mloc, pm[k]);
  } else {
    for (int c = tid; c < nchunks; c += kFkvThreads) mloc = fmaxf(mloc, part[(size_t)c * kPart]);
  }
  mloc = wave_max(mloc);
  if ((tid & 63) == 0) mx[tid >> 6] = mloc;
  __syncthreads();
  float M = mx[0];
#pragma unroll
  for (int w = 1; w < kFkvThreads / 64; ++w) M = fmaxf(M, mx[w]);
  float l = 0.0f, y = 0.0f;
  if (in_regs) {
#pragma unroll
    for (int k = 0; k < kMergeRegs; ++k)
      if (sl + k * S < nchunks) {
        const float a = expf(pm[k] - M);
        l = fmaf(a, pl[k], l);
        y = fmaf(a, py[k], y);
      }
  } else {
#pragma unroll 4
    for (int c = sl; c < nchunks; c += S) {
      const float* pc = part + (size_t)c * kPart;
      const float a = expf(pc[0] - M);
      l = fmaf(a, pc[1], l);
      y = fmaf(a, pc[4 + dim], y);
    }
  }
  yls[sl][dd] = y;
  if (dd == 0) ls[sl] = l;
  __syncthreads();
  if (sl == 0) {
    float yt = yls[0][dd], lt = ls[0];
#pragma unroll
    for (int s2 = 1; s2 < S; ++s2) {
      yt += yls[s2][dd];
      lt += ls[s2];
    }
    const float o = yt / lt;
    if (out_bf16) {
      bf16x2f p = __builtin_convertvector((float __attribute__((ext_vector_type(2)))){o, 0.0f}, bf16x2f);
      static_cast<uint16_t*>(out)[(size_t)h * D + dim] = (uint16_t)(__builtin_bit_cast(uint32_t, p) & 0xFFFFu);
    } else {
      static_cast<float*>(out)[(size_t)h * D + dim] = o;
    }
  }
}

// Waves and positions per workgroup of phase 1.  Up to two sub-chunks per CU:
// one sub-chunk per wave, and one wave per workgroup as long as that leaves at
// most 128 partials per head, which the merge reads in one pass wherever it
// splits the dims 16 ways (2500 positions of one head at d = 256 as 157
// partials 6.7 us, as 79 partials 5.9).  Beyond, four waves and as few rounds
// of one workgroup per CU as chunks of at most 512 positions need, all chunks
// alike: a chunk of the next power of two can leave a last round that a few
// CUs work through alone (4 heads of one group at d = 256, 70000 positions:
// 274 chunks of 256 positions 28.7 us, 244 of 288 19.9).  Two workgroups per
// CU, so half the chunk and twice the partials, were 1-7% slower over the
// Gemma3 stacks at 32K.  Past the number of partials that the static scratch
// holds, chunks of 512 positions, so that it serves the longest ranges it can.
struct FlowkvSplit {
  int waves, chunk;
};
constexpr size_t kStaticScratchBytes = Q4NX_FLOWKV_STATIC_BYTES;
static FlowkvSplit flowkv_split(int64_t n, int64_t H, int64_t G, int64_t d, int cus) {
  const int sp = sub_positions((int)d);
  const int64_t nsub = ceil_div(n, sp);
  if (nsub * G <= 2 * cus) {
    const int waves = nsub <= 128 ? 1 : nsub <= 256 ? 2 : 4;
    return {waves, waves * sp};
  }
  for (int64_t r = std::max<int64_t>(1, n * G / (512 * (int64_t)cus));; ++r) {
    const int64_t chunk = ceil_div(ceil_div(n, std::max<int64_t>(1, r * cus / G)), 4 * sp) * 4 * sp;
    if (chunk > 512) continue;
    const bool fits = (size_t)(H * ceil_div(n, chunk) * (d + 4)) * sizeof(float) <= kStaticScratchBytes;
    return {4, fits ? (int)chunk : 512};
  }
}

template <int D, int HG>
static void launch_flowkv(const uint16_t* q, const uint16_t* K, const uint16_t* V, int64_t L, int G, int j0, int j1,
                          float scale, float* work, void* out, int out_bf16, hipStream_t stream, int cus) {
  const FlowkvSplit sp = flowkv_split(j1 - j0, G * HG, G, D, cus);
  const int nchunks = (int)ceil_div(j1 - j0, sp.chunk);
  const auto chunks = [&](auto wc) {
    constexpr int W = decltype(wc)::value;
    hipLaunchKernelGGL((flowkv_chunk_kernel<W, D, HG>), dim3(nchunks, G), dim3(64 * W), 0, stream, q, K, V, L, j0, j1,
                       sp.chunk, scale, work);
  };
  switch (sp.waves) {
    case 1: chunks(std::integral_constant<int, 1>{}); break;
    case 2: chunks(std::integral_constant<int, 2>{}); break;
    default: chunks(std::integral_constant<int, 4>{}); break;
  }
  // Dims per merge workgroup: halved (down to 16) until there are at least
  // 128 workgroups.
  const int H = G * HG;
  int dw = D;
  while (dw > 16 && H * (D / dw) < 128) dw >>= 1;
  const dim3 mg(H, D / dw);
  // The one-pass merge where a slice takes at most kMergeRegs chunks.
  // Measured on MI355X over the Gemma3 layer stacks at 32K (same bits): 27B
  // 1.020 -> 0.995 ms, 4B 0.444 -> 0.436, 1B 0.330 -> 0.326.  (Both forms in
  // one kernel behind a run-time branch made the 1B stack 10% slower, so the
  // form is a template parameter.)
  const int slices = kFkvThreads / dw;
  const bool regs = nchunks <= slices * kMergeRegs;
  const auto merge = [&](auto dwc) {
    constexpr int DW = decltype(dwc)::value;
    if (regs)
      hipLaunchKernelGGL((flowkv_merge_kernel<D, DW, true>), mg, dim3(kFkvThreads), 0, stream, work, nchunks, out,
                         out_bf16);
    else
      hipLaunchKernelGGL((flowkv_merge_kernel<D, DW, false>), mg, dim3(kFkvThreads), 0, stream, work, nchunks, out,
                         out_bf16);
  };
  switch (dw) {
    case 256: merge(std::integral_constant<int, (D >= 256 ? 256 : D)>{}); break;
    case 128: merge(std::integral_constant<int, (D >= 128 ? 128 : D)>{}); break;
    case 64: merge(std::integral_constant<int, 64>{}); break;
    case 32: merge(std::integral_constant<int, 32>{}); break;
    default: merge(std::integral_constant<int, 16>{}); break;
  }
}

template <int D>
static bool dispatch_hg(int hg, const uint16_t* q, const uint16_t* K, const uint16_t* V, int64_t L, int G, int j0,
                        int j1, float scale, float* work, void* out, int out_bf16, hipStream_t stream, int cus) {
  switch (hg) {
    case 1: launch_flowkv<D, 1>(q, K, V, L, G, j0, j1, scale, work, out, out_bf16, stream, cus); return true;
    case 2: launch_flowkv<D, 2>(q, K, V, L, G, j0, j1, scale, work, out, out_bf16, stream, cus); return true;
    case 4: launch_flowkv<D, 4>(q, K, V, L, G, j0, j1, scale, work, out, out_bf16, stream, cus); return true;
    case 8: launch_flowkv<D, 8>(q, K, V, L, G, j0, j1, scale, work, out, out_bf16, stream, cus); return true;
    default: return false;
  }
}

// ---- scratch of the entry point that allocates nothing ----------------------
// q4nx_flowkv_decode_static keeps the chunk partials in this array instead of
// a caller workspace.  Each device holds its own copy, at its own address,
// for the life of the process.  Host code never passes the array's name to a
// kernel (on the host it is only a stand-in for the symbol): the device
// address comes from hipGetSymbolAddress, taken once per device with that
// device current.
static __device__ __align__(256) float scratch[kStaticScratchBytes / sizeof(float)];

static q4nx_status static_scratch(float** out) {
  static std::once_flag once[kMaxDevices];
  static float* ptr[kMaxDevices] = {};
  static hipError_t err[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
    return fail(Q4NX_ERR_HIP, "q4nx_flowkv_decode_static: no current device");
  std::call_once(once[dev], [&] {
    void* p = nullptr;
    err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    ptr[dev] = static_cast<float*>(p);
  });
  if (err[dev] != hipSuccess || ptr[dev] == nullptr)
    return fail(Q4NX_ERR_HIP, std::string("q4nx_flowkv_decode_static: hipGetSymbolAddress: ") +
                                  hipGetErrorString(err[dev]));
  *out = ptr[dev];
  return Q4NX_OK;
}

// Validation and launch shared by both entry points.  Every argument is
// checked before any HIP call.  work == nullptr selects the static scratch,
// whose need is sized by the chunk length the launch will use; a caller
// workspace is sized by the smallest chunk (q4nx_flowkv_workspace_size, which
// callers use to allocate before the chunk length is known).
static q4nx_status flowkv_entry(const uint16_t* d_q, const uint16_t* d_k, const uint16_t* d_v, int64_t H, int64_t G,
                                int64_t d, int64_t L, int64_t t, int64_t window, float scale, void* d_o,
                                q4nx_dtype o_dtype, float* work, size_t work_bytes, hipStream_t stream,
                                const char* fn) {
  const std::string f(fn);
  if (!d_q || !d_k || !d_v || !d_o) return fail(Q4NX_ERR_INVALID_ARG, f + ": NULL pointer");
  if (o_dtype != Q4NX_F32 && o_dtype != Q4NX_BF16) return fail(Q4NX_ERR_INVALID_ARG, f + ": unknown o_dtype");
  if (!std::isfinite(scale)) return fail(Q4NX_ERR_INVALID_ARG, f + ": scale must be finite");
  if (H <= 0 || G <= 0 || H % G != 0 || G > 65535) return fail(Q4NX_ERR_SHAPE, f + ": H must be a positive multiple of G");
  const int64_t hg = H / G;
  if (hg != 1 && hg != 2 && hg != 4 && hg != 8) return fail(Q4NX_ERR_SHAPE, f + ": H/G must be 1, 2, 4 or 8");
  if (d != 64 && d != 128 && d != 256) return fail(Q4NX_ERR_SHAPE, f + ": d must be 64, 128 or 256");
  if (L <= 0 || L > (int64_t(1) << 30) || t < 0 || t >= L || window < 0)
    return fail(Q4NX_ERR_SHAPE, f + ": need 0 <= t < L <= 2^30 and window >= 0");
  if (!aligned(d_q, 16) || !aligned(d_k, 16) || !aligned(d_v, 16) || !aligned(d_o, 4))
    return fail(Q4NX_ERR_ALIGNMENT, f + ": q, K and V need 16-byte alignment, o 4-byte");
  const int64_t j1 = t + 1, j0 = window == 0 ? 0 : std::max<int64_t>(0, j1 - window);
  if (work && work_bytes < q4nx_flowkv_workspace_size(H, d, j1 - j0))
    return fail(Q4NX_ERR_BUFFER_TOO_SMALL, f + ": workspace smaller than q4nx_flowkv_workspace_size");
  const int cus = current_device_cus();
  if (!work) {
    const size_t need = (size_t)H * (size_t)ceil_div(j1 - j0, flowkv_split(j1 - j0, H, G, d, cus).chunk) *
                        (size_t)(d + 4) * sizeof(float);
    if (need > kStaticScratchBytes)
      return fail(Q4NX_ERR_BUFFER_TOO_SMALL, f + ": the chunk partials (" + std::to_string(need) +
                                                 " bytes) exceed the static scratch (" +
                                                 std::to_string(kStaticScratchBytes) + " bytes)");
    if (q4nx_status st = static_scratch(&work)) return st;
  }
  const int ob = o_dtype == Q4NX_BF16;
  bool ok = false;
  if (d == 64) ok = dispatch_hg<64>((int)hg, d_q, d_k, d_v, L, (int)G, (int)j0, (int)j1, scale, work, d_o, ob, stream, cus);
  if (d == 128) ok = dispatch_hg<128>((int)hg, d_q, d_k, d_v, L, (int)G, (int)j0, (int)j1, scale, work, d_o, ob, stream, cus);
  if (d == 256) ok = dispatch_hg<256>((int)hg, d_q, d_k, d_v, L, (int)G, (int)j0, (int)j1, scale, work, d_o, ob, stream, cus);
  if (!ok) return fail(Q4NX_ERR_SHAPE, f + ": unsupported shape");
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(Q4NX_ERR_HIP, f + ": " + hipGetErrorString(e));
  return Q4NX_OK;
}

}  // namespace q4nx

using namespace q4nx;

extern "C" {

size_t q4nx_flowkv_workspace_size(int64_t H, int64_t d, int64_t n_keys) {
  if (H <= 0 || d <= 0 || n_keys <= 0 || H > (1 << 16) || d > 4096 || n_keys > (int64_t(1) << 30)) return 0;
  return (size_t)H * (size_t)ceil_div(n_keys, kMinChunk) * (size_t)(d + 4) * sizeof(float);
}

q4nx_status q4nx_flowkv_decode(const uint16_t* d_q, const uint16_t* d_k, const uint16_t* d_v, int64_t H, int64_t G,
                               int64_t d, int64_t L, int64_t t, int64_t window, float scale, void* d_o,
                               q4nx_dtype o_dtype, void* d_work, size_t work_bytes, hipStream_t stream) {
  clear_error();
  if (!d_work) return fail(Q4NX_ERR_INVALID_ARG, "q4nx_flowkv_decode: NULL pointer");
  if (!aligned(d_work, 16)) return fail(Q4NX_ERR_ALIGNMENT, "q4nx_flowkv_decode: workspace needs 16-byte alignment");
  return flowkv_entry(d_q, d_k, d_v, H, G, d, L, t, window, scale, d_o, o_dtype, static_cast<float*>(d_work),
                      work_bytes, stream, "q4nx_flowkv_decode");
}

q4nx_status q4nx_flowkv_decode_static(const uint16_t* d_q, const uint16_t* d_k, const uint16_t* d_v, int64_t H,
                                      int64_t G, int64_t d, int64_t L, int64_t t, int64_t window, float scale,
                                      void* d_o, q4nx_dtype o_dtype, hipStream_t stream) {
  clear_error();
  return flowkv_entry(d_q, d_k, d_v, H, G, d, L, t, window, scale, d_o, o_dtype, nullptr, 0, stream,
                      "q4nx_flowkv_decode_static");
}

}  // extern "C"
