// Kernels of the synthetic decode step: the stand-in for the paper's LLM
// decode victims (Sections 4.2-4.4; per-kernel latencies of one step as in
// Fig. 5).  A Llama-style decoder layer with random weights, batch <= 8.
//
// Weight streaming dominates a decode step, so the GEMV is the kernel that
// matters, and the step is built around it: the small element-wise stages
// ride inside the GEMVs instead of paying a launch (and a pipeline drain)
// each.
//
//   gemv_fused_kernel   BF16 weight rows x NB vectors, FP32 accumulation.
//     input  BF16: the vectors as given;
//            NORM: FP32 vectors RMS-normalised with a BF16 gain and rounded
//                  to BF16 while they are staged (every work-group computes
//                  the norms itself, in the same order as rmsnorm_kernel);
//     output PLAIN: FP32 rows, plus an optional residual (may alias);
//            SILU:  rows j and j + rows/2 of one wave are gate and up, the
//                   epilogue writes BF16 SiLU(gate) * up;
//            ROPE:  rows i and i + head_dim/2 of a head share a wave, the
//                   epilogue applies the rotary embedding and writes the
//                   query (FP32) or appends key and value (BF16) to the cache.
//   attn_partial_kernel  grouped-query attention over 64-position chunks:
//                        per chunk max, exp-sum and unnormalised output.
//   attn_combine_kernel  merges the chunks of one head, BF16 out.
//   rmsnorm_kernel, rope_append_kernel, silu_mul_kernel: the same stages as
//     stand-alone kernels (the unfused composition the fused path must
//     reproduce bit for bit; they share the arithmetic helpers below).
#include "internal.h"

#include <math.h>

#include <algorithm>

namespace ci {
namespace {

__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// FP32 -> BF16 bits, round to nearest even; NaN -> quiet NaN of the same sign.
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)(((u >> 16) & 0x8000u) | 0x7FC0u);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ uint32_t pack2(uint16_t lo, uint16_t hi) {
  return (uint32_t)lo | ((uint32_t)hi << 16);
}

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ float wave_max_f(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

__device__ __forceinline__ float dot8(uint4 w, uint4 x, float acc) {
  acc = __builtin_fmaf(bf_lo(w.x), bf_lo(x.x), acc);
  acc = __builtin_fmaf(bf_hi(w.x), bf_hi(x.x), acc);
  acc = __builtin_fmaf(bf_lo(w.y), bf_lo(x.y), acc);
  acc = __builtin_fmaf(bf_hi(w.y), bf_hi(x.y), acc);
  acc = __builtin_fmaf(bf_lo(w.z), bf_lo(x.z), acc);
  acc = __builtin_fmaf(bf_hi(w.z), bf_hi(x.z), acc);
  acc = __builtin_fmaf(bf_lo(w.w), bf_lo(x.w), acc);
  acc = __builtin_fmaf(bf_hi(w.w), bf_hi(x.w), acc);
  return acc;
}

// 16 bytes of each lane straight to LDS, lane l's to l + 16 * lane.
__device__ __forceinline__ void load_lds_16(const void* g, void* l) {
  __builtin_amdgcn_global_load_lds(g, l, 16, 0, 0);
}

constexpr int kWaitLoads = 0x0F70;     // s_waitcnt vmcnt(0)

// ---------------------------------------------- arithmetic shared by paths
__device__ __forceinline__ float sumsq_of_thread(const float* __restrict__ x, uint32_t n, uint32_t t) {
  const float4* x4 = reinterpret_cast<const float4*>(x);
  float ss = 0.0f;
  for (uint32_t i = t; i < n / 4; i += 256) {
    const float4 v = x4[i];
    ss = fmaf(v.x, v.x, ss);
    ss = fmaf(v.y, v.y, ss);
    ss = fmaf(v.z, v.z, ss);
    ss = fmaf(v.w, v.w, ss);
  }
  return ss;
}

// Sum of squares of x[0..n) by a 256-thread work-group: thread t takes the
// float4s t, t + 256, ..., then the waves' sums are added in a fixed order.
// Uniform control flow required (barriers).
__device__ float block_sumsq_256(const float* __restrict__ x, uint32_t n, float* s_part) {
  const float ss = wave_sum_f(sumsq_of_thread(x, n, threadIdx.x));
  if ((threadIdx.x & 63u) == 0) s_part[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float tot = (s_part[0] + s_part[1]) + (s_part[2] + s_part[3]);
  __syncthreads();
  return tot;
}

__device__ __forceinline__ float rms_factor(float sumsq, uint32_t n, float eps) {
  return 1.0f / sqrtf(sumsq / (float)n + eps);
}

__device__ __forceinline__ uint16_t norm_bf16(float x, float r, float g) {
#pragma clang fp contract(off)
  return f32_to_bf16_rne((x * r) * g);
}

// Pair i of a head turns by pos * base^(-2i/d): angle, cosine and sine in
// FP64, rounded to FP32; the rotation in FP32 without contraction.
__device__ __forceinline__ void rope_cos_sin(uint32_t pos, uint32_t i, uint32_t d, float base, float* cs,
                                             float* sn) {
  const double ang = (double)pos * pow((double)base, -2.0 * (double)i / (double)d);
  *cs = (float)cos(ang);
  *sn = (float)sin(ang);
}

__device__ __forceinline__ void rope_apply(float x1, float x2, float cs, float sn, float* y1, float* y2) {
#pragma clang fp contract(off)
  *y1 = x1 * cs - x2 * sn;
  *y2 = x2 * cs + x1 * sn;
}

__device__ __forceinline__ float silu_mul_f(float g, float u) {
#pragma clang fp contract(off)
  return g / (1.0f + expf(-g)) * u;
}

// ---------------------------------------------------------------- RMSNorm
// One 256-thread work-group per row; n a multiple of 4.
__global__ void __launch_bounds__(256) rmsnorm_kernel(const float* __restrict__ x,
                                                      const uint16_t* __restrict__ g,
                                                      uint16_t* __restrict__ y, uint32_t n,
                                                      float eps) {
  __shared__ float s_part[4];
  const float* xr = x + (size_t)blockIdx.x * n;
  const float r = rms_factor(block_sumsq_256(xr, n, s_part), n, eps);
  const float4* x4 = reinterpret_cast<const float4*>(xr);
  const uint2* g2 = reinterpret_cast<const uint2*>(g);
  uint2* y2 = reinterpret_cast<uint2*>(y + (size_t)blockIdx.x * n);
  for (uint32_t i = threadIdx.x; i < n / 4; i += 256) {
    const float4 v = x4[i];
    const uint2 gw = g2[i];
    y2[i] = make_uint2(pack2(norm_bf16(v.x, r, bf_lo(gw.x)), norm_bf16(v.y, r, bf_hi(gw.x))),
                       pack2(norm_bf16(v.z, r, bf_lo(gw.y)), norm_bf16(v.w, r, bf_hi(gw.y))));
  }
}

// ------------------------------------------------------------------- GEMV
constexpr int IN_BF16 = 0, IN_NORM = 1;
constexpr int EPI_PLAIN = 0, EPI_SILU = 1, EPI_ROPE = 2;

// Sums of N values over the 64 lanes, lane l getting value l / (64 / N): the
// butterfly of wave_sum_f for each of them, except that a lane group that holds
// several values keeps half of them at every level.
template <int N, int OFF = 32>
__device__ __forceinline__ float wave_sums(const float (&f)[N], uint32_t lane) {
  if constexpr (OFF == 0) {
    return f[0];
  } else if constexpr (N == 1) {
    const float g[1] = {f[0] + __shfl_xor(f[0], OFF, 64)};
    return wave_sums<1, OFF / 2>(g, lane);
  } else {
    float g[N / 2];
    const bool up = lane & OFF;
#pragma unroll
    for (int i = 0; i < N / 2; ++i)
      g[i] = (up ? f[i + N / 2] : f[i]) + __shfl_xor(up ? f[i] : f[i + N / 2], OFF, 64);
    return wave_sums<N / 2, OFF / 2>(g, lane);
  }
}

// The rows one wave computes at a time (a "unit"): PLAIN R consecutive rows;
// SILU / ROPE R / 2 row pairs.  The sums come out of wave_sums in groups of
// lanes: this lane's is that of row `r` of the unit and vector `b`.  For ROPE it
// carries its pair's cosine and sine.
template <int NB, int R, int EPI>
struct Unit {
  static constexpr uint32_t G = 64 / (NB * R);     // lanes per sum
  uint32_t first;          // first row (PLAIN) or pair
  const uint4* wr[R];
  bool live[R];
  float cs, sn;
  static __device__ __forceinline__ uint32_t r(uint32_t lane) { return lane / G / NB; }
  static __device__ __forceinline__ uint32_t b(uint32_t lane) { return lane / G % NB; }
};

template <int NB, int R, int EPI>
__device__ __forceinline__ void map_unit(const GemvArgs& a, uint32_t unit, uint32_t lane, Unit<NB, R, EPI>& u) {
  u.first = unit * (EPI == EPI_PLAIN ? R : R / 2);
  const uint32_t npairs = a.rows / 2, half = a.d / 2;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    uint32_t row = u.first + r;
    u.live[r] = row < a.rows;
    if constexpr (EPI != EPI_PLAIN) {
      const uint32_t jp = u.first + r / 2;
      u.live[r] = jp < npairs;
      if constexpr (EPI == EPI_SILU) row = r & 1 ? jp + npairs : jp;
      else row = jp / half * a.d + jp % half + (r & 1 ? half : 0);
    }
    u.wr[r] = reinterpret_cast<const uint4*>(a.w + (size_t)(u.live[r] ? row : 0) * a.k);
  }
}

template <int NB, int R, int EPI>
__device__ __forceinline__ void rope_factors(const GemvArgs& a, uint32_t lane, Unit<NB, R, EPI>& u) {
  if constexpr (EPI == EPI_ROPE) {
    u.cs = 1.0f;
    u.sn = 0.0f;
    const uint32_t half = a.d / 2, jp = u.first + u.r(lane) / 2, head = jp / half;
    if (jp < a.rows / 2 && u.b(lane) < a.batch && head < a.nq + a.nkv)
      rope_cos_sin((uint32_t)a.pos[u.b(lane)], jp - head * half, a.d, a.base, &u.cs, &u.sn);
  }
}

template <bool NTL>
__device__ __forceinline__ uint4 load_weights(const uint4* p) {
  if constexpr (NTL) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
  } else {
    return *p;
  }
}

// 16-byte chunks c = 64 (V j + v) + lane (v < V) of step j of the unit's rows.
template <bool NTL, int NB, int R, int V, int EPI>
__device__ __forceinline__ void load_step(const Unit<NB, R, EPI>& u, uint32_t j, uint32_t lane, uint32_t kc,
                                          uint4 (&wv)[R][V]) {
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const uint32_t c = 64u * (V * j + v) + lane;
      wv[r][v] = (u.live[r] && c < kc) ? load_weights<NTL>(u.wr[r] + c) : make_uint4(0, 0, 0, 0);
    }
}

template <int NB, int R, int EPI>
__device__ __forceinline__ void epilogue(const GemvArgs& a, const Unit<NB, R, EPI>& u, uint32_t lane,
                                         float (&acc)[R * NB]) {
  constexpr uint32_t G = Unit<NB, R, EPI>::G;
  const float sum = wave_sums<R * NB>(acc, lane);
  const uint32_t r = u.r(lane), b = u.b(lane);
  bool mine = lane % G == 0 && b < a.batch;
  if constexpr (EPI == EPI_PLAIN) {
    if (mine && u.first + r < a.rows) {
      const size_t o = (size_t)b * a.rows + u.first + r;
      a.out[o] = (a.res ? a.res[o] : 0.0f) + sum;
    }
  } else {
    const float second = __shfl(sum, lane + NB * G, 64);     // of the pair's second row
    const uint32_t jp = u.first + r / 2;
    mine = mine && r % 2 == 0 && jp < a.rows / 2;
    if constexpr (EPI == EPI_SILU) {
      if (mine) a.h[(size_t)b * (a.rows / 2) + jp] = f32_to_bf16_rne(silu_mul_f(sum, second));
    } else if (mine) {
      const uint32_t half = a.d / 2, head = jp / half, i = jp - head * half;
      const uint32_t pp = (uint32_t)a.pos[b];
      float y1 = sum, y2 = second;
      if (head < a.nq + a.nkv) rope_apply(sum, second, u.cs, u.sn, &y1, &y2);
      if (head < a.nq) {
        float* dst = a.q_out + ((size_t)b * a.nq + head) * a.d;
        dst[i] = y1;
        dst[i + half] = y2;
      } else {
        const bool key = head < a.nq + a.nkv;
        const uint32_t h = head - a.nq - (key ? 0 : a.nkv);
        uint16_t* dst = (key ? a.kc : a.vc) + (((size_t)b * a.nkv + h) * a.max_ctx + pp) * a.d;
        dst[i] = f32_to_bf16_rne(y1);
        dst[i + half] = f32_to_bf16_rne(y2);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < R * NB; ++i) acc[i] = 0.0f;
}

__device__ __forceinline__ uint2 norm4(const float4& x, float r, const uint2& g) {
  return make_uint2(pack2(norm_bf16(x.x, r, bf_lo(g.x)), norm_bf16(x.y, r, bf_hi(g.x))),
                    pack2(norm_bf16(x.z, r, bf_lo(g.y)), norm_bf16(x.w, r, bf_hi(g.y))));
}

// Stage chunks c0 .. c0 + nch - 1 of the NB vectors into LDS, normalised with
// factors s_r and gain g; zeros for b >= batch.
template <int NB, int TH>
__device__ __forceinline__ void stage_norm(const GemvArgs& a, uint32_t c0, uint32_t nch, uint32_t tc,
                                           const float* s_r, uint4* xs) {
  for (uint32_t i = threadIdx.x; i < NB * nch; i += TH) {
    const uint32_t b = i / nch, c = i - b * nch;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (b < a.batch) {
      const float4* xp = reinterpret_cast<const float4*>(a.x + (size_t)b * a.k) + 2 * (c0 + c);
      const float4 x0 = xp[0], x1 = xp[1];
      const uint4 gg = reinterpret_cast<const uint4*>(a.g)[c0 + c];
      const uint2 lo = norm4(x0, s_r[b], make_uint2(gg.x, gg.y)), hi = norm4(x1, s_r[b], make_uint2(gg.z, gg.w));
      val = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
    xs[b * tc + c] = val;
  }
}

// What a thread holds of the vectors between asking for them and staging them,
// so that the first weights can be asked for in between: a wave's loads return
// in order, and the vectors come from the L2 long before weights from memory.
// BF16: the whole tile, where one holds the vectors.
template <int NB, int TH>
struct HeldBf16 {
  static constexpr uint32_t kChunks = 8, TC = TH * kChunks / NB;
  uint4 x[kChunks];
  __device__ __forceinline__ void load(const GemvArgs& a, uint32_t kc) {
#pragma unroll
    for (uint32_t u = 0; u < kChunks; ++u) {
      const uint32_t i = threadIdx.x + TH * u, b = i / TC, c = i % TC;
      x[u] = c < kc && b < a.batch ? reinterpret_cast<const uint4*>(a.v + (size_t)b * a.k)[c] : make_uint4(0, 0, 0, 0);
    }
  }
  __device__ __forceinline__ void stage(uint32_t kc, uint4* xs) const {
#pragma unroll
    for (uint32_t u = 0; u < kChunks; ++u) {
      const uint32_t i = threadIdx.x + TH * u;
      if (i % TC < kc) xs[i] = x[u];
    }
    __syncthreads();
  }
};

// FP32: vectors of at most 4096 elements, 256 threads to a vector; they go to
// LDS normalised without a second read.  The norms are block_sumsq_256's.
template <int NB, int TH>
struct HeldNorm {
  static constexpr uint32_t kQuads = 4, G = TH / 256, Q = (NB + G - 1) / G;   // float4s per thread, vectors per 256
  float4 x[Q][kQuads];
  uint2 g[kQuads];
  static __device__ __forceinline__ bool fits(const GemvArgs& a) { return a.k <= 4 * 256 * kQuads; }
  __device__ __forceinline__ void load(const GemvArgs& a) {
    const uint32_t t = threadIdx.x & 255u, g0 = threadIdx.x >> 8, n4 = a.k / 4;
#pragma unroll
    for (uint32_t u = 0; u < kQuads; ++u) {
      const uint32_t i = t + 256 * u;
#pragma unroll
      for (uint32_t p = 0; p < Q; ++p) {
        const uint32_t b = g0 + G * p;
        x[p][u] = i < n4 && b < a.batch ? reinterpret_cast<const float4*>(a.x + (size_t)b * a.k)[i]
                                        : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      }
      g[u] = i < n4 ? reinterpret_cast<const uint2*>(a.g)[i] : make_uint2(0, 0);
    }
  }
  __device__ __forceinline__ void stage(const GemvArgs& a, uint32_t tc, float (*s_part)[4], uint4* xs) const {
    const uint32_t t = threadIdx.x & 255u, g0 = threadIdx.x >> 8, n4 = a.k / 4;
#pragma unroll
    for (uint32_t p = 0; p < Q; ++p) {
      float ss = 0.0f;
#pragma unroll
      for (uint32_t u = 0; u < kQuads; ++u)
        if (t + 256 * u < n4) {
          ss = fmaf(x[p][u].x, x[p][u].x, ss);
          ss = fmaf(x[p][u].y, x[p][u].y, ss);
          ss = fmaf(x[p][u].z, x[p][u].z, ss);
          ss = fmaf(x[p][u].w, x[p][u].w, ss);
        }
      ss = wave_sum_f(ss);
      if ((t & 63u) == 0 && g0 + G * p < NB) s_part[g0 + G * p][t >> 6] = ss;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t p = 0; p < Q; ++p) {
      const uint32_t b = g0 + G * p;
      if (b >= NB) break;
      const float* sp = s_part[b];
      const float r = b < a.batch ? rms_factor((sp[0] + sp[1]) + (sp[2] + sp[3]), a.k, a.eps) : 0.0f;
      uint2* dst = reinterpret_cast<uint2*>(xs + b * tc);
#pragma unroll
      for (uint32_t u = 0; u < kQuads; ++u)
        if (t + 256 * u < n4) dst[t + 256 * u] = norm4(x[p][u], r, g[u]);
    }
    __syncthreads();
  }
};

// out = W x (rows of BF16 weights times NB vectors), FP32 accumulation.
// Work-group: TH / 64 waves.  K is walked in steps of 64 V 16-byte chunks (V KiB
// contiguous per row per wave); the vectors are staged in LDS in tiles of 128
// bytes per thread, read by all waves of the work-group.  A tile is whole steps.
// Each lane's products are summed in increasing chunk order, then over the 64
// lanes by a butterfly: the result does not depend on NB, R, TH or the grid.
//   One tile (k * NB * 2 <= 128 TH): the grid is persistent; wave gw takes units
//     gw, gw + waves, ...; the next step's weights (next step, or step 0 of the
//     next unit) are loaded before the current step's products.
//   Several, BF16 input: one unit per wave; half a tile is filled straight from
//     memory while the waves read the other half.
//   Several, normalised input: one unit per wave, tiles staged in turn.
// NTL: non-temporal weight loads.
// What bounds it: memory for one to four vectors, the multiply-adds and the
// unpacking of the vectors for eight.  Times, cold weights, one vector: 28672 x
// 4096 with norm and SiLU 39 us (6.0 TB/s), 128256 x 4096 with norm 157 (6.7),
// 4096 x 14336 20, 6144 x 4096 with norm and rotary embedding 12.6, 4096 x 4096
// 7.6; before (staging waited for in turn, a butterfly and a store for each row
// and vector, cached loads, eight vectors of 4096 in two tiles) 44, 178, 25, 15.5
// and 9.4.  Four vectors: 44, 167, 25, 18 and 9.2 (56, 202, 32, 25 and 14.6);
// eight: 55, 215, 34, 27 and 14 (152, 599, 51, 54 and 20).
template <int NB, int R, int TH, int IN, int EPI, bool NTL>
__global__ void __launch_bounds__(TH) gemv_fused_kernel(GemvArgs a, uint32_t units) {
  constexpr int V = NB * R * 4 > 32 || (EPI == EPI_ROPE && NB == 4) ? 2 : 4;   // at most 128 registers where it matters
  constexpr uint32_t TC = TH * 8 / NB;
  static_assert(TC % (64 * V) == 0, "a tile must be whole steps");
  __shared__ uint4 xs[NB * TC];
  __shared__ float s_part[NB][4];
  __shared__ float s_r[NB];
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t gw = blockIdx.x * (TH / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t nwaves = gridDim.x * (TH / 64);
  const uint32_t kc = a.k / 8;
  const uint32_t nsteps = (kc + 64 * V - 1) / (64 * V);
  float acc[R * NB];
#pragma unroll
  for (int i = 0; i < R * NB; ++i) acc[i] = 0.0f;
  Unit<NB, R, EPI> cur;
  uint4 wcur[R][V], wnext[R][V];
  map_unit(a, gw, lane, cur);
  const bool single = kc <= TC;
  auto first_weights = [&] {
    __builtin_amdgcn_sched_barrier(0);
    load_step<NTL>(cur, 0, lane, kc, wcur);
    rope_factors(a, lane, cur);
  };
  if constexpr (IN == IN_BF16) {
    if (single) {
      HeldBf16<NB, TH> held;
      held.load(a, kc);
      first_weights();
      held.stage(kc, xs);
    } else {
      first_weights();
    }
  } else if (single && HeldNorm<NB, TH>::fits(a)) {
    HeldNorm<NB, TH> held;
    held.load(a);
    first_weights();
    held.stage(a, TC, s_part, xs);
  } else {
    first_weights();
#pragma unroll 1
    for (uint32_t b = threadIdx.x >> 8; b < NB; b += TH / 256) {
      const uint32_t t = threadIdx.x & 255u;
      float ss = 0.0f;
      if (b < a.batch) ss = sumsq_of_thread(a.x + (size_t)b * a.k, a.k, t);
      ss = wave_sum_f(ss);
      if ((t & 63u) == 0) s_part[b][t >> 6] = ss;
    }
    __syncthreads();
    if (threadIdx.x < NB) {
      const float* sp = s_part[threadIdx.x];
      s_r[threadIdx.x] =
          threadIdx.x < a.batch ? rms_factor((sp[0] + sp[1]) + (sp[2] + sp[3]), a.k, a.eps) : 0.0f;
    }
    __syncthreads();
    if (single) {
      stage_norm<NB, TH>(a, 0, kc, TC, s_r, xs);
      __syncthreads();
    }
  }
  auto multiply = [&](uint32_t j, uint32_t c0, uint32_t tc) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const uint32_t c = 64u * (V * j + v) + lane;
      if (c >= kc) break;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const uint4 xv = xs[b * tc + (c - c0)];
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r * NB + b] = dot8(wcur[r][v], xv, acc[r * NB + b]);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int v = 0; v < V; ++v) wcur[r][v] = wnext[r][v];
  };
  if (single) {
    uint32_t unit = gw, j = 0;
    while (unit < units) {
      const bool wrap = j + 1 == nsteps;
      const uint32_t nunit = wrap ? unit + nwaves : unit;
      if (nunit < units) {
        if (wrap) {
          Unit<NB, R, EPI> t;      // weights only: the rotary factors come with the unit itself
          map_unit(a, nunit, lane, t);
          load_step<NTL>(t, 0, lane, kc, wnext);
        } else {
          load_step<NTL>(cur, j + 1, lane, kc, wnext);
        }
      }
      multiply(j, 0, TC);
      if (wrap) {
        epilogue(a, cur, lane, acc);
        map_unit(a, nunit, lane, cur);
        if (nunit < units) rope_factors(a, lane, cur);
      }
      unit = nunit;
      j = wrap ? 0 : j + 1;
    }
    return;
  }
  if constexpr (IN == IN_BF16) {
    constexpr uint32_t TH2 = TC / 2;       // chunks of a half: one is filled while the other is read
    const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nhalf = (kc + TH2 - 1) / TH2;
    auto fill = [&](uint32_t h) {
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t piece = w * 4 + i, b = piece / (TH2 / 64), c = piece % (TH2 / 64) * 64;
        const uint4* src = reinterpret_cast<const uint4*>(a.v + (size_t)min(b, a.batch - 1) * a.k);
        load_lds_16(src + min(h * TH2 + c + lane, kc - 1), xs + ((h & 1) * NB + b) * TH2 + c);
      }
    };
    fill(0);
    uint32_t j = 0;
    for (uint32_t h = 0; h < nhalf; ++h) {
      __builtin_amdgcn_s_waitcnt(kWaitLoads);   // this wave's part of the half is in
      __syncthreads();
      if (h + 1 < nhalf) fill(h + 1);
      const uint32_t end = min(nsteps, (h + 1) * (TH2 / (64 * V)));
      const uint32_t c0 = h * TH2 - (h & 1) * NB * TH2;    // xs index of chunk c: c - c0 (mod 2^32)
      for (; j < end; ++j) {
        if (j + 1 < nsteps) load_step<NTL>(cur, j + 1, lane, kc, wnext);
        multiply(j, c0, TH2);
      }
    }
    if (gw < units) epilogue(a, cur, lane, acc);
    return;
  }
  for (uint32_t j = 0; j < nsteps; ++j) {
    const uint32_t cr = 64u * V * j;       // first chunk of the step
    const uint32_t c0 = cr - cr % TC;      // first chunk of its tile
    if (cr == c0) {
      __syncthreads();
      stage_norm<NB, TH>(a, c0, min(TC, kc - c0), TC, s_r, xs);
      __syncthreads();
    }
    if (j + 1 < nsteps) load_step<NTL>(cur, j + 1, lane, kc, wnext);
    multiply(j, c0, TC);
  }
  if (gw < units) epilogue(a, cur, lane, acc);
}

// ------------------------------------------------------------- RoPE + cache
// Stand-alone form.  grid (batch, n_q + 2 n_kv), block head_dim / 2.
// qkv: batch x (n_q + 2 n_kv) heads x head_dim FP32 (query heads, key heads,
// value heads).  Cache (one layer): batch x n_kv x max_ctx x head_dim BF16.
__global__ void __launch_bounds__(128) rope_append_kernel(const float* __restrict__ qkv,
                                                          Positions pos,
                                                          float* __restrict__ q_out,
                                                          uint16_t* __restrict__ kc,
                                                          uint16_t* __restrict__ vc, uint32_t nq,
                                                          uint32_t nkv, uint32_t d,
                                                          uint32_t max_ctx, float base) {
  const uint32_t b = blockIdx.x, h = blockIdx.y, i = threadIdx.x, half = d / 2;
  const uint32_t p = (uint32_t)pos.at(b);
  const float* src = qkv + ((size_t)b * (nq + 2 * nkv) + h) * d;
  const float x1 = src[i], x2 = src[i + half];
  if (h >= nq + nkv) {
    uint16_t* dst = vc + (((size_t)b * nkv + (h - nq - nkv)) * max_ctx + p) * d;
    dst[i] = f32_to_bf16_rne(x1);
    dst[i + half] = f32_to_bf16_rne(x2);
    return;
  }
  float cs, sn, y1, y2;
  rope_cos_sin(p, i, d, base, &cs, &sn);
  rope_apply(x1, x2, cs, sn, &y1, &y2);
  if (h < nq) {
    float* dst = q_out + ((size_t)b * nq + h) * d;
    dst[i] = y1;
    dst[i + half] = y2;
  } else {
    uint16_t* dst = kc + (((size_t)b * nkv + (h - nq)) * max_ctx + p) * d;
    dst[i] = f32_to_bf16_rne(y1);
    dst[i + half] = f32_to_bf16_rne(y2);
  }
}

// -------------------------------------------------------------- attention
// grid (chunks, n_kv, batch): a work-group takes positions t0 .. t0 + 63 of one
// key/value head and all query heads of its group (n_q / n_kv <= 16), HB of
// them per wave.  Keys go straight to LDS, 16 bytes per lane, the 16-byte chunk
// c of row t at chunk c ^ (t & 15); lane t scores position t0 + t.  Values go
// straight to registers, a row's words across the lanes.  The operand that all
// lanes share, a query element or a position's weight, is one lane of a
// register that holds 16 of them in each row of 16 lanes.  Sums run over
// positions and dimensions in increasing order, whatever HB.  Output per
// (batch, head, chunk): {max, exp-sum, D unnormalised outputs}; nothing for a
// chunk beyond its sequence's end.
// Long contexts are bound by reading the cache, short ones by one chunk's
// chain of load, score, weight and sum.  Eight sequences of up to 8064
// positions: 32 query and 8 key heads of 128 30.8 us (5.4 TB/s; 42.6 with keys
// and values staged through registers to LDS and one head per wave), 32 key
// heads 119 us (214), 16 and 8 of 256 65 us (170); one of 128 positions 4.2 us
// (4.7).
constexpr uint32_t kAttnChunk = 64;

// Multiply-adds with one lane of each row of 16 as an operand, one rounding
// each: %[o] += (lane 16 (l / 16) + %[l] of %[p]) * %[v].  Such an instruction
// must not follow within two wait states of the one that writes its %[p], and
// the compiler, which pads its own, does not look into assembly: a copy, a
// reload or an accumulator read may stand right before it.  So each statement
// begins with the wait itself and holds every multiply-add of four words; none
// of them writes a %[p].  (One instruction a statement and no wait: eight
// sequences of up to 8064 positions 32.3 us, 32.2 with it; four of up to 1000
// 6.3 and 5.8.)
#define CI_FMA(o, p, v, l) \
  "\n\tv_fmac_f32_dpp %[" o "], %[" p "], %[" v "] row_newbcast:%[" l "] row_mask:0xf bank_mask:0xf"
#define CI_WORDS(w) \
  [x0] "v"(bf_lo(w[0])), [y0] "v"(bf_hi(w[0])), [x1] "v"(bf_lo(w[1])), [y1] "v"(bf_hi(w[1])), \
  [x2] "v"(bf_lo(w[2])), [y2] "v"(bf_hi(w[2])), [x3] "v"(bf_lo(w[3])), [y3] "v"(bf_hi(w[3]))

// s[i] += sum over j of (lane L + j of q[i]) * element j of the four words.
#define CI_S1(v, l) CI_FMA("s0", "q0", v, l)
#define CI_S2(v, l) CI_S1(v, l) CI_FMA("s1", "q1", v, l)
#define CI_S4(v, l) CI_S2(v, l) CI_FMA("s2", "q2", v, l) CI_FMA("s3", "q3", v, l)
#define CI_SCORE(S) \
  "s_nop 1" S("x0", "l0") S("y0", "l1") S("x1", "l2") S("y1", "l3") S("x2", "l4") S("y2", "l5") S("x3", "l6") S("y3", "l7")
template <int L, int HB>
__device__ __forceinline__ void score_8(const uint32_t (&w)[4], const float (&q)[HB], float (&s)[HB]) {
  static_assert(HB == 1 || HB == 2 || HB == 4, "heads of a wave");
#define CI_LANES \
  [l0] "n"(L), [l1] "n"(L + 1), [l2] "n"(L + 2), [l3] "n"(L + 3), [l4] "n"(L + 4), [l5] "n"(L + 5), [l6] "n"(L + 6), [l7] "n"(L + 7)
  if constexpr (HB == 1)
    asm(CI_SCORE(CI_S1) : [s0] "+&v"(s[0]) : [q0] "v"(q[0]), CI_WORDS(w), CI_LANES);
  else if constexpr (HB == 2)
    asm(CI_SCORE(CI_S2) : [s0] "+&v"(s[0]), [s1] "+&v"(s[1]) : [q0] "v"(q[0]), [q1] "v"(q[1]), CI_WORDS(w), CI_LANES);
  else
    asm(CI_SCORE(CI_S4)
        : [s0] "+&v"(s[0]), [s1] "+&v"(s[1]), [s2] "+&v"(s[2]), [s3] "+&v"(s[3])
        : [q0] "v"(q[0]), [q1] "v"(q[1]), [q2] "v"(q[2]), [q3] "v"(q[3]), CI_WORDS(w), CI_LANES);
#undef CI_LANES
}

// a[i], b[i] += sum over j of (lane L + j of p[i]) * the halves of word j.
#define CI_A1(j) CI_FMA("a0", "p0", "x" #j, "l" #j) CI_FMA("b0", "p0", "y" #j, "l" #j)
#define CI_A2(j) CI_A1(j) CI_FMA("a1", "p1", "x" #j, "l" #j) CI_FMA("b1", "p1", "y" #j, "l" #j)
#define CI_A4(j) \
  CI_A2(j) CI_FMA("a2", "p2", "x" #j, "l" #j) CI_FMA("b2", "p2", "y" #j, "l" #j) \
  CI_FMA("a3", "p3", "x" #j, "l" #j) CI_FMA("b3", "p3", "y" #j, "l" #j)
#define CI_ADD(A) "s_nop 1" A(0) A(1) A(2) A(3)
template <int L, int HB>
__device__ __forceinline__ void add_4(const uint32_t (&w)[4], const float (&p)[HB], float (&a)[HB], float (&b)[HB]) {
  static_assert(HB == 1 || HB == 2 || HB == 4, "heads of a wave");
#define CI_LANES [l0] "n"(L), [l1] "n"(L + 1), [l2] "n"(L + 2), [l3] "n"(L + 3)
  if constexpr (HB == 1)
    asm(CI_ADD(CI_A1) : [a0] "+&v"(a[0]), [b0] "+&v"(b[0]) : [p0] "v"(p[0]), CI_WORDS(w), CI_LANES);
  else if constexpr (HB == 2)
    asm(CI_ADD(CI_A2)
        : [a0] "+&v"(a[0]), [b0] "+&v"(b[0]), [a1] "+&v"(a[1]), [b1] "+&v"(b[1])
        : [p0] "v"(p[0]), [p1] "v"(p[1]), CI_WORDS(w), CI_LANES);
  else
    asm(CI_ADD(CI_A4)
        : [a0] "+&v"(a[0]), [b0] "+&v"(b[0]), [a1] "+&v"(a[1]), [b1] "+&v"(b[1]), [a2] "+&v"(a[2]), [b2] "+&v"(b[2]),
          [a3] "+&v"(a[3]), [b3] "+&v"(b[3])
        : [p0] "v"(p[0]), [p1] "v"(p[1]), [p2] "v"(p[2]), [p3] "v"(p[3]), CI_WORDS(w), CI_LANES);
#undef CI_LANES
}
#undef CI_ADD
#undef CI_A4
#undef CI_A2
#undef CI_A1
#undef CI_SCORE
#undef CI_S4
#undef CI_S2
#undef CI_S1
#undef CI_WORDS
#undef CI_FMA

// A rounded product: it must not merge into the subtraction that follows.
__device__ __forceinline__ float scaled(float s, float scale) {
#pragma clang fp contract(off)
  return s * scale;
}

// Value rows in registers, W = D / 128 words per lane each; rows past the
// chunk's end read as zero (out of the buffer's range).
template <int D>
struct ValueRows {
  static constexpr uint32_t W = D / 128, kRows = 32 / W;
  uint32_t v[kRows][W];
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t r0, uint32_t lane) {
#pragma unroll
    for (uint32_t r = 0; r < kRows; ++r) {
      const uint32_t at = (r0 + r) * (D * 2);
      if constexpr (W == 1) {
        v[r][0] = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4 + at, 0, 0);
      } else {
        const auto t = __builtin_amdgcn_raw_buffer_load_b64(rs, lane * 8 + at, 0, 0);
        v[r][0] = t[0];
        v[r][1] = t[1];
      }
    }
  }
  // o[2 u], o[2 u + 1]: of word u, per head; p[r]: the weights of rows 16 r .. + 15
  template <uint32_t R0, uint32_t R, int HB>
  __device__ __forceinline__ void add(const float (&p)[4][HB], float (&o)[2 * W][HB]) const {
    if constexpr (R < kRows) {
#pragma unroll
      for (uint32_t u = 0; u < W; ++u) {
        const uint32_t w[4] = {v[R][u], v[R + 1][u], v[R + 2][u], v[R + 3][u]};
        add_4<(R0 + R) % 16, HB>(w, p[(R0 + R) / 16], o[2 * u], o[2 * u + 1]);
      }
      __builtin_amdgcn_sched_barrier(0);
      add<R0, R + 4, HB>(p, o);
    }
  }
};

// s += q . k over the 16 dimensions of two 16-byte chunks; q: lane l of each
// register holds dimension l % 16.
template <int HB>
__device__ __forceinline__ void score_16(const uint4& a, const uint4& b, const float (&q)[HB], float (&s)[HB]) {
  score_8<0, HB>({a.x, a.y, a.z, a.w}, q, s);
  score_8<8, HB>({b.x, b.y, b.z, b.w}, q, s);
}

template <int D, int HB>
__global__ void __launch_bounds__(1024 / HB) __attribute__((amdgpu_waves_per_eu(4)))
attn_partial_kernel(const float* __restrict__ q, const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc,
                    Positions pos, float* __restrict__ part, uint32_t nq, uint32_t nkv, uint32_t max_ctx,
                    uint32_t nchunks, float scale) {
  using Rows = ValueRows<D>;
  constexpr uint32_t kRow4 = D / 8;                       // 16-byte chunks per cached row
  constexpr uint32_t kPieces = kAttnChunk * kRow4 / 64;   // 1 KiB each
  __shared__ uint4 ks[kAttnChunk * kRow4];
  const uint32_t chunk = blockIdx.x, kvh = blockIdx.y, b = blockIdx.z;
  const uint32_t group = nq / nkv, waves = blockDim.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t T = __builtin_amdgcn_readfirstlane(pos.at(b)) + 1u, t0 = chunk * kAttnChunk;
  if (t0 >= T) return;
  const uint32_t n = min(kAttnChunk, T - t0);
  const size_t base = (((size_t)b * nkv + kvh) * max_ctx + t0) * D;
  const uint8_t* kb = reinterpret_cast<const uint8_t*>(kc + base);
  for (uint32_t i = w; i < kPieces; i += waves) {         // rows past the end repeat the last
    const uint32_t at = i * 64 + lane, t = at / kRow4, c = (at % kRow4) ^ (t & 15u);
    load_lds_16(kb + (min(t, n - 1) * kRow4 + c) * 16, ks + i * 64);
  }
  const uint32_t h0 = w * HB;
  float qr[D / 16][HB];
#pragma unroll
  for (uint32_t i = 0; i < HB; ++i) {
    const float* qh = q + ((size_t)b * nq + kvh * group + min(h0 + i, group - 1)) * D;
#pragma unroll
    for (uint32_t j = 0; j < D / 16; ++j) qr[j][i] = qh[16 * j + (lane & 15u)];
  }
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(vc + base), 0, n * (D * 2), 0x00027000);
  Rows va, vn;
  va.load(rs, 0, lane);
  __builtin_amdgcn_s_waitcnt(kWaitLoads);                 // this wave's loads are in
  __syncthreads();
  vn.load(rs, Rows::kRows, lane);
  float s[HB];
#pragma unroll
  for (uint32_t i = 0; i < HB; ++i) s[i] = 0.0f;
#pragma unroll
  for (uint32_t c = 0; c < kRow4; c += 2)
    score_16<HB>(ks[lane * kRow4 + (c ^ (lane & 15u))], ks[lane * kRow4 + ((c + 1) ^ (lane & 15u))], qr[c / 2], s);
  const bool valid = lane < n;
  float m[HB], l[HB], p[4][HB], o[2 * Rows::W][HB];
#pragma unroll
  for (uint32_t i = 0; i < HB; ++i) {
    s[i] = valid ? scaled(s[i], scale) : -INFINITY;
    m[i] = wave_max_f(s[i]);
  }
#pragma unroll
  for (uint32_t i = 0; i < HB; ++i) {
    const float e = valid ? expf(s[i] - m[i]) : 0.0f;
    l[i] = wave_sum_f(e);
#pragma unroll
    for (uint32_t r = 0; r < 4; ++r) p[r][i] = __shfl(e, 16 * r + (lane & 15u), 64);
#pragma unroll
    for (uint32_t j = 0; j < 2 * Rows::W; ++j) o[j][i] = 0.0f;
  }
  va.template add<0, 0, HB>(p, o);
  if constexpr (D == 256) va.load(rs, 2 * Rows::kRows, lane);
  vn.template add<Rows::kRows, 0, HB>(p, o);
  if constexpr (D == 256) {
    vn.load(rs, 3 * Rows::kRows, lane);
    va.template add<2 * Rows::kRows, 0, HB>(p, o);
    vn.template add<3 * Rows::kRows, 0, HB>(p, o);
  }
#pragma unroll
  for (uint32_t i = 0; i < HB; ++i) {
    if (h0 + i >= group) break;
    float* dst = part + (((size_t)b * nq + kvh * group + h0 + i) * nchunks + chunk) * (D + 2);
    if (lane == 0) {
      dst[0] = m[i];
      dst[1] = l[i];
    }
    float2* d2 = reinterpret_cast<float2*>(dst + 2) + lane * Rows::W;
#pragma unroll
    for (uint32_t u = 0; u < Rows::W; ++u) d2[u] = make_float2(o[2 * u][i], o[2 * u + 1][i]);
  }
}

// grid (n_q, batch), block 256: merge the chunks of one head.  Thread t
// takes chunk maxima t, t+256, ... (block maximum M), then per tile of 256
// chunks the weights e_c = exp(m_c - M) go to LDS and thread t accumulates
// dimension pair t mod (D/2) over chunks t / (D/2), + 256/(D/2), ...; the
// partial sums of the chunk groups are added in a fixed order.
template <int D>
__global__ void __launch_bounds__(256) attn_combine_kernel(const float* __restrict__ part,
                                                           Positions pos,
                                                           uint16_t* __restrict__ out, uint32_t nq,
                                                           uint32_t nchunks) {
  constexpr uint32_t kPairs = D / 2;            // dimension pairs
  constexpr uint32_t kGroups = 256 / kPairs;    // chunk groups (4 for D=128, 2 for D=256)
  __shared__ float s_e[256];
  __shared__ float s_red[4];
  __shared__ float2 s_o[kGroups][kPairs];
  const uint32_t h = blockIdx.x, b = blockIdx.y, t = threadIdx.x;
  const uint32_t nc = (uint32_t)pos.at(b) / 64u + 1u;
  const float* src = part + ((size_t)b * nq + h) * nchunks * (D + 2);
  float mx = -INFINITY;
  for (uint32_t c = t; c < nc; c += 256) mx = fmaxf(mx, src[(size_t)c * (D + 2)]);
  mx = wave_max_f(mx);
  if ((t & 63u) == 0) s_red[t >> 6] = mx;
  __syncthreads();
  const float M = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
  __syncthreads();
  const uint32_t dp = t % kPairs, grp = t / kPairs;
  float lsum = 0.0f;
  float2 o = make_float2(0.0f, 0.0f);
  for (uint32_t c0 = 0; c0 < nc; c0 += 256) {
    const uint32_t n = min(256u, nc - c0);
    float e = 0.0f;
    if (t < n) {
      const float* pc = src + (size_t)(c0 + t) * (D + 2);
      e = expf(pc[0] - M);
      lsum = fmaf(pc[1], e, lsum);
    }
    s_e[t] = e;
    __syncthreads();
#pragma unroll 4
    for (uint32_t c = grp; c < n; c += kGroups) {
      const float ec = s_e[c];
      const float2 v = reinterpret_cast<const float2*>(src + (size_t)(c0 + c) * (D + 2) + 2)[dp];
      o.x = fmaf(v.x, ec, o.x);
      o.y = fmaf(v.y, ec, o.y);
    }
    __syncthreads();
  }
  lsum = wave_sum_f(lsum);
  if ((t & 63u) == 0) s_red[t >> 6] = lsum;
  s_o[grp][dp] = o;
  __syncthreads();
  const float L = (s_red[0] + s_red[1]) + (s_red[2] + s_red[3]);
  if (t < kPairs) {
    float2 acc = s_o[0][t];
#pragma unroll
    for (uint32_t g = 1; g < kGroups; ++g) {
      acc.x += s_o[g][t].x;
      acc.y += s_o[g][t].y;
    }
    uint32_t* dst = reinterpret_cast<uint32_t*>(out + ((size_t)b * nq + h) * D);
    dst[t] = pack2(f32_to_bf16_rne(acc.x / L), f32_to_bf16_rne(acc.y / L));
  }
}

// ------------------------------------------------------------------- SiLU
// Stand-alone form.  gu: batch x 2f FP32 (gate columns, then up columns);
// h: batch x f BF16.
__global__ void __launch_bounds__(256) silu_mul_kernel(const float* __restrict__ gu,
                                                       uint16_t* __restrict__ h, uint32_t f,
                                                       uint32_t batch) {
  const uint64_t n = (uint64_t)batch * f;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) {
    const uint64_t b = i / f, j = i - b * f;
    h[i] = f32_to_bf16_rne(silu_mul_f(gu[b * 2 * f + j], gu[b * 2 * f + f + j]));
  }
}

// Work-groups of `kernel` that fit on the device at once, at most `most` on a
// CU: the size of a persistent grid.
uint32_t resident_wgs(const void* kernel, int threads, int most) {
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, 0) != hipSuccess)
    return 256;
  return (uint32_t)std::max(1, cus * std::min(std::max(per, 1), most));
}

template <int NB, int R, int TH, int IN, int EPI, bool NTL>
uint32_t resident_of() {
  // two rows a wave leave enough in flight with three groups of four waves:
  // 28672 x 4096 39.3 us with three, 41.1 with four, 41.3 with two
  constexpr int kMost = R == 2 && TH == 256 ? 3 : 32;
  static const uint32_t n =
      resident_wgs(reinterpret_cast<const void*>(gemv_fused_kernel<NB, R, TH, IN, EPI, NTL>), TH, kMost);
  return n;
}

template <int NB, int R, int TH, int IN, int EPI, bool NTL>
hipError_t gemv_launch(const GemvArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const uint32_t units = EPI == EPI_PLAIN ? (a.rows + R - 1) / R : a.rows / 2;
  uint32_t grid = (units + TH / 64 - 1) / (TH / 64);
  if (a.k / 8 <= TH * 8 / NB) grid = std::min(grid, resident_of<NB, R, TH, IN, EPI, NTL>());
  if (grid == 0) grid = 1;
  return xlaunch(gemv_fused_kernel<NB, R, TH, IN, EPI, NTL>, dim3(grid), dim3(TH), 0, s, e0, e1, a, units);
}

template <int NB, int IN, int EPI, bool NTL>
hipError_t gemv_rows_r(const GemvArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  // Eight waves share a staging, and twice the LDS: 2 x 28672 rows 39.9 us
  // against 41.2 for four, 4 x 128256 165 against 179.  Four where the rotary
  // factors' registers would leave a CU one work-group of eight (2 x 6144 rows
  // 14.6 us against 16.7), and for one vector (1 x 28672 38.6 against 41.7).
  constexpr int TH = NB == 1 || (NB == 2 && EPI == EPI_ROPE) ? 256 : 512;
  // plain rows: one row per wave while the resident grid still has a wave
  // for every row, two rows otherwise
  if constexpr (EPI == EPI_PLAIN) {
    if (a.rows <= TH / 64 * resident_of<NB, 1, TH, IN, EPI, NTL>())
      return gemv_launch<NB, 1, TH, IN, EPI, NTL>(a, s, e0, e1);
  }
  return gemv_launch<NB, 2, TH, IN, EPI, NTL>(a, s, e0, e1);
}

template <int NB, int IN, int EPI>
hipError_t gemv_stream(const GemvArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  return a.stream ? gemv_rows_r<NB, IN, EPI, true>(a, s, e0, e1) : gemv_rows_r<NB, IN, EPI, false>(a, s, e0, e1);
}

template <int IN, int EPI>
hipError_t gemv_nb(const GemvArgs& a, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (a.batch <= 1) return gemv_stream<1, IN, EPI>(a, s, e0, e1);
  if (a.batch <= 2) return gemv_stream<2, IN, EPI>(a, s, e0, e1);
  if (a.batch <= 4) return gemv_stream<4, IN, EPI>(a, s, e0, e1);
  return gemv_stream<8, IN, EPI>(a, s, e0, e1);
}

}  // namespace

hipError_t launch_gemv_fused(const GemvArgs& a, int input_norm, int epilogue, hipStream_t s, hipEvent_t e0,
                             hipEvent_t e1) {
  if (a.batch == 0 || a.batch > 8 || a.rows == 0 || a.k == 0 || a.k % 8) return hipErrorInvalidValue;
  if (input_norm) {
    switch (epilogue) {
      case EPI_PLAIN: return gemv_nb<IN_NORM, EPI_PLAIN>(a, s, e0, e1);
      case EPI_SILU: return gemv_nb<IN_NORM, EPI_SILU>(a, s, e0, e1);
      case EPI_ROPE: return gemv_nb<IN_NORM, EPI_ROPE>(a, s, e0, e1);
      default: return hipErrorInvalidValue;
    }
  }
  switch (epilogue) {
    case EPI_PLAIN: return gemv_nb<IN_BF16, EPI_PLAIN>(a, s, e0, e1);
    case EPI_SILU: return gemv_nb<IN_BF16, EPI_SILU>(a, s, e0, e1);
    case EPI_ROPE: return gemv_nb<IN_BF16, EPI_ROPE>(a, s, e0, e1);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rmsnorm_bf16(const float* x, const uint16_t* g, uint16_t* y, uint32_t rows,
                               uint32_t n, float eps, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  return xlaunch(rmsnorm_kernel, dim3(rows), dim3(256), 0, s, e0, e1, x, g, y, n, eps);
}

hipError_t launch_rope_append(const float* qkv, const Positions& pos, float* q_out, uint16_t* kc,
                              uint16_t* vc, uint32_t batch, uint32_t nq, uint32_t nkv, uint32_t d,
                              uint32_t max_ctx, float base, hipStream_t s, hipEvent_t e0,
                              hipEvent_t e1) {
  return xlaunch(rope_append_kernel, dim3(batch, nq + 2 * nkv), dim3(d / 2), 0, s, e0, e1, qkv, pos,
                 q_out, kc, vc, nq, nkv, d, max_ctx, base);
}

hipError_t launch_attn_partial(const float* q, const uint16_t* kc, const uint16_t* vc,
                               const Positions& pos, float* part, uint32_t batch, uint32_t nq,
                               uint32_t nkv, uint32_t d, uint32_t max_ctx, uint32_t nchunks,
                               uint32_t used_chunks, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const dim3 grid(used_chunks, nkv, batch);
  const float scale = (float)(1.0 / sqrt((double)d));
  const uint32_t group = nq / nkv;
  auto go = [&](auto kernel, uint32_t hb) {
    return xlaunch(kernel, grid, dim3(64 * ((group + hb - 1) / hb)), 0, s, e0, e1, q, kc, vc, pos, part, nq, nkv,
                   max_ctx, nchunks, scale);
  };
  // Heads per wave.  One leaves the most waves, two unpack a key or value word
  // once for both: 32 query and 8 key heads of 128, 512 work-groups 6.0 us with
  // one (7.1), 1008 9.5 with one (8.2), 8064 35 (30.8).  At most four waves a
  // work-group, as each reads all values through the L1: 16 heads per key head,
  // 20 work-groups 9.2 us with one, 8.0 with two, 6.7 with four.
  const uint32_t hb = group > 8 ? 4 : group > 4 || (group > 1 && used_chunks * nkv * batch > 512) ? 2 : 1;
  if (d == 128)
    return go(hb == 1 ? attn_partial_kernel<128, 1> : hb == 2 ? attn_partial_kernel<128, 2> : attn_partial_kernel<128, 4>, hb);
  if (d == 256)
    return go(hb == 1 ? attn_partial_kernel<256, 1> : hb == 2 ? attn_partial_kernel<256, 2> : attn_partial_kernel<256, 4>, hb);
  return hipErrorInvalidValue;
}

hipError_t launch_attn_combine(const float* part, const Positions& pos, uint16_t* out, uint32_t batch,
                               uint32_t nq, uint32_t d, uint32_t nchunks, hipStream_t s, hipEvent_t e0,
                               hipEvent_t e1) {
  if (d == 128)
    return xlaunch(attn_combine_kernel<128>, dim3(nq, batch), dim3(256), 0, s, e0, e1, part, pos, out, nq,
                   nchunks);
  if (d == 256)
    return xlaunch(attn_combine_kernel<256>, dim3(nq, batch), dim3(256), 0, s, e0, e1, part, pos, out, nq,
                   nchunks);
  return hipErrorInvalidValue;
}

hipError_t launch_silu_mul(const float* gu, uint16_t* h, uint32_t f, uint32_t batch, hipStream_t s,
                           hipEvent_t e0, hipEvent_t e1) {
  const uint64_t n = (uint64_t)batch * f;
  uint64_t g = (n + 255) / 256;
  if (g > 4096) g = 4096;
  if (g == 0) g = 1;
  return xlaunch(silu_mul_kernel, dim3((uint32_t)g), dim3(256), 0, s, e0, e1, gu, h, f, batch);
}

}  // namespace ci
