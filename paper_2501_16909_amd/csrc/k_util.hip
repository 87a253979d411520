// Output checksums, per-tensor quantisation and the request-input fill used
// by the serving loop.
#include "internal.h"

namespace ci {
namespace {

// Output checksum: work-group p sums the contiguous range [p * len,
// (p + 1) * len) -- thread t the groups of four t, t + 256, ... of it, in
// order, then a fixed tree over the work-group -- and stores one {bits, sum}
// pair to pinned host memory, where the host adds the pairs in order
// (checksum_total): no second kernel, and the FP64 sum is the same on every
// run.  *stamp (optional) takes the device clock as the kernel starts, which
// is the end of whatever ran before it in the stream.
// Bound by HBM reads: four non-temporal 16-byte loads per thread in flight on
// up to 1024 work-groups (four per CU) read 1 GiB in 153 us, 7.0 TB/s (cached
// loads 177 us, 512 or 2048 work-groups the same); one 4-byte load per thread
// took 503 us.  More work-groups only add stores to host memory (1 M words:
// 4.0 us with 1024, 5.7 with 2048, 10 with 4096).  The loads need only 4-byte
// alignment, so any FP32 pointer takes this path.
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr uint32_t kSumThreads = 256;
constexpr uint32_t kSumUnroll = 4;

__device__ __forceinline__ void sum4(f4u v, uint64_t& bits, double& sum) {
  bits += (uint64_t)__float_as_uint(v.x) + __float_as_uint(v.y);
  bits += (uint64_t)__float_as_uint(v.z) + __float_as_uint(v.w);
  sum += (double)v.x;
  sum += (double)v.y;
  sum += (double)v.z;
  sum += (double)v.w;
}

__global__ void __launch_bounds__(kSumThreads) checksum_kernel(const float* __restrict__ x, uint64_t n,
                                                               uint64_t len, SumPart* parts,
                                                               uint64_t* stamp) {
  __shared__ uint64_t sb[kSumThreads / 64];
  __shared__ double ss[kSumThreads / 64];
  if (stamp && blockIdx.x == 0 && threadIdx.x == 0) *stamp = dev_now();
  const uint64_t lo = (uint64_t)blockIdx.x * len;
  const uint64_t hi = lo + len < n ? lo + len : n;
  uint64_t bits = 0;
  double sum = 0.0;
  if (lo < hi) {
    const uint64_t n4 = (hi - lo) / 4;
    const f4u* x4 = reinterpret_cast<const f4u*>(x + lo);
    uint64_t i = threadIdx.x;
    for (; i + (kSumUnroll - 1) * kSumThreads < n4; i += kSumUnroll * kSumThreads) {
      f4u v[kSumUnroll];
#pragma unroll
      for (uint32_t u = 0; u < kSumUnroll; ++u) v[u] = __builtin_nontemporal_load(x4 + i + u * kSumThreads);
#pragma unroll
      for (uint32_t u = 0; u < kSumUnroll; ++u) sum4(v[u], bits, sum);
    }
    for (; i < n4; i += kSumThreads) sum4(x4[i], bits, sum);
    const uint64_t rest = lo + 4 * n4 + threadIdx.x;   // fewer than four words, in the last range only
    if (rest < hi) {
      const float v = x[rest];
      bits += (uint64_t)__float_as_uint(v);
      sum += (double)v;
    }
  }
  for (int off = 32; off > 0; off >>= 1) {
    bits += __shfl_xor(bits, off, 64);
    sum += __shfl_xor(sum, off, 64);
  }
  if ((threadIdx.x & 63u) == 0) {
    sb[threadIdx.x >> 6] = bits;
    ss[threadIdx.x >> 6] = sum;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    parts[blockIdx.x].bits = (sb[0] + sb[1]) + (sb[2] + sb[3]);
    parts[blockIdx.x].sum = (ss[0] + ss[1]) + (ss[2] + ss[3]);
  }
}

// Per-tensor quantisation in two kernels, both bound by HBM: amax_kernel
// leaves one maximum per work-group (the checksum's ranges and loads), and
// every work-group of to_fp8_kernel reduces those (4 KiB, from L2) before it
// converts, so no launch sits between them.  For 8192 x 8192 values the
// maximum takes 43 us (6.3 TB/s; 116 us with 4-byte loads) and the conversion
// 54 us (6.2 TB/s read and written; 86 us with 1-byte stores and integer
// rounding).
__global__ void __launch_bounds__(256) amax_kernel(const float* __restrict__ x, uint64_t n, uint64_t len,
                                                   float* part) {
  __shared__ float sm[4];
  const uint64_t lo = (uint64_t)blockIdx.x * len;
  const uint64_t hi = lo + len < n ? lo + len : n;
  float m = 0.0f;
  auto max4 = [&m](f4u v) { m = fmaxf(fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w))); };
  if (lo < hi) {
    const uint64_t n4 = (hi - lo) / 4;
    const f4u* x4 = reinterpret_cast<const f4u*>(x + lo);
    uint64_t i = threadIdx.x;
    for (; i + 3 * 256 < n4; i += 4 * 256) {
      f4u v[4];
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(x4 + i + u * 256);
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) max4(v[u]);
    }
    for (; i < n4; i += 256) max4(x4[i]);
    const uint64_t rest = lo + 4 * n4 + threadIdx.x;
    if (rest < hi) m = fmaxf(m, fabsf(x[rest]));
  }
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  if ((threadIdx.x & 63u) == 0) sm[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
}

// FP32 -> BF16, round to nearest even by integer arithmetic on the bit
// pattern; NaN -> quiet NaN of the same sign.
__device__ __forceinline__ uint16_t to_bf16(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)(((u >> 16) & 0x8000u) | 0x7FC0u);
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// Four at once with the conversion instruction, which rounds as to_bf16 does
// for every FP32 value but NaN (all 2^32 patterns compared); a sum that is
// NaN sends the four through to_bf16 (a NaN among them, or opposite
// infinities).
typedef uint16_t us4 __attribute__((ext_vector_type(4), aligned(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ us4 to_bf16_4(f4u v) {
  const float s = (v.x + v.y) + (v.z + v.w);
  if (__builtin_expect(s != s, 0)) return us4{to_bf16(v.x), to_bf16(v.y), to_bf16(v.z), to_bf16(v.w)};
  const f4v a = v;
  return __builtin_bit_cast(us4, __builtin_convertvector(a, bf4v));
}

// Tiles of kTile elements per work-group, four 16-byte loads per thread in
// flight; the last, partial tile is walked four elements, then one, at a time.
constexpr uint32_t kTile = 256 * 16;

template <typename F4, typename F1>
__device__ __forceinline__ void for_tiles(const float* __restrict__ x, uint64_t n, F4 four, F1 one) {
  const f4u* x4 = reinterpret_cast<const f4u*>(x);
  for (uint64_t t = blockIdx.x; t * kTile < n; t += gridDim.x) {
    const uint64_t i0 = t * (kTile / 4) + threadIdx.x;
    if ((t + 1) * kTile <= n) {
      f4u v[4];
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(x4 + i0 + u * 256);
#pragma unroll
      for (uint32_t u = 0; u < 4; ++u) four(i0 + u * 256, v[u]);
    } else {
      for (uint64_t i = i0; i < n / 4; i += 256) four(i, x4[i]);
      const uint64_t rest = (n & ~3ull) + threadIdx.x;
      if (rest < n) one(rest, x[rest]);
    }
  }
}

__global__ void __launch_bounds__(256) to_bf16_kernel(const float* __restrict__ x, uint64_t n,
                                                      uint16_t* __restrict__ out) {
  us4* o4 = reinterpret_cast<us4*>(out);
  for_tiles(x, n, [o4](uint64_t i, f4u v) { o4[i] = to_bf16_4(v); },
            [out](uint64_t i, float v) { out[i] = to_bf16(v); });
}

// FP32 -> OCP E4M3FN with round-to-nearest-even and saturation at +-448.
// Normal range (|y| >= 2^-6): keep 3 of the 23 mantissa bits, rounding on the
// 20 dropped bits; subnormal range: |y| * 2^9 rounded to an integer (exact
// scaling, v_rndne rounding), which also yields 2^-6 (code 8) on carry.
__device__ __forceinline__ uint8_t to_e4m3(float y) {
  const uint32_t u = __float_as_uint(y);
  const uint8_t sign = (uint8_t)((u >> 24) & 0x80u);
  const uint32_t a = u & 0x7FFFFFFFu;
  if (a > 0x7F800000u) return sign | 0x7Fu;          // NaN
  if (a >= 0x43E00000u) return sign | 0x7Eu;         // >= 448 (incl. inf): saturate
  const int e = (int)(a >> 23) - 127;
  if (e >= -6) {
    const uint32_t m = a & 0x7FFFFFu;
    uint32_t code = ((uint32_t)(e + 7) << 3) | (m >> 20);
    const uint32_t rem = m & 0xFFFFFu;
    if (rem > 0x80000u || (rem == 0x80000u && (code & 1u))) ++code;
    if (code > 0x7Eu) code = 0x7Eu;
    return sign | (uint8_t)code;
  }
  const float s = __uint_as_float(a) * 512.0f;       // exact
  const uint32_t q = (uint32_t)__builtin_rintf(s);  // nearest, ties to even
  return sign | (uint8_t)q;
}

// Four products x * inv at once: clamped to +-448, the conversion instruction
// gives to_e4m3's code for every FP32 value but NaN (all 2^32 patterns
// compared), which takes to_e4m3 itself.
typedef uint32_t u32u __attribute__((aligned(1)));

__device__ __forceinline__ uint32_t to_e4m3_4(f4u v, float inv) {
  const float a = __fmul_rn(v.x, inv), b = __fmul_rn(v.y, inv);   // lone products: nothing to contract
  const float c = __fmul_rn(v.z, inv), d = __fmul_rn(v.w, inv);
  const float s = (a + b) + (c + d);
  if (__builtin_expect(s != s, 0))
    return (uint32_t)to_e4m3(a) | (uint32_t)to_e4m3(b) << 8 | (uint32_t)to_e4m3(c) << 16 | (uint32_t)to_e4m3(d) << 24;
  const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_fmed3f(a, -448.0f, 448.0f),
                                                 __builtin_amdgcn_fmed3f(b, -448.0f, 448.0f), 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_fmed3f(c, -448.0f, 448.0f),
                                                   __builtin_amdgcn_fmed3f(d, -448.0f, 448.0f), lo, true);
}

__global__ void __launch_bounds__(256) to_fp8_kernel(const float* __restrict__ x, uint64_t n,
                                                     const float* __restrict__ part, uint32_t nparts,
                                                     float* amax, uint8_t* __restrict__ out) {
  __shared__ float sm[4];
  float m = 0.0f;
  for (uint32_t i = threadIdx.x; i < nparts; i += 256) m = fmaxf(m, part[i]);
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  if ((threadIdx.x & 63u) == 0) sm[threadIdx.x >> 6] = m;
  __syncthreads();
  m = fmaxf(fmaxf(sm[0], sm[1]), fmaxf(sm[2], sm[3]));
  if (blockIdx.x == 0 && threadIdx.x == 0) *amax = m;
  const float inv = (m > 0.0f && m <= 3.402823466e38f) ? __fdiv_rn(448.0f, m) : 1.0f;
  u32u* o4 = reinterpret_cast<u32u*>(out);
  for_tiles(x, n, [o4, inv](uint64_t i, f4u v) { o4[i] = to_e4m3_4(v, inv); },
            [out, inv](uint64_t i, float v) { out[i] = to_e4m3(__fmul_rn(v, inv)); });
}

__device__ __forceinline__ float uniform_from_word(uint64_t z) {
#pragma clang fp contract(off)
  const float k = (float)(uint32_t)(z >> 40);  // 24-bit integer: exact
  const float scaled = k * 0x1.0p-23f;          // exact
  return scaled - 1.0f;                         // exact
}

// Request inputs of the serving loop: SplitMix64 (Steele, Lea and Flood,
// OOPSLA 2014) in counter form, word i of stream `seed` = mix(seed + (i+1)G),
// mapped to a uniform value on [-1, 1) with 24 random bits, and rounded to BF16
// where the request reads BF16.  Four elements per thread: one multiplication
// less for three of them, and 16-byte stores.
// The 64-bit multiplications bound it: 2^28 elements FP32 194 us (5.5 TB/s; 243
// with one element per thread), 7424^2 in BF16 53 us (106 through FP32).
constexpr uint64_t kGolden = 0x9E3779B97F4A7C15ull;

__device__ __forceinline__ float uniform_at(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return uniform_from_word(z);
}

template <typename T>
__global__ void __launch_bounds__(256) fill_uniform_kernel(T* __restrict__ dst, uint64_t n, uint64_t seed) {
  const uint64_t stride = (uint64_t)gridDim.x * 256;
  for (uint64_t t = (uint64_t)blockIdx.x * 256 + threadIdx.x; 4 * t < n; t += stride) {
    uint64_t z = seed + (4 * t + 1) * kGolden;
    f4u v;
#pragma unroll
    for (int u = 0; u < 4; ++u, z += kGolden) v[u] = uniform_at(z);
    if (4 * t + 4 <= n) {
      if constexpr (sizeof(T) == 4) reinterpret_cast<f4u*>(dst)[t] = v;
      else reinterpret_cast<us4*>(dst)[t] = to_bf16_4(v);
    } else {
      for (uint32_t u = 0; u < n - 4 * t; ++u) {
        if constexpr (sizeof(T) == 4) dst[4 * t + u] = v[u];
        else dst[4 * t + u] = to_bf16(v[u]);
      }
    }
  }
}

uint32_t grid_for(uint64_t n) {
  uint64_t g = (n + 255) / 256;
  if (g > 16384) g = 16384;
  if (g == 0) g = 1;
  return (uint32_t)g;
}

}  // namespace

uint32_t checksum_parts(uint64_t n) {
  // at least sixteen words per thread, at most four work-groups per CU
  const uint64_t p = (n + 4095) / 4096;
  return (uint32_t)(p < 1 ? 1 : p > kSumParts ? kSumParts : p);
}

hipError_t launch_checksum_f32(const float* x, uint64_t n, SumPart* parts, uint64_t* stamp, hipStream_t s,
                               hipEvent_t done) {
  const uint32_t np = checksum_parts(n);
  const uint64_t len = ((n + np - 1) / np + 3) & ~3ull;   // whole groups of four
  return xlaunch(checksum_kernel, dim3(np), dim3(kSumThreads), 0, s, nullptr, done, x, n, len, parts, stamp);
}

void checksum_total(const volatile SumPart* parts, uint64_t n, uint64_t* bits, double* sum) {
  const uint32_t np = checksum_parts(n);
  uint64_t b = 0;
  double t = 0.0;
  for (uint32_t i = 0; i < np; ++i) {
    b += parts[i].bits;
    t += parts[i].sum;
  }
  *bits = b;
  *sum = t;
}

namespace {
// Work-groups of the tiled kernels: four per CU walk whatever is more (the
// FP8 conversion of 8192 x 8192 ran 3-5 us slower with 2048 to 16384).
uint32_t tile_grid(uint64_t n) {
  const uint64_t t = (n + kTile - 1) / kTile;
  return (uint32_t)(t > 1024 ? 1024 : t);
}
}  // namespace

hipError_t launch_to_bf16(const float* x, uint64_t n, uint16_t* out, hipStream_t s) {
  if (n == 0) return hipSuccess;
  return xlaunch(to_bf16_kernel, dim3(tile_grid(n)), dim3(256), 0, s, nullptr, nullptr, x, n, out);
}

hipError_t launch_quantize_fp8(const float* x, uint64_t n, float* part, float* amax, uint8_t* out, hipStream_t s) {
  const uint32_t np = checksum_parts(n);
  const uint64_t len = ((n + np - 1) / np + 3) & ~3ull;
  const hipError_t e = xlaunch(amax_kernel, dim3(np), dim3(256), 0, s, nullptr, nullptr, x, n, len, part);
  if (e != hipSuccess) return e;
  return xlaunch(to_fp8_kernel, dim3(tile_grid(n)), dim3(256), 0, s, nullptr, nullptr, x, n, part, np, amax, out);
}

// dst: 16-byte aligned
hipError_t launch_fill_uniform(float* dst, uint64_t n, uint64_t seed, hipStream_t s) {
  if (n == 0) return hipSuccess;
  return xlaunch(fill_uniform_kernel<float>, dim3(grid_for((n + 3) / 4)), dim3(256), 0, s, nullptr, nullptr, dst, n, seed);
}

hipError_t launch_fill_uniform_bf16(uint16_t* dst, uint64_t n, uint64_t seed, hipStream_t s) {
  if (n == 0) return hipSuccess;
  return xlaunch(fill_uniform_kernel<uint16_t>, dim3(grid_for((n + 3) / 4)), dim3(256), 0, s, nullptr, nullptr, dst, n,
                 seed);
}

}  // namespace ci
