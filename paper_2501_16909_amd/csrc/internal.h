// Internal declarations shared by the libcoloc translation units: the
// device-side stressor protocol (stressor_dev.h) and the host launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <tuple>
#include <utility>

#include "../../include/coloc.h"

#include "stressor_dev.h"

namespace ci {

// ------------------------------------------------------------ host launchers

template <typename Tup, size_t... I>
inline void fill_args(Tup& t, void** argv, std::index_sequence<I...>) {
  ((argv[I] = static_cast<void*>(&std::get<I>(t))), ...);
}

// Launch with optional start/stop events (kernel-exact timing); returns the
// runtime's status instead of discarding it.
template <typename... KArgs, typename... Args>
inline hipError_t xlaunch(void (*kernel)(KArgs...), dim3 grid, dim3 block, uint32_t shmem,
                          hipStream_t s, hipEvent_t e0, hipEvent_t e1, Args... args) {
  static_assert(sizeof...(KArgs) == sizeof...(Args), "kernel argument count");
  void* argv[sizeof...(Args) + 1];
  std::tuple<KArgs...> tup{static_cast<KArgs>(args)...};
  fill_args(tup, argv, std::index_sequence_for<KArgs...>{});
  if (!e0 && !e1)   // plain launch: capturable into a HIP graph
    return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, argv, shmem, s);
  return hipExtLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, argv, shmem, s,
                            e0, e1, 0);
}
// Loads a kernel's code, which its first launch would otherwise do between a
// timed call's begin stamp and the kernel (2 ms for a module, 10 us for a kernel).
template <typename Kernel>
inline hipError_t preload(Kernel kernel) {
  hipFuncAttributes a;
  return hipFuncGetAttributes(&a, reinterpret_cast<const void*>(kernel));
}
hipError_t preload_triad_victim();
hipError_t preload_dense();
// Each returns hipSuccess or the launch error.  `grid` work-groups.
hipError_t launch_zero(void* p, size_t bytes, hipStream_t s);
hipError_t launch_stamp(uint64_t* slot, hipStream_t s);
// mix: CI_HBM_TRIAD / READ / COPY / WRITE (anything else: triad); chunk:
// 16-byte accesses per lane and stream in one wave-chunk (1, 2 or 4)
// strided: the read-only mix takes fixed per-wave strides instead of tickets
hipError_t launch_stream_stressor(const KCtrl& c, uint32_t mix, uint32_t chunk, const float* b,
                                  const float* cc, float* a, uint64_t n, uint32_t threads,
                                  bool streaming, bool strided, hipStream_t s, hipEvent_t e0,
                                  hipEvent_t e1);
// in_kernel: the passes loop inside one launch (each wave re-sweeps its own
// chunks) instead of one launch per pass
hipError_t launch_triad_victim(const float* b, const float* c, float* a, uint64_t n,
                               uint32_t passes, bool in_kernel, uint32_t num_cus, hipStream_t s,
                               hipEvent_t e0, hipEvent_t e1);
hipError_t launch_cache_stressor(const KCtrl& c, const uint32_t* region, uint64_t region_words,
                                 uint64_t slice_words, uint32_t batch, uint32_t threads,
                                 hipStream_t s,
    hipEvent_t e0, hipEvent_t e1);
hipError_t launch_lds_stressor(const KCtrl& c, const uint32_t* window, uint32_t vw, uint32_t stride,
                               bool load_only, uint32_t threads, hipStream_t s, hipEvent_t e0,
                               hipEvent_t e1);
hipError_t launch_valu_stressor(const KCtrl& c, float* out, uint32_t ilp, uint64_t iters,
                                float fa, float fb, uint32_t threads, hipStream_t s,
    hipEvent_t e0, hipEvent_t e1);
hipError_t launch_valu64_stressor(const KCtrl& c, double* out, uint32_t ilp, uint64_t iters,
                                  double fa, uint32_t threads, hipStream_t s, hipEvent_t e0,
                                  hipEvent_t e1);
hipError_t launch_mfma_stressor(const KCtrl& c, int dtype, const void* a, const void* b,
                                float* out, uint32_t accs, uint64_t iters, uint32_t threads,
                                hipStream_t s,
    hipEvent_t e0, hipEvent_t e1);
hipError_t launch_chase_stressor(const KCtrl& c, const uint32_t* next, uint64_t n, uint32_t* end,
                                 uint32_t chains, uint64_t hops, uint32_t threads, hipStream_t s,
    hipEvent_t e0, hipEvent_t e1);
hipError_t launch_dispatch_empty(uint32_t nwg, hipStream_t s, hipEvent_t e0, hipEvent_t e1);
hipError_t launch_dispatch_count(uint32_t nwg, uint64_t* counter, hipStream_t s, hipEvent_t e0,
                                 hipEvent_t e1);
hipError_t launch_dispatch_announce(HostCtrl* host, hipStream_t s);
hipError_t launch_hog(const KCtrl& c, uint32_t lds_bytes, uint32_t threads, hipStream_t s,
    hipEvent_t e0, hipEvent_t e1);
hipError_t launch_probe(uint32_t nwg, uint32_t* out, hipStream_t s);
hipError_t launch_mfma_probe(int dtype, const void* a, const void* b, const float* c, float* d,
                             uint32_t ntiles, hipStream_t s);
// Checksum of n words: the kernel leaves checksum_parts(n) <= kSumParts pairs
// in `parts` (pinned host memory); once it has finished, checksum_total adds
// them.  `done` (optional) is recorded at the kernel's end.
struct SumPart {
  uint64_t bits;
  double sum;
};
constexpr uint32_t kSumParts = 1024;
uint32_t checksum_parts(uint64_t n);
hipError_t launch_checksum_f32(const float* x, uint64_t n, SumPart* parts, uint64_t* stamp, hipStream_t s,
                               hipEvent_t done);
void checksum_total(const volatile SumPart* parts, uint64_t n, uint64_t* bits, double* sum);
hipError_t launch_to_bf16(const float* x, uint64_t n, uint16_t* out, hipStream_t s);
// n > 0; part: kSumParts floats of device scratch; *amax (pinned) = max |x|
hipError_t launch_quantize_fp8(const float* x, uint64_t n, float* part, float* amax, uint8_t* out,
                               hipStream_t s);
hipError_t launch_gemm(int dtype, const void* a, const void* b, float* c, uint64_t m, uint64_t n,
                       uint64_t k, float scale, hipStream_t s, hipEvent_t e0, hipEvent_t e1);
hipError_t launch_gemv_bf16(const uint16_t* w, const uint16_t* x, float* y, uint64_t n,
                            uint64_t k, uint64_t copies, hipStream_t s, hipEvent_t e0, hipEvent_t e1);
hipError_t launch_fill_uniform(float* dst, uint64_t n, uint64_t seed, hipStream_t s);
hipError_t launch_fill_uniform_bf16(uint16_t* dst, uint64_t n, uint64_t seed, hipStream_t s);
// decode step
hipError_t launch_rmsnorm_bf16(const float* x, const uint16_t* g, uint16_t* y, uint32_t rows,
                               uint32_t n, float eps, hipStream_t s, hipEvent_t e0, hipEvent_t e1);
// Fused decode GEMV (see k_decode.hip): out / h / (q_out, kc, vc) from rows
// of w times batch vectors, given as BF16 v or as FP32 x normalised with g.
struct GemvArgs {
  const uint16_t* w;
  const uint16_t* v;      // BF16 input: batch x k
  const float* x;         // normalised input: batch x k FP32, gain g, eps
  const uint16_t* g;
  const float* res;       // PLAIN: optional residual (may alias out)
  float* out;             // PLAIN: batch x rows FP32
  uint16_t* h;            // SILU: batch x rows/2 BF16
  const int32_t* pos;     // ROPE: device positions; q_out FP32, caches BF16
  float* q_out;
  uint16_t* kc;
  uint16_t* vc;
  uint32_t rows, k, batch;
  uint32_t nq, nkv, d, max_ctx;
  float eps, base;
  bool stream;            // weights beyond the caches: non-temporal loads
};
// Whether weights that a program reads over and over are more than the Infinity
// Cache (256 MiB) keeps: then they are loaded non-temporally (28672 x 4096 cold
// 39 us against 42, 128256 x 4096 157 against 175); what fits is faster cached.
constexpr bool beyond_cache(uint64_t bytes) { return bytes > (256ull << 20); }
constexpr int kEpiPlain = 0, kEpiSilu = 1, kEpiRope = 2;
hipError_t launch_gemv_fused(const GemvArgs& a, int input_norm, int epilogue, hipStream_t s,
                             hipEvent_t e0, hipEvent_t e1);
// Positions of the batch's sequences: by value in the kernel's arguments (no
// copy to wait for), or in device memory (dev != NULL: a captured graph reads
// each replay's own).
struct Positions {
  const int32_t* dev;
  int32_t val[8];
  __device__ __forceinline__ int32_t at(uint32_t b) const { return dev ? dev[b] : val[b]; }
};
hipError_t launch_rope_append(const float* qkv, const Positions& pos, float* q_out, uint16_t* kc,
                              uint16_t* vc, uint32_t batch, uint32_t nq, uint32_t nkv, uint32_t d,
                              uint32_t max_ctx, float base, hipStream_t s, hipEvent_t e0,
                              hipEvent_t e1);
hipError_t launch_attn_partial(const float* q, const uint16_t* kc, const uint16_t* vc,
                               const Positions& pos, float* part, uint32_t batch, uint32_t nq,
                               uint32_t nkv, uint32_t d, uint32_t max_ctx, uint32_t nchunks,
                               uint32_t used_chunks, hipStream_t s, hipEvent_t e0, hipEvent_t e1);
hipError_t launch_attn_combine(const float* part, const Positions& pos, uint16_t* out, uint32_t batch,
                               uint32_t nq, uint32_t d, uint32_t nchunks, hipStream_t s, hipEvent_t e0,
                               hipEvent_t e1);
hipError_t launch_silu_mul(const float* gu, uint16_t* h, uint32_t f, uint32_t batch, hipStream_t s,
                           hipEvent_t e0, hipEvent_t e1);

// Victim constraints checked on the host before any launch.
constexpr uint32_t kTriadThreads = 256;

}  // namespace ci
