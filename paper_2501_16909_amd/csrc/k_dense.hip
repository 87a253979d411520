// Dense victims: GEMM C = s * A B^T on the matrix cores, and the BF16 GEMV
// y = W x.  The paper's shared-memory experiment uses a GEMM as the victim
// (Section 4.4.1, Figure 4) and its LLM decode victims are dominated by
// matrix-vector products that stream weights from memory (Sections 4.2-4.3).
//
// GEMM layout: A is M x K and B is N x K, both row-major (K contiguous), C is
// M x N FP32 row-major.  Three kernels, one summation order (each output is
// the MFMA chain over K in increasing order, so they agree bit for bit):
//   gemm_tile_kernel  tiles of 64 x 64, 128 x 64 or 128 x 128, four waves;
//                     every shape;
//   gemm256d_kernel   BF16 and FP8, 256 x 256 tiles, eight waves in two
//                     alternating groups;
//   gemm256f_kernel   FP32, 256 x 256 tiles, eight waves.
// All move operands straight from global memory into LDS, 16 bytes per lane.
// K * element size must be a multiple of 16; any M and N work.
#include <type_traits>

#include "internal.h"

namespace ci {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// A K-stage in LDS: 128 bytes of each row, so that every row of a load is a
// whole cache line (64-byte stages reached three quarters of the rate from
// L2).  The 16-byte chunk c of row r sits at chunk c ^ ((r >> 1) & 7): the 16
// rows a fragment read touches at a time fall on 16 distinct chunk positions
// of the banks, and a 1 KiB load (eight rows, lane l filling bytes 16 l) still
// fills its rows in place.
constexpr uint32_t kStage = 128;

__device__ __forceinline__ uint32_t stage_at(uint32_t row, uint32_t byte) {
  return row * kStage + ((((byte >> 4) ^ (row >> 1)) & 7u) << 4) + (byte & 15u);
}

// Logical chunk that lane `lane` of a load carries for row `row`.
__device__ __forceinline__ uint32_t lane_chunk(uint32_t lane, uint32_t row) {
  return ((lane & 7u) ^ (row >> 1)) & 7u;
}

__device__ __forceinline__ void load16_lds(const uint8_t* g, uint8_t* l) {
  __builtin_amdgcn_global_load_lds(g, l, 16, 0, 0);
}

// Operand fragments and products.  kStep: K bytes one fragment covers (k-step);
// off: the lane's byte offset inside it; cut: zero what lies past `rem` bytes.
template <int DT>
struct Op;

// FP32: a fragment is one 16-byte chunk, four k and two instructions; both
// halves of the wave read it whole and half h takes k = 2 t + h.
template <>
struct Op<CI_DT_F32> {
  using T = f32x4;
  static constexpr int kElem = 4;
  static constexpr int kStep = 16;
  __device__ static uint32_t off(uint32_t) { return 0; }
  __device__ static T ld(const uint8_t* p, uint32_t row, uint32_t kb) {
    return *reinterpret_cast<const f32x4*>(p + stage_at(row, kb));
  }
  __device__ static void cut(T& f, uint32_t kb, uint32_t rem) {
    if (kb + 16 > rem) f = f32x4{0, 0, 0, 0};
  }
  __device__ static f32x16 mma(const T& a, const T& b, f32x16 c, uint32_t lane) {
    const bool h = lane >= 32;
    c = __builtin_amdgcn_mfma_f32_32x32x2f32(h ? a.y : a.x, h ? b.y : b.x, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x2f32(h ? a.w : a.z, h ? b.w : b.z, c, 0, 0, 0);
  }
};

template <>
struct Op<CI_DT_BF16> {
  using T = bf16x8;
  static constexpr int kElem = 2;
  static constexpr int kStep = 32;
  __device__ static uint32_t off(uint32_t lane) { return (lane >> 5) * 16; }
  __device__ static T ld(const uint8_t* p, uint32_t row, uint32_t kb) {
    return *reinterpret_cast<const bf16x8*>(p + stage_at(row, kb));
  }
  __device__ static void cut(T& f, uint32_t kb, uint32_t rem) {
    if (kb + 16 > rem) f = __builtin_bit_cast(bf16x8, i32x4{0, 0, 0, 0});
  }
  __device__ static f32x16 mma(const T& a, const T& b, f32x16 c, uint32_t) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};

template <>
struct Op<CI_DT_FP8E4M3> {
  using T = i32x8;
  static constexpr int kElem = 1;
  static constexpr int kStep = 64;
  __device__ static uint32_t off(uint32_t lane) { return (lane >> 5) * 32; }
  __device__ static T ld(const uint8_t* p, uint32_t row, uint32_t kb) {
    const i32x4 a0 = *reinterpret_cast<const i32x4*>(p + stage_at(row, kb));
    const i32x4 a1 = *reinterpret_cast<const i32x4*>(p + stage_at(row, kb + 16));
    return i32x8{a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
  }
  __device__ static void cut(T& f, uint32_t kb, uint32_t rem) {
    const int lo = kb + 16 <= rem ? -1 : 0, hi = kb + 32 <= rem ? -1 : 0;
    f = f & i32x8{lo, lo, lo, lo, hi, hi, hi, hi};
  }
  __device__ static f32x16 mma(const T& a, const T& b, f32x16 c, uint32_t) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
  }
};

// s_waitcnt operands: vector-memory count n with no other wait, and LDS reads.
constexpr int kWaitLds = 0xC07F;
constexpr int wait_vm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// Map the work-group index to a C tile.  Work-groups are dealt to the 8
// XCDs round-robin, so first each XCD gets a contiguous range of tile
// numbers t; then t runs down bands of 4 tile rows (column by column within
// a band), so the tiles an XCD computes at one time form a 4 x 8 block that
// shares 4 A panels and 8 B panels in that XCD's L2 (a 2 x 16 row-major
// block would need 18).
template <uint32_t kBand = 4>
__device__ __forceinline__ void tile_of(uint32_t bid, uint32_t nbm, uint32_t nbn, uint32_t& tm,
                                        uint32_t& tn) {
  const uint32_t nb = nbm * nbn;
  uint32_t t = bid;
  if ((nb & 7u) == 0) t = (bid & 7u) * (nb >> 3) + (bid >> 3);
  const uint32_t band = kBand * nbn, group = t / band;
  const uint32_t first = group * kBand, rows = min(nbm - first, kBand), r = t - group * band;
  tm = first + r % rows;
  tn = r / rows;
}

// General tile kernel: a work-group of four waves (2 x 2, each TM/2 x TN/2)
// owns a TM x TN tile of C, SL K-stages in LDS (2 or 4).  A stage is two halves of
// k-steps with a fragment buffer each: while one half multiplies, the other's
// fragments are read, across stage boundaries too.  One barrier per stage:
// after it the next stage is in LDS and the finished one's slot takes the
// stage SL on.  With two, LDS per work-group is 32, 48 or 64 KiB, so two to five share a
// CU and cover each other's barriers and load latency; a third slot instead of
// the second work-group was slower (BF16 4096^3 166 against 135 us).
// What bounds it: at one work-group per CU the chain of load, barrier and
// fragment read of every stage (BF16 512^3: 5.8 us against 12.7 us for the
// register-staged 128 x 128 kernel it replaces, 1024^3 9.1 against 20.5); with
// several, the matrix core (FP32 1416 x 1402 x 1416 67 against 118 us, where
// 132 tiles of 128 x 128 left half the CUs idle; floor 36 us).
// Rows past the edge repeat the last one and feed outputs that are not
// stored; in a short last stage, chunks past its end repeat its last one and
// the fragments there are zeroed.
template <int DT, int TM, int TN, int SL>
__global__ void __launch_bounds__(256, TM * TN >= 128 * 128 ? 2 : 1)
gemm_tile_kernel(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, float* __restrict__ C, uint32_t M,
                 uint32_t N, uint32_t K, float scale) {
  using F = Op<DT>;
  constexpr int W = 4, IN = TM / 64, JN = TN / 64;                 // waves; 32 x 32 tiles per wave
  constexpr int kOpA = TM * kStage, kSlot = (TM + TN) * kStage;
  constexpr int OA = TM / 8 / W, OPS = (TM + TN) / 8 / W;          // 1 KiB loads per wave and stage: A, all
  constexpr int NS = kStage / F::kStep / 2;                        // k-steps per half stage
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const uint32_t nbm = (M + TM - 1) / TM, nbn = (N + TN - 1) / TN;
  uint32_t tm, tn;
  tile_of<8>(blockIdx.x, nbm, nbn, tm, tn);
  const uint32_t lane = threadIdx.x & 63u, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t wm = wid >> 1, wn = wid & 1u;
  const uint64_t rowBytes = (uint64_t)K * F::kElem;
  const uint32_t nst = (uint32_t)((rowBytes + kStage - 1) / kStage);
  const uint32_t rem = (uint32_t)(rowBytes - (uint64_t)(nst - 1) * kStage);   // bytes of the last stage, 16..128
  // load o of a wave fills rows 8 (wid + W o) .. + 7 of an operand, lane l row l / 8
  auto load_row = [&](int o) { return 8u * (wid + W * (o < OA ? o : o - OA)) + (lane >> 3); };
  const uint8_t* src[OPS];      // this lane's 16 bytes of the next stage to load
#pragma unroll
  for (int o = 0; o < OPS; ++o) {
    const uint32_t r = load_row(o);
    const uint64_t g = o < OA ? min(tm * TM + r, M - 1) : min(tn * TN + r, N - 1);
    src[o] = (o < OA ? A : B) + g * rowBytes + lane_chunk(lane, r) * 16u;
  }
  auto issue = [&](uint32_t st) {
    uint8_t* slot = smem + (st % SL) * kSlot;
    if (st + 1 == nst && rem < kStage) {
#pragma unroll
      for (int o = 0; o < OPS; ++o) {
        const uint32_t c = lane_chunk(lane, load_row(o));
        src[o] -= (c - min(c, rem / 16 - 1)) * 16u;
      }
    }
#pragma unroll
    for (int o = 0; o < OPS; ++o) {
      load16_lds(src[o], slot + (o < OA ? (wid + W * o) * 1024u : kOpA + (wid + W * (o - OA)) * 1024u));
      src[o] += kStage;
    }
  };
  f32x16 acc[IN][JN];
#pragma unroll
  for (int i = 0; i < IN; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
  const uint32_t frow = lane & 31u, fk = F::off(lane);
  typename F::T fa[2][NS][IN], fb[2][NS][JN];
  auto read_ks = [&](uint32_t st, auto half, int s) {
    constexpr int b = decltype(half)::value;
    const uint8_t* slot = smem + (st % SL) * kSlot;
    const uint32_t kb = b * (kStage / 2) + fk + s * F::kStep;
#pragma unroll
    for (int i = 0; i < IN; ++i) fa[b][s][i] = F::ld(slot, wm * (TM / 2) + i * 32 + frow, kb);
#pragma unroll
    for (int j = 0; j < JN; ++j) fb[b][s][j] = F::ld(slot + kOpA, wn * (TN / 2) + j * 32 + frow, kb);
  };
  auto mma_ks = [&](auto half, int s) {
    constexpr int b = decltype(half)::value;
#pragma unroll
    for (int i = 0; i < IN; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j) acc[i][j] = F::mma(fa[b][s][i], fb[b][s][j], acc[i][j], lane);
  };
  using H0 = std::integral_constant<int, 0>;
  using H1 = std::integral_constant<int, 1>;
#pragma unroll
  for (uint32_t q = 0; q < SL; ++q)
    if (q < nst) issue(q);
  if (nst >= SL) __builtin_amdgcn_s_waitcnt(wait_vm((SL - 1) * OPS));
  else __builtin_amdgcn_s_waitcnt(wait_vm(0));
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < NS; ++s) read_ks(0, H0{}, s);
  uint32_t st = 0;
  for (; st + 1 < nst; ++st) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      read_ks(st, H1{}, s);
      mma_ks(H0{}, s);
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kWaitLds);     // this wave's reads of the slot are done
    if (st + SL <= nst) __builtin_amdgcn_s_waitcnt(wait_vm((SL - 2) * OPS));   // its part of stage st + 1 has landed
    else __builtin_amdgcn_s_waitcnt(wait_vm(0));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      read_ks(st + 1, H0{}, s);
      if (s == NS - 1 && st + SL < nst) issue(st + SL);
      mma_ks(H1{}, s);
    }
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) read_ks(st, H1{}, s);
  if (rem < kStage) {
    auto cut_half = [&](auto half) {
      constexpr int b = decltype(half)::value;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const uint32_t kb = b * (kStage / 2) + fk + s * F::kStep;
#pragma unroll
        for (int i = 0; i < IN; ++i) F::cut(fa[b][s][i], kb, rem);
#pragma unroll
        for (int j = 0; j < JN; ++j) F::cut(fb[b][s][j], kb, rem);
      }
    };
    cut_half(H0{});
    cut_half(H1{});
  }
#pragma unroll
  for (int s = 0; s < NS; ++s) mma_ks(H0{}, s);
  if (rem > kStage / 2)
#pragma unroll
    for (int s = 0; s < NS; ++s) mma_ks(H1{}, s);
#pragma unroll
  for (int i = 0; i < IN; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      const uint32_t col = tn * TN + wn * (TN / 2) + j * 32 + (lane & 31u);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t row = tm * TM + wm * (TM / 2) + i * 32 + 8u * (v / 4) + 4u * (lane >> 5) + (v % 4);
        if (row < M && col < N) C[(uint64_t)row * N + col] = acc[i][j][v] * scale;
      }
    }
}

// Large-tile kernel of BF16 and FP8: one work-group per CU owns a 256 x 256
// tile, eight waves in a 2 x 4 grid, each 128 x 64 (4 x 2 MFMA tiles), two
// K-stages of 64 KiB in LDS.  The two rows of waves (wm 0 and 1, one wave of
// each per SIMD) run one phase apart: in a phase one row reads half a stage's
// fragments and issues loads while the other multiplies its half, and a
// barrier ends the phase, so the matrix core of every SIMD always has one
// wave's sixteen (FP8: eight) MFMAs ahead of it.
//   Loads of stage st + 1 go into the slot of st - 1, free once the later row
// has read its second half: half of them with the first fragment reads of st,
// half behind the first MFMAs, which spreads them over the load path.
//   FAR (more tiles than CUs): each stage also touches its share of the lines
// that the XCD's block of tiles needs kAhead stages later.  The 32 tiles an
// XCD computes at a time share their panels, so without this only two stages
// of each panel are ever on their way into its L2, and their latency, not a
// bandwidth, sets the rate (loads alone: 8192^3 780 us without, 567 with).
// Edge tiles start early and overlap their neighbour, so every row read
// exists; rows or columns that are the neighbour's are not stored.
// What bounds it: with random operands the part lowers its clock under MFMA
// load (1.6-1.9 GHz measured in the loop), and the loop with its loads left out
// runs 8192^3 BF16 in 737 us; with them a phase takes 705 clocks instead of
// 566, the load path being shared with the fragment reads.  On a part that
// other work has not warmed, against the one-group ring before it: BF16 8192^3
// 828 us (1330 TF; 970), FP8 397 (2770 TF; 483), BF16 4096^3 110 (128); after
// seconds of load BF16 8192^3 takes 920 us (1200 TF), FP8 485.
// At most 192 registers per wave and 129 KiB of LDS, so that two 64-register
// stressor waves per SIMD and up to 31 KiB of LDS still fit beside it.
constexpr uint32_t kBig = 256;
constexpr uint32_t kBigOp = kBig * kStage;          // one operand of a stage
constexpr uint32_t kBigSlot = 2 * kBigOp;
constexpr uint32_t kBigLds = 2 * kBigSlot + 256;    // and 256 bytes that FAR's touches land in
constexpr uint32_t kAhead = 4;
static_assert(kBigLds <= 129 * 1024, "the slots must leave LDS for a co-resident work-group");

template <int DT, bool FAR>
__global__ void __launch_bounds__(512, 1) __attribute__((amdgpu_num_vgpr(192)))
gemm256d_kernel(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, float* __restrict__ C, uint32_t M,
                uint32_t N, uint32_t K, float scale) {
  using F = Op<DT>;
  constexpr int IN = 4, JN = 2, NS = kStage / F::kStep / 2;
  constexpr uint32_t BAND = FAR ? 4 : 8;
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const uint32_t nbm = (M + kBig - 1) / kBig, nbn = (N + kBig - 1) / kBig;
  uint32_t tm, tn;
  tile_of<BAND>(blockIdx.x, nbm, nbn, tm, tn);
  const uint32_t lane = threadIdx.x & 63u, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t wm = wid >> 2, wn = wid & 3u;
  const uint32_t rowBytes = K * F::kElem;           // at most kBigMaxRow
  const uint32_t nhalf = (rowBytes + kStage / 2 - 1) / (kStage / 2), nst = (nhalf + 1) / 2;
  const uint32_t last = (rowBytes - (nst - 1) * kStage) / 16 - 1;      // last chunk of the last stage
  const bool cut_last = rowBytes % (kStage / 2) != 0;
  const uint32_t m0 = min(tm * kBig, M - kBig), n0 = min(tn * kBig, N - kBig);
  const uint8_t* baseA = A + (uint64_t)m0 * rowBytes;
  const uint8_t* baseB = B + (uint64_t)n0 * rowBytes;
  // load h of a wave and operand fills rows 8 (wid + 8 h) .. + 7: one lane
  // offset serves all, the rest of the address is uniform
  const uint32_t lrow = 8u * wid + (lane >> 3);
  uint32_t vo = lrow * rowBytes + lane_chunk(lane, lrow) * 16u;
  const uint64_t step = 64ull * rowBytes;
  auto issue = [&](uint32_t st, int h0, int h1) {
    uint8_t* slot = smem + (st & 1u) * kBigSlot;
    const uint64_t k = (uint64_t)st * kStage;
    if (h0 == 0 && st + 1 == nst && last < 7) {   // chunks past the end of a short last stage repeat its last one
      const uint32_t t = threadIdx.x & 63u, c = lane_chunk(t, 8u * wid + (t >> 3));
      vo -= (c - min(c, last)) * 16u;
    }
#pragma unroll
    for (int h = h0; h < h1; ++h) {
      const uint32_t blk = (wid + 8u * h) * 1024u;
      load16_lds(baseA + k + h * step + vo, slot + blk);
      load16_lds(baseB + k + h * step + vo, slot + kBigOp + blk);
    }
  };
  // touched per stage: 32 rows of A (its panel is shared by the 8 tiles of a
  // band's row that run together) and 64 of B (shared by 4), waves 0-3 and 4-7
  const uint32_t far_n = wid < 4 ? 8u : 16u;
  const uint32_t far_row = (wid < 4 ? (tn & 7u) * 32u : (tm & 3u) * 64u) + (wid & 3u) * far_n;
  const uint8_t* far = (wid < 4 ? baseA : baseB) + (uint64_t)far_row * rowBytes;
  const uint32_t far_o = min(lane, far_n - 1) * rowBytes;
  auto touch = [&](uint32_t st) {
    if constexpr (FAR)
      __builtin_amdgcn_global_load_lds(far + min(st * kStage, rowBytes - 16u) + far_o, smem + 2 * kBigSlot, 4, 0, 0);
  };
  f32x16 acc[IN][JN];
#pragma unroll
  for (int i = 0; i < IN; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
  const uint32_t frow = lane & 31u, fk = F::off(lane);
  typename F::T fa[NS][IN], fb[NS][JN];
  auto read_half = [&](uint32_t st, uint32_t half) {
    const uint8_t* slot = smem + (st & 1u) * kBigSlot;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const uint32_t kb = half * (kStage / 2) + fk + s * F::kStep;
#pragma unroll
      for (int i = 0; i < IN; ++i) fa[s][i] = F::ld(slot, wm * 128 + i * 32 + frow, kb);
#pragma unroll
      for (int j = 0; j < JN; ++j) fb[s][j] = F::ld(slot + kBigOp, wn * 64 + j * 32 + frow, kb);
    }
  };
  // zero what a short last stage holds past the end of the rows
  auto clear_tail = [&](uint32_t st) {
    uint8_t* slot = smem + (st & 1u) * kBigSlot;
    int z;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));     // made here: a constant would hold four registers through the loop
    for (uint32_t row = threadIdx.x & (kBig - 1); row < 2 * kBig; row += kBig)     // rows of A, then of B
      for (uint32_t c = last + 1; c < 8; ++c)
        *reinterpret_cast<i32x4*>(slot + stage_at(row, c * 16u)) = i32x4{z, z, z, z};
    __builtin_amdgcn_s_waitcnt(kWaitLds);
  };
  auto multiply = [&] {
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int i = 0; i < IN; ++i)
#pragma unroll
        for (int j = 0; j < JN; ++j) acc[i][j] = F::mma(fa[s][i], fb[s][j], acc[i][j], lane);
  };
  // The phases are fenced: nothing moves across a barrier.
  auto phase_end = [] {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr int kTouch = FAR ? 1 : 0;     // the newest load of a stage is its touch, which nobody waits for
  const bool late = wm != 0;
  issue(0, 0, 4);
  if constexpr (FAR)
#pragma unroll
    for (uint32_t q = 2; q <= kAhead; ++q) touch(q);
  __builtin_amdgcn_s_waitcnt(wait_vm(FAR ? kAhead - 1 : 0));
  phase_end();
  if (late) phase_end();
  for (uint32_t st = 0; st < nst; ++st) {
    const bool more = st + 1 < nst;
    if (cut_last && !more) {      // one phase more: the earlier row clears, the later one waits
      if (!late) clear_tail(st);
      phase_end();
    }
    read_half(st, 0);
    if (more) issue(st + 1, 0, 2);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(kWaitLds);
    phase_end();
    __builtin_amdgcn_s_setprio(1);
    if (more) issue(st + 1, 2, 4);
    touch(st + kAhead + 1);
    multiply();
    __builtin_amdgcn_s_setprio(0);
    phase_end();
    if (2 * st + 1 < nhalf) {
      read_half(st, 1);
      __builtin_amdgcn_sched_barrier(0);
      // stage st + 1 must have landed, for both rows, before the earlier row reads it
      if (late) __builtin_amdgcn_s_waitcnt(wait_vm(kTouch));
      __builtin_amdgcn_s_waitcnt(kWaitLds);
      phase_end();
      __builtin_amdgcn_s_setprio(1);
      multiply();
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      if (!late) __builtin_amdgcn_s_waitcnt(wait_vm(kTouch));
      phase_end();
    }
  }
  if (!late) phase_end();
  __builtin_amdgcn_s_waitcnt(wait_vm(0));   // no load may reach LDS after this work-group's end
  const uint32_t row0 = m0 + wm * 128 + 4u * (lane >> 5), col0 = n0 + wn * 64 + (lane & 31u);
  const bool whole = m0 == tm * kBig && n0 == tn * kBig;
#pragma unroll
  for (int i = 0; i < IN; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t row = row0 + i * 32 + 8u * (v / 4) + (v % 4), col = col0 + j * 32;
        if (whole || (row >= tm * kBig && col >= tn * kBig)) C[(uint64_t)row * N + col] = acc[i][j][v] * scale;
      }
}

// Large-tile kernel of FP32: 256 x 256 tiles, eight waves (2 x 4, each 128 x
// 64; two per SIMD) and a ring of four K-stages of 64 bytes per row.  Rows are
// stored unpadded; the 16-byte chunk c of row r sits at chunk
// c ^ ((r >> 2) & 3).  Two fragment buffers of one k-step (two k) each: a
// k-step's block is its first MFMA, then the next k-step's reads, then its
// other MFMAs, fenced in that order, so that the reads have seven MFMAs to
// land (4 % over the compiler's order).  One bare barrier per stage: each wave
// first waits for its own loads of the stage, so after the barrier the whole
// stage is in LDS; the reads of a stage's last k-step are waited for after the
// next stage's barrier, so that barrier frees the slot of the stage before:
// stage t + 2 is issued at the barrier of stage t into the slot of t - 2.
// A short last stage ends after its last whole chunk (two k-steps); its loads
// past the row's end repeat the row's last chunk.
// What bounds it: the matrix core, at 86 % of its rate (4096^3 1010 us, 136
// TF; tiles of 128 x 128 take 1130 us).  Its MFMAs are four times as long as
// BF16's for the same bytes, so neither loads nor barriers weigh enough for the
// alternating groups of the other types (1237 us).
// Four slots of 32 KiB: 128 KiB of the CU's 160 KiB, leaving 31 KiB (LDS is
// given out in pieces of 1280 bytes) for a co-resident stressor work-group.
constexpr int kRingStages = 4;
constexpr int kDStage = 64;                         // K bytes per stage per row
constexpr int kDOperand = kBig * kDStage;           // one operand, one stage (16 KiB)
constexpr int kDSlot = 2 * kDOperand;               // A and B of one stage
static_assert(kRingStages * kDSlot <= 128 * 1024, "the ring must leave LDS for a co-resident work-group");

__device__ __forceinline__ float ring_ld(const uint8_t* p, uint32_t row, uint32_t byte) {
  return *reinterpret_cast<const float*>(p + row * kDStage + ((((byte >> 4) ^ (row >> 2)) & 3u) << 4) + (byte & 15u));
}

// BAND: tile rows per band of the tile order (tile_of).
template <uint32_t BAND>
__global__ void __launch_bounds__(512, 1) gemm256f_kernel(const uint8_t* __restrict__ A,
                                                          const uint8_t* __restrict__ B,
                                                          float* __restrict__ C, uint32_t M,
                                                          uint32_t N, uint32_t K, float scale) {
  constexpr int WN = 4, JN = 2;           // 8 waves: 2 x 4, each 128 x 64
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const uint32_t nbm = (M + kBig - 1) / kBig, nbn = (N + kBig - 1) / kBig;
  uint32_t tm, tn;
  tile_of<BAND>(blockIdx.x, nbm, nbn, tm, tn);
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
  const uint32_t wm = wid / WN, wn = wid % WN;
  const uint32_t rowBytes = K * 4;                  // at most kBigMaxRow
  const uint32_t nstages = (rowBytes + kDStage - 1) / kDStage;
  // Wave w fills 1 KiB blocks w and w + 8 of each operand (16 blocks of 16
  // rows); lane l lands on row 16 q + l / 4, physical chunk l % 4.
  uint32_t lrow[2], lchunk[2];
  const uint8_t* srcA[2];
  const uint8_t* srcB[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t q = wid + 8u * h;
    lrow[h] = 16u * q + (lane >> 2);
    lchunk[h] = ((lane & 3u) ^ (lrow[h] >> 2)) & 3u;    // logical chunk for this slot
    const uint32_t gm = min(tm * kBig + lrow[h], M - 1), gn = min(tn * kBig + lrow[h], N - 1);
    srcA[h] = A + (uint64_t)gm * rowBytes;
    srcB[h] = B + (uint64_t)gn * rowBytes;
  }
  auto issue = [&](uint32_t st) {
    uint8_t* slot = smem + (st % kRingStages) * kDSlot;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t blk = (wid + 8u * h) * 1024u;
      const uint32_t k = min(st * kDStage + lchunk[h] * 16u, rowBytes - 16u);    // past a row's end: not multiplied
      load16_lds(srcA[h] + k, slot + blk);
      load16_lds(srcB[h] + k, slot + kDOperand + blk);
    }
  };
  f32x16 acc[4][JN];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
  const uint32_t frow = lane & 31u, fk = (lane >> 5) * 4u;
  constexpr int NS = kDStage / 8;         // k-steps per stage
  // Wait until this wave's loads of stage t are done (at most one later stage
  // of 4 instructions may be pending), then a bare barrier: a fence would also
  // wait for the later stage's loads.
  auto wait_stage = [&](uint32_t t) {
    if (t + 1 < nstages) __builtin_amdgcn_s_waitcnt(wait_vm(4));
    else __builtin_amdgcn_s_waitcnt(wait_vm(0));
    __builtin_amdgcn_s_barrier();
  };
  for (uint32_t st = 0; st < 2 && st < nstages; ++st) issue(st);
  float fa[2][4], fb[2][JN];
  auto read_ks = [&](uint32_t t, int s, auto buf) {
    constexpr int b = decltype(buf)::value;
    const uint8_t* slot = smem + (t % kRingStages) * kDSlot;
    const uint32_t kb = fk + s * 8;
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[b][i] = ring_ld(slot, wm * 128 + i * 32 + frow, kb);
#pragma unroll
    for (int j = 0; j < JN; ++j) fb[b][j] = ring_ld(slot + kDOperand, wn * 64 + j * 32 + frow, kb);
  };
  // MFMAs of one k-step: the first, or the others
  auto mma_part = [&](auto buf, bool first) {
    constexpr int b = decltype(buf)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < JN; ++j)
        if ((i == 0 && j == 0) == first)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[b][i], fb[b][j], acc[i][j], 0, 0, 0);
  };
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  using B0 = std::integral_constant<int, 0>;
  using B1 = std::integral_constant<int, 1>;
  // stage t, its first k-step already in buffer 0; with `more`, the last
  // k-step's MFMAs overlap the next stage's barrier and first reads
  auto stage_body = [&](uint32_t t, bool more) {
#pragma unroll
    for (int s = 0; s < NS; s += 2) {
      if (!more && t * kDStage + s * 8 >= rowBytes) break;     // a short last stage: whole chunks, two k-steps each
      mma_part(B0{}, true);
      fence();
      read_ks(t, s + 1, B1{});
      fence();
      mma_part(B0{}, false);
      fence();
      mma_part(B1{}, true);
      fence();
      if (s + 2 < NS) {
        read_ks(t, s + 2, B0{});
      } else if (more) {
        wait_stage(t + 1);
        if (t + 3 < nstages) issue(t + 3);
        read_ks(t + 1, 0, B0{});
      }
      fence();
      mma_part(B1{}, false);
      fence();
    }
  };
  wait_stage(0);
  if (2 < nstages) issue(2);
  read_ks(0, 0, B0{});
  // no branch around the reads in the steady state, so that each MFMA block
  // waits only for its own buffer's reads
  uint32_t st = 0;
  for (; st + 1 < nstages; ++st) stage_body(st, true);
  stage_body(st, false);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < JN; ++j) {
      const uint32_t col = tn * kBig + wn * 64 + j * 32 + (lane & 31u);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t row = tm * kBig + wm * 128 + i * 32 + 8u * (v / 4) + 4u * (lane >> 5) + (v % 4);
        if (row < M && col < N) C[(uint64_t)row * N + col] = acc[i][j][v] * scale;
      }
    }
}

// GEMV: wave w handles rows w, w + W, ...; lane l reads 16-byte chunks
// l, l + 64, ... of the row (8 BF16 each), four chunks in flight, and keeps
// an FP32 running sum; the 64 partial sums are combined by a fixed butterfly.
// Memory bounds it: 8192 x 8192 23.5 us (5.7 TB/s), 16384 x 16384 84 us (6.4
// TB/s); eight chunks in flight, two or four rows a wave and loads that run
// ahead over rows are no faster (25-32 and 84-109 us where this form took 25
// and 86).
// NTL: non-temporal weight loads, for matrices that no cache can hold.
__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ float dot8(uint4 w, uint4 x, float acc) {
  acc = __builtin_fmaf(bf16lo(w.x), bf16lo(x.x), acc);
  acc = __builtin_fmaf(bf16hi(w.x), bf16hi(x.x), acc);
  acc = __builtin_fmaf(bf16lo(w.y), bf16lo(x.y), acc);
  acc = __builtin_fmaf(bf16hi(w.y), bf16hi(x.y), acc);
  acc = __builtin_fmaf(bf16lo(w.z), bf16lo(x.z), acc);
  acc = __builtin_fmaf(bf16hi(w.z), bf16hi(x.z), acc);
  acc = __builtin_fmaf(bf16lo(w.w), bf16lo(x.w), acc);
  acc = __builtin_fmaf(bf16hi(w.w), bf16hi(x.w), acc);
  return acc;
}

template <bool NTL>
__device__ __forceinline__ uint4 ld_chunk(const uint4* p) {
  if constexpr (NTL) {
    const i32x4 v = __builtin_nontemporal_load(reinterpret_cast<const i32x4*>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
  } else {
    return *p;
  }
}

template <bool NTL>
__global__ void __launch_bounds__(256) gemv_bf16_kernel(const uint16_t* __restrict__ W,
                                                        const uint16_t* __restrict__ x,
                                                        float* __restrict__ y, uint64_t n,
                                                        uint64_t k) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint64_t gw = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const uint64_t nw = ((uint64_t)gridDim.x * blockDim.x) >> 6;
  const uint64_t nch = k / 8;   // 16-byte chunks per row
  const uint4* x4 = reinterpret_cast<const uint4*>(x);
  for (uint64_t r = gw; r < n; r += nw) {
    const uint4* w4 = reinterpret_cast<const uint4*>(W + r * k);
    float acc = 0.0f;
    uint64_t c = lane;
    for (; c + 192 < nch; c += 256) {
      uint4 w[4], xv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = ld_chunk<NTL>(w4 + c + 64 * u);
#pragma unroll
      for (int u = 0; u < 4; ++u) xv[u] = x4[c + 64 * u];
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = dot8(w[u], xv[u], acc);
    }
    for (; c < nch; c += 64) acc = dot8(ld_chunk<NTL>(w4 + c), x4[c], acc);
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane == 0) y[r] = acc;
  }
}

}  // namespace

namespace {

// Tile choice.  A work-group per CU at a time costs about u per tile and K,
// and v once (its share of launch, first loads and last stores); tiles that
// fill the last round of CUs poorly cost the whole round.  Rows that are not
// whole 128-byte lines straddle two per stage, which costs the smaller tiles,
// with more bytes per product, the most: a second set.  Fitted in microseconds
// per K = 1024 to all four tilings on 81 square shapes from 512 to 8192:
//   BF16, whole lines  64 x 64: 512^3 4.6, 1024^3 7.4, 1536^3 16; 128 x 64:
//              2048^3 26 (64 x 64 28, 128 x 128 27); 128 x 128: 2560^3 41 (59,
//              54; 256 x 256 59), 4352^3 188 (204); 256 x 256: 5120^3 248
//              (290), 8192^3 880 (1060);
//   BF16, others  128 x 128: 2488^3 46 (85, 76; 256 x 256 71); 256 x 256:
//              8184^3 930 (2940, 1760, 1250);
//   FP32       64 x 64: 1024^3 29 (128 x 64 48), 3072^3 534 (573, 643; 256 x
//              256 785), 4004^3 990 with 256 x 256 (1067 with 128 x 128).
// FP8 follows BF16 at half the time.
// 256 x 256 is offered only where its tiles are a CU's worth each or more (sides
// from about 3841): its 128 KiB of LDS shut out co-runners that hold more than
// 31 KiB.  Below that line it would take BF16 3328^3 from 99 to 74 us and FP32
// 3712^3 from 910 to 894, but a victim beside the LDS stressor on every CU, 2.5
// to 4 times its time with smaller tiles, would wait for the stressor to end.
// Two work-groups of 128 x 128 share a CU, so BF16's and FP8's fourth round
// rides on the third (3456^3, three rounds, 104 us; 3520^3, four, 103).
struct TileCost {
  float u, v;
};
constexpr uint32_t kTileM[4] = {64, 128, 128, 256}, kTileN[4] = {64, 64, 128, 256};
constexpr uint32_t kCus = 256;
constexpr TileCost kCost16[2][4] = {{{2.95f, 2.0f}, {4.4f, 3.6f}, {8.2f, 4.6f}, {26.2f, 1.0f}},
                                    {{5.2f, 0.5f}, {7.1f, 4.0f}, {10.4f, 2.5f}, {29.5f, 0.5f}}};
constexpr TileCost kCost32[2][4] = {{{18.7f, 9.0f}, {37.5f, 4.0f}, {70.0f, 8.0f}, {250.0f, 2.0f}},
                                    {{19.4f, 8.0f}, {36.0f, 10.0f}, {66.0f, 10.0f}, {250.0f, 2.0f}}};
// Row bytes for which the offsets of a lane fit 32 bits (63 rows and 112 bytes
// at the most): 256 tiles of longer rows do not fit the device.  4096^2 with
// BF16 rows of 2^23 + 128 bytes take 128 ms, 264 with tiles of 128 x 128.
constexpr uint64_t kBigMaxRow = 1u << 26;

int tile_choice(bool f32, bool whole_lines, uint64_t m, uint64_t n, bool big_ok) {
  const TileCost* t = (f32 ? kCost32 : kCost16)[whole_lines ? 0 : 1];
  int best = 0;
  float cost = 0.0f;
  bool prev_over = false;   // the best so far is beyond what a launch can hold
  for (int i = 0; i < (big_ok ? 4 : 3); ++i) {
    const uint64_t tiles = ((m + kTileM[i] - 1) / kTileM[i]) * ((n + kTileN[i] - 1) / kTileN[i]);
    float rounds = (float)((tiles + kCus - 1) / kCus);
    if (i == 2 && !f32 && rounds == 4.0f) rounds = 3.25f;
    const float c = rounds * t[i].u + t[i].v;
    const bool fits = tiles * (i < 3 ? 256 : 512) < (1ull << 32);   // a launch's work-items are 32 bits
    if (i == 0 || (fits && c <= cost) || prev_over) {
      best = i;
      cost = c;
      prev_over = !fits;
    }
  }
  return best;
}

struct GemmCall {
  const uint8_t *a, *b;
  float* c;
  uint32_t m, n, k;
  float scale;
  hipStream_t s;
  hipEvent_t e0, e1;
};

template <typename Kernel>
hipError_t launch_tiles(Kernel kernel, uint32_t tm, uint32_t tn, uint32_t threads, uint32_t lds, const GemmCall& g) {
  const uint64_t nb = (uint64_t)((g.m + tm - 1) / tm) * ((g.n + tn - 1) / tn);
  return xlaunch(kernel, dim3((uint32_t)nb), dim3(threads), lds, g.s, g.e0, g.e1, g.a, g.b, g.c, g.m, g.n, g.k, g.scale);
}

template <int DT>
hipError_t launch_gemm_dt(const GemmCall& g) {
  const uint64_t row = (uint64_t)g.k * Op<DT>::kElem;
  constexpr bool f32 = DT == CI_DT_F32;
  const uint64_t big_tiles = (uint64_t)((g.m + kBig - 1) / kBig) * ((g.n + kBig - 1) / kBig);
  const bool big_ok = g.m >= kBig && g.n >= kBig && big_tiles >= kCus && row <= kBigMaxRow;
  switch (tile_choice(f32, row % kStage == 0, g.m, g.n, big_ok)) {
    case 0: {
      // Four slots instead of two where a BF16 tile has its CU to itself and its
      // short stages leave a load little to hide behind: 1024^3 9.1 us, 9.8 with
      // two, 512^3 6.0 and 6.2; FP32 the same with both, FP8 0.2 us apart.  Tiles
      // of 128 x 128 would gain more (BF16 2048^3 15 %, FP32 5 %), but their 128
      // KiB shut out co-runners that hold 64 KiB of LDS, as the LDS stressor does.
      if constexpr (DT == CI_DT_BF16) {
        if ((uint64_t)((g.m + 63) / 64) * ((g.n + 63) / 64) <= kCus)
          return launch_tiles(gemm_tile_kernel<DT, 64, 64, 4>, 64, 64, 256, 4 * 128 * kStage, g);
      }
      return launch_tiles(gemm_tile_kernel<DT, 64, 64, 2>, 64, 64, 256, 2 * 128 * kStage, g);
    }
    case 1: return launch_tiles(gemm_tile_kernel<DT, 128, 64, 2>, 128, 64, 256, 2 * 192 * kStage, g);
    case 2: return launch_tiles(gemm_tile_kernel<DT, 128, 128, 2>, 128, 128, 256, 2 * 256 * kStage, g);
    default: break;
  }
  // Every tile at once or not: bands of 8 tile rows when it is (BF16 4096^3
  // 114 us against 116 with FAR), of 4 with FAR otherwise (8192^3 881 against
  // 926 us, FP8 412 against 465).
  const bool far = big_tiles > kCus;
  if constexpr (f32) {
    const uint32_t lds = kRingStages * kDSlot;
    return far ? launch_tiles(gemm256f_kernel<4>, kBig, kBig, 512, lds, g)
               : launch_tiles(gemm256f_kernel<8>, kBig, kBig, 512, lds, g);
  } else {
    return far ? launch_tiles(gemm256d_kernel<DT, true>, kBig, kBig, 512, kBigLds, g)
               : launch_tiles(gemm256d_kernel<DT, false>, kBig, kBig, 512, kBigLds, g);
  }
}

}  // namespace

hipError_t launch_gemm(int dtype, const void* a, const void* b, float* c, uint64_t m, uint64_t n,
                       uint64_t k, float scale, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  const GemmCall g{(const uint8_t*)a, (const uint8_t*)b, c, (uint32_t)m, (uint32_t)n, (uint32_t)k, scale, s, e0, e1};
  switch (dtype) {
    case CI_DT_F32: return launch_gemm_dt<CI_DT_F32>(g);
    case CI_DT_BF16: return launch_gemm_dt<CI_DT_BF16>(g);
    case CI_DT_FP8E4M3: return launch_gemm_dt<CI_DT_FP8E4M3>(g);
    default: return hipErrorInvalidValue;
  }
}

// Non-temporal weight loads when the copies that the launches rotate over are
// more than the 256 MiB Infinity Cache: 3 x 8192^2 23.5 us against 25.9, one
// 16384^2 84 against 93; below it the cache serves: 3 x 5888^2 14.4 us against
// 16.5, one 8192^2 21.5 against 22.0.
hipError_t launch_gemv_bf16(const uint16_t* w, const uint16_t* x, float* y, uint64_t n, uint64_t k,
                            uint64_t copies, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  uint64_t g = (n + 3) / 4;   // one wave per row, four waves per work-group
  if (g > 8192) g = 8192;
  if (g == 0) g = 1;
  const bool cached = (double)copies * (double)n * (double)k * 2.0 <= 256.0 * 1048576.0;
  return xlaunch(cached ? gemv_bf16_kernel<false> : gemv_bf16_kernel<true>, dim3((uint32_t)g), dim3(256), 0, s, e0, e1, w, x, y, n, k);
}

namespace {

template <int DT>
hipError_t preload_gemm() {
  hipError_t e[5] = {preload(gemm_tile_kernel<DT, 64, 64, 2>), preload(gemm_tile_kernel<DT, 128, 64, 2>),
                     preload(gemm_tile_kernel<DT, 128, 128, 2>), hipSuccess, hipSuccess};
  if constexpr (DT == CI_DT_F32) {
    e[3] = preload(gemm256f_kernel<4>);
    e[4] = preload(gemm256f_kernel<8>);
  } else {
    e[3] = preload(gemm256d_kernel<DT, true>);
    e[4] = preload(gemm256d_kernel<DT, false>);
  }
  for (const hipError_t x : e)
    if (x != hipSuccess) return x;
  return hipSuccess;
}

}  // namespace

hipError_t preload_dense() {
  for (const hipError_t e : {preload_gemm<CI_DT_F32>(), preload_gemm<CI_DT_BF16>(), preload_gemm<CI_DT_FP8E4M3>(),
                             preload(gemm_tile_kernel<CI_DT_BF16, 64, 64, 4>), preload(gemv_bf16_kernel<false>),
                             preload(gemv_bf16_kernel<true>)})
    if (e != hipSuccess) return e;
  return hipSuccess;
}

}  // namespace ci
