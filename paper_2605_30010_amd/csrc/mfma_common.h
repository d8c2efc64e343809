// Device helpers shared by the matrix kernels: MFMA and conversion wrappers, direct global -> LDS
// loads, explicit waits, the GELU of the fused epilogues.  Device code only.
//
// MFMA shapes, per 64-lane wavefront:
// v_mfma_f32_32x32x16_bf16, with g = lane / 32 and r = lane % 32:
//   operand "A" (32 x 16): lane holds row r,    k = 8g .. 8g+7   (8 bf16 = one 16-byte vector)
//   operand "B" (16 x 32): lane holds column r, k = 8g .. 8g+7
//   accumulator (32 x 32): lane holds column r, rows (i / 4) * 8 + 4g + (i % 4), i = 0..15
// v_mfma_f32_16x16x32_bf16, with g = lane / 16 and r = lane % 16:
//   operand "A" (16 x 32): lane holds row r,    k = 8g .. 8g+7
//   operand "B" (32 x 16): lane holds column r, k = 8g .. 8g+7
//   accumulator (16 x 16): lane holds column r, rows 4g + i, i = 0..3
// The second one takes less power per multiply-add: in a loop of MFMAs alone on all compute units the board's cap
// holds 1.83 GHz with the first shape (1.87 PFLOP/s) and 2.06 GHz with the second (2.06 PFLOP/s).
#pragma once
#include "et_common.h"

namespace et {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  bf16x2 v;
  v.x = (__bf16)lo;
  v.y = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ f32x16 mfma32(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ f32x4 mfma16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ float gelu_tanh_f(float u) {
  // 0.5 u (1 + tanh(y)) = u / (1 + exp(-2y)),  y = sqrt(2/pi) (u + 0.044715 u^3)
  // exp(-2y) = exp2(u (c1 + c3 u^2)) with the factor -2 log2(e) sqrt(2/pi) folded into c1, c3;
  // hardware exp2 and reciprocal (1 ulp) are ample for a result that is rounded to bf16.
  const float c1 = -2.0f * 1.4426950408889634f * 0.7978845608028654f;
  const float c3 = c1 * 0.044715f;
  const float t = u * fmaf(u * u, c3, c1);
  return u * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(t));
}

// LDS transpose read: every lane of a 16-lane group supplies the address of four consecutive 16-bit
// elements; lane j of the group receives element j % 4 of the lanes j / 4, 4 + j / 4, 8 + j / 4 and
// 12 + j / 4 (layout checked on the device).  With lane s of a group pointing at row s / 4, columns
// 4 (s % 4) .. + 3 of a row-major matrix, lane j gets column j of four consecutive rows.
__device__ __forceinline__ uint2 lds_read_tr16(const uint16_t *p) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
  return __builtin_bit_cast(uint2, v);
#else
  return make_uint2(0u, 0u);
#endif
}

// Direct global -> LDS loads (no staging registers): one wavefront moves 64 x 4 or 64 x 16 bytes to consecutive LDS.  The
// immediate offset moves the global AND the LDS address and has to be a literal.
#define ET_LDS_DMA4(gptr, lptr)                                                              \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gptr),   \
                                   (__attribute__((address_space(3))) void *)(lptr), 4, 0, 0)

#define ET_LDS_DMA16_OFF(gptr, lptr, imm)                                                    \
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)(gptr),   \
                                   (__attribute__((address_space(3))) void *)(lptr), 16, (imm), 0)

// The same load, unknown to the compiler: it has every LDS transpose read behind a direct load that it knows wait for that
// load (as if the read could overlap it), which undoes a prefetch.  The caller's own waits (wait_vmcnt) cover it; the
// compiler's waits for its own loads stay right, since an operation that it does not count only makes them longer.  M0 is
// written behind its back: not beside the macros above in one kernel.  (s_nop: the wait states that the base needs if a
// vector instruction has just written it, and M0, which the compiler sees to for loads that it knows.)
__device__ __forceinline__ void lds_dma16_untracked(const uint16_t *base, uint32_t byte_off, uint16_t *dst) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t to = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t *)dst;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %2"
               ::"v"(byte_off), "s"(__builtin_amdgcn_readfirstlane(to)), "s"(base) : "memory");
#endif
}

// The i-th of a group of four loads that share one LDS base (M0 cannot be rewritten before the
// previous load has read it): `src` has to be lowered by (i % 4) KiB by the caller.
__device__ __forceinline__ void lds_dma16_of4(const char *src, uint16_t *dst, int i) {
  switch (i & 3) {
    case 0: ET_LDS_DMA16_OFF(src, dst, 0); break;
    case 1: ET_LDS_DMA16_OFF(src, dst, 1024); break;
    case 2: ET_LDS_DMA16_OFF(src, dst, 2048); break;
    default: ET_LDS_DMA16_OFF(src, dst, 3072); break;
  }
}

// Sum over the eight lanes of an aligned group, in every one of them (lane ^ 1, lane ^ 2, mirror of the eight).
template <int CTRL>
__device__ __forceinline__ float dpp_plus(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float sum_of_8_lanes(float v) { return dpp_plus<0x141>(dpp_plus<0x4E>(dpp_plus<0xB1>(v))); }

// (mean, sum of squares about it) of the 64 bf16 values that eight lanes hold, eight each.  A mean that has left float32
// is given as 0, so that means can be subtracted; the sum of squares is infinite then, or NaN where a value is not finite.
__device__ __forceinline__ float2 piece_moments(u32x4 v) {
  float x[8], s = 0.f, q = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    x[2 * e] = bf16lo_to_f32(v[e]);
    x[2 * e + 1] = bf16hi_to_f32(v[e]);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) s += x[e];
  const float mean = sum_of_8_lanes(s) * (1.0f / 64.0f);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float d = x[e] - mean;
    q = fmaf(d, d, q);
  }
  return make_float2(fabsf(mean) < INFINITY ? mean : 0.f, sum_of_8_lanes(q));
}

// Combines the pieces of one row, in ascending order.  The pieces' means are taken relative to the first one's: nothing
// cancels when the row's mean is many standard deviations.  Where a square or a piece's sum leaves float32 (values beyond
// 1e18) the variance is infinite and the scale 0, as in rowstats_kernel; a NaN or an infinity in the row gives NaN.
struct PieceSum {
  float ref = 0.f, s1 = 0.f, s2 = 0.f;                   // ref: the first piece's mean, set by the caller
  __device__ __forceinline__ void add(float2 p) {
    const float d = p.x - ref;
    s1 += d;
    s2 = fmaf(64.f * d, d, s2 + p.y);
  }
  __device__ __forceinline__ float scale(int pieces, float eps) const {       // 1 / sqrt(var + eps)
    const float n = (float)pieces, m2 = s2 == INFINITY ? s2 : fmaf(-64.f * s1, s1 / n, s2);
    return 1.0f / sqrtf((m2 < 0.f ? 0.f : m2) / (64.f * n) + eps);             // (NaN stays NaN)
  }
};

// What a GEMM kernel needs for its first loads, as arguments of their own in front of the GemmArgs: the command processor
// hands the first 14 words of scalar arguments over in registers (-amdgpu-kernarg-preload-count; structures stay in memory),
// so that no load waits for the argument block, which is in no cache yet.  Kernels whose arguments are plain scalars have them
// so by themselves; narrow_blocks_kernel, with a structure alone, loads its own.  Measured, us per call: one frame through 27 blocks 1819 -> 1779, eight frames 3595 -> 3511.
#define ET_GEMM_FIRST                                                                                                       \
  const uint16_t *first_A, const uint16_t *first_W, int first_lda, int first_K, int first_M, int tiles_m, int tiles_n,      \
      int first_stats_ld, const float2 *first_stats, const float *first_scale
#define ET_GEMM_GIVE_FIRST(g) (g).A, (g).W, (g).lda, (g).K, (g).M, tiles_m, tiles_n, (g).stats_ld, (g).stats_in, (g).row_scale
#define ET_GEMM_TAKE_FIRST(g)                                                                                               \
  (g).A = first_A, (g).W = first_W, (g).lda = first_lda, (g).K = first_K, (g).M = first_M, (g).stats_ld = first_stats_ld,   \
  (g).stats_in = first_stats, (g).row_scale = first_scale

// Row scale of one row per lane: 1 / sqrt(var + eps) from the statistics of the row's pieces, or g.row_scale, or 1
// (fma(1, acc, bias) == acc + bias exactly).  fetch() issues the loads, value() combines them, so that a kernel
// can put its first operand loads between.
template <int BATCH>                                    // pieces in flight
struct RowScale {
  float2 v[BATCH];
  uint32_t off;                                         // byte offset of the row in a piece
  __device__ __forceinline__ float2 piece(const GemmArgs &g, int c) const {
    return *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(g.stats_in + (size_t)c * g.stats_ld) + off);
  }
  __device__ __forceinline__ void fetch(const GemmArgs &g, int m) {
    const int mc = m < g.M ? m : g.M - 1;
    off = (uint32_t)mc * (uint32_t)sizeof(float2);
    if (g.stats_in) {
#pragma unroll
      for (int u = 0; u < BATCH; ++u) v[u] = piece(g, u < g.K / 64 ? u : g.K / 64 - 1);   // (no branch; past the end unused)
    } else {
      v[0].x = g.row_scale ? g.row_scale[mc] : 1.0f;
    }
  }
  __device__ __forceinline__ float value(const GemmArgs &g) {
    if (!g.stats_in) return v[0].x;
    const int pieces = g.K / 64;
    PieceSum sum;
    sum.ref = v[0].x;
    for (int c = 0;;) {
#pragma unroll
      for (int u = 0; u < BATCH; ++u)
        if (c + u < pieces) sum.add(v[u]);
      c += BATCH;
      if (c >= pieces) break;
#pragma unroll
      for (int u = 0; u < BATCH; ++u)
        if (c + u < pieces) v[u] = piece(g, c + u);
    }
    return sum.scale(pieces, g.ln_eps);
  }
};

// Stores 16 bytes of a result, past the XCD's L2 (write-through) if `through` (the same for the whole launch).  Results left
// dirty there are written back when the kernel ends, in front of the next one: 22 MB of them cost 2.2 us; a store past
// it is waited for longer at a wavefront's end.  For whole 128-byte segments only (the memory side merges nothing).
// (s_nop: the store reads its data after it has issued, so two wait states have to pass before a vector instruction may
// overwrite them; the compiler sees to that for stores that it knows.)
__device__ __forceinline__ void store16(uint16_t *p, u32x4 v, bool through) {
  if (through) asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(v) : "memory");
  else *reinterpret_cast<u32x4 *>(p) = v;
}

// Order of a quarter of a k-tile (gemm_stream_kernel, gemm_duo_kernel): one MFMA in front of each LDS read, then the direct loads GAP MFMAs apart, the rest behind them.
template <int READS, int LOADS, int MFMAS>
__device__ __forceinline__ void mfma_between() {
  constexpr int GAP = LOADS ? ((MFMAS - READS) / (LOADS + 1) > 0 ? (MFMAS - READS) / (LOADS + 1) : 1) : 0;
#pragma unroll
  for (int i = 0; i < READS; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
  }
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, GAP, 0);
    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
  }
  if constexpr (MFMAS - READS - LOADS * GAP > 0) __builtin_amdgcn_sched_group_barrier(0x008, MFMAS - READS - LOADS * GAP, 0);
}

// Waits until at most N of this wavefront's vector-memory operations are outstanding.
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N <= 63, "vmcnt is a 6-bit counter");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Waits until all of its vector-memory and LDS operations are done.  In front of a barrier behind which LDS is refilled: that
// a read's result is used in front of the barrier in the source does not keep its wait there.
__device__ __forceinline__ void wait_all() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

}  // namespace et
