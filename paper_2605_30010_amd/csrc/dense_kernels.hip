// Dense encoder kernels for gfx950: LayerNorm, patch extraction, the bf16 MFMA GEMM with fused
// epilogues (bias | bias + GELU-tanh | bias + residual) and per-frame multi-head attention.
//
// The MFMA operand layouts are described in mfma_common.h.
#include <atomic>
#include <type_traits>

#include "gemm_choice.h"
#include "gemm_small.h"

namespace et {

namespace {

// ---------------------------------------------------------------------------------------
// LayerNorm: one wavefront per row, row held in registers, fp32 statistics (two passes over
// the registers: mean, then biased variance about the mean).
// ---------------------------------------------------------------------------------------
constexpr int kLnRows = 4;

template <int NV>
__global__ __launch_bounds__(kLnRows * kWave) void layernorm_kernel(
    const uint16_t *__restrict__ x, const float *__restrict__ gamma, const float *__restrict__ beta,
    float eps, int rows, int D, uint16_t *__restrict__ y) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kLnRows + (threadIdx.x >> 6);
  if (row >= rows) return;
  uint4 raw[NV];
  Row<NV> r;
  load_row<NV>(x + (size_t)row * D, D, lane, raw);
  unpack_row<NV>(raw, r);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NV * 8; ++i) s += r.v[i];           // pad lanes hold zeros
  const float mean = wave_sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if ((j * kWave + lane) * 8 < D) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float d = r.v[j * 8 + e] - mean;
        q = fmaf(d, d, q);
      }
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)D + eps);
  uint16_t *out = y + (size_t)row * D;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int c = (j * kWave + lane) * 8;
    if (c < D) {
      const float4 g0 = *reinterpret_cast<const float4 *>(gamma + c);
      const float4 g1 = *reinterpret_cast<const float4 *>(gamma + c + 4);
      const float4 b0 = *reinterpret_cast<const float4 *>(beta + c);
      const float4 b1 = *reinterpret_cast<const float4 *>(beta + c + 4);
      const float *v = &r.v[j * 8];
      uint4 o;
      o.x = cvt_pk_bf16((v[0] - mean) * rstd * g0.x + b0.x, (v[1] - mean) * rstd * g0.y + b0.y);
      o.y = cvt_pk_bf16((v[2] - mean) * rstd * g0.z + b0.z, (v[3] - mean) * rstd * g0.w + b0.w);
      o.z = cvt_pk_bf16((v[4] - mean) * rstd * g1.x + b1.x, (v[5] - mean) * rstd * g1.y + b1.y);
      o.w = cvt_pk_bf16((v[6] - mean) * rstd * g1.z + b1.z, (v[7] - mean) * rstd * g1.w + b1.w);
      *reinterpret_cast<uint4 *>(out + c) = o;
    }
  }
}

// The row statistics alone: 1 / sqrt(var + eps) per row (same arithmetic as layernorm_kernel), for
// GEMMs that have the LayerNorm folded into their weights and epilogue.
template <int NV>
__global__ __launch_bounds__(kLnRows * kWave) void rowstats_kernel(const uint16_t *__restrict__ x, float eps, int rows,
                                                                   int D, float *__restrict__ rstd_out) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kLnRows + (threadIdx.x >> 6);
  if (row >= rows) return;
  uint4 raw[NV];
  Row<NV> r;
  load_row<NV>(x + (size_t)row * D, D, lane, raw);
  unpack_row<NV>(raw, r);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NV * 8; ++i) s += r.v[i];           // pad lanes hold zeros
  const float mean = wave_sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if ((j * kWave + lane) * 8 < D) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float d = r.v[j * 8 + e] - mean;
        q = fmaf(d, d, q);
      }
    }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)D + eps);
  if (lane == 0) rstd_out[row] = rstd;
}

// The statistics of rows that no GEMM has written (after a merge or selection), by pieces of 64 columns as the
// residual epilogues leave them and with the same arithmetic: stats[p * ld + row] = (mean, sum of squares about it).
template <int NV>
__global__ __launch_bounds__(kLnRows * kWave) void piece_stats_kernel(const uint16_t *__restrict__ x, int rows, int D, int ld,
                                                                      float2 *__restrict__ stats) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kLnRows + (threadIdx.x >> 6);
  if (row >= rows) return;
  uint4 raw[NV];
  load_row<NV>(x + (size_t)row * D, D, lane, raw);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const float2 st = piece_moments(u32x4{raw[j].x, raw[j].y, raw[j].z, raw[j].w});
    const int piece = j * 8 + (lane >> 3);
    if ((lane & 7) == 0 && piece < D / 64) stats[(size_t)piece * ld + row] = st;
  }
}

// The row scales that RowScale combines from those pieces, in the same order.
template <int NV>
__global__ __launch_bounds__(kLnRows * kWave) void piece_scale_kernel(const uint16_t *__restrict__ x, float eps, int rows, int D,
                                                                      float *__restrict__ rstd_out) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kLnRows + (threadIdx.x >> 6);
  if (row >= rows) return;
  uint4 raw[NV];
  load_row<NV>(x + (size_t)row * D, D, lane, raw);
  PieceSum sum;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const float2 st = piece_moments(u32x4{raw[j].x, raw[j].y, raw[j].z, raw[j].w});
    if (j == 0) sum.ref = __shfl(st.x, 0);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float2 p = make_float2(__shfl(st.x, u * 8), __shfl(st.y, u * 8));
      if (j * 8 + u < D / 64) sum.add(p);
    }
  }
  if (lane == 0) rstd_out[row] = sum.scale(D / 64, eps);
}

// ---------------------------------------------------------------------------------------
// Patch extraction: frames fp32 [T, C, H, W] -> bf16 [T * L, Kpad]; row (t, gy, gx), column
// (c, py, px) flattened; columns >= C*P*P are zero.  One thread writes 8 columns (16 bytes).
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void im2col_kernel(const float *__restrict__ frames, int T, int C, int H,
                                                     int W, int P, int GX, int L, int Kreal, int Kpad,
                                                     uint16_t *__restrict__ out) {
  const int chunks = Kpad / 8;
  const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (size_t)T * L * chunks) return;
  const int ch = (int)(idx % chunks);
  const size_t row = idx / chunks;
  const int l = (int)(row % L), t = (int)(row / L);
  const int gy = l / GX, gx = l % GX;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int kk = ch * 8 + e;
    float val = 0.f;
    if (kk < Kreal) {
      const int c = kk / (P * P), rem = kk % (P * P);
      const int py = rem / P, px = rem % P;
      val = frames[(((size_t)t * C + c) * H + (gy * P + py)) * W + (gx * P + px)];
    }
    v[e] = val;
  }
  uint4 o;
  o.x = cvt_pk_bf16(v[0], v[1]); o.y = cvt_pk_bf16(v[2], v[3]);
  o.z = cvt_pk_bf16(v[4], v[5]); o.w = cvt_pk_bf16(v[6], v[7]);
  *reinterpret_cast<uint4 *>(out + row * Kpad + ch * 8) = o;
}

// The same through LDS, one workgroup per (frame, row of patches): the C * P image rows of the stripe
// are read as whole rows (float4, coalesced), kept in LDS as bf16, and the stripe's GX output rows are
// written as whole 16-byte chunks - both sides of the copy are contiguous, where the kernel above reads
// P-pixel runs.  Needs W % 4 == 0, 16-byte aligned frames and C * P * W * 2 bytes of LDS.
__global__ __launch_bounds__(1024) void im2col_stripe_kernel(const float *__restrict__ frames, int C, int H, int W, int P,
                                                            int GX, int GY, int Kreal, int Kpad,
                                                            uint16_t *__restrict__ out) {
  extern __shared__ __align__(16) uint16_t stripe[];           // [C * P][W] bf16
  const int t = blockIdx.x / GY, gy = blockIdx.x % GY;
  const int w4 = W / 4, n4 = C * P * w4;
  for (int i = threadIdx.x; i < n4; i += blockDim.x) {
    const int r = i / w4, x4 = i % w4, c = r / P, py = r % P;
    const float4 v = *reinterpret_cast<const float4 *>(frames + (((size_t)t * C + c) * H + (gy * P + py)) * W + x4 * 4);
    uint2 o;
    o.x = cvt_pk_bf16(v.x, v.y);
    o.y = cvt_pk_bf16(v.z, v.w);
    *reinterpret_cast<uint2 *>(stripe + r * W + x4 * 4) = o;
  }
  __syncthreads();
  const int chunks = Kpad / 8;
  uint16_t *orow = out + ((size_t)t * GY + gy) * GX * Kpad;
  for (int i = threadIdx.x; i < GX * chunks; i += blockDim.x) {
    const int gx = i / chunks, ch = i % chunks;
    uint16_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int kk = ch * 8 + e;
      uint16_t val = 0;
      if (kk < Kreal) {
        const int r = kk / P, px = kk % P;                       // r = c * P + py
        val = stripe[r * W + gx * P + px];
      }
      v[e] = val;
    }
    uint4 o;
    o.x = v[0] | ((uint32_t)v[1] << 16); o.y = v[2] | ((uint32_t)v[3] << 16);
    o.z = v[4] | ((uint32_t)v[5] << 16); o.w = v[6] | ((uint32_t)v[7] << 16);
    *reinterpret_cast<uint4 *>(orow + (size_t)gx * Kpad + ch * 8) = o;
  }
}

// ---------------------------------------------------------------------------------------
// GEMM  C[m, n] = sum_k A[m, k] W[n, k] + bias[n]  (+ epilogue), bf16 operands, fp32 accumulate.
// Both operands are k-contiguous, so both feed MFMA as 16-byte vectors straight from LDS.
// The weight tile is MFMA operand "A" (rows = n) and the activation tile operand "B"
// (columns = m): each lane then owns 4 consecutive n of one output row m per accumulator
// quad, which packs to an 8-byte bf16 piece.
// ---------------------------------------------------------------------------------------
// acc[a][b] is the 16 x 16 tile at columns n_base + 16 a (MFMA rows) and rows m_base + 16 b (MFMA columns): the lane owns
// output row m = .. + lane % 16 and the four consecutive columns n = .. + 4 (lane / 16) + (0..3).
// Epilogue for wavefront tiles 64 columns wide, staged through a private 4 KiB LDS slice per
// wavefront so that every global access is a full 128-byte row segment (8 lanes x 16 bytes)
// instead of 8-byte pieces scattered over 16 rows.  Per 32-row block: (residual only) the
// residual block is fetched coalesced into the slice; each lane then adds bias (+GELU | +its
// residual values read back from the slice) in fp32, rounds once to bf16 and writes its 4-column
// pieces to the slice; finally the slice is read row-wise and stored.  16-byte slots of a row are
// XOR-swizzled by (row >> 1) & 7.  LDS operations of one wavefront execute in order, so the phases
// need no barrier.
// Bias and row scales of the tile come to the slice before (see fetch_constants in the kernel).  STATS: the residual epilogue
// leaves the rows' statistics; for the others the row scales are written by a wavefront that has combined them.
constexpr int kBiasInSlice = 512;            // floats
template <int EPI, bool STATS, int MS, int NS>
__device__ __forceinline__ void gemm_epilogue_lds(f32x4 (&acc)[NS][MS], const GemmArgs &g, int m_base,
                                                  int n_base, int lane, uint16_t *slice) {
  static_assert(NS == 4 && MS % 2 == 0, "the staged epilogue handles 64-column wavefront tiles in blocks of 32 rows");
  const int r16 = lane & 15, g4 = lane >> 4;
  const int prow = lane >> 3, pch = lane & 7;                 // row-wise phase: 8 rows x 8 chunks per pass
  // Bias and row scales lie in the slice (kBiasInSlice floats from its start, and at its start); read before it takes results.
  const float *in_slice = reinterpret_cast<const float *>(slice);
  float rsv[MS];                                              // row scales of this lane's rows
#pragma unroll
  for (int b = 0; b < MS; ++b)                                // (no LayerNorm in front of a residual GEMM; fma(1, acc, bias) == acc + bias)
    rsv[b] = EPI != EPI_BIAS_RES && (STATS || g.row_scale) ? in_slice[b * 16 + r16] : 1.0f;
  const int n_lane = n_base + pch * 8;
  const bool n_ok = n_lane < g.n_store;                       // n_store is a multiple of 8 on this path
  float4 bi[NS];
#pragma unroll
  for (int a = 0; a < NS; ++a) bi[a] = *reinterpret_cast<const float4 *>(in_slice + kBiasInSlice + a * 16 + g4 * 4);
  asm volatile("" ::: "memory");
  u32x4 rv[4];
  auto fetch_res = [&](int b) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int m = m_base + b * 32 + j * 8 + prow;
      rv[j] = u32x4{0u, 0u, 0u, 0u};
      if (m < g.M && n_ok)
        rv[j] = *reinterpret_cast<const u32x4 *>(g.res + (size_t)(m % g.res_mod) * g.ldr + n_lane);
    }
  };
  if (EPI == EPI_BIAS_RES) fetch_res(0);
#pragma unroll
  for (int b = 0; b < MS / 2; ++b) {
    const int mb = m_base + b * 32;
    if (mb >= g.M) break;                                     // wave-uniform: whole block past the last row
    if (EPI == EPI_BIAS_RES) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = j * 8 + prow;
        *reinterpret_cast<u32x4 *>(slice + row * 64 + ((pch ^ ((row >> 1) & 7)) * 8)) = rv[j];
      }
      if (b + 1 < MS / 2) fetch_res(b + 1);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int row = h * 16 + r16;
      const float rs = rsv[b * 2 + h];
#pragma unroll
      for (int a = 0; a < NS; ++a) {
        const f32x4 av = acc[a][b * 2 + h];
        float v0 = fmaf(rs, av[0], bi[a].x), v1 = fmaf(rs, av[1], bi[a].y);
        float v2 = fmaf(rs, av[2], bi[a].z), v3 = fmaf(rs, av[3], bi[a].w);
        if (EPI == EPI_BIAS_GELU) {
          v0 = gelu_tanh_f(v0); v1 = gelu_tanh_f(v1); v2 = gelu_tanh_f(v2); v3 = gelu_tanh_f(v3);
        }
        uint2 *cell = reinterpret_cast<uint2 *>(slice + row * 64 + (((a * 2 + (g4 >> 1)) ^ ((row >> 1) & 7)) * 8) + (g4 & 1) * 4);
        if (EPI == EPI_BIAS_RES) {
          const uint2 rr = *cell;
          v0 += bf16lo_to_f32(rr.x); v1 += bf16hi_to_f32(rr.x);
          v2 += bf16lo_to_f32(rr.y); v3 += bf16hi_to_f32(rr.y);
        }
        uint2 o;
        o.x = cvt_pk_bf16(v0, v1);
        o.y = cvt_pk_bf16(v2, v3);
        *cell = o;
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = j * 8 + prow, m = mb + row;
      const u32x4 v = *reinterpret_cast<const u32x4 *>(slice + row * 64 + ((pch ^ ((row >> 1) & 7)) * 8));
      if (m < g.M && n_ok) store16(g.C + (size_t)m * g.ldc + n_lane, v, g.through);
      if (EPI == EPI_BIAS_RES && STATS) {                     // (n_store is a multiple of 64 then)
        const float2 st = piece_moments(v);
        if (pch == 0 && m < g.M && n_ok) g.stats_out[(size_t)(n_base >> 6) * g.stats_ld + m] = st;
        asm volatile("" ::: "memory");                          // (one piece at a time: the accumulators leave no registers)
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// Operands are brought in by direct global -> LDS loads (global_load_lds_dwordx4): no staging
// registers and no LDS write instructions.  One wavefront load moves 64 x 16 bytes to 1 KiB of
// consecutive LDS, i.e. 8 tile rows of 64 bf16; lane L lands at row L / 8, slot L % 8 and fetches
// the global 16-byte chunk (slot ^ swz(row)), an XOR swizzle that spreads the MFMA fragment reads
// (same k-chunk, consecutive rows) over the banks.  Waits are explicit (vmcnt) because the loads are
// asynchronous to the wavefront: a piece is complete once this wavefront's loads have landed AND the
// workgroup barrier after that wait has been passed.
//
// The kernel is persistent: one workgroup per compute-unit slot walks over its output tiles
// t = b, b + G, b + 2G, ... and treats their k-tiles as ONE stream through two LDS stages, so the
// loads of the next output tile are already in flight (and its first fragments already in
// registers) while the finished tile's epilogue runs.  That removes the per-tile prologue latency
// and the workgroup relaunch between tiles.
//
// A wavefront goes over its 64-deep k-tile in quarters: (upper half of its rows, k 0-31), (upper, 32-63), (lower, 0-31),
// (lower, 32-63); the fragments of a quarter are read from LDS under the MFMAs of the one before.  The weight fragments of
// both k-steps stay in registers for the whole k-tile, so after the first quarter the weights and the upper rows of the
// stage have been read by everyone and are refilled with the k-tile after the next, two loads per wavefront and quarter
// among the MFMAs: a compute unit takes 58 bytes of operands per clock, 1100 clocks per k-tile, and a burst of loads
// blocks whoever issues it.  The lower rows follow in the next k-tile's first quarter.  Two barriers per k-tile, a few
// MFMAs before a quarter's end, so that these are at hand behind them.
// Bound: the board's power cap where all compute units work; in launches of one round the fixed parts (launch 1-4 us,
// first loads 3 us, epilogue 3-7 us) and the barriers (120 of 600 clocks per quarter pair).  Measured against
// 32x32x16 MFMAs with whole stages refilled in one burst, us per launch (one box): 23328 rows, QKV 184.8 -> 176.8, fc1
// 238.7 -> 227.4, out-projection 73.5 -> 69.3, fc2 231.4 -> 215.3; 3276 rows, QKV 35.5 -> 33.5, fc1 39.6 -> 38.3.
// ---------------------------------------------------------------------------------------
// STATS, residual epilogue: leaves g.stats_out.  STATS, others: the row scales come from g.stats_in: one wavefront per
// 64 rows combines them (a row per lane) before the k-loop and leaves them, with the last k-tile, in the epilogue slices
// of the wavefronts that need them.  Only for launches of one tile per workgroup: further tiles' scales cost more than a launch that computes them
// (fetched beside the k-loop, 46656 rows: QKV 292 -> 324 us, fc1 445 -> 475).
template <int BM, int BN, int WAVES_M, int WAVES_N, int MINB, int EPI, bool STATS>
__global__ __launch_bounds__(WAVES_M *WAVES_N * 64, MINB) void gemm_stream_kernel(ET_GEMM_FIRST, GemmArgs g) {
  ET_GEMM_TAKE_FIRST(g);
  constexpr int BK = 64, STAGES = 2;
  constexpr int NW = WAVES_M * WAVES_N;
  constexpr int WTM = BM / WAVES_M, WTN = BN / WAVES_N;
  constexpr int MS = WTM / 16, NS = WTN / 16, MH = MS / 2;
  constexpr int STAGE_ELEMS = (BM + BN) * BK;
  constexpr int WL = BN / 8 / NW, AL = BM / 16 / NW;                 // 1 KiB loads per wavefront: of the weight tile, of either half of the activation tile
  constexpr int LOADS = WL + 2 * AL;
  static_assert(WTN == 64, "the staged epilogue handles 64-column wavefront tiles");
  static_assert(WL == 4 && AL == 2 && (WTM / 2) % (8 * AL) == 0, "loads are issued two per quarter, in groups that share one M0 value");
  extern __shared__ __align__(16) uint16_t lds[];

  const int n_tiles = tiles_m * tiles_n;
  const int G = gridDim.x;
  const int n_my = (n_tiles - (int)blockIdx.x + G - 1) / G;       // >= 1: the grid never exceeds n_tiles
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: LDS destinations of the loads stay scalar
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int r16 = lane & 15, g4 = lane >> 4;
  const int lrow = lane >> 3, lslot = lane & 7;

  // j-th tile of this workgroup.  Tiles are ordered in bands of 8 tile rows, inside a band in
  // column blocks of 4 tile columns, inside a block row-major; within a round of G tiles each XCD
  // (blockIdx % 8) takes a contiguous run of that order.  The ~32 tiles an XCD works on at once
  // then form an 8 x 4 patch that shares 8 activation and 4 weight k-slices through its L2
  // (12 slice fetches per 32 tiles instead of 19 for a 2 x 17 strip).
  auto tile_of = [&](int j, int &m0, int &n0) {
    const int base = j * G;
    const int cnt = (n_tiles - base < G) ? (n_tiles - base) : G;
    const int per = cnt / 8, rem = cnt % 8, xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
    const int t = base + xcd * per + (xcd < rem ? xcd : rem) + slot;
    const int band = t / (8 * tiles_n), r = t - band * 8 * tiles_n;
    const int hb = (tiles_m - band * 8 < 8) ? (tiles_m - band * 8) : 8;
    const int cb = r / (hb * 4), r2 = r - cb * hb * 4;
    const int wcb = (tiles_n - cb * 4 < 4) ? (tiles_n - cb * 4) : 4;
    m0 = (band * 8 + r2 / wcb) * BM;
    n0 = (cb * 4 + r2 % wcb) * BN;
  };

  // Source of this lane for each of the wavefront's loads: a wave-uniform tile origin (scalar
  // registers) plus a 32-bit per-lane byte offset, so that each load is issued with a scalar base
  // and needs no vector address arithmetic.  Only the activation offsets depend on the tile (rows
  // past M are clamped to the last row).
  // The instruction's immediate offset moves the global AND the LDS address, and the LDS base sits
  // in M0, which cannot be rewritten before the previous load has read it: loads are therefore
  // issued in groups of four that share one M0 value and step through LDS by immediates of 1 KiB,
  // with the lane offsets lowered by the same amount (kOffBias keeps them non-negative; the tile
  // origins are lowered by it).
  constexpr uint32_t kOffBias = 4096;
  const char *a_base = nullptr, *w_base = nullptr;
  uint32_t a_off[2 * AL], w_off[WL];
  // activation rows of this wavefront's loads: half h (rows h * WTM / 2 .. of every wavefront tile), i-th load
  constexpr int WPH = WTM / 2 / (8 * AL);                         // wavefronts that load one wavefront row's half
  const int a_row0 = (wave / WPH) * WTM + (wave % WPH) * 8 * AL;  // half 0; half 1: + WTM / 2
#pragma unroll
  for (int i = 0; i < WL; ++i) {
    const int row = (wave * WL + i) * 8 + lrow;
    w_off[i] = (uint32_t)(((size_t)row * g.K + ((lslot ^ ((row >> 1) & 7)) * 8)) * 2) + kOffBias - i * 1024;
  }
  auto set_load_tile = [&](int j) {
    int m0, n0;
    tile_of(j, m0, n0);
    a_base = reinterpret_cast<const char *>(g.A + (size_t)m0 * g.lda) - kOffBias;
    w_base = reinterpret_cast<const char *>(g.W + (size_t)n0 * g.K) - kOffBias;
    asm volatile("" : "+s"(a_base), "+s"(w_base));      // (keeps the bias out of the loads' address expressions)
#pragma unroll
    for (int i = 0; i < 2 * AL; ++i) {
      const int row = a_row0 + (i / AL) * (WTM / 2) + (i % AL) * 8 + lrow;
      const int rc = (m0 + row < g.M) ? row : g.M - 1 - m0;       // m0 < M always
      a_off[i] = (uint32_t)(((size_t)rc * g.lda + ((lslot ^ ((row >> 1) & 7)) * 8)) * 2) + kOffBias - (i % AL) * 1024;
    }
  };
  const int kt_n = g.K / BK;
  int load_tile = 0, load_kt = 0;                   // next k-tile of the stream to be fetched
  auto load_w = [&](int stage, int i0, int i1) {
    const char *b = w_base + (size_t)load_kt * (BK * 2);
    uint16_t *dst = lds + stage * STAGE_ELEMS + BM * BK + wave * WL * 512;
#pragma unroll
    for (int i = i0; i < i1; ++i) {
      asm volatile("" : "+v"(w_off[i]));
      lds_dma16_of4(b + w_off[i], dst, i);
    }
  };
  auto load_a = [&](int stage, int h) {
    const char *b = a_base + (size_t)load_kt * (BK * 2);
    uint16_t *dst = lds + stage * STAGE_ELEMS + (a_row0 + h * (WTM / 2)) * 64;
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      asm volatile("" : "+v"(a_off[h * AL + i]));
      lds_dma16_of4(b + a_off[h * AL + i], dst, i);
    }
  };
  auto advance = [&]() {
    if (++load_kt == kt_n) {                        // past the stream's end the last k-tile is re-read (unused)
      if (load_tile + 1 < n_my) {
        load_kt = 0;
        set_load_tile(++load_tile);
      } else {
        load_kt = kt_n - 1;
      }
    }
  };

  const int fx = (r16 >> 1) & 7;
  int a_addr[2], w_addr[2];                         // element offsets of this lane's fragments, by k-step
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int ko = ((4 * ks + g4) ^ fx) * 8;
    a_addr[ks] = (wm * WTM + r16) * 64 + ko;
    w_addr[ks] = BM * BK + (wn * WTN + r16) * 64 + ko;
  }

  f32x4 acc[NS][MS];
  auto clear_acc = [&]() {
#pragma unroll
    for (int a = 0; a < NS; ++a)
#pragma unroll
      for (int b = 0; b < MS; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  constexpr bool LNF = STATS && EPI != EPI_BIAS_RES;
  static_assert(!LNF || (WTM % 64 == 0 && BM / 64 <= NW), "one wavefront per 64 rows");
  float my_scale = 1.0f;
  RowScale<18> scale;
  if (LNF && wave < BM / 64) {
    int m0, n0;
    tile_of(0, m0, n0);
    scale.fetch(g, m0 + wave * 64 + lane);
  }
  // The bias of the wavefront's 64 columns and the scales of its rows, by direct loads into its epilogue slice while the
  // tile's k-loop runs: fetched in the epilogue they cost its wavefronts a trip to memory, behind all operand loads in flight.
  uint16_t *const slices = lds + STAGES * STAGE_ELEMS;
  uint16_t *const slice = slices + wave * (32 * 64);
  auto fetch_constants = [&](int j) {
    int m0, n0;
    tile_of(j, m0, n0);
    ET_LDS_DMA4(g.bias + n0 + wn * WTN + lane, slice + kBiasInSlice * 2);
    if (EPI != EPI_BIAS_RES && !STATS && g.row_scale) {
#pragma unroll
      for (int i = 0; i < WTM / 64; ++i) {
        const int m = m0 + wm * WTM + i * 64 + lane;
        ET_LDS_DMA4(g.row_scale + (m < g.M ? m : g.M - 1), slice + i * 128);
      }
    }
  };
  fetch_constants(0);
  set_load_tile(0);
#pragma unroll
  for (int st = 0; st < 2; ++st) {
    load_w(st, 0, WL);
    load_a(st, 0);
    if (st == 0) {
      load_a(st, 1);
      advance();
    }
  }

  u32x4 fw[2][NS], fa[2][MH];
  auto read_w = [&](int stage, int ks) {
    const uint16_t *p = lds + stage * STAGE_ELEMS + w_addr[ks];
#pragma unroll
    for (int a = 0; a < NS; ++a) fw[ks][a] = *reinterpret_cast<const u32x4 *>(p + a * 16 * 64);
  };
  auto read_a = [&](int buf, int stage, int h, int ks) {
    const uint16_t *p = lds + stage * STAGE_ELEMS + a_addr[ks] + h * (WTM / 2) * 64;
#pragma unroll
    for (int b = 0; b < MH; ++b) fa[buf][b] = *reinterpret_cast<const u32x4 *>(p + b * 16 * 64);
  };
  auto mfma_rows = [&](int buf, int h, int ks, int b0, int b1) {
#pragma unroll
    for (int b = b0; b < b1; ++b)
#pragma unroll
      for (int a = 0; a < NS; ++a) acc[a][h * MH + b] = mfma16(fw[ks][a], fa[buf][b], acc[a][h * MH + b]);
  };
  constexpr int N_ST = (MS / 2) * 4;                 // global stores per wavefront in the staged epilogue
  int relax = 0;
  auto landed = [&](auto newest) {                              // all but the newest LOADS loads of this wavefront, then everyone's
    if (relax > 0) {
      wait_vmcnt<decltype(newest)::value + N_ST>();
      --relax;
    } else {
      wait_vmcnt<decltype(newest)::value>();
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  wait_vmcnt<LOADS>();
  __builtin_amdgcn_sched_barrier(0);
  if (LNF && wave < BM / 64) {
    my_scale = scale.value(g);
    asm volatile("" : "+v"(my_scale));
  }
  clear_acc();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_w(0, 0);
  read_a(0, 0, 0, 0);

  int stage = 0, kt = 0, my_tile = 0;
  const int units = n_my * kt_n;
  for (int u = 0; u < units; ++u) {
    read_a(1, stage, 0, 1);
    read_w(stage, 1);
    load_a(stage ^ 1, 1);
    mfma_rows(0, 0, 0, 0, MH - 1);
    mfma_between<MH + NS, AL, NS * (MH - 1)>();
    __builtin_amdgcn_sched_barrier(0);
    advance();
    landed(std::integral_constant<int, LOADS>());
    __builtin_amdgcn_sched_barrier(0);
    mfma_rows(0, 0, 0, MH - 1, MH);
    read_a(0, stage, 1, 0);
    load_w(stage, 0, 2);
    mfma_rows(1, 0, 1, 0, MH);
    __builtin_amdgcn_sched_group_barrier(0x008, NS, 0);
    mfma_between<MH, 2, NS * MH>();
    __builtin_amdgcn_sched_barrier(0);
    read_a(1, stage, 1, 1);
    load_w(stage, 2, 4);
    mfma_rows(0, 1, 0, 0, MH - 1);
    mfma_between<MH, 2, NS * (MH - 1)>();
    __builtin_amdgcn_sched_barrier(0);
    if (LNF && wave < BM / 64 && kt + 1 == kt_n) {
      uint16_t *dst = slices + (wave * 64 / WTM) * WAVES_N * (32 * 64);
#pragma unroll
      for (int w = 0; w < WAVES_N; ++w) reinterpret_cast<float *>(dst + w * (32 * 64))[(wave * 64) % WTM + lane] = my_scale;
    }
    landed(std::integral_constant<int, LOADS - AL>());
    __builtin_amdgcn_sched_barrier(0);
    mfma_rows(0, 1, 0, MH - 1, MH);
    read_w(stage ^ 1, 0);
    read_a(0, stage ^ 1, 0, 0);
    load_a(stage, 0);
    mfma_rows(1, 1, 1, 0, MH);
    __builtin_amdgcn_sched_group_barrier(0x008, NS, 0);
    mfma_between<MH + NS, AL, NS * MH>();
    __builtin_amdgcn_sched_barrier(0);
    stage ^= 1;
    if (++kt == kt_n) {                             // an output tile is complete
      int m0, n0;
      tile_of(my_tile, m0, n0);
      wait_vmcnt<LOADS>();                          // (the tile's bias and row scales are older than its last k-tile's loads)
      gemm_epilogue_lds<EPI, STATS, MS, NS>(acc, g, m0 + wm * WTM, n0 + wn * WTN, lane, slice);
      if (m0 + BM <= g.M && n0 + BN <= g.n_store) relax = 2;
      if (++my_tile == n_my) break;
      fetch_constants(my_tile);
      kt = 0;
      clear_acc();
    }
  }
  wait_vmcnt<0>();                     // drain the padding loads before the workgroup's LDS is released
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int MINB>
int launch_gemm_stream_cfg(const GemmArgs &g, hipStream_t s) {
  constexpr int NT = WAVES_M * WAVES_N * 64;
  // two k-tile stages plus one 4 KiB epilogue slice per wavefront
  constexpr size_t lds_bytes = (size_t)2 * (BM + BN) * 64 * sizeof(uint16_t) +
                               (size_t)WAVES_M * WAVES_N * 32 * 64 * sizeof(uint16_t);
  static_assert(lds_bytes <= 160 * 1024, "LDS budget");
  const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.n_store + BN - 1) / BN;
  const int n_tiles = tiles_m * tiles_n;
  const int slots = device_cus() * MINB;
  const dim3 grid(n_tiles < slots ? n_tiles : slots), block(NT);
  if (g.stats_in && n_tiles > slots) {
    set_error("gemm: row statistics by pieces need one tile per workgroup (%d tiles, %d slots)", n_tiles, slots);
    return ET_ERR_INVALID_ARG;
  }
#define ET_GEMM_LAUNCH(E, STATS)                                                                  \
  {                                                                                              \
    constexpr auto kern = gemm_stream_kernel<BM, BN, WAVES_M, WAVES_N, MINB, E, STATS>;          \
    if (int rc = allow_lds<kern>(lds_bytes)) return rc;                                          \
    hipLaunchKernelGGL(kern, grid, block, lds_bytes, s, ET_GEMM_GIVE_FIRST(g), g);                    \
  }
  switch (g.epilogue) {
    case EPI_BIAS:
      if (g.stats_in) ET_GEMM_LAUNCH(EPI_BIAS, true) else ET_GEMM_LAUNCH(EPI_BIAS, false)
      break;
    case EPI_BIAS_GELU:
      if (g.stats_in) ET_GEMM_LAUNCH(EPI_BIAS_GELU, true) else ET_GEMM_LAUNCH(EPI_BIAS_GELU, false)
      break;
    case EPI_BIAS_RES:
      if (g.stats_out) ET_GEMM_LAUNCH(EPI_BIAS_RES, true) else ET_GEMM_LAUNCH(EPI_BIAS_RES, false)
      break;
    default: set_error("unknown epilogue %d", g.epilogue); return ET_ERR_INVALID_ARG;
  }
#undef ET_GEMM_LAUNCH
  ET_LAUNCH_CHECK();
  return ET_OK;
}

// ---------------------------------------------------------------------------------------
// Attention: softmax(Q K^T / sqrt(hd)) V inside one frame, one head per workgroup column.
// Flash-style streaming over 64-key tiles.  Everything is computed transposed: S^T = K Q^T puts the
// query on the accumulator's lane axis, so the exponentials' reference and the running sum are per-lane
// scalars, and the exponentiated accumulator registers are, without any data movement, MFMA operand "B" of
// O^T = V^T P^T.  The reference is the maximum of the first keys and stays (quick_block); where that does not
// serve, a second pass takes a running maximum and rescales (tile).
// ---------------------------------------------------------------------------------------
constexpr int kAttWaves = 4;
constexpr int kAttBQ = kAttWaves * 32;
constexpr int kAttBKV = 64;

// Workgroups go to the 8 XCDs round-robin by index.  A one-dimensional grid whose order puts
// workgroups that share data next to each other is therefore remapped first: XCD x takes the x-th
// contiguous run of the order (a bijection of [0, total)), and neighbours share an L2.
__device__ __forceinline__ int xcd_contiguous_index(int total) {
  const int per = total / 8, rem = total % 8, xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  return xcd * per + (xcd < rem ? xcd : rem) + slot;
}

// ---------------------------------------------------------------------------------------
// attention_dma_kernel: K and V tiles are brought in by direct global -> LDS loads, one tile ahead, two
// LDS stages, one barrier per 64-key tile; up to three workgroups share a compute unit (168 registers).  Frames have
// equal length n (frame f = rows f n ..) or, with `cu` given, the row ranges cu[f] .. cu[f+1]
// (decoupled selection: the grid is sized for the longest frame and workgroups past a frame's
// end leave at once).
// Both tiles sit in LDS as they are in memory, rows back to back (row stride = head_dim * 2
// bytes; 144 bytes for head_dim 72 spreads 16-byte reads of consecutive rows over all banks).
// MFMA wants the contraction index (the key) contiguous per lane for the P V product, i.e. V^T:
// its fragments are taken from the row-major tile with the LDS transpose read of gfx950
// (ds_read_b64_tr_b16), two per fragment, so V is never transposed in memory.  When head_dim is
// not a multiple of 16 the last contraction chunk of a K row runs 16 bytes into the next row;
// those slots carry the reference maximum (see below).  O^T row blocks past head_dim read
// whatever follows a V row; that only reaches accumulator rows >= head_dim, which are never
// stored (MFMA output rows are independent).
// No maximum is kept over the tiles (quick_block); a workgroup whose first reference did not last walks its tiles again
// with an online maximum (tile).  Bound on many frames: the matrix and the vector unit are busy 40 % of the cycles each, 38 %
// of the former at the same time, with the board near its power cap (back to back 1370 of 1400 W at 1.9 GHz); on few
// the chain of a wavefront.  Measured against an online maximum in every tile (heads of 72, us per launch):
// 64 x 729 320 -> 285, 32 x 729 140 -> 125, 23 x 729 99 -> 89, 8 x 729 36.9 -> 34.1, 9 x 364 16.7 -> 15.0; heads of 64,
// 16 x 196 12.3 -> 11.7.  (Two query blocks per wavefront spill: 170.)  The second pass, per workgroup that has a query with a
// later logit some 41 (2^60 in weight) above its first 32, or anything that is not finite; launches in which every workgroup
// has one, against a single pass with an online maximum: 64 x 729 288 -> 481, 8 x 729 36 -> 58, 2 x 729 16.9 -> 26.0, 1 x 729 12.8 ->
// 18.5, heads of 64, 16 x 196, 12.8 -> 18.8; up to that jump nothing (by 30: 36.4 -> 33.1, 12.7 -> 11.4).
// ---------------------------------------------------------------------------------------
// A flag in LDS that any wavefront of the workgroup can raise: cleared at the kernel's start by one thread, whose write
// is waited for in front of the first barrier; read behind a later one.
__device__ __forceinline__ void clear_flag(int &flag) {
  if (threadIdx.x == 0) flag = 0;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}
__device__ __forceinline__ void raise_flag(int &flag, bool mine) {
  if (__any(mine) && (threadIdx.x & 63) == 0) flag = 1;
}

// What one wavefront keeps and does for its 32 queries, shared by the kernels below.
template <int HD>
struct AttentionRows {
  static constexpr int NC = (HD + 15) / 16;
  static constexpr int NDB = (HD + 31) / 32;
  // When head_dim is not a multiple of 32 the last O^T row block has spare rows: the V^T fragment
  // of row head_dim is overridden with ones, and accumulator row head_dim of O^T is the softmax
  // denominator (the sum of the bf16-rounded probabilities, exactly what the numerator used), for free.
  static constexpr bool SUM_BY_MFMA = (HD % 32) != 0;
  // When head_dim is not a multiple of 16 the Q K^T contraction has spare slots: slot head_dim of
  // every K row is read as 1 and slot head_dim of a query holds minus its reference maximum, so
  // the MFMA delivers s - m_ref.  Otherwise the subtraction is a vector instruction per logit.
  static constexpr bool REF_IN_PAD = (HD % 16) != 0;
  // Reference maximum of the online softmax, per query, in exponent units.  It is moved only when
  // the maximum of a 32-key block exceeds it by more than kLazy (probabilities then stay below
  // 2^kLazy, harmless in fp32 / bf16), so the rescaling of O^T is rare after the first block.  With
  // REF_IN_PAD it is kept bf16-representable (any reference serves as long as numerator and
  // denominator use the same one).
  static constexpr float kLazy = 8.0f;
  u32x4 qf[NC];
  f32x16 o_acc[NDB];
  float m_ref, l_run;
  // Lanes whose query has met no logit above minus infinity yet (wave-uniform mask; all of them before the first keys).
  // Their reference stays 0 and their accumulators 0; the first such logit sets the reference without a rescaling.
  unsigned long long fresh;

  // Q is scaled by log2(e) / sqrt(head_dim) once, here, and rounded back to bf16: the logits leave
  // the MFMA already in the exponent's units.
  __device__ __forceinline__ void start(const uint16_t *qbase, int q_first, int n, int ld, float scale_log2, int r32, int grp) {
    const int q = q_first + r32;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int d = c * 16 + grp * 8;
      u32x4 raw = u32x4{0u, 0u, 0u, 0u};
      if (q < n && d < HD) raw = *reinterpret_cast<const u32x4 *>(qbase + (size_t)q * ld + d);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        qf[c][e] = cvt_pk_bf16(bf16lo_to_f32(raw[e]) * scale_log2, bf16hi_to_f32(raw[e]) * scale_log2);
    }
#pragma unroll
    for (int b = 0; b < NDB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) o_acc[b][i] = 0.f;
    m_ref = l_run = 0.f;
    fresh = ~0ull;
  }

  // Order of the keys: row r of a 32-row MFMA tile is key key_of_row(r) of its 32.  The keys of the four rows that half a
  // wavefront's transpose read touches, rows 8 h + 4 g + (0..3) of a 16-row chunk, lie KEY_STEP apart, so that their
  // 64-byte pieces fall into different banks (row strides of 36, 40, 48 and 16 banks; 64 and 128 take no order).
  static constexpr int KEY_STEP = HD == 72 ? 4 : HD == 80 ? 2 : 1;
  static __device__ __forceinline__ constexpr int key_of_row(int r) {
    const int j = r & 3, g = (r >> 2) & 1, h = (r >> 3) & 1;
    return (r & 16) + (KEY_STEP == 4 ? 4 * j + 2 * h + g : KEY_STEP == 2 ? 2 * j + g + 8 * h : r & 15);
  }
  // V^T fragment of 16-key chunk c, row block b = two transpose reads.  P's k-slots 0-3 of lane group
  // grp are rows 16 c + 4 grp + (0..3), slots 4-7 rows 16 c + 8 + 4 grp + (0..3); lane s of a 16-lane
  // group points at the key of row + s / 4, features 32 b + 16 (group % 2) + 4 (s % 4) .. + 3.
  static __device__ __forceinline__ u32x4 read_vfrag(const uint16_t *vs, int c, int b, int lane) {
    const int vr_off = key_of_row(4 * (lane >> 5) + ((lane & 15) >> 2)) * HD + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    const uint16_t *p = vs + vr_off + c * 16 * HD + b * 32;
    const uint2 lo = lds_read_tr16(p), hi = lds_read_tr16(p + key_of_row(8) * HD);
    u32x4 v = u32x4{lo.x, lo.y, hi.x, hi.y};
    if (SUM_BY_MFMA && b == NDB - 1 && (lane & 31) == HD % 32) v = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
    return v;
  }

  // Moves the reference to the maximum mx of the new logits s (relative to the old one).
  template <class Logits>
  __device__ __forceinline__ void move_reference(float mx, int lane, Logits subtract) {
    const bool mine = (fresh >> lane) & 1ull, none = mine && mx == -INFINITY;
    // (keys past the frame can make a block of minus infinities: it moves nothing)
    float target = m_ref + (none ? 0.f : mine ? mx : fmaxf(mx, 0.f));
    if (REF_IN_PAD) target = bf16lo_to_f32(cvt_pk_bf16(target, 0.f));
    const float delta = target - m_ref;
    if (fresh != ~0ull) {               // (something accumulated: delta >= 0 in those lanes)
      const float alpha = mine ? 1.0f : __builtin_amdgcn_exp2f(-delta);
      l_run *= alpha;
#pragma unroll
      for (int b = 0; b < NDB; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) o_acc[b][i] *= alpha;
    }
    subtract(delta);
    m_ref = target;
    if (REF_IN_PAD && (lane >> 5)) qf[NC - 1][0] = cvt_pk_bf16(-target, 0.f);
    fresh = __ballot(none);
  }

  // A whole 64-key tile.  A wavefront alone is bound by latency: LDS reads, dependent MFMAs and
  // the softmax chain follow one another.  Both 32-key blocks are taken together: all K fragments are read up
  // front, the two MFMA chains fill each other's gaps, one maximum and one reference check serve 64 keys.
  __device__ __forceinline__ void tile(const uint16_t *ks, const uint16_t *vs, int kv0, int n, int lane) {
    const int r32 = lane & 31, grp = lane >> 5;
    const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    u32x4 kf[NC][2];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        kf[c][kb] = *reinterpret_cast<const u32x4 *>(ks + (kb * 32 + key_of_row(r32)) * HD + c * 16 + grp * 8);
        if (REF_IN_PAD && c == NC - 1 && grp) kf[c][kb] = u32x4{0x3F80u, 0u, 0u, 0u};   // slot head_dim reads 1, the rest 0
      }
    u32x4 vf[2][NDB];
#pragma unroll
    for (int b = 0; b < NDB; ++b) vf[0][b] = read_vfrag(vs, 0, b, lane);
    f32x16 s[2];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) s[kb] = mfma32(kf[c][kb], qf[c], c == 0 ? zero16 : s[kb]);
    if (!REF_IN_PAD) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[kb][i] -= m_ref;
    }
    if (kv0 + kAttBKV > n) {               // only the last tile can hold keys past the frame
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kv0 + kb * 32 + key_of_row((i >> 2) * 8 + grp * 4 + (i & 3)) >= n) s[kb][i] = -INFINITY;
    }
    float m4[4];                           // four chains of maxima
#pragma unroll
    for (int u = 0; u < 4; ++u) m4[u] = s[u >> 1][(u & 1) * 8];
#pragma unroll
    for (int i = 1; i < 8; ++i)
#pragma unroll
      for (int u = 0; u < 4; ++u) m4[u] = fmaxf(m4[u], s[u >> 1][(u & 1) * 8 + i]);
    const uint32_t mb = __float_as_uint(fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3])));
    const auto r = __builtin_amdgcn_permlane32_swap(mb, mb, false, false);
    const float mx = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));      // relative to m_ref
    if (fresh || __any(mx > kLazy))     // wave-uniform: move the reference
      move_reference(mx, lane, [&](float delta) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
          for (int i = 0; i < 16; ++i) s[kb][i] -= delta;
      });
    // P V by 16-key chunks: the exponentials of chunk c + 1 run beside the MFMAs of chunk c
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      if (c + 1 < 4) {
#pragma unroll
        for (int b = 0; b < NDB; ++b) vf[(c + 1) & 1][b] = read_vfrag(vs, c + 1, b, lane);
      }
      float p[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        p[i] = __builtin_amdgcn_exp2f(s[c >> 1][(c & 1) * 8 + i]);
        if (!SUM_BY_MFMA) l_run += p[i];
      }
      u32x4 pf;
      pf.x = cvt_pk_bf16(p[0], p[1]); pf.y = cvt_pk_bf16(p[2], p[3]);
      pf.z = cvt_pk_bf16(p[4], p[5]); pf.w = cvt_pk_bf16(p[6], p[7]);
#pragma unroll
      for (int b = 0; b < NDB; ++b) o_acc[b] = mfma32(vf[c & 1][b], pf, o_acc[b]);
    }
  }

  // The 32 keys kv0 + 32 kb .. without an online maximum: the reference is the maximum of the first such block (`first`) and
  // stays.  A probability is then 2^(s - reference), whatever its size: float32 and bf16 carry the exponent, so nothing is
  // lost until a later logit exceeds the first block's maximum by some 2^60, which `sound` finds out at the end.  This
  // leaves one exponential and half a conversion per logit on the vector unit.  EDGE: the first tile, and the last one,
  // which can hold keys past the frame.
  template <bool EDGE>
  __device__ __forceinline__ void quick_block(const uint16_t *ks, const uint16_t *vs, int kb, int kv0, int n, int lane, bool first) {
    const int r32 = lane & 31, grp = lane >> 5;
    u32x4 kf[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      kf[c] = *reinterpret_cast<const u32x4 *>(ks + (kb * 32 + key_of_row(r32)) * HD + c * 16 + grp * 8);
      if (REF_IN_PAD && c == NC - 1 && grp) kf[c] = u32x4{0x3F80u, 0u, 0u, 0u};   // slot head_dim reads 1, the rest 0
    }
    u32x4 vf[2][NDB];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int b = 0; b < NDB; ++b) vf[hh][b] = read_vfrag(vs, 2 * kb + hh, b, lane);
    f32x16 s;                                // (where no slot is spare the reference is subtracted in the accumulator)
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = REF_IN_PAD ? 0.f : -m_ref;
#pragma unroll
    for (int c = 0; c < NC; ++c) s = mfma32(kf[c], qf[c], s);
    if (EDGE && kv0 + kAttBKV > n) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (kv0 + kb * 32 + key_of_row((i >> 2) * 8 + grp * 4 + (i & 3)) >= n) s[i] = -INFINITY;
    }
    if (EDGE && first) {
      float m = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) m = fmaxf(m, s[i]);
      const uint32_t mb = __float_as_uint(m);
      const auto r = __builtin_amdgcn_permlane32_swap(mb, mb, false, false);
      m = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
      if (!(fabsf(m) < INFINITY)) m = 0.f;      // (no finite maximum: `sound` finds a later one, or a NaN or an infinity)
      if (REF_IN_PAD) m = bf16lo_to_f32(cvt_pk_bf16(m, 0.f));
      m_ref = m;
      if (REF_IN_PAD && grp) qf[NC - 1][0] = cvt_pk_bf16(-m, 0.f);
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] -= m;
    }
    float p[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      p[i] = __builtin_amdgcn_exp2f(s[i]);
      if (!SUM_BY_MFMA) l_run += p[i];
    }
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      u32x4 pf;
      pf.x = cvt_pk_bf16(p[hh * 8 + 0], p[hh * 8 + 1]); pf.y = cvt_pk_bf16(p[hh * 8 + 2], p[hh * 8 + 3]);
      pf.z = cvt_pk_bf16(p[hh * 8 + 4], p[hh * 8 + 5]); pf.w = cvt_pk_bf16(p[hh * 8 + 6], p[hh * 8 + 7]);
#pragma unroll
      for (int b = 0; b < NDB; ++b) o_acc[b] = mfma32(vf[hh][b], pf, o_acc[b]);
    }
  }

  // Whether quick_block's result stands: the weights' sums are of ordinary size and everything is finite.
  __device__ __forceinline__ bool sound(int r32) const {
    const float l = denominator(r32);
    float z = 0.f;
#pragma unroll
    for (int b = 0; b < NDB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (b * 32 + (i >> 2) * 8 < HD) z = fmaf(o_acc[b][i], 0.f, z);          // (rows past head_dim hold anything)
    return l > 0x1p-60f && l < 0x1p60f && z == 0.f;
  }

  // Softmax denominator of this lane's query.
  __device__ __forceinline__ float denominator(int r32) const {
    if (SUM_BY_MFMA) {                        // accumulator row head_dim of O^T: lane group (row % 8) / 4, register (row / 8) * 4 + row % 4
      constexpr int ROW = HD % 32;
      return __shfl(o_acc[NDB - 1][(ROW / 8) * 4 + (ROW % 4)], r32 + 32 * ((ROW % 8) / 4), 64);
    }
    return l_run + __shfl_xor(l_run, 32, 64);
  }
};

// QUICK: the pass without an online maximum first (see launch_attention_hd).
template <int HD, int MINB, bool QUICK>
__global__ __launch_bounds__(kAttWaves * 64, MINB) void attention_dma_kernel(
    const uint16_t *__restrict__ qkv, const int32_t *__restrict__ cu, int n, int n_heads, int n_qblk, float scale_log2,
    uint16_t *__restrict__ out) {
  using Rows = AttentionRows<HD>;
  constexpr int NDB = Rows::NDB;
  constexpr int STAGES = 2;
  constexpr int T_LOADS = HD / 8;            // 1 KiB pieces of a K (or V) tile: 64 keys * HD * 2 bytes
  constexpr int PW = (T_LOADS + kAttWaves - 1) / kAttWaves;   // pieces per wavefront
  constexpr int K_ELEMS = kAttBKV * HD, V_ELEMS = kAttBKV * HD;
  constexpr int STAGE = K_ELEMS + V_ELEMS;
  // tail pad: the last V row's fragments of row blocks past head_dim read up to NDB * 32 - HD elements
  // behind the tile (rounded up generously).
  constexpr int PAD = (NDB * 32 - HD) * kAttBKV + 64;
  __shared__ __align__(16) uint16_t lds[STAGES * STAGE + PAD];
  __shared__ int redo;
  if (QUICK) clear_flag(redo);

  // One-dimensional grid over (frame, head, query block), query block fastest, so that the query blocks
  // of one (frame, head) - which read the same K and V - run on one XCD and share its L2.
  const int v = xcd_contiguous_index(gridDim.x);
  const int q0 = (v % n_qblk) * kAttBQ, h = (v / n_qblk) % n_heads, f = v / (n_qblk * n_heads);
  int start = f * n;
  if (cu) {                                            // ragged frames (workgroup-uniform)
    start = cu[f];
    n = cu[f + 1] - start;
    if (q0 >= n) return;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps load dispatch scalar
  const int r32 = lane & 31, grp = lane >> 5;
  const int D = n_heads * HD, ld = 3 * D;
  const uint16_t *qbase = qkv + (size_t)start * ld + h * HD;
  const uint16_t *kbase = qbase + D;                    // (V: + D again)
  const int n_tiles = (n + kAttBKV - 1) / kAttBKV;

  // Pieces j = wave, wave + 4, ... of a tile belong to this wavefront: K and V by direct global -> LDS loads.  A scalar
  // origin that advances by a constant per tile plus 32-bit lane offsets; the last tile has offsets of its own, with the
  // key rows clamped to the frame (masked later, in bounds).  V's origin is K's + D.
  uint32_t off[PW], off_last[PW];            // bytes from the tile's origin
#pragma unroll
  for (int j = 0; j < PW; ++j) {
    const int q = min(j * kAttWaves + wave, T_LOADS - 1) * 64 + lane, key = q / (HD / 8), ch = q % (HD / 8);
    off[j] = (uint32_t)(key * ld + ch * 8) * 2u;
    off_last[j] = (uint32_t)(min(key, n - 1 - (n_tiles - 1) * kAttBKV) * ld + ch * 8) * 2u;
  }
  auto issue = [&](int t) {                            // tile t into stage t % 2
    const uint16_t *k0 = kbase + (size_t)t * kAttBKV * ld;
    uint16_t *dst = lds + (t & 1) * STAGE;
    const bool last = t + 1 == n_tiles;
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int piece = j * kAttWaves + wave;          // (wave-uniform)
      if (piece < T_LOADS) {
        const uint32_t o = last ? off_last[j] : off[j];
        lds_dma16_untracked(k0, o, dst + piece * 512);
        lds_dma16_untracked(k0 + D, o, dst + K_ELEMS + piece * 512);
      }
    }
  };
  Rows rows;
  const bool active = q0 + wave * 32 < n;              // (wave-uniform: past the frame's queries a wavefront only loads)
  // One pass over the key tiles; tile(t, K, V) takes them in order.
  auto pass = [&](auto tile) {
    issue(0);
    rows.start(qbase, q0 + wave * 32, n, ld, scale_log2, r32, grp);
    for (int t = 0; t < n_tiles; ++t) {
      wait_all();                              // tile t has landed, and the reads of tile t-1 have returned
      __builtin_amdgcn_s_barrier();            // ... for every wavefront: the loads behind it may overwrite tile t-1
      asm volatile("" ::: "memory");
      if (t + 1 < n_tiles) issue(t + 1);
      const uint16_t *ks = lds + (t & 1) * STAGE;
      if (active) tile(t, ks, ks + K_ELEMS);
    }
  };
  auto careful = [&](int t, const uint16_t *ks, const uint16_t *vs) { rows.tile(ks, vs, t * kAttBKV, n, lane); };
  if constexpr (QUICK) {
    pass([&](int t, const uint16_t *ks, const uint16_t *vs) {
      const int kv0 = t * kAttBKV;
      const bool edge = t == 0 || t + 1 == n_tiles;
#pragma unroll                                         // (in this form the registers suffice: no spill in the loop)
      for (int kb = 0; kb < 2; ++kb) {
        if (edge) {
          if (kb == 0 || kv0 + 32 < n) rows.template quick_block<true>(ks, vs, kb, kv0, n, lane, t == 0 && kb == 0);
        } else {
          rows.template quick_block<false>(ks, vs, kb, kv0, n, lane, false);
        }
      }
    });
    raise_flag(redo, active && !rows.sound(r32));
    __syncthreads();
    if (__builtin_expect(redo, 0)) pass(careful);
  } else {
    pass(careful);
  }

  const float inv = 1.0f / rows.denominator(r32);
  const int q = q0 + wave * 32 + r32;
  if (q < n) {
    uint16_t *orow = out + ((size_t)start + q) * D + h * HD;
#pragma unroll
    for (int b = 0; b < NDB; ++b)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const int d = b * 32 + qd * 8 + grp * 4;
        if (d < HD) {
          const f32x16 &o = rows.o_acc[b];
          uint2 w;
          w.x = cvt_pk_bf16(o[qd * 4 + 0] * inv, o[qd * 4 + 1] * inv);
          w.y = cvt_pk_bf16(o[qd * 4 + 2] * inv, o[qd * 4 + 3] * inv);
          *reinterpret_cast<uint2 *>(orow + d) = w;
        }
      }
  }
}

// Workgroup `idx` of `count` reads its share of the ranges, eight 16-byte loads per thread in flight.
__device__ __forceinline__ void read_ahead(const WarmRanges &w, int idx, int count) {
#pragma unroll 1
  for (int r = 0; r < WarmRanges::kMax; ++r) {
    const u32x4 *p = static_cast<const u32x4 *>(w.ptr[r]);
    const uint32_t n = w.bytes[r] / 16u, step = (uint32_t)count * blockDim.x;
    if (n == 0) continue;
#pragma unroll 1
    for (uint32_t i = (uint32_t)idx * blockDim.x + threadIdx.x; i < n; i += 8 * step) {
      u32x4 v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = p[min(i + u * step, n - 1)];
#pragma unroll
      for (int u = 0; u < 8; ++u) asm volatile("" ::"v"(v[u]));
    }
  }
}

// ---------------------------------------------------------------------------------------
// The same for few queries, where a workgroup per 128 queries leaves most of the chip idle and walks all key tiles
// one after the other (1.4 us per tile): the 8 wavefronts of a workgroup form KG groups; a group takes 256 / KG
// queries, one block of 32 per wavefront, and every KG-th key tile, with LDS stages of its own.  The groups'
// partial results (reference maximum, denominator, O^T) meet in LDS; a thread finishes 8 features of a query
// and stores 16 bytes.  (Without the online maximum: 1 x 729 12.1 -> 11.4 us, 2 x 729 16.4 -> 14.9, 3 x 364 10.5 -> 10.0.)
// (One query block per workgroup, its tiles split over 4 wavefronts with private slots, loads every
// tile once per 32 queries: 729 tokens x 16 heads 18.0 -> 13.6 us, and slower than the kernel above from two frames on.)
// ---------------------------------------------------------------------------------------
template <int HD, int KG>
struct GroupShape {
  static constexpr int WPG = 8 / KG, NDB = (HD + 31) / 32, TILE = kAttBKV * HD;
  static constexpr int GROUP = 4 * TILE + 64;               // elements: two stages of K and V, and what the last fragments read past them
  static constexpr int O_LD = NDB * 32 + 4;                 // floats of a query's partial row: no bank conflicts on 16-byte cells
  static constexpr size_t kStages = (size_t)KG * GROUP * 2, kPartials = (size_t)8 * 32 * O_LD * 4;
  static constexpr size_t kLdsBytes = kStages > kPartials ? kStages : kPartials;
  static constexpr bool kFits = kLdsBytes + 8 * 32 * sizeof(float2) + sizeof(int) <= 160 * 1024;
};

template <int HD, int KG>
__global__ __launch_bounds__(512, 1) void attention_group_kernel(
    const uint16_t *__restrict__ qkv, const int32_t *__restrict__ cu, int n, int n_heads, int n_qblk, float scale_log2,
    uint16_t *__restrict__ out, WarmRanges warm, int n_work) {
  using S = GroupShape<HD, KG>;
  using Rows = AttentionRows<HD>;
  constexpr int WPG = S::WPG, T_LOADS = HD / 8, PW = (T_LOADS + WPG - 1) / WPG;
  extern __shared__ __align__(16) uint16_t lds[];
  __shared__ float2 ml[8][32];
  __shared__ int redo;
  clear_flag(redo);
  if ((int)blockIdx.x >= n_work) return read_ahead(warm, blockIdx.x - n_work, gridDim.x - n_work);
  const int v = xcd_contiguous_index(n_work);
  const int q0 = (v % n_qblk) * (32 * WPG), h = (v / n_qblk) % n_heads, f = v / (n_qblk * n_heads);
  int start = f * n;
  if (cu) {                                            // ragged frames (workgroup-uniform)
    start = cu[f];
    n = cu[f + 1] - start;
    if (q0 >= n) return;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp_k = wave / WPG, wi = wave % WPG;       // group (its key tiles) and query block inside the workgroup
  const int r32 = lane & 31, grp = lane >> 5;
  const int D = n_heads * HD, ld = 3 * D;
  const uint16_t *qbase = qkv + (size_t)start * ld + h * HD;
  const uint16_t *kbase = qbase + D;                    // (V: + D again)
  const int n_tiles = (n + kAttBKV - 1) / kAttBKV;
  uint16_t *mem = lds + grp_k * S::GROUP;

  // Pieces wi, wi + WPG, ... of the group's tiles by direct loads (see above).  Key rows past the frame are clamped to
  // its last one (masked later).
  uint32_t off[PW], off_last[PW];                      // bytes from the tile's origin
#pragma unroll
  for (int j = 0; j < PW; ++j) {
    const int piece = min(j * WPG + wi, T_LOADS - 1) * 64 + lane, key = piece / (HD / 8), ch = piece % (HD / 8);
    off[j] = (uint32_t)(key * ld + ch * 8) * 2u;
    off_last[j] = (uint32_t)(min(key, n - 1 - (n_tiles - 1) * kAttBKV) * ld + ch * 8) * 2u;
  }
  auto issue = [&](int t, int stage) {
    const uint16_t *k0 = kbase + (size_t)t * kAttBKV * ld;
    uint16_t *dst = mem + stage * 2 * S::TILE;
    const bool last = t + 1 == n_tiles;
#pragma unroll
    for (int j = 0; j < PW; ++j) {
      const int piece = j * WPG + wi;                  // (wave-uniform)
      if (piece < T_LOADS) {
        const uint32_t o = last ? off_last[j] : off[j];
        lds_dma16_untracked(k0, o, dst + piece * 512);
        lds_dma16_untracked(k0 + D, o, dst + S::TILE + piece * 512);
      }
    }
  };
  Rows rows;
  const bool has_tiles = grp_k < n_tiles;              // (wave-uniform)
  auto pass = [&](auto tile) {
    if (has_tiles) issue(grp_k, 0);
    rows.start(qbase, q0 + wi * 32, n, ld, scale_log2, r32, grp);
    int stage = 0;
    for (int t0 = 0; t0 < n_tiles; t0 += KG, stage ^= 1) {
      const int t = t0 + grp_k;
      wait_all();                                      // tile t has landed, and the reads of the other stage have returned
      __builtin_amdgcn_s_barrier();                    // ... for every wavefront: the loads behind it may overwrite that stage
      asm volatile("" ::: "memory");
      if (t + KG < n_tiles) issue(t + KG, stage ^ 1);
      const uint16_t *ks = mem + stage * 2 * S::TILE;
      if (t < n_tiles) tile(t, ks, ks + S::TILE);
    }
  };
  pass([&](int t, const uint16_t *ks, const uint16_t *vs) {
    const int kv0 = t * kAttBKV;
    const bool edge = t == grp_k || t + 1 == n_tiles;
    if (edge) {
#pragma unroll 1                                       // (code that runs once or twice is kept short: it comes in cold)
      for (int kb = 0; kb < (kv0 + 32 < n ? 2 : 1); ++kb) rows.template quick_block<true>(ks, vs, kb, kv0, n, lane, t == grp_k && kb == 0);
    } else {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) rows.template quick_block<false>(ks, vs, kb, kv0, n, lane, false);
    }
  });
  // (a group without a tile, or with nothing but minus infinities, has no part in the sum)
  auto leave = [&](bool nothing) {
    const float l = rows.denominator(r32);
    if (grp == 0) ml[wave][r32] = nothing ? make_float2(-INFINITY, 0.f) : make_float2(rows.m_ref, l);
  };
  leave(!has_tiles);
  raise_flag(redo, has_tiles && !rows.sound(r32));
  __syncthreads();                                     // the stages have been read
  if (__builtin_expect(redo, 0)) {
    pass([&](int t, const uint16_t *ks, const uint16_t *vs) { rows.tile(ks, vs, t * kAttBKV, n, lane); });
    leave((rows.fresh >> lane) & 1ull);
    __syncthreads();
  }
  float *part = reinterpret_cast<float *>(lds);
#pragma unroll
  for (int b = 0; b < S::NDB; ++b)
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
      const f32x16 &a = rows.o_acc[b];
      *reinterpret_cast<f32x4 *>(part + (wave * 32 + r32) * S::O_LD + b * 32 + qd * 8 + grp * 4) =
          f32x4{a[qd * 4], a[qd * 4 + 1], a[qd * 4 + 2], a[qd * 4 + 3]};
    }
  __syncthreads();
  for (int i = tid; i < 32 * WPG * (HD / 8); i += 512) {
    const int q = i / (HD / 8), ch = i % (HD / 8);     // (q = 32 * wavefront of the group + query)
    if (q0 + q >= n) continue;
    float m = -INFINITY, den = 0.f, fac[KG];
#pragma unroll
    for (int k = 0; k < KG; ++k) m = fmaxf(m, ml[k * WPG + (q >> 5)][q & 31].x);
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      const float2 w = ml[k * WPG + (q >> 5)][q & 31];
      fac[k] = __builtin_amdgcn_exp2f(w.x - m);
      den = fmaf(fac[k], w.y, den);
    }
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      const float *p = part + (k * WPG * 32 + q) * S::O_LD + ch * 8;
      lo += *reinterpret_cast<const f32x4 *>(p) * fac[k];
      hi += *reinterpret_cast<const f32x4 *>(p + 4) * fac[k];
    }
    const float inv = 1.0f / den;
    u32x4 r;
    r.x = cvt_pk_bf16(lo[0] * inv, lo[1] * inv); r.y = cvt_pk_bf16(lo[2] * inv, lo[3] * inv);
    r.z = cvt_pk_bf16(hi[0] * inv, hi[1] * inv); r.w = cvt_pk_bf16(hi[2] * inv, hi[3] * inv);
    *reinterpret_cast<u32x4 *>(out + ((size_t)start + q0 + q) * D + h * HD + ch * 8) = r;
  }
}

}  // namespace

int device_cus() {
  static std::atomic<int> known[64];       // by device; 0: not asked yet
  int dev = 0, n = 0;
  const bool have_dev = hipGetDevice(&dev) == hipSuccess;
  std::atomic<int> &slot = known[dev & 63];
  if (have_dev && (n = slot.load(std::memory_order_relaxed)) > 0) return n;
  if (!have_dev || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
    (void)hipGetLastError();
    return 256;
  }
  slot.store(n, std::memory_order_relaxed);
  return n;
}

int launch_layernorm(const uint16_t *x, const float *g, const float *b, float eps, int rows, int D,
                     uint16_t *y, hipStream_t s) {
  if (rows <= 0) return ET_OK;
  dim3 grid((rows + kLnRows - 1) / kLnRows), block(kLnRows * kWave);
  ET_DISPATCH_NV(D, hipLaunchKernelGGL(layernorm_kernel<NV>, grid, block, 0, s, x, g, b, eps, rows, D, y));
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_rowstats(const uint16_t *x, float eps, int rows, int D, float *rstd, hipStream_t s) {
  if (rows <= 0) return ET_OK;
  dim3 grid((rows + kLnRows - 1) / kLnRows), block(kLnRows * kWave);
  ET_DISPATCH_NV(D, hipLaunchKernelGGL(rowstats_kernel<NV>, grid, block, 0, s, x, eps, rows, D, rstd));
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_piece_stats(const uint16_t *x, int rows, int D, int ld, float2 *stats, hipStream_t s) {
  if (rows <= 0) return ET_OK;
  dim3 grid((rows + kLnRows - 1) / kLnRows), block(kLnRows * kWave);
  ET_DISPATCH_NV(D, hipLaunchKernelGGL(piece_stats_kernel<NV>, grid, block, 0, s, x, rows, D, ld, stats));
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_piece_scale(const uint16_t *x, float eps, int rows, int D, float *rstd, hipStream_t s) {
  if (rows <= 0) return ET_OK;
  dim3 grid((rows + kLnRows - 1) / kLnRows), block(kLnRows * kWave);
  ET_DISPATCH_NV(D, hipLaunchKernelGGL(piece_scale_kernel<NV>, grid, block, 0, s, x, eps, rows, D, rstd));
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_im2col(const float *frames, int T, int C, int H, int W, int P, int Kpad, uint16_t *out,
                  hipStream_t s) {
  const int GX = W / P, GY = H / P, L = GX * GY;
  const size_t stripe_bytes = (size_t)C * P * W * sizeof(uint16_t);
  if (W % 4 == 0 && reinterpret_cast<uintptr_t>(frames) % 16 == 0 && stripe_bytes <= 64 * 1024) {
    // A workgroup's copy is a chain of a few loads per thread: more wavefronts per workgroup while there are few
    // workgroups (256 / 512 / 1024 threads, us: 27 workgroups of 384-pixel images 18 / 12 / 9, 216 21 / 14 / 12, 432
    // 24 / 19 / 17, 864 33 / 28 / 30, 1728 52 / 46 / 50).
    hipLaunchKernelGGL(im2col_stripe_kernel, dim3((unsigned)(T * GY)), dim3(T * GY <= 512 ? 1024 : 512), stripe_bytes, s, frames, C, H, W, P,
                       GX, GY, C * P * P, Kpad, out);
    ET_LAUNCH_CHECK();
    return ET_OK;
  }
  const size_t n = (size_t)T * L * (Kpad / 8);
  hipLaunchKernelGGL(im2col_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, frames, T, C, H, W, P,
                     GX, L, C * P * P, Kpad, out);
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int gemm_config_count() { return kCfgStrip; }     // (what et_gemm_bf16 can ask for)

static int launch_gemm_id(const GemmArgs &g, hipStream_t s, int cfg) {
  switch (cfg) {
    case kCfgBig: return launch_gemm_stream_cfg<256, 256, 2, 4, 1>(g, s);
    case kCfg128: return launch_gemm_stream_cfg<128, 128, 2, 2, 2>(g, s);
    case kCfgWave: return launch_gemm_wave(g, s);
    case kCfgPair64: return launch_gemm_pair64(g, s);
    case kCfgPair128: return launch_gemm_pair128(g, s);
    case kCfgHalf: return launch_gemm_half(g, s);
    case kCfgStrip: return launch_gemm_strip(g, s);
    default: set_error("unknown gemm tile configuration %d", cfg); return ET_ERR_INVALID_ARG;
  }
}

// Whether a GEMM over `rows` rows is best done in one round of tiles, i.e. takes the statistics of its rows by
// pieces (launch_gemm accepts them for any size; beyond one round the row scales' own launch is cheaper).
bool gemm_takes_pieces(int rows, int cols) { return one_round(kCfgBig, rows, cols, device_cus()); }

int launch_gemm(const GemmArgs &args, hipStream_t s, int force_cfg, bool one_tile) {
  GemmArgs g = args;
  // from 1 MB of results on (0.7 MB: two launches 19.3 us without, 19.7 with; 1.7 to 6.3 MB, a 27-block encoder: 1984, 1930)
  g.through = (size_t)g.M * g.n_store * sizeof(uint16_t) >= (1u << 20);
  if (g.M <= 0) return ET_OK;
  if (g.K % 64 != 0 || g.n_store % 8 != 0) {
    set_error("gemm: K = %d must be a multiple of 64 and n_store = %d of 8", g.K, g.n_store);
    return ET_ERR_INVALID_ARG;
  }
  if ((g.stats_in && (g.row_scale || g.epilogue == EPI_BIAS_RES)) || (g.stats_out && (g.epilogue != EPI_BIAS_RES || g.n_store % 64 != 0))) {
    set_error("gemm: row statistics asked of an epilogue that has none");
    return ET_ERR_INVALID_ARG;
  }
  if (force_cfg >= 0) return launch_gemm_id(g, s, force_cfg);
  const GemmPlan plan = plan_gemm(GemmRules{g.K, device_cus(), g.epilogue != EPI_BIAS_RES || g.res_mod >= g.M, g.stats_in != nullptr || one_tile, g.epilogue == EPI_BIAS_RES}, g.M, g.n_store);
  for (int i = 0; i < plan.n; ++i) {
    const GemmPart &t = plan.part[i];
    GemmArgs part = g;
    part.M = t.rows;
    part.n_store = t.cols;
    part.A = g.A + (size_t)t.row0 * g.lda;
    part.W = g.W + (size_t)t.col0 * g.K;
    part.bias = g.bias + t.col0;
    part.C = g.C + (size_t)t.row0 * g.ldc + t.col0;
    if (g.res) part.res = g.res + (size_t)t.row0 * g.ldr + t.col0;
    if (g.row_scale) part.row_scale = g.row_scale + t.row0;
    if (g.stats_out) part.stats_out = g.stats_out + (size_t)(t.col0 / 64) * g.stats_ld + t.row0;
    const int rc = launch_gemm_id(part, s, t.cfg);
    if (rc != ET_OK) return rc;
  }
  return ET_OK;
}

bool head_dim_supported(int hd) {
  return hd == 16 || hd == 32 || hd == 64 || hd == 72 || hd == 80 || hd == 96 || hd == 128;
}

template <int HD, int KG>
static int launch_attention_group(const uint16_t *qkv, const int32_t *cu, int n, int n_tiles, int n_heads, int n_qblk, long long pairs,
                                  float scale_log2, uint16_t *out, hipStream_t s, const WarmRanges *warm) {
  constexpr size_t bytes = GroupShape<HD, KG>::kLdsBytes;
  constexpr auto kern = attention_group_kernel<HD, KG>;
  if (int rc = allow_lds<kern>(bytes)) return rc;
  // One workgroup per compute unit: the idle ones read ahead what read_ahead_of allows them.  (Where the attention has several
  // workgroups per compute unit, or beside the QKV projection, reading ahead costs what it gives.)
  const int work = (int)(n_qblk * pairs), idle = device_cus() - work;
  const WarmRanges ahead = warm ? read_ahead_of(*warm, idle, (n_tiles + KG - 1) / KG) : WarmRanges{};
  const int more = ahead.bytes[0] ? idle : 0;
  hipLaunchKernelGGL(kern, dim3(work + more), dim3(512), bytes, s, qkv, cu, n, n_heads, n_qblk, scale_log2, out, ahead, work);
  ET_LAUNCH_CHECK();
  return ET_OK;
}

// cu == nullptr: frames of `len` rows each; else row ranges cu[f] .. cu[f + 1] of at most `len` rows.
template <int HD>
static int launch_attention_hd(const uint16_t *qkv, const int32_t *cu, int n_frames, int len, int n_heads, uint16_t *out,
                               hipStream_t s, const WarmRanges *warm) {
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)HD);
  const long long pairs = (long long)n_heads * n_frames, cus = device_cus();
  const int n = cu ? 0 : len;
  auto blocks = [&](int rows) { return (len + rows - 1) / rows; };
  // Key tiles split over groups of wavefronts while that still makes one workgroup per compute unit at most, and
  // while a group keeps enough tiles for the exchange to pay.  Measured, microseconds per launch against the
  // kernel of 128 queries (heads of 72): 1 x 729 (192 workgroups of four groups) 17.3 -> 12.8, 2 x 729 (192 of two groups)
  // 17.0 -> 15.3, 3 x 364 (144) 12.1 -> 10.6; heads of 64: 1 x 196 8.7 -> 6.8, 4 x 98 6.3 -> 6.0.  Past the line: 4 x 729
  // 23.9 -> 30.0, 8 x 182 (3 tiles, two groups) 8.1 -> 8.6.
  const int n_tiles = blocks(kAttBKV);
  if constexpr (GroupShape<HD, 4>::kFits) {
    if (n_tiles >= 2 && blocks(64) * pairs <= cus)
      return launch_attention_group<HD, 4>(qkv, cu, n, n_tiles, n_heads, blocks(64), pairs, scale_log2, out, s, warm);
  }
  if constexpr (GroupShape<HD, 2>::kFits) {
    if (n_tiles >= 5 && blocks(128) * pairs <= cus)
      return launch_attention_group<HD, 2>(qkv, cu, n, n_tiles, n_heads, blocks(128), pairs, scale_log2, out, s, warm);
  }
  // Three workgroups per compute unit where the registers suffice without a spill: with both passes up to heads of 72, with the
  // online maximum alone also heads of 80 (150 registers; both passes take 186, held to 168 they spill).  Those take it from the
  // first workgroup that two per compute unit leave waiting.  us per launch, two with both passes / three with one: 47 x 59
  // (12 heads) 9.3 / 7.7, 18 x 172 17.5 / 14.0, 15 x 325 21.0 / 18.6, 29 x 322 32.2 / 29.8, 57 x 829 (12 heads) 227 / 216, 9 x
  // 761 46.6 / 48.5, 11 x 678 (12 heads) 41.4 / 42.5; up to two per compute unit two are the faster ones (5 x 777, 12 heads,
  // 23.7 / 26.4; 11 x 148 10.1 / 10.7).
  const long long work = blocks(kAttBQ) * pairs;
  auto launch = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)work), dim3(kAttWaves * 64), 0, s, qkv, cu, n, n_heads, blocks(kAttBQ), scale_log2, out);
  };
  bool three = false;
  if constexpr (HD == 80) {
    three = work > 2 * cus;
    if (three) launch(attention_dma_kernel<HD, 3, false>);
  }
  if (!three) launch(attention_dma_kernel<HD, (HD <= 72 ? 3 : HD <= 96 ? 2 : 1), true>);
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_attention(const uint16_t *qkv, const int32_t *cu, int n_frames, int len, int n_heads, int head_dim, uint16_t *out,
                     hipStream_t s, const WarmRanges *warm) {
  if (n_frames <= 0 || len <= 0) return ET_OK;
  switch (head_dim) {
    case 16: return launch_attention_hd<16>(qkv, cu, n_frames, len, n_heads, out, s, warm);
    case 32: return launch_attention_hd<32>(qkv, cu, n_frames, len, n_heads, out, s, warm);
    case 64: return launch_attention_hd<64>(qkv, cu, n_frames, len, n_heads, out, s, warm);
    case 72: return launch_attention_hd<72>(qkv, cu, n_frames, len, n_heads, out, s, warm);
    case 80: return launch_attention_hd<80>(qkv, cu, n_frames, len, n_heads, out, s, warm);
    case 96: return launch_attention_hd<96>(qkv, cu, n_frames, len, n_heads, out, s, warm);
    case 128: return launch_attention_hd<128>(qkv, cu, n_frames, len, n_heads, out, s, warm);
    default: set_error("head_dim %d is not instantiated", head_dim); return ET_ERR_UNSUPPORTED;
  }
}

int launch_attention_uniform(const uint16_t *qkv, int n_frames, int len, int n_heads, int head_dim, uint16_t *out, hipStream_t s,
                             const WarmRanges *warm) {
  return launch_attention(qkv, nullptr, n_frames, len, n_heads, head_dim, out, s, warm);
}

}  // namespace et
