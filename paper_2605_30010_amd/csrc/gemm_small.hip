// GEMM kernels for few rows (a short clip, or the blocks on the kept tokens), where the output has
// too few tiles to fill the chip: the contraction is split over the wavefronts of a workgroup and
// the partial sums meet in LDS, so nothing but the result goes through memory.  (gemm_half_kernel and
// gemm_strip_kernel split no k: k ascending in one accumulator, as the persistent kernel does it.)
//
// What bounds these launches (measured): a launch costs 2.2 us before it does anything; after that
// a compute unit takes its operands through one 64-byte-per-clock path (59 B/clk reached, and only
// with rows of 128 bytes: 64-byte row segments halve it), i.e. 256 cycles per 64 x 64 x 64 step and
// 512 per 128 x 128 x 64, against 128 and 512 cycles of the matrix unit.  What cost the time before
// was neither: a 64 x 128 workgroup tile walked its k-tiles one after the other, each a chain of
// barrier, LDS reads waited for one by one, two MFMAs per wait (0.6-1.2 us per k-tile).

#include "gemm_small.h"

namespace et {

namespace {

// Workgroups go to the 8 XCDs round-robin by index; XCD x takes the x-th contiguous run of tiles
// (bands of 8 tile rows, column by column inside a band), so that the tiles an XCD works on at
// once share operand slices through its L2.
__device__ __forceinline__ void small_tile_of(int tiles_m, int tiles_n, int &tm, int &tn) {
  const int total = tiles_m * tiles_n, per = total / 8, rem = total % 8, xcd = blockIdx.x % 8, slot = blockIdx.x / 8;
  const int v = xcd * per + (xcd < rem ? xcd : rem) + slot;
  const int band = v / (8 * tiles_n), r = v - band * 8 * tiles_n;
  const int hb = (tiles_m - band * 8 < 8) ? (tiles_m - band * 8) : 8;
  tm = band * 8 + r % hb;
  tn = r / hb;
}

// The lane offsets of the direct loads are lowered by the immediate of their group of four (see
// lds_dma16_of4); the bias keeps them non-negative and is taken off the scalar base.
constexpr uint32_t kOffBias = 4096;

// Byte offset of this lane's piece of row `row` (stride `ld` elements) in the i-th 1 KiB load of an
// operand: lane L lands at row L / 8, slot L % 8 of the 8-row piece and fetches 16-byte chunk
// slot ^ (row >> 1) % 8, an XOR swizzle that spreads the fragment reads over the banks.
__device__ __forceinline__ uint32_t piece_offset(int row, int src_row, int ld, int slot, int i) {
  return (uint32_t)src_row * (uint32_t)ld * 2u + (uint32_t)((slot ^ ((row >> 1) & 7)) * 16) + kOffBias - (uint32_t)(i % 4) * 1024u;
}

// Sum of the SUM partial 64 x 64 tiles of one output tile and the epilogue.  put() writes the wavefront's
// accumulators to 16 KiB of LDS per partial tile (fragment order, 16-byte cells); wavefront
// `rank` of the PARTS that share the output tile finishes 64 / PARTS rows, reading the cells row by row so that residual loads
// and stores are 128-byte row segments.  Partial sums are added in ascending order of the wavefronts:
// the result does not depend on timing.  rs_tile (LDS): the row scales of the 64 rows, written before the barrier.
// The cell of (column octet c, lane l) sits at l ^ (c << 1):
// both the writes (fixed c) and the row-wise reads (8 octets x 8 rows) are then conflict-free.
template <int PARTS, int SUM, int STRIDE, int EPI, class Put>
__device__ __forceinline__ void finish_rows(Put put, const GemmArgs &g, f32x4 *xch, int first, int rank, int m_tile, int n_tile,
                                            int lane, const float *rs_tile) {
  constexpr int ROWS = 64 / PARTS, PASS = ROWS / 8;
  const int pr = lane >> 3, oct = lane & 7;
  const int n = n_tile + oct * 8, row0 = rank * ROWS + pr;
  const bool n_ok = n < g.n_store;                       // n_store is a multiple of 8
  u32x4 res[PASS];
#pragma unroll
  for (int p = 0; p < PASS; ++p) {                       // fetched before the exchange: the latency is hidden by it
    const int m = m_tile + row0 + p * 8;
    res[p] = u32x4{0u, 0u, 0u, 0u};
    if (EPI == EPI_BIAS_RES && m < g.M && n_ok)
      res[p] = *reinterpret_cast<const u32x4 *>(g.res + (size_t)(m % g.res_mod) * g.ldr + n);
  }
  f32x4 b0 = {0.f, 0.f, 0.f, 0.f}, b1 = b0;
  if (n_ok) {
    b0 = *reinterpret_cast<const f32x4 *>(g.bias + n);
    b1 = *reinterpret_cast<const f32x4 *>(g.bias + n + 4);
  }
  put();
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PASS; ++p) {
    const int ml = row0 + p * 8, m = m_tile + ml, r = ml & 31;
    const float rs = EPI == EPI_BIAS_RES ? 1.0f : rs_tile[ml];       // (no LayerNorm in front of a residual GEMM)
    const f32x4 *cell = xch + first * 1024 + ((ml >> 5) * 8 + oct) * 64;
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
    for (int j = 0; j < SUM; ++j) {
      lo += cell[j * STRIDE * 1024 + (r ^ (oct << 1))];
      hi += cell[j * STRIDE * 1024 + ((32 + r) ^ (oct << 1))];
    }
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f32x4 &s = e < 2 ? lo : hi, &bi = e < 2 ? b0 : b1;
      float x0 = fmaf(rs, s[(e & 1) * 2], bi[(e & 1) * 2]), x1 = fmaf(rs, s[(e & 1) * 2 + 1], bi[(e & 1) * 2 + 1]);
      if (EPI == EPI_BIAS_GELU) {
        x0 = gelu_tanh_f(x0);
        x1 = gelu_tanh_f(x1);
      }
      if (EPI == EPI_BIAS_RES) {
        x0 += bf16lo_to_f32(res[p][e]);
        x1 += bf16hi_to_f32(res[p][e]);
      }
      o[e] = cvt_pk_bf16(x0, x1);
    }
    if (m < g.M && n_ok) store16(g.C + (size_t)m * g.ldc + n, o, g.through);
    if (EPI == EPI_BIAS_RES && g.stats_out) {              // (n_store is a multiple of 64 then)
      const float2 st = piece_moments(o);
      if (oct == 0 && m < g.M && n_ok) g.stats_out[(size_t)(n_tile >> 6) * g.stats_ld + m] = st;
    }
  }
}

// One 32 x 32 accumulator (columns 32 a, rows 32 b of the 64 x 64 tile) to the cells above.
__device__ __forceinline__ void put_quadrant(const f32x16 &acc, f32x4 *cells, int a, int b, int lane) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int c = a * 4 + q;
    cells[(b * 8 + c) * 64 + (lane ^ (c << 1))] = f32x4{acc[q * 4], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]};
  }
}
// One 16 x 16 accumulator (columns 16 a, rows 16 b of the 64 x 64 tile) to the same cells.
__device__ __forceinline__ void put_tile16(const f32x4 &acc, f32x4 *cells, int a, int b, int lane) {
  const int r = (b & 1) * 16 + (lane & 15), g4 = lane >> 4, c = a * 2 + (g4 >> 1);
  cells[((b >> 1) * 8 + c) * 64 + (((g4 & 1) * 32 + r) ^ (c << 1))] = acc;
}
template <int PARTS, int STRIDE, int EPI>
__device__ __forceinline__ void finish_tile64(const f32x16 (&acc)[2][2], const GemmArgs &g, f32x4 *xch, int wave, int first,
                                              int rank, int m_tile, int n_tile, int lane, const float *rs_tile) {
  auto put = [&]() {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a) put_quadrant(acc[a][b], xch + wave * 1024, a, b, lane);
  };
  finish_rows<PARTS, PARTS, STRIDE, EPI>(put, g, xch, first, rank, m_tile, n_tile, lane, rs_tile);
}

// ---------------------------------------------------------------------------------------
// 64 x 64 tile, 4 wavefronts, two workgroups per compute unit.  Every wavefront computes the WHOLE
// tile over its own k-tiles (t = wave, wave + 4, ...) from its own 16 KiB LDS slot, so the k-loop
// has no barrier: wait for the slot's loads, read all 16 fragments at once, refill the slot, 16
// MFMAs under which the refill is in flight.  The wavefronts drift apart and fill each other's gaps.
// Measured per launch (back to back, weights cold; before: the 64 x 128 workgroup tile):
//   729 rows, 1152 x 1152: 12.8 -> 7.1 us; 1152 x 4352: 50 -> 18 us; 64 rows, 3456 x 1152: 12.0 -> 6.9.
// Eight wavefronts per workgroup (128 KiB of slots) are level for one tile per compute unit and
// 20-40 % slower from two on.
// ---------------------------------------------------------------------------------------
template <int EPI>
__global__ __launch_bounds__(256, 2) void gemm_wave_kernel(ET_GEMM_FIRST, GemmArgs g) {
  ET_GEMM_TAKE_FIRST(g);
  constexpr int NW = 4;
  extern __shared__ __align__(16) uint16_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, grp = lane >> 5, lrow = lane >> 3, lslot = lane & 7;
  int m0, n0;
  small_tile_of(tiles_m, tiles_n, m0, n0);
  m0 *= 64;
  n0 *= 64;
  const int kt_n = g.K / 64;
  const char *a_base = reinterpret_cast<const char *>(g.A + (size_t)m0 * g.lda) - kOffBias;
  const char *w_base = reinterpret_cast<const char *>(g.W + (size_t)n0 * g.K) - kOffBias;
  uint32_t a_off[8], w_off[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int row = i * 8 + lrow;
    a_off[i] = piece_offset(row, (m0 + row < g.M) ? row : g.M - 1 - m0, g.lda, lslot, i);   // rows past M: the last row again
    w_off[i] = piece_offset(row, row, g.K, lslot, i);
  }
  uint16_t *slot = lds + wave * 8192;                    // 64 rows of A, 64 rows of W, 128 bytes each
  auto issue = [&](int t) {
    const char *ab = a_base + (size_t)t * 128, *wb = w_base + (size_t)t * 128;
    asm volatile("" : "+s"(ab), "+s"(wb));               // scalar base + 32-bit lane offset form of the load
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      asm volatile("" : "+v"(a_off[i]));
      lds_dma16_of4(ab + a_off[i], slot + (i & ~3) * 512, i);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      asm volatile("" : "+v"(w_off[i]));
      lds_dma16_of4(wb + w_off[i], slot + 4096 + (i & ~3) * 512, i);
    }
  };
  float *rs_tile = reinterpret_cast<float *>(lds + NW * 8192);
  RowScale<18> scale;
  const bool scales = EPI != EPI_BIAS_RES && wave == 0;
  if (scales) scale.fetch(g, m0 + lane);
  __builtin_amdgcn_sched_barrier(0);
  if (wave < kt_n) issue(wave);
  if (scales) rs_tile[lane] = scale.value(g);
  f32x16 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
  const int fx = (r32 >> 1) & 7;
  u32x4 fa[4][2], fw[4][2];
  for (int t = wave; t < kt_n; t += NW) {
    wait_vmcnt<0>();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const uint16_t *p = slot + r32 * 64 + ((2 * ks + grp) ^ fx) * 8;
#pragma unroll
      for (int b = 0; b < 2; ++b) fa[ks][b] = *reinterpret_cast<const u32x4 *>(p + b * 2048);
#pragma unroll
      for (int a = 0; a < 2; ++a) fw[ks][a] = *reinterpret_cast<const u32x4 *>(p + 4096 + a * 2048);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the slot has been read: it may be refilled
    __builtin_amdgcn_sched_barrier(0);
    if (t + NW < kt_n) issue(t + NW);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = mfma32(fw[ks][a], fa[ks][b], acc[a][b]);
  }
  // (a wavefront's 16 KiB of the exchange are its own slot: no barrier before they are written)
  finish_tile64<NW, 1, EPI>(acc, g, reinterpret_cast<f32x4 *>(lds), wave, 0, wave, m0, n0, lane, rs_tile);
}

// ---------------------------------------------------------------------------------------
// 64 x 64 tile, 4 wavefronts with a quadrant each, k ascending in one accumulator per element: the order of the persistent
// kernel and of gemm_half_kernel, for the last tile rows of a matrix whose other rows run there (gemm_choice.h).
// Four 16 KiB slots, one barrier per k-tile: all fragments of k-tile t are read at once, under the MFMAs of t - 1,
// and the loads of t + 3 go to the slot that everyone has left.  Bound by the operand path of the compute unit, like the
// kernel above (256 cycles per k-tile; the matrix unit 256 as well).  Measured per launch against 64 x 128 tiles of the
// persistent kernel and against the kernel above, which splits k: 32 rows, 3456 x 1152: 12.7 / 6.9 -> 7.4 us; 288 rows,
// 4352 x 1152: 14.0 / 11.1 -> 10.4; 341 rows, 3584 x 3584: 32.6 / 22.1 -> 21.5; 96 rows, 1152 x 4352: 38.8 / 15.1 -> 18.1.
// (One wavefront per tile: as slow as the 64 x 128 tile, its SIMD's matrix unit takes 1024 cycles per k-tile.)
// ---------------------------------------------------------------------------------------
template <int EPI>
__global__ __launch_bounds__(256, 2) void gemm_strip_kernel(ET_GEMM_FIRST, GemmArgs g) {
  ET_GEMM_TAKE_FIRST(g);
  constexpr int ST = 4, SLOT = 8192;                     // slots; elements of one: 64 rows of A, 64 of W, 128 bytes each
  extern __shared__ __align__(16) uint16_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, r16 = lane & 15, g4 = lane >> 4, lrow = lane >> 3, lslot = lane & 7;
  int m0, n0;
  small_tile_of(tiles_m, tiles_n, m0, n0);
  m0 *= 64;
  n0 *= 64;
  const int kt_n = g.K / 64;
  const char *a_base = reinterpret_cast<const char *>(g.A + (size_t)m0 * g.lda) - kOffBias;
  const char *w_base = reinterpret_cast<const char *>(g.W + (size_t)n0 * g.K) - kOffBias;
  uint32_t a_off[2], w_off[2];                           // 1 KiB loads 2 wave, 2 wave + 1 of either operand
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (wave * 2 + i) * 8 + lrow;
    a_off[i] = piece_offset(row, (m0 + row < g.M) ? row : g.M - 1 - m0, g.lda, lslot, i);   // rows past M: the last row again
    w_off[i] = piece_offset(row, row, g.K, lslot, i);
  }
  auto issue = [&](int slot, int t) {
    uint16_t *as = lds + slot * SLOT + wave * 1024, *ws = as + 4096;
    const char *ab = a_base + (size_t)t * 128, *wb = w_base + (size_t)t * 128;
    asm volatile("" : "+s"(ab), "+s"(wb));
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      asm volatile("" : "+v"(a_off[i]));
      lds_dma16_of4(ab + a_off[i], as, i);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      asm volatile("" : "+v"(w_off[i]));
      lds_dma16_of4(wb + w_off[i], ws, i);
    }
  };
  float *rs_tile = reinterpret_cast<float *>(lds + ST * SLOT);
  RowScale<18> scale;
  const bool scales = EPI != EPI_BIAS_RES && wave == 0;
  if (scales) scale.fetch(g, m0 + lane);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < ST - 1; ++t)
    if (t < kt_n) issue(t, t);
  if (scales) rs_tile[lane] = scale.value(g);
  f32x4 acc[2][2];                                       // [16 columns][16 rows] of the quadrant
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int fx = (r16 >> 1) & 7, a_row = (wm * 32 + r16) * 64, w_row = 4096 + (wn * 32 + r16) * 64;
  u32x4 fa[2][2][2], fw[2][2][2];                        // [buffer][k-step][16 rows or columns]
  auto mfmas = [&](int buf) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = mfma16(fw[buf][ks][a], fa[buf][ks][b], acc[a][b]);
  };
  int slot = 0;
  // k-tile t into fragment buffer `buf`; the MFMAs of t - 1 (the other buffer) follow the reads
  auto step = [&](int buf, int t) {
    if (t + 2 < kt_n) wait_vmcnt<8>();                   // k-tile t has landed (this wavefront's share), two more in flight
    else if (t + 1 < kt_n) wait_vmcnt<4>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();                        // ... everyone's; and everyone has read k-tile t - 1
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    const uint16_t *sp = lds + slot * SLOT;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int ko = ((4 * ks + g4) ^ fx) * 8;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[buf][ks][i] = *reinterpret_cast<const u32x4 *>(sp + a_row + i * 1024 + ko);
        fw[buf][ks][i] = *reinterpret_cast<const u32x4 *>(sp + w_row + i * 1024 + ko);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (t + ST - 1 < kt_n) issue(slot == 0 ? ST - 1 : slot - 1, t + ST - 1);
    __builtin_amdgcn_sched_barrier(0);
    if (t > 0) mfmas(buf ^ 1);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0): the reads have returned before the next barrier
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    slot = slot + 1 == ST ? 0 : slot + 1;
  };
  for (int t = 0; t < kt_n; t += 2) {
    step(0, t);
    if (t + 1 < kt_n) step(1, t + 1);
  }
  if (kt_n & 1) mfmas(0);
  else mfmas(1);
  __syncthreads();                                       // the slots have been read: their room takes the results
  f32x4 *xch = reinterpret_cast<f32x4 *>(lds);
  auto put = [&]() {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) put_tile16(acc[a][b], xch, wn * 2 + a, wm * 2 + b, lane);
  };
  finish_rows<4, 1, 1, EPI>(put, g, xch, 0, wave, m0, n0, lane, rs_tile);
}

// ---------------------------------------------------------------------------------------
// BM x BN tile (128 x 128 or 128 x 64), 8 wavefronts with 64 x 64 wavefront tiles: KG = 2 or 4 groups
// of wavefronts split the contraction, half of the groups (one wavefront per SIMD) reads fragments
// while the other half runs its 16 MFMAs, a barrier after each phase.  Operands are shared inside
// a group, so the load path carries half (128 x 128) or three quarters (128 x 64) of what four
// 64 x 64 tiles would.  A set of k-tiles (one per group of a half) is loaded four phases ahead (three
// stages: two phases).  Measured, one workgroup per compute unit (before: 64 x 128 workgroup tile):
//   729 rows, 3456 x 1152 (162 workgroups of 128 x 128): 14.0 -> 12.0 us; 3276 rows, 1152 x 4352 (234 of 128 x 128): 54 -> 38 us.
// As 128 x 64 it serves odd numbers of k-tiles only (gemm_duo_kernel below the even ones): 2048 rows, 1024 x 1088, 11.0 us; there
// with 1152, 10.1.
// ---------------------------------------------------------------------------------------
template <int BM, int BN>
struct PairShape {
  static constexpr int WPG = (BM / 64) * (BN / 64), KG = 8 / WPG, KH = KG / 2;   // wavefronts per group, groups, groups per half
  static constexpr int TILE = (BM + BN) * 64, SET = KH * TILE;                  // elements of one k-tile, of one stage
  static constexpr int ST = KH == 1 ? 5 : 3;
  static constexpr size_t kLdsBytes = (size_t)ST * SET * 2;
  static_assert(kLdsBytes <= 160 * 1024 && kLdsBytes >= 8 * 16384 + BM * 4, "stages fit, and the exchange and the row scales fit over them");
};

template <int BM, int BN, int EPI>
__global__ __launch_bounds__(512, 1) void gemm_pair_kernel(ET_GEMM_FIRST, GemmArgs g) {
  ET_GEMM_TAKE_FIRST(g);
  using S = PairShape<BM, BN>;
  constexpr int WN = BN / 64, WPG = S::WPG, KH = S::KH, ST = S::ST;
  constexpr int A_BLK = BM / 8 / WPG, W_BLK = BN / 8 / WPG, LOADS = A_BLK + W_BLK;     // 1 KiB loads per wavefront and k-tile
  static_assert(ST % 2 == 1, "the k-tiles of a half are loaded by that half");
  extern __shared__ __align__(16) uint16_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = wave >> 2, gi = (wave & 3) / WPG, wi = (wave & 3) % WPG, wm = wi / WN, wn = wi % WN;
  const int r32 = lane & 31, grp = lane >> 5, lrow = lane >> 3, lslot = lane & 7;
  int m0, n0;
  small_tile_of(tiles_m, tiles_n, m0, n0);
  m0 *= BM;
  n0 *= BN;
  const int kt_n = g.K / 64, n_sets = (kt_n + KH - 1) / KH;
  const char *a_base = reinterpret_cast<const char *>(g.A + (size_t)m0 * g.lda) - kOffBias;
  const char *w_base = reinterpret_cast<const char *>(g.W + (size_t)n0 * g.K) - kOffBias;
  uint32_t a_off[A_BLK], w_off[W_BLK];
#pragma unroll
  for (int i = 0; i < A_BLK; ++i) {
    const int row = (wi * A_BLK + i) * 8 + lrow;
    a_off[i] = piece_offset(row, (m0 + row < g.M) ? row : g.M - 1 - m0, g.lda, lslot, i);
  }
#pragma unroll
  for (int i = 0; i < W_BLK; ++i) {
    const int row = (wi * W_BLK + i) * 8 + lrow;
    w_off[i] = piece_offset(row, row, g.K, lslot, i);
  }
  // Set s = k-tiles s * KH .. of the contraction; sets of even / odd index belong to half 0 / 1.
  auto has = [&](int s) { return s * KH + gi < kt_n; };
  auto issue = [&](int stage, int s) {
    uint16_t *as = lds + stage * S::SET + gi * S::TILE, *ws = as + BM * 64;
    const size_t ko = (size_t)(s * KH + gi) * 128;
    const char *ab = a_base + ko, *wb = w_base + ko;
    asm volatile("" : "+s"(ab), "+s"(wb));
#pragma unroll
    for (int i = 0; i < A_BLK; ++i) {
      asm volatile("" : "+v"(a_off[i]));
      lds_dma16_of4(ab + a_off[i], as + (wi * A_BLK + (i & ~3)) * 512, i);
    }
#pragma unroll
    for (int i = 0; i < W_BLK; ++i) {
      asm volatile("" : "+v"(w_off[i]));
      lds_dma16_of4(wb + w_off[i], ws + (wi * W_BLK + (i & ~3)) * 512, i);
    }
  };
  // (the row scales stay in a register: with five stages LDS has room for them only once the k-loop is over)
  float *rs_tile = reinterpret_cast<float *>(lds + 8 * 8192);
  RowScale<18> scale;
  float my_scale = 1.0f;
  const bool scales = EPI != EPI_BIAS_RES && wave < BM / 64;
  if (scales) scale.fetch(g, m0 + wave * 64 + lane);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < ST - 1; ++s)
    if ((s & 1) == half && has(s)) issue(s, s);
  if (scales) my_scale = scale.value(g);
  asm volatile("" : "+v"(my_scale));

  const int fx = (r32 >> 1) & 7;
  const int a_row = gi * S::TILE + (wm * 64 + r32) * 64, w_row = gi * S::TILE + BM * 64 + (wn * 64 + r32) * 64;
  f32x16 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
  u32x4 fa[4][2], fw[4][2];
  // Set s has landed (this wavefront's share): younger loads in flight are those of set s + 2, which
  // with three stages has not been issued yet when this is asked.
  auto wait_set = [&](int s) {
    if (ST > 3 && has(s + 2)) wait_vmcnt<LOADS>();
    else wait_vmcnt<0>();
  };
  auto phase_end = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // Phase p: half p % 2 reads set p, the other half runs the MFMAs of set p - 1.
  wait_set(half);
  phase_end();
  if (half) phase_end();
  int stage = half, fill = half ? 0 : ST - 1;            // fill: stage of the previous set, read by everyone
  for (int s = half; s < n_sets; s += 2) {
    if (has(s)) {
      const uint16_t *sp = lds + stage * S::SET;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const int ko = ((2 * ks + grp) ^ fx) * 8;
#pragma unroll
        for (int b = 0; b < 2; ++b) fa[ks][b] = *reinterpret_cast<const u32x4 *>(sp + a_row + b * 2048 + ko);
#pragma unroll
        for (int a = 0; a < 2; ++a) fw[ks][a] = *reinterpret_cast<const u32x4 *>(sp + w_row + a * 2048 + ko);
      }
    }
    if (has(s + ST - 1)) issue(fill, s + ST - 1);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    phase_end();
    if (has(s)) {
      __builtin_amdgcn_s_setprio(1);                     // (wave priority: the other half is reading and loading)
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < 2; ++b) acc[a][b] = mfma32(fw[ks][a], fa[ks][b], acc[a][b]);
      __builtin_amdgcn_s_setprio(0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (s + 2 < n_sets) wait_set(s + 2);
    phase_end();
    stage += 2;
    if (stage >= ST) stage -= ST;
    fill += 2;
    if (fill >= ST) fill -= ST;
  }
  // Half 0 has passed 1 + 2 ceil(n_sets / 2) barriers, half 1 two plus 2 floor(n_sets / 2): level them.
  if (half == (n_sets & 1)) phase_end();
  if (scales) rs_tile[wave * 64 + lane] = my_scale;
  finish_tile64<S::KG, WPG, EPI>(acc, g, reinterpret_cast<f32x4 *>(lds), wave, wi, half * KH + gi, m0 + wm * 64, n0 + wn * 64,
                                 lane, rs_tile + wm * 64);
}

// ---------------------------------------------------------------------------------------
// 128 x 64 tile for an even number of k-tiles, 8 wavefronts in two groups that take the k-tiles in turn, each with two LDS
// stages of its own; the four wavefronts of a group as 2 x 2 with 64 x 32 wavefront tiles.  The k-loop is
// gemm_stream_kernel's (quarters of a k-tile, half stages refilled among the MFMAs, two barriers), one k-tile of either
// group at a time, so that the loads are never in a burst.  Bound: the operand path, 24 KiB per k-tile at 58 bytes per
// clock, 424 clocks against 256 of the matrix unit.  Measured per launch against gemm_pair_kernel<128, 64>: 1092 rows, 1152 x
// 1152: 9.7 -> 8.4 us; 1152 x 4352: 26.7 -> 25.7; 686 rows, 2304 x 768: 8.5 -> 7.8.  (As 128 x 128 tiles against
// gemm_pair_kernel<128, 128>: 3276 rows, 1152 x 4352 level, 2184 rows 32.6 -> 34.7: there the operand path, LDS and the
// matrix unit are all about as long.)
// ---------------------------------------------------------------------------------------
struct DuoShape {
  static constexpr int BM = 128, BN = 64, STAGE = (BM + BN) * 64, GROUP = 2 * STAGE;      // elements
  static constexpr int SCALES = 2 * GROUP;                       // the row scales lie behind the stages
  static constexpr size_t kLdsBytes = (size_t)SCALES * 2 + BM * sizeof(float);
  static_assert(kLdsBytes <= 160 * 1024 && SCALES >= 4 * 8192, "stages fit, and the exchange fits over them");
};

template <int EPI>
__global__ __launch_bounds__(512, 1) void gemm_duo_kernel(ET_GEMM_FIRST, GemmArgs g) {
  ET_GEMM_TAKE_FIRST(g);
  using S = DuoShape;
  constexpr int BM = S::BM, BN = S::BN, MS = 4, MH = 2, NS = BN / 32;
  constexpr int WL = BN / 32, AL = 2, LOADS = WL + 2 * AL;       // 1 KiB loads per wavefront: of the weight tile, of either half of the activation tile
  extern __shared__ __align__(16) uint16_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave >> 2, w = wave & 3, wm = w >> 1, wn = w & 1;
  const int r16 = lane & 15, g4 = lane >> 4, lrow = lane >> 3, lslot = lane & 7;
  int m0, n0;
  small_tile_of(tiles_m, tiles_n, m0, n0);
  m0 *= BM;
  n0 *= BN;
  const int units = g.K / 128;
  uint16_t *mem = lds + group * S::GROUP;
  const char *a_base = reinterpret_cast<const char *>(g.A + (size_t)m0 * g.lda + group * 64) - kOffBias;
  const char *w_base = reinterpret_cast<const char *>(g.W + (size_t)n0 * g.K + group * 64) - kOffBias;
  const int a_row0 = wm * 64 + wn * 16;                          // half 0 of the activation rows; half 1: + 32
  uint32_t a_off[2 * AL], w_off[WL];
#pragma unroll
  for (int i = 0; i < 2 * AL; ++i) {
    const int row = a_row0 + (i / AL) * 32 + (i % AL) * 8 + lrow;
    a_off[i] = piece_offset(row, (m0 + row < g.M) ? row : g.M - 1 - m0, g.lda, lslot, i % AL);
  }
#pragma unroll
  for (int i = 0; i < WL; ++i) {
    const int row = (w * WL + i) * 8 + lrow;
    w_off[i] = piece_offset(row, row, g.K, lslot, i);
  }
  int load_u = 0;                                                // next k-tile of this group to be fetched
  auto load_w = [&](int stage, int i0, int i1) {
    const char *b = w_base + (size_t)load_u * 256;
    uint16_t *dst = mem + stage * S::STAGE + BM * 64 + w * WL * 512;
    asm volatile("" : "+s"(b));
#pragma unroll
    for (int i = i0; i < i1; ++i) {
      asm volatile("" : "+v"(w_off[i]));
      lds_dma16_of4(b + w_off[i], dst, i);
    }
  };
  auto load_a = [&](int stage, int h) {
    const char *b = a_base + (size_t)load_u * 256;
    uint16_t *dst = mem + stage * S::STAGE + (a_row0 + h * 32) * 64;
    asm volatile("" : "+s"(b));
#pragma unroll
    for (int i = 0; i < AL; ++i) {
      asm volatile("" : "+v"(a_off[h * AL + i]));
      lds_dma16_of4(b + a_off[h * AL + i], dst, i);
    }
  };
  auto advance = [&]() { load_u = load_u + 1 < units ? load_u + 1 : load_u; };     // (past the end the last one is re-read, unused)
  RowScale<18> scale;
  float my_scale = 1.0f;
  const bool scales = EPI != EPI_BIAS_RES && wave < BM / 64;
  if (scales) scale.fetch(g, m0 + wave * 64 + lane);
  __builtin_amdgcn_sched_barrier(0);
  load_w(0, 0, WL);
  load_a(0, 0);
  load_a(0, 1);
  advance();
  load_w(1, 0, WL);
  load_a(1, 0);

  const int fx = (r16 >> 1) & 7;
  int a_addr[2], w_addr[2];                                      // element offsets of this lane's fragments, by k-step
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int ko = ((4 * ks + g4) ^ fx) * 8;
    a_addr[ks] = (wm * 64 + r16) * 64 + ko;
    w_addr[ks] = BM * 64 + (wn * (BN / 2) + r16) * 64 + ko;
  }
  f32x4 acc[NS][MS];
#pragma unroll
  for (int a = 0; a < NS; ++a)
#pragma unroll
    for (int b = 0; b < MS; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 fw[2][NS], fa[2][MH];
  auto read_w = [&](int stage, int ks) {
    const uint16_t *p = mem + stage * S::STAGE + w_addr[ks];
#pragma unroll
    for (int a = 0; a < NS; ++a) fw[ks][a] = *reinterpret_cast<const u32x4 *>(p + a * 1024);
  };
  auto read_a = [&](int buf, int stage, int h, int ks) {
    const uint16_t *p = mem + stage * S::STAGE + a_addr[ks] + h * 32 * 64;
#pragma unroll
    for (int b = 0; b < MH; ++b) fa[buf][b] = *reinterpret_cast<const u32x4 *>(p + b * 1024);
  };
  auto mfma_quarter = [&](int buf, int h, int ks) {
#pragma unroll
    for (int b = 0; b < MH; ++b)
#pragma unroll
      for (int a = 0; a < NS; ++a) acc[a][h * MH + b] = mfma16(fw[ks][a], fa[buf][b], acc[a][h * MH + b]);
  };
  auto meet = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  wait_vmcnt<LOADS>();
  __builtin_amdgcn_sched_barrier(0);
  if (scales) my_scale = scale.value(g);
  asm volatile("" : "+v"(my_scale));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_w(0, 0);
  read_a(0, 0, 0, 0);
  int stage = 0;
  for (int u = 0; u < units; ++u) {
    read_a(1, stage, 0, 1);
    read_w(stage, 1);
    load_a(stage ^ 1, 1);
    mfma_quarter(0, 0, 0);
    mfma_between<NS * MH - AL, AL, NS * MH>();
    __builtin_amdgcn_sched_barrier(0);
    advance();
    wait_vmcnt<LOADS>();                                         // the lower rows of this k-tile have landed
    meet();                                                      // ... everyone's; weights and upper rows have been read
    read_a(0, stage, 1, 0);
    load_w(stage, 0, WL / 2);
    mfma_quarter(1, 0, 1);
    mfma_between<MH, WL / 2, NS * MH>();
    __builtin_amdgcn_sched_barrier(0);
    read_a(1, stage, 1, 1);
    load_w(stage, WL / 2, WL);
    mfma_quarter(0, 1, 0);
    mfma_between<MH, WL / 2, NS * MH>();
    __builtin_amdgcn_sched_barrier(0);
    wait_vmcnt<LOADS - AL>();                                    // the next k-tile's weights and upper rows have landed
    meet();                                                      // ... everyone's; the lower rows have been read
    read_w(stage ^ 1, 0);
    read_a(0, stage ^ 1, 0, 0);
    load_a(stage, 0);
    mfma_quarter(1, 1, 1);
    mfma_between<NS * MH - AL, AL, NS * MH>();
    __builtin_amdgcn_sched_barrier(0);
    stage ^= 1;
  }
  wait_vmcnt<0>();                                               // (the loads past the end)
  __syncthreads();                                               // the stages take the partial sums
  float *rs_tile = reinterpret_cast<float *>(lds + S::SCALES);
  if (scales) rs_tile[wave * 64 + lane] = my_scale;
  f32x4 *xch = reinterpret_cast<f32x4 *>(lds);
  const int tile = group * 2 + wm;                               // the 64 x 64 partial tile that this wavefront writes half of
  auto put = [&]() {
#pragma unroll
    for (int a = 0; a < NS; ++a)
#pragma unroll
      for (int b = 0; b < MS; ++b) put_tile16(acc[a][b], xch + tile * 1024, wn * NS + a, b, lane);
  };
  finish_rows<4, 2, 2, EPI>(put, g, xch, wm, group * 2 + wn, m0 + wm * 64, n0, lane, rs_tile + wm * 64);
}

// ---------------------------------------------------------------------------------------
// 256 x 128 tile, 8 wavefronts with 64 x 64 wavefront tiles, one k-tile stream for all: half 0 owns the
// upper 128 rows, half 1 the lower ones.  The halves alternate as above (phase 2 u: half 0 reads
// k-tile u while half 1 runs the MFMAs of u - 1; phase 2 u + 1: the other way round), so the load path
// carries 48 KiB per 1024 cycles of the matrix unit instead of 32 per 512.  Three stages of 48 KiB; a
// stage is refilled when both halves have read it, three phases before it is needed again.  Pays where
// this tiling makes one full round (or two) and 128 x 128 a started second one: 5832 rows, 1152 x 4352
// (207 workgroups): 64 -> 59 us; 13122 rows: 131 -> 124 us; 1456 rows, 3456 x 1152: 20 -> 18.8 us.
// ---------------------------------------------------------------------------------------
template <int EPI>
__global__ __launch_bounds__(512, 1) void gemm_half_kernel(ET_GEMM_FIRST, GemmArgs g) {
  ET_GEMM_TAKE_FIRST(g);
  constexpr int BM = 256, BN = 128, ST = 3, STAGE = (BM + BN) * 64;
  constexpr int A_BLK = BM / 64, W_BLK = BN / 64, LOADS = A_BLK + W_BLK;      // 1 KiB loads per wavefront and k-tile
  extern __shared__ __align__(16) uint16_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = wave >> 2, wm = wave >> 1, wn = wave & 1;
  const int r16 = lane & 15, g4 = lane >> 4, lrow = lane >> 3, lslot = lane & 7;
  int m0, n0;
  small_tile_of(tiles_m, tiles_n, m0, n0);
  m0 *= BM;
  n0 *= BN;
  const int kt_n = g.K / 64;
  const char *a_base = reinterpret_cast<const char *>(g.A + (size_t)m0 * g.lda) - kOffBias;
  const char *w_base = reinterpret_cast<const char *>(g.W + (size_t)n0 * g.K) - kOffBias;
  uint32_t a_off[A_BLK], w_off[W_BLK];
#pragma unroll
  for (int i = 0; i < A_BLK; ++i) {
    const int row = (wave * A_BLK + i) * 8 + lrow;
    a_off[i] = piece_offset(row, (m0 + row < g.M) ? row : g.M - 1 - m0, g.lda, lslot, i);
  }
#pragma unroll
  for (int i = 0; i < W_BLK; ++i) {
    const int row = (wave * W_BLK + i) * 8 + lrow;
    w_off[i] = piece_offset(row, row, g.K, lslot, i);
  }
  auto issue = [&](int stage, int t) {
    uint16_t *as = lds + stage * STAGE + wave * A_BLK * 512, *ws = lds + stage * STAGE + BM * 64 + wave * W_BLK * 512;
    const char *ab = a_base + (size_t)t * 128, *wb = w_base + (size_t)t * 128;
    asm volatile("" : "+s"(ab), "+s"(wb));
#pragma unroll
    for (int i = 0; i < A_BLK; ++i) {
      asm volatile("" : "+v"(a_off[i]));
      lds_dma16_of4(ab + a_off[i], as, i);
    }
#pragma unroll
    for (int i = 0; i < W_BLK; ++i) {
      asm volatile("" : "+v"(w_off[i]));
      lds_dma16_of4(wb + w_off[i], ws, i);
    }
  };
  float *rs_tile = reinterpret_cast<float *>(lds + 3 * STAGE);
  RowScale<18> scale;
  const bool scales = EPI != EPI_BIAS_RES && wave < BM / 64;
  if (scales) scale.fetch(g, m0 + wave * 64 + lane);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < ST - 1; ++t)
    if (t < kt_n) issue(t, t);
  if (scales) rs_tile[wave * 64 + lane] = scale.value(g);
  const int fx = (r16 >> 1) & 7;
  const int a_row = (wm * 64 + r16) * 64, w_row = BM * 64 + (wn * 64 + r16) * 64;
  f32x4 acc[4][4];                                       // [16 columns][16 rows] of the wavefront tile
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 fa[2][4], fw[2][4];
  // k-tile t has landed (this wavefront's share); the loads of t + 1 may still be in flight
  auto wait_tile = [&](int t) {
    if (t + 1 < kt_n) wait_vmcnt<LOADS>();
    else wait_vmcnt<0>();
  };
  auto phase_end = [&]() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  wait_tile(0);
  phase_end();
  if (half) phase_end();
  int stage = 0;
  for (int t = 0; t < kt_n; ++t) {
    const uint16_t *sp = lds + stage * STAGE;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int ko = ((4 * ks + g4) ^ fx) * 8;
#pragma unroll
      for (int b = 0; b < 4; ++b) fa[ks][b] = *reinterpret_cast<const u32x4 *>(sp + a_row + b * 1024 + ko);
#pragma unroll
      for (int a = 0; a < 4; ++a) fw[ks][a] = *reinterpret_cast<const u32x4 *>(sp + w_row + a * 1024 + ko);
    }
    // (both halves have read k-tile t - 1 by now: its stage takes t + 2)
    if (t + ST - 1 < kt_n) issue(stage == 0 ? ST - 1 : stage - 1, t + ST - 1);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (half && t + 1 < kt_n) wait_tile(t + 1);
    phase_end();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mfma16(fw[ks][a], fa[ks][b], acc[a][b]);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    if (!half && t + 1 < kt_n) wait_tile(t + 1);
    phase_end();
    stage = (stage + 1 == ST) ? 0 : stage + 1;
  }
  if (!half) phase_end();
  f32x4 *xch = reinterpret_cast<f32x4 *>(lds);
  auto put = [&]() {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) put_tile16(acc[a][b], xch + wave * 1024, a, b, lane);
  };
  finish_rows<1, 1, 1, EPI>(put, g, xch, wave, 0, m0 + wm * 64, n0 + wn * 64, lane, rs_tile + wm * 64);
}

}  // namespace

template <void (*KERN)(ET_GEMM_FIRST, GemmArgs)>
static int launch_small(const GemmArgs &g, hipStream_t s, int bm, int bn, int threads, size_t lds_bytes) {
  if (int rc = allow_lds<KERN>(lds_bytes)) return rc;
  const int tiles_m = (g.M + bm - 1) / bm, tiles_n = (g.n_store + bn - 1) / bn;
  hipLaunchKernelGGL(KERN, dim3(tiles_m * tiles_n), dim3(threads), lds_bytes, s, ET_GEMM_GIVE_FIRST(g), g);
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_gemm_wave(const GemmArgs &g, hipStream_t s) {
  constexpr size_t kWaveLds = 4 * 16384 + 64 * 4;        // slots and row scales
  switch (g.epilogue) {
    case EPI_BIAS: return launch_small<gemm_wave_kernel<EPI_BIAS>>(g, s, 64, 64, 256, kWaveLds);
    case EPI_BIAS_GELU: return launch_small<gemm_wave_kernel<EPI_BIAS_GELU>>(g, s, 64, 64, 256, kWaveLds);
    case EPI_BIAS_RES: return launch_small<gemm_wave_kernel<EPI_BIAS_RES>>(g, s, 64, 64, 256, kWaveLds);
    default: set_error("unknown epilogue %d", g.epilogue); return ET_ERR_INVALID_ARG;
  }
}

int launch_gemm_strip(const GemmArgs &g, hipStream_t s) {
  constexpr size_t bytes = 4 * 16384 + 64 * 4;           // slots and row scales
  switch (g.epilogue) {
    case EPI_BIAS: return launch_small<gemm_strip_kernel<EPI_BIAS>>(g, s, 64, 64, 256, bytes);
    case EPI_BIAS_GELU: return launch_small<gemm_strip_kernel<EPI_BIAS_GELU>>(g, s, 64, 64, 256, bytes);
    case EPI_BIAS_RES: return launch_small<gemm_strip_kernel<EPI_BIAS_RES>>(g, s, 64, 64, 256, bytes);
    default: set_error("unknown epilogue %d", g.epilogue); return ET_ERR_INVALID_ARG;
  }
}

template <int BM, int BN>
static int launch_pair_shape(const GemmArgs &g, hipStream_t s) {
  constexpr size_t bytes = PairShape<BM, BN>::kLdsBytes;
  switch (g.epilogue) {
    case EPI_BIAS: return launch_small<gemm_pair_kernel<BM, BN, EPI_BIAS>>(g, s, BM, BN, 512, bytes);
    case EPI_BIAS_GELU: return launch_small<gemm_pair_kernel<BM, BN, EPI_BIAS_GELU>>(g, s, BM, BN, 512, bytes);
    case EPI_BIAS_RES: return launch_small<gemm_pair_kernel<BM, BN, EPI_BIAS_RES>>(g, s, BM, BN, 512, bytes);
    default: set_error("unknown epilogue %d", g.epilogue); return ET_ERR_INVALID_ARG;
  }
}
int launch_gemm_half(const GemmArgs &g, hipStream_t s) {
  constexpr size_t bytes = 3 * (256 + 128) * 64 * 2 + 256 * 4;      // stages and row scales
  switch (g.epilogue) {
    case EPI_BIAS: return launch_small<gemm_half_kernel<EPI_BIAS>>(g, s, 256, 128, 512, bytes);
    case EPI_BIAS_GELU: return launch_small<gemm_half_kernel<EPI_BIAS_GELU>>(g, s, 256, 128, 512, bytes);
    case EPI_BIAS_RES: return launch_small<gemm_half_kernel<EPI_BIAS_RES>>(g, s, 256, 128, 512, bytes);
    default: set_error("unknown epilogue %d", g.epilogue); return ET_ERR_INVALID_ARG;
  }
}
static int launch_duo(const GemmArgs &g, hipStream_t s) {
  switch (g.epilogue) {
    case EPI_BIAS: return launch_small<gemm_duo_kernel<EPI_BIAS>>(g, s, 128, 64, 512, DuoShape::kLdsBytes);
    case EPI_BIAS_GELU: return launch_small<gemm_duo_kernel<EPI_BIAS_GELU>>(g, s, 128, 64, 512, DuoShape::kLdsBytes);
    case EPI_BIAS_RES: return launch_small<gemm_duo_kernel<EPI_BIAS_RES>>(g, s, 128, 64, 512, DuoShape::kLdsBytes);
    default: set_error("unknown epilogue %d", g.epilogue); return ET_ERR_INVALID_ARG;
  }
}
int launch_gemm_pair128(const GemmArgs &g, hipStream_t s) { return launch_pair_shape<128, 128>(g, s); }
int launch_gemm_pair64(const GemmArgs &g, hipStream_t s) { return g.K % 128 == 0 ? launch_duo(g, s) : launch_pair_shape<128, 64>(g, s); }

}  // namespace et
