// Attention-received token scores (Sec. 3.3 / Alg. 2: the "per-token attention scores" A that the
// selection ranks).  The paper does not define how a per-token score is taken from the attention
// maps; this build's reading: score[f][j] = mean over heads h and queries i of
// softmax_h(Q K^T / sqrt(hd))[i][j] inside frame f, i.e. the attention token j RECEIVES.
//
// Input: the q and k thirds of a [frames * L, 3 D] bf16 activation (every frame has L rows).  Frames
// whose keys fit the registers of one workgroup (attn_score_kernel) are done in one pass over the
// queries; longer ones in two:
//   1. row statistics: for every (frame, head, query) the maximum m of the scaled logits (log2
//      domain) and 1 / sum_j exp2(s_j - m), by an online pass over 32-key tiles;
//   2. column sums: for every (frame, head, key) the sum over queries of exp2(s - m_i) / l_i,
//      accumulated in a fixed order inside one wavefront.
// Either way the per-head sums meet in attn_score_reduce_kernel in a fixed order, divided by
// heads * L (no atomics anywhere: bit-reproducible).  The two-pass kernels load their fragments
// straight from global memory (16-byte pieces of q / k rows); the head dimension is padded to a
// multiple of 16 with zero fragments.
#include <type_traits>

#include "mfma_common.h"

namespace et {

namespace {

constexpr int kScoreWaves = 4;
constexpr int kMaxKSteps = 8;        // head_dim <= 128

// 16-byte piece `chunk` (8 head dimensions) of a q / k row; zero past the head dimension.
__device__ __forceinline__ u32x4 load_piece(const uint16_t *row, int chunk, int head_dim) {
  if (chunk * 8 < head_dim) return *reinterpret_cast<const u32x4 *>(row + chunk * 8);
  return u32x4{0u, 0u, 0u, 0u};
}

// ---------------------------------------------------------------------------------------
// One pass.  A workgroup of 8 wavefronts owns one (frame, head) and a contiguous share of the 32-query
// blocks; wavefront w owns the NB 32-key blocks w, w + 8, ..., whose K fragments stay in registers.
// Per query block every wavefront computes S^T = K Q^T for its keys (the query on the accumulator's
// lane axis), exponentiates against its OWN maximum, and leaves (maximum, sum) per query in LDS; after one barrier each
// knows the factor exp2(m_w - m) / l that turns its exponentials into probabilities and adds them to its column sums, which
// stay in registers to the end: one exponential and one logit per (query, key) instead of two.  (The reference 0 in place of the
// maxima, while the sums stay within 2^+-60, saves 4 us of the 94 below and costs precision where logits are large: up to 14 %
// larger errors for standard normal q and k times 1.5 to 3; and a call of large logits has its blocks computed twice, 97 -> 165 us.)
// The query blocks come to LDS as fragments (KSTEPS * 1 KiB) by direct loads, three blocks ahead.
// Bound by the vector unit: per 16 accumulator values 16 maxima, fma, exponentials (at half rate), additions and fma, 350 to 380
// clocks against 160 of the matrix unit, which works on the next block in between; at 729 tokens a tenth of a workgroup's time is its
// keys' way from memory (one compute unit takes 40 KB per us), the rest the loop.  K and Q are read once per workgroup.
// Measured against the two passes (all launches of a call): 32 frames x 16 heads x 729 tokens of 72: 373 -> 94 us; 8 x
// 16 x 729: 114 -> 41; one frame: 63 -> 34; 32 x 12 x 196 of 64: 38 -> 21.
// ---------------------------------------------------------------------------------------
constexpr int kPassWaves = 8;
constexpr int kMaxSplits = 3;        // shares of a (frame, head)'s queries: their partial sums take the room of the two-pass statistics

// Sum over each row of 16 lanes, in all of them.
template <int CTRL>
__device__ __forceinline__ float dpp_rotated(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_sum(float v) {       // row_ror:8, 4, 2, 1
  return dpp_rotated<0x121>(dpp_rotated<0x122>(dpp_rotated<0x124>(dpp_rotated<0x128>(v))));
}
// {this lane's value, the value of the same query in the other lane half}, in half order
__device__ __forceinline__ float2 both_halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int KSTEPS, int NB>
__global__ __launch_bounds__(kPassWaves * 64, NB == 1 ? 4 : 2) void attn_score_kernel(
    const uint16_t *__restrict__ qkv, int L, int D, int n_heads, int head_dim, float scale_log2, int splits,
    float *__restrict__ partial) {
  constexpr int RING = 4;                                // query blocks in LDS
  __shared__ __align__(16) uint16_t qs[RING][KSTEPS * 512];          // fragments, 1 KiB each, 16 bytes per lane
  __shared__ float2 ex[2][kPassWaves][32];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, grp = lane >> 5;
  // neighbouring workgroups (shares of a head, heads of a frame) go to one XCD
  const int total = gridDim.x, per = total / 8, rem = total % 8, xcd = blockIdx.x % 8;
  const int v = xcd * per + (xcd < rem ? xcd : rem) + blockIdx.x / 8;
  const int sp = v % splits, h = (v / splits) % n_heads, f = v / (splits * n_heads);
  const int n_qb = (L + 31) / 32, qb0 = n_qb * sp / splits, qb1 = n_qb * (sp + 1) / splits;
  const size_t row_stride = (size_t)3 * D;
  const uint16_t *head = qkv + (size_t)f * L * row_stride + (size_t)h * head_dim;

  // The fragments of a query block come by direct loads, one per wavefront, three blocks ahead; nothing else is loaded in
  // the loop and the waits are explicit.  (Through registers, one block ahead, the loop waited for memory: 2 us per block.)
  // Rows past the frame are its last one; pieces past head_dim are taken from inside the row and zeroed behind LDS.
  const int n_pieces = head_dim / 8;
  const bool loads = wave < KSTEPS, pad_last = n_pieces < 2 * KSTEPS;
  const uint32_t piece_off = (uint32_t)min(2 * wave + grp, n_pieces - 1) * 16u;
  const uint32_t off_full = (uint32_t)r32 * (uint32_t)row_stride * 2u + piece_off;
  const uint32_t off_last = (uint32_t)min(r32, L - 1 - (n_qb - 1) * 32) * (uint32_t)row_stride * 2u + piece_off;
  auto issue = [&](int qb) {
    const int block = min(qb, n_qb - 1);                 // (past the share's end: loaded and not used)
    const uint64_t base = (uint64_t)(uintptr_t)(head + (size_t)block * 32 * row_stride);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)base), hi = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
    if (loads)
      lds_dma16_untracked(reinterpret_cast<const uint16_t *>((uintptr_t)((uint64_t)hi << 32 | lo)), block == n_qb - 1 ? off_last : off_full,
                          qs[(qb - qb0) % RING] + wave * 512);
  };
  u32x4 kf[NB][KSTEPS];
#pragma unroll
  for (int i = 0; i < RING - 1; ++i) issue(qb0 + i);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int k = (wave + b * kPassWaves) * 32 + r32;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      kf[b][ks] = u32x4{0u, 0u, 0u, 0u};
      if (k < L) kf[b][ks] = load_piece(head + (size_t)k * row_stride + D, 2 * ks + grp, head_dim);
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0), known to the compiler: it has no waits for the keys in the loop
  const bool any_key = wave * 32 < L;                    // wave-uniform; a wavefront without keys only keeps the barriers
  f32x16 acc[NB];
  float col[NB][16];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) col[b][i] = 0.f;
  auto query = [&](int slot, int ks) {
    u32x4 q = *reinterpret_cast<const u32x4 *>(qs[slot] + ks * 512 + lane * 8);
    if (ks == KSTEPS - 1 && pad_last && grp) q = u32x4{0u, 0u, 0u, 0u};
    return q;
  };
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // Query block qb, whose logits are in acc; leaves those of the next one there if the share has MORE.  (The last block's matrix work on
  // a next one, for nothing: shares of one block 4.1-4.3 us per launch, without it 3.8-4.0; 32 frames of 60 tokens, 12 heads, 6.3 -> 6.1.)
  auto block = [&](auto more, int qb, int buf) {
    constexpr bool MORE = decltype(more)::value;
    float p[NB][16];
    float m = -INFINITY, l = 0.f;
    const int next = (qb + 1 - qb0) % RING;
    u32x4 q_now;
    auto step = [&](int b, int ks) {                     // of the next block's logits of key block b
      if (!MORE) return;
      acc[b] = mfma32(kf[b][ks], q_now, ks ? acc[b] : zero16);
      q_now = query(next, ks + 1 < KSTEPS ? ks + 1 : 0);
    };
    if (any_key) {
      if (MORE) q_now = query(next, 0);
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const int k0 = (wave + b * kPassWaves) * 32;
        if (k0 + 32 > L) {                               // (wave-uniform) keys past the frame
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (k0 + (i / 4) * 8 + 4 * grp + (i % 4) >= L) acc[b][i] = -INFINITY;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) m = fmaxf(m, acc[b][i]);
      }
      // The wavefront's reference is a whole number, so the factor between two wavefronts' references is an
      // exact power of two.
      const float2 mm = both_halves(m);
      m = ceilf(fmaxf(mm.x, mm.y) * scale_log2);         // (scale_log2 > 0: the order is kept)
      const float m_ref = m == -INFINITY ? 0.f : m;      // no finite logit here: exponentials are 0, not NaN
      // The matrix unit works on the next block under the exponentials: of key block b - 1 as soon as its logits are used.
      float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
          __builtin_amdgcn_sched_barrier(0);
          if (b > 0) step(b - 1, ks);
#pragma unroll
          for (int i = 16 * ks / KSTEPS; i < 16 * (ks + 1) / KSTEPS; ++i) {
            p[b][i] = __builtin_amdgcn_exp2f(fmaf(acc[b][i], scale_log2, -m_ref));
            part[i & 3] += p[b][i];
          }
        }
      __builtin_amdgcn_sched_barrier(0);
      const float2 ll = both_halves((part[0] + part[1]) + (part[2] + part[3]));
      l = ll.x + ll.y;
    }
    if (grp == 0) ex[buf][wave][r32] = make_float2(m, l);
    wait_vmcnt<RING - 3>();                              // the fragment of the block after the next has landed
    __syncthreads();
    // (ex[buf] is written again two blocks on, behind the next barrier; a query block's room is loaded again behind the
    // barrier that follows its last read)
    if (any_key) {
      float2 o[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) o[w] = ex[buf][grp * 4 + w][r32];    // each lane half combines four wavefronts
      const float2 mm = both_halves(fmaxf(fmaxf(o[0].x, o[1].x), fmaxf(o[2].x, o[3].x)));
      const float mt = fmaxf(mm.x, mm.y);
      float lt = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) lt += o[w].y * __builtin_amdgcn_exp2f(o[w].x - mt);
      const float2 ll = both_halves(lt);
      const float fac = qb * 32 + r32 < L ? __builtin_amdgcn_exp2f(m - mt) / (ll.x + ll.y) : 0.f;      // queries past L add nothing
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) {
        __builtin_amdgcn_sched_barrier(0);
        step(NB - 1, ks);
#pragma unroll
        for (int i = NB * 16 * ks / KSTEPS; i < NB * 16 * (ks + 1) / KSTEPS; ++i) col[i / 16][i % 16] = fmaf(p[i / 16][i % 16], fac, col[i / 16][i % 16]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  __syncthreads();
  if (any_key) {
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
      const u32x4 q = query(0, ks);
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[b] = mfma32(kf[b][ks], q, ks ? acc[b] : zero16);
    }
  }
  int qb = qb0, buf = 0;
  for (; qb + 1 < qb1; ++qb, buf ^= 1) {
    issue(qb + RING - 1);
    block(std::true_type(), qb, buf);
  }
  block(std::false_type(), qb, buf);
  wait_vmcnt<0>();                                       // (the loads past the end)
  // Sums over the 32 queries of each lane half.  Two values of a key block share a register after the first exchange
  // (accumulator rows i in the even, i + 8 in the odd rows of 16 lanes); lane j of a row then stores the j-th sum.
  float *dst = partial + (((size_t)f * n_heads + h) * splits + sp) * L;
  const int j = lane & 15, odd_row = (lane >> 4) & 1;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    float mine = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(col[b][i]), __float_as_uint(col[b][i + 8]), false, false);
      const float c = row_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
      mine = j == i ? c : mine;
    }
    const int k = (wave + b * kPassWaves) * 32 + odd_row * 16 + (j >> 2) * 8 + 4 * grp + (j & 3);
    if (j < 8 && k < L) dst[k] = mine;
  }
}

// Pass 1.  grid (ceil(L / 128), heads, frames), 4 wavefronts, 32 queries per wavefront.
// S^T = K Q^T: keys on the accumulator's row axis, the query on its lane axis, so the running
// maximum and sum are per-lane scalars; the two lane halves see different keys and are combined
// at the end.  stats[(f * H + h) * L + i] = (m_i, 1 / l_i).
template <int KSTEPS>
__global__ __launch_bounds__(kScoreWaves * 64) void attn_rowstats_kernel(
    const uint16_t *__restrict__ qkv, int L, int D, int n_heads, int head_dim, float scale_log2,
    float2 *__restrict__ stats) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r32 = lane & 31, grp = lane >> 5;
  const int h = blockIdx.y, f = blockIdx.z;
  const int q0 = (blockIdx.x * kScoreWaves + wave) * 32;
  if (q0 >= L) return;                                         // wave-uniform
  const size_t row_stride = (size_t)3 * D;
  const uint16_t *frame = qkv + (size_t)f * L * row_stride + (size_t)h * head_dim;
  const int qi = q0 + r32 < L ? q0 + r32 : L - 1;              // clamped: rows past L are computed and dropped
  u32x4 qf[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) qf[ks] = load_piece(frame + (size_t)qi * row_stride, 2 * ks + grp, head_dim);

  float m = -INFINITY, l = 0.f;
  for (int k0 = 0; k0 < L; k0 += 32) {
    const int kj = k0 + r32 < L ? k0 + r32 : L - 1;
    const uint16_t *krow = frame + (size_t)kj * row_stride + D;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) acc = mfma32(load_piece(krow, 2 * ks + grp, head_dim), qf[ks], acc);
    float sv[16], tmax = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int key = k0 + (i / 4) * 8 + 4 * grp + (i % 4);
      sv[i] = key < L ? acc[i] * scale_log2 : -INFINITY;
      tmax = fmaxf(tmax, sv[i]);
    }
    if (tmax > m) {                                            // (a tile of this half with no valid key leaves m alone)
      l *= __builtin_amdgcn_exp2f(m - tmax);                   // exp2(-inf) = 0 on the first tile
      m = tmax;
    }
    if (m > -INFINITY) {
#pragma unroll
      for (int i = 0; i < 16; ++i) l += __builtin_amdgcn_exp2f(sv[i] - m);
    }
  }
  const float m_o = __shfl_xor(m, 32), l_o = __shfl_xor(l, 32);
  const float mt = fmaxf(m, m_o);
  const float lt = (m > -INFINITY ? l * __builtin_amdgcn_exp2f(m - mt) : 0.f) +
                   (m_o > -INFINITY ? l_o * __builtin_amdgcn_exp2f(m_o - mt) : 0.f);
  if (grp == 0 && q0 + r32 < L) stats[((size_t)f * n_heads + h) * L + q0 + r32] = make_float2(mt, 1.0f / lt);
}

// Pass 2.  grid (ceil(L / 128), heads, frames), 4 wavefronts, 32 keys per wavefront; loops over
// 32-query tiles.  S = Q K^T: queries on the accumulator's row axis, the key on its lane axis.
// partial[(f * H + h) * L + j] = sum over queries i of softmax_h[i][j].
template <int KSTEPS>
__global__ __launch_bounds__(kScoreWaves * 64) void attn_colsum_kernel(
    const uint16_t *__restrict__ qkv, int L, int D, int n_heads, int head_dim, float scale_log2,
    const float2 *__restrict__ stats, float *__restrict__ partial) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r32 = lane & 31, grp = lane >> 5;
  const int h = blockIdx.y, f = blockIdx.z;
  const int k0 = (blockIdx.x * kScoreWaves + wave) * 32;       // (a wavefront past the last key computes on clamped rows and stores nothing)
  const size_t row_stride = (size_t)3 * D;
  const uint16_t *head = qkv + (size_t)f * L * row_stride + (size_t)h * head_dim;
  const float2 *st = stats + ((size_t)f * n_heads + h) * L;
  // the four wavefronts see the same 32 queries: their (m, 1/l) pairs go through LDS once per tile
  // instead of 16 scattered loads per lane; two buffers, so one barrier per tile is enough
  __shared__ float2 qstat[2][32];
  const int kj = k0 + r32 < L ? k0 + r32 : L - 1;
  u32x4 kf[KSTEPS];
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) kf[ks] = load_piece(head + (size_t)kj * row_stride + D, 2 * ks + grp, head_dim);
  float col = 0.f;
  int buf = 0;
  for (int q0 = 0; q0 < L; q0 += 32, buf ^= 1) {
    if (threadIdx.x < 32) {
      const int q = q0 + (int)threadIdx.x;
      qstat[buf][threadIdx.x] = q < L ? st[q] : make_float2(INFINITY, 0.f);  // rows past L: exp2(-inf) * 0 = 0
    }
    const int qi = q0 + r32 < L ? q0 + r32 : L - 1;
    const uint16_t *qrow = head + (size_t)qi * row_stride;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) acc = mfma32(load_piece(qrow, 2 * ks + grp, head_dim), kf[ks], acc);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float2 ml = qstat[buf][(i / 4) * 8 + 4 * grp + (i % 4)];
      col += __builtin_amdgcn_exp2f(acc[i] * scale_log2 - ml.x) * ml.y;
    }
  }
  col += __shfl_xor(col, 32);
  if (grp == 0 && k0 + r32 < L) partial[((size_t)f * n_heads + h) * L + k0 + r32] = col;
}

// score[f][j] = (sum over heads and their shares of partial) / (heads * L); parts = heads * shares.  Eight sums over
// every eighth part, then a tree: eight loads in flight per lane, and the error of a short sum.
__global__ __launch_bounds__(256) void attn_score_reduce_kernel(const float *__restrict__ partial, int n_frames,
                                                                int L, int n_heads, int parts, float *__restrict__ score) {
  const int idx = blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n_frames * L) return;
  const int f = idx / L, j = idx - f * L;
  const float *p = partial + (size_t)f * parts * L + j;
  float t[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int h = 0; h < parts; h += 8)
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (h + u < parts) t[u] += p[(size_t)(h + u) * L];
#pragma unroll
  for (int w = 4; w > 0; w >>= 1)
#pragma unroll
    for (int u = 0; u < w; ++u) t[u] += t[u + w];
  score[idx] = t[0] / ((float)n_heads * (float)L);
}

}  // namespace

// row statistics (float2) followed by the per-head column sums (float)
size_t attention_scores_workspace_bytes(int n_frames, int L, int n_heads) {
  return (size_t)n_frames * n_heads * L * (sizeof(float2) + sizeof(float));
}

int launch_attention_scores(const uint16_t *qkv, int n_frames, int L, int n_heads, int head_dim, void *stats_ws,
                            float *score, hipStream_t s) {
  if (n_frames <= 0 || L <= 0) return ET_OK;
  ET_REQUIRE(head_dim % 8 == 0 && head_dim >= 8 && head_dim <= kMaxKSteps * 16,
             "head_dim = %d must be a multiple of 8 in [8, %d]", head_dim, kMaxKSteps * 16);
  const int D = n_heads * head_dim;
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)head_dim);
  const int ksteps = (head_dim + 15) / 16;
  const dim3 reduce_grid((n_frames * L + 255) / 256);
  // One pass while a workgroup's registers hold the frame's K fragments, 3 blocks of 32 keys per wavefront
  // (2 above head_dim 96), and the one-dimensional grid stays far below its limit.  Its direct loads to LDS need rows at multiples
  // of 16 bytes; a caller's tensor that begins elsewhere goes by ordinary loads, which the hardware takes at any address.
  if (reinterpret_cast<uintptr_t>(qkv) % 16 == 0 && L <= 32 * kPassWaves * (ksteps <= 6 ? 3 : 2) && n_frames <= 65535 && n_heads <= 65535 && (long)n_frames * n_heads <= (1L << 20)) {
    const int nb = (L + 32 * kPassWaves - 1) / (32 * kPassWaves), n_qb = (L + 31) / 32;
    // Shares per (frame, head): the fewest query blocks on the busiest compute unit, a workgroup's own start
    // (K fragments from memory, reduction of the column sums) counted as two.
    int splits = 1;
    long best = -1;
    for (int sp = 1; sp <= kMaxSplits && sp <= n_qb; ++sp) {
      const long slots = device_cus(), wgs = (long)n_frames * n_heads * sp;
      const long cost = ((wgs + slots - 1) / slots) * ((n_qb + sp - 1) / sp + 2);
      if (best < 0 || cost < best) { best = cost; splits = sp; }
    }
    float *partial = static_cast<float *>(stats_ws);
    const dim3 grid((unsigned)(n_frames * n_heads * splits)), block(kPassWaves * 64);
#define ET_PASS(KS, B)                                                                                               \
  if (ksteps == KS && nb == B)                                                                                      \
    hipLaunchKernelGGL((attn_score_kernel<KS, B>), grid, block, 0, s, qkv, L, D, n_heads, head_dim, scale_log2, splits, partial)
#define ET_PASS2(KS) ET_PASS(KS, 1); ET_PASS(KS, 2)
#define ET_PASS3(KS) ET_PASS2(KS); ET_PASS(KS, 3)
    ET_PASS3(1); ET_PASS3(2); ET_PASS3(3); ET_PASS3(4); ET_PASS3(5); ET_PASS3(6); ET_PASS2(7); ET_PASS2(8);
#undef ET_PASS3
#undef ET_PASS2
#undef ET_PASS
    hipLaunchKernelGGL(attn_score_reduce_kernel, reduce_grid, dim3(256), 0, s, partial, n_frames, L, n_heads,
                       n_heads * splits, score);
    ET_LAUNCH_CHECK();
    return ET_OK;
  }
  float2 *stats = static_cast<float2 *>(stats_ws);
  float *partial = reinterpret_cast<float *>(stats + (size_t)n_frames * n_heads * L);
  const int blocks = (L + kScoreWaves * 32 - 1) / (kScoreWaves * 32);
  const dim3 g1(blocks, n_heads, n_frames), block(kScoreWaves * 64);
  switch (ksteps) {
#define ET_SCORE_CASE(KS)                                                                                           \
  case KS:                                                                                                          \
    hipLaunchKernelGGL(attn_rowstats_kernel<KS>, g1, block, 0, s, qkv, L, D, n_heads, head_dim, scale_log2, stats);  \
    hipLaunchKernelGGL(attn_colsum_kernel<KS>, g1, block, 0, s, qkv, L, D, n_heads, head_dim, scale_log2, stats,     \
                       partial);                                                                                    \
    break;
    ET_SCORE_CASE(1) ET_SCORE_CASE(2) ET_SCORE_CASE(3) ET_SCORE_CASE(4)
    ET_SCORE_CASE(5) ET_SCORE_CASE(6) ET_SCORE_CASE(7) ET_SCORE_CASE(8)
#undef ET_SCORE_CASE
    default: set_error("head_dim = %d unsupported", head_dim); return ET_ERR_INVALID_ARG;
  }
  hipLaunchKernelGGL(attn_score_reduce_kernel, reduce_grid, dim3(256), 0, s, partial, n_frames, L, n_heads, n_heads, score);
  ET_LAUNCH_CHECK();
  return ET_OK;
}

}  // namespace et
