// Encoder blocks of narrow encoders (a width of 64, frames of up to 64 tokens, an MLP of up to 256): between two stages of
// the compression every frame is on its own, so one workgroup takes a frame through a whole run of blocks and the frame's
// rows stay in LDS.
//
// Bound: such a block is 7 MFLOP per frame; as five launches it costs what the launches cost (about 20 us, whatever the number of
// frames), here the chain of its eight phases, each a barrier, LDS reads and a few MFMAs per wavefront: 16 500 clocks or 7 us, of
// which q | k | v 4300 (under the block's weights: 170 KB through one compute unit's vector memory path), attention 2800, GELU 3500.
// The weights come straight to registers as MFMA operands, issued a phase or more ahead, and lie in that order: as rows, half a
// cache line per row and load, the same loads took 10 000 clocks.  The bounds on width, tokens and MLP are this split's: a wavefront
// holds its 16 columns' weights of a whole block, 160 registers with an MLP of 64 to 240 of the 256 with one of 256, and its 32 of the 64
// rows' accumulators beside them.  A larger block needs weights in chunks, which has not been tried; wide encoders fill the chip from
// their GEMMs' tiles instead, and a single compute unit would walk their weights for longer than the launches take.
#include "mfma_common.h"

namespace et {

namespace {

constexpr int kW = kNarrowWidth, kRows = kNarrowTokens;
constexpr int kXLd = kW + 8, kQkvLd = 3 * kW + 8, kHidLd = kNarrowMlp + 8;     // LDS row strides: 4 banks (mod 64) from row to row, a permutation of them

// Maximum over the four lanes of a column (lane % 16), in every one of them.
__device__ __forceinline__ float across_groups(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  const auto q = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
}

// Runs blocks 0 .. n_layers - 1 of `a` on frame blockIdx.x.  Roundings to bf16 as in the launches of wider encoders: q | k | v, the
// scaled q, the probabilities, the attention's result, the residual stream after either half, the MLP's hidden
// values; all sums in float32, the MFMA steps k-ascending (q | k | v have the bits of gemm_strip_kernel on the scales of
// piece_scale_kernel).  The stream's rows past the frame's end hold whatever the blocks make of zeros (with ln_eps = 0 not even
// finite values); their q | k | v are set to zero, so that no query meets them: a probability of 0 times a NaN would be one.
// JN: the MLP's width in units of 64.
template <int HD, int JN>
__global__ __launch_bounds__(512, 1) void narrow_blocks_kernel(NarrowArgs a) {
  constexpr int HEADS = kW / HD, KC = (HD + 31) / 32, FT = HD / 16, MLP = JN * 64;
  __shared__ __align__(16) uint16_t xs[kRows * kXLd];
  __shared__ __align__(16) uint16_t buf[kRows * kHidLd];      // q | k | v (the attention's result over q), then the MLP's hidden values
  __shared__ float scales[kRows];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, g4 = lane >> 4;
  const int start = a.cu ? a.cu[blockIdx.x] : (int)blockIdx.x * a.len;
  const int n = a.cu ? a.cu[blockIdx.x + 1] - start : a.len;            // at most kRows
  const int mh = wave & 1, nq = wave >> 1;                    // GEMMs: rows 32 mh .., 16-column tiles nq, nq + 4, ..

  // A block's parameters lie in one piece (NarrowPack): one address, in registers throughout, and constants from there.  (With
  // an address per matrix each fetch first waited for scalar loads of the kernel's arguments, 4 us per block.)
  const char *const pack = a.pack;
  const int pack_bytes = (int)NarrowPack::bytes(MLP);
  auto weights = [&](const char *block, int off, int k_steps, int tile, int ks) {
    return *reinterpret_cast<const u32x4 *>(block + off + (tile * k_steps + ks) * 1024 + lane * 16);
  };
  auto bias4 = [&](const char *block, int off, int tile) { return *reinterpret_cast<const f32x4 *>(block + off + (tile * 16 + g4 * 4) * 4); };
  u32x4 wq[3][2], wo[2], w1[JN][2], w2[2 * JN];
  f32x4 bq[3], bo, b1[JN], b2;
  auto fetch_attention_half = [&](int layer) {
    const char *p = pack + (size_t)layer * pack_bytes;
#pragma unroll
    for (int j = 0; j < 3; ++j) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) wq[j][ks] = weights(p, NarrowPack::wqkv(), 2, nq + 4 * j, ks);
      bq[j] = bias4(p, NarrowPack::bqkv(MLP), nq + 4 * j);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) wo[ks] = weights(p, NarrowPack::wo(), 2, nq, ks);
    bo = bias4(p, NarrowPack::bo(MLP), nq);
  };
  auto fetch_mlp_half = [&](int layer) {
    const char *p = pack + (size_t)layer * pack_bytes;
#pragma unroll
    for (int j = 0; j < JN; ++j) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) w1[j][ks] = weights(p, NarrowPack::w1(), 2, nq + 4 * j, ks);
      b1[j] = bias4(p, NarrowPack::b1(MLP), nq + 4 * j);
    }
#pragma unroll
    for (int ks = 0; ks < 2 * JN; ++ks) w2[ks] = weights(p, NarrowPack::w2(MLP), 2 * JN, nq, ks);
    b2 = bias4(p, NarrowPack::b2(MLP), nq);
  };
  auto meet = [&]() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  const int row = tid >> 3, oct = tid & 7;                    // row-wise phases: eight lanes per row
  uint16_t *const own = xs + row * kXLd + oct * 8;
  auto leave_scale = [&](u32x4 v) {
    PieceSum sum;
    const float2 st = piece_moments(v);
    sum.ref = st.x;
    sum.add(st);
    if (oct == 0) scales[row] = sum.scale(1, a.ln_eps);
  };
  // Activation operand: rows 32 mh + 16 b .., columns 32 ks .. of an LDS matrix.
  auto rows_of = [&](const uint16_t *m, int ld, int b, int ks) {
    return *reinterpret_cast<const u32x4 *>(m + (mh * 32 + b * 16 + r16) * ld + ks * 32 + g4 * 8);
  };

  u32x4 mine = u32x4{0u, 0u, 0u, 0u};
  if (row < n) mine = *reinterpret_cast<const u32x4 *>(a.x + ((size_t)start + row) * kW + oct * 8);
  fetch_attention_half(0);
  *reinterpret_cast<u32x4 *>(own) = mine;
  leave_scale(mine);
  meet();

  for (int li = 0; li < a.n_layers; ++li) {
    fetch_mlp_half(li);
    {                                                         // q | k | v
      f32x4 acc[3][2];
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const u32x4 x0 = rows_of(xs, kXLd, b, 0), x1 = rows_of(xs, kXLd, b, 1);
#pragma unroll
        for (int j = 0; j < 3; ++j) acc[j][b] = mfma16(wq[j][1], x1, mfma16(wq[j][0], x0, f32x4{0.f, 0.f, 0.f, 0.f}));
      }
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int m = mh * 32 + b * 16 + r16;
        const float rs = scales[m];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const int c = (nq + 4 * j) * 16 + g4 * 4;
          uint2 o;
          o.x = cvt_pk_bf16(fmaf(rs, acc[j][b][0], bq[j][0]), fmaf(rs, acc[j][b][1], bq[j][1]));
          o.y = cvt_pk_bf16(fmaf(rs, acc[j][b][2], bq[j][2]), fmaf(rs, acc[j][b][3], bq[j][3]));
          if (m >= n) o = make_uint2(0u, 0u);
          if (li + 1 == a.n_layers && m < n) *reinterpret_cast<uint2 *>(a.qkv + ((size_t)start + m) * 3 * kW + c) = o;
          *reinterpret_cast<uint2 *>(buf + m * kQkvLd + c) = o;
        }
      }
    }
    meet();
    // Attention by units of one head and 16 queries: S^T = K Q^T on 16 x 16 tiles, two of which are, exponentiated, the
    // operand of 32 keys of O^T = V^T P^T (k-slots 8 g4 + j: rows 4 g4 + j of the first tile, then of the second).  A wavefront takes
    // its units side by side: each is a chain of latencies.  Queries past the frame are computed too.
    if (HEADS * 4 >= 8 || wave < HEADS * 4) {
      constexpr int UNITS = HEADS * 4 >= 8 ? HEADS / 2 : 1;
      uint16_t *q_cell[UNITS];
      const uint16_t *kv[UNITS];
      u32x4 qf[UNITS][KC], pf[UNITS][2];
      f32x4 s[UNITS][4], o[UNITS][FT], sum[UNITS];
#pragma unroll
      for (int u = 0; u < UNITS; ++u) {
        const int h = (wave + 8 * u) >> 2, q0 = ((wave + 8 * u) & 3) * 16;
        q_cell[u] = buf + (q0 + r16) * kQkvLd + h * HD;
        kv[u] = buf + kW + h * HD;
#pragma unroll
        for (int c = 0; c < KC; ++c) {
          // (heads of 16 leave half of the contraction's slots empty: zeros on both sides)
          const u32x4 raw = *reinterpret_cast<const u32x4 *>(q_cell[u] + c * 32 + (HD == 16 ? g4 & 1 : g4) * 8);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            qf[u][c][e] = cvt_pk_bf16(bf16lo_to_f32(raw[e]) * a.scale_log2, bf16hi_to_f32(raw[e]) * a.scale_log2);
            if (HD == 16 && g4 >= 2) qf[u][c][e] = 0u;
          }
        }
      }
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
          s[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < KC; ++c) {
            u32x4 kf = *reinterpret_cast<const u32x4 *>(kv[u] + (t * 16 + r16) * kQkvLd + c * 32 + (HD == 16 ? g4 & 1 : g4) * 8);
            if (HD == 16 && g4 >= 2) kf = u32x4{0u, 0u, 0u, 0u};
            s[u][t] = mfma16(kf, qf[u][c], s[u][t]);
          }
        }
      if (n < kRows) {                                        // keys past the frame
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (t * 16 + g4 * 4 + i >= n) {
#pragma unroll
              for (int u = 0; u < UNITS; ++u) s[u][t][i] = -INFINITY;
            }
      }
#pragma unroll
      for (int u = 0; u < UNITS; ++u) {
        float mx = s[u][0][0];
#pragma unroll
        for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[u][i >> 2][i & 3]);
        mx = across_groups(mx);
        const float ref = mx == -INFINITY ? 0.f : mx;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            pf[u][t >> 1][(t & 1) * 2 + i] = cvt_pk_bf16(__builtin_amdgcn_exp2f(s[u][t][2 * i] - ref), __builtin_amdgcn_exp2f(s[u][t][2 * i + 1] - ref));
      }
      const u32x4 ones = u32x4{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u};
#pragma unroll
      for (int u = 0; u < UNITS; ++u) {                       // the denominator: the sum of the probabilities as rounded, in every row
        sum[u] = mfma16(ones, pf[u][1], mfma16(ones, pf[u][0], f32x4{0.f, 0.f, 0.f, 0.f}));
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) {
          o[u][ft] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const uint16_t *vp = kv[u] + kW + (c * 32 + g4 * 4 + (r16 >> 2)) * kQkvLd + ft * 16 + (r16 & 3) * 4;
            const uint2 lo = lds_read_tr16(vp), hi = lds_read_tr16(vp + 16 * kQkvLd);
            o[u][ft] = mfma16(u32x4{lo.x, lo.y, hi.x, hi.y}, pf[u][c], o[u][ft]);
          }
        }
      }
#pragma unroll
      for (int u = 0; u < UNITS; ++u) {
        const float inv = 1.0f / sum[u][0];
#pragma unroll
        for (int ft = 0; ft < FT; ++ft) {
          uint2 w;                                            // (over this unit's own queries, which nobody else reads)
          w.x = cvt_pk_bf16(o[u][ft][0] * inv, o[u][ft][1] * inv);
          w.y = cvt_pk_bf16(o[u][ft][2] * inv, o[u][ft][3] * inv);
          *reinterpret_cast<uint2 *>(q_cell[u] + ft * 16 + g4 * 4) = w;
        }
      }
    }
    meet();
    // Adds acc + bias to the residual stream, in place: an element has one owner.
    auto add_to_stream = [&](const f32x4 &acc, const f32x4 &bias, int b) {
      uint2 *cell = reinterpret_cast<uint2 *>(xs + (mh * 32 + b * 16 + r16) * kXLd + nq * 16 + g4 * 4);
      const uint2 r = *cell;
      uint2 o;
      o.x = cvt_pk_bf16(acc[0] + bias[0] + bf16lo_to_f32(r.x), acc[1] + bias[1] + bf16hi_to_f32(r.x));
      o.y = cvt_pk_bf16(acc[2] + bias[2] + bf16lo_to_f32(r.y), acc[3] + bias[3] + bf16hi_to_f32(r.y));
      *cell = o;
    };
#pragma unroll
    for (int b = 0; b < 2; ++b) {                             // out-projection
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) acc = mfma16(wo[ks], rows_of(buf, kQkvLd, b, ks), acc);
      add_to_stream(acc, bo, b);
    }
    if (li + 1 < a.n_layers) fetch_attention_half(li + 1);
    meet();
    leave_scale(*reinterpret_cast<const u32x4 *>(own));
    meet();
#pragma unroll
    for (int b = 0; b < 2; ++b) {                             // fc1, GELU
      const u32x4 x0 = rows_of(xs, kXLd, b, 0), x1 = rows_of(xs, kXLd, b, 1);
      const int m = mh * 32 + b * 16 + r16;
      const float rs = scales[m];
#pragma unroll
      for (int j = 0; j < JN; ++j) {
        const f32x4 acc = mfma16(w1[j][1], x1, mfma16(w1[j][0], x0, f32x4{0.f, 0.f, 0.f, 0.f}));
        uint2 o;
        o.x = cvt_pk_bf16(gelu_tanh_f(fmaf(rs, acc[0], b1[j][0])), gelu_tanh_f(fmaf(rs, acc[1], b1[j][1])));
        o.y = cvt_pk_bf16(gelu_tanh_f(fmaf(rs, acc[2], b1[j][2])), gelu_tanh_f(fmaf(rs, acc[3], b1[j][3])));
        *reinterpret_cast<uint2 *>(buf + m * kHidLd + (nq + 4 * j) * 16 + g4 * 4) = o;
      }
    }
    meet();
#pragma unroll
    for (int b = 0; b < 2; ++b) {                             // fc2
      f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 2 * JN; ++ks) acc = mfma16(w2[ks], rows_of(buf, kHidLd, b, ks), acc);
      add_to_stream(acc, b2, b);
    }
    meet();
    mine = *reinterpret_cast<const u32x4 *>(own);
    if (li + 1 < a.n_layers) {
      leave_scale(mine);
      meet();
    }
  }

  if (row >= n) return;
  uint16_t *dst = a.out + ((size_t)start + row) * kW + oct * 8;
  if (!a.final_g) {
    *reinterpret_cast<u32x4 *>(dst) = mine;
    return;
  }
  float v[8], s = 0.f, q = 0.f;                               // the final LayerNorm, as layernorm_kernel computes it
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[2 * e] = bf16lo_to_f32(mine[e]);
    v[2 * e + 1] = bf16hi_to_f32(mine[e]);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) s += v[e];
  const float mean = sum_of_8_lanes(s) / (float)kW;
#pragma unroll
  for (int e = 0; e < 8; ++e) q = fmaf(v[e] - mean, v[e] - mean, q);
  const float rstd = 1.0f / sqrtf(sum_of_8_lanes(q) / (float)kW + a.ln_eps);
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int c = oct * 8 + 2 * e;
    o[e] = cvt_pk_bf16((v[2 * e] - mean) * rstd * a.final_g[c] + a.final_b[c], (v[2 * e + 1] - mean) * rstd * a.final_g[c + 1] + a.final_b[c + 1]);
  }
  *reinterpret_cast<u32x4 *>(dst) = o;
}

}  // namespace

template <int HD>
static int launch_heads(const NarrowArgs &a, int n_frames, hipStream_t s) {
  const dim3 grid((unsigned)n_frames), block(512);
  switch (a.mlp / 64) {
    case 1: hipLaunchKernelGGL((narrow_blocks_kernel<HD, 1>), grid, block, 0, s, a); break;
    case 2: hipLaunchKernelGGL((narrow_blocks_kernel<HD, 2>), grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL((narrow_blocks_kernel<HD, 3>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((narrow_blocks_kernel<HD, 4>), grid, block, 0, s, a); break;
  }
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_narrow_blocks(const NarrowArgs &a, int n_frames, int n_heads, hipStream_t s) {
  if (n_frames <= 0 || a.n_layers <= 0) return ET_OK;
  ET_REQUIRE(a.len >= 1 && a.len <= kNarrowTokens && a.mlp >= 64 && a.mlp <= kNarrowMlp && a.mlp % 64 == 0,
             "narrow blocks: %d tokens, MLP %d out of range", a.len, a.mlp);
  switch (kNarrowWidth / n_heads) {
    case 16: return launch_heads<16>(a, n_frames, s);
    case 32: return launch_heads<32>(a, n_frames, s);
    case 64: return launch_heads<64>(a, n_frames, s);
    default: set_error("narrow blocks: %d heads", n_heads); return ET_ERR_UNSUPPORTED;
  }
}

}  // namespace et
