// The encoder object and et_encode_clip: weight packing, workspace layout, the layer loop with
// the compression stage spliced in after `merge_layer` blocks, and optional per-kernel timing.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <utility>
#include <vector>

#include "et_common.h"
#include "gemm_choice.h"

namespace et {

static inline int round_up(int v, int a) { return (v + a - 1) / a * a; }
static inline size_t align256(size_t v) { return (v + 255) / 256 * 256; }

static uint16_t host_f32_to_bf16(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

struct LayerDev {
  uint16_t *wqkv, *wo, *w1, *w2;
  float *bqkv, *bo, *b1, *b2;
};

}  // namespace et

struct et_encoder {
  et_config cfg;
  int L, D, hd, Mhp, Kp, Kp_pad, max_frames;
  std::vector<void *> allocs;
  uint16_t *patch_w = nullptr, *pos_emb = nullptr;
  float *patch_b = nullptr, *final_g = nullptr, *final_b = nullptr;
  std::vector<et::LayerDev> layers;
  char *narrow_pack = nullptr;          // see pack_narrow (NULL: not a narrow encoder)
  et::Profiler prof;
  int32_t *count_host = nullptr;        // pinned: segment count read back in the middle of the compression stage
  hipEvent_t count_ready = nullptr;
};

namespace et {

// LayerNorm folded into the linear layer that follows it.  With mu, rstd the row statistics,
//   LN(x) W^T + b = rstd (x - mu) (W . gamma)^T + (W beta + b) = rstd * (x Wf^T) + c,
//   Wf[n][k] = W[n][k] gamma[k] - mean_k(W[n][:] gamma),   c[n] = sum_k W[n][k] beta[k] + b[n]:
// subtracting each folded row's mean makes the mu term vanish (sum_k (x_k - mu) w_k = sum_k x_k (w_k - mean w)),
// so the GEMM reads the residual stream itself and its epilogue multiplies by the row's rstd.
// The folded weights are rounded to bfloat16 here, along each row with the rounding error carried
// into the next element (first-order error diffusion, k ascending, every step through the nearest
// float32): a row of rounded weights then still sums to zero within one step of one element, where
// independent rounding would leave ~sqrt(K) half-steps that a row's mean multiplies.
static void fold_layernorm(const float *W, const float *bias, const float *gamma, const float *beta, int N, int K,
                           std::vector<float> &Wf, std::vector<float> &c) {
  Wf.resize((size_t)N * K);
  c.resize(N);
  std::vector<double> row(K);
  for (int n = 0; n < N; ++n) {
    double mean = 0.0, cb = bias[n];
    for (int k = 0; k < K; ++k) {
      row[k] = (double)W[(size_t)n * K + k] * gamma[k];
      mean += row[k];
      cb += (double)W[(size_t)n * K + k] * beta[k];
    }
    mean /= K;
    double carry = 0.0;
    for (int k = 0; k < K; ++k) {
      const double t = row[k] - mean + carry;
      const uint32_t bits = (uint32_t)host_f32_to_bf16((float)t) << 16;
      float y;
      memcpy(&y, &bits, 4);
      Wf[(size_t)n * K + k] = y;
      carry = t - (double)y;
    }
    c[n] = (float)cb;
  }
}

// Uploads a host fp32 matrix [rows, cols] as bf16 [rows_pad, cols_pad], zero padded.
static int upload_bf16(et_encoder *e, const float *src, int rows, int cols, int rows_pad, int cols_pad,
                       uint16_t **out) {
  std::vector<uint16_t> h((size_t)rows_pad * cols_pad, 0);
  for (int r = 0; r < rows; ++r)
    for (int c = 0; c < cols; ++c) h[(size_t)r * cols_pad + c] = host_f32_to_bf16(src[(size_t)r * cols + c]);
  void *d = nullptr;
  if (hipMalloc(&d, h.size() * sizeof(uint16_t)) != hipSuccess) {
    (void)hipGetLastError();
    set_error("device allocation of %zu bytes failed", h.size() * sizeof(uint16_t));
    return ET_ERR_ALLOC;
  }
  e->allocs.push_back(d);
  ET_HIP(hipMemcpy(d, h.data(), h.size() * sizeof(uint16_t), hipMemcpyHostToDevice));
  *out = static_cast<uint16_t *>(d);
  return ET_OK;
}

static int upload_f32(et_encoder *e, const float *src, int n, int n_pad, float **out) {
  std::vector<float> h((size_t)n_pad, 0.f);
  memcpy(h.data(), src, (size_t)n * sizeof(float));
  void *d = nullptr;
  if (hipMalloc(&d, h.size() * sizeof(float)) != hipSuccess) {
    (void)hipGetLastError();
    set_error("device allocation of %zu bytes failed", h.size() * sizeof(float));
    return ET_ERR_ALLOC;
  }
  e->allocs.push_back(d);
  ET_HIP(hipMemcpy(d, h.data(), h.size() * sizeof(float), hipMemcpyHostToDevice));
  *out = static_cast<float *>(d);
  return ET_OK;
}

struct EncWs {
  uint16_t *x, *qkv, *att, *hid;
  void *merge;
  // row statistics and per-head column sums of the attention-received scores.  The statistics of the residual
  // stream live there too, from a residual GEMM to the GEMM that follows it (no scores are computed between):
  void *score_ws;
  float *rstd;         // [R]: 1 / sqrt(var + eps) of the rows of x, or
  float2 *pieces;      // [D / 64][piece_ld]: see GemmArgs::stats_out
  int piece_ld;
  float *att_score;    // [T, L]
  size_t bytes;
};

static EncWs carve_encoder(const et_encoder *e, void *ws, int T) {
  char *base = static_cast<char *>(ws);
  size_t off = 0;
  auto take = [&](size_t bytes) -> void * {
    void *p = base ? base + off : nullptr;
    off += align256(bytes);
    return p;
  };
  const size_t R = (size_t)T * e->L;
  EncWs w;
  w.x = static_cast<uint16_t *>(take(R * e->D * 2));
  w.qkv = static_cast<uint16_t *>(take(R * 3 * e->D * 2));
  w.att = static_cast<uint16_t *>(take(R * e->D * 2));
  const size_t hid_cols = (size_t)(e->Mhp > e->Kp_pad ? e->Mhp : e->Kp_pad);
  w.hid = static_cast<uint16_t *>(take(R * hid_cols * 2));
  w.merge = take(carve_merge(nullptr, T, e->L, e->D).bytes);
  const size_t score_bytes = attention_scores_workspace_bytes(T, e->L, e->cfg.n_heads), piece_bytes = R * (e->D / 64) * sizeof(float2);
  w.score_ws = take(score_bytes > piece_bytes ? score_bytes : piece_bytes);
  w.rstd = static_cast<float *>(w.score_ws);
  w.pieces = static_cast<float2 *>(w.score_ws);
  w.piece_ld = (int)R;
  w.att_score = static_cast<float *>(take(R * sizeof(float)));
  w.bytes = off;
  return w;
}

#define ET_TIMED(kind, call) ET_TIMED_P(&e->prof, kind, call)

static bool takes_pieces(const et_encoder *e, int rows) {
  return gemm_takes_pieces(rows, 3 * e->D) && gemm_takes_pieces(rows, e->Mhp);
}

// have_pieces: w.pieces holds the statistics of w.x (only looked at where takes_pieces(rows)).
// with_scores: also leave the attention each token receives in this block in w.att_score (frames of
// equal length only).
static int run_block(et_encoder *e, int layer, const EncWs &w, int rows, const int32_t *cu,
                     int n_frames, int max_len, bool ragged, bool have_pieces, hipStream_t s, bool with_scores = false) {
  const et_config &c = e->cfg;
  const int D = e->D;
  const LayerDev &lw = e->layers[layer];
  // LayerNorm 1 and 2 are folded into the QKV and fc1 weights (fold_layernorm): only the row scales are needed.  On
  // few rows (`by_pieces`) the GEMMs that write the residual stream leave its statistics by pieces of 64 columns
  // and the next GEMM combines them; after a merge or selection the pieces are computed here.  On many rows the scales
  // have a launch of their own, small beside the GEMMs.
  const bool by_pieces = takes_pieces(e, rows);
  auto normed = [&](GemmArgs g) {
    if (by_pieces) {
      g.stats_in = w.pieces;
      g.stats_ld = w.piece_ld;
      g.ln_eps = c.ln_eps;
    } else {
      g.row_scale = w.rstd;
    }
    return g;
  };
  auto leaving_pieces = [&](GemmArgs g) {
    if (by_pieces) {
      g.stats_out = w.pieces;
      g.stats_ld = w.piece_ld;
    }
    return g;
  };
  if (!by_pieces) ET_TIMED(ET_K_LAYERNORM, launch_rowstats(w.x, c.ln_eps, rows, D, w.rstd, s));
  else if (!have_pieces) ET_TIMED(ET_K_LAYERNORM, launch_piece_stats(w.x, rows, D, w.piece_ld, w.pieces, s));
  GemmArgs g = normed(GemmArgs{w.x, D, lw.wqkv, lw.bqkv, nullptr, 0, 1, w.qkv, 3 * D, rows, 3 * D, D, EPI_BIAS});
  ET_TIMED(ET_K_GEMM_QKV, launch_gemm(g, s));
  if (with_scores)
    ET_TIMED(ET_K_SCORE, launch_attention_scores(w.qkv, n_frames, max_len, c.n_heads, e->hd, w.score_ws, w.att_score, s));
  // the weights that the launches behind the attention read, for its idle compute units
  const uint32_t mlp_bytes = (uint32_t)D * e->Mhp * 2u;
  WarmRanges warm{{lw.wo, lw.w1, lw.w2, nullptr}, {(uint32_t)D * D * 2u, mlp_bytes, mlp_bytes, 0u}};
  if (layer + 1 < c.n_layers) {
    warm.ptr[3] = e->layers[layer + 1].wqkv;
    warm.bytes[3] = 3u * D * D * 2u;
  }
  if (ragged) {   // frames of different lengths (decoupled selection): row ranges from cu
    ET_TIMED(ET_K_ATTENTION, launch_attention(w.qkv, cu, n_frames, max_len, c.n_heads, e->hd, w.att, s, &warm));
  } else {        // every frame has max_len tokens
    ET_TIMED(ET_K_ATTENTION, launch_attention_uniform(w.qkv, n_frames, max_len, c.n_heads, e->hd, w.att, s, &warm));
  }
  g = leaving_pieces(GemmArgs{w.att, D, lw.wo, lw.bo, w.x, D, rows, w.x, D, rows, D, D, EPI_BIAS_RES});
  ET_TIMED(ET_K_GEMM_OUT, launch_gemm(g, s));
  if (!by_pieces) ET_TIMED(ET_K_LAYERNORM, launch_rowstats(w.x, c.ln_eps, rows, D, w.rstd, s));
  g = normed(GemmArgs{w.x, D, lw.w1, lw.b1, nullptr, 0, 1, w.hid, e->Mhp, rows, e->Mhp, D, EPI_BIAS_GELU});
  ET_TIMED(ET_K_GEMM_FC1, launch_gemm(g, s));
  g = leaving_pieces(GemmArgs{w.hid, e->Mhp, lw.w2, lw.b2, w.x, D, rows, w.x, D, rows, D, e->Mhp, EPI_BIAS_RES});
  ET_TIMED(ET_K_GEMM_FC2, launch_gemm(g, s));
  return ET_OK;
}

// Whether every frame of the encoder fits the kernel that takes a frame through a run of blocks (narrow_blocks.hip).  A rule
// on the encoder, not on the call: the stages of one clip, and et_encoder_block_qkv, see the same arithmetic throughout.
// An encoder of 4 blocks and 64 tokens per frame, merge after two, us per call by launches / by frames: 1 frame 149 / 79, 8 frames 158 / 84, 64 frames
// 160 / 88; nothing merged, 256 frames 190 / 84, 600 335 / 158, 2000 836 / 393 (a grid of many rounds); half the tokens kept in
// front of the first block, 256 frames 183 / 114, 2000 589 / 549.
static bool is_narrow(const et_encoder *e) {
  return e->D == kNarrowWidth && e->L <= kNarrowTokens && e->Mhp <= kNarrowMlp && (e->hd == 16 || e->hd == 32 || e->hd == 64);
}

// Blocks first .. last - 1 on the frames of w.x; leaves the stream in `out`, normalised if `final_norm`, and q | k | v of
// the last block in w.qkv.
static int run_narrow_blocks(et_encoder *e, int first, int last, const EncWs &w, const int32_t *cu, int n_frames, int max_len, bool final_norm,
                             uint16_t *out, hipStream_t s) {
  NarrowArgs a{};
  a.pack = e->narrow_pack + (size_t)first * NarrowPack::bytes(e->Mhp);
  a.n_layers = last - first;
  a.x = w.x;
  a.out = out;
  a.qkv = w.qkv;
  a.cu = cu;
  a.len = max_len;
  a.mlp = e->Mhp;
  a.ln_eps = e->cfg.ln_eps;
  a.scale_log2 = 1.4426950408889634f / sqrtf((float)e->hd);
  if (final_norm) {
    a.final_g = e->final_g;
    a.final_b = e->final_b;
  }
  ET_TIMED(ET_K_MISC, launch_narrow_blocks(a, n_frames, e->cfg.n_heads, s));
  return ET_OK;
}

// The parameters of all blocks once more, as that kernel reads them.
static int pack_narrow(et_encoder *e) {
  const int mlp = e->Mhp, D = kNarrowWidth;
  std::vector<char> host((size_t)e->cfg.n_layers * NarrowPack::bytes(mlp));
  std::vector<uint16_t> plain((size_t)mlp * D > (size_t)3 * D * D ? (size_t)mlp * D : (size_t)3 * D * D);
  for (int i = 0; i < e->cfg.n_layers; ++i) {
    char *p = host.data() + (size_t)i * NarrowPack::bytes(mlp);
    const LayerDev &l = e->layers[i];
    const struct { int off; const uint16_t *src; int rows, cols; } mats[] = {{NarrowPack::wqkv(), l.wqkv, 3 * D, D}, {NarrowPack::wo(), l.wo, D, D},
                                                                             {NarrowPack::w1(), l.w1, mlp, D}, {NarrowPack::w2(mlp), l.w2, D, mlp}};
    for (const auto &m : mats) {
      ET_HIP(hipMemcpy(plain.data(), m.src, (size_t)m.rows * m.cols * 2, hipMemcpyDeviceToHost));
      for (int r = 0; r < m.rows; ++r)
        for (int c = 0; c < m.cols; c += 8)
          memcpy(p + m.off + ((r / 16) * (m.cols / 32) + c / 32) * 1024 + ((c / 8 % 4) * 16 + r % 16) * 16, plain.data() + (size_t)r * m.cols + c, 16);
    }
    const struct { int off; const float *src; int n; } biases[] = {{NarrowPack::bqkv(mlp), l.bqkv, 3 * D}, {NarrowPack::bo(mlp), l.bo, D},
                                                                   {NarrowPack::b1(mlp), l.b1, mlp}, {NarrowPack::b2(mlp), l.b2, D}};
    for (const auto &b : biases) ET_HIP(hipMemcpy(p + b.off, b.src, (size_t)b.n * 4, hipMemcpyDeviceToHost));
  }
  void *d = nullptr;
  if (hipMalloc(&d, host.size()) != hipSuccess) {
    (void)hipGetLastError();
    set_error("device allocation of %zu bytes failed", host.size());
    return ET_ERR_ALLOC;
  }
  e->allocs.push_back(d);
  e->narrow_pack = static_cast<char *>(d);
  ET_HIP(hipMemcpy(d, host.data(), host.size(), hipMemcpyHostToDevice));
  return ET_OK;
}

}  // namespace et

using namespace et;

extern "C" {

int et_encoder_create(const et_config *config, const et_weights *weights, int32_t max_frames,
                      et_encoder **out) {
  ET_REQUIRE(config && weights && out, "config, weights or out is NULL");
  *out = nullptr;
  const et_config &c = *config;
  ET_REQUIRE(c.n_layers >= 0 && c.n_layers <= 1024, "n_layers = %d out of range", c.n_layers);
  ET_REQUIRE(c.d_model >= 8 && c.n_heads >= 1 && c.d_mlp >= 1, "d_model/n_heads/d_mlp must be positive");
  ET_REQUIRE(c.d_model % c.n_heads == 0, "d_model %d is not a multiple of n_heads %d", c.d_model, c.n_heads);
  ET_REQUIRE(c.patch >= 1 && c.channels >= 1, "patch and channels must be positive");
  ET_REQUIRE(c.image_h >= c.patch && c.image_w >= c.patch, "image %dx%d smaller than one %d-pixel patch",
             c.image_h, c.image_w, c.patch);
  ET_REQUIRE(c.ln_eps >= 0.f && isfinite(c.ln_eps), "ln_eps must be finite and non-negative");
  ET_REQUIRE(max_frames >= 1, "max_frames = %d must be at least 1", max_frames);
  const int L = (c.image_h / c.patch) * (c.image_w / c.patch);
  ET_REQUIRE((double)max_frames * L * c.d_model * 3 < 2.0e9, "max_frames * L * 3 * d_model exceeds 2^31 elements");
  ET_REQUIRE(weights->patch_w && weights->patch_b && weights->pos_emb, "a patch-embedding weight is NULL");
  ET_REQUIRE(c.n_layers == 0 || (weights->ln1_g && weights->ln1_b && weights->wqkv && weights->bqkv &&
                                 weights->wo && weights->bo && weights->ln2_g && weights->ln2_b &&
                                 weights->w1 && weights->b1 && weights->w2 && weights->b2),
             "a per-layer weight table is NULL");
  ET_REQUIRE(!c.has_final_ln || (weights->final_ln_g && weights->final_ln_b),
             "has_final_ln is set but final_ln_g/final_ln_b is NULL");
  if (c.d_model % 64 != 0 || c.d_model > 4096) {
    set_error("d_model = %d: only multiples of 64 up to 4096 are supported", c.d_model);
    return ET_ERR_UNSUPPORTED;
  }
  if (!head_dim_supported(c.d_model / c.n_heads)) {
    set_error("head_dim = %d is not instantiated (16, 32, 64, 72, 80, 96, 128)", c.d_model / c.n_heads);
    return ET_ERR_UNSUPPORTED;
  }
  if (L > 15360) {
    set_error("tokens per frame = %d above the supported 15360", L);
    return ET_ERR_UNSUPPORTED;
  }
  for (int i = 0; i < c.n_layers; ++i) {
    ET_REQUIRE(weights->ln1_g[i] && weights->ln1_b[i] && weights->wqkv[i] && weights->bqkv[i] &&
                   weights->wo[i] && weights->bo[i] && weights->ln2_g[i] && weights->ln2_b[i] &&
                   weights->w1[i] && weights->b1[i] && weights->w2[i] && weights->b2[i],
               "a weight pointer of layer %d is NULL", i);
  }

  et_encoder *e = new (std::nothrow) et_encoder();
  if (!e) { set_error("host allocation failed"); return ET_ERR_ALLOC; }
  e->cfg = c;
  e->L = L;
  e->D = c.d_model;
  e->hd = c.d_model / c.n_heads;
  e->Mhp = round_up(c.d_mlp, 64);
  e->Kp = c.channels * c.patch * c.patch;
  e->Kp_pad = round_up(e->Kp, 64);
  e->max_frames = max_frames;
  const int D = e->D, Dn = round_up(D, 256);
  int rc = ET_OK;
#define ET_TRY(x) if ((rc = (x)) != ET_OK) { et_encoder_destroy(e); return rc; }
  ET_TRY(upload_bf16(e, weights->patch_w, D, e->Kp, Dn, e->Kp_pad, &e->patch_w));
  ET_TRY(upload_f32(e, weights->patch_b, D, Dn, &e->patch_b));
  ET_TRY(upload_bf16(e, weights->pos_emb, L, D, L, D, &e->pos_emb));
  if (c.has_final_ln) {
    ET_TRY(upload_f32(e, weights->final_ln_g, D, D, &e->final_g));
    ET_TRY(upload_f32(e, weights->final_ln_b, D, D, &e->final_b));
  }
  e->layers.resize(c.n_layers);
  for (int i = 0; i < c.n_layers; ++i) {
    LayerDev &l = e->layers[i];
    std::vector<float> wf, cf;
    fold_layernorm(weights->wqkv[i], weights->bqkv[i], weights->ln1_g[i], weights->ln1_b[i], 3 * D, D, wf, cf);
    ET_TRY(upload_bf16(e, wf.data(), 3 * D, D, round_up(3 * D, 256), D, &l.wqkv));
    ET_TRY(upload_f32(e, cf.data(), 3 * D, round_up(3 * D, 256), &l.bqkv));
    ET_TRY(upload_bf16(e, weights->wo[i], D, D, Dn, D, &l.wo));
    ET_TRY(upload_f32(e, weights->bo[i], D, Dn, &l.bo));
    // MLP width padded to a multiple of 64 with zero rows / bias (GELU(0) = 0) and zero columns
    fold_layernorm(weights->w1[i], weights->b1[i], weights->ln2_g[i], weights->ln2_b[i], c.d_mlp, D, wf, cf);
    ET_TRY(upload_bf16(e, wf.data(), c.d_mlp, D, round_up(e->Mhp, 256), D, &l.w1));
    ET_TRY(upload_f32(e, cf.data(), c.d_mlp, round_up(e->Mhp, 256), &l.b1));
    ET_TRY(upload_bf16(e, weights->w2[i], D, c.d_mlp, Dn, e->Mhp, &l.w2));
    ET_TRY(upload_f32(e, weights->b2[i], D, Dn, &l.b2));
  }
  if (is_narrow(e) && c.n_layers > 0) ET_TRY(pack_narrow(e));
#undef ET_TRY
  if (hipEventCreateWithFlags(&e->count_ready, hipEventDisableTiming) != hipSuccess ||
      hipHostMalloc(reinterpret_cast<void **>(&e->count_host), 64, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    et_encoder_destroy(e);
    set_error("creating the read-back event or its pinned word failed");
    return ET_ERR_HIP;
  }
  *out = e;
  return ET_OK;
}

void et_encoder_destroy(et_encoder *e) {
  if (!e) return;
  if (e->count_ready) (void)hipEventDestroy(e->count_ready);
  if (e->count_host) (void)hipHostFree(e->count_host);
  for (void *p : e->allocs) (void)hipFree(p);
  e->prof.destroy();
  delete e;
}

size_t et_workspace_bytes(const et_encoder *e, int32_t T) {
  if (!e || T < 1 || T > e->max_frames) return 0;
  return carve_encoder(e, nullptr, T).bytes;
}

}  // extern "C"

// Shared body of et_encode_clip (policy == nullptr: simple stage with sim_threshold / keep_ratio)
// and et_encode_clip_policy.
// With a policy, `merge_layers[0..n_merge)` (ascending) are the layers where Stage I runs and
// `merge_layer` is the layer of Stage II (>= the last Stage I layer).
static int encode_impl(et_encoder *e, const float *frames_dev, int32_t T, int32_t merge_layer,
                       float sim_threshold, float keep_ratio, const et_policy *policy,
                       const int32_t *merge_layers, int32_t n_merge, void *workspace_dev,
                       size_t workspace_bytes, void *hip_stream, et_output *out, et_plan_out *plan) {
  ET_REQUIRE(e != nullptr, "encoder is NULL");
  ET_REQUIRE(frames_dev != nullptr, "frames_dev is NULL");
  ET_REQUIRE(T >= 1 && T <= e->max_frames, "T = %d outside [1, max_frames = %d]", T, e->max_frames);
  ET_REQUIRE(merge_layer <= e->cfg.n_layers, "merge_layer = %d above n_layers = %d", merge_layer,
             e->cfg.n_layers);
  ET_REQUIRE(out != nullptr, "out is NULL");
  ET_REQUIRE(out->tokens_dev && out->kept_idx_dev && out->cu_tokens_dev && out->seg_start_dev,
             "an output buffer is NULL (tokens_dev, kept_idx_dev, cu_tokens_dev, seg_start_dev are required)");
  const bool compress = merge_layer >= 0;
  bool by_attention = false;
  if (compress && policy) {
    int prc = check_policy(policy);
    if (prc) return prc;
    by_attention = policy->score_mode == ET_SCORE_ATTENTION;
    if (by_attention) {
      ET_REQUIRE(merge_layer >= 1, "attention scores need an encoder block before the selection (select layer >= 1)");
      for (int i = 0; i < n_merge; ++i)
        ET_REQUIRE(merge_layers[i] != merge_layer,
                   "attention scores need a block between the last merge and the selection (both at layer %d)",
                   merge_layer);
    }
  } else if (compress) {
    ET_REQUIRE(!isnan(sim_threshold), "sim_threshold is NaN");
    ET_REQUIRE(keep_ratio > 0.f && keep_ratio <= 1.f, "keep_ratio = %g outside (0, 1]", (double)keep_ratio);
  }
  ET_REQUIRE(workspace_dev != nullptr, "workspace_dev is NULL");
  const size_t need = et_workspace_bytes(e, T);
  if (workspace_bytes < need) {
    set_error("workspace of %zu bytes is smaller than the %zu needed", workspace_bytes, need);
    return ET_ERR_WORKSPACE;
  }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const et_config &c = e->cfg;
  const int L = e->L, D = e->D;
  EncWs w = carve_encoder(e, workspace_dev, T);
  uint16_t *spare = carve_merge(w.merge, T, L, D).merged;      // the other place of the residual stream (policy stages)
  e->prof.kinds.clear();
  e->prof.phase = 0;

  int rows = T * L, n_frames = T, max_len = L, k = L;
  (void)k;
  const int32_t *cu = nullptr;             // row ranges of the frames, once they differ in length
  if (!compress) {
    ET_TIMED(ET_K_MISC, launch_identity_maps(T, L, out->kept_idx_dev, out->cu_tokens_dev,
                                             out->seg_start_dev, s));
  }

  const bool narrow = is_narrow(e);
  bool finished = false;                   // out->tokens_dev is written
  // patch embedding: x = patches * Wp^T + bp + pos_emb[l]
  ET_TIMED(ET_K_IM2COL, launch_im2col(frames_dev, T, c.channels, c.image_h, c.image_w, c.patch, e->Kp_pad, w.hid, s));
  {
    GemmArgs g{w.hid, e->Kp_pad, e->patch_w, e->patch_b, e->pos_emb, D, L, w.x, D, T * L, D, e->Kp_pad, EPI_BIAS_RES};
    if (!narrow && takes_pieces(e, T * L)) {
      g.stats_out = w.pieces;
      g.stats_ld = w.piece_ld;
    }
    ET_TIMED(ET_K_GEMM_PATCH, launch_gemm(g, s));
  }

  bool ragged = false, selected = false, first_stage = true;
  bool have_pieces = true;         // w.pieces belongs to w.x: not after a stage has replaced it
  int n_segments = T, next_merge = 0;
  auto merges_at = [&](int i) { return compress && policy && !selected && next_merge < n_merge && merge_layers[next_merge] == i; };
  auto selects_at = [&](int i) { return compress && !selected && i == merge_layer; };
  for (int i = 0; i <= c.n_layers; ++i) {
    const bool merge_here = merges_at(i), select_here = selects_at(i);
    if (merge_here || select_here) have_pieces = false;
    if (policy && (merge_here || select_here)) {
      MergeWs mw = carve_merge(w.merge, T, L, D);
      int32_t *info = mw.n_seg + 8;
      mw.merged = spare;
      const PlanStep step{merge_here ? 1 : 0, select_here ? 1 : 0, first_stage ? 1 : 0, T};
      HostCell cell;
      int rc = enqueue_policy_stage(w.x, n_frames, L, D, *policy, step, mw, first_stage ? out->frame_sim_dev : nullptr,
                                    out->seg_start_dev, out->kept_idx_dev, out->cu_tokens_dev, w.x, info, s,
                                    &e->prof, select_here ? plan : nullptr, cell.ptr, cell.ptr ? e->count_ready : nullptr,
                                    (select_here && by_attention) ? w.att_score : nullptr);
      if (rc) return rc;
      if (!select_here) std::swap(w.x, spare);      // frames keep all L tokens: the merged frames are the residual stream
      int32_t hi[5] = {0, 0, 0, 0, 0};
      if (cell.ptr) {        // the counts are final after the plan: merge and selection still run while the next blocks are enqueued
        ET_HIP(hipEventSynchronize(e->count_ready));
        memcpy(hi, cell.ptr, sizeof(hi));
        cell.done = true;
      } else {
        ET_HIP(hipMemcpyAsync(hi, info, sizeof(hi), hipMemcpyDeviceToHost, s));
        ET_HIP(hipStreamSynchronize(s));
      }
      if (hi[0] < 1 || hi[0] > n_frames || hi[1] < 1 || hi[1] > T) {
        set_error("plan read back from the device is inconsistent (N = %d, segments = %d)", hi[0], hi[1]);
        return ET_ERR_HIP;
      }
      n_frames = hi[0];
      n_segments = hi[1];
      first_stage = false;
      if (merge_here) ++next_merge;
      if (select_here) {
        if (hi[2] < hi[0] || hi[2] > T * L || hi[3] < 1 || hi[3] > L || hi[4] < 1 || hi[4] > L) {
          set_error("token counts read back from the device are inconsistent (tokens = %d)", hi[2]);
          return ET_ERR_HIP;
        }
        rows = hi[2];
        max_len = hi[3] > hi[4] ? hi[3] : hi[4];
        ragged = policy->select_mode == ET_SELECT_DECOUPLED && hi[3] != hi[4];
        cu = out->cu_tokens_dev;
        selected = true;
        e->prof.phase = 1;
      } else {
        rows = n_frames * L;     // still L tokens per frame
      }
    } else if (select_here) {
      const MergeWs mw = carve_merge(w.merge, T, L, D);
      k = et_keep_count(L, keep_ratio);
      // The segment count is final after the scan: the host waits for that kernel only and enqueues the
      // next blocks while the merge, the selection and the compaction still run.
      const EarlyCount early{e->count_host, e->count_ready};
      *e->count_host = 0;
      int rc = enqueue_merge_stage(w.x, T, L, D, sim_threshold, k, mw, out->frame_sim_dev, out->seg_start_dev,
                                   out->kept_idx_dev, out->cu_tokens_dev, w.x, s, &e->prof, &early);
      if (rc) return rc;
      ET_HIP(hipEventSynchronize(e->count_ready));
      const int32_t n_seg = *e->count_host;
      if (n_seg < 1 || n_seg > T) {
        set_error("segment count %d read back from the device is outside [1, T = %d]", n_seg, T);
        return ET_ERR_HIP;
      }
      n_frames = n_segments = n_seg;
      rows = n_seg * k;
      max_len = k;
      cu = out->cu_tokens_dev;
      selected = true;
      e->prof.phase = 1;
    }
    if (i < c.n_layers && narrow) {        // all blocks up to the next stage
      int last = i + 1;
      while (last < c.n_layers && !merges_at(last) && !selects_at(last)) ++last;
      finished = last == c.n_layers && !merges_at(last) && !selects_at(last);
      int rc = run_narrow_blocks(e, i, last, w, ragged ? cu : nullptr, n_frames, max_len, finished && c.has_final_ln, finished ? out->tokens_dev : w.x, s);
      if (rc) return rc;
      if (by_attention && !selected && last == merge_layer)
        ET_TIMED(ET_K_SCORE, launch_attention_scores(w.qkv, n_frames, max_len, c.n_heads, e->hd, w.score_ws, w.att_score, s));
      i = last - 1;
    } else if (i < c.n_layers) {
      const bool with_scores = by_attention && !selected && i == merge_layer - 1;
      int rc;
      if ((rc = run_block(e, i, w, rows, cu, n_frames, max_len, ragged, have_pieces, s, with_scores))) return rc;
      have_pieces = true;
    }
  }
  if (plan) plan->n_segments = n_segments;
  if (finished) {
    // (by the last run of blocks)
  } else if (c.has_final_ln) {
    ET_TIMED(ET_K_LAYERNORM, launch_layernorm(w.x, e->final_g, e->final_b, c.ln_eps, rows, D,
                                              out->tokens_dev, s));
  } else {
    ET_HIP(hipMemcpyAsync(out->tokens_dev, w.x, (size_t)rows * D * 2, hipMemcpyDeviceToDevice, s));
  }
  ET_HIP(hipStreamSynchronize(s));
  int rc = e->prof.collect();
  if (rc) return rc;
  out->n_frames_out = n_frames;
  out->n_tokens = rows;
  return ET_OK;
}

extern "C" {

int et_encode_clip(et_encoder *e, const float *frames_dev, int32_t T, int32_t merge_layer,
                   float sim_threshold, float keep_ratio, void *workspace_dev, size_t workspace_bytes,
                   void *hip_stream, et_output *out) {
  return encode_impl(e, frames_dev, T, merge_layer, sim_threshold, keep_ratio, nullptr, nullptr, 0,
                     workspace_dev, workspace_bytes, hip_stream, out, nullptr);
}

int et_encode_clip_policy(et_encoder *e, const float *frames_dev, int32_t T, int32_t merge_layer,
                          const et_policy *policy, void *workspace_dev, size_t workspace_bytes,
                          void *hip_stream, et_output *out, et_plan_out *plan) {
  ET_REQUIRE(merge_layer < 0 || policy != nullptr, "policy is NULL");
  const int32_t layers[1] = {merge_layer};
  return encode_impl(e, frames_dev, T, merge_layer, 0.f, 1.f, policy, layers, merge_layer >= 0 ? 1 : 0,
                     workspace_dev, workspace_bytes, hip_stream, out, plan);
}

int et_encode_clip_multi(et_encoder *e, const float *frames_dev, int32_t T, const int32_t *merge_layers,
                         int32_t n_merge_layers, int32_t select_layer, const et_policy *policy,
                         void *workspace_dev, size_t workspace_bytes, void *hip_stream, et_output *out,
                         et_plan_out *plan) {
  ET_REQUIRE(e != nullptr, "encoder is NULL");
  ET_REQUIRE(policy != nullptr, "policy is NULL");
  ET_REQUIRE(n_merge_layers >= 0 && n_merge_layers <= 64, "n_merge_layers = %d outside [0, 64]", n_merge_layers);
  ET_REQUIRE(n_merge_layers == 0 || merge_layers != nullptr, "merge_layers is NULL");
  ET_REQUIRE(select_layer >= 0 && select_layer <= e->cfg.n_layers, "select_layer = %d outside [0, n_layers = %d]",
             select_layer, e->cfg.n_layers);
  for (int i = 0; i < n_merge_layers; ++i) {
    ET_REQUIRE(merge_layers[i] >= 0 && merge_layers[i] <= select_layer,
               "merge_layers[%d] = %d outside [0, select_layer = %d]", i, merge_layers[i], select_layer);
    ET_REQUIRE(i == 0 || merge_layers[i] > merge_layers[i - 1], "merge_layers must be strictly ascending");
  }
  return encode_impl(e, frames_dev, T, select_layer, 0.f, 1.f, policy, merge_layers, n_merge_layers,
                     workspace_dev, workspace_bytes, hip_stream, out, plan);
}

int et_profile_enable(et_encoder *e, int32_t on) {
  ET_REQUIRE(e != nullptr, "encoder is NULL");
  e->prof.on = on != 0;
  return ET_OK;
}

int et_profile_read(et_encoder *e, double *ms, int64_t *launches, int32_t reset) {
  ET_REQUIRE(e && ms && launches, "a pointer argument is NULL");
  for (int i = 0; i < 2 * ET_K_COUNT; ++i) {
    ms[i] = e->prof.ms[i];
    launches[i] = e->prof.launches[i];
    if (reset) { e->prof.ms[i] = 0; e->prof.launches[i] = 0; }
  }
  return ET_OK;
}

const char *et_kernel_name(int32_t kind) {
  static const char *names[ET_K_COUNT] = {"im2col", "gemm_patch", "layernorm", "gemm_qkv", "attention",
                                          "gemm_out", "gemm_fc1", "gemm_fc2", "similarity", "scan",
                                          "merge", "select", "compact", "misc", "score"};
  return (kind >= 0 && kind < ET_K_COUNT) ? names[kind] : "?";
}

size_t et_attention_scores_scratch_bytes(int32_t n_frames, int32_t L, int32_t n_heads) {
  if (n_frames < 0 || L < 0 || n_heads < 1) return 0;
  return attention_scores_workspace_bytes(n_frames, L, n_heads);
}

int et_attention_scores(const uint16_t *qkv_dev, int32_t n_frames, int32_t L, int32_t n_heads, int32_t head_dim,
                        void *scratch_dev, float *score_dev, void *hip_stream) {
  ET_REQUIRE(qkv_dev && scratch_dev && score_dev, "a pointer argument is NULL");
  ET_REQUIRE(n_frames >= 0 && L >= 1 && n_heads >= 1 && (int64_t)n_frames * L <= (1 << 24),
             "n_frames = %d, L = %d, n_heads = %d out of range", n_frames, L, n_heads);
  return launch_attention_scores(qkv_dev, n_frames, L, n_heads, head_dim, scratch_dev, score_dev,
                                 static_cast<hipStream_t>(hip_stream));
}

int et_encoder_block_qkv(et_encoder *e, int32_t layer, const uint16_t *x_dev, int32_t rows, float *rstd_dev,
                         uint16_t *qkv_dev, void *hip_stream) {
  ET_REQUIRE(e != nullptr, "encoder is NULL");
  ET_REQUIRE(layer >= 0 && layer < e->cfg.n_layers, "layer = %d outside [0, n_layers = %d)", layer, e->cfg.n_layers);
  ET_REQUIRE(x_dev && rstd_dev && qkv_dev, "a pointer argument is NULL");
  ET_REQUIRE(rows >= 0 && (double)rows * e->D * 3 < 2.0e9, "rows = %d out of range", rows);
  if (rows == 0) return ET_OK;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int D = e->D;
  const LayerDev &lw = e->layers[layer];
  int rc;
  if (is_narrow(e)) {                      // (the arithmetic of narrow_blocks_kernel)
    if ((rc = launch_piece_scale(x_dev, e->cfg.ln_eps, rows, D, rstd_dev, s))) return rc;
    return launch_gemm(GemmArgs{x_dev, D, lw.wqkv, lw.bqkv, nullptr, 0, 1, qkv_dev, 3 * D, rows, 3 * D, D, EPI_BIAS, rstd_dev}, s, kCfgStrip);
  }
  // run_block's two ways to the row scales; where it takes them from the pieces of a row, they are combined here by a kernel
  // of its own, with the same arithmetic, and the projection runs in the tiling that takes pieces
  const bool by_pieces = takes_pieces(e, rows);
  if (by_pieces) rc = launch_piece_scale(x_dev, e->cfg.ln_eps, rows, D, rstd_dev, s);
  else rc = launch_rowstats(x_dev, e->cfg.ln_eps, rows, D, rstd_dev, s);
  if (rc) return rc;
  const GemmArgs g{x_dev, D, lw.wqkv, lw.bqkv, nullptr, 0, 1, qkv_dev, 3 * D, rows, 3 * D, D, EPI_BIAS, rstd_dev};
  return launch_gemm(g, s, -1, by_pieces);
}

int et_layernorm(const uint16_t *x_dev, const float *gamma_dev, const float *beta_dev, float eps,
                 int32_t rows, int32_t D, uint16_t *y_dev, void *hip_stream) {
  ET_REQUIRE(x_dev && gamma_dev && beta_dev && y_dev, "a pointer argument is NULL");
  ET_REQUIRE(rows >= 0 && D >= 8 && D % 8 == 0, "rows = %d, D = %d out of range", rows, D);
  return launch_layernorm(x_dev, gamma_dev, beta_dev, eps, rows, D, y_dev, static_cast<hipStream_t>(hip_stream));
}

int et_attention(const uint16_t *qkv_dev, const int32_t *cu_tokens_dev, int32_t n_frames, int32_t max_len,
                 int32_t n_heads, int32_t head_dim, uint16_t *out_dev, void *hip_stream) {
  ET_REQUIRE(qkv_dev && cu_tokens_dev && out_dev, "a pointer argument is NULL");
  ET_REQUIRE(n_frames >= 0 && max_len >= 0 && n_heads >= 1, "n_frames/max_len/n_heads out of range");
  if (!head_dim_supported(head_dim)) {
    set_error("head_dim = %d is not instantiated (16, 32, 64, 72, 80, 96, 128)", head_dim);
    return ET_ERR_UNSUPPORTED;
  }
  return launch_attention(qkv_dev, cu_tokens_dev, n_frames, max_len, n_heads, head_dim, out_dev,
                          static_cast<hipStream_t>(hip_stream));
}

int et_attention_uniform(const uint16_t *qkv_dev, int32_t n_frames, int32_t len, int32_t n_heads,
                         int32_t head_dim, uint16_t *out_dev, void *hip_stream) {
  ET_REQUIRE(qkv_dev && out_dev, "a pointer argument is NULL");
  ET_REQUIRE(n_frames >= 0 && len >= 0 && n_heads >= 1, "n_frames/len/n_heads out of range");
  if (!head_dim_supported(head_dim)) {
    set_error("head_dim = %d is not instantiated (16, 32, 64, 72, 80, 96, 128)", head_dim);
    return ET_ERR_UNSUPPORTED;
  }
  ET_REQUIRE((double)n_frames * len * n_heads * head_dim * 3 < 2.0e9, "qkv exceeds 2^31 elements");
  if (n_frames == 0 || len == 0) return ET_OK;
  return launch_attention_uniform(qkv_dev, n_frames, len, n_heads, head_dim, out_dev,
                                  static_cast<hipStream_t>(hip_stream));
}

int et_gemm_bf16(const uint16_t *a_dev, const uint16_t *w_dev, const float *bias_dev, const uint16_t *res_dev,
                 int32_t M, int32_t N, int32_t K, int32_t epilogue, int32_t tile_config, uint16_t *c_dev,
                 void *hip_stream) {
  ET_REQUIRE(tile_config >= -1 && tile_config < gemm_config_count(), "tile_config = %d unknown", tile_config);
  ET_REQUIRE(a_dev && w_dev && bias_dev && c_dev, "a pointer argument is NULL");
  ET_REQUIRE(M >= 1 && N >= 8 && K >= 8 && N % 8 == 0 && K % 8 == 0, "M = %d, N = %d, K = %d out of range", M, N, K);
  ET_REQUIRE(epilogue >= 0 && epilogue <= 2, "epilogue = %d unknown", epilogue);
  ET_REQUIRE(epilogue != EPI_BIAS_RES || res_dev, "res_dev is NULL for the residual epilogue");
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int Kp = round_up(K, 64), Np = round_up(N, 256);
  uint16_t *a = nullptr, *w = nullptr;
  float *b = nullptr;
  int rc = ET_OK;
  hipError_t he;
  if ((he = hipMalloc((void **)&a, (size_t)M * Kp * 2)) != hipSuccess ||
      (he = hipMalloc((void **)&w, (size_t)Np * Kp * 2)) != hipSuccess ||
      (he = hipMalloc((void **)&b, (size_t)Np * 4)) != hipSuccess) {
    (void)hipGetLastError();
    set_error("device allocation failed in et_gemm_bf16");
    rc = ET_ERR_ALLOC;
  }
  auto step = [&](hipError_t err, const char *what) {
    if (rc == ET_OK && err != hipSuccess) rc = hip_fail(err, what, __FILE__, __LINE__);
  };
  if (rc == ET_OK) {
    step(hipMemsetAsync(a, 0, (size_t)M * Kp * 2, s), "memset a");
    step(hipMemsetAsync(w, 0, (size_t)Np * Kp * 2, s), "memset w");
    step(hipMemsetAsync(b, 0, (size_t)Np * 4, s), "memset bias");
    step(hipMemcpy2DAsync(a, (size_t)Kp * 2, a_dev, (size_t)K * 2, (size_t)K * 2, M, hipMemcpyDeviceToDevice, s), "copy a");
    step(hipMemcpy2DAsync(w, (size_t)Kp * 2, w_dev, (size_t)K * 2, (size_t)K * 2, N, hipMemcpyDeviceToDevice, s), "copy w");
    step(hipMemcpyAsync(b, bias_dev, (size_t)N * 4, hipMemcpyDeviceToDevice, s), "copy bias");
  }
  if (rc == ET_OK) {
    GemmArgs g{a, Kp, w, b, res_dev, N, M, c_dev, N, M, N, Kp, epilogue};
    rc = launch_gemm(g, s, tile_config);
  }
  hipError_t se = hipStreamSynchronize(s);
  if (rc == ET_OK && se != hipSuccess) rc = hip_fail(se, "hipStreamSynchronize", __FILE__, __LINE__);
  if (a) (void)hipFree(a);
  if (w) (void)hipFree(w);
  if (b) (void)hipFree(b);
  return rc;
}

}  // extern "C"
