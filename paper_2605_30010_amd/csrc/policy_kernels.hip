// Paper-exact compression stage: Eq. 1 with smoothing, Alg. 1 (head and tail of a segment kept,
// middle frames fused pairwise with similarity weights, Eq. 2-3), Alg. 2 (dynamic frames: global
// top-k with the re-scaled count of Eq. 5; static frames: arg-max per local window, Eq. 6) and
// the gather of Eq. 7 with per-frame token counts.
//
// Readings of points the paper leaves open are stated at plan_kernel.  The similarity kernel of
// the simple path is reused; this file adds the plan builder (all lanes of a wavefront up to 64 frames, O(T) steps on
// one lane above), a weighted-range merge, the per-frame selection with two modes and a ragged gather.
#include "select_common.h"

namespace et {

namespace {

constexpr int kRowsPerBlock = 4;

// ---------------------------------------------------------------------------------------
// Plan builder.  info[0] = N output frames, info[1] = segments, info[2] = total kept tokens,
// info[3] = tokens per dynamic frame, info[4] = tokens per static frame.
//  - Eq. 1: s_hat restarts at every segment start (first pair of a segment: s_hat = s_t); a NaN
//    value opens a segment.
//  - Alg. 1: the pair (F_i, F_{i+1}) is eligible only if both are middle frames of the segment;
//    fused with weights s_i / (s_i + s_{i+1}), s_{i+1} / (s_i + s_{i+1}), s_i = Sim(F_i, F_{i+1}).
//  - Eq. 5 (as a count): r_hat = clamp(floor(ratio * T * L / N + 0.5), 1, L).
//  - Eq. 6: w = L / r_hat (integer division), M = ceil(L / w) windows.
// ---------------------------------------------------------------------------------------
// What the one lane builds: segments, then the output frames as (first, count) over the current frames.
struct PlanLists {
  int32_t *seg, *first, *count, *dyn;
  float *w;
};

// Eq. 1.  The contraction is written out: left to the compiler, which of the two products is rounded first depends on how
// it unrolls a loop, and a similarity that sits on the threshold would fall on one side or the other with the clip's length.
__device__ __forceinline__ float smoothed(float alpha, float now, float prev) { return fmaf(1.0f - alpha, prev, alpha * now); }

__device__ __forceinline__ void build_plan(const float *sim, int T, const PolicyArgs &p, const PlanLists &o, int &n_seg_out, int &n_out) {
  int n_seg = 0, N = 0;
  o.seg[0] = 0;
  float prev = 0.f;
  bool fresh = true;
  for (int t = 1; t < T; ++t) {
    const float sv = sim[t - 1];
    const float cur = fresh ? sv : smoothed(p.alpha, sv, prev);
    if (!(cur >= p.tau_seg)) {
      o.seg[++n_seg] = t;
      fresh = true;
    } else {
      prev = cur;
      fresh = false;
    }
  }
  o.seg[++n_seg] = T;
  auto emit = [&](int first, int count, float w0, float w1, int dyn) {
    o.first[N] = first;
    o.count[N] = count;
    o.dyn[N] = dyn;
    o.w[2 * N] = w0;
    o.w[2 * N + 1] = w1;
    ++N;
  };
  for (int sgi = 0; sgi < n_seg; ++sgi) {
    const int a = o.seg[sgi], b = o.seg[sgi + 1];
    if (p.merge_mode == ET_MERGE_MEAN) {
      emit(a, b - a, 0.f, 0.f, 1);                 // uniform weights: handled as sum / count
      continue;
    }
    const int k = b - a - 1;
    emit(a, 1, 1.f, 0.f, 1);
    int i = 1;
    while (i < k) {
      const float si = sim[a + i];                 // Sim(F_i, F_{i+1})
      if (i + 1 <= k - 1 && si > p.tau_merge && si > sim[a + i + 1]) {
        const float sj = sim[a + i + 1];
        emit(a + i, 2, si / (si + sj), sj / (si + sj), 0);
        i += 2;
      } else {
        emit(a + i, 1, 1.f, 0.f, 0);
        i += 1;
      }
    }
    if (k >= 1) emit(a + k, 1, 1.f, 0.f, 1);
  }
  n_seg_out = n_seg;
  n_out = N;
}

// The same for up to 64 frames, one per lane: only the smoothing of Eq. 1 is a chain (a few scalar steps per frame); the
// left-to-right walk of Alg. 1 takes the lowest eligible pair, strikes out its two frames and goes on, on a bit
// mask; positions are population counts.
__device__ __forceinline__ void build_plan_64(const float *sim, int T, const PolicyArgs &p, const PlanLists &o, int lane,
                                              int &n_seg_out, int &n_out) {
  const float s = lane < T - 1 ? sim[lane] : 0.f;
  auto of_lane = [&](int t) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), t)); };
  unsigned long long starts = 1ull;
  float prev = 0.f;
  bool fresh = true;
  for (int t = 1; t < T; ++t) {
    const float sv = of_lane(t - 1);
    const float cur = fresh ? sv : smoothed(p.alpha, sv, prev);
    if (!(cur >= p.tau_seg)) {
      starts |= 1ull << t;
      fresh = true;
    } else {
      prev = cur;
      fresh = false;
    }
  }
  const unsigned long long below = (1ull << lane) - 1ull, mine = 1ull << lane, later = starts & ~(below | mine);
  const int b = later ? __builtin_ctzll(later) : T;             // end of this lane's segment
  const bool head = (starts & mine) != 0, tail = lane == b - 1;
  const int a = 63 - __builtin_clzll(starts & (below | mine));
  unsigned long long fused = 0ull, emits = starts;
  const float s_next = __shfl_down(s, 1);
  if (p.merge_mode != ET_MERGE_MEAN) {
    // F_i and F_{i+1} both middle frames
    unsigned long long left = __ballot(lane < T && lane > a && lane + 1 <= b - 2 && s > p.tau_merge && s > s_next);
    while (left) {
      const int i = __builtin_ctzll(left);
      fused |= 1ull << i;
      left &= ~(3ull << i);
    }
    emits = (T < 64 ? (1ull << T) - 1ull : ~0ull) & ~(fused << 1);
  }
  if (emits & mine) {
    const int n = __popcll(emits & below);
    const bool pair = (fused & mine) != 0, mean = p.merge_mode == ET_MERGE_MEAN;
    o.first[n] = lane;
    o.count[n] = mean ? b - a : (pair ? 2 : 1);
    o.dyn[n] = head || tail;
    o.w[2 * n] = mean ? 0.f : (pair ? s / (s + s_next) : 1.f);
    o.w[2 * n + 1] = pair ? s_next / (s + s_next) : 0.f;
  }
  if (head) o.seg[__popcll(starts & below)] = lane;
  n_seg_out = __popcll(starts);
  n_out = __popcll(emits);
}

// One workgroup.  With st.do_plan all its wavefronts first take the frames' similarities from the sums that the similarity kernel
// left.  The rest is one wavefront's: up to 64 frames are planned by all lanes, longer clips by lane 0 on LDS copies (T <= kPlanLds) or
// on global memory, where every step is a round trip; the arrays are written by all lanes.  Bound: a chain of round trips.  40
// frames: 3.7 us for the means, a launch boundary and 7.0 us for the plan -> 8.0 us; the stage's call 99.3 -> 96.4.
constexpr int kPlanLds = 1024, kPlanThreads = 1024;

// Behind it every lane of the wavefront sees what its lanes wrote, in LDS or in memory.
__device__ __forceinline__ void wave_meets() {
  __threadfence_block();
  __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(kPlanThreads) void plan_kernel(
    const float *__restrict__ part, int n_part, float *sim, int T, int L, PolicyArgs p, int k_uniform, PlanStep st, int32_t *__restrict__ seg_start,
    int32_t *__restrict__ frame_first, int32_t *__restrict__ frame_count, int32_t *__restrict__ frame_dyn,
    float *__restrict__ frame_w, int32_t *orig_first, int32_t *orig_count, int32_t *__restrict__ cu_tokens, int32_t *__restrict__ info,
    PlanOut out) {
  // T = current number of frames.  st.do_plan: build segments and output frames from part [T-1, n_part] (else the
  // identity plan over the T current frames, dynamic flags left as they are).  st.do_counts: token
  // counts and offsets of the selection.  orig_first / orig_count: range of ORIGINAL frames behind
  // each current frame (st.init_orig: identity, first stage), updated in place; seg_start is
  // written in original frame indices.  out: copies of the final plan for the caller (each may be NULL).
  __shared__ float l_sim[kPlanLds], l_w[2 * kPlanLds];
  __shared__ int32_t l_seg[kPlanLds + 1], l_first[kPlanLds], l_count[kPlanLds], l_dyn[kPlanLds];
  __shared__ int head[2];
  const int lane = threadIdx.x;                    // (the plan's own wavefront)
  int N = T, n_segments = T;
  int my_first = lane, my_count = 1, my_dyn = 1;   // of output frame `lane`: up to 64 frames nothing is read back
  if (st.do_plan) {
    mean_over_positions(part, n_part, T, L, sim, l_sim, kPlanLds);
    __threadfence_block();
    __syncthreads();
  }
  if (threadIdx.x >= kWave) return;                // (no barrier of the workgroup behind this line)
  if (st.do_plan) {
    const bool in_lds = T <= kPlanLds;             // (uniform)
    if (T <= kWave) {
      int n_seg = 0, n = 0;
      build_plan_64(l_sim, T, p, PlanLists{l_seg, l_first, l_count, l_dyn, l_w}, lane, n_seg, n);
      if (lane == 0) {
        head[0] = n_seg;
        head[1] = n;
      }
    } else if (lane == 0) {
      int n_seg = 0, n = 0;
      if (in_lds) build_plan(l_sim, T, p, PlanLists{l_seg, l_first, l_count, l_dyn, l_w}, n_seg, n);
      else build_plan(sim, T, p, PlanLists{seg_start, frame_first, frame_count, frame_dyn, frame_w}, n_seg, n);
      head[0] = n_seg;
      head[1] = n;
    }
    wave_meets();
    const int n_seg = n_segments = head[0];
    N = head[1];
    // segment starts and frame ranges in original frame indices: 64 entries at a time are read before they are
    // written, and entry n only needs entries >= n
    for (int i0 = 0; i0 < n_seg; i0 += kWave) {
      const int i = i0 + lane;
      if (i < n_seg) {
        const int f = in_lds ? l_seg[i] : seg_start[i];
        seg_start[i] = st.init_orig ? f : orig_first[f];
      }
    }
    if (lane == 0) seg_start[n_seg] = st.t_orig;
    for (int n0 = 0; n0 < N; n0 += kWave) {
      const int n = n0 + lane;
      int of = 0, oe = 0, dyn = 0;
      if (n < N) {
        const int f = in_lds ? l_first[n] : frame_first[n], c = in_lds ? l_count[n] : frame_count[n], l = f + c - 1;
        of = st.init_orig ? f : orig_first[f];
        oe = st.init_orig ? l + 1 : orig_first[l] + orig_count[l];
        dyn = in_lds ? l_dyn[n] : frame_dyn[n];
        if (in_lds) {
          frame_first[n] = f;
          frame_count[n] = c;
          frame_dyn[n] = dyn;
          frame_w[2 * n] = l_w[2 * n];
          frame_w[2 * n + 1] = l_w[2 * n + 1];
        }
      }
      if (!st.init_orig) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (all 64 entries have been read)
      if (n0 == 0) my_first = of, my_count = oe - of, my_dyn = dyn;
      if (n < N) {
        orig_first[n] = of;
        orig_count[n] = oe - of;
      }
    }
    if (lane == 0) info[1] = n_seg;
  } else {
    for (int n = lane; n < N; n += kWave) {
      frame_first[n] = n;
      frame_count[n] = 1;
      frame_w[2 * n] = 1.f;
      frame_w[2 * n + 1] = 0.f;
      if (st.init_orig) {
        frame_dyn[n] = 1;
        orig_first[n] = n;
        orig_count[n] = 1;
      }
    }
    if (st.init_orig) {
      for (int i = lane; i <= T; i += kWave) seg_start[i] = i;
      if (lane == 0) info[1] = T;
    } else {
      n_segments = info[1];
      if (lane < N) {
        my_first = orig_first[lane];
        my_count = orig_count[lane];
        my_dyn = frame_dyn[lane];
      }
    }
  }
  if (lane == 0) info[0] = N;
  if (lane == 0 && out.header) {
    out.header[0] = N;
    out.header[1] = n_segments;
  }
  if (N > kWave) wave_meets();
  for (int n = lane; n < N; n += kWave) {
    if (out.first) out.first[n] = N > kWave ? orig_first[n] : my_first;
    if (out.count) out.count[n] = N > kWave ? orig_count[n] : my_count;
    if (out.dyn) out.dyn[n] = N > kWave ? frame_dyn[n] : my_dyn;
  }
  if (!st.do_counts) return;
  int n_dyn_tok, n_sta_tok;
  if (p.select_mode == ET_SELECT_UNIFORM) {
    n_dyn_tok = n_sta_tok = k_uniform;
  } else {
    double v = floor((double)p.ratio * (double)st.t_orig * (double)L / (double)N + 0.5);
    int r_hat = v < 1.0 ? 1 : (v > (double)L ? L : (int)v);
    const int w = L / r_hat;
    n_dyn_tok = r_hat;
    n_sta_tok = (L + w - 1) / w;
  }
  int total = 0;                                   // tokens before the 64 frames at n0
  for (int n0 = 0; n0 < N; n0 += kWave) {
    const int n = n0 + lane, here = N - n0 < kWave ? N - n0 : kWave;
    const bool dyn = n < N && (p.select_mode == ET_SELECT_UNIFORM || (N > kWave ? frame_dyn[n] : my_dyn));
    const unsigned long long m = __ballot(dyn);
    const int before = __popcll(m & ((1ull << lane) - 1ull)), all = __popcll(m);
    if (n < N) cu_tokens[n] = total + before * n_dyn_tok + (lane - before) * n_sta_tok;
    total += all * n_dyn_tok + (here - all) * n_sta_tok;
  }
  if (lane == 0) {
    cu_tokens[N] = total;
    info[2] = total;
    info[3] = n_dyn_tok;
    info[4] = n_sta_tok;
    if (out.header) {
      out.header[2] = total;
      out.header[3] = n_dyn_tok;
      out.header[4] = n_sta_tok;
    }
  }
}

// ---------------------------------------------------------------------------------------
// Weighted-range merge: output frame n = sum over its source frames.  Three cases, all fp32 with
// one rounding to bf16 and the score taken from the unrounded value: a single source frame
// (bit copy), a uniform mean (ascending-t sum divided by the count, exactly the simple path's
// arithmetic), a fused pair w0 x0 + w1 x1 (Eq. 3).
// ---------------------------------------------------------------------------------------
template <int NV>
__global__ __launch_bounds__(kRowsPerBlock * kWave) void plan_merge_kernel(
    const uint16_t *__restrict__ x, int L, int D, const int32_t *__restrict__ info,
    const int32_t *__restrict__ frame_first, const int32_t *__restrict__ frame_count,
    const float *__restrict__ frame_w, int uniform_mean, uint16_t *__restrict__ merged,
    float *__restrict__ score) {
  const int n = blockIdx.y;
  if (n >= info[0]) return;
  const int lane = threadIdx.x & 63;
  const int l = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
  if (l >= L) return;
  const int a = frame_first[n], cnt = frame_count[n];
  const size_t frame_stride = (size_t)L * D;
  const uint16_t *p = x + (size_t)a * frame_stride + (size_t)l * D;
  Row<NV> acc, r;
  uint4 raw[NV];
  if (uniform_mean || cnt == 1) {
#pragma unroll
    for (int i = 0; i < NV * 8; ++i) acc.v[i] = 0.f;
    for (int t = 0; t < cnt; ++t) {
      load_row<NV>(p + (size_t)t * frame_stride, D, lane, raw);
      unpack_row<NV>(raw, r);
#pragma unroll
      for (int i = 0; i < NV * 8; ++i) acc.v[i] += r.v[i];
    }
    const float len = (float)cnt;
#pragma unroll
    for (int i = 0; i < NV * 8; ++i) acc.v[i] = acc.v[i] / len;
  } else {                                           // cnt == 2 by construction
    const float w0 = frame_w[2 * n], w1 = frame_w[2 * n + 1];
    load_row<NV>(p, D, lane, raw);
    unpack_row<NV>(raw, r);
#pragma unroll
    for (int i = 0; i < NV * 8; ++i) acc.v[i] = w0 * r.v[i];
    load_row<NV>(p + frame_stride, D, lane, raw);
    unpack_row<NV>(raw, r);
#pragma unroll
    for (int i = 0; i < NV * 8; ++i) acc.v[i] = fmaf(w1, r.v[i], acc.v[i]);
  }
  float z = 0.f;
  uint16_t *q = merged + ((size_t)n * L + l) * D;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const float *m = &acc.v[j * 8];
#pragma unroll
    for (int e = 0; e < 8; ++e) z = fmaf(m[e], m[e], z);
    const int c = (j * kWave + lane) * 8;
    if (c < D) {
      uint4 o;
      o.x = pack_bf16x2(m[0], m[1]); o.y = pack_bf16x2(m[2], m[3]);
      o.z = pack_bf16x2(m[4], m[5]); o.w = pack_bf16x2(m[6], m[7]);
      *reinterpret_cast<uint4 *>(q + c) = o;
    }
  }
  z = wave_sum(z);
  if (lane == 0) score[(size_t)n * L + l] = z;
}

// ---------------------------------------------------------------------------------------
// Per-frame selection with ragged output.  Dynamic frames (and every frame in uniform mode): the
// radix select of the simple path (select_common.h) with k = cu[n+1] - cu[n].  Static frames: one thread per local
// window of w consecutive positions, arg-max of the key, lowest position on ties.
// ---------------------------------------------------------------------------------------
__global__ __launch_bounds__(kSelThreads) void select_policy_kernel(
    const float *__restrict__ score, const int32_t *__restrict__ info, const int32_t *__restrict__ frame_dyn,
    const int32_t *__restrict__ cu_tokens, int L, int all_topk, int32_t *__restrict__ kept) {
  extern __shared__ uint32_t keys[];     // [L]
  __shared__ SelectShared sh;

  const int n = blockIdx.x;
  const int tid = threadIdx.x;
  // (fetched before the frame count is known: entry n < gridDim.x lies inside every buffer whether or not the frame exists, and the
  // loads overlap)
  const int n_frames = info[0], r_hat = info[3], dyn = frame_dyn[n], out0 = cu_tokens[n], out1 = cu_tokens[n + 1];
  stage_keys(score + (size_t)n * L, L, keys);
  if (n >= n_frames) return;
  const int k = out1 - out0;
  __syncthreads();
  int32_t *dst = kept + out0;

  if (!all_topk && !dyn) {                  // static frame: local windows (Eq. 6)
    const int w = L / r_hat;
    for (int j = tid; j < k; j += kSelThreads) {
      const int lo = j * w, hi = min(lo + w, L);
      int best = lo;
      uint32_t kb = keys[lo];
      for (int i = lo + 1; i < hi; ++i) {
        const uint32_t ki = keys[i];
        if (ki > kb) { kb = ki; best = i; }
      }
      dst[j] = best;
    }
    return;
  }

  radix_select_emit(keys, L, k, dst, sh);
}

// Gather with per-frame counts: out[cu[n] + j, :] = merged[n, kept[cu[n] + j], :].
__global__ __launch_bounds__(kRowsPerBlock * kWave) void compact_ragged_kernel(
    const uint16_t *__restrict__ merged, const int32_t *__restrict__ kept, const int32_t *__restrict__ info,
    const int32_t *__restrict__ cu_tokens, int L, int D, uint16_t *__restrict__ out) {
  const int n = blockIdx.y;
  const int n_frames = info[0], out0 = cu_tokens[n], out1 = cu_tokens[n + 1];      // (n < T: inside the array)
  asm volatile("" ::"s"(n_frames), "s"(out0), "s"(out1));                          // (the three loads overlap)
  if (n >= n_frames) return;
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
  if (j >= out1 - out0) return;
  const size_t orow = (size_t)out0 + j;
  const int l = kept[orow];
  if (l < 0 || l >= L) return;
  const uint4 *src = reinterpret_cast<const uint4 *>(merged + ((size_t)n * L + l) * D);
  uint4 *dst = reinterpret_cast<uint4 *>(out + orow * D);
  for (int c = lane; c < D / 8; c += kWave) dst[c] = src[c];
}

}  // namespace

int launch_plan(const float *part, int n_part, float *sim, int T, int L, const PolicyArgs &p, int k_uniform, const PlanStep &st,
                int32_t *seg_start, int32_t *frame_first, int32_t *frame_count, int32_t *frame_dyn,
                float *frame_w, int32_t *orig_first, int32_t *orig_count, int32_t *cu_tokens, int32_t *info,
                const PlanOut &out, hipStream_t s) {
  hipLaunchKernelGGL(plan_kernel, dim3(1), dim3(st.do_plan ? kPlanThreads : kWave), 0, s, part, n_part, sim, T, L, p, k_uniform, st, seg_start, frame_first,
                     frame_count, frame_dyn, frame_w, orig_first, orig_count, cu_tokens, info, out);
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_plan_merge(const uint16_t *x, int T, int L, int D, const int32_t *info, const int32_t *frame_first,
                      const int32_t *frame_count, const float *frame_w, bool uniform_mean, uint16_t *merged,
                      float *score, hipStream_t s) {
  dim3 grid((L + kRowsPerBlock - 1) / kRowsPerBlock, T), block(kRowsPerBlock * kWave);
  ET_DISPATCH_NV(D, hipLaunchKernelGGL(plan_merge_kernel<NV>, grid, block, 0, s, x, L, D, info, frame_first,
                                       frame_count, frame_w, uniform_mean ? 1 : 0, merged, score));
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_select_policy(const float *score, int T, const int32_t *info, const int32_t *frame_dyn,
                         const int32_t *cu_tokens, int L, bool all_topk, int32_t *kept, hipStream_t s) {
  if (L > 15360) {
    set_error("tokens per frame %d above the supported 15360", L);
    return ET_ERR_UNSUPPORTED;
  }
  hipLaunchKernelGGL(select_policy_kernel, dim3(T), dim3(kSelThreads), (size_t)L * sizeof(uint32_t), s, score,
                     info, frame_dyn, cu_tokens, L, all_topk ? 1 : 0, kept);
  ET_LAUNCH_CHECK();
  return ET_OK;
}

int launch_compact_ragged(const uint16_t *merged, const int32_t *kept, int T, const int32_t *info,
                          const int32_t *cu_tokens, int L, int D, uint16_t *out, hipStream_t s) {
  dim3 grid((L + kRowsPerBlock - 1) / kRowsPerBlock, T);
  hipLaunchKernelGGL(compact_ragged_kernel, grid, dim3(kRowsPerBlock * kWave), 0, s, merged, kept, info,
                     cu_tokens, L, D, out);
  ET_LAUNCH_CHECK();
  return ET_OK;
}

}  // namespace et
