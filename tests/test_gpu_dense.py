"""GPU parity of the dense encoder kernels (LayerNorm, MFMA GEMM + epilogues, attention)
against the CPU oracle's definitions, on bf16-representable inputs.

Tolerances: the kernels accumulate in float32 and round the result once to bf16
(relative step 2^-8), so element errors are bounded by about 2^-8 of the result's
magnitude plus float32 accumulation noise; relative L2 errors stay below 4e-3.
"""
import math

import numpy as np
import pytest
import torch

import paper_2605_30010_amd as et
from et_inputs import bf16_bits_to_f32, f32_to_bf16_bits
from oracle import earlytom_oracle as O
from tests._util import bits_to_dev, dev_to_bits, dev_to_f64, rel_l2

pytestmark = pytest.mark.gpu


def _bf(rng, shape, scale=1.0, shift=0.0):
    bits = f32_to_bf16_bits((rng.standard_normal(shape) * scale + shift).astype(np.float32))
    return bits, bf16_bits_to_f32(bits).astype(np.float64)


@pytest.mark.parametrize("rows,D", [(1, 64), (37, 64), (1000, 1152), (5, 4096), (9, 520)])
def test_layernorm_matches_oracle(rows, D):
    rng = np.random.default_rng(rows + D)
    bits, x = _bf(rng, (rows, D), scale=3.0, shift=1.5)
    g = (1 + 0.1 * rng.standard_normal(D)).astype(np.float32)
    b = (0.1 * rng.standard_normal(D)).astype(np.float32)
    ref = O.layer_norm(x, g.astype(np.float64), b.astype(np.float64), 1e-6)
    y = et.et_layernorm(bits_to_dev(bits), torch.from_numpy(g).cuda(), torch.from_numpy(b).cuda(), 1e-6)
    got = dev_to_f64(y)
    assert np.max(np.abs(got - ref) - 2 ** -8 * np.abs(ref)) < 2e-5
    assert rel_l2(got, ref) < 3e-3


@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (300, 192, 128), (1000, 1152, 1152), (257, 4304, 1152),
                                   (513, 1152, 4304), (5, 8, 8), (2050, 3456, 1152), (700, 1152, 592)])
@pytest.mark.parametrize("epi", [0, 1, 2])
def test_gemm_matches_oracle(M, N, K, epi):
    rng = np.random.default_rng(M + N + K + epi)
    a_bits, a = _bf(rng, (M, K))
    w_bits, w = _bf(rng, (N, K), scale=0.05)
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    r_bits, r = _bf(rng, (M, N))
    ref = a @ w.T + bias.astype(np.float64)
    if epi == 1:
        ref = O.gelu_tanh(ref)
    if epi == 2:
        ref = ref + r
    c = et.et_gemm_bf16(bits_to_dev(a_bits), bits_to_dev(w_bits), torch.from_numpy(bias).cuda(), epi,
                        residual=bits_to_dev(r_bits) if epi == 2 else None)
    got = dev_to_f64(c)
    scale = np.sqrt(K) * 0.05 + 1.0
    assert np.max(np.abs(got - ref) - 2 ** -8 * np.abs(ref)) < 2e-4 * scale
    assert rel_l2(got, ref) < 4e-3


@pytest.mark.parametrize("cfg", [0, 1, 2])
def test_gemm_every_tile_configuration(cfg):
    """Each workgroup tiling, on a shape with ragged M, several k-tiles and a partial N tile."""
    rng = np.random.default_rng(cfg)
    M, N, K = 777, 1160, 448
    a_bits, a = _bf(rng, (M, K))
    w_bits, w = _bf(rng, (N, K), scale=0.05)
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    r_bits, r = _bf(rng, (M, N))
    ref = O.gelu_tanh(a @ w.T + bias.astype(np.float64))
    c = et.et_gemm_bf16(bits_to_dev(a_bits), bits_to_dev(w_bits), torch.from_numpy(bias).cuda(), 1,
                        tile_config=cfg)
    got = dev_to_f64(c)
    assert np.max(np.abs(got - ref) - 2 ** -8 * np.abs(ref)) < 5e-4
    assert rel_l2(got, ref) < 4e-3
    ref2 = a @ w.T + bias.astype(np.float64) + r
    c2 = et.et_gemm_bf16(bits_to_dev(a_bits), bits_to_dev(w_bits), torch.from_numpy(bias).cuda(), 2,
                         residual=bits_to_dev(r_bits), tile_config=cfg)
    assert rel_l2(dev_to_f64(c2), ref2) < 4e-3


def test_gemm_residual_in_place():
    rng = np.random.default_rng(5)
    M, N, K = 333, 128, 64
    a_bits, a = _bf(rng, (M, K))
    w_bits, w = _bf(rng, (N, K), scale=0.1)
    r_bits, r = _bf(rng, (M, N))
    bias = torch.zeros(N, dtype=torch.float32, device="cuda")
    res = bits_to_dev(r_bits)
    lib = et.load_library()
    import ctypes as C
    a_d, w_d = bits_to_dev(a_bits), bits_to_dev(w_bits)
    rc = lib.et_gemm_bf16(C.c_void_p(a_d.data_ptr()), C.c_void_p(w_d.data_ptr()), C.c_void_p(bias.data_ptr()),
                          C.c_void_p(res.data_ptr()), M, N, K, 2, -1, C.c_void_p(res.data_ptr()),
                          C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, et.et_last_error()
    assert rel_l2(dev_to_f64(res), a @ w.T + r) < 4e-3


def _attention_ref(qkv, cu, n_heads, hd):
    D = n_heads * hd
    out = np.zeros((qkv.shape[0], D))
    for f in range(len(cu) - 1):
        a, b = cu[f], cu[f + 1]
        if b == a:
            continue
        q = qkv[a:b, :D].reshape(b - a, n_heads, hd).transpose(1, 0, 2)
        k = qkv[a:b, D:2 * D].reshape(b - a, n_heads, hd).transpose(1, 0, 2)
        v = qkv[a:b, 2 * D:].reshape(b - a, n_heads, hd).transpose(1, 0, 2)
        p = O.softmax_rows(q @ k.transpose(0, 2, 1) / math.sqrt(hd))
        out[a:b] = (p @ v).transpose(1, 0, 2).reshape(b - a, D)
    return out


@pytest.mark.parametrize("n_heads,hd", [(4, 16), (16, 72), (2, 64), (2, 128), (3, 32), (2, 80), (2, 96)])
def test_attention_matches_oracle(n_heads, hd):
    rng = np.random.default_rng(n_heads * hd)
    lens = [5, 64, 131, 729, 1, 128, 364, 182] if hd in (16, 72) else [5, 130, 64, 1]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows, D = int(cu[-1]), n_heads * hd
    # logits with a spread of several units so that the softmax is far from uniform
    bits, qkv = _bf(rng, (rows, 3 * D), scale=1.0)
    qkv_s = qkv.copy()
    qkv_s[:, :D] *= 2.0
    bits = f32_to_bf16_bits(qkv_s.astype(np.float32))
    qkv_s = bf16_bits_to_f32(bits).astype(np.float64)
    ref = _attention_ref(qkv_s, cu, n_heads, hd)
    out = et.et_attention(bits_to_dev(bits), torch.from_numpy(cu).cuda(), max(lens), n_heads, hd)
    got = dev_to_f64(out)
    assert rel_l2(got, ref) < 6e-3
    assert np.max(np.abs(got - ref)) < 0.05
    # a one-token frame attends to itself only: output = its own v, exactly
    one = int(cu[lens.index(1)])
    assert np.array_equal(got[one], qkv_s[one, 2 * D:])


@pytest.mark.parametrize("n_heads,hd,n_frames,length", [(16, 72, 3, 729), (16, 72, 5, 364), (16, 72, 2, 182),
                                                        (4, 16, 8, 64), (4, 16, 2, 32), (2, 64, 3, 130),
                                                        (2, 128, 2, 70), (3, 32, 2, 1), (2, 80, 2, 129),
                                                        (2, 96, 2, 65), (16, 72, 1, 218),
                                                        # several rounds of workgroups
                                                        (16, 72, 11, 729), (4, 16, 130, 70), (2, 80, 90, 300)])
def test_attention_uniform_matches_oracle(n_heads, hd, n_frames, length):
    rng = np.random.default_rng(n_heads * hd + length)
    D, rows = n_heads * hd, n_frames * length
    _, qkv = _bf(rng, (rows, 3 * D))
    qkv[:, :D] *= 2.0
    bits = f32_to_bf16_bits(qkv.astype(np.float32))
    qkv = bf16_bits_to_f32(bits).astype(np.float64)
    cu = (np.arange(n_frames + 1) * length).astype(np.int32)
    ref = _attention_ref(qkv, cu, n_heads, hd)
    out = et.et_attention_uniform(bits_to_dev(bits), n_frames, length, n_heads, hd)
    got = dev_to_f64(out)
    assert np.all(np.isfinite(got))
    assert rel_l2(got, ref) < 6e-3
    assert np.max(np.abs(got - ref)) < 0.05
    # the ragged entry point (row ranges from cu_tokens) agrees on the same input
    gen = et.et_attention(bits_to_dev(bits), torch.from_numpy(cu).cuda(), length, n_heads, hd)
    assert rel_l2(dev_to_f64(gen), got) < 6e-3


@pytest.mark.parametrize("order", ["rising", "falling", "negative_first", "spike_last"])
def test_attention_uniform_moving_maxima(order):
    """The exponentials refer to the maximum of the first 32 keys.  These inputs make the row maxima climb past it by some 2^47 over
    the frame (rising) or by 2^41 in the last, partly filled tile (spike_last), which the weights carry without another reference, never
    exceed it (falling), or start so far below the rest (negative_first) that the weights leave their range and the tiles are walked
    again with an online maximum."""
    n_heads, hd, length = 16, 72, 729
    n_frames = 11 if order in ("rising", "spike_last") else 2    # 11 frames: 128 queries per workgroup; two: groups of wavefronts
    rng = np.random.default_rng({"rising": 1, "falling": 2, "negative_first": 3, "spike_last": 4}[order])
    D, rows = n_heads * hd, n_frames * length
    _, qkv = _bf(rng, (rows, 3 * D))
    pos = np.tile(np.arange(length), n_frames).astype(np.float64)
    # logits = q . k / sqrt(72): a shared direction u with |u| = 1 gives q.k ~ a_q * a_k
    u = np.zeros(D)
    u.reshape(n_heads, hd)[:, 0] = 1.0
    ramp = {"rising": pos / 64.0 * 3.0, "falling": (length - pos) / 64.0 * 3.0,
            "negative_first": np.where(pos < 64, -40.0, 0.0), "spike_last": np.where(pos >= 720, 30.0, 0.0)}[order]
    qkv[:, :D] = qkv[:, :D] * 0.5 + 8.0 * u                      # q . u = 8 per head
    qkv[:, D:2 * D] = qkv[:, D:2 * D] * 0.5 + ramp[:, None] * u  # k . u = ramp -> logit shift 8 ramp / sqrt(72)
    bits = f32_to_bf16_bits(qkv.astype(np.float32))
    qkv = bf16_bits_to_f32(bits).astype(np.float64)
    cu = (np.arange(n_frames + 1) * length).astype(np.int32)
    ref = _attention_ref(qkv, cu, n_heads, hd)
    got = dev_to_f64(et.et_attention_uniform(bits_to_dev(bits), n_frames, length, n_heads, hd))
    assert np.all(np.isfinite(got))
    assert rel_l2(got, ref) < 1e-2
    assert np.max(np.abs(got - ref)) < 0.05


@pytest.mark.parametrize("cfg", [0, 1, 2])
def test_gemm_persistent_configs_walk_several_tiles_per_workgroup(cfg):
    """More output tiles than compute units, so each persistent workgroup finishes a tile, clears its
    accumulators and goes on; ragged last tile row and column; all three epilogues."""
    rng = np.random.default_rng(100 + cfg)
    M, N, K = 4500, 4304, 320                       # 18 x 17 = 306 tiles of 256 x 256
    a_bits, a = _bf(rng, (M, K))
    w_bits, w = _bf(rng, (N, K), scale=0.05)
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    r_bits, r = _bf(rng, (M, N))
    lin = a @ w.T + bias.astype(np.float64)
    a_d, w_d, b_d = bits_to_dev(a_bits), bits_to_dev(w_bits), torch.from_numpy(bias).cuda()
    for epi, ref in ((0, lin), (1, O.gelu_tanh(lin)), (2, lin + r)):
        c = et.et_gemm_bf16(a_d, w_d, b_d, epi, residual=bits_to_dev(r_bits) if epi == 2 else None,
                            tile_config=cfg)
        got = dev_to_f64(c)
        assert np.max(np.abs(got - ref) - 2 ** -8 * np.abs(ref)) < 5e-4, epi
        assert rel_l2(got, ref) < 4e-3, epi


@pytest.mark.parametrize("M,N,K", [(4500, 4304, 64), (4500, 4304, 128), (4353, 4168, 192), (511, 264, 576)])
def test_gemm_short_contractions_in_a_stream_of_tiles(M, N, K):
    """One, two and three k-tiles per output tile (the operand stream crosses an output tile at every one, two or
    three of them, the stores of a tile still in flight), an odd and an even count; the tilings in k order agree bit for
    bit.  Exact products, float32 sums of K terms (K * 2^-24 of their absolute sum, below 1e-5 here), one rounding to bf16."""
    rng = np.random.default_rng(M + K)
    a_bits, a = _bf(rng, (M, K))
    w_bits, w = _bf(rng, (N, K), scale=0.05)
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    r_bits, r = _bf(rng, (M, N))
    lin = (a.astype(np.float32) @ w.astype(np.float32).T + bias).astype(np.float64)
    a_d, w_d, b_d, r_d = bits_to_dev(a_bits), bits_to_dev(w_bits), torch.from_numpy(bias).cuda(), bits_to_dev(r_bits)
    for epi, ref in ((0, lin), (2, lin + r)):
        outs = [et.et_gemm_bf16(a_d, w_d, b_d, epi, residual=r_d if epi == 2 else None, tile_config=cfg) for cfg in (0, 1, 5)]
        got = dev_to_f64(outs[0])
        assert np.max(np.abs(got - ref) - 2 ** -8 * np.abs(ref)) < 5e-4, epi
        for other in outs[1:]:
            assert torch.equal(outs[0].view(torch.int16), other.view(torch.int16)), epi


def test_gemm_fc2_shape_with_residual_at_encoder_row_counts():
    """The fc2 step as the encoder runs it (K = 4304, bias + residual) on the kept-token and the all-token
    row counts: every element against exact products summed in float64."""
    rng = np.random.default_rng(4304)
    N, K = 1152, 4304
    w_bits, w = _bf(rng, (N, K), scale=0.02)
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    w_d, b_d = bits_to_dev(w_bits), torch.from_numpy(bias).cuda()
    for M in (2912, 23328):
        a_bits, a = _bf(rng, (M, K))
        r_bits, r = _bf(rng, (M, N))
        ref = a @ w.T + bias.astype(np.float64) + r
        c = et.et_gemm_bf16(bits_to_dev(a_bits), w_d, b_d, 2, residual=bits_to_dev(r_bits))
        got = dev_to_f64(c)
        assert np.max(np.abs(got - ref) - 2 ** -8 * np.abs(ref)) < 5e-4, M
        assert rel_l2(got, ref) < 4e-3, M


@pytest.mark.parametrize("N,epi", [(3456, 0), (4304, 1), (4304, 2), (1152, 2)])
def test_gemm_library_choice_at_encoder_row_count(N, epi):
    """32 x 729 rows with the library's own tiling, which splits a nearly empty last tile row or a partly
    filled last tile column off into launches of their own: every output element against the oracle."""
    rng = np.random.default_rng(N + epi)
    M, K = 23328, 128
    a_bits, a = _bf(rng, (M, K))
    w_bits, w = _bf(rng, (N, K), scale=0.1)
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    ref = a.astype(np.float32) @ w.astype(np.float32).T + bias            # exact products, float32 sums of 128 terms
    res = None
    if epi == 1:
        ref = O.gelu_tanh(ref.astype(np.float64))
    if epi == 2:
        r_bits, r = _bf(rng, (M, N))
        ref = ref + r.astype(np.float32)
        res = bits_to_dev(r_bits)
    c = et.et_gemm_bf16(bits_to_dev(a_bits), bits_to_dev(w_bits), torch.from_numpy(bias).cuda(), epi, residual=res)
    got = bf16_bits_to_f32(dev_to_bits(c))
    assert np.max(np.abs(got - ref) - 2 ** -8 * np.abs(ref)) < 5e-4
    assert rel_l2(got.astype(np.float64), ref.astype(np.float64)) < 4e-3


@pytest.mark.parametrize("rows,d_in,d_hidden,d_out", [(4949, 1152, 3584, 3584), (300, 64, 104, 72), (1, 128, 8, 8)])
def test_projector_matches_oracle(rows, d_in, d_hidden, d_out):
    """The two-layer projector (Sec. 3.1) on as many tokens as the paper's layout keeps of a 32-frame clip,
    at the widths of a 7B language model, and on small ragged widths; the hidden activation passes through
    bfloat16 once, hence 1e-2."""
    rng = np.random.default_rng(rows + d_out)
    x_bits, x = _bf(rng, (rows, d_in))
    w1_bits, w1 = _bf(rng, (d_hidden, d_in), scale=1.0 / math.sqrt(d_in))
    w2_bits, w2 = _bf(rng, (d_out, d_hidden), scale=1.0 / math.sqrt(d_hidden))
    b1 = (0.1 * rng.standard_normal(d_hidden)).astype(np.float32)
    b2 = (0.1 * rng.standard_normal(d_out)).astype(np.float32)
    proj = et.Projector(w1, b1, w2, b2)
    got = dev_to_f64(proj.project(bits_to_dev(x_bits)))
    proj.close()
    ref = O.project_tokens(x, w1, b1.astype(np.float64), w2, b2.astype(np.float64))
    assert got.shape == ref.shape
    assert rel_l2(got, ref) < 1e-2
    assert np.max(np.abs(got - ref)) < 0.05 * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("cfg", [2, 3, 4, 5])
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (63, 72, 128), (64, 64, 192), (65, 136, 320), (257, 200, 448), (130, 1152, 4352)])
def test_gemm_split_over_wavefronts(cfg, M, N, K):
    """The kernels for few rows: fewer k-tiles than wavefront groups, k-tiles that do not divide among them, ragged
    rows and columns; in fp64 against bf16 inputs (one rounding of an fp32 sum: 2^-8 relative + accumulation noise)."""
    rng = np.random.default_rng(M + N + K)
    a_bits, a = _bf(rng, (M, K))
    w_bits, w = _bf(rng, (N, K), scale=0.05)
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    r_bits, r = _bf(rng, (M, N))
    plain = a @ w.T + bias.astype(np.float64)
    a_d, w_d, b_d, r_d = bits_to_dev(a_bits), bits_to_dev(w_bits), torch.from_numpy(bias).cuda(), bits_to_dev(r_bits)
    for epi, ref in ((0, plain), (1, O.gelu_tanh(plain)), (2, plain + r)):
        got = dev_to_f64(et.et_gemm_bf16(a_d, w_d, b_d, epi, residual=r_d if epi == 2 else None, tile_config=cfg))
        assert np.max(np.abs(got - ref) - 2 ** -8 * np.abs(ref)) < 2e-4 * (np.sqrt(K) * 0.05 + 1.0)
        assert rel_l2(got, ref) < 4e-3


@pytest.mark.parametrize("M,N,K", [(1, 8, 128), (63, 72, 128), (129, 64, 256), (257, 200, 384), (300, 136, 1152)])
def test_gemm_two_groups_of_wavefronts_in_turn(M, N, K):
    """128 x 64 tiles with an even number of k-tiles (one, two, three and nine per group of wavefronts), ragged rows and
    columns; in fp64 against bf16 inputs, bounds as above."""
    test_gemm_split_over_wavefronts(3, M, N, K)


@pytest.mark.parametrize("n_heads,hd,lens", [
    (16, 72, [729]),                      # key tiles over four groups of wavefronts, uneven shares, ragged last tile
    (4, 64, [65, 0, 1, 128, 129]),        # the same: fewer tiles than groups, an empty and a one-token frame
    (2, 16, [300] * 3), (3, 32, [511, 64]), (1, 72, [70]),
    (16, 72, [729, 700]),                 # two groups
    (2, 80, [400, 321]), (2, 96, [330]), (1, 128, [577]),
    (16, 72, [729, 33, 515, 256, 1, 700, 257, 640, 90, 729, 600]),   # ragged, several rounds of workgroups
    (2, 80, [70] * 256), (2, 80, [70] * 257), (4, 80, [129, 33] * 32), (4, 80, [129, 33] * 33),   # heads of 80: two and three workgroups per compute unit
])
def test_attention_split_and_ragged_forms(n_heads, hd, lens):
    """Same bounds as the oracle test above: probabilities pass through bf16 once, the output is rounded once; partial
    results of the groups are combined in float32."""
    rng = np.random.default_rng(n_heads * hd + len(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows, D = int(cu[-1]), n_heads * hd
    _, qkv = _bf(rng, (rows, 3 * D))
    qkv[:, :D] *= 2.0
    bits = f32_to_bf16_bits(qkv.astype(np.float32))
    qkv = bf16_bits_to_f32(bits).astype(np.float64)
    ref = _attention_ref(qkv, cu, n_heads, hd)
    got = [et.et_attention(bits_to_dev(bits), torch.from_numpy(cu).cuda(), max(lens), n_heads, hd)]
    if len(set(lens)) == 1:
        got.append(et.et_attention_uniform(bits_to_dev(bits), len(lens), lens[0], n_heads, hd))
    for out in got:
        assert rel_l2(dev_to_f64(out), ref) < 6e-3
        assert np.max(np.abs(dev_to_f64(out) - ref)) < 0.05


@pytest.mark.parametrize("M,N,K,epi", [
    (729 * 7, 3456, 1152, 0), (729 * 14, 3456, 1152, 0), (729 * 16, 4352, 1152, 1), (729 * 24, 1152, 1152, 2),
    (729 * 24, 1152, 4352, 2), (729 * 27, 4352, 1152, 1), (729 * 32, 3456, 1152, 0), (729 * 32, 4352, 1152, 1),
    (729 * 64, 3456, 1152, 0),                                   # a strip of rows and one of columns
    (729 * 14, 3456, 1216, 0),                                   # an odd number of k-tiles
    (23040 + 1, 4352, 1152, 1), (23040 + 65, 4352, 1152, 1), (4608 + 63, 3456, 1152, 0),
    (729 * 5, 1152, 4352, 2), (729, 3456, 1152, 0),              # one launch, its k split over wavefronts
])
def test_equal_rows_have_equal_bits_wherever_they_lie(M, N, K, epi):
    """The library's choice may split the last tile rows off; every row is summed over k in one order all the same: a
    pattern of 81 rows, repeated through the matrix, gives the same bits in every repeat."""
    P = 81
    rng = np.random.default_rng(N + K + epi)
    a_bits, a = _bf(rng, (P, K))
    w_bits, w = _bf(rng, (N, K), scale=0.05)
    r_bits, r = _bf(rng, (P, N))
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    rows = torch.arange(M, device="cuda") % P
    c = et.et_gemm_bf16(bits_to_dev(a_bits)[rows], bits_to_dev(w_bits), torch.from_numpy(bias).cuda(), epi,
                        residual=bits_to_dev(r_bits)[rows] if epi == 2 else None)
    assert torch.equal(c.view(torch.int16), c[:P].view(torch.int16)[rows])
    ref = a @ w.T + bias.astype(np.float64)
    ref = O.gelu_tanh(ref) if epi == 1 else ref + r if epi == 2 else ref
    assert rel_l2(dev_to_f64(c[:P]), ref) < 4e-3


@pytest.mark.parametrize("n_heads,hd,lens,dead", [
    (16, 72, [729], (64, 128)), (4, 64, [300], (64, 128)), (2, 16, [300], (128, 192)),       # first tile of one of four groups
    (16, 72, [729], (64, 200)), (2, 32, [130], (0, 64)),                                     # ... and more of its tiles; of the first group
    (16, 72, [729, 700], (64, 128)), (2, 96, [330], (64, 128)), (2, 80, [400, 321], (0, 130)),       # two groups
    (16, 72, [729] * 5, (0, 64)), (16, 64, [130] * 30, (0, 100)), (2, 128, [70], (0, 32)),           # 128 queries per workgroup
    (16, 72, [150] * 96, (0, 96)), (16, 16, [70] * 96, (0, 32)), (16, 80, [129] * 96, (0, 64)),      # ... and many rounds of workgroups
])
@pytest.mark.parametrize("shift", [0.0, -16.0])
def test_attention_with_logits_of_minus_infinity(n_heads, hd, lens, dead, shift):
    """Keys whose logits are minus infinity for every query have probability 0, wherever they lie: the first 32 keys, the
    whole first key tile of a frame or of a group of wavefronts.  With `shift` all other logits are below -150, where a
    reference maximum that had stayed at 0 would leave no probability.  Bounds as in the oracle test."""
    rng = np.random.default_rng(n_heads * hd + len(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows, D = int(cu[-1]), n_heads * hd
    qkv = rng.standard_normal((rows, 3 * D))
    qkv[:, :D] = np.abs(qkv[:, :D]) + 0.5
    qkv[:, D:2 * D] += shift
    for f in range(len(lens)):
        qkv[cu[f] + dead[0]:min(cu[f] + dead[1], cu[f + 1]), D:2 * D] = -3.0e38
    bits = f32_to_bf16_bits(qkv.astype(np.float32))
    ref = _attention_ref(bf16_bits_to_f32(bits).astype(np.float64), cu, n_heads, hd)
    got = [et.et_attention(bits_to_dev(bits), torch.from_numpy(cu).cuda(), max(lens), n_heads, hd)]
    if len(set(lens)) == 1:
        got.append(et.et_attention_uniform(bits_to_dev(bits), len(lens), lens[0], n_heads, hd))
    for out in got:
        assert rel_l2(dev_to_f64(out), ref) < 6e-3
        assert np.max(np.abs(dev_to_f64(out) - ref)) < 0.05


@pytest.mark.parametrize("n_heads,hd,lens", [
    (16, 72, [729] * 32), (16, 16, [70] * 96), (12, 64, [129] * 130), (16, 32, [64] * 96), (16, 80, [1] * 96),
    (16, 72, [257, 0, 1, 255, 64, 33] * 9), (24, 80, [300] * 33), (16, 64, [256, 31] * 48),
])
def test_attention_over_several_rounds_of_workgroups(n_heads, hd, lens):
    """More workgroups of 128 queries than the compute units hold at a time (three each), in frames of one length and in ragged
    ones: wavefronts past a frame's queries, workgroups past its end, frames of a few tokens.  Bounds as in the oracle test."""
    assert -(-max(lens) // 128) * n_heads * len(lens) >= 1536
    rng = np.random.default_rng(n_heads * hd + len(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows, D = int(cu[-1]), n_heads * hd
    _, qkv = _bf(rng, (rows, 3 * D))
    qkv[:, :D] *= 2.0
    bits = f32_to_bf16_bits(qkv.astype(np.float32))
    ref = _attention_ref(bf16_bits_to_f32(bits).astype(np.float64), cu, n_heads, hd)
    got = [et.et_attention(bits_to_dev(bits), torch.from_numpy(cu).cuda(), max(lens), n_heads, hd)]
    if len(set(lens)) == 1:
        got.append(et.et_attention_uniform(bits_to_dev(bits), len(lens), lens[0], n_heads, hd))
    for out in got:
        assert rel_l2(dev_to_f64(out), ref) < 6e-3
        assert np.max(np.abs(dev_to_f64(out) - ref)) < 0.05


@pytest.mark.parametrize("n_heads,hd,lens", [
    (16, 72, [729] * 11), (16, 72, [729]), (16, 72, [729, 700]),        # 128 queries per workgroup; four and two groups
    (12, 64, [196] * 30), (4, 64, [65, 1, 129]), (2, 16, [300] * 3), (3, 32, [511, 64]), (2, 80, [400, 321]), (2, 96, [330]),
    (1, 128, [577]),
])
@pytest.mark.parametrize("jump,v_scale", [(100.0, 1.0), (28.0, 1.0e28), (-100.0, 1.0)])
def test_attention_where_the_first_reference_does_not_last(n_heads, hd, lens, jump, v_scale):
    """The reference maximum is the one of a frame's (or of a group of wavefronts') first 32 keys.  Later keys of every
    second query exceed it by e^100 (the weights' sum leaves its range), by e^28 with values of 1e28 (the sum stays, the
    weighted values leave float32), or lie e^100 below (nothing happens): the result is the oracle's in all of them.
    Bounds as in the oracle test, relative to the values' scale."""
    rng = np.random.default_rng(n_heads * hd + len(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows, D = int(cu[-1]), n_heads * hd
    qkv = rng.standard_normal((rows, 3 * D))
    late = np.concatenate([np.arange(n) >= n * 0.55 for n in lens])
    heads = qkv.reshape(rows, 3, n_heads, hd)
    heads[:, 0, :, 0] = np.where(np.arange(rows) % 2 == 0, 8.0, 0.0)[:, None]      # q . u
    heads[:, 1, :, 0] = np.where(late, jump * math.sqrt(hd) / 8.0, 0.0)[:, None]   # k . u: the logit is shifted by `jump`
    heads[:, 2] *= v_scale
    bits = f32_to_bf16_bits(qkv.astype(np.float32))
    ref = _attention_ref(bf16_bits_to_f32(bits).astype(np.float64), cu, n_heads, hd)
    got = [et.et_attention(bits_to_dev(bits), torch.from_numpy(cu).cuda(), max(lens), n_heads, hd)]
    if len(set(lens)) == 1:
        got.append(et.et_attention_uniform(bits_to_dev(bits), len(lens), lens[0], n_heads, hd))
    for out in got:
        assert rel_l2(dev_to_f64(out), ref) < 6e-3
        assert np.max(np.abs(dev_to_f64(out) - ref)) < 0.05 * v_scale


@pytest.mark.parametrize("n_heads,hd,lens,stride", [
    (16, 72, [729], 4), (16, 72, [729, 700], 2), (16, 72, [729] * 11, 1),          # four and two groups of wavefronts; 128 queries per workgroup
    (4, 64, [729], 4), (12, 64, [330] * 30, 1), (2, 16, [729] * 3, 4), (16, 16, [380] * 40, 1), (3, 32, [729], 4), (12, 32, [380] * 40, 1),
    (2, 80, [729], 2), (16, 80, [380] * 7, 1), (16, 80, [380] * 10, 1),            # the latter: the online maximum alone
    (2, 96, [729], 2), (16, 96, [380] * 6, 1), (1, 128, [729], 2), (16, 128, [380] * 6, 1),
])
def test_attention_rescales_what_still_counts(n_heads, hd, lens, stride):
    """The pass with an online maximum (a key far above the first reference forces it: the last key, for every 32nd query) moves its
    reference when a key tile exceeds it by 2^8, and rescales what it has summed up.  The other queries' logits climb by 7 (2^10)
    in every third tile of a group of wavefronts, there in one key only, so that the keys below it keep a share s of the weight of
    0.15 to 0.25; their values are 1, the high key's -1.  The scaled q is rounded to bf16, and here one component of it makes the
    whole step: 7 * 2^-9 in the logit, the same for all keys of a level, with another 2^-8 from the probabilities' own rounding.  That moves the result 1 - 2s by
    2 s (1 - s) * 0.018, 1.3 % of it at s = 0.25; with the oracle test's 6e-3 the bound is 2e-2.  An oracle whose keys below the last
    step are left out, or are not scaled down, is ten times further off."""
    rng = np.random.default_rng(n_heads * hd + len(lens))
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows, D = int(cu[-1]), n_heads * hd
    pos = np.concatenate([np.arange(n) for n in lens])
    last = np.concatenate([np.arange(n) == n - 1 for n in lens])
    tile = pos // 64 // stride                                     # tiles of a group in its own order
    step = (tile % 3 == 2) & (pos % 64 == 5)                       # the key that leads to the next level
    level = tile // 3 + step
    forced = pos % 32 == 7
    heads = (0.2 * rng.standard_normal((rows, 3, n_heads, hd)))
    heads[:, 0, :, 0] = np.where(forced, 8.0, 0.0)[:, None]
    heads[:, 1, :, 0] = np.where(last, 100.0 * math.sqrt(hd) / 8.0, 0.0)[:, None]
    heads[:, 0, :, 1] = np.where(forced, 0.0, 8.0)[:, None]
    heads[:, 1, :, 1] = np.where(last, 0.0, 7.0 * level * math.sqrt(hd) / 8.0)[:, None]
    heads[:, 2] += np.where(step, -1.0, 1.0)[:, None, None]
    bits = f32_to_bf16_bits(heads.reshape(rows, 3 * D).astype(np.float32))
    qkv = bf16_bits_to_f32(bits).astype(np.float64)
    ref = _attention_ref(qkv, cu, n_heads, hd)
    got = [et.et_attention(bits_to_dev(bits), torch.from_numpy(cu).cuda(), max(lens), n_heads, hd)]
    if len(set(lens)) == 1:
        got.append(et.et_attention_uniform(bits_to_dev(bits), len(lens), lens[0], n_heads, hd))
    for out in got:
        assert rel_l2(dev_to_f64(out), ref) < 2e-2
        assert np.max(np.abs(dev_to_f64(out) - ref)) < 0.05
    top = np.concatenate([np.full(n, level[cu[f]:cu[f + 1]].max()) for f, n in enumerate(lens)])
    below = level < top
    for wrong in (-60.0, 7.0 * math.sqrt(hd) / 8.0):               # the last rescaling by 0, and by 1
        planted = qkv.copy()
        planted.reshape(rows, 3, n_heads, hd)[below & ~last, 1, :, 1] += wrong
        mistaken = _attention_ref(planted, cu, n_heads, hd)
        assert rel_l2(mistaken[~forced], ref[~forced]) > 0.2
