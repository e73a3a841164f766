"""GPU parity: gr_beam_attn_fp8kv (shared-prefix beam attention over a prompt cache stored as FP8 E4M3 codes with one
scale per tensor; paper Section 5.1's separated cache with its shared half at one byte per element) against the
oracle's unified-cache attention on the widened values (code * scale as fp32).  Quantisation is part of the INPUT
here, so the bar is the one of the bf16 path: max-abs <= 2e-2 on bf16 outputs, LSE within 2e-3."""
import numpy as np
import pytest

import gr_synth
from gpu_util import bf16_to_dev, rand_attn_case, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gr():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2512_11529_amd as gr
    gr.load_library()
    return gr


def _quantise(bits):
    x = gr_synth.bf16_bits_to_f32(bits)
    scale = np.float32(max(float(np.abs(x).max()), 1e-6) / 448.0)
    codes = gr_synth.f32_to_e4m3_bits(x / scale)
    return codes, scale


def _check(gr, oracle_lib, a, sm_scale, triples=None):
    import torch
    B, W, Hq, d = a["q"].shape
    k8, ks = _quantise(a["k_shared"])
    v8, vs = _quantise(a["v_shared"])
    cu = a["cu_seqlens"]
    lse = torch.empty((B, W, Hq), dtype=torch.float32, device="cuda:0")
    out, _ = gr.gr_beam_attn_fp8kv(bf16_to_dev(a["q"]), to_dev(k8), to_dev(v8), float(ks), float(vs), to_dev(cu),
                                   bf16_to_dev(a["k_unshared"]), bf16_to_dev(a["v_unshared"]), a["u"], sm_scale,
                                   int(np.diff(cu).max()) if len(cu) > 1 else 0, int(cu[-1]), lse_out=lse)
    torch.cuda.synchronize()
    out, lse = out.float().cpu().numpy(), lse.cpu().numpy()
    kf = (gr_synth.e4m3_bits_to_f32(k8) * ks).astype(np.float32)
    vf = (gr_synth.e4m3_bits_to_f32(v8) * vs).astype(np.float32)
    ref, ref_lse = oracle_lib.attn_unified_f32kv(a["q"], kf, vf, cu, a["k_unshared"], a["v_unshared"], a["u"], sm_scale, triples)
    if triples is None:
        got, got_lse = out.reshape(-1, d), lse.reshape(-1)
    else:
        got, got_lse = out[triples[:, 0], triples[:, 1], triples[:, 2]], lse[triples[:, 0], triples[:, 1], triples[:, 2]]
    err = np.abs(got - ref).max()
    assert err <= 2e-2, f"max-abs {err}"
    fin = np.isfinite(ref_lse)
    np.testing.assert_allclose(got_lse[fin], ref_lse[fin], rtol=0, atol=2e-3)


@pytest.mark.parametrize("B,W,Hq,Hkv,d,u,lens", [
    (2, 5, 8, 2, 128, 2, (7, 150)),
    (3, 24, 4, 4, 64, 1, (64, 1, 130)),
    (1, 70, 8, 2, 128, 3, (333,)),
    (2, 16, 16, 4, 128, 3, (0, 200)),           # a request with no prompt: only its own tokens
    (1, 40, 4, 4, 64, 0, (257,)),               # no own tokens: the prompt loop alone (scales still applied)
    (2, 96, 32, 8, 128, 3, (100, 1500)),        # enough rows for the L split
])
def test_fp8kv_matches_oracle(gr, oracle_lib, B, W, Hq, Hkv, d, u, lens):
    a = rand_attn_case(300 + B + W + d, B, W, Hq, Hkv, d, 3, u, lens)
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,segments", [(128, 1), (256, 1), (128, 3), (256, 2)])
def test_fp8kv_every_launch_plan(gr, oracle_lib, d, rows, segments):
    B, W, Hq, Hkv = 2, 160, 8, 2
    a = rand_attn_case(400 + d + rows + segments, B, W, Hq, Hkv, d, 3, 2, (333, 1100))
    rng = np.random.default_rng(6)
    n = 200
    tri = np.stack([rng.integers(0, B, n), rng.integers(0, W, n), rng.integers(0, Hq, n)], axis=1).astype(np.int32)
    tri[:4] = [[0, 0, 0], [1, W - 1, Hq - 1], [0, 63, 7], [1, 64, 0]]
    gr.gr_diag_attn_plan(rows, segments)
    try:
        _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))), tri)
    finally:
        gr.gr_diag_attn_plan(0, 0)


@pytest.mark.parametrize("d,B", [(64, 11), (64, 36), (128, 11), (128, 36)])
def test_fp8kv_one_and_two_sets_of_wavefronts(gr, oracle_lib, d, B):
    """88 row blocks (two sets of wavefronts share each one's prompt: no, one, odd and even numbers of tiles) and 288 (one set)."""
    lens = ((0, 1, 64, 65, 128, 129, 192, 200, 256, 320, 321) * 4)[:B]
    a = rand_attn_case(500 + d + B, B, 20, 8, 8, d, 3, 2, lens)
    rng = np.random.default_rng(9)
    tri = np.stack([np.arange(400) % B, rng.integers(0, 20, 400), rng.integers(0, 8, 400)], axis=1).astype(np.int32)
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))), tri)


def test_fp8kv_every_code_is_widened_exactly(gr, oracle_lib):
    """All 254 finite codes appear in K and V (one dominant key per query picks single V rows, so a wrong code -> value
    map or a wrong byte order inside the 8-byte pieces shows up at full magnitude)."""
    import torch
    B, W, Hq, Hkv, d, L = 1, 8, 2, 1, 64, 128
    a = rand_attn_case(9, B, W, Hq, Hkv, d, 3, 0, (L,))
    codes = np.array([c for c in range(256) if (c & 0x7F) != 0x7F], dtype=np.uint8)
    rng = np.random.default_rng(2)
    k8 = rng.choice(codes, size=(L, Hkv, d)).astype(np.uint8)
    v8 = np.resize(codes, (L, Hkv, d)).astype(np.uint8)
    ks, vs = np.float32(2.0 ** -9), np.float32(2.0 ** -6)
    cu = a["cu_seqlens"]
    out, _ = gr.gr_beam_attn_fp8kv(bf16_to_dev(a["q"]), to_dev(k8), to_dev(v8), float(ks), float(vs), to_dev(cu),
                                   bf16_to_dev(a["k_unshared"]), bf16_to_dev(a["v_unshared"]), 0, 1.0, L, L)
    torch.cuda.synchronize()
    kf = (gr_synth.e4m3_bits_to_f32(k8) * ks).astype(np.float32)
    vf = (gr_synth.e4m3_bits_to_f32(v8) * vs).astype(np.float32)
    ref, _ = oracle_lib.attn_unified_f32kv(a["q"], kf, vf, cu, a["k_unshared"], a["v_unshared"], 0, 1.0)
    err = np.abs(out.float().cpu().numpy().reshape(-1, d) - ref).max()
    assert err <= 2e-2, f"max-abs {err}"


def test_fp8kv_rejects_bad_scales(gr):
    a = rand_attn_case(1, 1, 2, 2, 2, 64, 3, 1, (5,))
    k8, _ = _quantise(a["k_shared"])
    for ks, vs in ((0.0, 1.0), (1.0, -1.0), (float("nan"), 1.0), (1.0, float("inf"))):
        with pytest.raises(gr.GrError) as e:
            gr.gr_beam_attn_fp8kv(bf16_to_dev(a["q"]), to_dev(k8), to_dev(k8), ks, vs, to_dev(a["cu_seqlens"]),
                                  bf16_to_dev(a["k_unshared"]), bf16_to_dev(a["v_unshared"]), 1, 1.0, 5, 5)
        assert e.value.status == -1


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,factor", [(128, 3.0), (128, 7.0), (256, 7.0), (128, 12.0), (256, 12.0)])
def test_fp8kv_scores_that_jump_inside_the_prompt(gr, oracle_lib, d, rows, factor):
    """Keys far above everything before them: the reference is raised after the tile, or the wavefront computes its columns again."""
    lens, W, Hq, Hkv = (330, 460), 40, 8, 2
    a = rand_attn_case(950 + d + rows, len(lens), W, Hq, Hkv, d, 3, 2, lens)
    q, k = gr_synth.bf16_bits_to_f32(a["q"]), gr_synth.bf16_bits_to_f32(a["k_shared"]).copy()
    for b, (w, head, tok) in enumerate([(3, 1, 70), (0, 4, 300)]):
        k[a["cu_seqlens"][b] + tok, head // (Hq // Hkv)] = factor * q[b, w, head]
    a["k_shared"] = gr_synth.f32_to_bf16_bits(k)
    gr.gr_diag_attn_plan(rows, 1)
    try:
        _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))))
    finally:
        gr.gr_diag_attn_plan(0, 0)


@pytest.mark.parametrize("W", [64, 80])
def test_fp8kv_many_workgroups_of_either_size(gr, oracle_lib, W):
    """256 workgroups of 256 query rows or more: 256 rows, and 128 rows where they leave fewer unused."""
    B = 33
    a = rand_attn_case(970 + W, B, W, 32, 8, 128, 3, 2, tuple(1 + 9 * (b % 16) for b in range(B)))
    rng = np.random.default_rng(9)
    n = 300
    tri = np.stack([np.arange(n) % B, rng.integers(0, W, n), rng.integers(0, 32, n)], axis=1).astype(np.int32)
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(128))), tri)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("uniform", [True, False])
@pytest.mark.parametrize("factor", [3.0, 12.0])
def test_fp8kv_scores_that_jump_in_many_workgroups(gr, oracle_lib, d, uniform, factor):
    """More than 256 workgroups of 128 rows: one set of four wavefronts, its requests of one length or found by rank."""
    B, W, H = 40, 20, 8
    lens = tuple(260 if uniform else 130 + 9 * (b % 16) for b in range(B))
    a = rand_attn_case(1300 + d, B, W, H, H, d, 3, 2, lens)
    q, k = gr_synth.bf16_bits_to_f32(a["q"]), gr_synth.bf16_bits_to_f32(a["k_shared"]).copy()
    tri = []
    for b in range(B):
        w, head, tok = b % W, b % H, (70 + 3 * b) % lens[b]
        k[a["cu_seqlens"][b] + tok, head] = factor * q[b, w, head]
        tri += [(b, w, head), (b, (w + 1) % W, head), (b, w, (head + 1) % H)]
    a["k_shared"] = gr_synth.f32_to_bf16_bits(k)
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))), np.array(tri, dtype=np.int32))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("factor", [4.0, 12.0])
def test_fp8kv_a_token_that_is_nearly_all_of_the_sum(gr, d, rows, factor):
    """The output is that token's V row: codes of values between 1 and 2, times a scale that is a power of two."""
    lens, W, H = (330, 460), 20, 4
    a = rand_attn_case(1400 + d + rows, len(lens), W, H, H, d, 3, 2, lens)
    rng = np.random.default_rng(12)
    v = (rng.choice([-1.0, 1.0], a["v_shared"].shape) * (1.0 + rng.integers(0, 8, a["v_shared"].shape) / 8.0)).astype(np.float32)
    q, k = gr_synth.bf16_bits_to_f32(a["q"]), gr_synth.bf16_bits_to_f32(a["k_shared"]).copy()
    rows_of = []
    for b in range(len(lens)):
        for i, tok in enumerate([5, 70, 129, 200, 250, lens[b] - 1]):
            for head in range(H):
                k[a["cu_seqlens"][b] + tok, head] = factor * q[b, 3 * i + b, head]
                rows_of.append((b, 3 * i + b, head, a["cu_seqlens"][b] + tok))
    codes, scale = _quantise(gr_synth.f32_to_bf16_bits(k))
    gr.gr_diag_attn_plan(rows, 1)
    try:
        out, _ = gr.gr_beam_attn_fp8kv(bf16_to_dev(a["q"]), to_dev(codes), to_dev(gr_synth.f32_to_e4m3_bits(v)), float(scale), 0.25, to_dev(a["cu_seqlens"]),
                                       bf16_to_dev(a["k_unshared"]), bf16_to_dev(a["v_unshared"]), 2, float(np.float32(1 / np.sqrt(d))), 460, 790)
        out = out.float().cpu().numpy()
    finally:
        gr.gr_diag_attn_plan(0, 0)
    for b, w, head, at in rows_of:
        np.testing.assert_array_equal(out[b, w, head], 0.25 * v[at, head], err_msg=f"request {b}, beam {w}, head {head}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows", [128, 256])
@pytest.mark.parametrize("width", [4.0, 32.0])
def test_fp8kv_scores_that_are_wide_from_the_first_tile_on(gr, oracle_lib, d, rows, width):
    """Some wavefronts, or all, search from the first tile on."""
    lens, W, Hq, Hkv = (330, 65), 40, 8, 2
    a = rand_attn_case(1600 + d + rows, len(lens), W, Hq, Hkv, d, 3, 2, lens)
    a["q"] = gr_synth.f32_to_bf16_bits(width * gr_synth.bf16_bits_to_f32(a["q"]))
    gr.gr_diag_attn_plan(rows, 1)
    try:
        _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))))
    finally:
        gr.gr_diag_attn_plan(0, 0)
