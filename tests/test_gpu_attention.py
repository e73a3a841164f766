"""GPU parity: gr_beam_attn against the CPU oracle's unified-cache attention (Sections 5.1-5.2).

Bar: max-abs error <= 2e-2 on bf16 outputs (bf16 in, fp32 accumulate), plus a tighter bound derived
from the arithmetic: the output is a convex combination of bf16 values whose weights carry a bf16
rounding (2^-9 relative) and the result is rounded to bf16 once more, so |err| <= 2^-7 * max|V| with
a wide margin.
"""
import numpy as np
import pytest

import gr_synth
from gpu_util import rand_attn_case, run_attn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gr():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2512_11529_amd as gr
    gr.load_library()
    return gr


def _check(gr, oracle_lib, a, scale, triples=None):
    out, lse = run_attn(gr, a, scale)
    B, W, Hq, d = a["q"].shape
    ref, ref_lse = oracle_lib.attn_unified(a["q"], a["k_shared"], a["v_shared"], a["cu_seqlens"], a["k_unshared"],
                                           a["v_unshared"], a["u"], scale, triples)
    if triples is None:
        got, got_lse = out.reshape(-1, d), lse.reshape(-1)
    else:
        got = out[triples[:, 0], triples[:, 1], triples[:, 2]]
        got_lse = lse[triples[:, 0], triples[:, 1], triples[:, 2]]
    err = np.abs(got - ref).max()
    vmax = float(np.abs(gr_synth.bf16_bits_to_f32(a["v_shared"])).max()) if a["v_shared"].size else 1.0
    vmax = max(vmax, float(np.abs(gr_synth.bf16_bits_to_f32(a["v_unshared"])).max()))
    assert err <= 2e-2, f"max-abs {err}"
    assert err <= 2.0 ** -7 * vmax, f"max-abs {err} vs derived bound {2.0 ** -7 * vmax}"
    fin = np.isfinite(ref_lse)
    np.testing.assert_allclose(got_lse[fin], ref_lse[fin], rtol=0, atol=2e-3)
    return err


def test_tiny_config_all_steps(gr, oracle_lib):
    cfg = gr_synth.get_config(1)
    for step in range(cfg.ND):
        a = gr_synth.make_attention_inputs(cfg, step)
        _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(cfg.d))))


@pytest.mark.parametrize("B,W,Hq,Hkv,d,u,lens", [
    (2, 5, 8, 2, 128, 2, (70, 333)),          # ragged tails, GQA g=4, W*g = 20 rows (partial row block)
    (3, 24, 4, 4, 64, 1, (1, 64, 129)),       # g=1, d=64, one-token prompt, exact tile, tile+1
    (1, 70, 8, 2, 128, 3, (517,)),            # 280 rows: two row blocks
    (2, 16, 16, 4, 128, 3, (0, 200)),         # an empty prompt: only the beam's own tokens
    (1, 3, 2, 1, 64, 2, (1000,)),             # g=2
    (2, 96, 32, 8, 128, 3, (2048, 1500)),     # the benchmark head geometry; long enough to split L
    (1, 40, 4, 4, 64, 3, (100,)),             # g=1: 32 beams x 3 own tokens per wave = three unshared mini-tiles
    (2, 20, 4, 2, 128, 3, (64, 10)),          # g=2: 16 beams x 3 = 48 own-token rows, two mini-tiles
    (1, 30, 6, 2, 64, 2, (130,)),             # g=3: beams straddle wave boundaries (32 is not a multiple of g)
    (1, 300, 8, 2, 128, 3, (0,)),             # no prompt at all, several row blocks: own tokens only
    (1, 200, 4, 2, 64, 2, (300,)),            # d=64 with more than 128 rows per KV head: the 8-wave d=64 kernel
    (1, 8, 8, 2, 128, 1, (1500,)),            # 32 rows per KV head, long prompt: 4-wave kernel with L split in five
])
def test_random_shapes(gr, oracle_lib, B, W, Hq, Hkv, d, u, lens):
    a = rand_attn_case(B * 100 + W, B, W, Hq, Hkv, d, 3, u, lens)
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))))


def test_structured_inputs_give_order_one_outputs(gr, oracle_lib):
    # one dominant key per query makes the output a single V row (magnitude ~1), so layout or
    # indexing mistakes cannot hide under small averaged values
    B, W, Hq, Hkv, d = 2, 9, 8, 2, 128
    a = rand_attn_case(5, B, W, Hq, Hkv, d, 3, 3, (150, 97))
    rng = np.random.default_rng(0)
    q = gr_synth.bf16_bits_to_f32(a["q"])
    for b in range(B):
        lo, hi = a["cu_seqlens"][b], a["cu_seqlens"][b + 1]
        for hk in range(Hkv):
            j = int(rng.integers(lo, hi))
            a["k_shared"][j, hk] = gr_synth.f32_to_bf16_bits(8.0 * q[b, int(rng.integers(W)), hk * (Hq // Hkv)])
    for b in range(B):
        for w in range(0, W, 2):
            a["k_unshared"][b, w, 1, 0] = gr_synth.f32_to_bf16_bits(8.0 * q[b, w, 1])
    _check(gr, oracle_lib, a, 1.0)


def test_scores_rising_along_the_prompt_raise_the_reference_on_every_tile(gr, oracle_lib):
    # keys proportional to one query with a factor that grows with the position: that query's scores climb by ~15 bits per
    # 64-token tile (the lazily raised reference maximum and the O / row-sum rescale run on every tile), the last key
    # dominates, and for the opposite sign the first tile holds the maximum and everything later underflows
    B, W, Hq, Hkv, d, L = 1, 4, 4, 1, 64, 1000
    for sign in (1.0, -1.0):
        a = rand_attn_case(17, B, W, Hq, Hkv, d, 3, 2, (L,))
        q0 = gr_synth.bf16_bits_to_f32(a["q"])[0, 0, 0]
        ramp = (np.arange(L, dtype=np.float32) / 50.0)[:, None]
        a["k_shared"][:, 0] = gr_synth.f32_to_bf16_bits(sign * ramp * q0[None, :])
        _check(gr, oracle_lib, a, 0.125)


def test_wide_beam_sampled_rows(gr, oracle_lib):
    # W = 2048 beams (8192 query rows per KV head, 32 row blocks): sampled outputs against the oracle
    B, W, Hq, Hkv, d = 1, 2048, 8, 2, 64
    a = rand_attn_case(31, B, W, Hq, Hkv, d, 3, 3, (200,))
    rng = np.random.default_rng(3)
    tri = np.stack([np.zeros(300, np.int64), rng.integers(0, W, 300), rng.integers(0, Hq, 300)], axis=1).astype(np.int32)
    tri[:4] = [[0, 0, 0], [0, W - 1, Hq - 1], [0, 255, 3], [0, 256, 4]]
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))), tri)


def test_separated_cache_is_w_independent_of_other_beams(gr, oracle_lib):
    # changing one beam's own tokens must not change any other beam's output
    a = rand_attn_case(9, 1, 6, 4, 2, 64, 3, 2, (90,))
    out0, _ = run_attn(gr, a, 0.125)
    a2 = dict(a); a2["k_unshared"] = a["k_unshared"].copy(); a2["k_unshared"][0, 2] ^= 0x8000
    out1, _ = run_attn(gr, a2, 0.125)
    keep = [w for w in range(6) if w != 2]
    np.testing.assert_array_equal(out0[0, keep], out1[0, keep])
    assert not np.array_equal(out0[0, 2], out1[0, 2])


def test_argument_errors(gr):
    import torch
    from gpu_util import bf16_to_dev, to_dev
    a = rand_attn_case(1, 1, 2, 2, 2, 32, 3, 1, (5,))     # d = 32 unsupported
    with pytest.raises(gr.GrError) as e:
        run_attn(gr, a, 1.0)
    assert e.value.status == -2
    a = rand_attn_case(1, 1, 2, 2, 2, 64, 3, 1, (5,))
    a["u"] = 4
    with pytest.raises(gr.GrError) as e:
        run_attn(gr, a, 1.0)
    assert e.value.status == -1
    # a tensor that does not start on a 16-byte boundary is refused (the kernels move 16-byte pieces)
    a = rand_attn_case(2, 1, 2, 2, 2, 64, 3, 1, (5,))
    q = bf16_to_dev(a["q"])
    shifted = torch.empty(q.numel() + 8, dtype=torch.bfloat16, device=q.device)[1:1 + q.numel()].view(q.shape)
    shifted.copy_(q)
    assert shifted.data_ptr() % 16 == 2
    with pytest.raises(gr.GrError) as e:
        gr.gr_beam_attn(shifted, bf16_to_dev(a["k_shared"]), bf16_to_dev(a["v_shared"]), to_dev(a["cu_seqlens"]),
                        bf16_to_dev(a["k_unshared"]), bf16_to_dev(a["v_unshared"]), 1, 1.0, 5, 5)
    assert e.value.status == -1


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,segments", [(128, 1), (256, 1), (128, 3), (256, 2), (256, 16)])
def test_every_launch_plan_matches_oracle(gr, oracle_lib, d, rows, segments):
    """Both workgroup sizes and the L-split path of both head sizes, forced through the plan override (the built-in rule
    picks only one of them per shape): ragged batch, 640 query rows per KV head, a prompt that ends inside a tile."""
    B, W, Hq, Hkv = 2, 160, 8, 2
    a = rand_attn_case(50 + d + rows + segments, B, W, Hq, Hkv, d, 3, 2, (333, 1100))
    rng = np.random.default_rng(4)
    n = 240
    tri = np.stack([rng.integers(0, B, n), rng.integers(0, W, n), rng.integers(0, Hq, n)], axis=1).astype(np.int32)
    tri[:6] = [[0, 0, 0], [1, W - 1, Hq - 1], [0, 31, 3], [1, 32, 4], [0, 63, 7], [1, 64, 0]]
    gr.gr_diag_attn_plan(rows, segments)
    try:
        _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))), tri)
    finally:
        gr.gr_diag_attn_plan(0, 0)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("g,u", [(1, 3), (3, 2), (4, 0), (8, 1)])
def test_two_sets_of_wavefronts_split_the_prompt(gr, oracle_lib, d, g, u):
    """Few enough row blocks that two sets of wavefronts share each: prompts of no tile, one, an odd and an even number of tiles, each
    with a whole and a partial last one (the second set has no tile, one less than the first, or as many); g = 1 needs three passes of the
    own-token stage."""
    lens = (0, 1, 64, 65, 128, 129, 192, 200, 256, 320, 321)
    a = rand_attn_case(700 + d + g + u, len(lens), 33, g, 1, d, 3, u, lens)
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))))


@pytest.mark.parametrize("d,B", [(64, 32), (64, 33), (128, 32), (128, 33)])
def test_one_and_two_sets_of_wavefronts(gr, oracle_lib, d, B):
    """256 row blocks (one per CU, two sets each) and 264 (one set each)."""
    lens = tuple(70 + 9 * (b % 5) for b in range(B))
    a = rand_attn_case(800 + d + B, B, 20, 16, 8, d, 3, 2, lens)
    rng = np.random.default_rng(8)
    tri = np.stack([np.arange(300) % B, rng.integers(0, 20, 300), rng.integers(0, 16, 300)], axis=1).astype(np.int32)
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))), tri)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,segments", [(128, 1), (256, 1), (256, 2)])
@pytest.mark.parametrize("factor", [3.0, 7.0, 12.0])
def test_scores_that_jump_inside_the_prompt(gr, oracle_lib, d, rows, segments, factor):
    """Keys that one beam's queries meet 34 to 50 bits (factor 3), 80 (7, head size 64: its reference is raised after the tile), 114 (7, head size
    128) or 138 bits and more (12: the wavefront computes its columns again) above everything before them, in an early, a middle and the last tile of a prompt whose
    tiles are even or odd in number, for workgroups of one and of two sets of wavefronts."""
    lens, W, Hq, Hkv = (330, 400, 460), 40, 8, 2
    a = rand_attn_case(900 + d + rows, len(lens), W, Hq, Hkv, d, 3, 2, lens)
    q, k = gr_synth.bf16_bits_to_f32(a["q"]), gr_synth.bf16_bits_to_f32(a["k_shared"]).copy()
    for b, (w, head, tok) in enumerate([(3, 1, 70), (39, 6, 200), (0, 4, 459)]):
        k[a["cu_seqlens"][b] + tok, head // (Hq // Hkv)] = factor * q[b, w, head]
    a["k_shared"] = gr_synth.f32_to_bf16_bits(k)
    gr.gr_diag_attn_plan(rows, segments)
    try:
        _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))))
    finally:
        gr.gr_diag_attn_plan(0, 0)


@pytest.mark.parametrize("B,W,uniform", [(32, 80, False), (32, 64, False), (33, 64, False), (33, 64, True)])
def test_many_workgroups_of_either_size(gr, oracle_lib, B, W, uniform):
    """256 workgroups of 256 query rows or more: 128 rows where they leave fewer rows unused (80 beams x 4 heads), 256 rows in one round, 128
    rows for short prompts in more than one, with requests of one length and ordered by length."""
    lens = tuple(70 if uniform else 1 + 9 * (b % 16) for b in range(B))
    a = rand_attn_case(960 + B + W, B, W, 32, 8, 128, 3, 3, lens)
    rng = np.random.default_rng(9)
    n = 400
    tri = np.stack([np.arange(n) % B, rng.integers(0, W, n), rng.integers(0, 32, n)], axis=1).astype(np.int32)
    tri[:4, 1] = [0, W - 1, 31, min(W - 1, 32)]
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(128))), tri)


@pytest.mark.parametrize("B", [63, 64, 65, 127, 128, 129])
@pytest.mark.parametrize("lens", ["ragged", "two lengths", "one long"])
def test_requests_by_decreasing_length(gr, oracle_lib, B, lens):
    """More workgroups than CUs: every workgroup finds its request by rank (up to 128 requests; a kernel orders more); equal lengths,
    requests without a prompt, lengths around powers of two."""
    rng = np.random.default_rng(B)
    n = {"ragged": rng.integers(0, 150, B), "two lengths": np.where(rng.random(B) < 0.5, 63, 64), "one long": np.where(np.arange(B) == B - 1, 513, 1)}[lens]
    n[:2] = [128, 0]
    a = rand_attn_case(980 + B, B, 40, 8, 8, 64, 3, 1, tuple(int(x) for x in n))
    m = 3 * B
    tri = np.stack([np.arange(m) % B, rng.integers(0, 40, m), rng.integers(0, 8, m)], axis=1).astype(np.int32)
    _check(gr, oracle_lib, a, 0.125, tri)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,segments", [(128, 1), (256, 1), (128, 2)])
@pytest.mark.parametrize("power", [-118, 110])
def test_values_near_the_ends_of_the_range(gr, oracle_lib, d, rows, segments, power):
    """V times a power of two gives the output times that power, down to where products of V and probabilities meet fp32's smallest numbers
    and up to where the un-normalised sums do not overflow unless a reference is far below the maximum; also for queries whose scores
    jump by 34 to 50 bits inside the prompt or at an own token.  The bound is _check's: two roundings to bf16, 2^-7 max|V|."""
    lens, W, Hq, Hkv = (330, 400, 60), 40, 8, 2
    a = rand_attn_case(1000 + d + rows, len(lens), W, Hq, Hkv, d, 3, 2, lens)
    q, k, ko = (gr_synth.bf16_bits_to_f32(a[n]).copy() for n in ("q", "k_shared", "k_unshared"))
    for b, (w, head, tok) in enumerate([(3, 1, 70), (39, 6, 399)]):
        k[a["cu_seqlens"][b] + tok, head // (Hq // Hkv)] = 3.0 * q[b, w, head]
    for b, (w, head, tok) in enumerate([(4, 1, 0), (11, 6, 1), (20, 3, 1)]):
        ko[b, w, tok, head // (Hq // Hkv)] = 3.0 * q[b, w, head]
    a["k_shared"], a["k_unshared"] = gr_synth.f32_to_bf16_bits(k), gr_synth.f32_to_bf16_bits(ko)
    scale = float(np.float32(1 / np.sqrt(d)))
    gr.gr_diag_attn_plan(rows, segments)
    try:
        _check(gr, oracle_lib, a, scale)
        want, want_lse = run_attn(gr, a, scale)
        scaled = dict(a)
        for n in ("v_shared", "v_unshared"):
            scaled[n] = gr_synth.f32_to_bf16_bits(np.ldexp(gr_synth.bf16_bits_to_f32(a[n]), power))
        out, lse = run_attn(gr, scaled, scale)
    finally:
        gr.gr_diag_attn_plan(0, 0)
    vmax = max(float(np.abs(gr_synth.bf16_bits_to_f32(a[n])).max()) for n in ("v_shared", "v_unshared"))
    assert np.isfinite(out).all()
    assert np.abs(np.ldexp(out, -power) - want).max() <= 2.0 ** -7 * vmax
    np.testing.assert_allclose(lse, want_lse, rtol=0, atol=2e-3)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,segments", [(128, 1), (256, 1), (128, 2)])
@pytest.mark.parametrize("factor", [3.0, 7.0, 12.0])
def test_a_token_that_is_nearly_all_of_the_sum(gr, d, rows, segments, factor):
    """A key 34 bits or more above all others of its column, in the first tile, a later one, the last one or among the own tokens: the others
    add less than 2^-20 to values between 1 and 2, so the output is that token's V row, every bit of it.  (A probability that O takes
    rounded and the sum does not gives values a bit off.)"""
    lens, W, Hq, Hkv = (330, 400, 460), 40, 8, 2
    a = rand_attn_case(1100 + d + rows, len(lens), W, Hq, Hkv, d, 3, 2, lens)
    rng = np.random.default_rng(11)
    values = lambda shape: gr_synth.f32_to_bf16_bits((rng.choice([-1.0, 1.0], shape) * rng.uniform(1.0, 2.0, shape)).astype(np.float32))
    a["v_shared"], a["v_unshared"] = values(a["v_shared"].shape), values(a["v_unshared"].shape)
    q, k, ko = (gr_synth.bf16_bits_to_f32(a[n]).copy() for n in ("q", "k_shared", "k_unshared"))
    rows_of = []
    for b in range(len(lens)):
        toks = [5, 70, 129, 200, 250, lens[b] - 1, -1, -2]                   # -1 - t: own token t
        for i, tok in enumerate(toks):
            for kvh in range(Hkv):
                w, head = 5 * i + b, kvh * (Hq // Hkv) + i % (Hq // Hkv)
                if tok >= 0:
                    at = (a["cu_seqlens"][b] + tok, kvh)
                    k[at] = factor * q[b, w, head]
                else:
                    at = (b, w, -1 - tok, kvh)
                    ko[at] = factor * q[b, w, head]
                rows_of.append((b, w, head, tok, at))
    a["k_shared"], a["k_unshared"] = gr_synth.f32_to_bf16_bits(k), gr_synth.f32_to_bf16_bits(ko)
    gr.gr_diag_attn_plan(rows, segments)
    try:
        out, _ = run_attn(gr, a, float(np.float32(1 / np.sqrt(d))))
    finally:
        gr.gr_diag_attn_plan(0, 0)
    for b, w, head, tok, at in rows_of:
        want = gr_synth.bf16_bits_to_f32(a["v_shared" if tok >= 0 else "v_unshared"])[at]
        np.testing.assert_array_equal(out[b, w, head], want, err_msg=f"request {b}, beam {w}, head {head}, token {tok}")


@pytest.mark.parametrize("d,W", [(64, 16), (64, 40), (128, 40)])
@pytest.mark.parametrize("uniform", [True, False])
@pytest.mark.parametrize("factor", [3.0, 7.0, 12.0])
def test_scores_that_jump_in_many_workgroups(gr, oracle_lib, d, W, uniform, factor):
    """More than 256 workgroups of 128 rows: one set of four wavefronts, its requests of one length or found by rank.  Scores that jump by 34 to
    50, 80 to 114 (the reference is raised after the tile, or the wavefront computes its columns again) or 138 bits and more (again)."""
    B, H = 40, 8
    lens = tuple(260 if uniform else 130 + 9 * (b % 16) for b in range(B))
    a = rand_attn_case(1200 + d + W, B, W, H, H, d, 3, 2, lens)
    q, k = gr_synth.bf16_bits_to_f32(a["q"]), gr_synth.bf16_bits_to_f32(a["k_shared"]).copy()
    tri = []
    for b in range(B):
        w, head, tok = b % W, b % H, (70 + 3 * b) % lens[b]
        k[a["cu_seqlens"][b] + tok, head] = factor * q[b, w, head]
        tri += [(b, w, head), (b, (w + 1) % W, head), (b, w, (head + 1) % H), (b, W - 1, head)]
    a["k_shared"] = gr_synth.f32_to_bf16_bits(k)
    _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))), np.array(tri, dtype=np.int32))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,segments", [(128, 1), (256, 1), (128, 2)])
@pytest.mark.parametrize("width", [4.0, 32.0])
def test_scores_that_are_wide_from_the_first_tile_on(gr, oracle_lib, d, rows, segments, width):
    """Queries times 4, where some wavefronts' first tile passes 16 bits and makes them search from the start, and others search from a rise
    on or not at all; and times 32, where all of them do and scores go on to rise by tens of bits."""
    lens, W, Hq, Hkv = (330, 400, 65), 40, 8, 2
    a = rand_attn_case(1500 + d + rows, len(lens), W, Hq, Hkv, d, 3, 2, lens)
    a["q"] = gr_synth.f32_to_bf16_bits(width * gr_synth.bf16_bits_to_f32(a["q"]))
    gr.gr_diag_attn_plan(rows, segments)
    try:
        _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))))
    finally:
        gr.gr_diag_attn_plan(0, 0)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("W,Hq,Hkv", [(1, 2, 2), (31, 2, 2), (11, 6, 2), (43, 3, 1), (17, 8, 1), (257, 2, 2)])      # 1, 31, 33, 129, 136 and 257 rows per KV head
def test_partials_of_blocks_that_are_not_full(gr, oracle_lib, d, W, Hq, Hkv):
    # a segment's partials lie in blocks of up to 32 rows, column pieces first: rows that end inside a block, a line or a workgroup of the merge
    a = rand_attn_case(W, 2, W, Hq, Hkv, d, 3, 2, (330, 200))
    gr.gr_diag_attn_plan(128, 5)
    try:
        _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))))
    finally:
        gr.gr_diag_attn_plan(0, 0)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows,copies", [(128, 1), (128, 12), (256, 1)])      # two sets of wavefronts, workgroups of 4, of 8
def test_prompts_of_every_number_of_tiles(gr, oracle_lib, d, rows, copies):
    # tiles ahead are asked for in places that come round after two or three tiles: prompts of 1 to 8 tiles, whole and not
    lens = (1, 64, 65, 128, 129, 192, 193, 256, 257, 320, 321, 449) * copies
    a = rand_attn_case(d + rows, len(lens), 3, 4, 2, d, 3, 2, lens)
    gr.gr_diag_attn_plan(rows, 1)
    try:
        _check(gr, oracle_lib, a, float(np.float32(1 / np.sqrt(d))))
    finally:
        gr.gr_diag_attn_plan(0, 0)


@pytest.mark.parametrize("uniform", [True, False])
def test_segments_for_two_workgroups_per_cu(gr, oracle_lib, uniform):
    # 96 (request, KV head) pairs of one row block: split so that more workgroups run than there are CUs, in the order of their lengths where these differ
    B = 12
    lens = (1700,) * B if uniform else tuple(int(n) for n in np.random.default_rng(2).integers(1400, 1900, B))
    a = rand_attn_case(B, B, 20, 8, 8, 64, 3, 2, lens)
    assert gr.attn_workspace_bytes(B, 20, 8, 8, 64, max(lens), sum(lens)) >= 3 * B * 20 * 8 * (64 + 2) * 4       # (three segments or more: 288 workgroups)
    _check(gr, oracle_lib, a, 0.125)
