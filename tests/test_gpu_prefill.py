"""GPU parity: gr_prefill_attn (causal attention over packed prompts, paper Sections 2.2.1 / 5.1) against the
oracle's row-by-row definition.  Tolerances as for the decode attention: bf16 output, max-abs <= 2e-2 on
unit-variance inputs; LSE within 2e-3."""
import numpy as np
import pytest

import gr_synth
from gpu_util import bf16_to_dev, to_dev

pytestmark = pytest.mark.gpu


def _case(seed, lens, Hq, Hkv, d):
    rng = np.random.default_rng(seed)
    cu = np.zeros(len(lens) + 1, dtype=np.int32)
    cu[1:] = np.cumsum(lens)
    T = max(int(cu[-1]), 1)
    bf = lambda *s: gr_synth.f32_to_bf16_bits(rng.standard_normal(s, dtype=np.float32))
    return dict(q=bf(T, Hq, d), k=bf(T, Hkv, d), v=bf(T, Hkv, d), cu=cu)


def _run(gr, c, scale, want_lse=True):
    import torch
    T, Hq, d = c["q"].shape
    lens = np.diff(c["cu"])
    lse = torch.full((T, Hq), 7.0, dtype=torch.float32, device="cuda:0") if want_lse else None
    out = torch.full((T, Hq, d), 7.0, dtype=torch.bfloat16, device="cuda:0")
    gr.gr_prefill_attn(bf16_to_dev(c["q"]), bf16_to_dev(c["k"]), bf16_to_dev(c["v"]), to_dev(c["cu"]), scale,
                       int(lens.max()) if len(lens) else 0, int(c["cu"][-1]), out=out, lse_out=lse)
    torch.cuda.synchronize()
    return out.float().cpu().numpy(), (lse.cpu().numpy() if want_lse else None)


@pytest.mark.parametrize("lens,Hq,Hkv,d", [
    ((5, 19, 1, 33), 4, 2, 64),            # shorter than a tile, a one-token request
    ((70,), 8, 8, 64),                     # g = 1: 256 tokens per row block, ragged second tile
    ((130, 64, 257), 32, 8, 128),          # the benchmark's head geometry; several row blocks, block-aligned and ragged ends
    ((300,), 8, 2, 128),
    ((100, 37, 0, 129), 16, 2, 64),        # g = 8 and an empty request in the middle
    ((64, 128, 192), 4, 1, 128),           # tile-aligned lengths
])
def test_prefill_matches_oracle(oracle_lib, lens, Hq, Hkv, d):
    import paper_2512_11529_amd as gr
    gr.load_library()
    c = _case(hash((lens, Hq, Hkv, d)) % 1000, lens, Hq, Hkv, d)
    scale = float(np.float32(1 / np.sqrt(d)))
    out, lse = _run(gr, c, scale)
    ref, ref_lse = oracle_lib.prefill_attn_causal(c["q"], c["k"], c["v"], c["cu"], scale)
    T = int(c["cu"][-1])
    ref = ref.reshape(T, Hq, d)
    ref_lse = ref_lse.reshape(T, Hq)
    err = np.abs(out[:T] - ref).max()
    assert err <= 2e-2, f"max-abs {err}"
    np.testing.assert_allclose(lse[:T], ref_lse, rtol=0, atol=2e-3)


@pytest.mark.parametrize("lens,Hq,Hkv,max_L", [(*case, n) for n in (2048, 2049) for case in (      # head size 128: blocks of 128 and of 256 query rows
    ((1, 31, 33, 63, 65), 32, 8),          # g = 4: 32 and 64 tokens per row block
    ((257, 128, 129, 2), 4, 4),            # g = 1: row blocks of 128 and 256 tokens
    ((43, 86, 90), 6, 2),                  # g = 3: a token's heads lie in two row blocks
)] + [((n,), 8, 1, n) for n in (1280, 1281, 2048)])        # one (prompt, KV head) pair of 40 to 64 blocks of 256 rows: 128, 256, 256
def test_prefill_row_blocks_of_both_sizes(oracle_lib, lens, Hq, Hkv, max_L):
    """max_L is a bound that the longest prompt need not reach; it decides the size of a row block."""
    import paper_2512_11529_amd as gr
    import torch
    gr.load_library()
    d = 128
    c = _case(sum(lens), lens, Hq, Hkv, d)
    scale = float(np.float32(1 / np.sqrt(d)))
    T = int(c["cu"][-1])
    lse = torch.empty((T, Hq), dtype=torch.float32, device="cuda:0")
    out, _ = gr.gr_prefill_attn(bf16_to_dev(c["q"]), bf16_to_dev(c["k"]), bf16_to_dev(c["v"]), to_dev(c["cu"]), scale, max_L, T, lse_out=lse)
    torch.cuda.synchronize()
    ref, ref_lse = oracle_lib.prefill_attn_causal(c["q"], c["k"], c["v"], c["cu"], scale)
    assert np.abs(out.float().cpu().numpy() - ref.reshape(T, Hq, d)).max() <= 2e-2
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse.reshape(T, Hq), rtol=0, atol=2e-3)


def test_prefill_long_prompt_sampled_rows(oracle_lib):
    """L = 4096 at the benchmark's head geometry: 16 row blocks per KV head, up to 64 tiles per block.  Rows checked:
    the first and last token of every 64-token block (diagonal tiles, block edges) and a seeded sample, every head."""
    import paper_2512_11529_amd as gr
    gr.load_library()
    L, Hq, Hkv, d = 4096, 32, 8, 128
    c = _case(77, (L,), Hq, Hkv, d)
    scale = float(np.float32(1 / np.sqrt(d)))
    out, lse = _run(gr, c, scale)
    rng = np.random.default_rng(5)
    toks = sorted(set([0, 1, 2, L - 1] + [64 * k for k in range(L // 64)] + [64 * k + 63 for k in range(L // 64)] + list(rng.integers(0, L, 120))))
    tri = np.array([(0, i, h) for i in toks for h in range(Hq)], dtype=np.int32)
    ref, ref_lse = oracle_lib.prefill_attn_causal(c["q"], c["k"], c["v"], c["cu"], scale, tri)
    got = out[tri[:, 1], tri[:, 2]]
    err = np.abs(got - ref).max()
    assert err <= 2e-2, f"max-abs {err}"
    np.testing.assert_allclose(lse[tri[:, 1], tri[:, 2]], ref_lse, rtol=0, atol=2e-3)


def test_prefill_ragged_batch_touches_only_its_rows(oracle_lib):
    """Rows past total_L in the output buffer stay untouched; every row below is written."""
    import torch
    import paper_2512_11529_amd as gr
    gr.load_library()
    c = _case(9, (40, 200, 3), 8, 2, 64)
    T = int(c["cu"][-1])
    pad = 5
    q = torch.cat([bf16_to_dev(c["q"]), torch.zeros((pad, 8, 64), dtype=torch.bfloat16, device="cuda:0")])
    k = torch.cat([bf16_to_dev(c["k"]), torch.zeros((pad, 2, 64), dtype=torch.bfloat16, device="cuda:0")])
    v = k.clone(); v[:T] = bf16_to_dev(c["v"])
    out = torch.full_like(q, 7.0)
    gr.gr_prefill_attn(q, k, v, to_dev(c["cu"]), 0.125, 200, T, out=out)
    torch.cuda.synchronize()
    assert (out[T:] == 7.0).all()
    ref, _ = oracle_lib.prefill_attn_causal(c["q"], c["k"], c["v"], c["cu"], 0.125)
    assert np.abs(out[:T].float().cpu().numpy() - ref.reshape(T, 8, 64)).max() <= 2e-2


def test_prefill_rejects_bad_arguments():
    import torch
    import paper_2512_11529_amd as gr
    gr.load_library()
    dev = torch.device("cuda:0")
    q = torch.zeros((8, 4, 64), dtype=torch.bfloat16, device=dev)
    kv = torch.zeros((8, 2, 64), dtype=torch.bfloat16, device=dev)
    cu = torch.tensor([0, 8], dtype=torch.int32, device=dev)
    for scale in (0.0, -1.0, float("nan"), float("inf")):
        with pytest.raises(gr.GrError) as e:
            gr.gr_prefill_attn(q, kv, kv, cu, scale, 8, 8)
        assert e.value.status == -1
    q32 = torch.zeros((8, 4, 32), dtype=torch.bfloat16, device=dev)
    kv32 = torch.zeros((8, 2, 32), dtype=torch.bfloat16, device=dev)
    with pytest.raises(gr.GrError) as e:
        gr.gr_prefill_attn(q32, kv32, kv32, cu, 0.1, 8, 8)
    assert e.value.status == -2
    with pytest.raises(gr.GrError) as e:                 # total_L larger than B * max_L
        gr.gr_prefill_attn(q, kv, kv, cu, 0.1, 4, 8)
    assert e.value.status == -1
    out, _ = gr.gr_prefill_attn(q, kv, kv, torch.tensor([0, 0], dtype=torch.int32, device=dev), 0.1, 0, 0)     # empty batch: nothing to do
    torch.cuda.synchronize()


def test_prefill_ragged_long_batch_sampled_rows(oracle_lib):
    """Eight prompts of 512..8192 tokens (the length mix of the high-concurrency workload) at the benchmark's head
    geometry: the grid is sized by the longest prompt, so most row blocks of the short requests leave at once and the
    rest are dispatched heaviest first.  Rows checked per request: first, last, the last row of the first block, the
    rows on both sides of every 1024th token, and a seeded sample; every head."""
    import paper_2512_11529_amd as gr
    gr.load_library()
    Hq, Hkv, d = 32, 8, 128
    rng = np.random.default_rng(12)
    lens = tuple(int(x) for x in rng.integers(512, 8193, size=8))
    c = _case(78, lens, Hq, Hkv, d)
    scale = float(np.float32(1 / np.sqrt(d)))
    out, lse = _run(gr, c, scale)
    tri = []
    for b, L in enumerate(lens):
        toks = {0, L - 1, 63, 64} | {t for k in range(1024, L, 1024) for t in (k - 1, k)} | set(int(x) for x in rng.integers(0, L, 12))
        tri += [(b, i, h) for i in sorted(toks) for h in range(Hq)]
    tri = np.array(tri, dtype=np.int32)
    ref, ref_lse = oracle_lib.prefill_attn_causal(c["q"], c["k"], c["v"], c["cu"], scale, tri)
    rows = c["cu"][tri[:, 0]] + tri[:, 1]
    err = np.abs(out[rows, tri[:, 2]] - ref).max()
    assert err <= 2e-2, f"max-abs {err}"
    np.testing.assert_allclose(lse[rows, tri[:, 2]], ref_lse, rtol=0, atol=2e-3)
    assert np.isfinite(out[:int(c["cu"][-1])]).all()


@pytest.mark.parametrize("d,max_L", [(64, 330), (128, 330), (128, 2049)])      # blocks of 128, 128 and 256 query rows
@pytest.mark.parametrize("factor", [3.0, 7.0, 12.0])
def test_prefill_scores_that_jump_inside_the_prompt(oracle_lib, d, max_L, factor):
    """Keys far above everything before them, in a tile before and on a block's diagonal: the reference is raised after the tile, or
    the wavefront computes its columns again."""
    import torch
    import paper_2512_11529_amd as gr
    gr.load_library()
    c = _case(77 + d, (330, 200), 8, 2, d)
    q, k = gr_synth.bf16_bits_to_f32(c["q"]), gr_synth.bf16_bits_to_f32(c["k"]).copy()
    for row, head, tok in [(300, 1, 100), (329, 5, 328), (330 + 199, 0, 330 + 130)]:
        k[tok, head // 4] = factor * q[row, head]
    c["k"] = gr_synth.f32_to_bf16_bits(k)
    scale = float(np.float32(1 / np.sqrt(d)))
    out = torch.empty(c["q"].shape, dtype=torch.bfloat16, device="cuda:0")
    gr.gr_prefill_attn(bf16_to_dev(c["q"]), bf16_to_dev(c["k"]), bf16_to_dev(c["v"]), to_dev(c["cu"]), scale, max_L, 530, out=out)
    ref, _ = oracle_lib.prefill_attn_causal(c["q"], c["k"], c["v"], c["cu"], scale)
    err = np.abs(out.float().cpu().numpy() - ref.reshape(out.shape)).max()
    assert err <= 2e-2, f"max-abs {err}"


@pytest.mark.parametrize("B,Hq,Hkv,d,L_min,L_max", [
    (24, 8, 8, 64, 0, 300),         # head size 64, prompts without a block among them
    (64, 8, 8, 64, 100, 256),       # the most (request, KV head) pairs that are dealt by weight: 64 to an XCD
    (65, 8, 8, 64, 100, 256),       # one request more: pair by pair
    (8, 32, 8, 128, 1, 290),        # 8 pairs to an XCD
    (16, 32, 8, 128, 1, 200),       # 64 rows of a token, prompts of unlike length
    (16, 6, 3, 128, 300, 700),      # KV heads that do not divide the XCDs evenly
    (17, 16, 2, 128, 20, 220),      # 34 pairs: some XCDs have one more
    (8, 32, 8, 128, 256, 256),      # one length, every block full, all with a place at once (pair by pair)
    (8, 32, 8, 128, 288, 288),      # the same with more blocks
    (12, 32, 8, 128, 150, 200),     # 48 rows of a token to an XCD, the most of prompts of like length
    (13, 32, 8, 128, 150, 200),     # 52 of prompts of like length: pair by pair
    (13, 32, 8, 128, 1, 200),       # 52, and prompts of unlike length
    (17, 32, 8, 128, 1, 200),       # 68: pair by pair
    (32, 32, 8, 64, 100, 128),      # head size 64, 128 rows of a token, like lengths
    (33, 32, 8, 64, 100, 128),      # 132: pair by pair
    (33, 32, 8, 64, 0, 128),        # unlike lengths
])
def test_prefill_blocks_dealt_by_weight(oracle_lib, B, Hq, Hkv, d, L_min, L_max):
    """More row blocks than have a place at once, dealt heaviest first over all pairs of an XCD: every row of every request is written
    once and is right."""
    import paper_2512_11529_amd as gr
    gr.load_library()
    rng = np.random.default_rng(B + L_max)
    lens = rng.integers(L_min, L_max + 1, B)
    lens[B // 2] = L_max
    c = _case(B + d, tuple(int(n) for n in lens), Hq, Hkv, d)
    scale = float(np.float32(1 / np.sqrt(d)))
    out, lse = _run(gr, c, scale)
    ref, ref_lse = oracle_lib.prefill_attn_causal(c["q"], c["k"], c["v"], c["cu"], scale)
    T = int(c["cu"][-1])
    assert np.abs(out[:T] - ref.reshape(T, Hq, d)).max() <= 2e-2
    np.testing.assert_allclose(lse[:T], ref_lse.reshape(T, Hq), rtol=0, atol=2e-3)


@pytest.mark.parametrize("d,max_L", [(64, 330), (128, 330), (128, 2049)])      # blocks of 128, 128 and 256 query rows
@pytest.mark.parametrize("power", [-118, 110])
def test_prefill_values_near_the_ends_of_the_range(d, max_L, power):
    """V times a power of two gives the output times that power, also where a row's scores jump by 34 to 50 bits.  The bound: two roundings
    to bf16, 2^-7 max|V|."""
    import torch
    import paper_2512_11529_amd as gr
    gr.load_library()
    c = _case(79 + d, (330, 200), 8, 2, d)
    q, k, v = (gr_synth.bf16_bits_to_f32(c[n]).copy() for n in ("q", "k", "v"))
    for row, head, tok in [(300, 1, 100), (329, 5, 328), (330 + 199, 0, 330 + 130)]:
        k[tok, head // 4] = 3.0 * q[row, head]
    c["k"] = gr_synth.f32_to_bf16_bits(k)
    scale = float(np.float32(1 / np.sqrt(d)))

    def run(values):
        out = torch.empty(c["q"].shape, dtype=torch.bfloat16, device="cuda:0")
        gr.gr_prefill_attn(bf16_to_dev(c["q"]), bf16_to_dev(c["k"]), bf16_to_dev(gr_synth.f32_to_bf16_bits(values)), to_dev(c["cu"]), scale, max_L, 530, out=out)
        return out.float().cpu().numpy()

    want, out = run(v), run(np.ldexp(v, power))
    assert np.isfinite(out).all()
    assert np.abs(np.ldexp(out, -power) - want).max() <= 2.0 ** -7 * float(np.abs(v).max())


@pytest.mark.parametrize("d,max_L", [(64, 330), (128, 330), (128, 2049)])
@pytest.mark.parametrize("factor", [3.0, 12.0])
def test_prefill_a_token_that_is_nearly_all_of_the_sum(d, max_L, factor):
    """A key 34 bits or more above all others of a row: the output is its V row, every bit of it (values between 1 and 2)."""
    import torch
    import paper_2512_11529_amd as gr
    gr.load_library()
    c = _case(83 + d, (330, 200), 8, 2, d)
    rng = np.random.default_rng(13)
    v = (rng.choice([-1.0, 1.0], c["v"].shape) * rng.uniform(1.0, 2.0, c["v"].shape)).astype(np.float32)
    c["v"] = gr_synth.f32_to_bf16_bits(v)
    q, k = gr_synth.bf16_bits_to_f32(c["q"]), gr_synth.bf16_bits_to_f32(c["k"]).copy()
    rows_of = [(300, 1, 100), (329, 5, 328), (310, 6, 70), (200, 2, 5), (180, 3, 179), (160, 7, 140), (330 + 199, 0, 330 + 130), (330 + 150, 4, 330 + 149)]
    for row, head, tok in rows_of:
        k[tok, head // 4] = factor * q[row, head]
    c["k"] = gr_synth.f32_to_bf16_bits(k)
    out = torch.empty(c["q"].shape, dtype=torch.bfloat16, device="cuda:0")
    gr.gr_prefill_attn(bf16_to_dev(c["q"]), bf16_to_dev(c["k"]), bf16_to_dev(c["v"]), to_dev(c["cu"]), float(np.float32(1 / np.sqrt(d))), max_L, 530, out=out)
    out, v = out.float().cpu().numpy(), gr_synth.bf16_bits_to_f32(c["v"])
    for row, head, tok in rows_of:
        np.testing.assert_array_equal(out[row, head], v[tok, head // 4], err_msg=f"row {row}, head {head}")


def test_prefill_rows_do_not_depend_on_total_L(oracle_lib):
    """total_L only chooses a plan: a number that is too small leaves no row out, also where blocks are dealt by weight."""
    import torch
    import paper_2512_11529_amd as gr
    gr.load_library()
    c = _case(91, (290, 200, 250, 280, 210, 290, 260, 230), 32, 8, 128)
    scale = float(np.float32(1 / np.sqrt(128)))
    want, _ = _run(gr, c, scale)
    out = torch.full(c["q"].shape, 7.0, dtype=torch.bfloat16, device="cuda:0")
    gr.gr_prefill_attn(bf16_to_dev(c["q"]), bf16_to_dev(c["k"]), bf16_to_dev(c["v"]), to_dev(c["cu"]), scale, 290, 300, out=out)
    np.testing.assert_array_equal(out.float().cpu().numpy(), want)


@pytest.mark.parametrize("d,max_L", [(64, 330), (128, 330), (128, 2049)])
@pytest.mark.parametrize("width", [4.0, 32.0])
def test_prefill_scores_that_are_wide_from_the_first_tile_on(oracle_lib, d, max_L, width):
    """Some wavefronts, or all, search from the first tile on."""
    import torch
    import paper_2512_11529_amd as gr
    gr.load_library()
    c = _case(97 + d, (330, 65, 200), 8, 2, d)
    c["q"] = gr_synth.f32_to_bf16_bits(width * gr_synth.bf16_bits_to_f32(c["q"]))
    scale = float(np.float32(1 / np.sqrt(d)))
    out = torch.empty(c["q"].shape, dtype=torch.bfloat16, device="cuda:0")
    lse = torch.empty(c["q"].shape[:2], dtype=torch.float32, device="cuda:0")
    gr.gr_prefill_attn(bf16_to_dev(c["q"]), bf16_to_dev(c["k"]), bf16_to_dev(c["v"]), to_dev(c["cu"]), scale, max_L, 595, out=out, lse_out=lse)
    ref, ref_lse = oracle_lib.prefill_attn_causal(c["q"], c["k"], c["v"], c["cu"], scale)
    assert np.abs(out.float().cpu().numpy() - ref.reshape(out.shape)).max() <= 2e-2
    np.testing.assert_allclose(lse.cpu().numpy(), ref_lse.reshape(lse.shape), rtol=0, atol=2e-3)
