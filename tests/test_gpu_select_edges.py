"""GPU: the item step where its kernels change hands, bit-exact against the oracle - rows around the blocks and lines that a
streamed row is cut into, child counts around the limits of the gathered forms (scores kept, one wavefront, a workgroup) at
levels 1 and 2, more beams than the selection keeps single groups for, and fewer groups than beams."""
import numpy as np
import pytest
import torch

import gr_synth
from gpu_util import assert_select_equal, run_select, to_dev
from test_gpu_select import gr  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("step", [0, 1])
@pytest.mark.parametrize("W,V", [(3, 3), (5, 31), (4, 2047), (6, 2050), (5, 8191), (5, 8193), (4, 16387), (3, 24575), (2, 32768), (70, 515), (1030, 33)])
def test_streamed_rows_without_a_mask(gr, oracle_lib, W, V, step):  # noqa: F811
    # step 0 deals rows to 512 threads, a later step to 256; some beams are dead
    rng = np.random.default_rng(V + W + step)
    B = 2
    logits = (3.0 * rng.standard_normal((B, W, V))).astype(np.float32)
    logits[0, 0, V - 1] = 9.0                                      # the row's last token wins
    sc = (-3.0 * rng.random((B, W))).astype(np.float32)
    sc[:, 2::3] = -np.inf
    pf = np.full((B, W, 3), -1, np.int32)
    pf[:, :, :step] = 0
    rg = np.zeros((B, W, 2), np.int32)
    assert_select_equal(run_select(gr, None, logits, sc, pf, rg, step), oracle_lib.beam_select(None, logits, sc, pf, step))


def _children(rng, V, counts):
    """Sorted distinct tokens per entry of `counts`."""
    return [np.sort(rng.choice(V, size=n, replace=False)) for n in counts]


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("V,W", [(4100, 13), (4100, 600), (9001, 20)])
def test_child_counts_at_the_limits(gr, oracle_lib, V, W, flags):  # noqa: F811
    rng = np.random.default_rng(V + W)
    counts = [1, 15, 16, 17, 239, 240, 241, 1023, 1024, 1025, 2300, 3900]
    rows = []
    for t1, second in enumerate(_children(rng, V, counts)):        # level 1: first token t1 has counts[t1] children
        rows += [(t1, int(t2), int(rng.integers(V))) for t2 in second]
    last = len(counts)
    for t2, third in enumerate(_children(rng, V, counts)):         # level 2: pair (last, t2) has counts[t2] children
        rows += [(last, t2, int(t3)) for t3 in third]
    items = np.array(sorted(rows), dtype=np.int32)
    mask = gr.gr_item_mask_build(to_dev(items), V)
    sc, pf, rg = gr_synth.initial_beam_state(1, W, 3)
    for step in range(3):
        logits = (2.0 * rng.standard_normal((1, W, V))).astype(np.float32)
        if step == 1:
            logits[0, :, :len(counts)] += np.where(pf[0, :, 0] == last, 30.0, 0.0)[:, None].astype(np.float32)   # keep the pairs of `last`
        want = oracle_lib.beam_select(items, logits, sc, pf, step)
        assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, step, flags), want, f"step {step}")
        sc, pf, rg = want["scores"], want["prefix"], want["range"]


@pytest.mark.parametrize("spread", [1e-4, 1e-2, 40.0])
def test_scores_close_together_and_far_apart(gr, oracle_lib, spread):  # noqa: F811
    # the histograms adapt their bins to the range of the scores; 40 reaches past what 2048 bins of 1/64 cover
    rng = np.random.default_rng(5)
    B, W, V = 2, 48, 3000
    logits = (spread * rng.standard_normal((B, W, V))).astype(np.float32)
    sc = (-0.1 * spread * rng.random((B, W))).astype(np.float32)
    pf = np.full((B, W, 3), -1, np.int32)
    rg = np.zeros((B, W, 2), np.int32)
    for step in (0, 1):
        pf[:, :, :step] = 0
        assert_select_equal(run_select(gr, None, logits, sc, pf, rg, step), oracle_lib.beam_select(None, logits, sc, pf, step), f"step {step}")
    one = np.full((B, W), -np.inf, np.float32)
    one[:, 7] = 0.0                                                # a single live beam: fewer groups than beams
    assert_select_equal(run_select(gr, None, logits, one, pf, rg, 0), oracle_lib.beam_select(None, logits, one, pf, 0))


def _suppressed(pattern, n):
    """Positions in a child list of n whose logits are -inf."""
    at = np.arange(n)
    return dict(wave_0=(at % 2048) < 512,                          # every part of 512 that the first of four wavefronts takes
                wave_3=(at % 2048) >= 1536,
                all_but_last=at < n - 1, all_but_one=at != min(700, n - 1), all=at >= 0, second_half=at >= n // 2)[pattern]


@pytest.mark.parametrize("step", [1, 2])
@pytest.mark.parametrize("pattern", ["wave_0", "wave_3", "all_but_last", "all_but_one", "all", "second_half"])
def test_long_child_lists_with_suppressed_tokens(gr, oracle_lib, pattern, step):  # noqa: F811
    # -inf logits (a top-k or category filter in front of the item step) over whole parts of rows that a workgroup gathers
    rng = np.random.default_rng(step)
    V, counts = 8200, (300, 1025, 2049, 3000, 8192)
    lists = _children(rng, V, counts)
    if step == 1:
        items = np.array([(t1, t2, int(rng.integers(V))) for t1, lst in enumerate(lists) for t2 in lst], dtype=np.int32)
    else:
        items = np.array([(4, t2, t3) for t2, lst in enumerate(lists) for t3 in lst], dtype=np.int32)
    mask = gr.gr_item_mask_build(to_dev(items), V)
    W = 2 * len(counts)
    pf = np.full((2, W, 3), -1, np.int32)
    rg = np.zeros((2, W, 2), np.int32)
    end = np.cumsum(counts)
    logits = (2.0 * rng.standard_normal((2, W, V))).astype(np.float32)
    for w in range(W):
        i = w % len(counts)
        pf[:, w, :step] = [i] if step == 1 else [4, i]
        rg[:, w] = end[i] - counts[i], end[i]
        logits[0, w, lists[i][_suppressed(pattern, counts[i])]] = -np.inf
    logits[1] = logits[0]
    sc = (-3.0 * rng.random((2, W))).astype(np.float32)
    sc[1, np.arange(W) != 3] = -np.inf                             # request 1: a row of 3000 is its only live beam
    assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, step), oracle_lib.beam_select(items, logits, sc, pf, step))


@pytest.mark.parametrize("live,finite", [(200, 1), (20, 1), (3, 1), (1, 200), (12, 20), (256, 0)])
@pytest.mark.parametrize("masked", [False, True])
def test_fewer_finite_candidates_than_beams(gr, oracle_lib, live, finite, masked):  # noqa: F811
    # every live beam has `finite` finite logits, so that most slots of the new generation are dead
    rng = np.random.default_rng(live + finite)
    B, W, V = 2, 256, 8192
    logits = np.full((B, W, V), -np.inf, np.float32)
    items = mask = None
    pf = np.full((B, W, 3), -1, np.int32)
    rg = np.zeros((B, W, 2), np.int32)
    pf[:, :, 0] = 0
    if masked:                                                     # every first token has 5000 children
        children = _children(rng, V, [5000] * 4)
        items = np.array([(t1, t2, 7) for t1 in range(4) for t2 in children[t1]], dtype=np.int32)
        mask = gr.gr_item_mask_build(to_dev(items), V)
        pf[:, :, 0] = np.arange(W) % 4
        rg[:, :, 0], rg[:, :, 1] = 5000 * pf[:, :, 0], 5000 * (pf[:, :, 0] + 1)
    for b in range(B):
        for w in range(W):
            at = rng.choice(V if not masked else 5000, size=finite, replace=False)
            at = children[w % 4][at] if masked else at
            logits[b, w, at] = rng.standard_normal(finite)
    sc = np.full((B, W), -np.inf, np.float32)
    for b in range(B):
        sc[b, rng.choice(W, size=live, replace=False)] = -rng.random(live)
    assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, 1), oracle_lib.beam_select(items, logits, sc, pf, 1))


@pytest.mark.parametrize("flags", [0, 1])
def test_a_range_no_mask_produces_has_no_children(gr, oracle_lib, flags):  # noqa: F811
    # wider than the vocabulary, outside the table, or backwards: the beam is dead, the others are selected as without it
    rng = np.random.default_rng(3)
    V, W, children = 64, 8, 40
    thirds = _children(rng, V, [children] * 60)
    items = np.array([(0, t2, t3) for t2, lst in enumerate(thirds) for t3 in lst], dtype=np.int32)
    mask = gr.gr_item_mask_build(to_dev(items), V)
    logits = (2.0 * rng.standard_normal((1, W, V))).astype(np.float32)
    pf = np.full((1, W, 3), -1, np.int32)
    pf[:, :, 0], pf[:, :, 1] = 0, np.arange(W)
    rg = np.stack([children * np.arange(W), children * (np.arange(W) + 1)], 1).astype(np.int32)[None]
    sc = -rng.random((1, W)).astype(np.float32)
    bad = [1, 3, 4, 6]
    rg[0, bad] = [[0, V + 1], [0, len(items)], [len(items) - 3, len(items) + 1], [90, 80]]
    live = sc.copy()
    live[0, bad] = -np.inf
    assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, 2, flags), oracle_lib.beam_select(items, logits, live, pf, 2))


def _second_level(rng, W, V, widths, items, oracle_lib):
    """Inputs of the step after a first one: beams as the oracle selects them from logits of widths[0], logits of widths[1]."""
    sc, pf, rg = gr_synth.initial_beam_state(1, W, 3)
    logits = (widths[0] * rng.standard_normal((1, W, V))).astype(np.float32)
    first = oracle_lib.beam_select(items, logits, sc, pf, 0)
    logits = (widths[1] * rng.standard_normal((1, W, V))).astype(np.float32)
    return logits, first["scores"], first["prefix"], first["range"]


# widths of the logits at the first and the second level: few beams far ahead of the others, all close together, far apart
_WIDTHS = [(6.0, 1.0), (10.0, 2.0), (0.05, 0.05), (20.0, 20.0)]


@pytest.mark.parametrize("widths", _WIDTHS)
@pytest.mark.parametrize("W,V", [(128, 8192), (512, 8192), (300, 20000), (1100, 2000), (2048, 1024)])
def test_spread_of_beam_scores_without_a_mask(gr, oracle_lib, W, V, widths):  # noqa: F811
    logits, sc, pf, rg = _second_level(np.random.default_rng(W + V), W, V, widths, None, oracle_lib)
    assert_select_equal(run_select(gr, None, logits, sc, pf, rg, 1), oracle_lib.beam_select(None, logits, sc, pf, 1))


@pytest.mark.parametrize("widths", _WIDTHS)
@pytest.mark.parametrize("first,children,W", [(5, 5000, 256), (8, 8192, 512), (8, 8192, 2048), (40, 3000, 256), (600, 700, 512), (64, 200, 300), (9, 100, 1200)])
def test_spread_of_beam_scores_with_few_first_tokens(gr, oracle_lib, first, children, W, widths):  # noqa: F811
    rng = np.random.default_rng(first + W)
    V = 8192
    items = np.array([(13 * t1, t2, 5) for t1, lst in enumerate(_children(rng, V, [children] * first)) for t2 in lst], dtype=np.int32)
    mask = gr.gr_item_mask_build(to_dev(items), V)
    logits, sc, pf, rg = _second_level(rng, W, V, widths, items, oracle_lib)
    assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, 1), oracle_lib.beam_select(items, logits, sc, pf, 1))


@pytest.mark.parametrize("low", [-np.inf, np.finfo(np.float32).min, -1e9, -65504.0])
@pytest.mark.parametrize("W,live", [(128, 1), (128, 128), (700, 10)])
def test_filtered_logits(gr, oracle_lib, W, live, low):  # noqa: F811
    # 50 tokens of every row are left by a filter, the others are set to a lowest value that is a candidate of its own where finite
    rng = np.random.default_rng(W)
    V = 4100
    logits = np.full((2, W, V), low, np.float32)
    for b in range(2):
        for w in range(W):
            logits[b, w, rng.choice(V, size=50, replace=False)] = 2.0 * rng.standard_normal(50)
    sc = np.full((2, W), -np.inf, np.float32)
    sc[:, :live] = -rng.random((2, live))
    pf = np.full((2, W, 3), -1, np.int32)
    rg = np.zeros((2, W, 2), np.int32)
    for step in (0, 1):
        pf[:, :, :step] = 0
        assert_select_equal(run_select(gr, None, logits, sc, pf, rg, step), oracle_lib.beam_select(None, logits, sc, pf, step), f"step {step}")


def test_spread_of_beam_scores_does_not_change_the_time(gr):  # noqa: F811
    # the exact fallback takes 20 times as long as the selection it stands in for; it is for ties, not for score distributions
    import torch
    B, W, V = 8, 512, 8192
    g = torch.Generator(device="cuda:0")

    def time(widths, mask):
        g.manual_seed(7)
        sc = torch.full((B, W), -np.inf, device="cuda:0")
        sc[:, 0] = 0.0
        beams = dict(scores=sc, prefix=torch.full((B, W, 3), -1, dtype=torch.int32, device="cuda:0"),
                     range=torch.zeros(B, W, 2, dtype=torch.int32, device="cuda:0"))
        for step in (0, 1):
            x = torch.empty(B, W, V, device="cuda:0").normal_(generator=g).mul_(widths[step])
            run = lambda: gr.gr_beam_select(mask, x, beams["scores"], beams["prefix"], beams["range"], step)
            after = run()
            if step == 1:
                best = np.inf
                for _ in range(5):
                    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                    a.record()
                    for _ in range(5):
                        run()
                    b.record()
                    b.synchronize()
                    best = min(best, a.elapsed_time(b))
            beams = after
        return best

    children = _children(np.random.default_rng(1), V, [5000] * 12)
    mask = gr.gr_item_mask_build(to_dev(np.array([(t1, t2, 5) for t1, lst in enumerate(children) for t2 in lst], dtype=np.int32)), V)
    usual = time((3.0, 3.0), None)
    for widths in [(3.0, 1.0)] + _WIDTHS:
        assert time(widths, None) < 5 * usual, widths
        assert time(widths, mask) < 5 * usual, widths


@pytest.mark.parametrize("V,W", [(1, 1), (3, 1), (5, 16), (255, 16), (2048, 512), (2049, 1023), (8191, 256), (8192, 1024), (8192, 1025), (8193, 128)])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("pattern", ["normal", "equal", "close", "one far ahead", "one far below", "inf"])
def test_level_0_of_one_live_beam(gr, oracle_lib, V, W, masked, pattern):  # noqa: F811
    """The first beam of every request alone is live: its workgroup selects as well, unless the row is longer than a block, the beams
    are too many, or thousands of scores are as good as equal.  Around these limits, fewer tokens than beams, requests beside
    them that start otherwise (another beam, two beams, none)."""
    rng = np.random.default_rng(V + W)
    B = 5
    x = rng.standard_normal((B, W, V))
    if pattern == "equal":
        x[:] = 1.25
    elif pattern == "close":
        x = 1.0 + 1e-6 * x
    elif pattern == "one far ahead":
        x[:, :, V // 2] = 400.0
    elif pattern == "one far below":
        x[:, :, V // 3] = -1e6
    elif pattern == "inf":
        x[:, :, rng.random(V) < 0.5] = -np.inf
    logits = x.astype(np.float32)
    sc = np.full((B, W), -np.inf, np.float32)
    sc[:3, 0] = [0.0, -2.5, 7.0]
    sc[3, W - 1] = -1.0                                            # a beam that is not the first (or is: W = 1)
    if W > 1:
        sc[2, W - 1] = 6.5                                         # two; request 4 has none
    pf, rg = np.full((B, W, 3), -1, np.int32), np.zeros((B, W, 2), np.int32)
    items = mask = None
    if masked:
        t1 = np.flatnonzero(rng.random(V) < 0.6) if V > 1 else np.array([0])
        if len(t1) == 0:
            t1 = np.array([V - 1])
        items = np.stack([np.repeat(t1, 2), np.tile([0, V - 1], len(t1)), np.zeros(2 * len(t1), np.int64)], axis=1).astype(np.int32)
        items = np.unique(items, axis=0)
        mask = gr.gr_item_mask_build(to_dev(items), V)
    want = oracle_lib.beam_select(items, logits, sc, pf, 0)
    for _ in range(2):
        assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, 0), want)


@pytest.mark.parametrize("B,W,V", [(1, 16, 256), (5, 128, 8192), (600, 60, 64)])
def test_level_0_with_scores_in_place(gr, oracle_lib, B, W, V):  # noqa: F811
    """Scores written over the ones that came in, also for more rows than one look of every workgroup at its rows' scores covers (600 x 60):
    the incoming scores are read before any is written, so only the selection's own launch writes them."""
    rng = np.random.default_rng(B + W + V)
    logits = (3.0 * rng.standard_normal((B, W, V))).astype(np.float32)
    sc = np.full((B, W), -np.inf, np.float32)
    sc[:, 0] = -rng.random(B)
    pf, rg = np.full((B, W, 3), -1, np.int32), np.zeros((B, W, 2), np.int32)
    want = oracle_lib.beam_select(None, logits, sc, pf, 0)
    scores = to_dev(sc)
    i32 = lambda *shape: torch.empty(shape, dtype=torch.int32, device="cuda:0")
    out = {"parent": i32(B, W), "token": i32(B, W), "scores": scores, "prefix": i32(B, W, 3), "range": i32(B, W, 2), "item_index": i32(B, W)}
    gr.gr_beam_select(None, to_dev(logits), scores, to_dev(pf), to_dev(rg), 0, out=out)
    torch.cuda.synchronize()
    assert_select_equal({k: v.cpu().numpy() for k, v in out.items()}, want)


@pytest.mark.parametrize("W,counts", [(3, [1, 2, 5]), (40, [4, 5, 60, 64]), (128, [16, 17]), (129, [16, 17]), (500, [1, 4, 5]), (600, [1, 4, 5]), (1024, [1, 3]), (1030, [1, 3]),
                                      (64, [240]), (64, [240, 241])])
@pytest.mark.parametrize("close", [False, True])
def test_short_lists_taken_at_once(gr, oracle_lib, W, counts, close):  # noqa: F811
    """The last level with few scores (taken all at once, up to 512 quads), more of them (listed first) and a row that leaves keys; with
    dead beams among them or without, and with scores as good as equal."""
    rng = np.random.default_rng(W + sum(counts))
    V = max(300, W)
    rows = []
    for t1, third in enumerate(_children(rng, V, [counts[i % len(counts)] for i in range(W)])):
        rows += [(t1, 0, int(t3)) for t3 in third]
    items = np.array(rows, dtype=np.int32)
    mask = gr.gr_item_mask_build(to_dev(items), V)
    starts = np.searchsorted(items[:, 0], np.arange(W + 1))
    for dead in (False, True):
        logits = (1.25 + (1e-6 if close else 2.0) * rng.standard_normal((1, W, V))).astype(np.float32)     # (sums of 1 in fp32, not beside 0)
        sc = np.sort(-(0.0 if close else 3.0) * rng.random((1, W))).astype(np.float32)[:, ::-1].copy()
        if dead:
            sc[0, W // 2:: 3] = -np.inf
        pf = np.full((1, W, 3), -1, np.int32)
        pf[0, :, 0], pf[0, :, 1] = np.arange(W), 0
        rg = np.stack([starts[:-1], starts[1:]], axis=1)[None].astype(np.int32)
        want = oracle_lib.beam_select(items, logits, sc, pf, 2)
        assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, 2), want, f"dead {dead}")


@pytest.mark.parametrize("W,V", [(1, 1), (2, 64), (16, 256), (15, 1024), (16, 512), (16, 513), (16, 1024), (16, 1025), (17, 1024)])
@pytest.mark.parametrize("counts", [[1], [0, 3, 64], [240, 241, 512, 513], [10 ** 6]])
def test_requests_that_one_workgroup_gathers(gr, oracle_lib, W, V, counts):  # noqa: F811
    """Levels 1 and 2 around the most beams and the longest vocabulary that the selecting workgroup gathers itself: rows without children,
    with few, of every length up to the vocabulary; dead beams, a request of dead beams alone, scores in place."""
    rng = np.random.default_rng(W + V + len(counts))
    B, T = 3, min(V, 40)
    counts = [min(counts[i % len(counts)], V) for i in range(T)]
    second = _children(rng, V, counts)
    items = np.array([(t1, int(t2), int(t3)) for t1, row in enumerate(second) for t2 in row for t3 in sorted({0, V // 2, V - 1})], dtype=np.int32)
    if len(items) == 0:
        items = np.zeros((1, 3), np.int32)
    mask = gr.gr_item_mask_build(to_dev(items), V)
    sc = np.sort(-3.0 * rng.random((B, W)), axis=1)[:, ::-1].astype(np.float32).copy()
    sc[1, ::3] = -np.inf
    sc[2] = -np.inf
    pf, rg = np.full((B, W, 3), -1, np.int32), np.zeros((B, W, 2), np.int32)
    pf[:, :, 0] = rng.integers(0, T, (B, W))
    for step in (1, 2):
        logits = (3.0 * rng.standard_normal((B, W, V))).astype(np.float32)
        if step == 1:
            rg[:, :, 0], rg[:, :, 1] = np.searchsorted(items[:, 0], pf[:, :, 0]), np.searchsorted(items[:, 0], pf[:, :, 0] + 1)
        want = oracle_lib.beam_select(items, logits, sc, pf, step)
        got = run_select(gr, mask, logits, sc, pf, rg, step)
        assert_select_equal(got, want, f"step {step}")
        scores = to_dev(sc)
        out = {k: torch.empty_like(to_dev(v)) for k, v in got.items()}
        out["scores"] = scores
        gr.gr_beam_select(mask, to_dev(logits), scores, to_dev(pf), to_dev(rg), step, out=out)
        torch.cuda.synchronize()
        assert_select_equal({k: v.cpu().numpy() for k, v in out.items()}, want, f"step {step}, in place")
        sc, pf, rg = want["scores"], want["prefix"], want["range"]


@pytest.mark.parametrize("step", [0, 1, 2])
@pytest.mark.parametrize("where", ["scores one request further", "scores one request before", "prefix", "range"])
def test_outputs_that_lie_on_the_incoming_scores(gr, oracle_lib, step, where):  # noqa: F811
    """The incoming scores are read before any output is written, also where an output begins elsewhere in them: more requests than run at a
    time, so that first ones would be written while later ones have not been read."""
    rng = np.random.default_rng(step)
    B, W, V = 3000, 6, 64
    second = _children(rng, V, [1 + i % 5 for i in range(V)])
    items = np.array([(t1, int(t2), t3) for t1, row in enumerate(second) for t2 in row for t3 in (3, 40)], dtype=np.int32)
    mask = gr.gr_item_mask_build(to_dev(items), V)
    logits = (2.0 * rng.standard_normal((B, W, V))).astype(np.float32)
    sc = np.sort(-3.0 * rng.random((B, W)), axis=1)[:, ::-1].astype(np.float32).copy()
    pf, rg = np.full((B, W, 3), -1, np.int32), np.zeros((B, W, 2), np.int32)
    if step == 0:
        sc[:, 1:] = -np.inf
    else:
        pf[:, :, 0] = rng.integers(0, V, (B, W))
        if step == 1:
            rg[:, :, 0], rg[:, :, 1] = np.searchsorted(items[:, 0], pf[:, :, 0]), np.searchsorted(items[:, 0], pf[:, :, 0] + 1)
        else:
            pair = rng.integers(0, len(items) // 2, (B, W))
            pf[:, :, 0], pf[:, :, 1] = items[2 * pair, 0], items[2 * pair, 1]
            rg[:, :, 0], rg[:, :, 1] = 2 * pair, 2 * pair + 2
    want = oracle_lib.beam_select(items, logits, sc, pf, step)
    arena = torch.full((8 * B * W,), -7, dtype=torch.int32, device="cuda:0")
    at = {"scores one request further": W, "scores one request before": -W, "prefix": -(B * W) // 2 // W * W, "range": -W}[where]
    scores = arena[4 * B * W:5 * B * W].view(torch.float32).view(B, W)
    scores.copy_(to_dev(sc))
    i32 = lambda *shape: torch.empty(shape, dtype=torch.int32, device="cuda:0")
    out = {"parent": i32(B, W), "token": i32(B, W), "scores": torch.empty((B, W), dtype=torch.float32, device="cuda:0"), "prefix": i32(B, W, 3), "range": i32(B, W, 2),
           "item_index": i32(B, W)}
    lies = lambda *shape: arena[4 * B * W + at:4 * B * W + at + int(np.prod(shape))].view(*shape)
    if where == "prefix":
        out["prefix"] = lies(B, W, 3)
    elif where == "range":
        out["range"] = lies(B, W, 2)
    else:
        out["scores"] = lies(B, W).view(torch.float32)
    d_logits, d_pf, d_rg = to_dev(logits), to_dev(pf), to_dev(rg)
    gr.gr_beam_select(mask, d_logits, scores, d_pf, d_rg, step, out=out)
    torch.cuda.synchronize()
    assert_select_equal({k: v.cpu().numpy() for k, v in out.items()}, want, f"step {step}")


@pytest.mark.parametrize("V,W,first_tokens", [(256, 163, None), (256, 255, None), (256, 256, None), (256, 257, None), (2048, 1024, None), (2048, 1000, 900), (2049, 1024, None),
                                              (2052, 900, 880), (8192, 1024, 1023), (8192, 256, 8), (300, 16, 15), (300, 16, 16), (300, 16, 17)])
@pytest.mark.parametrize("spread", [1e-3, 3.0, 2000.0])
def test_level_0_with_about_as_many_beams_as_first_tokens(gr, oracle_lib, V, W, first_tokens, spread):  # noqa: F811
    """One live beam a request and a beam for most of its candidates, for all of them, or for more than there are: around the longest row that
    fits the list of the workgroup that selects."""
    rng = np.random.default_rng(V + W)
    B = 4
    logits = (1.25 + spread * rng.standard_normal((B, W, V))).astype(np.float32)
    logits[1, 0, ::7] = -np.inf
    sc = np.full((B, W), -np.inf, np.float32)
    sc[:, 0] = [0.0, -2.5, 7.0, -1.0]
    pf, rg = np.full((B, W, 3), -1, np.int32), np.zeros((B, W, 2), np.int32)
    items = mask = None
    if first_tokens:
        t1 = np.sort(rng.choice(V, first_tokens, replace=False))
        items = np.stack([t1, np.zeros_like(t1), np.zeros_like(t1)], axis=1).astype(np.int32)
        mask = gr.gr_item_mask_build(to_dev(items), V)
    want = oracle_lib.beam_select(items, logits, sc, pf, 0)
    assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, 0), want)


@pytest.mark.parametrize("W", [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 150, 151, 191, 192, 193])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("step_size", [0.0, 0.25])
def test_few_candidates_counted_against_each_other(gr, oracle_lib, W, masked, step_size):  # noqa: F811
    # as many candidates as a lane's share of the counting changes at, with and without scores that are equal; 600 tokens: the best of every four are as
    # many as 150 beams, and a row ends inside a load
    V, B = 602, 2
    rng = np.random.default_rng(W)
    pairs = np.stack([rng.integers(0, V, 4000), rng.integers(0, V, 4000), rng.integers(0, V, 4000)], axis=1)
    items = np.unique(pairs, axis=0).astype(np.int32)
    mask = gr.gr_item_mask_build(to_dev(items), V) if masked else None
    sc, pf, rg = gr_synth.initial_beam_state(B, W, 3)
    for step in range(3 if masked else 1):
        logits = (2.0 * rng.standard_normal((B, W, V))).astype(np.float32)
        if step_size:
            logits = (np.round(logits / step_size) * step_size).astype(np.float32)
        want = oracle_lib.beam_select(items if masked else None, logits, sc, pf, step)
        assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, step), want, f"step {step}")
        sc, pf, rg = want["scores"], want["prefix"], want["range"]


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("V", [64, 602])
def test_level_0_of_more_requests_than_workgroups(gr, oracle_lib, V, masked):  # noqa: F811
    """512 workgroups select from three requests each, one after the other, in the same LDS: every way a request can end (dead; other live rows; no
    finite logit; too many equal scores; few candidates; more than are counted against each other) is followed by every other."""
    rng = np.random.default_rng(V)
    B, W, grid = 1100, 20, 512
    logits = (2.0 * rng.standard_normal((B, W, V))).astype(np.float32)
    sc = np.full((B, W), -np.inf, np.float32)
    sc[:, 0] = -3.0 * rng.random(B)
    for b in range(B):
        kind = b % grid // 6 ** (b // grid) % 6
        if kind == 0:
            sc[b] = -np.inf
        elif kind == 1:
            sc[b, 1 + b % (W - 1)] = -1.5
        elif kind == 2:
            logits[b, 0] = -np.inf
        elif kind == 3:
            logits[b, 0] = 0.75
        elif kind == 5:                                        # fewer than W far ahead of many in one bin of the threshold, of several bins of the order
            logits[b, 0] = -100.0 + 0.4 * rng.random(V)
            logits[b, 0, rng.choice(V, W - 4, replace=False)] = 5.0 * rng.random(W - 4)
    pf, rg = np.full((B, W, 3), -1, np.int32), np.zeros((B, W, 2), np.int32)
    items = mask = None
    if masked:
        t1 = np.sort(rng.choice(V, V * 3 // 4, replace=False))
        items = np.stack([t1, t1 // 2, t1 // 3], axis=1).astype(np.int32)
        mask = gr.gr_item_mask_build(to_dev(items), V)
    want = oracle_lib.beam_select(items, logits, sc, pf, 0)
    assert_select_equal(run_select(gr, mask, logits, sc, pf, rg, 0), want)


@pytest.mark.parametrize("V,W", [(8192, 96), (8192, 544), (8192, 545), (8192, 1024), (4096, 544), (4096, 1024), (3264, 544), (3263, 544), (602, 100), (602, 101), (256, 97)])
@pytest.mark.parametrize("alike", [False, True])
def test_level_0_selects_beside_its_rows(gr, oracle_lib, V, W, alike):  # noqa: F811
    """Around the numbers of beams up to which the threshold is looked for among the best of every four logits: the workgroup's list holds what
    reaches it, also where the logits of a four are as good as equal, and the request is not left to the second kernel."""
    rng = np.random.default_rng(V + W)
    B = 3
    logits = (3.0 * rng.standard_normal((B, W, V))).astype(np.float32)
    if alike:
        logits = np.repeat(logits[:, :, ::4], 4, axis=2)[:, :, :V] + (1e-3 * rng.standard_normal((B, W, V))).astype(np.float32)
    sc, pf, rg = gr_synth.initial_beam_state(B, W, 3)
    workspace = torch.zeros(gr.select_workspace_bytes(B, W, V, 3), dtype=torch.uint8, device="cuda:0")
    r = gr.gr_beam_select(None, to_dev(logits), to_dev(sc), to_dev(pf), to_dev(rg), 0, workspace=workspace)
    torch.cuda.synchronize()
    assert_select_equal({k: v.cpu().numpy() for k, v in r.items()}, oracle_lib.beam_select(None, logits, sc, pf, 0))
    words = (4 * B * W + 255) // 256 * 64                      # (the rows' modes lie behind their biases)
    modes = workspace.view(torch.int32)[words:words + B * W].view(B, W)[:, 0].cpu() & 3
    assert (modes == 3).all()
