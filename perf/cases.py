"""The work that is timed on one MI355X: what a serving program has this library do, through its public calls.

`kind` of a case:
  decode   one item generated for every beam of every request: three decode steps, each the attention of all beams over the
           shared prompt and their own tokens, the item step, and the slot table's update between two steps
  attn     one attention call of a decode step (the prompt cache in bf16 or as FP8 codes)
  prefill  causal attention over a batch of packed prompts
  select   one item step at one level of the item tree (with the item mask or without)
  move     the surviving beams' own caches moved to their new places, after the first and after the second step
  mask     the item mask built from the sorted item table (when a catalogue is loaded)

Inputs are random: Q, K, V ~ N(0, 1) in bf16, logits ~ sigma * N(0, 1) in fp32, items with uniform or Zipf(1.1) first
tokens, prompts of one length or spread evenly over a range.  Prompt lengths follow from the case alone.
"""
import math
import random

import torch

import paper_2512_11529_amd as gr

STEPS = 3                                   # tokens of an item = decode steps = levels of the item tree
GEOMETRIES = ((32, 8, 128), (8, 8, 64), (8, 2, 128), (16, 4, 128), (16, 2, 128), (8, 2, 64))       # query heads, KV heads, head size


def listed():
    big = dict(Hq=32, Hkv=8, d=128)
    return [
        # the smallest call: one request of a small model; launches and latency are all there is
        dict(name="decode_tiny", kind="decode", B=1, L_min=256, L_max=256, W=16, Hq=8, Hkv=8, d=64, V=256, items=2000, zipf=False, sigma=2.0),
        # one user waits for an answer: a single request with an odd prompt length
        dict(name="decode_single", kind="decode", B=1, L_min=1531, L_max=1531, W=128, **big, V=8192, items=1_000_000, zipf=False, sigma=2.0),
        # a small batch of ordinary prompts
        dict(name="decode_small_batch", kind="decode", B=8, L_min=2048, L_max=2048, W=128, **big, V=8192, items=1_000_000, zipf=False, sigma=2.0),
        # the batch that throughput is quoted on
        dict(name="decode_batch", kind="decode", B=32, L_min=4096, L_max=4096, W=256, **big, V=8192, items=10_000_000, zipf=True, sigma=3.0),
        # many concurrent requests whose prompts differ in length by a factor of sixteen
        dict(name="decode_ragged", kind="decode", B=128, L_min=512, L_max=8192, W=256, **big, V=8192, items=10_000_000, zipf=True, sigma=3.0),
        # very long histories and wide beams, the prompt cache held in FP8
        dict(name="attn_long_fp8", kind="attn", B=4, L_min=16384, L_max=16384, W=512, **big, u=3, fp8=True),
        # prefill of short prompts of all lengths
        dict(name="prefill_short", kind="prefill", B=16, L_min=60, L_max=700, **big),
        # prefill of long prompts
        dict(name="prefill_long", kind="prefill", B=8, L_min=1024, L_max=8192, **big),
        # item step without an item table: every beam reads its whole row
        dict(name="select_free", kind="select", B=32, W=256, V=8192, items=0, zipf=False, sigma=3.0, level=2, noalloc=False),
        # item step of wide beams over a vocabulary of odd size, by a caller that allocates nothing
        dict(name="select_odd", kind="select", B=2, W=512, V=12003, items=3_000_000, zipf=True, sigma=3.0, level=1, noalloc=True),
        # the beams' own caches of the large batch follow their beams
        dict(name="move_batch", kind="move", B=32, W=256, Hkv=8, d=128),
        # a catalogue of ten million items is loaded
        dict(name="mask_build", kind="mask", V=8192, items=10_000_000, zipf=True),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, even over the logarithm."""
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _cost(case):
    w = work(case)
    return w["flops"] / 1e15 + w["bytes"] / 5e12


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= most:
            return c


def _draw(rng):
    kind = rng.choice(("decode",) * 6 + ("attn", "attn", "prefill", "prefill", "select", "select", "move", "mask"))
    Hq, Hkv, d = rng.choice((GEOMETRIES[0],) * 3 + GEOMETRIES)
    L_max = _spread(rng, 64, 16384)
    L_min = L_max if rng.random() < 0.4 else max(1, int(L_max * rng.uniform(0.05, 0.9)))
    V = rng.choice((1024, 2048, 4096, 8192, 8192, 8192, 16384)) if rng.random() < 0.6 else _spread(rng, 256, 20000)
    zipf = rng.random() < 0.5
    most_items = V * V if zipf else V ** 3 // 8     # (a Zipf table's commonest first token must not run out of items)
    items = min(_spread(rng, 2000, 12_000_000), most_items)
    sigma = rng.choice((2.0, 3.0))
    W = _spread(rng, 16, 512)
    B = _spread(rng, 1, 128)
    if kind == "decode":
        return dict(kind=kind, B=B, L_min=L_min, L_max=L_max, W=W, Hq=Hq, Hkv=Hkv, d=d, V=V, items=items, zipf=zipf, sigma=sigma)
    if kind == "attn":
        return dict(kind=kind, B=B, L_min=L_min, L_max=L_max, W=W, Hq=Hq, Hkv=Hkv, d=d, u=rng.randint(1, 3), fp8=rng.random() < 0.6)
    if kind == "prefill":
        return dict(kind=kind, B=B, L_min=L_min, L_max=L_max, Hq=Hq, Hkv=Hkv, d=d)
    if kind == "select":
        noalloc = rng.random() < 0.3 and B * W <= 12000
        return dict(kind=kind, B=B, W=W, V=V, items=items if rng.random() < 0.7 else 0, zipf=zipf, sigma=sigma, level=rng.randint(0, 2), noalloc=noalloc)
    if kind == "move":
        return dict(kind=kind, B=B, W=W, Hkv=Hkv, d=d)
    return dict(kind=kind, V=V, items=min(_spread(rng, 50_000, 12_000_000), most_items), zipf=zipf)


# ---------------------------------------------------------------------------------------------- inputs
def _lengths(c):
    if c["L_min"] == c["L_max"]:
        return [c["L_max"]] * c["B"]
    r = random.Random(c["B"] * 1_000_003 + c["L_max"] * 131 + c["L_min"])
    return [r.randint(c["L_min"], c["L_max"]) for _ in range(c["B"])]


def _cu(lens, dev):
    return torch.tensor([0] + lens, dtype=torch.int64).cumsum(0).to(torch.int32).to(dev)


def _bf16(g, *shape):
    return torch.empty(shape, dtype=torch.bfloat16, device=g.device).normal_(generator=g)


def _e4m3(g, scale, *shape):
    x = torch.empty(shape, dtype=torch.float32, device=g.device).normal_(generator=g)
    return (x / scale).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)


def _item_table(g, V, n, zipf):
    """n distinct items, sorted, int32 [n, 3]."""
    if zipf:
        p = torch.arange(1, V + 1, dtype=torch.float64, device=g.device).pow(-1.1)
        cdf = (p / p.sum()).cumsum(0)
        token_of_rank = torch.randperm(V, generator=g, device=g.device)
    keys = torch.empty(0, dtype=torch.int64, device=g.device)
    while keys.numel() < n:
        m = int((n - keys.numel()) * 1.3) + 1024
        if zipf:
            u = torch.rand(m, dtype=torch.float64, device=g.device, generator=g)
            t0 = token_of_rank[torch.searchsorted(cdf, u).clamp_(max=V - 1)]
        else:
            t0 = torch.randint(0, V, (m,), device=g.device, generator=g)
        rest = torch.randint(0, V * V, (m,), device=g.device, generator=g)
        keys = torch.unique(torch.cat([keys, t0 * (V * V) + rest]))
    if keys.numel() > n:
        keys = keys[torch.randperm(keys.numel(), device=g.device, generator=g)[:n]].sort().values
    return torch.stack([keys // (V * V), keys // V % V, keys % V], dim=1).to(torch.int32).contiguous()


def _fix_pairs(g, items, V, n_pairs):
    """The table with exactly n_pairs distinct (first, second) tokens and as many items as before: the items of surplus pairs
    are replaced by others of the remaining pairs, so that masks of tables of one case have parts of one size."""
    n = items.shape[0]
    keys = (items[:, 0].to(torch.int64) * V + items[:, 1]) * V + items[:, 2]
    pairs, of_item = torch.unique(keys // V, return_inverse=True)
    if pairs.numel() < n_pairs:
        raise ValueError("the table has too few distinct pairs")
    keep = torch.zeros(pairs.numel(), dtype=torch.bool, device=g.device)
    keep[torch.randperm(pairs.numel(), generator=g, device=g.device)[:n_pairs]] = True
    keys = keys[keep[of_item]]
    while keys.numel() < n:
        m = 2 * (n - keys.numel()) + 1024
        like = keys[torch.randint(0, keys.numel(), (m,), generator=g, device=g.device)]
        new = torch.unique(like // V * V + torch.randint(0, V, (m,), generator=g, device=g.device))
        new = new[keys[torch.searchsorted(keys, new).clamp_(max=keys.numel() - 1)] != new]
        new = new[torch.randperm(new.numel(), generator=g, device=g.device)[:n - keys.numel()]]
        keys = torch.cat([keys, new]).sort().values
    return torch.stack([keys // (V * V), keys // V % V, keys % V], dim=1).to(torch.int32).contiguous()


def _logits(g, c):
    return torch.empty((c["B"], c["W"], c["V"]), dtype=torch.float32, device=g.device).normal_(generator=g).mul_(c["sigma"])


def _first_beams(B, W, dev):
    scores = torch.full((B, W), -math.inf, dtype=torch.float32, device=dev)
    scores[:, 0] = 0.0
    return dict(scores=scores, prefix=torch.full((B, W, STEPS), -1, dtype=torch.int32, device=dev),
                range=torch.zeros((B, W, 2), dtype=torch.int32, device=dev))


def _beam_buffers(B, W, dev):
    i32 = lambda *s: torch.empty(s, dtype=torch.int32, device=dev)
    return dict(parent=i32(B, W), token=i32(B, W), scores=torch.empty((B, W), dtype=torch.float32, device=dev), prefix=i32(B, W, STEPS),
                range=i32(B, W, 2), item_index=i32(B, W))


def _bytes(n, dev):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=dev)


def _attn_state(g, c, fp8, n_q):
    dev = g.device
    lens = _lengths(c)
    B, W, Hq, Hkv, d, total = c["B"], c["W"], c["Hq"], c["Hkv"], c["d"], sum(lens)
    s = dict(max_L=max(lens), total_L=total, cu=_cu(lens, dev), scale=1.0 / math.sqrt(d))
    if fp8:
        s["k_scale"], s["v_scale"] = 0.017, 0.021
        s["k"], s["v"] = _e4m3(g, s["k_scale"], total, Hkv, d), _e4m3(g, s["v_scale"], total, Hkv, d)
    else:
        s["k"], s["v"] = _bf16(g, total, Hkv, d), _bf16(g, total, Hkv, d)
    s["k_own"], s["v_own"] = _bf16(g, B, W, STEPS, Hkv, d), _bf16(g, B, W, STEPS, Hkv, d)
    s["q"] = [_bf16(g, B, W, Hq, d) for _ in range(n_q)]
    s["out"] = [torch.empty((B, W, Hq, d), dtype=torch.bfloat16, device=dev) for _ in range(n_q)]
    s["attn_ws"] = _bytes(gr.attn_workspace_bytes(B, W, Hq, Hkv, d, s["max_L"], total), dev)
    return s


def prepare(case, seed):
    c = case
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed) * 7919 + 17)
    kind = c["kind"]
    if kind == "decode":
        s = _attn_state(g, c, False, STEPS)
        B, W, V = c["B"], c["W"], c["V"]
        s["mask"] = gr.gr_item_mask_build(_item_table(g, V, c["items"], c["zipf"]), V)
        s["logits"] = [_logits(g, c) for _ in range(STEPS)]
        s["first"] = _first_beams(B, W, dev)
        s["beams"] = [_beam_buffers(B, W, dev) for _ in range(STEPS)]
        s["slots"] = [torch.empty((B, W, STEPS), dtype=torch.int32, device=dev) for _ in range(STEPS - 1)]
        s["select_ws"] = _bytes(gr.select_workspace_bytes(B, W, V, STEPS), dev)
    elif kind == "attn":
        s = dict(_attn_state(g, c, c["fp8"], 1), u=c["u"], fp8=c["fp8"])
    elif kind == "prefill":
        lens = _lengths(c)
        total = sum(lens)
        s = dict(q=_bf16(g, total, c["Hq"], c["d"]), k=_bf16(g, total, c["Hkv"], c["d"]), v=_bf16(g, total, c["Hkv"], c["d"]), cu=_cu(lens, dev),
                 scale=1.0 / math.sqrt(c["d"]), max_L=max(lens), total_L=total,
                 out=torch.empty((total, c["Hq"], c["d"]), dtype=torch.bfloat16, device=dev))
    elif kind == "select":
        B, W, V = c["B"], c["W"], c["V"]
        mask = gr.gr_item_mask_build(_item_table(g, V, c["items"], c["zipf"]), V) if c["items"] else None
        beams = _first_beams(B, W, dev)
        for level in range(c["level"]):           # the beams that reach this level
            beams = gr.gr_beam_select(mask, _logits(g, c), beams["scores"], beams["prefix"], beams["range"], level)
        s = dict(mask=mask, first=beams, logits=_logits(g, c), level=c["level"], noalloc=c["noalloc"], beams=_beam_buffers(B, W, dev),
                 select_ws=_bytes(gr.select_workspace_bytes(B, W, V, STEPS), dev))
    elif kind == "move":
        B, W = c["B"], c["W"]
        s = dict(k_own=_bf16(g, B, W, STEPS, c["Hkv"], c["d"]), v_own=_bf16(g, B, W, STEPS, c["Hkv"], c["d"]),
                 parents=[torch.randint(0, W, (B, W), device=dev, generator=g).to(torch.int32) for _ in range(STEPS - 1)])
    else:
        V = c["V"]
        n_pairs = int(0.95 * _n_pairs(V, c["items"], c["zipf"]))
        items = _fix_pairs(g, _item_table(g, V, c["items"], c["zipf"]), V, n_pairs)
        head = gr.gr_item_mask_build(items, V)[:256].cpu().view(torch.int64).tolist()
        words = (V + 31) // 32
        # where the parts of the mask lie: bits of levels 0 and 1, row and pair offsets, pairs, third tokens
        sizes = (words, V * words, V + 1, V + 1, n_pairs, n_pairs + 1, c["items"])
        s = dict(items=items, V=V, parts=[(o, 4 * n) for o, n in zip(head[4:11], sizes)])
    return dict(s, kind=kind)


# ---------------------------------------------------------------------------------------------- one pass
def run(s):
    kind = s["kind"]
    if kind == "decode":
        beams, slot, answers = s["first"], None, []
        for step in range(STEPS):
            out, _ = gr.gr_beam_attn(s["q"][step], s["k"], s["v"], s["cu"], s["k_own"], s["v_own"], step + 1, s["scale"], s["max_L"], s["total_L"],
                                     out=s["out"][step], workspace=s["attn_ws"], slot=slot)
            beams = gr.gr_beam_select(s["mask"], s["logits"][step], beams["scores"], beams["prefix"], beams["range"], step,
                                      out=s["beams"][step], workspace=s["select_ws"])
            answers.append((out, beams))
            if step + 1 < STEPS:
                slot = gr.gr_beam_slot_update(beams["parent"], slot, step + 1, STEPS, out=s["slots"][step])
        return answers, s["slots"]
    if kind == "attn":
        if s["fp8"]:
            out, _ = gr.gr_beam_attn_fp8kv(s["q"][0], s["k"], s["v"], s["k_scale"], s["v_scale"], s["cu"], s["k_own"], s["v_own"], s["u"], s["scale"],
                                           s["max_L"], s["total_L"], out=s["out"][0], workspace=s["attn_ws"])
        else:
            out, _ = gr.gr_beam_attn(s["q"][0], s["k"], s["v"], s["cu"], s["k_own"], s["v_own"], s["u"], s["scale"], s["max_L"], s["total_L"],
                                     out=s["out"][0], workspace=s["attn_ws"])
        return out
    if kind == "prefill":
        out, _ = gr.gr_prefill_attn(s["q"], s["k"], s["v"], s["cu"], s["scale"], s["max_L"], s["total_L"], out=s["out"])
        return out
    if kind == "select":
        b = s["first"]
        if s["noalloc"]:
            return gr.gr_beam_select_noalloc(s["mask"], s["logits"], b["scores"], b["prefix"], b["range"], s["level"], s["beams"])
        return gr.gr_beam_select(s["mask"], s["logits"], b["scores"], b["prefix"], b["range"], s["level"], out=s["beams"], workspace=s["select_ws"])
    if kind == "move":
        for u, parent in enumerate(s["parents"], 1):
            gr.gr_beam_reorder(parent, s["k_own"], s["v_own"], u)
        return s["k_own"], s["v_own"]
    blob = gr.gr_item_mask_build(s["items"], s["V"])
    return [blob[o:o + n].view(torch.int32) for o, n in s["parts"]]


# ---------------------------------------------------------------------------------------------- what a pass cannot do without
def _attn_work(c, u, kv_bytes):
    total, rows = sum(_lengths(c)), c["B"] * c["W"]
    return dict(bytes=2 * kv_bytes * total * c["Hkv"] * c["d"] + 4 * rows * u * c["Hkv"] * c["d"] + 4 * rows * c["Hq"] * c["d"],
                flops=4 * c["W"] * c["Hq"] * c["d"] * (total + c["B"] * u))


def _select_bytes(c, level):
    """Logits of the live beams' valid tokens, those tokens as a list or as bits, and the beam state."""
    V = c["V"]
    live = min(c["W"], V ** level)
    if not c["items"]:
        per_row = 4 * V
    else:
        children = V if level == 0 else min(V, max(1, c["items"] / V)) if level == 1 else max(1, c["items"] / V / V)
        per_row = min(8 * children, 4 * V + V / 8)
    return c["B"] * (live * per_row + c["W"] * (6 * 4 + 10 * 4))


def _n_pairs(V, n, zipf):
    """Expected number of distinct (first, second) tokens of a table of n items."""
    if not zipf:
        return V * V * -math.expm1(-n / V / V)
    norm = sum(r ** -1.1 for r in range(1, V + 1))
    return sum(V * -math.expm1(-n * r ** -1.1 / norm / V) for r in range(1, V + 1))


def work(case):
    c, kind = case, case["kind"]
    if kind == "decode":
        parts = [_attn_work(c, step + 1, 2) for step in range(STEPS)]
        slots = 2 * 4 * c["B"] * c["W"] * (STEPS + 1 + STEPS)
        return dict(bytes=sum(p["bytes"] for p in parts) + sum(_select_bytes(c, level) for level in range(STEPS)) + slots,
                    flops=sum(p["flops"] for p in parts))
    if kind == "attn":
        return _attn_work(c, c["u"], 1 if c["fp8"] else 2)
    if kind == "prefill":
        lens = _lengths(c)
        return dict(bytes=2 * sum(lens) * c["d"] * (2 * c["Hq"] + 2 * c["Hkv"]), flops=sum(2 * c["Hq"] * c["d"] * n * (n + 1) for n in lens))
    if kind == "select":
        return dict(bytes=_select_bytes(c, c["level"]), flops=0)
    if kind == "move":
        return dict(bytes=c["B"] * c["W"] * (2 * 2 * (1 + 2) * c["Hkv"] * c["d"] * 2 + 2 * 4), flops=0)
    V, n = c["V"], c["items"]
    return dict(bytes=12 * n + V * V / 8 + V / 8 + 8 * V + 8 * 0.95 * _n_pairs(V, n, c["zipf"]) + 4 * n, flops=0)


def tolerance(case):
    """Attention against the same in 64 bits: 2.4e-3 (2-norm), 1.8e-2 (largest; short prefill rows), of which 1.7e-3 and 3.9e-3 are
    the rounding of the result to bf16.  Scores have one defined fp32 arithmetic, so beams differ for ties within its sums only."""
    kind = case["kind"]
    if kind in ("decode", "attn", "prefill"):
        return {"rel": 1e-2, "max": 7e-2, "differ": 1e-3}
    if kind == "select":
        return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
    return "exact"
