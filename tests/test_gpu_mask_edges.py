"""GPU: gr_item_mask_build where its passes change hands - the ends of a block of table rows (2048), first tokens that are
skipped in numbers (written lane by lane or by a whole wavefront), a table that does not start on a 16-byte boundary, and
enough blocks for their counts to be scanned by a kernel.  Every part of the blob against the definition, exactly."""
import numpy as np
import pytest
import torch

from gpu_util import to_dev
from test_gpu_select import _parse_blob, gr  # noqa: F401

pytestmark = pytest.mark.gpu


def _check_blob(m, items, V):
    first = items[:, 0]
    new_pair = np.ones(len(items), bool)
    new_pair[1:] = (items[1:, :2] != items[:-1, :2]).any(axis=1)
    start = np.flatnonzero(new_pair)
    pairs = items[start, :2]
    assert m["n_items"] == len(items) and m["n_pairs"] == len(start)
    np.testing.assert_array_equal(m["off1"], np.searchsorted(first, np.arange(V + 1), side="left"))
    np.testing.assert_array_equal(m["pair_off"], np.searchsorted(pairs[:, 0], np.arange(V + 1), side="left"))
    np.testing.assert_array_equal(m["pair_t2"], pairs[:, 1])
    np.testing.assert_array_equal(m["pair_row"], np.append(start, len(items)))
    np.testing.assert_array_equal(m["t3"], items[:, 2])
    unpack = lambda words: np.unpackbits(np.ascontiguousarray(words).view(np.uint8), bitorder="little")
    l0 = np.zeros(m["words"] * 32, np.uint8)
    l0[first] = 1
    np.testing.assert_array_equal(unpack(m["l0"]), l0)
    want = np.zeros((V, m["words"] * 32), np.uint8)
    want[pairs[:, 0], pairs[:, 1]] = 1
    np.testing.assert_array_equal(unpack(m["l1"]).reshape(V, -1), want)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("V,n,step", [(2, 1, 1), (40, 1, 40), (33, 2047, 1), (64, 2048, 1), (100, 2049, 7), (300, 4096, 60), (1000, 6145, 9),
                                      (2100, 3000, 8), (1031, 70000, 1)])
def test_blocks_gaps_and_alignment(gr, V, n, step, shift):  # noqa: F811
    rng = np.random.default_rng(V + n)
    firsts = np.arange(V - 1, -1, -step)[::-1]                   # first tokens `step` apart, the last one V - 1
    keys = np.sort(rng.choice(len(firsts) * V * V, size=n + shift, replace=False)).astype(np.int64)
    items = np.stack([firsts[keys // (V * V)], (keys // V) % V, keys % V], axis=1).astype(np.int32)
    dev = to_dev(items)[shift:]                                  # one row in: 12 bytes off a 16-byte boundary
    _check_blob(_parse_blob(gr.gr_item_mask_build(dev, V), V), items[shift:], V)


def test_counts_scanned_by_a_kernel(gr):  # noqa: F811
    V, n = 260, 8192 * 2048 + 5                                  # nearly every (t1, t2, t3) is an item
    rng = np.random.default_rng(3)
    drop = np.zeros(V ** 3, bool)
    drop[rng.choice(V ** 3, size=V ** 3 - n, replace=False)] = True
    keys = np.flatnonzero(~drop)
    items = np.stack([keys // (V * V), (keys // V) % V, keys % V], axis=1).astype(np.int32)
    _check_blob(_parse_blob(gr.gr_item_mask_build(to_dev(items), V), V), items, V)


@pytest.mark.parametrize("n", [1, 2048, 2049, 5000])
def test_bad_rows_in_any_block_are_refused(n):
    """A row that is not valid in the first, an inner or the last block of rows, or at a block's edge; the table itself is accepted, also by
    a call right after a refused one."""
    import paper_2512_11529_amd as gr
    V = 64
    flat = torch.arange(n, dtype=torch.int32, device="cuda:0") * 7
    good = torch.stack([flat // (V * V), flat // V % V, flat % V], dim=1).contiguous()
    blob = gr.gr_item_mask_build(good, V).clone()
    for row in sorted({0, min(2047, n - 1), min(2048, n - 1), n // 2, n - 1}):
        for column, value in ((0, -1), (2, V), (1, 2 ** 31 - 1)):
            bad = good.clone()
            bad[row, column] = value
            with pytest.raises(gr.GrError) as e:
                gr.gr_item_mask_build(bad, V)
            assert e.value.status == -4
        assert torch.equal(gr.gr_item_mask_build(good, V)[:96], blob[:96])


def test_large_table_whose_counts_are_scanned():
    """More blocks of rows than the second pass adds up by itself: every (t1, t2, t3) of V = 260, and the same with one row wrong."""
    import paper_2512_11529_amd as gr
    V = 260
    n = V ** 3
    flat = torch.arange(n, dtype=torch.int32, device="cuda:0")
    items = torch.stack([flat // (V * V), flat // V % V, flat % V], dim=1).contiguous()
    head = gr.gr_item_mask_build(items, V)
    off = head[:256].cpu().view(torch.int64).tolist()
    part = lambda k, count: head[off[k]:off[k] + 4 * count].view(torch.int32)
    assert off[3] == V * V
    assert torch.equal(part(8, V * V), flat[:V * V] % V)                       # pair_t2
    assert torch.equal(part(9, V * V + 1), torch.arange(V * V + 1, dtype=torch.int32, device="cuda:0") * V)      # pair_row
    assert torch.equal(part(10, n), flat % V)                                  # t3
    for row in (0, n // 2, n - 1):
        bad = items.clone()
        bad[row, 2] = V
        with pytest.raises(gr.GrError) as e:
            gr.gr_item_mask_build(bad, V)
        assert e.value.status == -4


def test_builds_from_several_threads():
    import threading
    import paper_2512_11529_amd as gr
    V = 64
    flat = torch.arange(5000, dtype=torch.int32, device="cuda:0") * 7
    good = torch.stack([flat // (V * V), flat // V % V, flat % V], dim=1).contiguous()
    bad = good.clone()
    bad[3000, 1] = -5
    torch.cuda.synchronize()
    wrong = []

    def work(refused):
        stream = torch.cuda.Stream()
        for _ in range(20):
            try:
                with torch.cuda.stream(stream):
                    gr.gr_item_mask_build(bad if refused else good, V)
                if refused:
                    wrong.append("a bad table was accepted")
            except gr.GrError as e:
                if not refused or e.status != -4:
                    wrong.append(str(e))

    threads = [threading.Thread(target=work, args=(i % 2 == 1,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
