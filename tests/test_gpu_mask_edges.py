"""GPU: gr_item_mask_build where its passes change hands - the ends of a block of table rows (2048), first tokens that are
skipped in numbers (written lane by lane or by a whole wavefront), a table that does not start on a 16-byte boundary, and
enough blocks for their counts to be scanned by a kernel.  Every part of the blob against the definition, exactly."""
import numpy as np
import pytest

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
