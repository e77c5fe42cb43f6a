"""Imports around the size of a counting part: new blocks take pool rows in
input order behind those already there, blocks already there keep theirs and
get the new data, the pending list names every touched block once, and of
several rows naming one block one is taken."""
import numpy as np
import pytest
import torch

from paper_1803_03949_amd import Volume
from tests.gpu_compare import to_dev

pytestmark = pytest.mark.gpu


def rows(n, seed, lo=-20):
    rng = np.random.default_rng(seed)
    cell = rng.permutation(20 ** 3)[:n]
    c = np.stack([cell % 20 + lo, cell // 20 % 20, cell // 400], 1).astype(np.int32)
    d = rng.uniform(-1, 1, (n, 512)).astype(np.float32)
    return c, d, rng.integers(0, 2, (n, 512)).astype(np.float32)


@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 1023, 2049])
def test_rows_append_in_order_across_parts(n):
    print(f"[import] {n}", flush=True)
    g = Volume(0.01, hash_log2=14, max_blocks=1 << 12, max_vertices=1 << 16)
    c, d, w = rows(n, n)
    first = c[::3], d[::3], w[::3]
    g.import_blocks(*to_dev(*first))
    g.extract(scope_all=True)  # the next import is another extraction's
    assert len(g.block_list("pending")) == 0
    d2 = (d + 1).astype(np.float32)
    g.import_blocks(*to_dev(c, d2, w))
    want = [tuple(x) for x in c[::3].tolist()]
    want += [t for t in map(tuple, c.tolist()) if t not in set(want)]
    b = g.export_blocks()
    assert [tuple(x) for x in b["coords"].tolist()] == want
    at = g.lookup(to_dev(c)[0]).long()
    assert torch.equal(b["d"][at], to_dev(d2)[0]) and torch.equal(b["w"][at], to_dev(w)[0])
    for which in ("frame", "pending"):
        assert [tuple(x) for x in g.block_list(which).tolist()] == [tuple(x) for x in c.tolist()]
    assert g.status()["error"] == 0


def test_one_of_several_rows_naming_a_block_is_taken():
    g = Volume(0.01, hash_log2=14, max_blocks=1 << 12, max_vertices=1 << 16)
    c, d, w = rows(300, 7)
    pick = np.concatenate([np.arange(300), np.arange(0, 300, 2), np.arange(0, 300, 5)])
    rng = np.random.default_rng(8)
    d3 = rng.uniform(-1, 1, (len(pick), 512)).astype(np.float32)
    g.import_blocks(*to_dev(c[pick], d3, w[pick]))
    b = g.export_blocks()
    assert len(b["coords"]) == 300 and len(g.block_list("pending")) == 300
    got = b["d"].cpu().numpy()
    named = {}
    for i, k in enumerate(pick):
        named.setdefault(tuple(c[k].tolist()), []).append(i)
    for i, t in enumerate(map(tuple, b["coords"].tolist())):
        assert any(np.array_equal(got[i], d3[j]) for j in named[t])
