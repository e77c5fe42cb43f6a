"""Imports inside a captured HIP graph that holds no reset: every replay
imports its rows again, whether the blocks were new to the volume at the first
replay or present before the capture, with the program's own work on the
volume between the replays."""
import numpy as np
import pytest
import torch

from paper_1803_03949_amd import Volume
from paper_1803_03949_amd.batch import canonical_vertices
from tests.gpu_compare import to_dev

pytestmark = pytest.mark.gpu


def field(seed, n):
    rng = np.random.default_rng(seed)
    return rng.uniform(-1, 1, (n, 512)).astype(np.float32)


def eager(coords, d, w):
    g = Volume(0.01, hash_log2=12, max_blocks=1024, max_vertices=1 << 20)
    g.import_blocks(*to_dev(coords, d, w))
    g.extract(scope_all=True)
    return canonical_vertices(*g.positions()), g.export_blocks()


@pytest.mark.parametrize("dims", [(1, 1, 1), (3, 2, 2), (7, 7, 6)])  # one part of rows and more
@pytest.mark.parametrize("present", [False, True])
def test_every_replay_imports(dims, present):
    print(f"[import replay] {dims} present {present}", flush=True)
    coords = np.stack(np.meshgrid(*[np.arange(n) for n in dims], indexing="ij"), -1)
    coords = coords.reshape(-1, 3).astype(np.int32)
    n = len(coords)
    g = Volume(0.01, hash_log2=12, max_blocks=1024, max_vertices=1 << 20)
    c, d, w = to_dev(coords, field(0, n), np.ones((n, 512), np.float32))
    rows = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    if present:
        g.import_blocks(c, d, w)
        g.extract(scope_all=True)
    pos, slot = g.positions()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.import_batch(None, c, d, w, rows)
        g.extract(scope_all=True)
        g.positions(pos, slot)
    for seed in (1, 2, 3):
        new = field(seed, n)
        d.copy_(torch.from_numpy(new))
        rows.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        want, blocks = eager(coords, new, np.ones((n, 512), np.float32))
        assert g.status()["error"] == 0
        assert np.array_equal(rows.cpu().numpy(), np.arange(n)), seed
        got = g.export_blocks()
        for k in ("d", "w", "cur"):
            assert torch.equal(got[k], blocks[k]), (seed, k)
        assert np.array_equal(canonical_vertices(pos, slot), want), seed
