"""A download with and without the counting launch (segments of more than
32,768 vertices of capacity, or more than 131,072 blocks, are counted first):
the same state on both sides of each line gives the same mesh in pool order,
with several chunks of slots per segment and of blocks."""
import numpy as np
import pytest
import torch

from paper_1803_03949_amd import Volume
from tests.gpu_compare import compare_all, to_dev
import oracle

pytestmark = pytest.mark.gpu


def field(dims, seed):
    """Planes through a third of the blocks, nothing in the others."""
    rng = np.random.default_rng(seed)
    c = np.stack(np.meshgrid(*[np.arange(n) for n in dims], indexing="ij"), -1).reshape(-1, 3)
    n, v = len(c), np.arange(512)
    xyz = np.stack([v % 8, v // 8 % 8, v // 64], 1) - 3.5
    nrm = rng.normal(size=(n, 3))
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    d = (nrm @ xyz.T) / 16 + rng.uniform(-0.2, 0.2, (n, 1))
    d[rng.uniform(size=n) < 0.66] = 0.7
    return c.astype(np.int32), d.astype(np.float32), np.ones((n, 512), np.float32)


# vertex segments: one per 256 blocks of capacity, at most 256
@pytest.mark.parametrize("dims,max_blocks,max_vertices", [
    ((5, 5, 5), 256, 32 * 1024), ((5, 5, 5), 256, 32 * 1024 + 1),         # one segment
    ((13, 13, 13), 4096, 16 * 32 * 1024), ((13, 13, 13), 4096, 16 * 32 * 1024 + 16),
    ((13, 13, 13), 128 * 1024, 256 * 4096), ((13, 13, 13), 128 * 1024 + 1, 256 * 4096)])
def test_both_sides_of_the_counting_rule(dims, max_blocks, max_vertices):
    print(f"[download] {dims} {max_blocks} {max_vertices}", flush=True)
    g = Volume(0.01, hash_log2=13, max_blocks=max_blocks, max_vertices=max_vertices)
    o = oracle.OracleVolume(0.01)
    for seed in (1, 2):  # the second field frees and recycles vertices
        a = field(dims, seed)
        for v, args in ((g, to_dev(*a)), (o, a)):
            v.import_blocks(*args)
            v.extract(scope_all=True)
        compare_all(g, o)
        verts, tris, keys = g.download()
        p = g.export_vertices()
        assert torch.equal(keys, p["keys"][p["ref"] > 0])
        assert len(tris) == g.status()["triangles"] > 0
    assert g.status()["error"] == 0
