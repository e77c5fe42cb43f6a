"""vm_reset_volume clears everything a new mesh reads, in one launch, at the
smallest and at ragged capacities: after a reset the volume is empty, keeps
its running totals, and meshes another scene as a fresh volume does."""
import numpy as np
import pytest

import scenes
from paper_1803_03949_amd import Volume
from tests.gpu_compare import gpu_blocks_sorted, gpu_live_vertices, gpu_triangle_keys, to_dev

pytestmark = pytest.mark.gpu


def mesh(vol, dims, seed):
    sv = scenes.sphere_volume(seed=seed, dims_blocks=dims, voxel_m=0.01,
                              radius=0.3 * 0.08 * min(dims) + 0.01,
                              center=0.04 * np.asarray(dims), jitter=0.004)
    vol.import_blocks(*to_dev(*sv.blocks()))
    vol.extract(scope_all=True)
    vol.extract()
    b = gpu_blocks_sorted(vol)
    return [b[k] for k in ("coords", "d", "w", "prev", "cur")] + list(gpu_live_vertices(vol)) + \
        [gpu_triangle_keys(vol)[0]]


@pytest.mark.parametrize("hash_log2,max_blocks,max_vertices", [
    (10, 1, 2048), (10, 3, 4096), (11, 65, 1 << 14), (13, 1023, 1 << 17)])
def test_reset_equals_a_fresh_volume(hash_log2, max_blocks, max_vertices):
    print(f"[reset] {hash_log2} {max_blocks} {max_vertices}", flush=True)
    kw = dict(hash_log2=hash_log2, max_blocks=max_blocks, max_vertices=max_vertices)
    big = (1, 1, max_blocks) if max_blocks < 65 else (4, 4, 4)
    vol = Volume(0.01, **kw)
    mesh(vol, big, 3)
    before = vol.totals()
    vol.reset()
    assert vol.totals() == before
    st = vol.status()
    for k in ("error", "blocks", "pending_blocks", "vertex_slots", "free_vertex_slots",
              "triangles", "tri_cubes", "max_segment_live"):
        assert st[k] == 0, k
    verts, tris, _ = vol.download()
    assert len(verts) == 0 and len(tris) == 0
    got = mesh(vol, (1, 1, 1), 4)
    want = mesh(Volume(0.01, **kw), (1, 1, 1), 4)
    for a, b in zip(got, want):
        assert a.shape == b.shape and np.array_equal(a, b)
