"""Block collection (Eq. 1) where a tile's blocks leave the usual window: an
unrelated depth at every pixel (more distinct blocks than a workgroup's table
holds), truncations whose boxes are wider than a window, depth steps inside
tiles, and images smaller than a tile or not a multiple of one."""
import numpy as np
import pytest

import oracle
import scenes
from paper_1803_03949_amd import Volume
from tests.gpu_compare import compare_all, to_dev

pytestmark = pytest.mark.gpu


def depth_image(kind, W, H):
    rng = np.random.default_rng(11)
    if kind == "noise":
        return rng.uniform(0.4, 3.0, (H, W)).astype(np.float32)
    steps = np.where((np.arange(W)[None, :] // 5 + np.arange(H)[:, None] // 7) % 2, 0.9, 2.3)
    return (steps + rng.normal(0, 0.002, (H, W))).astype(np.float32)


@pytest.mark.parametrize("kind,trunc,W,H,voxel", [
    ("noise", 4.0, 96, 64, 0.01), ("noise", 20.0, 33, 17, 0.02), ("steps", 4.0, 161, 47, 0.01),
    ("steps", 9.0, 64, 33, 0.02), ("noise", 4.0, 1, 1, 0.02), ("steps", 1.0, 31, 15, 0.03)])
def test_collected_blocks_match_oracle(kind, trunc, W, H, voxel):
    print(f"[collect] {kind} {trunc} {W}x{H}", flush=True)
    g = Volume(voxel, trunc_vox=trunc, hash_log2=17, max_blocks=1 << 15, max_vertices=1 << 21)
    o = oracle.OracleVolume(voxel, trunc)
    K = (525.0 * W / 640, 525.0 * W / 640, (W - 1) / 2, (H - 1) / 2) if W > 8 else (400.0, 400.0, 0.0, 0.0)
    pose = scenes.look_at((2.0, 2.0, 1.5), (3.0, 2.4, 1.2)).astype(np.float32)
    for k in range(2):  # the second frame finds its blocks in the hash
        depth = depth_image(kind, W, H)
        g.integrate(to_dev(depth)[0], K, pose, 0.4, 3.0)
        o.integrate(depth, K, pose, 0.4, 3.0)
        assert {tuple(x) for x in g.block_list("frame").tolist()} == \
            {tuple(x) for x in o.block_set("frame").tolist()}
        assert len(g.block_list("frame")) == len(o.block_set("frame"))
        g.extract()
        o.extract()
        compare_all(g, o)


@pytest.mark.parametrize("kind,trunc,W,H,voxel", [
    ("steps", 4.0, 512, 257, 0.02), ("steps", 9.0, 641, 239, 0.03), ("noise", 4.0, 520, 273, 0.04),
    ("steps", 4.0, 512, 256, 0.02), ("noise", 20.0, 545, 271, 0.06)])
def test_images_of_more_tiles_than_compute_units(kind, trunc, W, H, voxel):
    """Around the 256 tiles from which a lane takes two pixels."""
    test_collected_blocks_match_oracle(kind, trunc, W, H, voxel)
