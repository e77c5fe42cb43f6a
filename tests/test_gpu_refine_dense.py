"""Refinement where a block lists many cubes (dense sign fields with most
corners near zero, up to all 512 cubes), few or none, as a pass and within the
extraction, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1803_03949_amd import Volume
from tests.gpu_compare import compare_all, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flip, near", [(0.5, 0.9), (0.5, 1.0), (0.03, 0.7), (0.002, 1.0), (0.5, 0.0)])
@pytest.mark.parametrize("inside", [False, True])
def test_dense_fields_refine_like_the_oracle(flip, near, inside):
    print(f"[refine] {flip} {near} {inside}", flush=True)
    g = Volume(0.01, hash_log2=14, max_blocks=1 << 10, max_vertices=1 << 18)
    o = oracle.OracleVolume(0.01, 4.0, 0.5)
    rng = np.random.default_rng(5)
    c = np.stack(np.meshgrid(*[np.arange(3)] * 3, indexing="ij"), -1).reshape(-1, 3).astype(np.int32)
    v = np.arange(512)
    wall = (c[:, :1] * 8 + v % 8 - 11.5) > 0  # a plane: regular types under the noise
    for k in range(3):
        sign = np.where(wall ^ (rng.uniform(size=(27, 512)) < flip), 1.0, -1.0)
        size = np.where(rng.uniform(size=(27, 512)) < near, rng.uniform(0.01, 0.49, (27, 512)),
                        rng.uniform(0.51, 0.9, (27, 512)))
        d, w = (sign * size).astype(np.float32), np.ones((27, 512), np.float32)
        g.import_blocks(*to_dev(c, d, w))
        o.import_blocks(c, d, w)
        g.extract(refine=inside)
        o.extract(refine=inside)
        compare_all(g, o)
        g.refine()
        o.refine()
        compare_all(g, o)
    assert g.status()["error"] == 0
    assert near == 0.0 or g.totals()["refined_cubes"] > 0
