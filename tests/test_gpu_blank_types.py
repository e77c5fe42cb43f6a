"""Blocks whose previous types are all 0 and not written (new ones, free space,
ones whose surface came and went): exported types, vertices and triangles
against the oracle through imports, extractions, refinements and a reset, with
one block per wave and with many (the vertex pass then asks for triangle counts
before types)."""
import numpy as np
import pytest

import oracle
from paper_1803_03949_amd import Volume
from tests.gpu_compare import compare_all, to_dev

pytestmark = pytest.mark.gpu

S = 0.01


def blocks(dims, seed, empty):
    """A plane through a few blocks of a dims^3 box, the others (a share of
    `empty`) positive, negative or unobserved throughout."""
    rng = np.random.default_rng(seed)
    n = dims ** 3
    cell = np.arange(n)
    c = np.stack([cell % dims, cell // dims % dims, cell // dims ** 2], 1).astype(np.int32)
    v = np.arange(512)
    xyz = np.stack([v % 8, v // 8 % 8, v // 64], 1) - 3.5
    nrm = rng.normal(size=(n, 3))
    nrm /= np.linalg.norm(nrm, axis=1, keepdims=True)
    d = (nrm @ xyz.T) / 16 + rng.uniform(-0.2, 0.2, (n, 1))
    kind = rng.uniform(size=n)
    d[kind < empty] = 0.7
    d[kind < empty * 0.3] = -0.7
    w = np.ones((n, 512))
    w[kind > 1 - 0.1 * empty] = 0
    return c, d.astype(np.float32), w.astype(np.float32)


@pytest.mark.parametrize("dims, launch", [(1, None), (5, None), (13, dict(wave_group_size=2, wave_groups_per_cu=1))])
def test_types_of_blank_blocks(dims, launch):
    cap = 1 << 12
    g = Volume(S, hash_log2=14, max_blocks=cap, max_vertices=1 << 21)
    if launch:
        g.set_launch(**launch)
        groups = 256 * launch["wave_groups_per_cu"]
        assert dims ** 3 > 4 * groups * launch["wave_group_size"]
    o = oracle.OracleVolume(S, 4.0, 0.5)

    def take(seed, empty, keep=slice(None)):
        a = [x[keep] for x in blocks(dims, seed, empty)]
        g.import_blocks(*to_dev(*a))
        o.import_blocks(*a)

    def step(name, f):
        print(f"[blank] {dims} {name}", flush=True)
        f(g), f(o)
        return compare_all(g, o)

    take(1, 0.8)
    step("new", lambda v: None)
    step("refined before any extraction", lambda v: v.refine())
    info = step("extracted", lambda v: v.extract())
    assert dims == 1 or info["nv"] > 100
    step("refined", lambda v: v.refine())
    take(2, 0.95, slice(0, None, 2))
    step("new data", lambda v: None)
    step("refined before the extraction", lambda v: v.refine())
    step("extracted again", lambda v: v.extract())
    step("refined again", lambda v: v.refine())
    take(3, 1.0)
    step("all empty", lambda v: v.extract(scope_all=True))
    take(4, 0.5, slice(0, None, 3))
    step("refining extraction", lambda v: v.extract(refine=True))
    step("refined after it", lambda v: v.refine())
    g.reset()
    o = oracle.OracleVolume(S, 4.0, 0.5)
    take(5, 0.8, slice(1, None, 2))
    step("after a reset", lambda v: v.refine())
    step("extracted after a reset", lambda v: v.extract())
    step("refined after a reset", lambda v: v.refine())
    assert g.status()["error"] == 0
