"""vm_download_mesh at the edges of its work split: blocks with more triangles
than a wave lists at once (random signs), more blocks than a counting chunk,
more vertices than a chunk of slots, recycled slots between live ones, buffers
that are too small, and rows left from a larger mesh before a reset."""
import numpy as np
import pytest
import torch

import oracle
from paper_1803_03949_amd import Volume, VmError, binding
from tests.gpu_compare import compare_all, to_dev

pytestmark = pytest.mark.gpu


def noise(dims, seed):
    rng = np.random.default_rng(seed)
    c = np.stack(np.meshgrid(*[np.arange(n) for n in dims], indexing="ij"), -1).reshape(-1, 3)
    d = rng.uniform(-1, 1, (len(c), 512)).astype(np.float32)
    return c.astype(np.int32), d, np.ones_like(d)


def pool_order(vol):
    """Keys of the live pool entries in pool order."""
    p = vol.export_vertices()
    return p["keys"][p["ref"] > 0]


# capacities of one pool segment and of several
@pytest.mark.parametrize("dims,max_blocks,max_vertices", [
    ((1, 1, 1), 8, 4096), ((3, 2, 3), 300, 1 << 16), ((7, 6, 7), 1024, 1 << 20)])
def test_dense_signs_match_oracle_in_pool_order(dims, max_blocks, max_vertices):
    print(f"[download] {dims}", flush=True)
    g = Volume(0.01, hash_log2=12, max_blocks=max_blocks, max_vertices=max_vertices)
    o = oracle.OracleVolume(0.01)
    for seed in (1, 2):  # the second field frees and recycles most vertices
        a = noise(dims, seed)
        for v, args in ((g, to_dev(*a)), (o, a)):
            v.import_blocks(*args)
            v.extract(scope_all=True)
            v.gc()
        compare_all(g, o)
        verts, tris, keys = g.download()
        assert torch.equal(keys, pool_order(g))
        assert len(tris) == g.status()["triangles"] > 600 * len(a[0])
    # a call with too little room fills what fits and says so
    L, s = binding.lib(), binding._stream()
    import ctypes
    nv, nt = ctypes.c_int64(), ctypes.c_int64()
    v2 = torch.full((len(verts), 3), -1.0, device="cuda")
    t2 = torch.full((len(tris), 3), -7, dtype=torch.int32, device="cuda")
    m, n = len(verts) // 2, len(tris) // 3
    assert L.vm_download_mesh(g.h, v2.data_ptr(), None, t2.data_ptr(), m, n, ctypes.byref(nv),
                              ctypes.byref(nt), s) == -6
    assert (nv.value, nt.value) == (len(verts), len(tris))
    assert torch.equal(v2[:m], verts[:m]) and bool((v2[m:] == -1).all())
    assert torch.equal(t2[:n], tris[:n]) and bool((t2[n:] == -7).all())


def test_rows_of_a_mesh_before_a_reset_are_forgotten():
    """A vertex created after the last download has no row, whatever the slot
    held before: its upstream gradient is ignored."""
    g = Volume(0.01, hash_log2=12, max_blocks=64, max_vertices=1 << 16)
    big, small = to_dev(*noise((3, 3, 3), 3)), to_dev(*noise((1, 1, 1), 4))
    g.import_blocks(*big)
    g.extract(scope_all=True)
    n_big = len(g.download()[0])
    g.reset()
    g.import_blocks(*small)
    g.extract(scope_all=True)
    verts, _, keys = g.download()
    assert 0 < len(verts) < n_big
    want = g.extract_backward(torch.ones_like(verts))
    c, d, w = noise((1, 1, 2), 4)
    # a second block, meshed but not downloaded: the first one's gradient
    # comes from the downloaded vertices that are still there
    g.import_blocks(*to_dev(c[1:], d[1:], w[1:]))
    g.extract(scope_all=True)
    got = g.extract_backward(torch.ones_like(verts))
    fresh = g.lookup(to_dev(c[1:])[0])
    # edges owned by the new block have no row
    inner = got[fresh.long()].reshape(8, 8, 8)[1:, 1:, 1:]
    assert bool((inner == 0).all())
    assert bool((want != 0).any())


def test_sizes_follow_the_mesh_from_call_to_call():
    """The buffers of one download are sized by the one before: a larger, a
    smaller and an empty mesh after each other come back whole."""
    g = Volume(0.01, hash_log2=12, max_blocks=256, max_vertices=1 << 18)
    for dims in ((1, 1, 1), (4, 4, 4), (2, 1, 1), None, (3, 3, 3)):
        g.reset()
        if dims:
            g.import_blocks(*to_dev(*noise(dims, 5)))
        g.extract(scope_all=True)
        verts, tris, keys = g.download()
        st = g.status()
        assert len(verts) == len(keys) == st["vertex_slots"] - st["free_vertex_slots"]
        assert len(tris) == st["triangles"]
        assert torch.equal(keys, pool_order(g))
        if dims:
            assert int(tris.min()) >= 0 and int(tris.max()) == len(verts) - 1


@pytest.mark.parametrize("rows", [[0], [5, -1, 2], list(range(8))])
def test_backward_rows_equals_the_whole_backward(rows):
    g = Volume(0.01, hash_log2=12, max_blocks=64, max_vertices=1 << 16)
    g.import_blocks(*to_dev(*noise((2, 2, 2), 6)))
    g.extract(scope_all=True)
    verts, _, _ = g.download()
    dL = torch.rand(verts.shape, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    want = g.extract_backward(dL)
    r = torch.tensor(rows, dtype=torch.int32, device="cuda")
    got = g.extract_backward_rows(dL, r)
    for i, k in enumerate(rows):
        assert torch.equal(got[i], want[k] if k >= 0 else torch.zeros_like(want[0]))
    g.extract()
    assert g.extract_backward_rows(dL, r) is None


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 3, 2)])
def test_backward_of_dense_signs_matches_oracle(dims, shift):
    """Blocks with more vertices than the backward lists at once, into an
    output aligned to 16 bytes and to 4."""
    g = Volume(0.01, hash_log2=12, max_blocks=64, max_vertices=1 << 16)
    o = oracle.OracleVolume(0.01)
    a = noise(dims, 8)
    g.import_blocks(*to_dev(*a))
    g.extract(scope_all=True)
    o.import_blocks(*a)
    o.extract(scope_all=True)
    verts, _, _ = g.download()
    buf = torch.full((512 * len(a[0]) + 4,), 7.0, device="cuda")
    out = buf[shift:shift + 512 * len(a[0])].view(-1, 512)
    got = g.extract_backward(verts, out)  # dL/dp = p
    want = o.grad_tsdf64(o.positions64())
    rows = {tuple(c): i for i, c in enumerate(g.export_blocks()["coords"].tolist())}
    got = got.cpu().numpy()[[rows[tuple(c)] for c in o.blocks()["coords"].tolist()]]
    # |p| dt/dd with dt/dd up to 1/(da - db)^2: relative to each voxel's own sum
    assert np.all(np.abs(got - want) <= 1e-4 * np.abs(want) + 1e-4 * np.abs(want).max())
    assert bool((buf[:shift] == 7).all()) and bool((buf[shift + 512 * len(a[0]):] == 7).all())
