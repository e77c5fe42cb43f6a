"""Blocks whose import into bound storage was refused (their rows would not land
on their own pool rows): the error stands, and every later call finds them as
blocks that nothing was observed in, whatever the workspace held before."""
import ctypes

import numpy as np
import pytest
import torch

import scenes
from paper_1803_03949_amd import Volume, VmError, binding
from tests.gpu_compare import gpu_live_vertices, to_dev

pytestmark = pytest.mark.gpu

S = 0.008
RANGE = -8  # VM_ERR_RANGE


def download(g):
    cap, tcap = g.cfg.max_vertices, 5 * 512 * g.cfg.max_blocks
    verts = torch.empty((cap, 3), device="cuda")
    keys = torch.empty(cap, dtype=torch.int64, device="cuda")
    tris = torch.empty((tcap, 3), dtype=torch.int32, device="cuda")
    nv, nt = ctypes.c_int64(), ctypes.c_int64()
    r = binding.lib().vm_download_mesh(g.h, verts.data_ptr(), keys.data_ptr(), tris.data_ptr(), cap,
                                       tcap, ctypes.byref(nv), ctypes.byref(nt), binding._stream())
    return r, verts[:nv.value], keys[:nv.value], tris[:nt.value]


@pytest.mark.parametrize("scope_all", [False, True])
@pytest.mark.parametrize("refine", [False, True])
def test_refused_blocks_are_empty(scope_all, refine):
    v = scenes.sphere_volume(seed=1, dims_blocks=(5, 4, 4), voxel_m=S, radius=0.1,
                             center=np.array([0.16, 0.128, 0.128]))
    c, d, w = v.blocks()
    n, half = len(c), len(c) // 2
    kw = dict(hash_log2=12, max_blocks=n, max_vertices=1 << 16)
    f = Volume(S, **kw)
    f.import_blocks(*to_dev(c[:half], d[:half], w[:half]))
    g = Volume(S, **kw)
    td, tw = to_dev(d, w)
    g.bind_tsdf(td, tw)
    # what an earlier use left in the workspace: every block meshed, with dense
    # signs, before the reset
    td.copy_(torch.rand_like(td) - 0.5)
    g.import_blocks(to_dev(c)[0], td, tw)
    g.extract(scope_all=True)
    td.copy_(to_dev(d)[0])
    g.reset()
    g.import_blocks(to_dev(c[:half])[0], td, tw)
    g.import_blocks(to_dev(c[half:])[0], td, tw)
    for _ in range(2):
        for x in (f, g):
            x.extract(scope_all=scope_all, refine=refine)
            x.refine()
        r, verts, keys, tris = download(g)
        st = g.status(check=False)
        assert r == RANGE and st["error"] == RANGE and st["blocks"] == n
        assert st["triangles"] == f.status()["triangles"] == len(tris) > 0
        for a, b in zip(gpu_live_vertices(g), gpu_live_vertices(f)):
            assert np.array_equal(a, b)
        assert int(tris.min()) == 0 and int(tris.max()) == len(verts) - 1
        b = g.export_blocks()
        assert bool((b["cur"][half:] == 0).all()) and bool((b["prev"][half:] == 0).all())
        grad = g.extract_backward_rows(verts, torch.arange(half, n, dtype=torch.int32, device="cuda"))
        assert bool((grad == 0).all())
    with pytest.raises(VmError):
        g.download()
    g.reset()
    g.import_blocks(to_dev(c)[0], td, tw)
    g.extract()
    assert len(g.download()[0]) > len(keys)
