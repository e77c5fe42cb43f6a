"""The backward of a differentiable extraction reads its volume as the forward
left it: calls that leave the mesh as it was may come in between, after any
that may change it the backward raises instead of reading another mesh's rows.
And a download's gradients are as many as its rows."""
import numpy as np
import pytest
import torch

import scenes
from paper_1803_03949_amd import Volume, binding
from paper_1803_03949_amd.autograd import FusedMesh, TSDFMesh
from tests.gpu_compare import to_dev

pytestmark = pytest.mark.gpu

S = 0.01


def sphere(radius):
    sv = scenes.sphere_volume(seed=11, dims_blocks=(2, 2, 2), voxel_m=S, radius=radius,
                              center=np.full(3, 0.08), jitter=0.005)
    c = sv.meta["center"]
    pose = scenes.look_at(c + np.array([0.02, -0.30, 0.12]), c).astype(np.float32)
    sc = scenes.Scene([(c, radius)], [], None)
    depth = sc.render(pose.astype(np.float64), scenes.pixel_rays(), None, 0.1, 5.0)
    return (*to_dev(*sv.blocks()), to_dev(depth)[0], pose)


def volume():
    return Volume(S, hash_log2=12, max_blocks=1024, max_vertices=1 << 16)


def forward(kind, vol, case):
    """(leaf tensor, vertices)"""
    coords, tsdf, weight, depth, pose = case
    if kind == "tsdf":
        x = tsdf.clone().requires_grad_(True)
        return x, TSDFMesh.apply(x, weight, coords, vol)[0]
    x = tsdf.clone().requires_grad_(True)
    return x, FusedMesh.apply(depth, x, weight, coords, vol, scenes.K, pose, 0.1, 5.0)[0]


def keep(vol, case):
    vol.gc()
    vol.status()
    vol.download()
    vol.download_normals()
    vol.export_blocks()
    vol.bind_tsdf(None, None)  # as it is


def extract_again(vol, case):
    vol.extract()
    vol.extract(scope_all=True)


def extract_and_download_again(vol, case):
    vol.extract(scope_all=True)
    vol.extract()
    vol.download()


def import_again(vol, case):
    vol.import_blocks(case[0], case[1] * 0.5, case[2])


def import_extract_download(vol, case):
    import_again(vol, case)
    vol.extract()
    vol.download()


def integrate(vol, case):
    vol.integrate(case[3], scenes.K, case[4], 0.1, 5.0)


def refine(vol, case):
    vol.refine()


def refining_extraction(vol, case):
    vol.extract(refine=True)


def reset(vol, case):
    vol.reset()


def bind(vol, case):
    B = vol.cfg.max_blocks
    vol.bind_tsdf(torch.zeros((B, 512), device="cuda"), torch.zeros((B, 512), device="cuda"))


@pytest.mark.parametrize("kind", ["tsdf", "fused"])
@pytest.mark.parametrize("between", [keep, extract_again, extract_and_download_again])
def test_calls_that_leave_the_mesh(kind, between):
    case = sphere(0.05)
    grads = []
    for f in (lambda vol, case: None, between):
        vol = volume()
        x, verts = forward(kind, vol, case)
        f(vol, case)
        (verts * verts).sum().backward()
        assert bool((x.grad != 0).any())
        grads.append(x.grad)
    # each voxel's gradient is a sum in a fixed order of its own vertices'
    assert torch.equal(*grads)


@pytest.mark.parametrize("kind", ["tsdf", "fused"])
@pytest.mark.parametrize("between", [import_again, import_extract_download, integrate, refine,
                                     refining_extraction, reset, bind])
def test_calls_that_change_the_mesh(kind, between):
    case = sphere(0.05)
    vol = volume()
    x, verts = forward(kind, vol, case)
    between(vol, case)
    with pytest.raises(RuntimeError, match="another mesh"):
        verts.sum().backward()
    assert x.grad is None
    # and the volume serves the next forward
    x, verts = forward(kind, volume() if between is bind else vol, case)
    verts.sum().backward()
    assert bool((x.grad != 0).any())


@pytest.mark.parametrize("kind", ["tsdf", "fused"])
@pytest.mark.parametrize("r1,r2", [(0.03, 0.06), (0.06, 0.03), (0.05, 0.05)])
def test_two_forwards_on_one_volume(kind, r1, r2):
    vol = volume()
    a, va = forward(kind, vol, sphere(r1))
    b, vb = forward(kind, vol, sphere(r2))
    (vb * vb).sum().backward()
    want, vw = forward(kind, volume(), sphere(r2))
    (vw * vw).sum().backward()
    assert torch.equal(b.grad, want.grad)
    with pytest.raises(RuntimeError, match="another mesh"):
        (va * va).sum().backward()


def test_gradients_are_as_many_as_rows():
    vol = volume()
    coords, tsdf, weight, _, _ = sphere(0.05)
    assert vol.mesh_state()[1:] == (0, 0)
    vol.import_blocks(coords, tsdf, weight)
    vol.extract(scope_all=True)
    verts, _, _ = vol.download()
    cur, dl, n = vol.mesh_state()
    assert cur == dl > 0 and n == len(verts) > 10
    rows = torch.arange(8, dtype=torch.int32, device="cuda")
    for call in (vol.extract_backward, lambda g: vol.extract_backward_rows(g, rows)):
        for short in (verts[:-1], verts[:0]):
            with pytest.raises(ValueError, match=f"{n} vertices"):
                call(short)
        assert torch.equal(call(verts), call(torch.cat([verts, verts])))
    vol.extract(refine=True)  # another mesh; the rows are still the download's
    assert vol.mesh_state() == (cur + 1, dl, n)
    with pytest.raises(ValueError):
        vol.extract_backward(verts[:-1])
    vol.reset()
    assert vol.mesh_state()[1:] == (0, 0)


def test_no_gradients_for_a_mesh_is_an_argument_error():
    vol = volume()
    coords, tsdf, weight, _, _ = sphere(0.05)
    vol.import_blocks(coords, tsdf, weight)
    out = torch.zeros((8, 512), device="cuda")
    rows = torch.arange(8, dtype=torch.int32, device="cuda")
    L, s = binding.lib(), binding._stream()
    assert L.vm_extract_backward(vol.h, None, out.data_ptr(), s) == 0  # no row to read yet
    vol.extract(scope_all=True)
    assert len(vol.download()[0]) > 0
    assert L.vm_extract_backward(vol.h, None, out.data_ptr(), s) == binding.VM_ERR_ARG
    assert L.vm_extract_backward_rows(vol.h, None, rows.data_ptr(), 8, out.data_ptr(),
                                      s) == binding.VM_ERR_ARG
