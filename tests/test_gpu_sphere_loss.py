"""The batched loss gradient's kernel against the same operations in torch
(FP64 and FP32), over sizes around a workgroup, slots outside the table, and
the tensors it leaves to torch."""
import pytest
import torch

from paper_1803_03949_amd.batch import sphere_loss_grad
from paper_1803_03949_amd.binding import sphere_loss_grad_kernel

pytestmark = pytest.mark.gpu


def inputs(n, m, seed=1):
    g = torch.Generator().manual_seed(seed)
    pos = torch.rand((n, 3), generator=g) * 2
    slot = torch.randint(-1, m, (n,), generator=g, dtype=torch.int32)
    if n > 3:
        slot[1], slot[2] = 2 * m + 3, -m - 3
    pos[slot == -1] = 0
    return pos, slot, torch.rand((m, 3), generator=g), torch.rand(m, generator=g) + 0.1


def reference(pos, slot, centers, radii):
    c = torch.cat([centers, torch.zeros(1, 3)]).double()
    r = torch.cat([radii, torch.zeros(1)]).double()
    k = slot.long().remainder(len(r))
    d = pos.double() - c[k]
    dist = d.norm(dim=1).clamp_min(1e-30)
    return d * ((dist - r[k]) / dist * 2)[:, None]


@pytest.mark.parametrize("n,m", [(0, 2), (1, 1), (255, 3), (257, 64), (70001, 5)])
def test_kernel_matches_fp64(n, m):
    pos, slot, centers, radii = inputs(n, m)
    fn = sphere_loss_grad(centers.cuda(), radii.cuda())
    out = torch.full((n, 3), 7.0, device="cuda")
    got = fn(pos.cuda(), slot.cuda(), out)
    assert got is out
    want = reference(pos, slot, centers, radii)
    # d, its length and the scale carry a few roundings of 2^-24, the
    # difference to the radius up to |d| + r of them
    assert torch.all((out.cpu().double() - want).abs() <= 16 * 2.0 ** -24 * 4)
    assert torch.all(out.cpu()[slot == -1] == 0)
    # in place, and through torch (a strided output is not the kernel's)
    p = pos.cuda()
    assert torch.equal(fn(p, slot.cuda(), p), out)
    wide = torch.zeros((n, 4), device="cuda")[:, :3]
    fn(pos.cuda(), slot.cuda(), wide)
    assert torch.equal(wide, out)


def test_what_the_kernel_leaves_to_torch():
    pos, slot, centers, radii = (t.cuda() for t in inputs(100, 4))
    out = torch.empty_like(pos)
    buf = torch.zeros(400, device="cuda")
    for p, s, o in ((pos.double(), slot, out.double()), (pos, slot.long(), out),
                    (pos.cpu(), slot.cpu(), out.cpu()), (pos, slot, None),
                    (pos.t().contiguous().t(), slot, out), (pos[:50], slot, out),
                    (buf[:300].view(100, 3), slot, buf[30:330].view(100, 3)),
                    (pos.clone().requires_grad_(True), slot, out)):
        if o is None:
            continue
        assert not sphere_loss_grad_kernel(p, s, centers, radii, o)
    with torch.autograd.forward_ad.dual_level():
        assert not sphere_loss_grad_kernel(pos, slot, centers, radii, out)
    assert sphere_loss_grad_kernel(pos, slot, centers, radii, out)
    nan = pos.clone()
    nan[3] = float("nan")
    nan[4, 1] = float("inf")
    fn = sphere_loss_grad(centers, radii)
    a = fn(nan, slot, torch.empty_like(nan))
    b = fn(nan, slot.long(), torch.empty_like(nan))  # torch
    assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.nan_to_num(1.0), b.nan_to_num(1.0))
