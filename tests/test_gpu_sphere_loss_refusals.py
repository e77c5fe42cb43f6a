"""What the batched loss gradient refused or followed when it was torch
operations alone, it still refuses or follows beside its kernel."""
import pytest
import torch

from paper_1803_03949_amd.batch import sphere_loss_grad
from paper_1803_03949_amd.binding import sphere_loss_grad_kernel

pytestmark = pytest.mark.gpu


def inputs(n=70, m=3):
    g = torch.Generator().manual_seed(2)
    pos = torch.rand((n, 3), generator=g) * 2
    slot = torch.randint(-1, m, (n,), generator=g, dtype=torch.int32)
    pos[slot == -1] = 0
    return [t.cuda() for t in (pos, slot, torch.rand((m, 3), generator=g),
                               torch.rand(m, generator=g) + 0.1)]


@pytest.mark.parametrize("which", ["centers", "radii"])
def test_a_gradient_of_the_spheres_is_refused(which):
    pos, slot, centers, radii = inputs()
    want = sphere_loss_grad(centers, radii)(pos, slot, torch.empty_like(pos))
    (centers if which == "centers" else radii).requires_grad_(True)
    assert not sphere_loss_grad_kernel(pos, slot, centers, radii, torch.empty_like(pos))
    fn = sphere_loss_grad(centers, radii)
    with pytest.raises(RuntimeError, match="requires grad"):
        fn(pos, slot, torch.empty_like(pos))
    with torch.no_grad():
        assert torch.equal(fn(pos, slot, torch.empty_like(pos)), want)
