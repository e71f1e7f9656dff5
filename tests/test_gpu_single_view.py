"""A single view's image is the forward's buffer itself: gradients that arrive expanded, transposed or as a
plain copy are taken alike, and the image may be changed in place."""
import pytest

from paper_2509_07021_amd import render as R
from paper_2509_07021_amd import scenes as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("form", ["plain", "expanded", "transposed", "in_place"])
def test_gradient_of_one_view(form):
    scene, cams = S.make_workload("small_2k_128px")
    cams = [S.look_at((0.0, -4.0, 0.3), 101, 67)]
    ds = R.DeviceScene.from_scene(scene)
    g = torch.Generator(device="cuda").manual_seed(7)
    w = torch.rand(3, 67, 101, device="cuda", generator=g)
    if form == "expanded":
        w = w[:, :1, :1].expand(3, 67, 101)
    elif form == "transposed":
        w = w.transpose(1, 2).contiguous().transpose(1, 2)
    fr = R.forward(ds, cams, R.Config(16, 64))
    ref = R.backward(ds, fr, (w.contiguous() * (2.0 if form == "in_place" else 1.0)).reshape(-1))
    leaves = [(q, t.requires_grad_(True)) for q, t in ds.planes.items() if t is not None and t.numel()]
    (img,) = R.render(ds, cams, R.Config(16, 64))
    assert img.shape == (3, 67, 101) and torch.equal(img.detach().reshape(-1), fr.images)
    if form == "in_place":
        img.mul_(2.0)
    grads = torch.autograd.grad([img], [t for _, t in leaves], grad_outputs=[w])
    for (q, _), x in zip(leaves, grads):  # the float atomics add the same terms in another order
        assert float((x - ref[q]).norm()) <= 1e-5 * float(ref[q].norm()), q
