"""The photometric loss at the sizes where its strips change: widths around the 64 columns and the 5-pixel
halo of a strip, heights around the strips' 4 to 64 rows, images smaller than the window, several views."""
import numpy as np
import pytest

from test_gpu_train import T, _Size, _loss_case

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


@pytest.mark.parametrize("sizes", [
    [(1, 1)], [(1, 9), (9, 1)], [(5, 5), (11, 11)], [(63, 4), (64, 5), (65, 3)], [(69, 8), (70, 9), (74, 7)],
    [(127, 13), (128, 12), (129, 11), (133, 16)], [(700, 517)], [(963, 1081), (640, 33)], [(2113, 1301)],
], ids=lambda s: "+".join(f"{w}x{h}" for w, h in s))
def test_loss_at_strip_edges(sizes):
    _loss_case(sizes, 140 + len(sizes)) if sizes[0][0] >= 4 and sizes[0][1] >= 4 else _small(sizes)


def _small(sizes):
    """_loss_case without its equal corner, which needs four pixels (same bounds)."""
    from oracle import oracle as O
    rng = np.random.default_rng(7)
    xs = [rng.uniform(-0.1, 1.1, size=(3, h, w)).astype(np.float32) for w, h in sizes]
    ys = [rng.uniform(0.0, 1.0, size=x.shape).astype(np.float32) for x in xs]
    flat = lambda a: torch.from_numpy(np.concatenate([v.reshape(-1) for v in a])).cuda()
    loss, dl = T.photometric_loss(flat(xs), flat(ys), [_Size(w, h) for w, h in sizes])
    ref, grads = O.photometric_loss([x.astype(np.float64) for x in xs], [y.astype(np.float64) for y in ys], 0.2)
    np.testing.assert_allclose(float(loss), ref, rtol=1e-12)
    want = np.concatenate([g.reshape(-1) for g in grads])
    bound = 2.0 ** -23 * np.abs(want) + 1e-12 * np.abs(want).max()
    assert np.all(np.abs(dl.cpu().numpy().astype(np.float64) - want) <= bound)


def test_loss_without_gradient_and_repeated():
    """The loss alone and with its gradient are the same bits, and so are repeated calls."""
    g = torch.Generator(device="cuda").manual_seed(2)
    sizes = [_Size(321, 77), _Size(64, 130)]
    n = sum(3 * s.width * s.height for s in sizes)
    x, y = (torch.rand(n, device="cuda", generator=g) for _ in range(2))
    a, dl = T.photometric_loss(x, y, sizes)
    b, none = T.photometric_loss(x, y, sizes, with_grad=False)
    c, dl2 = T.photometric_loss(x, y, sizes)
    assert none is None and float(a) == float(b) == float(c) and torch.equal(dl, dl2)


@pytest.mark.parametrize("sizes", [
    # 16 x 16 tiles: edges of a tile and of its halo, several views, the narrowest and tallest
    [(16, 16)], [(17, 15), (15, 17), (32, 33)], [(21, 22), (26, 27), (5, 48)], [(1, 700), (2, 65)], [(640, 350)], [(33, 18)] * 64,
    # strips of 2 to 64 rows on wide images: edges of a strip's columns and halo
    [(4096, 1)], [(4097, 2)], [(4159, 3), (4160, 5)], [(4101, 9), (4155, 17)], [(703, 517)], [(961, 603), (64, 7)],
], ids=lambda s: f"{len(s)} of {s[0][0]}x{s[0][1]}")
def test_loss_in_tiles_and_in_strips(sizes):
    _small(sizes)
