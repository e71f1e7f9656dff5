"""Blending of short and odd lists: list lengths around the sub-tile backward's group of seven entries and
the blends' chunks of 64 list positions, every stage against the oracle on a ragged image; and the default
launch (blended per sub-tile in the tile's frame) against the per-tile kernels, bit for bit."""
import dataclasses

import numpy as np
import pytest

from paper_2509_07021_amd import _lib as L
from paper_2509_07021_amd import prune as P
from paper_2509_07021_amd import render as R
from paper_2509_07021_amd import scenes as S

from test_gpu_parity import _run_all_stages

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _faint_scene(n):
    """n Gaussians whose footprints cover most of the image, faint enough that hardly a pixel is opaque."""
    rng = np.random.default_rng(900 + n)
    sc = S.random_scene(rng, n, 1, False, spread=0.6, logscale_mu=-1.0)
    return dataclasses.replace(sc, op_logit=(0.5 * sc.op_logit - 3.0 - 0.4 * np.log2(n)).clip(-4.5, None).astype(np.float32))


@pytest.mark.parametrize("tile,subtile", [(16, 0), (32, 0), (16, 8), (32, 8)])
@pytest.mark.parametrize("n", [1, 6, 7, 8, 14, 15, 63, 64, 65, 70, 71, 128, 134, 300])
def test_list_lengths_at_group_and_chunk_edges(n, tile, subtile):
    cams = [S.look_at((0.0, -4.0, 0.3), 21, 13, bg=(0.3, 0.1, 0.2))]
    _run_all_stages(_faint_scene(n), cams, R.Config(tile, 64, subtile=subtile))


@pytest.mark.parametrize("tile", [16, 32])
@pytest.mark.parametrize("flags", [0, L.MEGS_FLAG_PERSISTENT, L.MEGS_FLAG_ONE_STAGE_SORT])
def test_default_launch_matches_the_per_tile_kernels(tile, flags):
    """waves = 0 against waves = 4 on uneven ragged views: images, final transmittances and last indices are
    the same bits (the same decisions over the same lists); importance sums and gradients add the same
    FP32 terms in another order, so each errs by at most a few roundings of its terms' absolute sum."""
    scene, cams = S.make_workload("small_2k_128px")
    cams = cams + [S.look_at((2.0, -3.0, 1.5), 101, 67, bg=(0.2, 0.3, 0.1)), S.look_at((0.2, -1.2, 0.1), 37, 41)]
    ds = R.DeviceScene.from_scene(scene)
    npix = sum(c.width * c.height for c in cams)
    dl = torch.rand(3 * npix, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    out = []
    for waves in (0, 4):
        cfg = R.Config(tile, 64, flags=flags, waves=waves)
        fr = R.forward(ds, cams, cfg)
        imgs = [fr.images.clone(), fr.buffer("T_final", npix, torch.float32).clone(),
                fr.buffer("last", npix, torch.int32).clone()]
        grads = R.backward(ds, fr, dl)
        imp_img, imp = P.importance(ds, cams, cfg)
        out.append((imgs, grads, imp_img, imp))
    (a, ga, ia, ma), (b, gb, ib, mb) = out
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    assert torch.equal(a[0], ia) and torch.equal(b[0], ib)
    # weights are positive, so a sum of m of them in any order errs by less than m ulps of itself; a score
    # adds at most a few thousand pixels, in partial sums of 64
    assert torch.allclose(ma, mb, rtol=2e-5, atol=1e-7)
    for p, g in ga.items():
        if g is not None and g.numel():
            assert float((g - gb[p]).norm() / gb[p].norm()) <= 1e-5, p


@pytest.mark.parametrize("tile,size", [(16, (121, 77)), (32, (121, 77)), (16, (1003, 803)), (32, (1003, 803)),
                                       (16, (640, 1025))])
@pytest.mark.parametrize("n", [400, 6000])
def test_long_lists_and_tile_order(tile, size, n):
    """Sub-tile lists queued by their flags against lists tested entry by entry (one-stage keys carry no
    flags), and the default launch against the per-tile kernels, on images of few and of many sub-tiles
    (run as numbered, or by list length) with remainders: the same decisions over the same lists, so the
    images, transmittances and last indices are the same bits."""
    rng = np.random.default_rng(n)
    sc = S.random_scene(rng, n, 1, False, spread=0.7, logscale_mu=-2.0)
    cams = [S.look_at((0.0, -4.0, 0.3), *size, bg=(0.3, 0.1, 0.2)), S.look_at((3.0, -2.0, 0.3), size[1], size[0])]
    ds = R.DeviceScene.from_scene(sc)
    npix = sum(c.width * c.height for c in cams)
    dl = torch.rand(3 * npix, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    for pair in ([R.Config(tile, 64, subtile=8), R.Config(tile, 64, subtile=8, flags=L.MEGS_FLAG_ONE_STAGE_SORT)],
                 [R.Config(tile, 64), R.Config(tile, 64, waves=4)]):
        out = []
        for cfg in pair:
            fr = R.forward(ds, cams, cfg)
            out.append(([fr.images.clone(), fr.buffer("T_final", npix, torch.float32).clone(),
                         fr.buffer("last", npix, torch.int32).clone()], R.backward(ds, fr, dl)))
        for x, y in zip(out[0][0], out[1][0]):
            assert torch.equal(x, y)
        for p, g in out[0][1].items():
            if g is not None and g.numel():
                assert float((g - out[1][1][p]).norm() / g.norm()) <= 1e-5, p


@pytest.mark.parametrize("tile,sizes", [(16, [(2048, 2048)]), (16, [(2049, 2048)]), (16, [(2113, 2100), (65, 4000), (2048, 2100)]),
                                        (16, [(4096, 4096)]), (16, [(4097, 4096)]), (32, [(4097, 4128)]), (32, [(8192, 8224)])])
def test_tile_order_in_slices(tile, sizes):
    """16,384 tiles (ordered in one piece), 16,512, 35,702 and 65,536 (two to four slices in the backward), 65,792
    (none), and with 32 x 32 tiles 16,641 and 65,792 (two and five slices in the forward): the sub-tile blends run in
    that order, with the two-stage and the one-stage sort, against the persistent launch, which runs the
    sub-tiles as numbered: the same decisions over the same lists, so the same bits, and every tile was run."""
    sc = S.random_scene(np.random.default_rng(5), 4000, 1, False, spread=1.5, logscale_mu=-3.0)
    cams = [S.look_at((0.0, -4.0, 0.3 + 0.2 * i), w, h, bg=(0.3, 0.1, 0.2)) for i, (w, h) in enumerate(sizes)]
    ds = R.DeviceScene.from_scene(sc)
    npix = sum(c.width * c.height for c in cams)
    dl = torch.rand(3 * npix, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    out = []
    for flags in (L.MEGS_FLAG_PERSISTENT, 0, L.MEGS_FLAG_ONE_STAGE_SORT):
        fr = R.forward(ds, cams, R.Config(tile, 64, subtile=8, flags=flags))
        assert int(fr.state.n_pairs) >= 8 * int(fr.state.n_tiles)  # (above 65,536 tiles only long lists are ordered)
        out.append(([fr.images.clone(), fr.buffer("T_final", npix, torch.float32).clone(),
                     fr.buffer("last", npix, torch.int32).clone()], R.backward(ds, fr, dl)))
    for other in out[1:]:
        for x, y in zip(out[0][0], other[0]):
            assert torch.equal(x, y)
        for p, g in out[0][1].items():
            if g is not None and g.numel():
                assert float((g - other[1][p]).norm() / g.norm()) <= 1e-5, p


@pytest.mark.parametrize("tile,subtile", [(16, 0), (32, 0), (16, 8), (32, 8)])
@pytest.mark.parametrize("sizes", [[(1003, 803)], [(121, 77)], [(33, 31)] * 63 + [(200, 17)]])
def test_tiles_with_empty_lists(tile, subtile, sizes):
    """A few small Gaussians on images whose tiles are mostly empty, ragged at both edges, one view and as many as there
    can be: every stage of the one view against the oracle, images and gradients against the per-tile kernels', and the
    background exact where nothing is included."""
    sc = S.random_scene(np.random.default_rng(11), 40, 1, False, spread=0.3, logscale_mu=-5.0)
    cams = [S.look_at((0.0, -4.0, 0.3 + 0.01 * i), w, h, bg=(0.3, 0.1 + 0.01 * i, 0.2)) for i, (w, h) in enumerate(sizes)]
    cfg = R.Config(tile, 64, subtile=subtile)
    if len(cams) == 1:
        _run_all_stages(sc, cams, cfg)
    ds = R.DeviceScene.from_scene(sc)
    npix = sum(c.width * c.height for c in cams)
    dl = torch.rand(3 * npix, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    out = []
    for c in (cfg, R.Config(tile, 64, waves=4)):
        torch.full((64 << 20,), float("nan"), device="cuda")  # what the allocator hands out next holds NaN
        fr = R.forward(ds, cams, c)
        out.append((fr.images.clone(), fr.buffer("T_final", npix, torch.float32).clone(),
                    fr.buffer("last", npix, torch.int32).clone(), R.backward(ds, fr, dl)))
    off = 0
    for c in cams:
        n = c.width * c.height
        none = out[0][2][off:off + n] == 0
        assert bool(none.any()) and bool(torch.equal(out[0][1][off:off + n][none], torch.ones_like(out[0][1][off:off + n][none])))
        for ch in range(3):
            plane = out[0][0][3 * off + ch * n:3 * off + (ch + 1) * n]
            assert bool((plane[none] == float(np.float32(c.bg[ch]))).all())
        off += n
    assert float((out[0][0] - out[1][0]).abs().max()) <= 1e-5
    for p, g in out[1][3].items():
        if g is not None and g.numel():
            assert float((g - out[0][3][p]).norm() / g.norm()) <= 1e-4, p


@pytest.mark.parametrize("tile,size,n,mu", [(32, (1311, 1311), 400, -5.5), (32, (1311, 1311), 4000, -3.5), (16, (1003, 803), 60, 0.3),
                                            (32, (1003, 803), 60, 0.3), (16, (1003, 803), 3000, -1.0), (32, (1003, 803), 3000, -1.0)])
def test_default_launch_where_it_runs_the_per_tile_kernels(tile, size, n, mu):
    """Short lists of 32 x 32 tiles, and few records that cover most of the image (the library's choice is then the
    per-tile kernels, in the forward, the importance or the backward), and sizes on the other side of that choice: images,
    transmittances and last indices as with waves = 4, sums and gradients to the rounding of their order."""
    sc = S.random_scene(np.random.default_rng(n), n, 1, False, spread=0.7, logscale_mu=mu)
    sc = dataclasses.replace(sc, op_logit=(sc.op_logit - 3.0).astype(np.float32))
    cams = [S.look_at((0.0, -4.0, 0.3), *size, bg=(0.3, 0.1, 0.2))]
    ds = R.DeviceScene.from_scene(sc)
    npix = size[0] * size[1]
    dl = torch.rand(3 * npix, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    out = []
    for cfg in (R.Config(tile, 64), R.Config(tile, 64, waves=4)):
        fr = R.forward(ds, cams, cfg)
        images, imp = P.importance(ds, cams, cfg)
        out.append(([fr.images.clone(), fr.buffer("T_final", npix, torch.float32).clone(),
                     fr.buffer("last", npix, torch.int32).clone(), images], imp, R.backward(ds, fr, dl)))
    for x, y in zip(out[0][0], out[1][0]):
        assert torch.equal(x, y)
    # a score sums at most 805,409 weights, first in partial sums of 64 or 256 and those one by one, of which
    # there are at most 12,585: in any order that errs by less than 12,585 x 2^-24 of the (positive) sum
    assert torch.allclose(out[0][1], out[1][1], rtol=7.5e-4, atol=1e-7)
    for p, g in out[1][2].items():
        if g is not None and g.numel():
            assert float((g - out[0][2][p]).norm() / g.norm()) <= 1e-4, p


@pytest.mark.parametrize("tile,subtile,flags,evaluated", [
    (8, 0, 0, 379_840), (16, 8, 0, 392_000), (32, 8, 0, 397_056), (16, 8, L.MEGS_FLAG_ONE_STAGE_SORT, 403_968),
    (32, 8, L.MEGS_FLAG_ONE_STAGE_SORT, 410_304), (32, 8, L.MEGS_FLAG_PERSISTENT, 397_056)])
def test_fragment_counts(tile, subtile, flags, evaluated):
    """The statistics' whole numbers on a fixed scene: the blended fragments are the same for every launch; those tested are
    the live pixels of the entries that the sub-tile flags, or without flags the footprint boxes, leave."""
    scene, cams = S.make_workload("small_2k_128px")
    fr = R.forward(R.DeviceScene.from_scene(scene), cams, R.Config(tile, 64, flags | L.MEGS_FLAG_STATS, subtile=subtile))
    torch.cuda.synchronize()
    st = fr.alloc.view(fr.state.device_status, 8, torch.int32).cpu().numpy()
    assert (int(st[4:6].view("uint64")[0]), int(st[6:8].view("uint64")[0])) == (80_458, evaluated)
