"""The key table at the sizes where the sorts and scans change their form: one workgroup (up to 8,192 items),
count tables summed by the scatter (up to 64 workgroups), 4, 8 or 16 keys a thread of a radix pass, scans whose second pass sums the totals
(up to 1,024 workgroups of 2,048), and the general form; and forwards from several threads at once."""
import threading

import numpy as np
import pytest

from gpu_util import IMG_TOL
from oracle import oracle as O
from paper_2509_07021_amd import _lib as L
from paper_2509_07021_amd import render as R
from paper_2509_07021_amd import scenes as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _table(ds, cams, cfg, n):
    fr = R.forward(ds, cams, cfg)
    st, nr = fr.state, n * len(cams)
    p = int(st.n_pairs)
    out = {"pairs": p, "counts": fr.counts(), "vals": fr.buffer("vals", p, torch.int32).cpu().numpy().view(np.uint32),
           "ranges": fr.buffer("ranges", 2 * int(st.n_tiles), torch.int32).cpu().numpy().reshape(-1, 2),
           "ntiles": fr.buffer("ntiles", nr, torch.int32).cpu().numpy(),
           "depth": fr.buffer("rgbd", 4 * nr, torch.float32).view(nr, 4)[:, 3].cpu().numpy().view(np.uint32),
           "images": fr.images.clone()}
    if st.tile_keys:
        out["tile"] = fr.buffer("tile_keys", p, torch.int32).cpu().numpy().view(np.uint32)
    else:
        out["tile"] = (fr.buffer("keys64", p, torch.int64).cpu().numpy().view(np.uint64) >> np.uint64(32)).astype(np.uint32)
    return out


@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 1024, 1025, 4096, 4097, 8191, 8192, 8193, 65_536, 65_537, 262_144, 262_145,
                               655_359, 655_360, 2_097_152, 2_097_153, 4_194_303, 4_194_304])
def test_key_table_at_the_sorts_size_limits(n):
    rng = np.random.default_rng(n)
    scene = S.random_scene(rng, n, 0, False, spread=1.5, logscale_mu=-5.0 if n > 100_000 else -3.0)
    # equal depths among the records, whose order is then the record index: rows of Gaussians facing the camera
    scene.pos[1] = np.round(scene.pos[1] * 20) / 20
    cams = [S.look_at((0.0, -4.0, 0.0), 93, 70)]
    ds = R.DeviceScene.from_scene(scene)
    planes = L.MEGS_FLAG_RECORD_PLANES
    a = _table(ds, cams, R.Config(16, 64, flags=planes), n)
    # every record's pairs, sorted by tile, depth bits and record
    assert a["pairs"] == int(a["ntiles"].astype(np.int64).sum()) == a["counts"]["pairs_needed"]
    assert np.array_equal(np.bincount(a["vals"], minlength=n), a["ntiles"])
    t, d, v = a["tile"].astype(np.uint64), a["depth"][a["vals"]].astype(np.uint64), a["vals"].astype(np.int64)
    key = (t << np.uint64(32)) | d
    assert np.all((key[1:] > key[:-1]) | ((key[1:] == key[:-1]) & (v[1:] > v[:-1])))
    first = np.searchsorted(a["tile"], np.arange(len(a["ranges"])), side="left")
    last = np.searchsorted(a["tile"], np.arange(len(a["ranges"])), side="right")
    empty = first == last
    assert np.array_equal(a["ranges"][~empty], np.stack([first, last], 1)[~empty]) and not a["ranges"][empty].any()
    b = _table(ds, cams, R.Config(16, 64, flags=planes | L.MEGS_FLAG_ONE_STAGE_SORT), n)
    assert np.array_equal(a["vals"], b["vals"]) and np.array_equal(a["tile"], b["tile"])
    assert np.array_equal(a["ranges"], b["ranges"]) and torch.equal(a["images"], b["images"])


@pytest.mark.parametrize("culled", [False, True])
@pytest.mark.parametrize("n", [1, 2, 64, 65, 1000, 1025, 8192])
def test_key_table_of_records_at_one_depth(n, culled):
    """Every depth key the same, so that no digit of the depth sort differs: a plane of Gaussians that faces the
    camera, and the same plane behind it (all culled). The depth order is the record order."""
    rng = np.random.default_rng(n)
    scene = S.random_scene(rng, n, 0, False, logscale_mu=-3.0)
    scene.pos[0], scene.pos[2] = rng.uniform(-1.0, 1.0, (2, n))
    scene.pos[1] = -9.0 if culled else 0.25
    scene.op_logit[:] = 1.0
    cams = [S.look_at((0.0, -4.0, 0.0), 93, 70)]
    ds = R.DeviceScene.from_scene(scene)
    planes = L.MEGS_FLAG_RECORD_PLANES
    a = _table(ds, cams, R.Config(16, 64, flags=planes), n)
    assert a["pairs"] == int(a["ntiles"].astype(np.int64).sum()) == a["counts"]["pairs_needed"]
    assert a["counts"]["culled"] == (n if culled else 0)
    if culled:
        assert a["pairs"] == 0 and not a["ranges"].any()
    else:
        assert np.all(a["ntiles"] > 0) and np.unique(a["depth"]).size == 1
    assert np.array_equal(np.bincount(a["vals"], minlength=n), a["ntiles"])
    key = (a["tile"].astype(np.int64) << 32) | a["vals"]  # by tile, and in a tile by record
    assert np.all(key[1:] > key[:-1])
    b = _table(ds, cams, R.Config(16, 64, flags=planes | L.MEGS_FLAG_ONE_STAGE_SORT), n)
    for name in ("vals", "tile", "ranges"):
        assert np.array_equal(a[name], b[name])
    assert torch.equal(a["images"], b["images"])
    ref = O.render(scene.widened(), scene.k, cams, 16)
    ok = ref["views"][0]["flag"] == 0
    img = a["images"].view(3, cams[0].height, cams[0].width).cpu().numpy()
    assert np.abs(img - ref["images"][0])[:, ok].max() <= IMG_TOL


def test_forwards_from_several_threads():
    """Sizing forwards (each waits for its own pair count) on eight threads and streams: the images are those
    of one thread."""
    scenes = [S.random_scene(np.random.default_rng(i), 300 * (i + 1) ** 2, 1, False, logscale_mu=-3.0) for i in range(8)]
    cams = [[S.look_at((0.0, -4.0, 0.1 * i), 40 + 9 * i, 33)] for i in range(8)]
    ds = [R.DeviceScene.from_scene(s) for s in scenes]
    ref = [R.forward(ds[i], cams[i], R.Config()).images.clone() for i in range(8)]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for r in range(6):
                k = (i + r) % 8
                fr = R.forward(ds[k], cams[k], R.Config())
                stream.synchronize()
                if not torch.equal(fr.images, ref[k]):
                    bad.append((i, r))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


@pytest.mark.parametrize("n,w,h", [(256, 2048, 1024), (256, 2048, 1025), (257, 2048, 2048), (257, 2056, 2048), (1, 2049, 1024)])
def test_ranges_where_few_records_meet_many_tiles(n, w, h):
    """Tile ranges cleared by the emission (up to 128 a thread: 32,768 tiles for 256 records, 65,536 for 257) or by
    a launch of their own: only the tiles that records list have a range. The forward before leaves other ranges
    in the memory that this one gets."""
    scene = S.random_scene(np.random.default_rng(n), n, 0, False, logscale_mu=-5.0)
    ds, dense = R.DeviceScene.from_scene(scene), R.DeviceScene.from_scene(S.random_scene(np.random.default_rng(1), 3000, 0, False))
    cams = [S.look_at((0.0, -4.0, 0.0), w, h)]
    R.forward(dense, cams, R.Config(8, 64, flags=L.MEGS_FLAG_RECORD_PLANES))
    a = _table(ds, cams, R.Config(8, 64, flags=L.MEGS_FLAG_RECORD_PLANES), n)
    first = np.searchsorted(a["tile"], np.arange(len(a["ranges"])), side="left")
    last = np.searchsorted(a["tile"], np.arange(len(a["ranges"])), side="right")
    empty = first == last
    assert a["pairs"] > 0 and np.array_equal(a["ranges"][~empty], np.stack([first, last], 1)[~empty])
    assert not a["ranges"][empty].any()


def test_emission_of_few_records_on_many_tiles_is_short():
    """256 records on 4.2 M tiles: the emission does not clear them all with one workgroup (0.51 ms). The shortest of
    five, against a bound far above what it takes."""
    ds = R.DeviceScene.from_scene(S.random_scene(np.random.default_rng(0), 256, 0, False, logscale_mu=-7.0))
    ms = []
    for _ in range(5):
        with R.Profile() as p:
            R.forward(ds, [S.look_at((0.0, -4.0, 0.3), 16384, 16384)], R.Config(8, 64))
            torch.cuda.synchronize()
        ms.append(p.ms["emit"])
    assert min(ms) < 0.2, ms
