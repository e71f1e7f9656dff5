"""The top-kappa selection and the compaction at the edges of their launches: one workgroup or several,
chunks with a remainder, ties that begin, end and cross workgroups, infinities, a long and a short
Gaussian count around the workgroup size, more lobes than are loaded together. Selections, index maps
and offsets are whole numbers and compared exactly."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2509_07021_amd import render as R
from paper_2509_07021_amd import scenes as S

from gpu_util import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_2509_07021_amd import prune as P  # noqa: E402


@pytest.mark.parametrize("n", [2, 1023, 1024, 1025, 16384, 16385, 18433, 524287, 524289, 700_001])
@pytest.mark.parametrize("kind", ["distinct", "two", "one", "inf", "one_exponent"])
def test_topk_sizes(n, kind):
    rng = np.random.default_rng(n)
    if kind == "distinct":
        score = rng.permutation(n).astype(np.float32) - n // 2  # below 2^24: exact, no ties
    elif kind == "two":
        score = rng.choice(np.float32([-1.5, 2.0]), size=n)
    elif kind == "one":
        score = np.full(n, -0.0, np.float32)
        score[::3] = 0.0
    elif kind == "inf":
        score = rng.choice(np.float32([-np.inf, np.inf, 3e38, -3e38, 1e-45]), size=n)
    else:
        score = (1.0 + rng.integers(0, 300, size=n) * 2.0 ** -23).astype(np.float32)
    dev = torch.from_numpy(np.concatenate([np.float32([0.0]), score])).cuda()[1:]  # 4-byte aligned only
    for kappa in sorted({1, n // 3, n // 2, n - 1} - {0}):
        log(f"topk n={n} {kind} kappa={kappa}")
        keep = P.select_topk(dev, kappa).cpu().numpy().astype(bool)
        np.testing.assert_array_equal(keep, O.topk_keep(score.astype(np.float64), kappa))


@pytest.mark.parametrize("n,k,ragged,dt", [(1, 1, False, "f32"), (511, 4, False, "f32"), (512, 5, False, "f16"),
                                           (513, 8, False, "f32"), (513, 8, True, "f32"), (1025, 4, True, "bf16"),
                                           (70_001, 6, True, "f16"), (1_100_000, 1, False, "f32")])
def test_compaction_sizes(n, k, ragged, dt):
    log(f"compaction n={n} k={k} ragged={ragged} {dt}")
    rng = np.random.default_rng(n + k)
    sc = S.ragged_scene(rng, n, k, masks=True) if ragged else S.make_scene(n, k, 5, clustered=False, masks=True)
    if sc.sharp.size:
        sc.sharp[rng.random(sc.sharp.shape) < 0.5] *= 0.01
    sc = sc.stored(dt, dt, dt)
    pl = sc.widened()
    o = 1 / (1 + np.exp(-pl["op_logit"])) / (1 + np.exp(-pl["pmask_logit"]))
    tau = float(np.median(o)) * (1 + 1e-7) if n > 1 else 0.0
    assert np.min(np.abs(o - tau)) > 1e-12  # no decision within the last places of exp
    cds, kept, lobe_src = P.compact(R.DeviceScene.from_scene(sc), tau, 1.0)
    ref = O.compact(pl, sc.k, tau, 1.0)
    np.testing.assert_array_equal(kept.cpu().numpy(), ref["kept"])
    np.testing.assert_array_equal(cds.lobe_off.cpu().numpy(), ref["lobe_off"])
    np.testing.assert_array_equal(lobe_src.cpu().numpy(), ref["lobe_src"])
    for q in ("pos", "logscale", "quat", "axis", "sharp"):  # copied bit for bit
        got = cds.planes[q].float().cpu().numpy().ravel()
        np.testing.assert_array_equal(got, ref[q].ravel().astype(np.float32), err_msg=q)
    ulp = {"f32": 2.0 ** -23, "f16": 2.0 ** -10, "bf16": 2.0 ** -7}[dt]  # one of the storage type
    for q in ("op_logit", "base", "amp"):
        got, r = cds.planes[q].double().cpu().numpy().ravel(), ref[q].ravel()
        assert np.all(np.abs(got - r) <= ulp * np.abs(r) + 6e-8), q
