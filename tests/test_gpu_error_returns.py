"""Calls that fail after the host has learned a counted total: the stream is idle when they return, so the caller may
free or reuse the memory it gave."""
import ctypes

import numpy as np
import pytest

from paper_2509_07021_amd import _lib as L
from paper_2509_07021_amd import render as R
from paper_2509_07021_amd import scenes as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)


def _blocks(refuse):
    """Allocation callback that refuses the block of that index (from 0), and the blocks it gave."""
    given = []

    def take(ctx, nbytes):
        if len(given) == refuse:
            given.append(None)
            return None
        given.append(torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
        return given[-1].data_ptr()

    return L.ALLOC_FN(take), given


@pytest.mark.parametrize("case", ["pairs refused", "malformed lobes"])
def test_a_forward_that_fails_on_its_count_leaves_the_stream_idle(case):
    """32 M records, whose scan runs on for a while after the total is known."""
    n, nv = 1 << 20, 32
    rng = np.random.default_rng(0)
    ragged = case == "malformed lobes"
    sc = S.random_scene(rng, n, 0, False, logscale_mu=-7.0)
    if ragged:
        off = np.minimum(np.arange(n + 1), 1000).astype(np.int32)
        off[7] = 5  # after a 6
        one = S.random_scene(rng, 1000, 1, False)
        sc.k, sc.axis, sc.sharp, sc.amp, sc.lobe_off = 1, one.axis[0], one.sharp[0], one.amp[0], off
    ds = R.DeviceScene.from_scene(sc)
    cams = [S.look_at((0.0, -4.0, 0.02 * i), 32, 32) for i in range(nv)]
    images = torch.empty(3 * nv * 32 * 32, dtype=torch.float32, device="cuda")
    scene, arr, cfg, state = ds.struct(), R.cameras_struct(cams), R.Config(16, 64).struct(), L.MegsState()
    lib = L.load()
    for _ in range(3):
        fn, given = _blocks(None if ragged else 1)
        torch.cuda.synchronize()
        stream = torch.cuda.current_stream()
        st = lib.megs_render_forward(ctypes.byref(scene), arr, nv, ctypes.byref(cfg), fn, None, images.data_ptr(),
                                     ctypes.byref(state), stream.cuda_stream)
        idle = stream.query()
        torch.cuda.synchronize()
        assert st == (L.MEGS_ERR_ARG if ragged else L.MEGS_ERR_ALLOC), lib.megs_last_error()
        assert idle and len(given) == (1 if ragged else 2)
