"""Blending of short and odd lists: list lengths around the sub-tile backward's group of seven entries and
the blends' chunks of 64 list positions, every stage against the oracle on a ragged image."""
import dataclasses

import numpy as np
import pytest

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


@pytest.mark.parametrize("tile", [16, 32])
@pytest.mark.parametrize("n", [1, 6, 7, 8, 14, 15, 63, 64, 65, 70, 71, 128, 134, 300])
def test_list_lengths_at_group_and_chunk_edges(n, tile):
    cams = [S.look_at((0.0, -4.0, 0.3), 21, 13, bg=(0.3, 0.1, 0.2))]
    _run_all_stages(_faint_scene(n), cams, R.Config(tile, 64, subtile=8))
