"""The first sizing forward of a process while another thread captures a stream in the global mode: the forward allocates
its pinned words without disturbing the capture. In a process of its own, since the words are allocated once."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = """
import threading
import numpy as np
import torch
from paper_2509_07021_amd import render as R
from paper_2509_07021_amd import scenes as S

ds = R.DeviceScene.from_scene(S.random_scene(np.random.default_rng(0), 500, 1, False, logscale_mu=-3.0))
cams = [S.look_at((0.0, -4.0, 0.1), 64, 48)]
side = torch.cuda.Stream()
with torch.cuda.stream(side):  # a fixed pair capacity waits for nothing; it also fills the stream's memory pool
    ref = R.forward(ds, cams, R.Config(pair_capacity=100_000)).images.clone()
    frames = [R.forward(ds, cams, R.Config(pair_capacity=100_000)) for _ in range(4)]
    del frames
torch.cuda.synchronize()
out, kept = [], []

def work():
    try:
        with torch.cuda.stream(side):
            kept.append(R.forward(ds, cams, R.Config()))
    except Exception as e:
        out.append(repr(e))

x = torch.ones(1000, device="cuda")
g = torch.cuda.CUDAGraph()
with torch.cuda.graph(g, capture_error_mode="global"):
    x.mul_(2.0)
    t = threading.Thread(target=work)
    t.start()
    t.join()
    x.add_(1.0)
torch.cuda.synchronize()
out += [bool(torch.equal(fr.images, ref)) for fr in kept]
for i in range(3):
    g.replay()
    torch.cuda.synchronize()
    fr = R.forward(ds, cams, R.Config())
    out.append(bool(torch.equal(fr.images, ref)))
print("forwards", out, "x", float(x[0]), flush=True)
"""


def test_first_sizing_forward_beside_a_capture():
    r = subprocess.run([sys.executable, "-c", CODE], cwd=ROOT, capture_output=True, text=True, timeout=100)
    print(r.stdout, r.stderr)
    assert r.returncode == 0, r.stderr[-2000:]
    assert "forwards [True, True, True, True] x 15.0" in r.stdout, r.stdout
