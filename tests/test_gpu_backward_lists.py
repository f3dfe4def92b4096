"""The blend backward's walks at the lengths where they can go wrong: a few
pixels (less than one tile, less than one quarter, ragged) under 2 to 700
leaves, so that a tile's list, and the list each 4x4 quarter walks two entries
at a time, passes the staged batch's and the 32-entry word's edges, against
the oracle's gradients at the parity tests' bounds; with floating-point
atomics and in the deterministic mode.  And a cotangent that is not finite on
one pixel stays on the splats that pixel can reach."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2406_12080_amd import synth
from test_gpu_parity import _grad_case

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("tuning", [(8, 8, 64, 0), (16, 8, 128, 0), (16, 16, 256, 1), (32, 16, 512, 0)])
@pytest.mark.parametrize("n", [2, 20, 33, 65, 130, 257, 700])
def test_short_and_odd_lists(n, tuning, det):
    if det:
        tuning = tuning[:3] + (0,)  # it launches one workgroup per tile
    h = synth.make_scene(1, n_leaves=n)
    w, hh = ((3, 2), (13, 11), (33, 17))[n % 3]
    # narrow: the whole cube fills the image, so that every tile sees most splats
    v = synth.look_at((0, 0, 3), (0, 0, 0), (0, 1, 0), w, hh, 0.15 * hh / 11)
    _grad_case(h, v, seed=n, tuning=tuning, det=det)


def test_nan_cotangent_stays_on_its_pixel():
    from paper_2406_12080_amd import hgs
    h = synth.make_scene(1)
    v = synth.make_views(1, tau=4.0)[0]
    r = hgs.Renderer(0)
    try:
        r.upload(h)
        grads = {k: torch.zeros_like(t) for k, t in hgs.params_to_device(h).items()}
        dL = torch.randn((v.height, v.width, 3), generator=torch.Generator().manual_seed(3)).cuda()
        dL[3, 5] = float("nan")  # a corner of the image that few splats reach
        r.render([v])
        r.backward([dL], grads)
        bad = torch.isnan(grads["sh"]).any(1)
        assert int(bad.sum()) < 0.05 * int((grads["sh"] != 0).any(1).sum())
        dL[3, 5] = 0.0
        clean = {k: torch.zeros_like(t) for k, t in grads.items()}
        r.render([v])
        r.backward([dL], clean)
        ok = ~bad
        for k in grads:
            # off the NaN pixel's splats: the same sums, in atomic order
            a, b = grads[k][ok].double(), clean[k][ok].double()
            assert torch.isfinite(a).all(), k
            assert float((a - b).norm()) <= 1e-6 * float(b.norm()), k
    finally:
        r.close()
