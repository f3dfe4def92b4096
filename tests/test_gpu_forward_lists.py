"""The forward blend's walks at the lengths where they can go wrong: 1 to 700
leaves over images of a few pixels and of ragged tiles, so that a quarter's
list passes the pair of entries taken at a time, the 32-entry history, the
128-entry chunk and the staged batch, and tiles with pixels that stop early
beside pixels that never do; image, transmittance, blended counts and
contributors against the oracle, the same for every tile."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2406_12080_amd import synth
import parity as PR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opaque", [False, True])
@pytest.mark.parametrize("n", [1, 2, 31, 33, 63, 65, 127, 129, 257, 700])
def test_walk_lengths(n, opaque):
    from paper_2406_12080_amd import hgs
    lv = synth.make_leaves(n, "cube", n)
    lv["scale"] = lv["scale"] * np.float32(12.0)  # each leaf over most of the image
    lv["opacity"] = np.full(n, 0.97 if opaque else 0.012, np.float32)
    h = synth.build_hierarchy(lv)
    w, hh = ((3, 2), (40, 24), (33, 17))[n % 3]
    v = PR.safe_tau(h, synth.look_at((0, 0, 3), (0, 0, 0), (0, 1, 0), w, hh, 0.0))
    o = O.render(h, v)
    r = hgs.Renderer(0)
    first = None
    try:
        r.upload(h)
        for tile in ((8, 8, 64), (16, 8, 256), (16, 16, 256), (32, 16, 512)):
            r.set_tuning(*tile)
            (img,), st = r.render([v])
            T = r.buffer(hgs.BUF_T_FINAL, torch.float32)
            nb = r.buffer(hgs.BUF_N_BLEND, torch.int32)
            last = r.buffer(hgs.BUF_N_LAST, torch.int32)
            res = PR.check_pixels(img.cpu().numpy().reshape(-1, 3).astype(np.float64),
                                  T.cpu().numpy().astype(np.float64), o)
            assert res["ok"], (tile, res)
            clean = o["nalt"] == 0
            assert np.array_equal(nb.cpu().numpy()[clean], o["nblend"][clean]), tile
            assert st["blended"] == int(nb.sum()) <= st["evaluated"]
            assert bool(((last == 0) == (nb == 0)).all()) and bool((last >= nb).all())
            state = (img.clone(), T, nb)
            if first is None:
                first = state
            assert all(torch.equal(a, b) for a, b in zip(first, state)), tile
    finally:
        r.close()
