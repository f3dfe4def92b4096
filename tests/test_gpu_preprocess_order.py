"""Views rendered together take their cut entries in another order than views
rendered alone, and a wave reads the SH records of its visible entries
together.  Both at the sizes where they can go wrong: one node to several runs
of nodes, 1 to 66 views, views that see everything, a part and nothing, and a
cut that outgrows the buffers of the render before.  The images of a batch are
those of its views alone to the last bit (per view the arithmetic and its
order are the same), and the colours of a sweep of visible counts are the
oracle's."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2406_12080_amd import synth
import parity as PR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _views(nv, tau):
    out = []
    for i in range(nv):
        a = 0.37 * i
        eye = (3 * np.cos(a), 3 * np.sin(a), 0.4)
        at = (0, 0, 0) if i % 5 != 3 else tuple(2 * np.asarray(eye))  # one in five looks away
        w, h = ((33, 17), (64, 40), (8, 8))[i % 3]
        out.append(synth.look_at(eye, at, (0, 0, 1), w, h, tau * (1 + i % 4)))
    return out


@pytest.mark.parametrize("n,nv,tau", [(1, 2, 0.0), (60, 3, 0.0), (700, 66, 0.0), (3000, 5, 1.0), (9000, 9, 0.0),
                                      (40000, 3, 0.5)])
def test_batch_equals_single_views(n, nv, tau):
    from paper_2406_12080_amd import hgs
    h = synth.build_hierarchy(synth.make_leaves(n, "cube", n))
    vs = _views(nv, tau)
    r = hgs.Renderer(0)
    try:
        r.upload(h)
        alone = [r.render([v])[0][0].clone() for v in vs]
        r.render(vs[:2])  # the batch's cut outgrows these buffers
        for _ in range(2):
            together, st = r.render(vs)
            for i, (a, b) in enumerate(zip(alone, together)):
                assert torch.equal(a, b), i
        assert st["cut"] >= nv
    finally:
        r.close()


@pytest.mark.parametrize("n", [1, 2, 15, 16, 17, 33, 47, 63, 64, 65, 130])
def test_colours_of_n_visible(n):
    from paper_2406_12080_amd import hgs
    lv = synth.make_leaves(n, "cube", n)
    lv["scale"] = lv["scale"] * np.float32(4.0)
    h = synth.build_hierarchy(lv)
    r = hgs.Renderer(0)
    try:
        r.upload(h)
        for tau in (0.0, 30.0):  # leaves only; interior nodes between their parents and children
            v = PR.safe_tau(h, synth.look_at((0, 0, 3), (0, 0, 0), (0, 1, 0), 40, 24, tau))
            o = O.render(h, v)
            (img,), _ = r.render([v])
            T = r.buffer(hgs.BUF_T_FINAL, torch.float32)
            res = PR.check_pixels(img.cpu().numpy().reshape(-1, 3).astype(np.float64),
                                  T.cpu().numpy().astype(np.float64), o)
            assert res["ok"], (tau, res)
    finally:
        r.close()
