"""The backward's gather at the sizes where it can go wrong: nodes whose
children take up several 64-node mask words or straddle two, 1 to 130 views
(the views of a word are kept 64 to a mask), views that see nothing, and
splats behind opaque ones, which have no gradient row.  One view against the
oracle's gradients at the parity tests' bounds; the gradients of a batch
against the sum of its views' own."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2406_12080_amd import synth
import scenes as SC
from test_gpu_parity import _grad_case
from test_gpu_preprocess_order import _views

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _fans(counts):
    """A root with len(counts) children, the k-th of them with counts[k] leaves."""
    m = len(counts)
    parent = [-1] + [0] * m + [1 + k for k in range(m) for _ in range(counts[k])]
    n = len(parent)
    rng = np.random.default_rng(n)
    mean, scale, rot, op, sh = SC.random_params(rng, n, (0, 0, 6), 0.7, -2.2)
    return SC.hierarchy(parent, mean, scale, rot, op, sh)


@pytest.mark.parametrize("counts", [(1,), (60, 2), (61, 3, 64), (62, 65, 128), (3, 130, 1), (300, 5), (64, 64, 64)])
@pytest.mark.parametrize("tau", [0.05, 12.0])  # leaves (their parents' share through t), and the inner nodes
def test_children_over_words(counts, tau):
    _grad_case(_fans(counts), SC.axis_view(24, 18, 20.0, tau), seed=len(counts))


@pytest.mark.parametrize("nv", [2, 9, 64, 66, 130])
@pytest.mark.parametrize("opaque", [False, True])
def test_batch_is_the_sum_of_its_views(nv, opaque):
    from paper_2406_12080_amd import hgs
    n = 900
    lv = synth.make_leaves(n, "cube", n)
    if opaque:  # most of the visible splats reach no pixel
        lv["scale"] = lv["scale"] * np.float32(6.0)
        lv["opacity"] = np.full(n, 0.99, np.float32)
    h = synth.build_hierarchy(lv)
    vs = _views(nv, 2.0)
    gen = torch.Generator().manual_seed(nv)
    dL = [torch.randn((v.height, v.width, 3), generator=gen).cuda() for v in vs]
    r = hgs.Renderer(0)
    try:
        r.upload(h)
        zero = {k: torch.zeros_like(t) for k, t in hgs.params_to_device(h).items()}
        total = {k: torch.zeros_like(t, dtype=torch.float64) for k, t in zero.items()}
        size = {k: 0.0 for k in zero}
        for v, d in zip(vs, dL):
            g = {k: torch.zeros_like(t) for k, t in zero.items()}
            r.render([v])
            r.backward([d], g)
            for k in g:
                total[k] += g[k].double()
                size[k] += float(g[k].double().norm())
        for _ in range(3):  # the graph's first run and its replays
            g = {k: torch.zeros_like(t) for k, t in zero.items()}
            r.render(vs)
            r.backward(dL, g)
            for k in g:
                # FP32 sums of at most nv terms in another order, each addition
                # within 2^-24 of a partial sum (4: entries that cancel in a view)
                d = float((g[k].double() - total[k]).norm())
                assert d <= 4 * (nv + 4) * 2.0 ** -24 * size[k], (k, d, size[k])
    finally:
        r.close()
