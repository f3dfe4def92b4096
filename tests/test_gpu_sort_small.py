"""The sort of a small list in one workgroup (at most 8192 pairs) against the
passes over many: the same views from a renderer whose buffers are small and
from one whose buffers a larger scene has grown.  Both sorts are stable, so
the images are the same bit for bit.  Sizes around a wave, the workgroup's
1024 lanes and the limit; several views, some of which see nothing; the
generation's sorts of 8192 leaves against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2406_12080_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def grown():
    from paper_2406_12080_amd import hgs
    r = hgs.Renderer(0)
    r.upload(synth.make_scene(1, n_leaves=9000))  # room for 9000 entries at the first render
    r.render([synth.make_views(1, tau=4.0)[0]])
    yield r
    r.close()


# leaves, views: the first render makes room for leaves x views entries
@pytest.mark.parametrize("leaves,views", [(1, 1), (64, 1), (65, 3), (1025, 1), (2000, 4), (8192, 1)])
def test_small_lists_sort_alike(grown, leaves, views):
    from paper_2406_12080_amd import hgs
    h = synth.make_scene(1, n_leaves=leaves)
    vs = [synth.look_at((3 * np.cos(a), 0.3, 3 * np.sin(a)), (0, 0, 0), (0, 1, 0), 120, 88, 0.5) for a in range(views)]
    if views > 1:
        vs[1] = synth.look_at((0, 0, 5), (0, 0, 9), (0, 1, 0), 120, 88, 0.5)  # looks away
    small = hgs.Renderer(0)
    try:
        small.upload(h)
        a = [o.clone() for o in small.render(vs)[0]]
    finally:
        small.close()
    grown.upload(h)
    b = grown.render(vs)[0]
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    assert float(a[0].abs().max()) > 0.0


def test_generation_at_the_limit():
    from paper_2406_12080_amd import hgs
    lv = synth.make_leaves(8192, "cube", 7)
    r = hgs.Renderer(0)
    try:
        r.build(lv)
        g = r.download(leaf_src=True)
    finally:
        r.close()
    o = O.build_hierarchy(lv)
    for k in ("parent", "child_begin", "child_count", "leaf_src", "bmin", "bmax"):
        assert np.array_equal(g[k], o[k]), k
