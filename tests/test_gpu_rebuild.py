"""Builds one after the other in one renderer, whose buffers a build of the
same counts writes over: the same leaves again, others of the same number,
fewer and more, after an upload, after parameters were bound, after a build
that was refused, and with work of the hierarchy before still queued on
another stream.  Every build and its image equal those of a renderer of its
own to the bit."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2406_12080_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

VIEWS = [synth.look_at((0.3 * i, 0, 3), (0, 0, 0), (0, 1, 0), 40, 24, 2.0) for i in range(3)]


def _state(r):
    d = r.download(leaf_src=True)
    imgs, _ = r.render(VIEWS)
    return d, [i.cpu().numpy() for i in imgs]


def _fresh(leaves):
    from paper_2406_12080_amd import hgs
    r = hgs.Renderer(0)
    try:
        r.build(leaves)
        return _state(r)
    finally:
        r.close()


def _same(a, b):
    assert a[0].keys() == b[0].keys()
    for k in a[0]:
        assert np.array_equal(np.asarray(a[0][k]), np.asarray(b[0][k])), k
    assert all(np.array_equal(x, y) for x, y in zip(a[1], b[1]))


@pytest.mark.parametrize("n", [1, 2, 65, 1000])
def test_builds_in_turn(n):
    from paper_2406_12080_amd import hgs
    A, B = synth.make_leaves(n, "cube", 1), synth.make_leaves(n, "cube", 2)
    C = {k: (v * np.float32(0.5) if k in ("pos", "scale") else v).copy() for k, v in A.items()}  # A's tree
    D = synth.make_leaves(3 * n + 5, "cube", 4)
    want = {k: _fresh(v) for k, v in dict(A=A, B=B, C=C, D=D).items()}
    r = hgs.Renderer(0)
    try:
        for name, lv in (("A", A), ("A", A), ("C", C), ("D", D), ("B", B), ("C", C), ("A", A)):
            dev = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in lv.items()}
            r.build(dev if name == "C" else lv)
            _same(_state(r), want[name])
        P = {k: torch.zeros((r.n_nodes, c) if c > 1 else r.n_nodes, device="cuda")
             for k, c in dict(mean=3, scale=3, rot=4, opacity=1, sh=48).items()}
        r.bind(*[P[k] for k in ("mean", "scale", "rot", "opacity", "sh")])
        r.build(C)
        _same(_state(r), want["C"])
        with pytest.raises(hgs.HgsError):
            r.build({k: v[:0] for k, v in A.items()})
        if n > 1:
            bad = {k: v.copy() for k, v in A.items()}
            bad["pos"][0, 0] = np.inf
            with pytest.raises(hgs.HgsError):
                r.build(bad)
        r.build(A)
        _same(_state(r), want["A"])
        r.upload(synth.make_scene(1, n_leaves=70))
        r.build(C)
        _same(_state(r), want["C"])
        # a backward of the hierarchy before still queued
        s = torch.cuda.Stream()
        r._check(r.L.hgs_set_stream(r.h, s.cuda_stream))
        imgs, _ = r.render(VIEWS)
        g = {k: torch.zeros_like(P[k]) for k in P}
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            r.backward([torch.ones_like(i) for i in imgs], g)
        r._check(r.L.hgs_set_stream(r.h, torch.cuda.current_stream().cuda_stream))
        r.build(A)
        _same(_state(r), want["A"])
    finally:
        r.close()
