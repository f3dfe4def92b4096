"""Bound parameters that begin in the middle of a 16-byte word, as groups of one
flat buffer do: images and gradients are those of aligned arrays to the bit."""
from __future__ import annotations

import pytest

from paper_2406_12080_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _flat(P, off):
    """The arrays one behind the other in one buffer, each `off` floats past a
    multiple of 16 bytes."""
    room = torch.full((sum(t.numel() + 8 for t in P.values()),), 1e30, device="cuda")
    out, at = {}, 0
    for k, t in P.items():
        at = (at + 3) // 4 * 4 + off
        out[k] = room[at:at + t.numel()].view(t.shape)
        out[k].copy_(t)
        assert out[k].data_ptr() % 16 == 4 * off
        at += t.numel()
    return out


@pytest.mark.parametrize("views", [1, 3])
@pytest.mark.parametrize("off", [1, 2, 3])
def test_offsets(off, views):
    from paper_2406_12080_amd import hgs
    h = synth.make_scene(1, n_leaves=3001)
    vs = [synth.look_at((0.2 * i, 0.3, 3), (0, 0, 0), (0, 1, 0), 100, 70, 6.0) for i in range(views)]
    r = hgs.Renderer(0)
    got = []
    try:
        r.upload(h)
        r.set_deterministic(True)
        P = hgs.params_to_device(h)
        for Q in (P, _flat(P, off)):
            r.bind(*[Q[k] for k in hgs.PARAM_FIELDS])
            imgs, st = r.render(vs)
            assert st["visible"] > 500
            g = {k: torch.zeros_like(t) for k, t in P.items()}
            r.backward([torch.ones_like(i) for i in imgs], g)
            got.append((imgs, g))
    finally:
        r.close()
    for a, b in zip(got[0][0], got[1][0]):
        assert torch.equal(a, b) and float(a.abs().max()) > 0.0
    for k in got[0][1]:
        assert torch.equal(got[0][1][k], got[1][1][k]), k
