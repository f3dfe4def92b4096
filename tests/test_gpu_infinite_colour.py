"""A splat whose colour is infinite (its SH sum overflows) belongs to the pixels
that blend it.  Every other pixel of its quarter, the finished ones behind an
opaque surface among them, is what a finite colour leaves it, to the bit."""
from __future__ import annotations

import numpy as np
import pytest

import scenes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TILES = [(8, 8, 64, 0), (16, 8, 128, 0), (16, 16, 256, 1), (32, 16, 512, 0)]
W = H = 40
F = 40.0
HUGE = 3.3e38


def _scene(splats):
    """Interior nodes (pixel x, pixel y, depth, peak alpha, red SH coefficient)
    that are a cut of their own: each with one leaf of the same size, under a
    root whose box holds the eye (t = 0).  Each is 0.05 px^2 wide, with the
    dilation 0.35, so that it takes pixels up to 2 px away."""
    n = len(splats)
    sp = np.array(splats, np.float64)
    z = sp[:, 2]
    x, y = (sp[:, 0] + 0.5 - W / 2) / F, (sp[:, 1] + 0.5 - H / 2) / F  # over z
    cov = 0.05 * np.array([[1 + x * x, x * y], [x * y, 1 + y * y]]).transpose(2, 0, 1)
    kappa = np.sqrt(np.linalg.det(cov) / np.linalg.det(cov + 0.3 * np.eye(2)))
    node = dict(mean=np.stack([x * z, y * z, z], 1), scale=np.repeat(np.sqrt(0.05) * z[:, None] / F, 3, 1),
                op=sp[:, 3] / kappa, sh=np.zeros((n, 48)))
    node["sh"][:, 0] = sp[:, 4]
    node["sh"][:, 1] = np.linspace(0.0, 1.0, n)
    node["sh"][:, [6, 18]] = np.where(sp[:, 4:5] >= HUGE, HUGE, 0.0)  # three coefficients whose sum overflows
    # root, the nodes, a leaf at the eye, the nodes' leaves
    a = {k: np.concatenate([v[:1], v, 0.0 * v[:1], v]) for k, v in node.items()}
    a["sh"][0] = 0.0
    return scenes.hierarchy([-1] + [0] * (n + 1) + list(range(1, n + 1)), a["mean"], np.maximum(a["scale"], 1e-3),
                            np.tile([1.0, 0, 0, 0], (2 * n + 2, 1)), a["op"], a["sh"])


def _render(h, tile):
    from paper_2406_12080_amd import hgs
    r = hgs.Renderer(0)
    r.upload(h)
    r.set_tuning(*tile)
    (img,), st = r.render([scenes.axis_view(W, H, F, tau=4.0)])
    assert st["cut"] == h.n_nodes // 2
    return r, img


@pytest.mark.parametrize("tile", TILES)
def test_image(tile):
    rng = np.random.default_rng(1)
    ground = [(x, y, 6.0 + 0.01 * rng.random(), 0.4, 0.5) for x in range(0, W, 2) for y in range(0, H, 2)]
    wall = [(x, y, 1.0 + 0.1 * k, 0.98, -0.2) for k in range(3) for x in range(18, 28) for y in range(16, 24)]
    at = [(5, 5), (14, 30), (17, 17), (28, 20), (33, 33)]  # the third and fourth beside the wall, behind it in part
    pictures = []
    for red in (1.0, 2.0, HUGE):
        r, img = _render(_scene(ground + wall + [(x, y, 4.0, 0.5, red) for x, y in at]), tile)
        pictures.append(img.cpu().numpy())
        r.close()
    one, two, inf = pictures
    touched = (one != two).any(2)
    assert 20 < touched.sum() < 200 and not touched[16:24, 18:28].any()
    assert np.isposinf(inf[..., 0][touched]).all()
    assert np.array_equal(inf[~touched], one[~touched])
    assert np.array_equal(inf[..., 1:][touched], one[..., 1:][touched])


@pytest.mark.parametrize("det", [False, True])
@pytest.mark.parametrize("tile", TILES)
def test_gradient(tile, det):
    """Pixel (16, 16) ends at the infinite splat, which no pixel of its quarter
    blends; splats on the quarter's far pixel, before and behind it, keep
    their gradients."""
    if det:
        tile = tile[:3] + (0,)
    from paper_2406_12080_amd import hgs
    got = []
    for red in (1.0, HUGE):
        h = _scene([(16, 16, 1.0, 2.0, 0.1), (16, 16, 1.1, 1.0 - 0.0108, 0.1), (19, 19, 2.0, 0.6, 0.7),
                    (15.2, 15.2, 3.0, 0.9, red), (19, 19, 4.0, 0.7, 0.3), (18, 18, 5.0, 0.7, 0.3)])
        r, img = _render(h, tile)
        try:
            r.set_deterministic(det)
            r.render([scenes.axis_view(W, H, F, tau=4.0)], out=[img])
            nb = r.buffer(hgs.BUF_N_BLEND, torch.int32).view(H, W)
            assert nb[16, 16] == 2 and nb[19, 19] >= 2
            assert bool(torch.isfinite(img[16:20, 16:20]).all())
            assert bool(torch.isfinite(img[15, 15]).all()) == (red < HUGE)
            g = {k: torch.zeros_like(t) for k, t in hgs.params_to_device(h).items()}
            dL = torch.ones_like(img)
            r.backward([dL], g)
            got.append({k: t.cpu().numpy() for k, t in g.items()})
        finally:
            r.close()
    for k in got[0]:
        for node in (3, 5, 6):
            a, b = got[0][k][node], got[1][k][node]
            assert np.isfinite(b).all(), (k, node)
            assert np.abs(a).max() > 0 or k == "rot", (k, node)
            assert np.allclose(a, b, rtol=1e-6, atol=1e-7 * np.abs(a).max()), (k, node)


def test_replayed():
    """Two views in one captured graph, the colour made infinite and finite again
    in place between the replays."""
    from paper_2406_12080_amd import hgs
    h = _scene([(x, y, 3.0 + 0.01 * x, 0.5, 0.5) for x in range(2, W, 5) for y in range(2, H, 5)])
    vs = [scenes.axis_view(W, H, F, tau=4.0), scenes.axis_view(W, H, F, tau=4.0, eye=(0.05, 0.0, 0.0))]
    r = hgs.Renderer(0)
    try:
        r.upload(h)
        P = hgs.params_to_device(h)
        r.bind(*[P[k] for k in hgs.PARAM_FIELDS])
        out = [torch.empty((H, W, 3), device="cuda") for _ in vs]
        sh = P["sh"].clone()
        pictures = []
        for huge in (False, True, False, True, True, False):
            P["sh"].copy_(sh)
            if huge:
                P["sh"][7, [0, 6, 18]] = HUGE
            r.render(vs, out=out)
            pictures.append([o.clone() for o in out])
        for k in range(2):
            a, b = pictures[0][k], pictures[1][k]
            inf = torch.isposinf(b[..., 0])
            assert 4 <= int(inf.sum()) <= 16
            assert torch.equal(a[~inf], b[~inf]) and torch.equal(a[..., 1:], b[..., 1:])
            for i, p in enumerate(pictures):
                assert torch.equal(p[k], pictures[1 if i in (1, 3, 4) else 0][k])
    finally:
        r.close()
