"""The cut's sweep, which skips runs of 64 nodes by the bounds of their
parents, against the oracle's top-down descent, node for node and for every
view of a batch: hierarchies of one node, of less than and just over one mask
word, and of many; 70 views in one batch (more than one group of 64), with
eyes inside the scene, beside it and far away, and tau from 0 upwards."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import oracle as O
from paper_2406_12080_amd import synth
import parity as PR

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 40, 46, 700, 3001])
def test_batched_cuts_match_oracle(n):
    from paper_2406_12080_amd import hgs
    h = synth.make_scene(1, n_leaves=n)
    rng = np.random.default_rng(n)
    views = []
    for k in range(70):
        far = (0.5, 1.5, 3.0, 40.0, 2000.0)[k % 5]
        eye = rng.normal(size=3)
        eye *= far / np.linalg.norm(eye)
        v = synth.look_at(eye, (0.01, 0.02, 0.0), (0, 1, 0), 16, 16, float(rng.choice([0.0, 0.05, 0.3, 1.0, 4.0])))
        views.append(PR.safe_tau(h, v))
    r = hgs.Renderer(0)
    try:
        r.upload(h)
        r.render(views)
        ids = r.buffer(hgs.BUF_CUT_IDS, torch.int32).cpu().numpy()
        t = r.buffer(hgs.BUF_CUT_T, torch.float64).cpu().numpy()
        base = r.buffer(hgs.BUF_CUT_BASE, torch.int32).cpu().numpy()
        for k, v in enumerate(views):
            oids, ot = O.cut(h, v)
            assert np.array_equal(ids[base[k]:base[k + 1]], oids), k
            assert np.abs(t[base[k]:base[k + 1]] - ot).max(initial=0) <= 1e-12
            one, _ = r.cut(v)
            assert np.array_equal(one.cpu().numpy(), oids), k
    finally:
        r.close()
