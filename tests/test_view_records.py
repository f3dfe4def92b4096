"""The view records that go to the library: many at once are the same bytes as
one at a time, below and from the number on where they are filled by column,
for arrays, lists, flat and square rotations and values beyond FP32."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2406_12080_amd import hgs, synth


@pytest.mark.parametrize("n", [1, 7, 8, 9, 65])
@pytest.mark.parametrize("kind", ["arrays", "lists", "mixed", "wide"])
def test_records(n, kind):
    vs = []
    for i in range(n):
        v = synth.look_at((i + 0.1, 0.3, 3), (0, 0, 0), (0, 1, 0), 64 + i, 48, 1.0 + i)
        if kind == "lists" or (kind == "mixed" and i % 2):
            v = v.replace(R=v.R.reshape(9).tolist(), eye=list(v.eye))
        if kind == "wide":
            v = v.replace(R=v.R.astype(np.float64), fx=1e39, cy=np.float32(2.5), tau=1e-50)
        vs.append(v)
    one = (hgs.View * n)(*[hgs.make_view(v) for v in vs])
    assert bytes(hgs.make_views(vs)) == bytes(one)
