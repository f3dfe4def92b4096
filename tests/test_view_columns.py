"""Many view records at once take what one at a time takes and refuse what it
refuses, whatever the number: anything that float() accepts as an intrinsic."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2406_12080_amd import hgs, synth

torch = pytest.importorskip("torch")


def _views(n):
    return [synth.look_at((i + 0.1, 0.3, 3), (0, 0, 0), (0, 1, 0), 64 + i, 48, 1.0 + i) for i in range(n)]


SCALARS = {
    "one-element array": lambda x: np.array([x]),
    "0-d array": lambda x: np.array(x),
    "one-element tensor": lambda x: torch.tensor([x], dtype=torch.float64),
    "0-d tensor": lambda x: torch.tensor(x),
    "tensor with gradient": lambda x: torch.tensor(x, requires_grad=True),
    "text": str,
    "integer": int,
}


@pytest.mark.parametrize("n", [7, 8])
@pytest.mark.parametrize("every", [1, 3])
@pytest.mark.parametrize("kind", SCALARS)
@pytest.mark.filterwarnings("ignore::DeprecationWarning")
@pytest.mark.filterwarnings("ignore::UserWarning")
def test_scalars(kind, every, n):
    vs = _views(n)
    for i in range(0, n, every):
        f = SCALARS[kind]
        vs[i] = vs[i].replace(fx=f(vs[i].fx), cy=f(vs[i].cy), tau=f(vs[i].tau))
    one = (hgs.View * n)(*[hgs.make_view(v) for v in vs])
    assert bytes(hgs.make_views(vs)) == bytes(one)
