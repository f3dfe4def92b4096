"""Many view records at once take what one at a time takes and refuse what it
refuses, whatever the number: anything that float() accepts as an intrinsic,
and rotations and eyes of their own size only."""
from __future__ import annotations

from fractions import Fraction

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
    "double of numpy": np.float64,
    "fraction": Fraction,
}


@pytest.mark.parametrize("n", [7, 8, 15, 16, 24])
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


def _refused(vs, error=ValueError):
    with pytest.raises(error):
        [hgs.make_view(v) for v in vs]
    with pytest.raises(error):
        hgs.make_views(vs)


@pytest.mark.parametrize("n", [7, 8, 15, 16, 24])
@pytest.mark.parametrize("field", ["R", "eye"])
def test_sizes_that_add_up(field, n):
    """Records of the wrong size, n of the right size in all."""
    vs = _views(n)
    size = 9 if field == "R" else 3
    all_of = np.arange(n * size, dtype=np.float32)
    cut = size + 1  # the first a value too long, the second a value too short
    vs[0] = vs[0].replace(**{field: all_of[:cut]})
    vs[1] = vs[1].replace(**{field: all_of[cut:2 * size]})
    vs[2:] = [v.replace(**{field: all_of[:size]}) for v in vs[2:]]
    _refused(vs)


@pytest.mark.parametrize("n", [8, 16, 24])
def test_blocks_that_add_up(n):
    """The same with rotations of 2 and 4 rows."""
    vs = _views(n)
    vs[0] = vs[0].replace(R=np.ones((2, 3), np.float32))
    vs[1] = vs[1].replace(R=np.ones((4, 3), np.float32))
    _refused(vs)


@pytest.mark.parametrize("n", [7, 8, 15, 16, 24])
def test_whole_numbers_beyond_64_bits(n):
    vs = _views(n)
    vs[3] = vs[3].replace(width=2 ** 70 + 5)
    one = (hgs.View * n)(*[hgs.make_view(v) for v in vs])
    assert bytes(hgs.make_views(vs)) == bytes(one)


@pytest.mark.parametrize("n", [7, 8, 16, 24])
@pytest.mark.parametrize("bad,error", [(None, TypeError), ([1.0, 2.0], TypeError), (1j, TypeError), ("x", ValueError)])
def test_no_numbers(n, bad, error):
    vs = _views(n)
    vs[2] = vs[2].replace(fy=bad)
    _refused(vs, error)


@pytest.mark.parametrize("n", [7, 16])
@pytest.mark.parametrize("size", [64.9, "64", np.int32(64), np.float32(64.5), True, Fraction(129, 2)])
def test_image_sizes(n, size):
    """int() of whatever it is."""
    vs = _views(n)
    vs[1] = vs[1].replace(width=size)
    one = (hgs.View * n)(*[hgs.make_view(v) for v in vs])
    assert bytes(hgs.make_views(vs)) == bytes(one) and one[1].width == int(size)
