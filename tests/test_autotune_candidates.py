"""The blend kernels differ by tile and work distribution only, whatever the
batch: the autotuner times each of them once and keeps the fastest."""
from __future__ import annotations

import time

import pytest

from paper_2406_12080_amd.autotune import CANDIDATES, autotune

torch = pytest.importorskip("torch")


class _Renderer:
    def __init__(self):
        self.set, self.steps = [], 0

    def set_tuning(self, *t):
        self.set.append(t)

    def step(self):
        self.steps += 1
        if self.set[-1][:2] != (16, 8) or self.set[-1][3]:
            time.sleep(0.002)


@pytest.mark.parametrize("candidates", [None, ((16, 16, 512, 0), (16, 8, 256, 0), (16, 8, 128, 0), (16, 16, 256, 1))])
def test_every_kernel_is_timed_once(monkeypatch, candidates):
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    r = _Renderer()
    out = autotune(r, [], r.step, reps=2) if candidates is None else autotune(r, [], r.step, 2, candidates)
    want = {(tw, th, p) for tw, th, _, p in (CANDIDATES if candidates is None else candidates)}
    timed = [(tw, th, p) for tw, th, _, p in r.set[:-1]]
    assert sorted(timed) == sorted(want)
    assert r.steps == 3 * len(want) == 3 * len(out["ms"])
    assert r.set[-1] == (out["tile_w"], out["tile_h"], out["batch"], out["persistent"])
    assert (out["tile_w"], out["tile_h"], out["persistent"]) == (16, 8, 0)
    assert r.set[-1] in (CANDIDATES if candidates is None else candidates)
