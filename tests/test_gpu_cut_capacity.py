"""The cut's nodes are queued behind the scan without a look at its total on
the host: a buffer that is one entry short, or empty, stays as it was and the
size is reported; one of the exact size is filled to its last entry.  Both
entry points, over sizes around one block of 1024 nodes, with and without
weights."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

from paper_2406_12080_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaves", [1, 512, 513, 5000])
@pytest.mark.parametrize("entry", ["hgs_cut", "hgs_cut_noalloc"])
def test_a_cut_is_written_whole_or_not_at_all(leaves, entry):
    from paper_2406_12080_amd import hgs
    r = hgs.Renderer(0)
    try:
        r.upload(synth.make_scene(1, n_leaves=leaves))
        view = synth.make_views(1, tau=1.0)[0]
        hv = hgs.make_view(view)
        want_ids, want_t = r.cut(view)
        want_ids, want_t = want_ids.cpu().numpy(), want_t.cpu().numpy()
        n = want_ids.shape[0]
        assert n > 0
        for cap in sorted({0, n - 1, n, n + 3}):
            for weights in (True, False):
                ids = torch.full((n + 8,), -5, dtype=torch.int32, device="cuda")
                t = torch.full((n + 8,), -5.0, dtype=torch.float32, device="cuda")
                count = ctypes.c_int64(-1)
                status = getattr(r.L, entry)(r.h, ctypes.byref(hv), ctypes.c_void_p(ids.data_ptr()),
                                             ctypes.c_void_p(t.data_ptr() if weights else 0), cap,
                                             ctypes.byref(count))
                got_ids, got_t = ids.cpu().numpy(), t.cpu().numpy()
                assert count.value == n
                k = n if cap >= n else 0
                assert status == (0 if cap >= n else hgs.ERR_CAPACITY)
                assert np.array_equal(got_ids[:k], want_ids[:k]) and (got_ids[k:] == -5).all()
                k = k if weights else 0
                assert np.array_equal(got_t[:k], want_t[:k]) and (got_t[k:] == -5.0).all()
    finally:
        r.close()
