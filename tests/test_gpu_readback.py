"""Read-backs above and below the size from which they go through pinned chunks,
against the plain copies of lbm_read_fields_noalloc, and chunk tails: bitwise."""
from __future__ import annotations

import threading

import numpy as np
import pytest

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

PHI, ALL = 1, 1 | 2 | 4 | 8 | 16


@pytest.mark.parametrize("shape,mask", [
    ((64, 64, 50), ALL),      # 31 rows of 1.6 MB: copies of less and of more than a chunk
    ((70, 71, 43), ALL),      # odd sizes
    ((128, 96, 85), PHI),     # 8.36 MB: just above the limit
    ((128, 96, 85), PHI | 4),
    ((64, 64, 17), PHI),      # plain copies
])
def test_chunked_read_back(shape, mask):
    require_gpu()
    from paper_2512_01032_amd import inputs, lbm
    lat = lbm.Lattice(inputs.random_small(*shape, seed=41, u_amp=0.002), storage="fp32_shift")
    lat.step(3)
    bits = [b for b in (1, 2, 4, 8, 16) if mask & b]
    got = lat.read(mask)
    # one array at a time fits the fixed staging of the other call
    for b in bits:
        if b in (8, 16):
            continue
        name = {1: "phi", 2: "P", 4: "u"}[b]
        one = lat.read(b, noalloc=True)
        assert np.array_equal(got[name], one[name]), name
    if mask & 24:
        h, g = lat.pops()
        assert np.array_equal(got["pops"], np.concatenate([h, g]))
        # phi = sum_i h_i: every row has come to its place
        assert np.abs(h.sum(axis=0) - got["phi"]).max() < 1e-5


def test_chunked_read_back_from_threads():
    """Two lattices read at the same time by two threads, and again in turn."""
    require_gpu()
    from paper_2512_01032_amd import inputs, lbm
    lats = [lbm.Lattice(inputs.random_small(96, 96, 50, seed=s, u_amp=0.002), storage="fp32_shift") for s in (42, 43)]
    for lat in lats:
        lat.step(2)
    out = [None, None]

    def run(k):
        out[k] = lats[k].fields()
    ts = [threading.Thread(target=run, args=(k,)) for k in (0, 1)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in (0, 1):
        for x, y in zip(out[k], lats[k].fields()):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("pinned", ["phi", "u", "phi u"])
def test_pinned_destination(pinned):
    """Destinations in pinned memory take plain copies, beside pageable ones in chunks."""
    require_gpu()
    import torch
    from paper_2512_01032_amd import inputs, lbm
    lat = lbm.Lattice(inputs.random_small(128, 96, 87, seed=44, u_amp=0.002), storage="fp32_shift")
    lat.step(2)
    want = lat.read(PHI | 4, noalloc=True)
    out = {k: torch.full(want[k].shape, 7.0, dtype=torch.float64, pin_memory=k in pinned) for k in want}
    lbm.check(lbm.lbm_read_fields(lat.h, PHI | 4, out["phi"].data_ptr(), None, out["u"].data_ptr(), None))
    for k in want:
        assert out[k].is_pinned() == (k in pinned)
        assert np.array_equal(out[k].numpy(), want[k]), k
