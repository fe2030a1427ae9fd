"""Which layout a lattice takes, and lattices at the edges of the rules, on the GPU."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest

from tests.gpu_util import require_gpu
from tests.test_gpu_walls_rounding import porous

pytestmark = pytest.mark.gpu


def separate(monkeypatch, wl, storage, tile_z=2, **kw):
    """The lattice as separate passes: a tile depth of its own selects them."""
    from paper_2512_01032_amd import lbm
    with monkeypatch.context() as m:
        m.setenv("LBM_TILE_Z", str(tile_z))
        return lbm.Lattice(wl, storage=storage, **kw)


def is_fused(lat, sep):
    """The two layouts differ in footprint."""
    return lat.info()["footprint"] != sep.info()["footprint"]


@pytest.mark.parametrize("shape,storage,fused", [
    ((64, 64, 64), "fp64", True),         # within the Infinity Cache
    ((104, 104, 104), "fp64", False),     # 297 MB of populations
    ((128, 128, 128), "fp32_shift", True),
    ((130, 131, 129), "fp32_shift", True),      # beyond the cache, up to 3 GB
    ((160, 160, 130), "fp16_shift_g", False),   # 313 MB
])
def test_hysteresis_layout(shape, storage, fused, monkeypatch):
    """Lattices with contact-angle hysteresis beyond the cache take the separate passes,
    where their history entries are hidden behind other waves, but for FP32."""
    require_gpu()
    from paper_2512_01032_amd import lbm
    wl = porous(*shape, 0.1, 7, hysteresis=1)
    a = lbm.Lattice(wl, storage=storage)
    b = separate(monkeypatch, wl, storage)
    assert is_fused(a, b) == fused
