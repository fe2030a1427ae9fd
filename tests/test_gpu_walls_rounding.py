"""Rounding of the near-wall arithmetic, on the GPU.

A porous medium has wall normals and corner nodes of every kind.  The digests in
tests/golden/porous_digests.json are those of the library whose wall pass was first
held to the oracle; the populations have to stay bitwise the same in either layout, as
the sign term of the mobility correction and the regularised unit vectors turn a
last-bit difference into a visible one within tens of steps."""
from __future__ import annotations

import hashlib
import json
import os

import numpy as np
import pytest

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "porous_digests.json")
OPTIONS = {"plain": {}, "hysteresis_1": {"hysteresis": 1}, "hysteresis_2": {"hysteresis": 2},
           "slip_0.3": {"slip_factor": 0.3}, "d3q19": {"q_phase": 19}}


def porous(nx=33, ny=20, nz=18, fraction=0.3, seed=4, **phys):
    """Solid nodes of three materials at random between pressure faces along z; every
    input is formed by additions, products and comparisons alone, so it is the same on
    every host."""
    import dataclasses
    from paper_2512_01032_amd import inputs
    rng = np.random.default_rng(seed)
    solid = (rng.random((nz, ny, nx)) < fraction).astype(np.uint8)
    solid[solid > 0] = 1 + (rng.random(int(solid.sum())) * 3).astype(np.uint8)
    solid[:3], solid[-3:] = 0, 0
    z = np.arange(nz, dtype=np.float64)[:, None, None]
    phi = np.clip((0.4 * nz - z) * 0.25 + 0.5 + 0.01 * (rng.random((nz, ny, nx)) - 0.5), 0.0, 1.0)
    ph = dataclasses.replace(inputs.optimised(inputs.Physics(nu_g=0.1)), **phys)
    faces = (None,) * 4 + ((ph.P_ref + 1e-4, 1e-6), (ph.P_ref, 0.0))
    return inputs.Workload("porous", nx, ny, nz, ph, phi, solid=solid, faces=faces,
                           theta_deg=(60.0, 100.0, 35.0) + (90.0,) * 13)


def digest(lat):
    h = hashlib.sha256()
    for a in lat.pops():
        assert np.isfinite(a).all()
        h.update(np.ascontiguousarray(a + 0.0).tobytes())
    return h.hexdigest()[:24]


@pytest.mark.parametrize("layout", ["default", "separate"])
@pytest.mark.parametrize("storage", ["fp64", "fp32_shift", "fp16_shift_g"])
@pytest.mark.parametrize("option", sorted(OPTIONS))
def test_porous_populations(option, storage, layout, monkeypatch):
    require_gpu()
    from paper_2512_01032_amd import lbm
    if layout == "separate":
        monkeypatch.setenv("LBM_TILE_Z", "2")   # a tile depth of its own selects the separate passes
    lat = lbm.Lattice(porous(**OPTIONS[option]), storage=storage)
    lat.step(7)
    with open(GOLDEN) as f:
        want = json.load(f)["digests"]
    assert digest(lat) == want["%s/%s" % (option, storage)]
