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


@pytest.mark.parametrize("storage", ["fp64", "fp32_shift"])
@pytest.mark.parametrize("shape,tiles", [
    ((64, 1, 40), 40),       # one row: tiles of 64 x 4, not of 32 x 8
    ((130, 6, 20), 100),     # 160 x 8 lanes in tiles of 32 x 8, 144 x 16 in narrower ones
    ((2, 2, 50), 50),        # equal lanes at every width: the narrowest
    ((96, 16, 10), 60),      # 3 x 2 tiles of 32 x 8
])
def test_idle_rows_count(shape, tiles, storage, monkeypatch):
    """Tiles of flat lattices leave few rows idle, and step like the separate passes."""
    require_gpu()
    from paper_2512_01032_amd import inputs, lbm
    wl = inputs.random_small(*shape, seed=9, u_amp=2e-4, optimised_model=True)
    a = lbm.Lattice(wl, storage=storage)
    b = separate(monkeypatch, wl, storage)
    assert a.info()["n_tiles"] == tiles
    for n in (1, 4):
        a.step(n)
        b.step(n)
        for x, y in zip(a.fields() + a.pops(), b.fields() + b.pops()):
            assert np.isfinite(y).all()
            assert np.array_equal(x, y)


@pytest.mark.parametrize("storage,shape,beyond", [
    ("fp32_shift", (120, 120, 120), False),    # 228 MB of populations in 243 MB of lines
    ("fp32_shift", (128, 128, 128), True),     # 277 MB
    ("fp32_shift", (17, 256, 256), True),      # 147 MB in 277 MB
    ("fp16_shift_g", (128, 128, 128), False),  # 197 MB
    ("fp16_shift_g", (33, 200, 300), True),    # 186 MB in 307 MB
])
def test_lines_beyond_the_cache(storage, shape, beyond, monkeypatch):
    """Lattices whose cache lines, not only whose populations, exceed the Infinity Cache
    take its tile order and read pass (whose second tile list shows in the footprint
    of a lattice without walls) and step like the separate passes."""
    require_gpu()
    from paper_2512_01032_amd import inputs, lbm
    z, y, x = np.ogrid[:shape[2], :shape[1], :shape[0]]
    r = np.sqrt((x - 0.5 * shape[0]) ** 2 + (y - 60.3) ** 2 + (z - 58.1) ** 2)
    wl = inputs.Workload("droplet", *shape, inputs.Physics(nu_g=0.1), inputs.tanh_profile(r - 7.0, 4.0))
    a = lbm.Lattice(wl, storage=storage)
    b = separate(monkeypatch, wl, storage)
    sh, sg = 4, 2 if storage == "fp16_shift_g" else 4
    info = a.info()
    row = [w for w in (64, 32, 16) if -(-shape[0] // w) * -(-shape[1] // (256 // w)) * shape[2] == info["n_tiles"]][0]
    up = lambda v: -(-v // 256) * 256
    n, nt = wl.n_nodes, info["n_tiles"]
    plain = 2 * up(-(-shape[0] // row) * row * shape[1] * shape[2] * 7 * sh)
    plain += up(-(-shape[0] // 64) * 64 * shape[1] * shape[2] * 19 * sg) + up(n) + up(4 * n) + up(32 * nt) + up(80 * nt)
    second = up(32 * (nt // shape[2]) * -(-shape[2] // 8))
    extra = info["footprint"] - plain
    assert (extra >= second) == beyond, (extra, second)
    for k in (1, 2, 8):
        a.step(k)
        b.step(k)
        for x, y in zip(a.fields(), b.fields()):
            assert np.isfinite(y).all()
            assert np.array_equal(x, y)


@pytest.mark.parametrize("diag_every", [0, 20])
@pytest.mark.parametrize("first", [0, 3])
def test_long_calls_replay_graphs(first, diag_every):
    """Calls of 64 steps and more replay 16-step graphs, from either parity and between
    diagnostic steps, shorter ones launch every step: the same state."""
    require_gpu()
    from paper_2512_01032_amd import inputs, lbm
    wl = inputs.static_droplet(n=24, R=7.0)
    a = lbm.Lattice(wl, storage="fp32_shift", diag_every=diag_every)
    b = lbm.Lattice(wl, storage="fp32_shift", diag_every=diag_every)
    a.step(first)
    a.step(83)
    a.step(64)
    for n in (first, 63, 20, 63, 1):
        b.step(n)
    assert a.t == b.t
    for x, y in zip(a.pops(), b.pops()):
        assert np.isfinite(y).all()
        assert np.array_equal(x, y)


@pytest.mark.parametrize("storage", ["fp64", "fp32_shift", "fp16_shift_g"])
@pytest.mark.parametrize("nx", [1, 16, 17, 33, 48, 49, 52, 56, 65, 97, 104, 113, 129])
def test_footprint_is_a_bound(nx, storage):
    """lbm_footprint bounds what a lattice takes in the layout it is given: rows a little
    past a tile or a block, without walls and with a wall link at almost every node."""
    require_gpu()
    from paper_2512_01032_amd import inputs, lbm
    for wl in (inputs.random_small(nx, 9, 8, seed=3), porous(nx, 40, 38, 0.3), porous(nx, 40, 38, 0.3, hysteresis=1)):
        lat = lbm.Lattice(wl, storage=storage)
        assert lat.info()["footprint"] <= lbm.footprint(wl, storage), wl.name


@pytest.mark.parametrize("storage,ny,nz", [("fp32_shift", 200, 300), ("fp16_shift_g", 220, 330)])
def test_footprint_bounds_narrow_porous_lattices(storage, ny, nz, monkeypatch):
    """Beyond the cache, rows of 33 in tiles of 64 with a wall link at almost every node
    would exceed the bound: they take narrower tiles, and step like the separate passes."""
    require_gpu()
    from paper_2512_01032_amd import lbm
    wl = porous(33, ny, nz, 0.2)
    a = lbm.Lattice(wl, storage=storage)
    b = separate(monkeypatch, wl, storage)
    assert a.info()["footprint"] <= lbm.footprint(wl, storage)
    for n in (1, 2):
        a.step(n)
        b.step(n)
        for x, y in zip(a.fields(), b.fields()):
            assert np.isfinite(y).all()
            assert np.array_equal(x, y)


def test_timing_of_the_one_kernel_step(monkeypatch):
    """A lattice in the fused layout has no phi pass to time."""
    require_gpu()
    from paper_2512_01032_amd import inputs, lbm
    wl = inputs.static_droplet(n=24, R=7.0)
    a, b = lbm.Lattice(wl, storage="fp32_shift"), separate(monkeypatch, wl, "fp32_shift")
    for lat, phi_pass in ((a, False), (b, True)):
        lat.set_timing()
        lat.step(6)
        phi_ms, sweep_ms, steps = lat.get_timing()
        assert steps == 6 and sweep_ms > 0.0
        assert (phi_ms > 0.0) == phi_pass
