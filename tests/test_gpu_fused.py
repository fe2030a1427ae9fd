"""The one-kernel step against the separate passes, on the GPU.

A lattice of this size takes the fused layout unless a tile depth is asked for,
which the separate passes alone have.  Both round alike (kernels_fused.hpp), so
every field and population has to agree bitwise; only the diagnostic sums, taken
tile by tile, may differ by their FP64 summation order."""
from __future__ import annotations

import dataclasses

import numpy as np
import pytest

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def _separate(monkeypatch, lbm, wl, storage, **kw):
    """The same lattice as separate passes: a tile depth of its own selects them."""
    with monkeypatch.context() as m:
        m.setenv("LBM_TILE_Z", "2")
        return lbm.Lattice(wl, storage=storage, **kw)


def _same(x, y):
    """Equal everywhere; a run that has blown up has NaN at the same nodes."""
    return np.array_equal(x, y, equal_nan=True)


def _phys(wl, **kw):
    return dataclasses.replace(wl, phys=dataclasses.replace(wl.phys, **kw))


def _workloads():
    from paper_2512_01032_amd import inputs
    rs = inputs.random_small
    full = dict(walls=True, open_x=True, optimised_model=True)
    return {
        # tile widths 64, 32 and 16; one node past, one short of and exactly a tile
        "periodic_65x5x3": (rs(65, 5, 3, seed=21), {}),
        "periodic_48x17x2": (rs(48, 17, 2, seed=22), {}),
        "periodic_16x17x2": (rs(16, 17, 2, seed=22), {}),
        "periodic_96x8x1": (rs(96, 8, 1, seed=23), {}),
        "one_row_70x1x23": (rs(70, 1, 23, seed=24), {}),
        "one_column_1x21x23": (rs(1, 21, 23, seed=24), {}),
        "plain_walls_63x9x7": (rs(63, 9, 7, seed=25, walls=True), {}),
        "walls_faces_129x11x9": (rs(129, 11, 9, seed=26, **full), {}),
        "walls_faces_96x24x10": (rs(96, 24, 10, seed=27, **full), {"diag_every": 3}),
        "force_35x37x41": (_phys(rs(35, 37, 41, seed=28, **full), F_ex=(1e-6, -2e-6, 3e-6)), {}),
        "hysteresis_1": (_phys(rs(40, 12, 10, seed=29, **full), hysteresis=1), {}),
        "hysteresis_2": (_phys(rs(64, 12, 10, seed=30, walls=True, optimised_model=True), hysteresis=2), {}),
        "partial_slip": (_phys(rs(64, 12, 10, seed=31, walls=True, optimised_model=True), slip_factor=0.4), {}),
        "channel_2d": (inputs.channel_filling_2d(130, 18), {}),
        "ramped_duct": (inputs.constricted_duct(40, 40, 72, step_z=36, ramp_to=2e-4, slug_offset=0.3), {}),
    }


NAMES = ["periodic_65x5x3", "periodic_48x17x2", "periodic_16x17x2", "periodic_96x8x1", "one_row_70x1x23",
         "one_column_1x21x23", "plain_walls_63x9x7",
         "walls_faces_129x11x9", "walls_faces_96x24x10", "force_35x37x41", "hysteresis_1", "hysteresis_2",
         "partial_slip", "channel_2d", "ramped_duct"]


@pytest.mark.parametrize("storage", ["fp64", "fp32", "fp32_shift", "fp16_shift_g"])
@pytest.mark.parametrize("name", NAMES)
def test_fused_equals_separate_passes(name, storage, monkeypatch):
    require_gpu()
    from paper_2512_01032_amd import lbm
    wl, kw = _workloads()[name]
    a = lbm.Lattice(wl, storage=storage, **kw)
    b = _separate(monkeypatch, lbm, wl, storage, **kw)
    assert a.info()["footprint"] != b.info()["footprint"]
    state = None
    for n in (0, 1, 2, 18):
        a.step(n)
        b.step(n)
        for x, y, what in zip(a.fields() + a.pops(), b.fields() + b.pops(), ("phi", "P", "u", "h", "g")):
            assert _same(x, y), (name, storage, a.t, what)
        if a.t == 3:
            state = np.concatenate(a.pops())
    da, db = a.diagnostics(), b.diagnostics()
    for k in ("step", "u_max", "n_nan", "n_liq", "n_gas"):
        assert _same(da[k], db[k]), k
    # at most 6e4 terms: |sum - sum'| <= 6e4 2^-53 sum |x| < 1e-11 sum |x|, and phi
    # and P keep one sign
    for k in ("phi_sum", "P_liq_mean", "P_gas_mean"):
        assert abs(da[k] - db[k]) <= 1e-11 * abs(db[k]) or _same(da[k], db[k]), k
    # populations of an odd step, restored into either layout
    c = lbm.Lattice(wl, storage=storage, pops=state, step=3, **kw)
    d = _separate(monkeypatch, lbm, wl, storage, pops=state, step=3, **kw)
    c.step(5)
    d.step(5)
    for x, y in zip(c.pops(), d.pops()):
        assert _same(x, y), (name, storage, "restored")


def test_small_arena_takes_separate_passes():
    """An arena of the separate passes' size, where the fused layout needs more
    (no walls, rows of whole blocks), serves the lattice as before."""
    require_gpu()
    import torch
    from paper_2512_01032_amd import inputs, lbm
    wl = inputs.random_small(64, 12, 10, seed=33)
    tiny = torch.zeros(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(lbm.LbmError) as e:
        lbm.Lattice(wl, storage="fp32_shift", arena=(tiny.data_ptr(), 256))
    size = int(str(e.value).rsplit(None, 1)[1])
    arena = torch.zeros(size, dtype=torch.uint8, device="cuda")
    a = lbm.Lattice(wl, storage="fp32_shift")
    b = lbm.Lattice(wl, storage="fp32_shift", arena=(arena.data_ptr(), size))
    assert b.info()["footprint"] == size < a.info()["footprint"]
    a.step(19)
    b.step(19)
    for x, y in zip(a.pops(), b.pops()):
        assert _same(x, y)
    b.close()


@pytest.mark.parametrize("storage,nx,ny,nz", [("fp32_shift", 130, 131, 133), ("fp16_shift_g", 160, 149, 131),
                                              ("fp64", 96, 101, 118)])
def test_tiles_both_ways(storage, nx, ny, nz, monkeypatch):
    """Lattices beyond the Infinity Cache (more than 285 MB of populations), whose
    tiles run plane by plane, backwards on odd steps: every tile once a step, and
    the parts of a plane that do not divide by eight."""
    require_gpu()
    from paper_2512_01032_amd import inputs, lbm
    wl = inputs.random_small(nx, ny, nz, seed=34, walls=True, open_x=True, optimised_model=True, u_amp=0.002)
    a = lbm.Lattice(wl, storage=storage)
    b = _separate(monkeypatch, lbm, wl, storage)
    for n in (1, 2, 18):
        a.step(n)
        b.step(n)
        for x, y, what in zip(a.fields(), b.fields(), ("phi", "P", "u")):
            assert _same(x, y), (storage, a.t, what)
