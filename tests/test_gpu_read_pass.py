"""Read-backs of fused-layout lattices beyond the Infinity Cache, whose read pass has
kernels and tiles of its own, against the separate passes: bitwise."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_util import require_gpu
from tests.test_gpu_walls_rounding import porous

pytestmark = pytest.mark.gpu


def _pair(monkeypatch, wl, storage, **kw):
    from paper_2512_01032_amd import lbm
    a = lbm.Lattice(wl, storage=storage, **kw)
    with monkeypatch.context() as m:
        m.setenv("LBM_TILE_Z", "2")   # a tile depth of its own selects the separate passes
        b = lbm.Lattice(wl, storage=storage, **kw)
    return a, b


def _workload(name):
    from paper_2512_01032_amd import inputs
    # 264 bytes of FP64, 132 of FP32 and 94 of FP16 g populations a node: more than
    # 285 MB each; depths that leave a short last tile
    if name == "porous":
        return porous(97, 105, 108, 0.15, 6)
    if name == "hysteresis":
        return porous(130, 131, 129, 0.1, 7, hysteresis=1)
    return inputs.static_droplet(n=147, R=37.3)


@pytest.mark.parametrize("name,storage", [("porous", "fp64"), ("hysteresis", "fp32_shift"), ("droplet", "fp32_shift"),
                                          ("droplet", "fp16_shift_g")])
def test_read_pass_equals_separate_passes(name, storage, monkeypatch):
    require_gpu()
    wl = _workload(name)
    a, b = _pair(monkeypatch, wl, storage)
    assert a.info()["footprint"] != b.info()["footprint"]
    state = None
    for n in (0, 1, 2):
        a.step(n)
        b.step(n)
        for mask in (1 | 2 | 4, 8, 16):
            x, y = a.read(mask), b.read(mask)
            for k in x:
                assert np.isfinite(y[k]).all(), (k, a.t)
                assert np.array_equal(x[k], y[k]), (k, a.t)
        da, db = a.diagnostics(), b.diagnostics()
        for k in ("step", "u_max", "n_nan", "n_liq", "n_gas"):
            assert da[k] == db[k], k
        # at most 3.1e6 terms: |sum - sum'| <= 3.1e6 2^-53 sum |x| < 1e-9 sum |x|
        for k in ("phi_sum", "P_liq_mean", "P_gas_mean"):
            assert abs(da[k] - db[k]) <= 1e-9 * abs(db[k]), k
        if a.t == 1:
            state = np.concatenate(a.pops())
    # reading has disturbed neither lattice; a restored one records the wall history in
    # its read pass
    a.step(3)
    b.step(3)
    c, d = _pair(monkeypatch, wl, storage, pops=state, step=1)
    for lat in (c, d):
        lat.step(3)
    for x, y in zip(a.pops() + c.pops(), b.pops() + d.pops()):
        assert np.array_equal(x, y)
