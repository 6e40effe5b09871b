"""The macroscopic sums are the same bits whichever fields a call asks for, and
within the rounding of their reduction of the exact sums of the nodes' values:
boxes that are walked and boxes that are summed tile by tile, below and above
the workgroup counts of either."""
import ctypes
import math

import numpy as np
import pytest

from paper_1611_02445_amd import _abi
from paper_1611_02445_amd.lattice import _vp

from helpers import log, new_lattice

pytestmark = pytest.mark.gpu


def _solid(kind):
    rng = np.random.default_rng(5)
    if kind == "one tile":
        return np.zeros((4, 4, 4), np.uint8)
    if kind == "few tiles":
        return (rng.random((12, 20, 36)) < 0.4).astype(np.uint8)
    if kind == "porous":  # 28 x 20 x 22 tiles, ragged along x for groups of four
        return (rng.random((112, 80, 88)) < 0.5).astype(np.uint8)
    if kind == "nearly empty":  # 1 tile in 40, more groups than 4 times the tiles
        tiles = rng.random((50, 48, 52)) < 0.025
        return 1 - np.kron(tiles, np.ones((4, 4, 4))).astype(np.uint8)
    assert kind == "large"  # 2,700 groups of four tiles
    return (rng.random((120, 120, 192)) < 0.3).astype(np.uint8)


def _sums(lat, rho=None, u=None, name="lbm_macroscopic_buf"):
    sums = (ctypes.c_double * 8)()
    rc = getattr(_abi.lib(), name)(lat.ctx, None, _vp(rho), _vp(u), sums)
    return rc, np.array(sums[:])


@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("kind", ["one tile", "few tiles", "porous", "nearly empty", "large"])
def test_sums_do_not_depend_on_the_fields_asked_for(kind, storage):
    import torch
    log(f"[case] sums {kind} {storage}")
    lat = new_lattice(_solid(kind), 0.8, 7, storage=storage, model="inc" if storage == "f32" else "qc")
    lat.init(u0=(0.02, -0.01, 0.015))
    lat.set_force((2e-5, -1e-5, 3e-5))
    lat.step(3)
    box = lat.dense_shape
    rho = torch.full(box, 7.0, dtype=torch.float64, device=lat.device)
    u = torch.full((3,) + box, 7.0, dtype=torch.float64, device=lat.device)
    _, every = _sums(lat, rho, u)
    for fields in (dict(), dict(rho=torch.empty_like(rho)), dict(u=torch.empty_like(u))):
        for name in ("lbm_macroscopic_buf", "lbm_macroscopic_noalloc"):
            _, got = _sums(lat, name=name, **fields)
            assert np.array_equal(got.view(np.int64), every.view(np.int64)), (sorted(fields), name, got - every)
        for k, v in fields.items():
            assert torch.equal(v, {"rho": rho, "u": u}[k])
    # nodes outside the kept tiles read 0; the sums are those of the fields' values
    r, v = rho.cpu().numpy().ravel(), u.cpu().numpy().reshape(3, -1)
    assert np.count_nonzero(r) == lat.n_fluid == every[4]
    # additions that round: 6 in the butterfly, 3 over the waves, 6 in the tree over the rows, and one each
    # where a lane's and a column's sum take in what was kept beside them; and a product's own rounding
    eps = 2.0 ** -53
    for got, x, extra in [(every[0], r, 0)] + [(every[1 + a], r * v[a], 1) for a in range(3)] + [(every[7], v[0], 0)]:
        assert abs(got - math.fsum(x)) <= (17 + 1 + 2 * extra) * eps * math.fsum(np.abs(x))
    # |u| by numpy and by the device, each with a few roundings
    assert abs(every[5] - np.sqrt((v * v).sum(0)).max()) <= 8 * eps * every[5]
    assert every[6] == 0


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_sums_of_non_finite_values(bad):
    """A sum that meets an infinity is that infinity, as plain additions give it."""
    import torch
    solid = _solid("porous")
    lat = new_lattice(solid, 0.8, 7, model="inc")
    lat.init()
    f = lat.get_state()
    z, y, x = (int(c[11]) for c in np.nonzero(solid == 0))
    f[0, z, y, x] = bad  # rho is that, and u (c_0 = 0 times it) is NaN
    lat.set_state(f)
    rho = torch.empty(lat.dense_shape, dtype=torch.float64, device=lat.device)
    for fields in (None, rho):
        rc, s = _sums(lat, fields)
        assert rc == _abi.STATUS_CODE["LBM_E_NUMERIC"] and s[6] == 1
        assert (np.isnan(s[0]) if np.isnan(bad) else s[0] == bad) and np.isnan(s[7])
