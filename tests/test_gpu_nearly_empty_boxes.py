"""Dense arrays of boxes with few kept tiles are cleared and then filled tile by
tile: the launches (on a runtime without a device), and the values on both
sides of the rule."""
import numpy as np
import pytest

import fake_hip
from helpers import log, new_lattice, perturbed_state


def _solid(kept, box=(40, 48, 64)):
    """`kept` tiles of 10 x 12 x 16, scattered, with random nodes of them fluid."""
    rng = np.random.default_rng(kept)
    tz, ty, tx = (v // 4 for v in box)
    tiles = np.zeros(tx * ty * tz, bool)
    tiles[rng.choice(tiles.size, kept, replace=False)] = True
    fluid = np.kron(tiles.reshape(tz, ty, tx), np.ones((4, 4, 4), bool)) & (rng.random(box) < 0.6)
    return 1 - fluid.astype(np.uint8)


# 480 groups of four tiles
@pytest.mark.parametrize("kept,walked", [(1, False), (239, False), (240, True)])
def test_way_over_the_box(tmp_path, kept, walked):
    np.save(tmp_path / "solid.npy", _solid(kept))
    fake_hip.run(tmp_path, f"""
import ctypes
import numpy as np
c = context(np.load({str(tmp_path / 'solid.npy')!r}))
assert c.tiles.contents.n_tiles == {kept}
out = ctypes.c_void_p(1 << 42)
walked = {walked}
for args in (("lbm_get_state", c.ctx, None, out), ("lbm_adjoint_get", c.ctx, out, out),
             ("lbm_field_to_dense", c.ctx, out, 0, out), ("lbm_tiles_to_dense", c.ctx, out, 2, 1, out)):
    hip.notes()
    call(*args)
    n = hip.notes()
    assert len(n) == (1 if walked else 2), (args[0], n)
    assert walked or "k_fill" in n[0], n
    assert ("DenseWalk" if walked else "TileWalk") in n[-1], n
c.destroy()
""")


@pytest.mark.gpu
@pytest.mark.parametrize("kept", [1, 239, 240])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
def test_values(kept, storage):
    import torch
    log(f"[case] nearly empty {kept} {storage}")
    solid = _solid(kept)
    lat = new_lattice(solid, 0.7, 7, storage=storage)
    assert lat.n_tiles == kept
    rng = np.random.default_rng(1)
    fluid = solid == 0
    f = perturbed_state(solid, 1)
    lat.set_state(f)
    got = lat.get_state().cpu().numpy()
    if storage == "f64":
        assert bool(np.array_equal(got, f))
    else:  # what a second load and save keep is what the first kept
        assert float(np.abs(got - f).max()) < 1e-3 and not got[:, ~fluid].any()
        lat.set_state(got)
        assert np.array_equal(lat.get_state().cpu().numpy(), got)
    g = np.where(fluid, rng.standard_normal((3,) + fluid.shape), 0.0).astype(np.float32).astype(np.float64)
    lat.set_force(torch.from_numpy(g).cuda())
    dense = lat.field_to_dense(lat.force_buf, dtype=0 if storage == "f64" else 1)
    assert np.array_equal(dense.cpu().numpy(), g)
    buf = torch.arange(kept * 2 * 64, dtype=torch.float32, device="cuda") + 1.0
    dense = lat.tiles_to_dense(buf, 2, dtype=1).cpu().numpy()
    order = lat.tiling.device_order()
    xyz = lat.tiling.arrays()["tile_xyz"][order]
    want = np.zeros_like(dense)
    tiles = buf.cpu().numpy().reshape(kept, 2, 4, 4, 4)
    for t, (x, y, z) in enumerate(xyz):
        want[:, z:z + 4, y:y + 4, x:x + 4] = tiles[t]
    assert np.array_equal(dense, np.where(fluid, want, 0.0))
