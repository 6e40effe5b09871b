"""Grids whose tiles are nearly all full: staging steps ask for LDS that holds
fewer waves on a compute unit (the launches, on a runtime without a device),
and store the same bytes."""
import numpy as np
import pytest

import fake_hip
from helpers import log, new_lattice
from test_gpu_staged_stores import _buffers, _check


def _box(kind):
    """24^3 tiles: all full; 60 of 64 nodes fluid; or 22^3 full ones."""
    solid = np.zeros((88, 88, 88) if kind == "small" else (96, 96, 96), np.uint8)
    if kind == "porous":
        solid[::4, ::4, :] = 1
    if kind == "walled":  # 62.7 of 64 nodes
        solid[0], solid[:, 0] = 1, 1
    return solid


# LDS bytes of a workgroup: 160 KB shared by as many as hold the waves, in units of 1280, at most 64 KB
@pytest.mark.parametrize("kind,storage,model,tpw,step,adjoint", [
    ("full", 0, 0, 0, 53760, 65536),     # 12 and 8 waves in workgroups of 4
    ("full", 0, 1, 1, 12800, 20480),
    ("full", 0, 0, 2, 26880, 40960),
    ("full", 0, 0, 8, 0, 0),             # 8 FP64 tiles do not fit the 64 KB
    ("full", 0, 2, 0, 53760, None),
    ("full", 1, 0, 0, 32000, 32000),     # 20 waves
    ("full", 1, 3, 1, 7680, 7680),
    ("full", 1, 0, 8, 65536, 65536),
    ("full", 2, 0, 0, 9728, None),       # 4 FP16 tiles: no limit
    ("walled", 0, 0, 0, 53760, 65536),
    ("walled", 0, 3, 0, 38912, None),    # 4 tiles
    ("walled", 1, 2, 0, 32000, 32000),
    ("porous", 0, 0, 0, 38912, 38912),
    ("porous", 1, 0, 0, 19456, 19456),
    ("small", 0, 0, 0, 38912, 38912),
    ("small", 1, 0, 0, 19456, 19456),
])
def test_lds_asked_for(tmp_path, kind, storage, model, tpw, step, adjoint):
    np.save(tmp_path / "solid.npy", _box(kind))
    fake_hip.run(tmp_path, f"""
import ctypes
import numpy as np
c = context(np.load({str(tmp_path / 'solid.npy')!r}), storage={storage}, model={model}, tiles_per_wg={tpw})
a, b, g = (ctypes.c_void_p(k << 40) for k in (4, 5, 6))
def lds(*args):
    hip.notes()
    call(*args)
    (n,) = hip.notes()
    return int(n.split()[3])
assert lds("lbm_step", c.ctx, 1) == {step}
if {model} == 0:  # the measurement kernels take the shape of an LBGK step
    assert lds("lbm_calib_step", c.ctx, 1, a, b) == lds("lbm_calib_step", c.ctx, 2, a, b) == {step}
if {adjoint} is not None:
    assert lds("lbm_adjoint_step", c.ctx, c.state[0], a, b, g) == {adjoint}
c.destroy()
""")


# 24^3 tiles with `nodes` fluid nodes each
@pytest.mark.parametrize("nodes,storage,model,lds", [(50, 0, 2, 9728), (50, 0, 3, 9728), (51, 0, 2, 0), (64, 0, 3, 0),
                                                     (51, 0, 0, 38912), (51, 1, 2, 19456)])
def test_mrt_adjoint_stores_directly(tmp_path, nodes, storage, model, lds):
    tile = (np.arange(64) >= nodes).astype(np.uint8).reshape(4, 4, 4)
    np.save(tmp_path / "solid.npy", np.tile(tile, (24, 24, 24)))
    fake_hip.run(tmp_path, f"""
import ctypes
import numpy as np
c = context(np.load({str(tmp_path / 'solid.npy')!r}), storage={storage}, model={model})
a, b, g = (ctypes.c_void_p(k << 40) for k in (4, 5, 6))
hip.notes()
call("lbm_adjoint_seed", c.ctx, c.state[0], a, g)
call("lbm_adjoint_step", c.ctx, c.state[0], a, b, g)
call("lbm_adjoint_final", c.ctx, b, a)
for n in hip.notes():
    assert int(n.split()[3]) == {lds} and ("direct" in n) == ({lds} == 0), n
c.destroy()
""")


@pytest.mark.gpu
@pytest.mark.parametrize("storage,item", [("f64", 8), ("f32", 4)])
@pytest.mark.parametrize("model", ["qc", "mrt-qc"])
@pytest.mark.parametrize("tpw", [0, 1, 2])
def test_same_bytes(storage, item, model, tpw):
    import torch
    log(f"[case] full grid {storage} {model} {tpw}")
    lat = new_lattice(_box("full"), 0.8, 7, storage=storage, model=model, tiles_per_wg=tpw)
    lat.init(u0=(0.02, -0.01, 0.015))
    lat.set_force((1e-5, -2e-5, 3e-5))
    lat.step(2)
    n, src = lat.sizes.state_bytes, lat.current_state()
    pairs = _buffers(lat, n, item)  # the second is off a 16-byte boundary: stored directly
    for whole, start in pairs:
        lat.step_buf(src, whole.data_ptr() + start)
    _check(pairs, n)
    eta = torch.rand(n // item, dtype=torch.float64 if item == 8 else torch.float32, device=lat.device)
    pairs, grads = _buffers(lat, n, item), []
    for whole, start in pairs:
        grads.append(lat.new_grad())
        lat.adjoint_step(src, eta.data_ptr(), whole.data_ptr() + start, grads[-1])
    _check(pairs, n)
    assert torch.equal(grads[0], grads[1])
