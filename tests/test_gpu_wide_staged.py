"""The kernels of lattices past 4 GiB, 64-bit offsets with staged stores: every
one is chosen where it should be (launches on a runtime without a device) and
stores the bytes of the 32-bit one, which are pinned to the direct stores.  The
same for FP16 with stochastic rounding and for the measurement kernels."""
import numpy as np
import pytest

import fake_hip
from helpers import log, new_lattice
from test_gpu_staged_stores import _buffers, _check, _solid


@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("tiles", [6143, 6144])
def test_kernels_chosen(tmp_path, wide, tiles):
    """k_step<storage, model, offset type (j 32 bits, m 64)> and the like, without "direct" from 6144 tiles on."""
    kept = np.zeros(4 * 4 * 400, bool)  # of 4 x 4 x 400 tiles
    kept[:tiles] = True
    half = np.arange(64).reshape(4, 4, 4) % 2  # tiles of 32 fluid nodes
    solid = 1 - np.kron(kept.reshape(4, 4, 400), half).astype(np.uint8)
    np.save(tmp_path / "solid.npy", solid)
    fake_hip.run(tmp_path, f"""
import ctypes
import numpy as np
solid = np.load({str(tmp_path / 'solid.npy')!r})
off, direct = "m" if {wide} else "j", {tiles} < 6144
a, b, g = (ctypes.c_void_p(k << 40) for k in (4, 5, 6))
for storage in (0, 1, 2):
    for model in (0, 1, 2, 3):
        c = context(solid, storage=storage, model=model, wide_offsets={wide})
        assert c.tiles.contents.n_tiles == {tiles}
        hip.notes()
        call("lbm_step_buf", c.ctx, a, b)
        call("lbm_calib_step", c.ctx, 1, a, b)
        call("lbm_calib_step", c.ctx, 2, a, b)
        names = ["k_step", "k_calib", "k_calib"]
        if storage < 2:
            call("lbm_adjoint_seed", c.ctx, a, b, g)
            call("lbm_adjoint_step", c.ctx, a, b, c.state[0], g)
            call("lbm_adjoint_final", c.ctx, a, b)
            names += ["k_adj_seed", "k_adj_step", "k_adj_final"]
        for name, note in zip(names, hip.notes()):
            kernel, _, _, lds = note.split()
            if name == "k_calib":
                s = "d" if storage == 0 else "f" if storage == 1 else "DF16_"
                assert kernel.startswith(f"_ZN4tlbm7k_calibI{{s}}") and f"E{{off}}Lb{{0 if direct else 1}}EE" in kernel, kernel
            else:
                n = name + ("_direct" if direct else "")
                m = 0 if name == "k_adj_final" else model
                assert kernel.startswith(f"_ZN4tlbm{{len(n)}}{{n}}ILi{{storage}}ELi{{m}}E{{off}}EE"), kernel
            assert (int(lds) == 0) == direct, note
        c.destroy()
""")


def _lattice(wide, storage, model, **kw):
    lat = new_lattice(_solid(), 0.8, 0, storage=storage, model=model, wide_offsets=wide, **kw)
    lat.init(u0=(0.02, -0.01, 0.015))
    lat.set_force((1e-5, -2e-5, 3e-5))
    return lat


@pytest.mark.gpu
@pytest.mark.parametrize("storage,item", [("f64", 8), ("f32", 4), ("f16s", 2)])
@pytest.mark.parametrize("model", ["qc", "inc", "mrt-qc", "mrt-inc"])
@pytest.mark.parametrize("open_faces", [False, True])
def test_wide_equals_narrow(storage, item, model, open_faces):
    import torch
    log(f"[case] wide staged {storage} {model} open={open_faces}")
    rounding = "stochastic" if model in ("qc", "mrt-inc") else "nearest"
    lats = [_lattice(w, storage, model, f16_rounding=rounding) for w in (False, True)]
    solid = _solid()
    for lat in lats:
        if open_faces:
            types = np.zeros_like(solid)
            types[:, :, 0] = np.where(solid[:, :, 0] == 0, 1, 0)
            types[:, :, -1] = np.where(solid[:, :, -1] == 0, 2, 0)
            lat.set_boundaries(types, u_in=(0.02, 0.0, 0.0), rho_out=1.0)
        lat.step(3)
    a, b = (lat.current_state() for lat in lats)
    assert torch.equal(a, b)
    n = lats[0].sizes.state_bytes
    for kind in () if open_faces else (1, 2):
        out = [torch.full((n,), 0xA5, dtype=torch.uint8, device=a.device) for _ in lats]
        for lat, o in zip(lats, out):
            lat.calib_step(kind, a, o)
        assert torch.equal(out[0], out[1]), kind
    if storage == "f16s" or open_faces:
        return
    eta = torch.rand(n // item, dtype=torch.float64 if item == 8 else torch.float32, device=a.device)
    outs = []
    for lat in lats:
        seed, step, final, grad = lat.new_adjoint(), lat.new_adjoint(), lat.new_adjoint(), lat.new_grad()
        lat.adjoint_seed(a, seed, grad)
        lat.adjoint_step(a, eta.data_ptr(), step, grad)
        lat.adjoint_final(eta.data_ptr(), final)
        outs.append((seed, step, final, grad))
    for x, y in zip(*outs):
        assert torch.equal(x, y)


@pytest.mark.gpu
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("model", ["qc", "mrt-inc"])
def test_stochastic_staged_equals_direct(wide, model):
    """Two contexts with equal launch counters draw the same bits; one stores directly, off a 16-byte boundary."""
    lats = [_lattice(wide, "f16s", model) for _ in range(2)]
    for lat in lats:
        lat.step(2)
    n = lats[0].sizes.state_bytes
    pairs = _buffers(lats[0], n, 2)
    for lat, (whole, start) in zip(lats, pairs):
        lat.step_buf(lat.current_state(), whole.data_ptr() + start)
    _check(pairs, n)


@pytest.mark.gpu
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("storage,item", [("f64", 8), ("f32", 4), ("f16s", 2)])
@pytest.mark.parametrize("kind", [1, 2])
def test_calib_staged_equals_direct(wide, storage, item, kind):
    lat = _lattice(wide, storage, "qc")
    lat.step(2)
    n = lat.sizes.state_bytes
    pairs = _buffers(lat, n, item)
    for whole, start in pairs:
        lat.calib_step(kind, lat.current_state(), whole.data_ptr() + start)
    _check(pairs, n)
