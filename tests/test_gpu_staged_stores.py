"""Stores staged through LDS, taken from 6144 tiles on to lattices on a 16-byte
boundary: bitwise the lattice that the direct stores write (to a buffer off
that boundary), over tiles of every fluid count, with nothing written outside
the lattice and every pad byte zero."""
import numpy as np
import pytest

from helpers import log, new_lattice

pytestmark = pytest.mark.gpu

CANARY = 0xA5


def _solid():
    """19^3 tiles whose fluid counts run over 1..64."""
    rng = np.random.default_rng(77)
    t = rng.random((19, 19, 19, 64)).argsort(-1).argsort(-1)  # ranks 0..63 in every tile
    k = rng.integers(1, 65, (19, 19, 19, 1))
    k[0, 0, :, 0] = np.arange(1, 20)
    k[0, 1, :, 0] = np.arange(46, 65)
    solid = (t >= k).astype(np.uint8).reshape(19, 19, 19, 4, 4, 4)
    return np.ascontiguousarray(solid.transpose(0, 3, 1, 4, 2, 5).reshape(76, 76, 76))


def _buffers(lat, nbytes, item):
    """Two buffers of nbytes within canaries: on a 16-byte boundary, and `item` bytes past one."""
    import torch
    out = []
    for shift in (0, item):
        whole = torch.full((nbytes + 512,), CANARY, dtype=torch.uint8, device=lat.device)
        start = (-whole.data_ptr()) % 256 + shift
        out.append((whole, start))
    return out


def _check(pairs, nbytes):
    import torch
    torch.cuda.synchronize()
    (wa, a), (wb, b) = pairs
    assert torch.equal(wa[a:a + nbytes], wb[b:b + nbytes])
    for whole, start in pairs:
        assert bool((whole[:start] == CANARY).all()) and bool((whole[start + nbytes:] == CANARY).all())
    assert not bool((wa[a:a + nbytes].view(torch.int32) == int.from_bytes(bytes([CANARY] * 4), "little", signed=True)).any())


@pytest.mark.parametrize("storage,item", [("f64", 8), ("f32", 4), ("f16s", 2)])
@pytest.mark.parametrize("model", ["qc", "mrt-inc"])
@pytest.mark.parametrize("open_faces", [False, True])
def test_staged_equals_direct(storage, item, model, open_faces):
    import torch
    solid = _solid()
    lat = new_lattice(solid, 0.8, 0, storage=storage, model=model, f16_rounding="nearest")
    assert lat.n_tiles == 19 ** 3 >= 6144
    lat.init(u0=(0.02, -0.01, 0.015))
    lat.set_force((1e-5, -2e-5, 3e-5))
    if open_faces:
        types = np.zeros_like(solid)
        types[:, :, 0] = np.where(solid[:, :, 0] == 0, 1, 0)
        types[:, :, -1] = np.where(solid[:, :, -1] == 0, 2, 0)
        lat.set_boundaries(types, u_in=(0.02, 0.0, 0.0), rho_out=1.0)
    lat.step(2)
    n = lat.sizes.state_bytes
    src = lat.current_state()
    pairs = _buffers(lat, n, item)
    for whole, start in pairs:
        lat.step_buf(src, whole.data_ptr() + start)
    _check(pairs, n)
    if storage == "f16s" or open_faces:
        return
    eta = torch.rand(n // item, dtype=torch.float64 if item == 8 else torch.float32, device=lat.device)
    for call in ("seed", "step", "final"):
        pairs = _buffers(lat, n, item)
        grads = []
        for whole, start in pairs:
            out, grad = whole.data_ptr() + start, lat.new_grad()
            if call == "seed":
                lat.adjoint_seed(src, out, grad)
            elif call == "step":
                lat.adjoint_step(src, eta.data_ptr(), out, grad)
            else:
                lat.adjoint_final(eta.data_ptr(), out)
            grads.append(grad)
        _check(pairs, n)
        assert torch.equal(grads[0], grads[1])
    log(f"[case] staged = direct: {storage} {model}")


@pytest.mark.parametrize("tiles_per_wg", [1, 2, 8])
def test_workgroup_sizes(tiles_per_wg):
    """Eight FP64 tiles need more LDS than a workgroup is sure to get: stored directly."""
    import torch
    solid = _solid()
    out = []
    for tpw in (0, tiles_per_wg):
        lat = new_lattice(solid, 0.7, 0, tiles_per_wg=tpw)
        lat.init(u0=(0.02, -0.01, 0.015))
        lat.step(3)
        out.append(lat.current_state().clone())
    assert torch.equal(out[0], out[1])
