"""A dense input that has to be converted first is converted on the current
stream: the load on the lattice's own stream comes after it, and the copy's
memory is not handed out again before the load."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

from paper_1611_02445_amd import lattice as M

SHAPE = (4, 4, 8)


class _Stream:
    def __init__(self, log):
        self.log = log

    def synchronize(self):
        pass

    def wait_stream(self, other):
        self.log.append("after the current stream")


@pytest.mark.parametrize("call", ["lbm_set_state", "lbm_adjoint_set", "lbm_set_force"])
@pytest.mark.parametrize("same_stream", [True, False])
@pytest.mark.parametrize("converted", [True, False])
def test_conversion_comes_first(monkeypatch, call, same_stream, converted):
    log = []
    own, other = _Stream(log), _Stream(log)
    lat = M.Lattice.__new__(M.Lattice)
    lat.ctx, lat.device, lat.stream, lat.force_buf = None, torch.device("cpu"), own, torch.empty(1)
    lat.tiling = SimpleNamespace(dense_shape=SHAPE)
    lat.torch = SimpleNamespace(as_tensor=torch.as_tensor, float64=torch.float64, Tensor=torch.Tensor,
                                cuda=SimpleNamespace(current_stream=lambda device: own if same_stream else other))
    monkeypatch.setattr(M, "call", lambda name, *args: log.append(name))
    monkeypatch.setattr(torch.Tensor, "record_stream", lambda t, s: log.append("kept for it" if s is own else "?"))
    x = torch.zeros((3 if call == "lbm_set_force" else 19,) + SHAPE, dtype=torch.float32 if converted else torch.float64)
    {"lbm_set_state": lat.set_state, "lbm_adjoint_set": lambda v: lat.adjoint_set(v, None),
     "lbm_set_force": lat.set_force}[call](x)
    before = ["after the current stream"] if converted and not same_stream else []
    # the other two calls wait for the load
    after = ["kept for it"] if call == "lbm_set_force" and not same_stream else []
    assert log == before + [call] + after


@pytest.mark.gpu
@pytest.mark.parametrize("what", ["state", "adjoint", "force"])
def test_slow_conversion(what):
    """The conversion is queued behind other work of the current stream; the lattice's stream is idle."""
    from helpers import new_lattice, padded, perturbed_state
    from paper_1611_02445_amd import inputs as I

    solid, _ = I.sphere_pack((48, 40, 44), 0.6, 3.0, 6.0, seed=8)
    sp = padded(solid, 7)
    want = perturbed_state(sp, 3).astype(np.float32)
    if what == "force":
        want = np.ascontiguousarray(want[:3])
    lat = new_lattice(solid, 0.7, 7, stream=torch.cuda.Stream())
    lat.init()
    adj = lat.new_adjoint()
    busy = torch.ones(1 << 26, device="cuda")
    x = torch.from_numpy(want).cuda()
    torch.cuda.synchronize()
    for _ in range(200):
        busy.mul_(1.0)
    if what == "state":
        lat.set_state(x)
        got = lat.get_state()
    elif what == "adjoint":
        lat.adjoint_set(x, adj)
        got = lat.adjoint_get(adj)
    else:
        lat.set_force(x)
        got = lat.field_to_dense(lat.force_buf)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), want.astype(np.float64))
