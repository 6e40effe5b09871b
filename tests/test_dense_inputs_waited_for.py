"""A dense array handed to set_state or adjoint_set has been read when the call
returns, whatever stream is current: the caller may free or overwrite it on any
stream, and nothing else orders that after the load."""
from types import SimpleNamespace

import pytest
import torch

from paper_1611_02445_amd import lattice as M

SHAPE = (4, 4, 8)


class _Stream:
    def __init__(self, log, name):
        self.log, self.name = log, name

    def synchronize(self):
        self.log.append(f"wait for {self.name}")

    def wait_stream(self, other):
        self.log.append(f"{self.name} after {other.name}")


def _lattice(monkeypatch, same_stream):
    """A Lattice without a device: library calls and stream operations are noted in order."""
    log = []
    own, other = _Stream(log, "own"), _Stream(log, "other")
    lat = M.Lattice.__new__(M.Lattice)
    lat.ctx, lat.device, lat.stream = None, torch.device("cpu"), own
    lat.tiling = SimpleNamespace(dense_shape=SHAPE)
    lat.torch = SimpleNamespace(as_tensor=torch.as_tensor, float64=torch.float64, Tensor=torch.Tensor,
                                cuda=SimpleNamespace(current_stream=lambda device: own if same_stream else other))
    monkeypatch.setattr(M, "call", lambda name, *args: log.append(name))
    return lat, log


@pytest.mark.parametrize("same_stream", [True, False])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_load_is_waited_for(monkeypatch, same_stream, dtype):
    lat, log = _lattice(monkeypatch, same_stream)
    f = torch.zeros((19,) + SHAPE, dtype=dtype)
    lat.set_state(f)
    assert log[-2:] == ["lbm_set_state", "wait for own"]
    lat.adjoint_set(f, None)
    assert log[-2:] == ["lbm_adjoint_set", "wait for own"]


@pytest.mark.gpu
@pytest.mark.parametrize("what", ["state", "adjoint"])
@pytest.mark.parametrize("then", ["overwrite", "free"])
def test_source_of_another_stream(what, then):
    """The lattice's stream is current, the source belongs to the default stream, and the load is queued
    behind other work."""
    import numpy as np
    from helpers import new_lattice, padded, perturbed_state
    from paper_1611_02445_amd import inputs as I

    solid, _ = I.sphere_pack((48, 40, 44), 0.6, 3.0, 6.0, seed=8)
    want = perturbed_state(padded(solid, 7), 3)
    s = torch.cuda.Stream()
    lat = new_lattice(solid, 0.7, 7, stream=s)
    lat.init()
    adj = lat.new_adjoint()
    torch.cuda.synchronize()
    f = torch.from_numpy(want).cuda()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        lat.step(400)
        lat.set_state(f) if what == "state" else lat.adjoint_set(f, adj)
    if then == "overwrite":
        f.zero_()
    else:
        shape = f.shape
        del f
        junk = [torch.zeros(shape, dtype=torch.float64, device="cuda") for _ in range(3)]  # noqa: F841
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        got = lat.get_state() if what == "state" else lat.adjoint_get(adj)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), want)
