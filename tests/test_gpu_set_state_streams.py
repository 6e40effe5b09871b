"""Loading a dense lattice that has to be converted first: the converted copy
outlives the call on the lattice's stream, the current one or another."""
import numpy as np
import pytest

from paper_1611_02445_amd import inputs as I

from helpers import new_lattice, padded, perturbed_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("own_stream", [False, True])
@pytest.mark.parametrize("what", ["state", "adjoint"])
def test_converted_input_lives_long_enough(own_stream, what):
    import torch
    solid, _ = I.sphere_pack((48, 40, 44), 0.6, 3.0, 6.0, seed=8)
    sp = padded(solid, 7)
    dev = torch.device("cuda")
    stream = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    lat = new_lattice(solid, 0.7, 7, stream=stream)
    lat.init()
    adj = lat.new_adjoint()
    torch.cuda.synchronize()
    for seed in range(4):
        f = torch.from_numpy(perturbed_state(sp, seed)).to(dev, torch.float32)
        torch.cuda.synchronize()
        if what == "state":
            lat.set_state(f)
        else:
            lat.adjoint_set(f, adj)
        # memory of the converted copy, if it was given back, is taken and written here
        junk = [torch.full(f.shape, float(seed), dtype=torch.float64, device=dev) for _ in range(3)]
        torch.cuda.synchronize()
        got = lat.get_state() if what == "state" else lat.adjoint_get(adj)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), f.double().cpu().numpy())
        del junk
