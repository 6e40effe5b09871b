"""Steps with and without open boundaries are kernels of their own: every
storage type, model and offset width of both, on a ragged channel whose
boundary nodes lie on a chosen axis with either flow direction, against the
oracle at the bounds of the boundary tests; taking the boundaries away again
brings back the closed step."""
import numpy as np
import pytest

import oracle as O

from helpers import log, new_lattice, padded, perturbed_state, rel_err_f

pytestmark = pytest.mark.gpu


def _channel(axis, flip):
    """Solid walls on the four other faces of a ragged box, velocity nodes on one face of `axis` and
    pressure nodes on the other."""
    n = [13, 11, 10]  # x, y, z
    n[axis] = 22
    solid = np.zeros((n[2], n[1], n[0]), np.uint8)
    for a in range(3):
        if a != axis:
            ix = [slice(None)] * 3
            for side in (0, -1):
                ix[2 - a] = side
                solid[tuple(ix)] = 1
    types = np.zeros_like(solid)
    base = 4 * axis + 1
    low, high = [slice(None)] * 3, [slice(None)] * 3
    low[2 - axis], high[2 - axis] = 0, -1
    types[tuple(low)] = base + (3 if flip else 0)
    types[tuple(high)] = base + (2 if flip else 1)
    types[solid == 1] = 0
    return solid, types


@pytest.mark.parametrize("axis,flip", [(0, False), (1, True), (2, False), (0, True)])
@pytest.mark.parametrize("storage", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("model", ["qc", "inc", "mrt-qc", "mrt-inc"])
def test_open_and_closed_steps(model, storage, axis, flip):
    import torch
    solid, types = _channel(axis, flip)
    sp = padded(solid, 0)
    bt = np.zeros_like(sp)
    bt[:types.shape[0], :types.shape[1], :types.shape[2]] = types
    tau, steps = 0.8, 12
    u = [0.001, -0.002, 0.0015]
    u[axis] = -0.02 if flip else 0.02
    g = (1e-6, -2e-6, 3e-6)
    f0 = perturbed_state(sp, 17)
    ref = O.run_bc(f0, sp, tau, steps, bt, u_in=tuple(u), rho_out=0.999, force=np.array(g), periodic=0,
                   model=O.MODELS[model])
    closed = O.run(f0, sp, tau, steps, force=np.array(g), periodic=0, model=O.MODELS[model])
    _, w, _ = O.lattice()
    fl = sp == 0
    for wide in (False, True):
        lat = new_lattice(solid, tau, 0, model=model, storage=storage, wide_offsets=wide)
        lat.init()
        lat.set_force(g)
        for boundaries, want in ((bt, ref), (None, closed), (bt, ref)):
            lat.set_boundaries(boundaries, u_in=tuple(u), rho_out=0.999)
            lat.set_state(torch.from_numpy(f0))
            lat.step(steps)
            got = lat.get_state().cpu().numpy()
            if storage == "f64":
                err, bound = rel_err_f(got, want, sp), 1e-12
            else:
                d = np.abs(want - w[:, None, None, None])[:, fl].max()
                err = float(np.abs(got - want)[:, fl].max())
                bound = steps * 2.0 ** -24 * d * 8 if storage == "f32" else steps * 2.0 ** -10 * d
            log(f"[case] {model} {storage} axis={axis} flip={flip} wide={wide} open={boundaries is not None}: "
                f"{err:.2e} (bound {bound:.2e})")
            assert err <= bound
