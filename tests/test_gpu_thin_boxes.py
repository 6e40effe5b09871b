"""Boxes of one tile along x: dense arrays are walked by groups of four tiles
along y, no lane without a node but at the end of a row of tiles.  The
launches on a runtime without a device, and the values by the checks of the
other boxes."""
import numpy as np
import pytest

import fake_hip
import test_gpu_dense_walk as walk
from paper_1611_02445_amd import inputs as I


@pytest.mark.parametrize("ny,groups", [(4, 1), (16, 1), (17, 2), (64, 4)])
def test_groups(tmp_path, ny, groups):
    fake_hip.run(tmp_path, f"""
import ctypes
import numpy as np
c = context(np.zeros((8, {ny}, 4)), periodic=0)
out = ctypes.c_void_p(1 << 42)
for args in (("lbm_get_state", c.ctx, None, out), ("lbm_field_to_dense", c.ctx, out, 0, out),
             ("lbm_macroscopic", c.ctx, out, out, (ctypes.c_double * 8)())):
    hip.notes()
    call(*args)
    n = hip.notes()
    assert n[0].split()[1:3] == ["{2 * groups}", "256"], n
c.destroy()
""")


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(4, 16, 4), (9, 13, 4), (5, 35, 3), (7, 70, 1), (90, 140, 4)])
@pytest.mark.parametrize("storage,model", [("f64", "qc"), ("f32", "inc"), ("f16s", "qc")])
def test_values(monkeypatch, shape, storage, model):
    monkeypatch.setattr(walk, "_geometry", lambda name: I.random_bitmap(shape, 0.4, shape[1]))
    walk.test_dense_outputs("", storage, model)
