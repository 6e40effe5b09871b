"""Tilings that no dense array of their box is walked for, on a runtime without
a device: a box too large for any array, of which a program steps a few tiles."""
import fake_hip

HEAD = """
import ctypes
import numpy as np
def tiling(n, corners):
    # a tiling made by the library whose tiles are put elsewhere in a larger box
    solid = np.ones((4, 4, 4 * len(corners)), np.uint8)
    solid[..., ::2] = 0
    c = fake_hip.context.__new__(fake_hip.context)
    t = ctypes.POINTER(abi.Tiles)()
    call("lbm_build_tiles", solid.ctypes.data_as(ctypes.c_void_p), solid.shape[2], 4, 4, 0, ctypes.byref(t))
    t.contents.nx = t.contents.ny = t.contents.nz = n
    t.contents.tx = t.contents.ty = t.contents.tz = (n + 3) // 4
    for k, at in enumerate(corners):
        for a in range(3):
            t.contents.tile_xyz[3 * k + a] = at[a]
    return t
def create(t):
    p, size, ctx = abi.Params(tau=0.7, rho0=1.0), abi.Sizes(), ctypes.c_void_p()
    call("lbm_required_bytes", t, ctypes.byref(p), ctypes.byref(size))
    mem = [np.zeros(int(b) + 256, np.uint8) for b in (size.table_bytes, size.scratch_bytes)]
    at = [ctypes.c_void_p((m.ctypes.data + 255) // 256 * 256) for m in mem]
    call("lbm_create", t, ctypes.byref(p), ctypes.c_void_p(1 << 40), ctypes.c_void_p(1 << 41), *at, None, ctypes.byref(ctx))
    return ctx, size, mem
"""


def test_box_too_large_for_a_map(tmp_path):
    fake_hip.run(tmp_path, HEAD + """
for n in (1 << 12, 1 << 16, 1 << 23, 0x7ffffffc):
    t = tiling(n, [(0, 0, 0), (n - 4, n - 8, n - 4)])
    ctx, size, mem = create(t)
    assert size.table_bytes <= 1 << 12, (n, size.table_bytes)
    hip.notes()
    call("lbm_step", ctx, 2)
    s = (ctypes.c_double * 8)()
    call("lbm_macroscopic", ctx, None, None, s)
    n = hip.notes()
    assert [x.split()[0][:20] for x in n[:2]] == [n[0].split()[0][:20]] * 2 and "k_sums" in n[2], n
    call("lbm_destroy", ctx)
""")


def test_two_tiles_at_one_place(tmp_path):
    """Every tile of the caller's tiling counts in the sums: the tiles are taken one by one."""
    fake_hip.run(tmp_path, HEAD + """
for corners, kernel in (([(0, 0, 0), (4, 0, 0), (4, 4, 4)], "k_fields"), ([(0, 0, 0), (4, 0, 0), (4, 0, 0)], "k_sums")):
    ctx, size, mem = create(tiling(8, corners))
    hip.notes()
    s = (ctypes.c_double * 8)()
    call("lbm_macroscopic", ctx, None, None, s)
    n = hip.notes()
    assert kernel in n[0], n
    call("lbm_destroy", ctx)
""")
