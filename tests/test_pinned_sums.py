"""Pinned host memory of the macroscopic sums, on a runtime without a device:
a context does without it when it cannot be had."""
import fake_hip


def test_failed_allocation_leaves_no_error(tmp_path):
    """The first launch after it does not report the allocation's error, and the sums come out of the scratch."""
    fake_hip.run(tmp_path, """
import numpy as np
hip.set(pinned_fails=1)
c = context(np.zeros((8, 8, 8)))
assert any(n.startswith("hipHostMalloc") for n in hip.notes())
call("lbm_init", c.ctx, 1.0, 0.0, 0.0, 0.0)
call("lbm_step", c.ctx, 2)
a, b = c.sums(), c.sums()
assert b[0] == a[0] + 1 and b[7] == b[0]
c.destroy()
""")
