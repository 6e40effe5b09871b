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


def test_destroy_frees_no_pinned_memory(tmp_path):
    """hipHostFree waits for every stream of the device: contexts come and go without it, on one block."""
    fake_hip.run(tmp_path, """
import numpy as np
for _ in range(200):
    c = context(np.zeros((4, 4, 4)))
    c.sums()
    c.destroy()
n = [x for x in hip.notes() if x.startswith("hipHost")]
assert n == ["hipHostMalloc 4096"], n
""")


def test_contexts_share_no_row(tmp_path):
    """More contexts at a time than the block has rows for, on several threads, some of them destroyed and made
    again: every call gets the sums of its own launch (a number of its own), and no more is allocated."""
    fake_hip.run(tmp_path, """
import threading
import numpy as np
seen, errors = [], []
def work(seed):
    try:
        rng = np.random.default_rng(seed)
        cs = [context(np.zeros((4, 4, 4))) for _ in range(30)]
        for _ in range(300):
            i = int(rng.integers(30))
            s = cs[i].sums()
            assert s[0] == s[7], s
            seen.append(s[0])
            if rng.random() < 0.2:
                cs[i].destroy()
                cs[i] = context(np.zeros((4, 4, 4)))
        for c in cs:
            c.destroy()
    except BaseException as e:
        errors.append(e)
ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
[t.start() for t in ts]; [t.join() for t in ts]
assert not errors, errors
assert len(seen) == len(set(seen)) == 1200
assert sum(x.startswith("hipHost") for x in hip.notes()) == 1
""")


def test_first_context_during_a_capture(tmp_path):
    """Another thread's global-mode capture forbids allocations, but in relaxed mode."""
    fake_hip.run(tmp_path, """
import numpy as np
hip.set(in_capture=1)
c = context(np.zeros((4, 4, 4)))
call("lbm_init", c.ctx, 1.0, 0.0, 0.0, 0.0)
hip.set()
c.sums()
c.destroy()
assert [x for x in hip.notes() if x.startswith("hipHost")] == ["hipHostMalloc 4096"]
""")
