"""A step reads its physics at a byte offset of its argument buffer: a kernel
signature that moves it does not compile (no GPU needed)."""
import os
import shutil
import subprocess

import pytest

from paper_1611_02445_amd import build as B


@pytest.mark.parametrize("change,compiles", [("", True), ("int more, ", False)])
def test_moved_argument_is_refused(tmp_path, change, compiles):
    if not (os.path.exists(B.HIPCC) or shutil.which(B.HIPCC)):
        pytest.skip("hipcc not available")
    text = open(os.path.join(B.CSRC, "kernels.hip")).read()
    at = "BC_PARAM Phys P)"
    assert text.count(at) == 1
    # the kernels alone: their launches do not pass the new argument
    text = text.replace(at, "BC_PARAM " + change + "Phys P)")
    text = text[:text.index("// launchers")] + "\n}\n"
    src = tmp_path / "kernels.hip"
    src.write_text(text)
    cmd = [B.HIPCC] + [f for f in B.FLAGS if f != "-shared"] + ["-I", B.INCLUDE, "-I", B.CSRC, "-fsyntax-only",
                                                               "--cuda-host-only", str(src)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert (r.returncode == 0) == compiles, r.stderr[-2000:]
    assert compiles or "StepPhys reads the physics" in r.stderr
