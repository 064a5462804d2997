"""What the compiler says of the kernels' sources (no GPU)."""
import os
import shutil
import subprocess

import pytest

from paper_1101_2065_amd import build

KERNELS = [s for s in build.SOURCES if s.endswith(".hip")]


@pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="hipcc not available")
@pytest.mark.parametrize("src", KERNELS)
def test_no_pointer_is_taken_for_a_better_aligned_one(src):
    """A complex array need only lie on its real type's boundaries, and the
    kernels' 16-byte accesses say so in their types; a type handed on without
    its alignment is an error of the device pass."""
    r = subprocess.run([build.HIPCC] + build.HIP_FLAGS + build.EXTRA.get(src, []) +
                       ["-x", "hip", "--cuda-device-only", "-fsyntax-only", "-Werror=align-mismatch",
                        os.path.join(build.CSRC, src)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
