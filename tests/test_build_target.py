"""The kernels build for gfx950 only (CPU): the order between the blocks of the
finalize kernel is argued from that chip's memory instructions, so another
target is refused at compile time."""
import os
import subprocess

import pytest

from paper_2603_18112_amd import _build


def test_another_target_is_refused():
    if not os.path.exists(_build.HIPCC):
        pytest.skip("hipcc not available")
    r = subprocess.run([_build.HIPCC, "--offload-arch=gfx942", "--offload-device-only", "-fsyntax-only",
                        "-std=c++17", "-I", _build.INCLUDE, "-I", _build.CSRC,
                        os.path.join(_build.CSRC, "ags_kernels.hip")], capture_output=True, text=True)
    assert r.returncode != 0 and "gfx950 only" in r.stderr
