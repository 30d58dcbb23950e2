"""The rule that chooses the streaming kernels' launch shape (CPU: the rule
is host code in a header, compiled here into a small program)."""
import collections
import os
import subprocess

import pytest

from paper_2603_18112_amd import _build

MIB = 1 << 20
Shape = collections.namedtuple("Shape", "step_blocks stats_blocks update_blocks stream_step "
                                        "stream_update stream_gbar grouped_step")


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    """shapes([(bytes of w and m, K, dtype, elementwise, lars), ...]) -> Shapes"""
    exe = str(tmp_path_factory.mktemp("shape") / "dump")
    here = os.path.dirname(os.path.abspath(__file__))
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", _build.INCLUDE, "-I", _build.CSRC, os.path.join(here, "launch_shape_dump.cpp"),
                    "-o", exe], check=True, capture_output=True)

    def ask(cases):
        text = "".join(f"{b // 8} {K} {int(dt == 'bf16')} {int(ew)} {int(lars)}\n"
                       for b, K, dt, ew, lars in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [Shape(*map(int, line.split())) for line in out.splitlines()]
    return ask


REPLICAS = [1, 2, 3, 4, 5, 7, 8, 12, 15, 16, 17, 24, 31, 32, 33, 48, 63, 64, 100, 1024]


def test_small_layouts_are_not_capped(shapes):
    """Layouts whose blocks the chip holds at once only lose from a cap on the
    blocks per CU: none up to 40 MiB of w and m with ordinary accesses, none
    with element scales while w and m fit the Infinity Cache, none for
    statistics and for LARS's update up to 64 MiB."""
    sizes = [2048, 193_872, MIB, 8 * MIB, 32 * MIB, 40 * MIB]
    cases = [(b, K, dt, ew, lars) for b in sizes for K in REPLICAS for dt in ("f32", "bf16")
             for ew, lars in ((0, 0), (1, 0), (0, 1))]
    for c, s in zip(cases, shapes(cases)):
        assert s.step_blocks == 0 or s.stream_step, (c, s)
        assert s.stats_blocks == 0 and s.update_blocks == 0, (c, s)
    cases = [(b, K, dt, 1, 0) for b in (85 * MIB, 256 * MIB) for K in REPLICAS for dt in ("f32", "bf16")]
    for c, s in zip(cases, shapes(cases)):
        assert s.step_blocks == 0 or s.stream_step, (c, s)
    cases = [(64 * MIB, K, dt, 0, 1) for K in REPLICAS for dt in ("f32", "bf16")]
    for c, s in zip(cases, shapes(cases)):
        assert s.stats_blocks == 0 and s.update_blocks == 0, (c, s)
