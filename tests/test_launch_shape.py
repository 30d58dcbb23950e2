"""The rule that chooses the streaming kernels' launch shape (CPU: the rule
is host code in a header, compiled here into a small program)."""
import collections
import os
import re
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
    blocks per CU: none up to 40 MiB of w and m, none for statistics up to 64
    MiB, nor for LARS's update where it reads the kept mean."""
    sizes = [2048, 193_872, MIB, 8 * MIB, 32 * MIB, 40 * MIB]
    cases = [(b, K, dt, ew, lars) for b in sizes for K in REPLICAS for dt in ("f32", "bf16")
             for ew, lars in ((0, 0), (1, 0), (0, 1))]
    for c, s in zip(cases, shapes(cases)):
        assert s.step_blocks == 0 or s.stream_step, (c, s)
        assert s.stats_blocks == 0 and s.update_blocks == 0, (c, s)
    cases = [(64 * MIB, K, dt, 0, 1) for K in REPLICAS for dt in ("f32", "bf16")]
    for c, s in zip(cases, shapes(cases)):
        keeps_mean = c[1] * (4 if c[2] == "f32" else 2) > 8
        assert s.stats_blocks == 0 and (s.update_blocks == 0) == keeps_mean, (c, s)


def test_layouts_that_fit_the_cache_are_capped_from_their_line_on(shapes):
    """Above 40 MiB of w and m four blocks per CU, with element scales too
    (for a few replicas the cap gains 1 to 5% there)."""
    cases = [(b, K, dt, ew, 0) for b in (40 * MIB + 8, 85 * MIB, 128 * MIB) for K in (1, 2, 4, 7)
             for dt in ("f32", "bf16") for ew in (0, 1)]
    assert all(s.step_blocks == 4 and not s.stream_step for s in shapes(cases))


@pytest.mark.parametrize("K,dtype,ew,line", [
    (16, "f32", 0, 8), (1024, "f32", 0, 8), (32, "bf16", 0, 8), (64, "bf16", 0, 8),
    (8, "f32", 0, 128), (15, "f32", 0, 128), (20, "bf16", 0, 256), (31, "bf16", 0, 256),
    (5, "f32", 0, 256), (7, "f32", 0, 256), (16, "bf16", 0, 512), (19, "bf16", 0, 512),
    (4, "f32", 0, 512), (1, "f32", 0, 256), (3, "f32", 0, 256),
    (1, "bf16", 0, None), (15, "bf16", 0, None),
    (16, "f32", 1, 128), (10, "f32", 1, 256), (15, "f32", 1, 256), (6, "f32", 1, 512), (9, "f32", 1, 512),
    (5, "f32", 1, None), (1, "f32", 1, None), (64, "bf16", 1, None), (1024, "bf16", 1, None)])
def test_streaming_is_taken_from_its_line_on(shapes, K, dtype, ew, line):
    """w and m are streamed only above the size from which that was measured
    to gain more, with other states in between, than it loses back to back."""
    sizes = [MIB, 8 * MIB, 64 * MIB, 128 * MIB, 195 * MIB, 256 * MIB, 280 * MIB, 450 * MIB, 512 * MIB,
             600 * MIB, 1056 * MIB]
    if line is not None:
        sizes += [line * MIB, line * MIB + 8]
    cases = [(b, K, dtype, ew, 0) for b in sizes]
    for c, s in zip(cases, shapes(cases)):
        assert bool(s.stream_step) == (line is not None and c[0] > line * MIB), (c, s)


def test_lars_streams_from_its_lines_on(shapes):
    """The update's w and m above 64 MiB, the mean once it outgrows the cache."""
    for line, field in ((64, "stream_update"), (512, "stream_gbar")):
        cases = [(line * MIB + d, K, dt, 0, 1) for d in (0, 8) for K in REPLICAS for dt in ("f32", "bf16")]
        for c, s in zip(cases, shapes(cases)):
            assert bool(getattr(s, field)) == (c[0] > line * MIB), (c, s)


def test_the_library_holds_exactly_the_kernels_that_can_be_launched(shapes):
    """Every instantiation of the step, update and correction kernels against
    what the rule, the kept replica mean (more than 8 replica bytes per
    element), carried weight norms and the small-batch choice can ask for."""
    from paper_2603_18112_amd import ags
    ags.load_library()
    nm = subprocess.run(["nm", "-C", _build.LIB], capture_output=True, text=True, check=True).stdout
    built = {m.group(1) for m in re.finditer(r"__device_stub__((?:step|update|correct)_kernel<[^>]*>)", nm)}

    lines = [8, 40, 64, 128, 256, 512]
    sizes = [MIB, 2048 * MIB] + [b * MIB + d for b in lines for d in (0, 8)]
    cases = [(b, K, dt, ew, lars) for b in sizes for K in sorted({*REPLICAS, *range(1, 70)})
             for dt in ("f32", "bf16") for ew, lars in ((0, 0), (1, 0), (0, 1))]

    def name(kernel, *args):
        return f"{kernel}_kernel<{', '.join(str(a).lower() for a in args)}>"

    want = set()
    for (_, K, dt, ew, lars), s in zip(cases, shapes(cases)):
        gt = "float" if dt == "f32" else "unsigned short"
        kt = K if K in (1, 2, 4, 8, 16, 32, 64) else 0
        keep = K * (4 if dt == "f32" else 2) > 8
        for r in range(3 if K > 1 else 2):
            want.add(name("step", gt, kt, r, False, False, False, False, 0))  # ags_stats
            if not lars:
                want.add(name("step", gt, kt, r, True, bool(ew), bool(s.stream_step), False, 0))
                continue
            for carried in (False, True):
                want.add(name("step", gt, kt, r, False, False, False, carried, 0))
                want.add(name("step", gt, kt, r, False, False, False, carried,
                              0 if not keep else 2 if s.stream_gbar else 1))
                want.add(name("update", gt, kt, not keep, carried, keep and bool(s.stream_update)))
        want.add(name("correct", gt, kt))
    assert built == want, (sorted(built - want), sorted(want - built))


def test_the_streaming_parity_cases_stream(shapes):
    """The layouts with which the GPU tests check the streaming kernels are
    above the lines from which they are taken (and not far above)."""
    import streaming_cases as sc

    def ask(cases, lars):
        return shapes([(8 * sc.layout(mib).n_flat, K, dt, int(cases is sc.ELEMENT_SCALES), lars)
                       for mib, K, dt, _ in cases])

    assert all(s.stream_step for s in ask(sc.STEP, 0))
    assert all(s.stream_step for s in ask(sc.ELEMENT_SCALES, 0))
    lars = ask(sc.LARS, 1)
    assert all(s.stream_update for s in lars) and lars[-1].stream_gbar
    assert all(K * (4 if dt == "f32" else 2) > 8 for _, K, dt, _ in sc.LARS)  # the mean is kept
