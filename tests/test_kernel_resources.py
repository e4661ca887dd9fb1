"""Registers, scratch memory and waves per SIMD of the compiled kernels, as the compiler reports
them for gfx950 (no GPU needed). The kernels below wait on memory or on chains of additions,
so that the waves a SIMD holds set their time: a second form compiled into one of them, or a
longer unroll, must not take the waves away."""
import functools
import os
import re
import subprocess

import pytest

from paper_1005_5198_amd import build


@functools.lru_cache(maxsize=None)
def _usage(source):
    """{demangled kernel name: {"waves", "scratch"}} of one HIP source."""
    cmd = [build.HIPCC, *build.COMPILE_FLAGS, "--cuda-device-only", "-c", os.path.join(build.CSRC, source),
           "-o", os.devnull, "-Rpass-analysis=kernel-resource-usage"]
    proc = subprocess.run(cmd, capture_output=True, text=True, check=True)
    out, cur = {}, None
    for line in proc.stderr.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
        for key, text in (("waves", r"Occupancy \[waves/SIMD\]"), ("scratch", r"ScratchSize \[bytes/lane\]")):
            m = re.search(r"remark: +" + text + r": (\d+)", line)
            if m and cur is not None:
                cur[key] = int(m.group(1))
    names = subprocess.run(["c++filt", *out], capture_output=True, text=True, check=True).stdout.split("\n")
    return {n.replace("(anonymous namespace)::", ""): u for n, u in zip(names, out.values())}


def _kernels(source, pattern):
    found = {n: u for n, u in _usage(source).items() if re.search(pattern, n)}
    assert found, f"no kernel of {source} matches {pattern}"
    return found


# (the figures are the kernels' own before they took a second form in)
@pytest.mark.parametrize("pattern,waves,scratch", [
    (r"recheck_scan_batch_kernel<1,", 2, 16),        # the batch's exact stage
    (r"recheck_exact_wave_kernel<\w+, .*ExactForm\)0>", 3, 0),   # a map's, chain
])
def test_exact_stage_keeps_its_waves(pattern, waves, scratch):
    for name, u in _kernels("recheck.hip", pattern).items():
        assert u["waves"] >= waves and u["scratch"] <= scratch, (name, u)


def test_stage_a_by_thread_keeps_its_waves():
    """Stage A with a thread per ray, in a kernel without the form for short queues (1: FORM_THREADS)."""
    for name, u in _kernels("recheck.hip", r"recheck_fast_kernel<\w+, .*StageAForm\)1>").items():
        assert u["waves"] >= 4 and u["scratch"] == 0, (name, u)


def test_the_stages_in_one_kernel_keep_three_waves():
    """Stage F with stages A and B in its kernel (small maps): a small map's queue is a wave or
    two per SIMD of loads and reductions, which a third hides."""
    for name, u in _kernels("farfield.hip", r"recheck_far_kernel<\w+, true>").items():
        assert u["waves"] >= 3 and u["scratch"] == 0, (name, u)
