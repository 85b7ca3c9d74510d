"""Sums over the lanes of a wave (over_lanes in device_utils.h): a rotation within 16 lanes stands for lane ^ O only where eight or
more lanes below are still to meet, so narrower groups are refused when they are compiled."""
import subprocess

import pytest

from paper_2509_23241_amd import build

SOURCE = """
#include "device_utils.h"
__global__ void sums(float* v) { v[threadIdx.x] = tp::sum_over_lanes<%d>(v[threadIdx.x]); }
"""


@pytest.mark.parametrize("lanes,accepted", [(32, True), (16, True), (8, True), (4, False), (2, False), (1, False)])
def test_widths_that_a_rotation_stands_for(tmp_path, lanes, accepted):
    source = tmp_path / "sums.hip"
    source.write_text(SOURCE % lanes)
    run = subprocess.run([build._hipcc(), "--offload-arch=gfx950", "--offload-device-only", "-fsyntax-only", "-std=c++17", "-I", build.CSRC,
                          "-x", "hip", str(source)], capture_output=True, text=True)
    assert (run.returncode == 0) == accepted, run.stderr
    assert accepted or "lane" in run.stderr
