"""Ticket streams of the persistent kernels: a launch needs a running workgroup
per stream, so their number must stay a small part of a grid that may fill the
chip (a stream restricted to part of it, two launches side by side)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2306_14337_amd", "csrc")

SOURCE = """
#include "kernels.h"
#include <cstdio>
int main() {
  for (int g = 1; g <= 4096; g++) std::printf("%d\\n", kktlu::ticket_streams(g));
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_streams_need_a_32nd_of_the_grid(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC,
                    str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    streams = [int(v) for v in subprocess.run([str(exe)], check=True, capture_output=True,
                                              text=True).stdout.split()]
    assert len(streams) == 4096
    for grid, s in enumerate(streams, 1):
        assert 1 <= s <= min(grid, 64)
        assert s <= max(8, grid // 32), (grid, s)
    assert streams[255] == 8      # a workgroup per CU: as many streams as XCDs
    assert streams[2047] == 64    # eight per CU


def test_every_launch_takes_the_rule():
    text = open(os.path.join(CSRC, "kernels.hip")).read()
    assert "std::min(TICKET_STREAMS, grid)" not in text
    assert text.count("ticket_streams(grid)") == 6
