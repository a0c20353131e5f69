"""Which calls of few faces take the device's second stream (csrc/side.h, host code):
those of a stream that has the device to itself, not those of streams that take turns."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_26137_amd", "csrc")
MAIN = r"""
#include <stdio.h>
#include "side.h"
// a line per call of the pattern given, repeated: 1 where it takes the second stream
int main(int argc, char** argv) {
    bake::SteadyCaller c;
    static int streams[26];
    for (int r = 0; r < 40; ++r)
        for (const char* p = argv[1]; *p; ++p) putchar(c.call(streams + (*p - 'A')) ? '1' : '0');
    return 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    d = tmp_path_factory.mktemp("side")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, "-o", str(d / "side"), str(d / "main.cpp"),
                    "-lpthread"], check=True)
    return str(d / "side")


def calls(exe, pattern):
    return subprocess.run([exe, pattern], check=True, capture_output=True, text=True).stdout


def test_alone(exe):
    assert calls(exe, "A" * 2) == "0" * 16 + "1" * 64


@pytest.mark.parametrize("pattern", ["AB", "AABB", "AAB", "ABCD", "AABBCCDD", "A" * 8 + "B" * 8, "A" * 16 + "B"])
def test_in_turn(exe, pattern):
    assert "1" not in calls(exe, pattern)


def test_another_call_between(exe):
    out = calls(exe, "A" * 30 + "B")
    assert out[:31] == "0" * 16 + "1" * 14 + "0" and out[31:47] == "0" * 16
