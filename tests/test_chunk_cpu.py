"""The halving of a chunk whose scratch cannot be had, on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "chunk.h"
int main(int, char **v)
{
    const long want = atol(v[1]), least = atol(v[2]), room = atol(v[3]);
    int calls = 0;
    const long got = tr::take_chunk(want, least, [&](long n) { ++calls; return n <= room; });
    printf("%ld %d\n", got, calls);
}
"""


@pytest.fixture(scope="module")
def prog(tmp_path_factory):
    d = tmp_path_factory.mktemp("chunk")
    (d / "m.cpp").write_text(SRC)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2105_09644_amd", "csrc"), "-o", str(d / "m"), str(d / "m.cpp")], check=True)
    return str(d / "m")


@pytest.mark.parametrize("want,least,room,got,calls", [
    (32768, 1024, 10 ** 9, 32768, 1),    # all of it
    (32768, 1024, 32767, 16384, 2),
    (32768, 1024, 1024, 1024, 6),        # the least
    (32768, 1024, 1023, 0, 6),           # not even that
    (5000, 1024, 1500, 1250, 3),
    (5000, 1024, 1100, 1024, 4),         # clamped to the least, not 625
    (7, 7, 7, 7, 1),
    (7, 7, 6, 0, 1),
    (1, 1, 0, 0, 1),
])
def test_take_chunk(prog, want, least, room, got, calls):
    out = subprocess.run([prog, str(want), str(least), str(room)], capture_output=True, text=True, check=True).stdout
    assert out.split() == [str(got), str(calls)]
