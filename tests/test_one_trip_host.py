"""Host-side check of the launch of the passes that go through in one trip (cdl_one_trip.h, compiled here for the CPU): wherever the rule lets one through, the
launch has fewer threads than 2^32, the most that HIP takes in one dimension, and every vector of the tensor has a thread and no block is idle."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2501_09849_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include "cdl_one_trip.h"
using namespace cdl;

int main()
{
    long long n;
    while (scanf("%lld", &n) == 1) {
        const long long grid = one_trip_grid(n), vectors = (long long)kOneTripThreads * kOneTripVectors;
        printf("%d %d %d\n", one_trip_fits(n) ? 1 : 0, grid * kOneTripThreads < 4294967296ll ? 1 : 0, grid * vectors >= n / 4 && (grid - 1) * vectors <= n / 4 ? 1 : 0);
    }
    return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_launches(tmp_path):
    source, program = tmp_path / "p.cpp", tmp_path / "p"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(source), "-o", str(program)], check=True)
    limit = 1 << 35      # entries with 2^32 threads
    sizes = [(1 << 21) + 1, 1 << 31, (1 << 31) + 4099, limit - 2049, limit - 2048, limit - 1, limit, limit + 1, 1 << 36, 1 << 40]
    out = subprocess.run([str(program)], input="\n".join(map(str, sizes)), capture_output=True, text=True, check=True).stdout.split("\n")
    for n, line in zip(sizes, out):
        fits, allowed, covered = (int(x) for x in line.split())
        assert covered and fits == allowed == (n < limit - 2048), n
