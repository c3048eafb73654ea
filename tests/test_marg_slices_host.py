"""Host-side check of histograms added up in slices (cdl_marg_slices.h, compiled here for the CPU): every block waits for blocks of lower numbers alone, so that a launch ends on a device that starts blocks in
order with as little room as one place, on one XCD or dealt over eight; and the slices cover the levels, sixteen at most.  What a call launches is checked against the roles (launch_recorder.py)."""
import shutil
import subprocess

import pytest

import launch_recorder as lr

CSRC = lr.ROOT + "/paper_2501_09849_amd/csrc"

PROGRAM = r"""
#include <stdio.h>
#include <vector>
#include "cdl_marg_slices.h"
using namespace cdl;

// Blocks start in order, on each of `xcds` its share of them, as long as one of its `places` is free; a block leaves when all that it waits for have left what they publish (which the blocks with entries do when
// they run, collectors when their rows are there).
static bool ends(const MargRoles &r, int places, int xcds)
{
    const int grid = r.grid();
    std::vector<int> state(grid, 0), next(xcds), held(xcds, 0);      // 0: not started, 1: running, 2: over
    for (int x = 0; x < xcds; ++x) next[x] = x;
    int left = grid;
    for (bool moved = true; moved && left > 0;) {
        moved = false;
        for (int x = 0; x < xcds; ++x)
            while (next[x] < grid && held[x] < places) { state[next[x]] = 1; next[x] += xcds; ++held[x]; moved = true; }
        for (int b = 0; b < grid; ++b) {
            if (state[b] != 1) continue;
            bool over = true;
            if (r.collects(b)) {
                for (int i = 0; i < r.rows_from(); ++i) over = over && state[i] == 2;
                for (int c = 0; c < r.terms_from(r.collector(b)); ++c) over = over && state[r.workers + c] == 2;
            }
            if (over) { state[b] = 2; --held[b % xcds]; --left; moved = true; }
        }
    }
    return left == 0;
}

int main()
{
    int workers, levels;
    while (scanf("%d %d", &workers, &levels) == 2) {
        const int lg = marg_lg_per(workers, levels);
        const MargRoles r{workers, marg_slices(levels, lg)};
        int later = 0;
        for (int b = 0; b < r.grid(); ++b)
            if (r.collects(b) && (r.rows_from() > b || (r.terms_from(r.collector(b)) > 0 && r.workers + r.terms_from(r.collector(b)) > b))) ++later;
        const bool all = ends(r, 1, 1) && ends(r, 2, 1) && ends(r, 1, 8) && ends(r, 3, 8);
        printf("%d %d %d %d %d\n", r.slices, later, all ? 1 : 0, (r.slices << lg) >= levels && ((r.slices - 1) << lg) < levels ? 1 : 0, r.grid());
    }
    return 0;
}
"""
needs_compiler = pytest.mark.skipif(shutil.which("g++") is None or shutil.which("c++filt") is None, reason="no host compiler")


def _roles(tmp_path, cases):
    source, program = tmp_path / "p.cpp", tmp_path / "p"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(source), "-o", str(program)], check=True)
    out = subprocess.run([str(program)], input="\n".join("%d %d" % c for c in cases), capture_output=True, text=True, check=True).stdout
    return [[int(v) for v in line.split()] for line in out.splitlines()]


@needs_compiler
def test_every_wait_is_for_lower_numbers(tmp_path):
    cases = [(w, lv) for w in (1, 2, 17, 64, 133, 250, 255, 256) for lv in (2, 3, 30, 31, 63, 64, 66, 127, 200, 255, 256)]
    for case, (slices, later, ends, covered, _) in zip(cases, _roles(tmp_path, cases)):
        assert slices <= 16 and later == 0 and ends and covered, case


@needs_compiler
def test_launches_have_the_collectors_behind_the_blocks_with_entries(tmp_path):
    # (blocks of 512 threads and four entries a trip, as many trips as leave 256 of them)
    workers = [171, 129, 256, 256, 17, 212]
    sizes = [(700_001, 30), (524_289, 255), (2_097_152, 255), (256 * 2048 - 4, 63), (17 * 2048 - 1, 256), (1_300_002, 66)]
    calls = []
    for n, levels in sizes:
        lo = 0 if levels > 255 else -(levels // 2)
        calls.append(("cdl_quantize_fwd", [(lr.POINTER, lr.A), (lr.INT64, n), (lr.QPARAMS, [lo, levels, 0.0625, 4.0 * 256.0, 0]), (lr.POINTER, lr.A), (lr.POINTER, lr.A), (lr.POINTER, lr.A), (lr.POINTER, lr.A),
                      (lr.POINTER, lr.A), (lr.SIZE, 1 << 30), (lr.POINTER, None)]))
    roles = _roles(tmp_path, list(zip(workers, (lv for _, lv in sizes))))
    for size, (launches, _), role in zip(sizes, lr.record(tmp_path, calls), roles):
        assert len(launches) == 1 and ", 2, 1>" in launches[0].name, (size, launches)      # (FORM = slices, one launch)
        assert launches[0].grid == (role[4], 1, 1), (size, launches, role)
