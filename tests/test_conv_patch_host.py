"""Host-side check of the activation gradient of convolutions from patches: the plan and the walk through the weights are the kernel's own
(cdl_conv_patch.h), compiled here for the CPU.  Every byte that a wave asks for, ahead of its multiplications too, lies in the weights of its
class, for every limb count and every part of the channels, and a patch has a thread for each word and room in LDS, over shapes of the whole range."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_09849_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include "cdl_conv_patch.h"
using namespace cdl;

int main()
{
    int B, H, W, C, N, R, S, stride, pad;
    while (scanf("%d %d %d %d %d %d %d %d %d", &B, &H, &W, &C, &N, &R, &S, &stride, &pad) == 9) {
        const int P = (H + 2 * pad - R) / stride + 1, Q = (W + 2 * pad - S) / stride + 1, Np = (N + 31) / 32 * 32, C32 = (C + 31) / 32 * 32;
        ConvDxGrid grids[4];
        bool unreached;
        const int n = conv_dx_classes(H, W, R, S, stride, pad, grids, unreached);
        const PatchPlan p = plan_patch(grids, n, B, P, Q, C, Np);
        long long over = 0;
        int parts = 0;
        for (int c = 0; p.served && c < n; ++c)
            for (int L = kPatchMinLimbs; L <= kPatchMaxLimbs; ++L) {
                const int taps = grids[c].Rc * grids[c].Sc, nc = p.nc[L], nk = taps * (nc / 32);
                if (Np / nc > parts) parts = Np / nc;
                const long long own = (long long)taps * Np * C32;      // bytes of the class
                for (int n0 = 0; n0 < Np; n0 += nc) {
                    PatchWeights w(n0, nc, Np, C32, nk);
                    for (int load = 0; load < patch_ahead(L) + ((nk + 1) & ~1); ++load) {
                        // the first nk loads are the class's entries of these channels, tap by tap
                        const long long at = ((long long)(load / (nc / 32)) * Np + n0 + 32 * (load % (nc / 32))) * C32;
                        if (load < nk && w.at != at) { printf("order %d %d %d\n", c, L, load); return 1; }
                        if (w.at < 0 || w.at + (long long)C32 * 32 - own > over) over = w.at + (long long)C32 * 32 - own;
                        w.next();
                    }
                }
            }
        // what the kernel takes for granted: a thread for each word of a pixel's row, LDS, 16-bit rows in the table
        int broken = 0;
        for (int L = kPatchMinLimbs; p.served && L <= kPatchMaxLimbs; ++L) {
            const int nc = p.nc[L], rows = patch_rows(p.wn);
            if (nc < 32 || nc % 32 != 0 || Np % nc != 0 || nc / 4 > kPatchThreads) broken |= 1;
            if (kPatchFixed + 2ll * n * (p.taps + 1) * rows + (long long)L * (p.px_max + 1) * (nc + 16) > kPatchLds) broken |= 2;
            if (p.px_max < 1 || p.px_max > 65535 || p.px_max > (long long)B * P * Q) broken |= 4;
        }
        printf("%d %d %lld %d\n", p.served ? 1 : 0, parts, over, broken);
    }
    return 0;
}
"""

# one part of 32 channels each (a prime number of them) and an odd number of taps: the furthest a walk can step
FAR = [(1, 11, 11, 1280, 992, 3, 3, 1, 1), (4, 7, 7, 1408, 544, 3, 3, 1, 0), (5, 5, 5, 1792, 544, 3, 3, 1, 0), (27, 3, 3, 500, 984, 3, 3, 1, 0),
       (4, 56, 56, 128, 224, 5, 5, 1, 2), (8, 28, 28, 96, 352, 3, 3, 2, 1)]


# few pixels of g and more channels than a block has words for: a fully connected head as a convolution
HEADS = [(1, 7, 7, 512, 2048, 7, 7, 1, 0), (4, 7, 7, 512, 1280, 7, 7, 1, 0), (8, 7, 7, 512, 2048, 7, 7, 1, 0), (16, 7, 7, 512, 1056, 7, 7, 1, 0),
         (2, 5, 5, 2048, 4096, 5, 5, 1, 0)]


def _shapes(count):
    rng = random.Random(11)
    out = FAR + HEADS
    while len(out) < count // 4:
        R, S = rng.randint(1, 7), rng.randint(1, 7)
        geom = (rng.randint(1, 24), R + rng.randint(0, 2), S + rng.randint(0, 2), 4 * rng.randint(1, 500), 4 * rng.randint(256, 1024), R, S, rng.choice([1, 2]), 0)
        if R * S * geom[4] <= 131071:
            out.append(geom)
    while len(out) < count:
        R, S, stride = rng.choice([1, 2, 3, 3, 4, 5, 7]), rng.choice([1, 2, 3, 3, 4, 5, 7]), rng.choice([1, 1, 2])
        H, W = rng.randint(max(R, 2), 60), rng.randint(max(S, 2), 60)
        pad = rng.randint(0, min(R, S) - 1)
        C, N = 4 * rng.randint(1, 500), 4 * rng.randint(1, 256)
        if R * S * N <= 131071:
            out.append((rng.randint(1, 64), H, W, C, N, R, S, stride, pad))
    return out


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_plan_and_walk(tmp_path):
    source, program = tmp_path / "walk.cpp", tmp_path / "walk"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(source), "-o", str(program)], check=True)
    shapes = _shapes(4000)
    res = subprocess.run([str(program)], input="\n".join(" ".join(map(str, s)) for s in shapes), stdout=subprocess.PIPE, text=True, check=True)
    lines = [tuple(map(int, line.split())) for line in res.stdout.splitlines()]
    assert len(lines) == len(shapes)
    assert all(served and parts > 1 for served, parts, *_ in lines[:len(FAR)])
    assert all(served for served, *_ in lines[len(FAR):len(FAR) + len(HEADS)])
    assert sum(served for served, *_ in lines) > 1000
    broken = [(s, line[3]) for s, line in zip(shapes, lines) if line[3]]
    assert not broken, broken[:5]
    over = [(s, line[2]) for s, line in zip(shapes, lines) if line[2] > 0]
    assert not over, "%d shapes, the furthest %s" % (len(over), max(over, key=lambda o: o[1]))
