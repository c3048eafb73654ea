"""Host-side check of the activation gradient of convolutions from patches: the plan and the walk through the weights are the kernel's own
(cdl_conv_patch.h), compiled here for the CPU.  Every byte that a wave asks for, ahead of its multiplications too, lies in the weights of its
class, for every limb count and every part of the channels, over shapes of the whole range."""
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
        printf("%d %d %lld\n", p.served ? 1 : 0, parts, over);
    }
    return 0;
}
"""

# one part of 32 channels each (a prime number of them) and an odd number of taps: the furthest a walk can step
FAR = [(1, 11, 11, 1280, 992, 3, 3, 1, 1), (4, 7, 7, 1408, 544, 3, 3, 1, 0), (5, 5, 5, 1792, 544, 3, 3, 1, 0), (27, 3, 3, 500, 984, 3, 3, 1, 0),
       (4, 56, 56, 128, 224, 5, 5, 1, 2), (8, 28, 28, 96, 352, 3, 3, 2, 1)]


def _shapes(count):
    rng = random.Random(11)
    out = list(FAR)
    while len(out) < count:
        R, S, stride = rng.choice([1, 2, 3, 3, 4, 5, 7]), rng.choice([1, 2, 3, 3, 4, 5, 7]), rng.choice([1, 1, 2])
        H, W = rng.randint(max(R, 2), 60), rng.randint(max(S, 2), 60)
        pad = rng.randint(0, min(R, S) - 1)
        C, N = 4 * rng.randint(1, 500), 4 * rng.randint(1, 256)
        if R * S * N <= 131071:
            out.append((rng.randint(1, 64), H, W, C, N, R, S, stride, pad))
    return out


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_weights_asked_for_lie_in_their_class(tmp_path):
    source, program = tmp_path / "walk.cpp", tmp_path / "walk"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(source), "-o", str(program)], check=True)
    shapes = _shapes(4000)
    res = subprocess.run([str(program)], input="\n".join(" ".join(map(str, s)) for s in shapes), stdout=subprocess.PIPE, text=True, check=True)
    lines = [tuple(map(int, line.split())) for line in res.stdout.splitlines()]
    assert len(lines) == len(shapes)
    assert all(served and parts > 1 for served, parts, _ in lines[:len(FAR)])
    assert sum(served for served, _, _ in lines) > 1000
    over = [(s, line[2]) for s, line in zip(shapes, lines) if line[2] > 0]
    assert not over, "%d shapes, the furthest %s" % (len(over), max(over, key=lambda o: o[1]))
