// Plan of the activation gradient of convolutions from patches of g: host arithmetic and the walk through the weights, which the kernel
// (cdl_conv_patch.hip) and the checks on the host share (not installed).
#pragma once

#include <stdint.h>

#include "cdl_anywhere.h"

namespace cdl {

// A class of input pixels (2 i + oa, 2 j + oc) and the taps (r0 + 2 r', s0 + 2 s'), r' < Rc, s' < Sc, that reach them (stride 1: one class,
// every pixel and tap, steps of 1).
struct ConvDxGrid { int oa, oc, Hc, Wc, pad_h, pad_w, Rc, Sc, r0, s0; };

// The classes of input pixels.  Stride 1: all of them, every tap.  Stride 2: input pixel (h, w) is reached only by the
// taps r = h + pad, s = w + pad (mod 2) - with all R x S taps three products in four would multiply zeros -, so the
// pixels (2 i + a, 2 j + c) of each parity (a, c) form a product of their own over the taps r = r0 + 2 r',
// s = s0 + 2 s' (r0 = (a + pad) mod 2, likewise s0), in which g is read at p = i + (a + pad - r0) / 2 - r'.
// Returns their number; unreached: there are pixels that no tap reaches.
inline int conv_dx_classes(int32_t H, int32_t W, int32_t R, int32_t S, int32_t stride, int32_t pad, ConvDxGrid (&grids)[4], bool &unreached)
{
    int n = 0;
    unreached = false;
    if (stride == 1) {
        grids[n++] = ConvDxGrid{0, 0, H, W, pad, pad, R, S, 0, 0};
        return n;
    }
    for (int pa = 0; pa < 2; ++pa)
        for (int pc = 0; pc < 2; ++pc) {
            const int Hc = (H - pa + 1) / 2, Wc = (W - pc + 1) / 2;
            if (Hc <= 0 || Wc <= 0) continue;
            const int r0 = (pa + pad) & 1, s0 = (pc + pad) & 1;
            const int Rc = r0 < R ? (R - r0 + 1) / 2 : 0, Sc = s0 < S ? (S - s0 + 1) / 2 : 0;
            if (Rc == 0 || Sc == 0) { unreached = true; continue; }
            grids[n++] = ConvDxGrid{pa, pc, Hc, Wc, (pa + pad - r0) / 2, (pc + pad - s0) / 2, Rc, Sc, r0, s0};
        }
    return n;
}

constexpr int kPatchThreads = 256;
constexpr int kPatchLds = 80 << 10;          // two blocks share a compute unit
constexpr int kPatchFixed = 64;              // bytes for the reductions
// At least four limbs: relative to a block's largest entry they leave 2^-32, below the rounding of the fp32 result.  (Three keep the bound where the
// steps and indices are small; outputs 2.5e-8 -> 9e-8 of their norm.)
constexpr int kPatchMinLimbs = 4, kPatchMaxLimbs = 6;

// Four waves: WN = 1, 2, 4 as (4 / WN) x WN, 32 pixels by 64 channels each, of the one class; WN = 0: a wave for each class, 32 grid
// pixels by 64 channels (four classes read the same patch, and no wave has to load weights behind stores: a wave's loads wait for
// its older stores, which take microseconds).
constexpr int patch_rows(int wn) { return wn == 0 ? 32 : 32 * (4 / wn); }
constexpr int patch_cols(int wn) { return wn == 0 ? 64 : 64 * wn; }

// The grid that the classes share, and what a pixel of it reads.
struct PatchGrid { int Hm, Wm, lo_h, hi_h, lo_w, hi_w; };

inline PatchGrid patch_grid(const ConvDxGrid *grids, int n)
{
    PatchGrid p{0, 0, 1 << 30, -(1 << 30), 1 << 30, -(1 << 30)};
    auto least = [](int &a, int b) { if (b < a) a = b; };
    auto most = [](int &a, int b) { if (b > a) a = b; };
    for (int i = 0; i < n; ++i) {
        const ConvDxGrid &s = grids[i];
        most(p.Hm, s.Hc);
        most(p.Wm, s.Wc);
        least(p.lo_h, s.pad_h - s.Rc + 1);
        most(p.hi_h, s.pad_h);
        least(p.lo_w, s.pad_w - s.Sc + 1);
        most(p.hi_w, s.pad_w);
    }
    return p;
}

// Pixels of g that a run of `rows` pixels of the grid needs, at most: from what the first one reads first to what the last one reads
// last, with what g's rows and images have more than the grid's at every end of a row and an image.
inline int64_t patch_pixels(const PatchGrid &s, int rows, int P, int Q, int64_t all)
{
    const int64_t hw = (int64_t)s.Hm * s.Wm, row_ends = (rows - 2 + s.Wm) / s.Wm, image_ends = (rows - 2 + hw) / hw;
    int64_t n = rows + (int64_t)(s.hi_h - s.lo_h) * Q + s.hi_w - s.lo_w;
    if (Q > s.Wm) n += row_ends * (Q - s.Wm);
    if (P > s.Hm) n += image_ends * (int64_t)(P - s.Hm) * Q;
    // (pixels beyond the last window: their range begins at the image's last row or pixel instead)
    if (s.Hm - 1 + s.lo_h > P - 1) n += (int64_t)(s.Hm + s.lo_h - P) * Q;
    if (s.Wm - 1 + s.lo_w > Q - 1) n += s.Wm + s.lo_w - Q;
    return n < all ? n : all;
}

struct PatchPlan {
    bool served;
    int wn, px_max, taps;
    int nc[kPatchMaxLimbs + 1];
};

// The tile of 32 x 256, 64 x 128 or 128 x 64 outputs that pads the channels least (of equals the widest, which needs the smallest
// patch; several classes: 32 x 64 of each), and the channels of a patch that fit LDS: all of them or an equal part, a multiple of 32, of at most
// four a thread (a thread makes the digits of one word of a pixel's row; more fit LDS where g has up to some eighteen pixels).
inline PatchPlan plan_patch(const ConvDxGrid *grids, int n_grids, int64_t B, int P, int Q, int C, int Np)
{
    PatchPlan best{};
    int64_t least = 0;
    const PatchGrid grid = patch_grid(grids, n_grids);
    if (n_grids < 1 || B * grid.Hm * grid.Wm > 2147483647LL) return best;
    for (int wn = n_grids > 1 ? 0 : 4; wn >= 0; wn = wn > 1 ? wn / 2 : -1) {
        const int rows = patch_rows(wn), cols = patch_cols(wn);
        const int64_t padded = (int64_t)((C + cols - 1) / cols) * cols;
        if (best.served && padded >= least) continue;
        PatchPlan p{};
        p.served = true;
        p.wn = wn;
        for (int i = 0; i < n_grids; ++i)
            if (grids[i].Rc * grids[i].Sc > p.taps) p.taps = grids[i].Rc * grids[i].Sc;
        const int64_t px = patch_pixels(grid, rows, P, Q, B * P * Q);
        if (px > 4096) continue;
        p.px_max = (int)px;
        for (int l = kPatchMinLimbs; l <= kPatchMaxLimbs; ++l) {
            p.nc[l] = 0;
            for (int parts = 1; parts <= Np / 32 && !p.nc[l]; ++parts)
                if (Np / 32 % parts == 0 && Np / parts <= 4 * kPatchThreads && kPatchFixed + 2ll * n_grids * (p.taps + 1) * rows + l * (px + 1) * (Np / parts + 16) <= kPatchLds) p.nc[l] = Np / parts;
            p.served = p.served && p.nc[l] != 0;
        }
        if (!p.served) continue;
        best = p;
        least = padded;
    }
    // A block takes about 12 us beside its k-steps (0.28 us each), which short contractions do not pay for once there are enough blocks for
    // the passes that this kernel does without (15 - 25 us) not to count.  Digits made beforehand / patches, us: 59 x 52 x 52 x 240 -> 48, 3 x 3
    // (18 steps, 5 K blocks)  129 / 150;  195 x 38 x 38 x 96 -> 24 (9, 4.4 K)  101 / 108;  19 x 45 x 45 x 208 -> 36 (18, 1.2 K)  49 / 45;
    // 27 x 56 x 56 x 64 -> 24 (9, 0.7 K)  44 / 31.
    int taps = 0;
    for (int i = 0; i < n_grids; ++i) taps += grids[i].Rc * grids[i].Sc;
    if (best.served && taps * (Np / 32) < 20) {
        const int rows = patch_rows(best.wn), cols = patch_cols(best.wn);
        if ((B * grid.Hm * grid.Wm + rows - 1) / rows * ((C + cols - 1) / cols) > 2000) best.served = false;
    }
    return best;
}

// The weights of one part of a patch's channels, [taps][channels / 32] k-steps, in the order in which they are multiplied: byte offset, from the
// class's weights on, of the step that is loaded next.  Behind the last step it stays there: what is asked for ahead is then the last step again.
struct PatchWeights {
    int64_t at, step, skip;      // skip: to the next tap's part
    int per_tap, in_tap, left;
    CDL_ANYWHERE PatchWeights(int n0, int nc, int Np, int C32, int steps)
        : at((int64_t)(n0 >> 5) * C32 * 32), step((int64_t)C32 * 32), skip((int64_t)((Np - nc) >> 5) * C32 * 32), per_tap(nc >> 5), in_tap(nc >> 5), left(steps) {}
    CDL_ANYWHERE void next()
    {
        --in_tap;
        --left;
        at += left > 0 ? step + (in_tap == 0 ? skip : 0) : 0;
        in_tap = in_tap == 0 ? per_tap : in_tap;
    }
};
// k-steps ahead of their multiplication that weights are asked for; a wave asks for as many more than the steps that it carries out, which are
// an even number: an odd one is followed by one on rows of zeros.
constexpr int patch_ahead(int limbs) { return limbs <= 4 ? 4 : (limbs == 5 ? 2 : 1); }

}  // namespace cdl
