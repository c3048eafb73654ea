// Histograms that are added up in slices of the levels: which blocks do it, and for whom they wait (not installed; compiles without HIP).
#pragma once

#include <stdint.h>

#include "cdl_anywhere.h"

namespace cdl {

// Most blocks that finish a grid's histograms between them.
constexpr int kMargCollectors = 16;

// Levels of a slice, as a power of two: up to sixteen slices of 16 to 32 KB of what the blocks leave (8 bytes a level and block; one round of loads of 512 threads), or one of all.
// us of the forward pass, slices of 16 to 32 KB / at most 16 / at most 8: 1 M entries of 63 levels 9.6 / 10.3 / 10.9, 400 K of 40 8.4 / 9.0 / 9.2, 65536 of 255 7.8 / 8.2 / 8.6, 2.1 M of 255
// 13.0 / 13.0 / 13.3.
inline int marg_lg_per(int64_t blocks, int n_levels)
{
    int lg = 2;
    while ((1 << lg) < n_levels && ((n_levels + (1 << lg) - 1) >> lg > kMargCollectors || (blocks << lg) < 2048)) ++lg;
    return lg;
}
inline int marg_slices(int n_levels, int lg_per) { return (n_levels + (1 << lg_per) - 1) >> lg_per; }

// A launch has `workers` blocks, which share the entries and wait for nobody, and behind them `slices` collectors without entries: a collector waits for the rows of blocks
// 0 .. rows_from(), the last one also for the entropy terms of collectors 0 .. terms_from().  So all wait for blocks of lower numbers alone, and where blocks start in the order of their numbers
// (on each XCD: its share of them) a launch ends with any number of places, one among them: whoever waits has taken no place from those that it waits for.  (Collectors that have entries too need each
// other's rows: with fewer places than collectors nobody would end.)
struct MargRoles {
    int workers, slices;
    CDL_ANYWHERE bool collects(int block) const { return block >= workers; }
    CDL_ANYWHERE int collector(int block) const { return block - workers; }
    CDL_ANYWHERE int rows_from() const { return workers; }
    CDL_ANYWHERE int terms_from(int collector) const { return collector == slices - 1 ? slices - 1 : 0; }
    CDL_ANYWHERE int grid() const { return workers + slices; }
};

}  // namespace cdl
