// Direct-gather accumulators of a single problem.
#include "accum.h"

namespace spg {

// (the other kind is instantiated in its own file)
extern template hipError_t launch_acc_wave_t<true>(const KArgs &, int, int, bool, bool, bool,
                                                   hipStream_t);
extern template hipError_t launch_heavy_t<true>(const KArgs &, int, int, bool, bool, bool,
                                                hipStream_t, bool, long long, int, int);

// work items of a wave bin: 64 columns (one per lane: ESC sub-bins 0 and 1),
// groups of columns (the other ESC sub-bins) or columns (sort bins)
int wave_bin_items(int bin, int ncols) {
    if (bin >= BIN_ESC0 && bin < BIN_ESC0 + kLaneSubBins) return ceil_div(ncols, 64);
    if (bin >= BIN_ESC0 && bin < BIN_ESC0 + kEscBins) return ceil_div(ncols, 64 >> (bin - BIN_ESC0));
    return ncols;
}

// The heavy columns' launches one part at a time (the caller interleaves them
// with other streams' launches): windows take the map of windows, the
// expansion and the windowed sort; the radix ESC the expansion and the sort.
int heavy_parts(bool radix) { return radix ? 2 : 3; }
// the first part a launch needs: the windows' map is written by the place
// kernel of a planned launch, and stays from the counting launch to the
// filling ones that follow it
int heavy_first_part(bool radix, bool mapped) { return !radix && mapped ? 1 : 0; }

template hipError_t launch_acc_wave_t<false>(const KArgs &, int, int, bool, bool, bool, hipStream_t);
template hipError_t launch_heavy_t<false>(const KArgs &, int, int, bool, bool, bool, hipStream_t,
                                          bool, long long, int, int);

}  // namespace spg
