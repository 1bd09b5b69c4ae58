// Direct-gather accumulators of a single problem.
#include "accum.h"

namespace spg {

// (the other kind is instantiated in its own file)
extern template hipError_t launch_acc_light_t<true>(const KArgs &, unsigned, int, bool, bool, bool,
                                               hipStream_t);
extern template hipError_t launch_acc_one_t<true>(const KArgs &, int, int, bool, bool, bool, hipStream_t);
extern template hipError_t launch_heavy_t<true>(const KArgs &, int, int, bool, bool, bool, hipStream_t,
                                           bool, long long, int, int, int);

// work items of the light bins of `mask` with these column counts
int light_items(const int32_t *bin_count, unsigned mask) {
    int n = 0;
    for (int i = 0; i < kLightBins; ++i)
        if ((mask >> i) & 1u) n += ceil_div(bin_count[BIN_ESC0 + i], light_columns(i));
    return n;
}

// The heavy columns' launches one part at a time (the caller interleaves them
// with other streams' launches): windows take the map of windows, the
// expansion and the windowed sort; the radix ESC the expansion and the sort.
int heavy_parts(bool radix) { return radix ? 2 : 3; }
// the first part a launch needs: the windows' map is written by the place
// kernel of a planned launch, and stays from the counting launch to the
// filling ones that follow it
int heavy_first_part(bool radix, bool mapped) { return !radix && mapped ? 1 : 0; }

template hipError_t launch_acc_light_t<false>(const KArgs &, unsigned, int, bool, bool, bool,
                                        hipStream_t);
template hipError_t launch_acc_one_t<false>(const KArgs &, int, int, bool, bool, bool, hipStream_t);
template hipError_t launch_heavy_t<false>(const KArgs &, int, int, bool, bool, bool, hipStream_t,
                                    bool, long long, int, int, int);

}  // namespace spg
