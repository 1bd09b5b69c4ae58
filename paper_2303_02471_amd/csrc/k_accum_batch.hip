// Direct-gather accumulators of a batch of problems.
#include "accum.h"

namespace spg {

// (the other kind is instantiated in its own file)
extern template hipError_t launch_acc_light_t<false>(const KArgs &, unsigned, int, bool, bool, bool,
                                               hipStream_t);
extern template hipError_t launch_acc_one_t<false>(const KArgs &, int, int, bool, bool, bool, hipStream_t);
extern template hipError_t launch_heavy_t<false>(const KArgs &, int, int, bool, bool, bool, hipStream_t,
                                           bool, long long, int, int, int);

template hipError_t launch_acc_light_t<true>(const KArgs &, unsigned, int, bool, bool, bool,
                                        hipStream_t);
template hipError_t launch_acc_one_t<true>(const KArgs &, int, int, bool, bool, bool, hipStream_t);
template hipError_t launch_heavy_t<true>(const KArgs &, int, int, bool, bool, bool, hipStream_t,
                                    bool, long long, int, int, int);

}  // namespace spg
