// Instantiations of the replicated-sharing DReLU / ReLU kernel (Alg. drelu2)
// for 64-bit share storage, one kernel per window count N = l_x + 1 in
// [30, 33] (a source of its own, so that the two compile side by side).
#include "rss_kernel.h"

namespace bc {

hipError_t launch_rss_u64_top(const RssLaunch& L, hipStream_t st) {
    return launch_rss_range<uint64_t, 30, 33>(L, st);
}

}  // namespace bc
