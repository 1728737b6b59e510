// The front propagation kernel (omap_front.h) and its launch.
#include "omap_front.h"

#include <initializer_list>

namespace omap {

hipError_t launch_front(const RoundArgs& a, int32_t grid, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    RoundArgs b = a;
    b.wave_stride = grid;   // tiles (visiting blocks) per pass over the list
    const auto kernel = a.dense ? (a.n_slots == 1 ? k_front<true, true> : k_front<false, true>)
                                : (a.n_slots == 1 ? k_front<true, false> : k_front<false, false>);
    if (e0 != nullptr)
        hipExtLaunchKernelGGL(kernel, dim3(grid + 1), dim3(kFrontThreads), 0, s, e0, e1, 0, b);
    else
        hipLaunchKernelGGL(kernel, dim3(grid + 1), dim3(kFrontThreads), 0, s, b);
    return hipGetLastError();
}

int front_blocks_per_cu() {
    int least = 0;
    for (auto kernel : {k_front<true, false>, k_front<false, false>, k_front<true, true>, k_front<false, true>}) {
        int blocks = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, kernel, kFrontThreads, 0) != hipSuccess) return 0;
        least = least == 0 || blocks < least ? blocks : least;
    }
    return least;
}

}  // namespace omap
