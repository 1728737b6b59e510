// The front propagation kernel (omap_front.h) and its launch.
#include "omap_front.h"

namespace omap {

hipError_t launch_front(const RoundArgs& a, int32_t grid, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    RoundArgs b = a;
    b.wave_stride = grid;   // tiles (visiting blocks) per pass over the list
    const auto kernel = a.n_slots == 1 ? k_front<true> : k_front<false>;
    if (e0 != nullptr)
        hipExtLaunchKernelGGL(kernel, dim3(grid + 1), dim3(kFrontThreads), 0, s, e0, e1, 0, b);
    else
        hipLaunchKernelGGL(kernel, dim3(grid + 1), dim3(kFrontThreads), 0, s, b);
    return hipGetLastError();
}

int front_blocks_per_cu() {
    int one = 0, many = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&one, k_front<true>, kFrontThreads, 0) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&many, k_front<false>, kFrontThreads, 0) != hipSuccess)
        return 0;
    return one < many ? one : many;
}

}  // namespace omap
