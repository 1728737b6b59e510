// The front propagation kernel (omap_front.h) and its launch.
#include "omap_front.h"

namespace omap {

hipError_t launch_front(const RoundArgs& a, int32_t grid, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
    RoundArgs b = a;
    b.wave_stride = grid;   // tiles (visiting blocks) per pass over the list
    if (e0 != nullptr)
        hipExtLaunchKernelGGL(k_front, dim3(grid + 1), dim3(kFrontThreads), 0, s, e0, e1, 0, b);
    else
        hipLaunchKernelGGL(k_front, dim3(grid + 1), dim3(kFrontThreads), 0, s, b);
    return hipGetLastError();
}

int front_blocks_per_cu() {
    int blocks = 0;
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k_front, kFrontThreads, 0);
    return e == hipSuccess ? blocks : 0;
}

}  // namespace omap
