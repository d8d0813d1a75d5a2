// The two-launch step: its moment launch and the collision launch without totals.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "split_launch.hpp"

namespace lbm {

size_t split_scratch_bytes(int storage_bytes, long long plane_nodes)
{
    return (size_t)plane_nodes * (2 * sizeof(double) + 5 * (size_t)storage_bytes);
}

void split_tile(int& tx, int& ty)
{
    tx = kSplitTX;
    ty = kSplitTY;
}

hipError_t launch_split_moments(int storage_bytes, const void* src, void* scratch, const StepGeom& g,
                                const Phys& ph, const StepAux& aux, hipStream_t st)
{
    const unsigned n = (unsigned)g.nx * (unsigned)g.ny * (unsigned)g.nz;
    const dim3 grid((n + kSplitThreads - 1) / kSplitThreads), block(kSplitThreads);
    const int ext = split_launch::ext_of(ph);
#define LBM_SPLIT_MOMENTS(T, EXT)                                                                        \
    hipLaunchKernelGGL((k_split_moments<19, T, T, EXT>), grid, block, 0, st, (const T*)src, scratch, g,  \
                       ph, aux)
    if (storage_bytes == 4) {
        if (ext == kExtTable) LBM_SPLIT_MOMENTS(float, kExtTable);
        else if (ext == kExtWalls) LBM_SPLIT_MOMENTS(float, kExtWalls);
        else LBM_SPLIT_MOMENTS(float, kExtNone);
    } else {
        if (ext == kExtTable) LBM_SPLIT_MOMENTS(double, kExtTable);
        else if (ext == kExtWalls) LBM_SPLIT_MOMENTS(double, kExtWalls);
        else LBM_SPLIT_MOMENTS(double, kExtNone);
    }
#undef LBM_SPLIT_MOMENTS
    return hipGetLastError();
}

hipError_t launch_split_collide(int storage_bytes, const void* src, void* dst, const void* scratch,
                                const StepGeom& g, const Phys& ph, const StepAux& aux, hipStream_t st)
{
    if (storage_bytes == 4)
        return split_launch::collide<float, float, false>(src, dst, scratch, g, ph, aux, st);
    return split_launch::collide<double, double, false>(src, dst, scratch, g, ph, aux, st);
}

}  // namespace lbm
