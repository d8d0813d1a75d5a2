// Instantiation choice of the two-launch step, shared by the plain launches and those that also
// form the state's totals.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "split_kernel.hpp"

namespace lbm {
namespace split_launch {

// 0 periodic, 1 walls or body force, 2 tabulated equation of state
inline int ext_of(const Phys& ph)
{
    if (ph.eos != 0) return kExtTable;
    return ph.walls || ph.g[0] != 0.0 || ph.g[1] != 0.0 || ph.g[2] != 0.0 ? kExtWalls : kExtNone;
}

template <class S, class R, int NMODE, bool RED>
hipError_t collide_n(const void* src, void* dst, const void* scratch, const StepGeom& g, const Phys& ph,
                     const StepAux& aux, hipStream_t st)
{
    const dim3 grid((unsigned)(g.ntx * g.nty * g.nchunks)), block(kSplitThreads);
#define LBM_SPLIT_COLLIDE(EXT)                                                                          \
    hipLaunchKernelGGL((k_split_collide<19, S, R, NMODE, EXT, RED>), grid, block, 0, st, (const S*)src, \
                       (S*)dst, scratch, g, ph, aux)
    switch (ext_of(ph)) {
    case kExtTable: LBM_SPLIT_COLLIDE(kExtTable); break;
    case kExtWalls: LBM_SPLIT_COLLIDE(kExtWalls); break;
    default: LBM_SPLIT_COLLIDE(kExtNone); break;
    }
#undef LBM_SPLIT_COLLIDE
    return hipGetLastError();
}

// tau = 1 with BGK does not read the density populations again
template <class S, class R, bool RED>
hipError_t collide(const void* src, void* dst, const void* scratch, const StepGeom& g, const Phys& ph,
                   const StepAux& aux, hipStream_t st)
{
    if (ph.collision != 0) return collide_n<S, R, kMrt, RED>(src, dst, scratch, g, ph, aux, st);
    if (ph.omega == 1.0) return collide_n<S, R, kTauOne, RED>(src, dst, scratch, g, ph, aux, st);
    return collide_n<S, R, kTauAny, RED>(src, dst, scratch, g, ph, aux, st);
}

}  // namespace split_launch
}  // namespace lbm
