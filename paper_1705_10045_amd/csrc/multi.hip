// Launches of several D2Q9 steps at once (multi_kernel.hpp).
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "multi_kernel.hpp"

namespace lbm {

int multi_nodes() { return kMultiNodes; }

namespace {

template <class S, int NMODE>
hipError_t launch_n(const void* src, void* dst, const StepGeom& g, const MultiGeom& mg, const Phys& ph,
                    const StepAux& aux, hipStream_t st)
{
    const dim3 grid((unsigned)(g.ntx * g.nty)), block((unsigned)((mg.rx * mg.ry + 63) / 64 * 64));
#define LBM_MULTI(EXT)                                                                                \
    hipLaunchKernelGGL((k_multi_step<S, NMODE, EXT>), grid, block, 0, st, (const S*)src, (S*)dst, g, mg, \
                       ph, aux)
    if (ph.eos != 0) LBM_MULTI(kExtTable);
    else if (ph.g[0] != 0.0 || ph.g[1] != 0.0 || ph.g[2] != 0.0) LBM_MULTI(kExtWalls);
    else LBM_MULTI(kExtNone);
#undef LBM_MULTI
    return hipGetLastError();
}

template <class S>
hipError_t launch_s(const void* src, void* dst, const StepGeom& g, const MultiGeom& mg, const Phys& ph,
                    const StepAux& aux, hipStream_t st)
{
    if (ph.collision != 0) return launch_n<S, kMrt>(src, dst, g, mg, ph, aux, st);
    if (ph.omega == 1.0) return launch_n<S, kTauOne>(src, dst, g, mg, ph, aux, st);
    return launch_n<S, kTauAny>(src, dst, g, mg, ph, aux, st);
}

}  // namespace

hipError_t launch_multi(int storage_bytes, const void* src, void* dst, const StepGeom& g, const MultiGeom& mg,
                        const Phys& ph, const StepAux& aux, hipStream_t st)
{
    if (mg.rx * mg.ry > kMultiNodes || mg.steps < 1) return hipErrorInvalidValue;
    if (storage_bytes == 4) return launch_s<float>(src, dst, g, mg, ph, aux, st);
    return launch_s<double>(src, dst, g, mg, ph, aux, st);
}

}  // namespace lbm
