// The collision launch of the two-launch step that also forms the totals of the state it writes.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "split_launch.hpp"

namespace lbm {

hipError_t launch_split_collide_totals(int storage_bytes, const void* src, void* dst, const void* scratch,
                                       const StepGeom& g, const Phys& ph, const StepAux& aux, double* out,
                                       hipStream_t st)
{
    if (!aux.partials || !out) return hipErrorInvalidValue;
    const hipError_t e = storage_bytes == 4
                             ? split_launch::collide<float, float, true>(src, dst, scratch, g, ph, aux, st)
                             : split_launch::collide<double, double, true>(src, dst, scratch, g, ph, aux, st);
    if (e != hipSuccess) return e;
    return launch_sum_partials(aux.partials, step_workgroups(g), out, st);
}

}  // namespace lbm
