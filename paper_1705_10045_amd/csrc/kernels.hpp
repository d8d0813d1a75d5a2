// Launch interface between the host library and the device kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "physics.hpp"

namespace lbm {

// Geometry of one fused step launch.
struct StepGeom {
    int nx, ny, nz;
    int pitch;              // elements between consecutive x rows of a plane (>= nx)
    long long plane;        // elements between consecutive population planes
    int ntx, nty;           // tiles along x and y
    int chunk;              // z planes per workgroup
    int nchunks;
    int resident;           // workgroups of one round of the placement, 0 for the whole launch: what the GPU holds at
                            // once (D2Q9: of two per CU; rounds of one to eight made 3% of difference)
    double inv_nx, inv_ny, inv_ntx, inv_nty;   // reciprocals for index divisions (set_reciprocals)
};

inline void set_reciprocals(StepGeom& g)
{
    g.inv_nx = 1.0 / g.nx;
    g.inv_ny = 1.0 / g.ny;
    g.inv_ntx = 1.0 / g.ntx;
    g.inv_nty = 1.0 / g.nty;
}

// Read-only tables and the error word shared by every step launch of a simulation.
struct StepAux {
    const double* __restrict__ maxwell;  // band-limit table (reduced densities)
    double tab_s0, tab_inv_ds;
    int* err;                            // device error word (atomicOr)
    const double* __restrict__ eos_p;    // tabulated EOS (Phys::eos = 1): reduced pressures
    const double* __restrict__ eos_coex; // and its coexistence band per row
    double* partials;                    // steps that also form the state's totals: 5 per
                                         // workgroup (mass, momentum x/y/z, energy)
};

int step_variants(int Q, int storage_bytes);
void step_tile(int Q, int storage_bytes, int variant, int& tx, int& ty, int& per_cu);
hipError_t launch_step(int Q, int storage_bytes, int variant, const void* src, void* dst,
                       const StepGeom& g, const Phys& ph, const StepAux& aux, hipStream_t st);
// The same step, which also sums the totals of the state it writes (as launch_reduce would sum
// them) into aux.partials, one entry of 5 per workgroup, and then into out[5].  Exists for the
// default variants (0 of every lattice and storage, 2 of D2Q9, 5 of FP32 D3Q19); the others
// return hipErrorNotSupported before launching anything.
hipError_t launch_step_totals(int Q, int storage_bytes, int variant, const void* src, void* dst,
                              const StepGeom& g, const Phys& ph, const StepAux& aux, double* out,
                              hipStream_t st);
// The two-launch D3Q19 step (split_kernel.hpp) on states under 4 GB: the moments of src into
// `scratch` (split_scratch_bytes for plane_nodes = pitch * ny * nz elements), then the collision
// launch on the tiles of split_tile; the second form also sums the totals of the state it writes
// into aux.partials (5 per workgroup) and then into out[5].
size_t split_scratch_bytes(int storage_bytes, long long plane_nodes);
void split_tile(int& tx, int& ty);
hipError_t launch_split_moments(int storage_bytes, const void* src, void* scratch, const StepGeom& g,
                                const Phys& ph, const StepAux& aux, hipStream_t st);
hipError_t launch_split_collide(int storage_bytes, const void* src, void* dst, const void* scratch,
                                const StepGeom& g, const Phys& ph, const StepAux& aux, hipStream_t st);
hipError_t launch_split_collide_totals(int storage_bytes, const void* src, void* dst, const void* scratch,
                                       const StepGeom& g, const Phys& ph, const StepAux& aux, double* out,
                                       hipStream_t st);
// A launch of several D2Q9 steps at once (multi_kernel.hpp): tiles of tx x ty nodes (StepGeom::ntx,
// nty of them) with a halo of 3 steps - 1 nodes, a region of rx x ry <= multi_nodes() nodes.
struct MultiGeom {
    int tx, ty, steps;
    int margin;             // 3 * steps - 1
    int rx, ry;             // tx + 2 margin, ty + 2 margin (1 in a box of one row)
    double inv_rx;
};
int multi_nodes();
hipError_t launch_multi(int storage_bytes, const void* src, void* dst, const StepGeom& g, const MultiGeom& mg,
                        const Phys& ph, const StepAux& aux, hipStream_t st);
// workgroups of one step launch (the entries of aux.partials it writes)
inline long long step_workgroups(const StepGeom& g) { return (long long)g.ntx * g.nty * g.nchunks; }
// Row pitch of the population planes: x rows padded to whole 128-byte lines, so that rows of
// every width start line-aligned (a tile row then loads and stores whole lines).
inline int row_pitch(int nx, int storage_bytes)
{
    const int per_line = 128 / storage_bytes;
    return (nx + per_line - 1) / per_line * per_line;
}
hipError_t launch_init(int Q, int storage_bytes, void* buf, const double* rho0, const double* u0,
                       const double* T0, int nx, int ny, int nz, int pitch, long long plane,
                       double c_v, int walls, hipStream_t st);
hipError_t launch_moments(int Q, int storage_bytes, const void* buf, double* scratch, int nx, int ny,
                          int nz, int pitch, long long plane, const Phys& ph, const double* eos_p,
                          int* err, double* rho, double* us, double* E, double* T, hipStream_t st);
int reduce_blocks(long long n);
// n: buffer elements of one population plane to sum (row padding is zero; a multiple of 16
// bytes' worth of elements, as the row pitch makes it)
hipError_t launch_reduce(int Q, int storage_bytes, const void* buf, long long n, long long plane,
                         double* partials, int nblocks, double* out, hipStream_t st);
// out[0..4] = the sums over nblocks entries of 5 partial totals, in a fixed order
hipError_t launch_sum_partials(const double* partials, long long nblocks, double* out, hipStream_t st);

}  // namespace lbm
