// Device kernels of the thermal multiphase LBM library and their launchers.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "lattice.hpp"
#include "physics.hpp"
#include "step_launch.hpp"

namespace lbm {

using step_launch::launch_step_t;

namespace {

// Node of thread `id` (x fastest) of a box, and its neighbours' coordinates on the periodic axes.
// The extents' reciprocals come from the host: three integer remainders per direction, in 64 bits,
// took the moment kernels as long as their memory traffic.
struct BoxIndex {
    int nx, ny, nz, pitch;
    double inv_nx, inv_ny;
};

BoxIndex box_index(int nx, int ny, int nz, int pitch)
{
    return BoxIndex{nx, ny, nz, pitch, 1.0 / nx, 1.0 / ny};
}

struct NodeIndex {
    int x[3], y[3], z[3];   // coordinate - 1, itself, + 1, wrapped
    __device__ __forceinline__ NodeIndex(unsigned id, const BoxIndex& b)
    {
        const unsigned row = div_by(id, b.inv_nx), zz = div_by(row, b.inv_ny);
        x[1] = (int)(id - row * (unsigned)b.nx);
        y[1] = (int)(row - zz * (unsigned)b.ny);
        z[1] = (int)zz;
        x[0] = wrap_dec(x[1], b.nx); x[2] = wrap_inc(x[1], b.nx);
        y[0] = wrap_dec(y[1], b.ny); y[2] = wrap_inc(y[1], b.ny);
        z[0] = wrap_dec(z[1], b.nz); z[2] = wrap_inc(z[1], b.nz);
    }
    // element of the node displaced by (dx, dy, dz) in a field with rows of the given length
    __device__ __forceinline__ unsigned at(int dx, int dy, int dz, int row, int ny) const
    {
        return (unsigned)x[1 + dx] + (unsigned)row * ((unsigned)y[1 + dy] + (unsigned)ny * (unsigned)z[1 + dz]);
    }
};

// Equilibrium initial state N_k = rho0 P_k(u0), g_k = rho0 c_v T0 P_k(u0) (eq:feq, section 4),
// stored in pull form: node y keeps, for direction k, the value belonging to node y + c_k.  Each
// node reads its five fields once and scatters (gathering them from the 18 neighbours took twice
// as long).
template <int Q, class S>
__global__ void k_init(S* __restrict__ buf, const double* __restrict__ rho0,
                       const double* __restrict__ u0, const double* __restrict__ T0, const BoxIndex box,
                       long long plane, double c_v, int walls)
{
    using L = Lattice<Q>;
    const unsigned n = (unsigned)box.nx * (unsigned)box.ny * (unsigned)box.nz;
    const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const NodeIndex node(i, box);
    const int z = node.z[1];
    const unsigned own = node.at(0, 0, 0, box.pitch, box.ny);
    const double rho = rho0[i];
    const double ux = u0[i], uy = u0[(long long)n + i], uz = u0[2 * (long long)n + i];
    const double E = rho * c_v * T0[i];
    const double uu = ux * ux + uy * uy + uz * uz;
    // the node scatters its own equilibrium: direction k of it is stored at the node it is pulled
    // from, or, where that is beyond a wall, at the node itself as the opposite direction
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const bool bounced = walls && (z - L::cz[k] < 0 || z - L::cz[k] >= box.nz);
        const int kd = bounced ? opposite<Q>(k) : k;
        const unsigned b = bounced ? own : node.at(-L::cx[k], -L::cy[k], -L::cz[k], box.pitch, box.ny);
        const double cu = L::cx[k] * ux + L::cy[k] * uy + L::cz[k] * uz;
        const double P = eq_poly(weight<Q>(k), cu, uu);
        buf[(long long)kd * plane + b] = S(rho * P);
        buf[(long long)(Q + kd) * plane + b] = S(E * P);
    }
}

// Moments of the current state in FP64, one node per thread: rho, E and T where an output is
// given; for u*, Phi into the scratch and j into the u* output itself, which the second kernel turns
// into u* in place.  That kernel takes rho from the caller's output only where no other overlaps it
// (launch_moments).  Bound by its traffic (152 bytes read and 56 written per FP32 D3Q19 node; with rho
// in the scratch too 64, 3 to 5% more time).
struct MomentOut {
    double *rho, *us, *E, *T;       // any may be null
    double *rho_us, *phi;           // with us: where the second kernel finds rho and Phi
};

template <int Q, class S>
__global__ void k_moments_a(const S* __restrict__ buf, const MomentOut out, const BoxIndex box,
                            long long plane, Phys ph, const double* __restrict__ eos_p, int* err)
{
    using L = Lattice<Q>;
    const unsigned n = (unsigned)box.nx * (unsigned)box.ny * (unsigned)box.nz;
    const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const NodeIndex node(i, box);
    const int z = node.z[1];
    const unsigned own = node.at(0, 0, 0, box.pitch, box.ny);
    double rho = 0, jx = 0, jy = 0, jz = 0, E = 0;
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        unsigned j = node.at(-L::cx[k], -L::cy[k], -L::cz[k], box.pitch, box.ny);
        long long pk = (long long)k * plane;
        if (L::cz[k] != 0 && ph.walls && (z - L::cz[k] < 0 || z - L::cz[k] >= box.nz)) {   // bounce-back at a wall
            pk = (long long)opposite<Q>(k) * plane;
            j = own;
        }
        const double nk = double(buf[pk + j]);
        rho += nk;
        if (L::cx[k]) jx += L::cx[k] * nk;
        if (L::cy[k]) jy += L::cy[k] * nk;
        if (L::cz[k]) jz += L::cz[k] * nk;
        E += double(buf[(long long)Q * plane + pk + j]);
    }
    const double T = E / (rho * ph.c_v);
    const double Te = (ph.flags & kBaro) ? ph.T0_baro : T;
    bool inside = true;
    const double p = ph.eos ? ph.p_c * table_pressure(rho * ph.inv_rho_c, Te * ph.inv_T_c, ph, eos_p, inside)
                            : vdw_pressure(rho, Te, ph);
    double phi2 = fma(rho, kTheta, -p);
    if (!inside || !(phi2 > 0.0) || !(rho * ph.inv_rho_c < 3.0) || !(rho > 0.0) || !(E == E)) {
        atomicOr(err, 1);
        phi2 = 0.0;
    }
    if (out.rho) out.rho[i] = rho;
    if (out.E) out.E[i] = E;
    if (out.T) out.T[i] = T;
    if (out.us) {
        if (out.rho_us != out.rho) out.rho_us[i] = rho;
        out.phi[i] = sqrt(phi2);
        out.us[i] = jx;
        out.us[(long long)n + i] = jy;
        out.us[2 * (long long)n + i] = jz;
    }
}

// u* = (j + F/2)/rho (eq:ustar) in place of j, with the force of section 3 from the Phi field
// (mirrored beyond walls) plus the body force rho g.
template <int Q>
__global__ void k_moments_b(const MomentOut out, const BoxIndex box, Phys ph)
{
    using L = Lattice<Q>;
    const unsigned n = (unsigned)box.nx * (unsigned)box.ny * (unsigned)box.nz;
    const unsigned i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    NodeIndex node(i, box);
    if (ph.walls) {
        if (node.z[1] == 0) node.z[0] = 0;
        if (node.z[1] == box.nz - 1) node.z[2] = box.nz - 1;
    }
    const double* __restrict__ Phi = out.phi;
    double s1[3] = {0, 0, 0}, s2[3] = {0, 0, 0};
#pragma unroll
    for (int k = 1; k < Q; ++k) {
        const double p = Phi[node.at(L::cx[k], L::cy[k], L::cz[k], box.nx, box.ny)];
        const double G = force_coef<Q>(k);
        const int c[3] = {L::cx[k], L::cy[k], L::cz[k]};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            if (c[a] == 0) continue;
            s1[a] += G * p * p * c[a];
            s2[a] += G * p * c[a];
        }
    }
    const double rho = out.rho_us[i];
    const double phi = Phi[i];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double F = (ph.A * s1[a] + (1.0 - 2.0 * ph.A) * phi * s2[a]) * ph.inv_alpha + rho * ph.g[a];
        double* u = out.us + (long long)a * n + i;
        *u = (*u + 0.5 * F) / rho;
    }
}

constexpr int kReduceThreads = 256;

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Block partial sums of mass, momentum and internal energy (FP64): per-thread grid-stride
// sums over 16-byte vectors of consecutive nodes (a population plane's rows are padded to
// whole 128-byte lines, so the plane's element count is a multiple of the vector and every
// plane starts aligned), 64-lane wavefront shuffles, then the waves in order.
template <int Q, class S>
__global__ void __launch_bounds__(kReduceThreads)
k_reduce_partial(const S* __restrict__ buf, long long n, long long plane, double* __restrict__ part)
{
    using L = Lattice<Q>;
    constexpr int VEC = 16 / (int)sizeof(S);
    typedef S V __attribute__((ext_vector_type(VEC)));
    const long long nv = n / VEC;
    double acc[5] = {0, 0, 0, 0, 0};
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < nv;
         i += (long long)gridDim.x * blockDim.x) {
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const V a = *(const V*)(buf + (long long)k * plane + i * VEC);
            const V b = *(const V*)(buf + (long long)(Q + k) * plane + i * VEC);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const double nk = double(a[e]);
                acc[0] += nk;
                if (L::cx[k]) acc[1] += L::cx[k] * nk;
                if (L::cy[k]) acc[2] += L::cy[k] * nk;
                if (L::cz[k]) acc[3] += L::cz[k] * nk;
                acc[4] += double(b[e]);
            }
        }
    }
    __shared__ double wsum[kReduceThreads / 64][5];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        const double v = wave_sum(acc[c]);
        if (lane == 0) wsum[wave][c] = v;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        double s = 0;
        for (int w = 0; w < kReduceThreads / 64; ++w) s += wsum[w][threadIdx.x];
        part[blockIdx.x * 5 + threadIdx.x] = s;
    }
}

// Sum of per-block partial totals (5 per block) in a fixed order: thread t adds the entries
// t, t + 256, ... (independent loads in flight together), then a fixed tree over the threads.
__global__ void __launch_bounds__(kReduceThreads)
k_sum_partials(const double* __restrict__ part, long long nblocks, double* __restrict__ out)
{
    __shared__ double red[5][kReduceThreads];
    double acc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (long long b = threadIdx.x; b < nblocks; b += kReduceThreads) {
#pragma unroll
        for (int q = 0; q < 5; ++q) acc[q] += part[b * 5 + q];
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) red[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int h = kReduceThreads / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
#pragma unroll
            for (int q = 0; q < 5; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x < 5) out[threadIdx.x] = red[threadIdx.x][0];
}

inline unsigned blocks_for(long long n, int threads)
{
    return (unsigned)((n + threads - 1) / threads);
}

}  // namespace

// Launch shapes of the fused step.  Variant 0 is the default per (lattice, storage); the
// others are selected for tuning.  Tile shape, thread count and the order of the loads do not
// change the per-node arithmetic, so every variant gives bitwise-identical results.
// `per_cu` is the number of workgroups of the variant resident per compute unit (set by its
// registers and LDS); the automatic z chunk aims at about 256 * per_cu workgroups.
// FP32 variant 5 is the default launch with plain global addressing, which variant 0 falls
// back to for states of 4 GB and more; variant 7 is the same on 64 x 8 tiles (816 moment slots,
// the 48 beyond the 768 threads on threads without collision work), which lbm_init picks for
// such states where 64-wide tiles leave no more x columns idle than 32-wide ones.
struct TileShape { int tx, ty, threads; bool pipe, stash; int per_cu; };
static const TileShape kVariants19f[] = {
    {32, 16, 768, true, true, 1}, {32, 16, 768, false, true, 1}, {32, 16, 768, true, false, 1},
    {32, 16, 768, false, false, 1}, {32, 8, 512, false, false, 2}, {32, 16, 768, true, true, 1},
    {32, 8, 256, false, false, 2}, {64, 8, 768, false, true, 1}};
constexpr int kNumVariants19f = sizeof(kVariants19f) / sizeof(kVariants19f[0]);
// FP64 D3Q19: twice the registers and LDS per node
static const TileShape kVariants19d[] = {
    {32, 8, 512, false, true, 1}, {32, 8, 512, false, false, 1}, {32, 8, 256, false, false, 1},
    {32, 4, 128, false, false, 2}};
constexpr int kNumVariants19d = sizeof(kVariants19d) / sizeof(kVariants19d[0]);
// D2Q9 (one plane, no z march): the moment stage pulls the tile plus a 2-node halo, 1.69x the
// tile's nodes on 32x8 and 1.41x on 32x16
static const TileShape kVariants9[] = {
    {32, 8, 256, true, false, 2}, {32, 16, 512, true, false, 1}, {64, 8, 512, true, false, 1}};
constexpr int kNumVariants9 = sizeof(kVariants9) / sizeof(kVariants9[0]);

int step_variants(int Q, int storage_bytes)
{
    if (Q == 19) return storage_bytes == 4 ? kNumVariants19f : kNumVariants19d;
    return kNumVariants9;
}

void step_tile(int Q, int storage_bytes, int variant, int& tx, int& ty, int& per_cu)
{
    const TileShape* t = nullptr;
    if (Q == 19 && storage_bytes == 4 && variant >= 0 && variant < kNumVariants19f) t = &kVariants19f[variant];
    if (Q == 19 && storage_bytes == 8 && variant >= 0 && variant < kNumVariants19d) t = &kVariants19d[variant];
    if (Q == 9 && variant >= 0 && variant < kNumVariants9) t = &kVariants9[variant];
    if (t) {
        tx = t->tx;
        ty = t->ty;
        per_cu = t->per_cu;
        return;
    }
    tx = 32;
    ty = 8;
    per_cu = 2;
}

hipError_t launch_step(int Q, int storage_bytes, int variant, const void* src, void* dst,
                       const StepGeom& g, const Phys& ph, const StepAux& aux, hipStream_t st)
{
    if (Q == 19 && storage_bytes == 4) {
        switch (variant) {
        case 0: return launch_step_t<19, float, float, 32, 16, 768, true, true>(src, dst, g, ph, aux, st);
        case 1: return launch_step_t<19, float, float, 32, 16, 768, false, true>(src, dst, g, ph, aux, st);
        case 2: return launch_step_t<19, float, float, 32, 16, 768, true>(src, dst, g, ph, aux, st);
        case 3: return launch_step_t<19, float, float, 32, 16, 768, false>(src, dst, g, ph, aux, st);
        case 4: return launch_step_t<19, float, float, 32, 8, 512, false>(src, dst, g, ph, aux, st);
        case 5: return launch_step_t<19, float, float, 32, 16, 768, true, true, true>(src, dst, g, ph, aux, st);
        case 6: return launch_step_t<19, float, float, 32, 8, 256, false>(src, dst, g, ph, aux, st);
        case 7: return launch_step_t<19, float, float, 64, 8, 768, false, true, true>(src, dst, g, ph, aux, st);
        default: return hipErrorInvalidValue;
        }
    }
    if (Q == 19 && storage_bytes == 8) {
        switch (variant) {
        case 0: return launch_step_t<19, double, double, 32, 8, 512, false, true>(src, dst, g, ph, aux, st);
        case 1: return launch_step_t<19, double, double, 32, 8, 512, false>(src, dst, g, ph, aux, st);
        case 2: return launch_step_t<19, double, double, 32, 8, 256, false>(src, dst, g, ph, aux, st);
        case 3: return launch_step_t<19, double, double, 32, 4, 128, false>(src, dst, g, ph, aux, st);
        default: return hipErrorInvalidValue;
        }
    }
    // D2Q9 FP32 populations with FP64 arithmetic: in 2D the registers allow it, and FP32
    // arithmetic tripled the error of the stored-FP32 state alone (u* 9e-6 to 1e-5 against a
    // floor of 3e-6 on a 100-step slab)
    if (Q == 9 && storage_bytes == 4) {
        switch (variant) {
        case 0: return launch_step_t<9, float, double, 32, 8, 256, true>(src, dst, g, ph, aux, st);
        case 1: return launch_step_t<9, float, double, 32, 16, 512, true>(src, dst, g, ph, aux, st);
        case 2: return launch_step_t<9, float, double, 64, 8, 512, true>(src, dst, g, ph, aux, st);
        default: return hipErrorInvalidValue;
        }
    }
    if (Q == 9 && storage_bytes == 8) {
        switch (variant) {
        case 0: return launch_step_t<9, double, double, 32, 8, 256, false>(src, dst, g, ph, aux, st);
        case 1: return launch_step_t<9, double, double, 32, 16, 512, false>(src, dst, g, ph, aux, st);
        case 2: return launch_step_t<9, double, double, 64, 8, 512, false>(src, dst, g, ph, aux, st);
        default: return hipErrorInvalidValue;
        }
    }
    return hipErrorInvalidValue;
}

hipError_t launch_init(int Q, int storage_bytes, void* buf, const double* rho0, const double* u0,
                       const double* T0, int nx, int ny, int nz, int pitch, long long plane,
                       double c_v, int walls, hipStream_t st)
{
    const long long n = (long long)nx * ny * nz;
    const dim3 grid(blocks_for(n, 256)), block(256);
    const BoxIndex box = box_index(nx, ny, nz, pitch);
    if (Q == 19 && storage_bytes == 4) hipLaunchKernelGGL((k_init<19, float>), grid, block, 0, st, (float*)buf, rho0, u0, T0, box, plane, c_v, walls);
    else if (Q == 19 && storage_bytes == 8) hipLaunchKernelGGL((k_init<19, double>), grid, block, 0, st, (double*)buf, rho0, u0, T0, box, plane, c_v, walls);
    else if (Q == 9 && storage_bytes == 4) hipLaunchKernelGGL((k_init<9, float>), grid, block, 0, st, (float*)buf, rho0, u0, T0, box, plane, c_v, 0);
    else if (Q == 9 && storage_bytes == 8) hipLaunchKernelGGL((k_init<9, double>), grid, block, 0, st, (double*)buf, rho0, u0, T0, box, plane, c_v, 0);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_moments(int Q, int storage_bytes, const void* buf, double* scratch, int nx, int ny,
                          int nz, int pitch, long long plane, const Phys& ph, const double* eos_p,
                          int* err, double* rho, double* us, double* E, double* T, hipStream_t st)
{
    const long long n = (long long)nx * ny * nz;
    const dim3 grid(blocks_for(n, 256)), block(256);
    const BoxIndex box = box_index(nx, ny, nz, pitch);
    const auto apart = [&](const double* other, long long m) { return !other || rho + n <= other || other + m <= rho; };
    const bool own = rho && apart(us, 3 * n) && apart(E, n) && apart(T, n);
    const MomentOut out{rho, us, E, T, own ? rho : scratch, scratch + n};
    if (Q == 19 && storage_bytes == 4) hipLaunchKernelGGL((k_moments_a<19, float>), grid, block, 0, st, (const float*)buf, out, box, plane, ph, eos_p, err);
    else if (Q == 19 && storage_bytes == 8) hipLaunchKernelGGL((k_moments_a<19, double>), grid, block, 0, st, (const double*)buf, out, box, plane, ph, eos_p, err);
    else if (Q == 9 && storage_bytes == 4) hipLaunchKernelGGL((k_moments_a<9, float>), grid, block, 0, st, (const float*)buf, out, box, plane, ph, eos_p, err);
    else if (Q == 9 && storage_bytes == 8) hipLaunchKernelGGL((k_moments_a<9, double>), grid, block, 0, st, (const double*)buf, out, box, plane, ph, eos_p, err);
    else return hipErrorInvalidValue;
    if (us) {
        if (Q == 19) hipLaunchKernelGGL((k_moments_b<19>), grid, block, 0, st, out, box, ph);
        else hipLaunchKernelGGL((k_moments_b<9>), grid, block, 0, st, out, box, ph);
    }
    return hipGetLastError();
}

int reduce_blocks(long long n)
{
    long long b = (n + kReduceThreads * 8 - 1) / (kReduceThreads * 8);
    return (int)(b < 1 ? 1 : (b > 2048 ? 2048 : b));
}

hipError_t launch_reduce(int Q, int storage_bytes, const void* buf, long long n, long long plane,
                         double* partials, int nblocks, double* out, hipStream_t st)
{
    const dim3 grid(nblocks), block(kReduceThreads);
    if (Q == 19 && storage_bytes == 4) hipLaunchKernelGGL((k_reduce_partial<19, float>), grid, block, 0, st, (const float*)buf, n, plane, partials);
    else if (Q == 19 && storage_bytes == 8) hipLaunchKernelGGL((k_reduce_partial<19, double>), grid, block, 0, st, (const double*)buf, n, plane, partials);
    else if (Q == 9 && storage_bytes == 4) hipLaunchKernelGGL((k_reduce_partial<9, float>), grid, block, 0, st, (const float*)buf, n, plane, partials);
    else if (Q == 9 && storage_bytes == 8) hipLaunchKernelGGL((k_reduce_partial<9, double>), grid, block, 0, st, (const double*)buf, n, plane, partials);
    else return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kReduceThreads), 0, st, (const double*)partials,
                       (long long)nblocks, out);
    return hipGetLastError();
}

hipError_t launch_sum_partials(const double* partials, long long nblocks, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(kReduceThreads), 0, st, partials, nblocks, out);
    return hipGetLastError();
}

}  // namespace lbm
