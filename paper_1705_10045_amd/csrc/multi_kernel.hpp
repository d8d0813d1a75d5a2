// Several time steps of the D2Q9 thermal multiphase LBM in one launch, for boxes whose step is
// bound by latency rather than bytes.
//
// A step of a small box is a launch, one round of loads and a chain of dependent FP64 arithmetic,
// 6 to 7 us whatever its size, with most of the chip idle (bound by that chain, here 2.1 us of
// each step of 1000 nodes).  Here a workgroup takes a tile with a
// halo of 3 nodes per step (a node's update reaches populations 3 nodes away), loads it once, and
// takes `steps` steps on a region that shrinks by 3 nodes each, with the populations of the steps
// between in LDS.  One thread owns one node of the region for the whole launch, so all of the
// node's quantities stay in registers, and redundant halo nodes cost only lanes that would idle.
// The per-node arithmetic is that of the fused step (node_math.hpp), and populations are rounded
// to the storage type after every step, so the fields are bitwise those of single steps.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "lattice.hpp"
#include "node_math.hpp"
#include "physics.hpp"
#include "step_kernel.hpp"

namespace lbm {

// Nodes of a region: one thread each.  At 168 VGPRs a CU holds 12 wavefronts, and the LDS of one
// workgroup is 129 KB for FP64 populations.
constexpr int kMultiNodes = 704;

template <class S, int NMODE, int EXT>
__global__ void __launch_bounds__(kMultiNodes)
k_multi_step(const S* __restrict__ src, S* __restrict__ dst, const StepGeom g, const MultiGeom mg,
             const Phys ph, const StepAux aux)
{
    using L = Lattice<9>;
    using R = double;
    constexpr int Q = 9;
    constexpr bool WN = NMODE != kTauOne;
    constexpr bool kTable = EXT == kExtTable;
    __shared__ S pop[2 * Q][kMultiNodes];
    __shared__ double sPhi[kMultiNodes];
    __shared__ R sRho[kMultiNodes], sT[kMultiNodes], sUx[kMultiNodes], sUy[kMultiNodes];

    const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
    const int tiy = div_uniform(lb, g.inv_ntx), tix = lb - tiy * g.ntx;
    const int x0 = tix * mg.tx, y0 = tiy * mg.ty;
    const PopIO<S, kAddrBuf> io(src, dst, g.plane, 2 * Q);
    const int tid = threadIdx.x;
    // the node: position in the region, distance from the tile (a box of one row has no y halo:
    // its rows above and below are the row itself, stride 0)
    const int py = (int)div_by((unsigned)tid, mg.inv_rx), px = tid - py * mg.rx;
    const int W = mg.ry == 1 ? 0 : mg.rx;
    const int my = mg.ry == 1 ? 0 : mg.margin;
    const int dx = max(max(mg.margin - px, px - mg.margin - mg.tx + 1), 0);
    const int dy = max(max(my - py, py - my - mg.ty + 1), 0);
    const int d = tid < mg.rx * mg.ry ? max(dx, dy) : 1 << 20;
    const int ox = x0 - mg.margin + px, oy = y0 - my + py;
    const int gx = wrap_near(ox, g.nx), gy = wrap_near(oy, g.ny);
    const bool has_g = EXT != kExtNone && (ph.g[0] != 0.0 || ph.g[1] != 0.0 || ph.g[2] != 0.0);
    const R omega_E = ph.omega_E, keepN = 1.0 - ph.omega, keepG = 1.0 - ph.omega_E;
    const unsigned flags = ph.flags;
    const bool pseudo = (flags & kPseudo) != 0;

    S pn[Q], pe[Q];
    if (d <= mg.margin) {
        const int xs[3] = {wrap_dec(gx, g.nx), gx, wrap_inc(gx, g.nx)};
        const int ys[3] = {wrap_dec(gy, g.ny) * g.pitch, gy * g.pitch, wrap_inc(gy, g.ny) * g.pitch};
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const int off = ys[1 - L::cy[k]] + xs[1 - L::cx[k]];
            pn[k] = io.load(k, off);
            pe[k] = io.load(Q + k, off);
        }
    }
    for (int left = mg.steps - 1; left >= 0; --left) {
        const int h = 3 * left;   // the collision's region: the tile and h nodes around it
        double dr = 1.0, dE = 1.0, p = 0.0;
        R jx = 0.0, jy = 0.0, jz = 0.0;
        if (d <= h + 2) {
            if (left != mg.steps - 1) {
#pragma unroll
                for (int k = 0; k < Q; ++k) {
                    const int e = tid - L::cx[k] - W * L::cy[k];
                    pn[k] = pop[k][e];
                    pe[k] = pop[Q + k][e];
                }
            }
            double dT, phi2;
            bool ok;
            moment_sums<Q>(pn, pe, dr, jx, jy, jz, dE);
            eos_phi2<kTable>(dr, dE, ph, flags, aux, dT, p, phi2, ok);
            if (!ok) {
                atomicOr(aux.err, 1);
                phi2 = 0.0;
            }
            sPhi[tid] = sqrt(phi2);
            sRho[tid] = dr;
            sT[tid] = dT;
        }
        __syncthreads();
        R Fx = 0.0, Fy = 0.0, Fz = 0.0;
        const R inv_rho = R(1) / dr;
        if (d <= h + 1) {
            force_at<Q>(sPhi, sPhi, sPhi, tid, W, ph.A, ph.inv_alpha, Fx, Fy, Fz);
            if (has_g) {
                Fx = fma(dr, ph.g[0], Fx);
                Fy = fma(dr, ph.g[1], Fy);
                Fz = fma(dr, ph.g[2], Fz);
            }
            sUx[tid] = (jx + 0.5 * Fx) * inv_rho;
            sUy[tid] = (jy + 0.5 * Fy) * inv_rho;
        }
        __syncthreads();
        if (d <= h) {
            const R div = 0.5 * (sUx[tid + 1] - sUx[tid - 1]) + 0.5 * (sUy[tid + W] - sUy[tid - W]);
            const R dS = energy_source<2, R, kTable>(p, div, dr, sT[tid], 0.0, sRho, 0.0, 0.0, sT, 0.0, tid, W,
                                                     ph.cond_half, flags, ph, aux);
            R rn[Q], re[Q];
#pragma unroll
            for (int k = 1; k < Q; ++k) {
                re[k] = R(pe[k]);
                rn[k] = WN ? R(pn[k]) : R(0);
            }
            NodeCollision<Q, S, R, WN, NMODE == kMrt> c;
            c.setup(dr, dE, jx, jy, jz, Fx, Fy, Fz, inv_rho, dS, keepN, keepG, omega_E, pseudo);
            c.mrt_prepare(rn, ph);
            const bool last = left == 0;
            const bool stored = last && ox < g.nx && oy < g.ny;
            const int own = gy * g.pitch + gx;
            auto put = [&](int pk, S v) {
                if (!last) pop[pk][tid] = v;
                else if (stored) io.store(pk, own, v);
            };
#pragma unroll
            for (int k = 1; k < Q; ++k) {
                const int ko = opposite<Q>(k);
                if (ko < k) continue;
                S out[4];
                c.dir_pair(k, rn, re, out);
                put(k, out[0]);
                put(Q + k, out[1]);
                put(ko, out[2]);
                put(Q + ko, out[3]);
            }
            S n0, g0;
            c.rest(dr, dE, dS, n0, g0);
            put(0, n0);
            put(Q, g0);
        }
        if (left != 0) __syncthreads();
    }
}

}  // namespace lbm
