// Two-launch time step of the D3Q19 thermal multiphase LBM: a moment launch over all nodes, then
// a launch for the force, the energy source and the collisions.
//
// The fused step (step_kernel.hpp) moves the fewest bytes but runs one workgroup of 768 threads
// per CU in lockstep stages: each z plane of a tile column costs one serial chain of loads,
// barriers, force, collision and stores (5 us on an idle chip), every chunk of planes pays four
// extra iterations, and tiles of 32 x 16 leave small and ragged boxes with a few busy CUs.  Here
//   - k_split_moments gives one thread to one node: its 38 pulls are all in flight at once and
//     every population is pulled by exactly one thread; rho, j, T, p and Phi go to a scratch
//     (36 bytes per node for FP32);
//   - k_split_collide marches 32 x 8 tiles through a few planes with the scratch's halo in LDS
//     (38 KB, 49 for FP64, instead of 147: registers allow three and two workgroups per CU), pulls the
//     node's energy populations (and the density ones unless tau = 1) once more, and stores.
// Both are bound by what they move between L2 and memory: 200 x 150 x 97 FP32 1.68 times the algorithmic bytes
// at 4.8 TB/s, 121 and 186 us (96^3 FP64, tau = 0.8: 1.74 times at 5.5 TB/s, 62 and 107 us); a box that leaves
// the chip idle by one workgroup's chain (32^3 3.8 and 7.6 us).
// The per-node arithmetic is that of node_math.hpp in the same order, so the fields are bitwise
// those of the fused step.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.hpp"
#include "lattice.hpp"
#include "node_math.hpp"
#include "physics.hpp"
#include "step_kernel.hpp"

namespace lbm {

// Moments of one state, structure of arrays with the row pitch of the populations: Phi and rho
// in FP64 (the force is a small difference of Phi^2 values, the rest populations close the mass
// balance in FP64), T, p and j in the collision's type R.  `nodes` is the elements of one array
// (pitch * ny * nz); byte offsets of the arrays fit 32 bits (the state is under 4 GB, and the
// scratch is smaller).
template <class R>
struct SplitFields {
    __amdgpu_buffer_rsrc_t rs;
    unsigned nodes;
    __device__ SplitFields(void* base, unsigned n) : nodes(n)
    {
        const unsigned bytes = n * (unsigned)(2 * sizeof(double) + 5 * sizeof(R));
        rs = __builtin_amdgcn_make_buffer_rsrc(base, (short)0, __builtin_bit_cast(int, bytes), bufio::kWord3);
    }
    // byte offsets of the arrays
    __device__ unsigned phi() const { return 0; }
    __device__ unsigned rho() const { return nodes * 8u; }
    __device__ unsigned T() const { return nodes * 16u; }
    __device__ unsigned p() const { return nodes * (16u + (unsigned)sizeof(R)); }
    __device__ unsigned j(int a) const { return nodes * (16u + (2u + a) * (unsigned)sizeof(R)); }
    // element `i` (per lane) of the array at byte offset `f` plus `z` elements (uniform)
    template <class V>
    __device__ __forceinline__ V load(unsigned f, unsigned i, unsigned z) const
    {
        return bufio::load<V>(rs, i * (unsigned)sizeof(V), f + z * (unsigned)sizeof(V));
    }
    template <class V>
    __device__ __forceinline__ void store(unsigned f, unsigned i, V v) const
    {
        if constexpr (sizeof(V) == 4)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, (int)(i * 4u), (int)f, 0);
        else
            __builtin_amdgcn_raw_buffer_store_b64(
                __builtin_bit_cast(__attribute__((ext_vector_type(2))) unsigned, v), rs, (int)(i * 8u), (int)f, 0);
    }
};

// Wavefronts of 256-thread workgroups, one node per thread.
constexpr int kSplitThreads = 256;

// Moments of node `id` (x fastest) of the box described by g.
template <int Q, class S, class R, int EXT>
__device__ __forceinline__ void split_moments_node(const S* __restrict__ src, void* __restrict__ scratch,
                                                   const StepGeom& g, const Phys& ph, const StepAux& aux,
                                                   const unsigned id)
{
    using L = Lattice<Q>;
    const unsigned n = (unsigned)g.nx * (unsigned)g.ny * (unsigned)g.nz;
    if (id >= n) return;
    const PopIO<S, kAddrBuf> io(src, nullptr, g.plane, 2 * Q);
    const unsigned nxy = (unsigned)g.pitch * (unsigned)g.ny;
    const SplitFields<R> f(scratch, nxy * (unsigned)g.nz);
    const unsigned rowid = div_by(id, g.inv_nx);
    const int x = (int)(id - rowid * (unsigned)g.nx);
    const int z = (int)div_by(rowid, g.inv_ny);
    const int y = (int)(rowid - (unsigned)z * (unsigned)g.ny);
    // wrapped x, y * pitch, z * plane of (node - c) for c = +1, 0, -1 (index 1 - c)
    const int xs[3] = {wrap_dec(x, g.nx), x, wrap_inc(x, g.nx)};
    const int ys[3] = {wrap_dec(y, g.ny) * g.pitch, y * g.pitch, wrap_inc(y, g.ny) * g.pitch};
    const unsigned zs[3] = {(unsigned)wrap_dec(z, g.nz) * nxy, (unsigned)z * nxy, (unsigned)wrap_inc(z, g.nz) * nxy};
    const bool has_walls = EXT != kExtNone && ph.walls != 0;
    const bool bb_lo = has_walls && z == 0, bb_hi = has_walls && z == g.nz - 1;
    const unsigned own = zs[1] + (unsigned)(ys[1] + x);
    S pn[Q], pe[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        const unsigned off = zs[1 - L::cz[k]] + (unsigned)(ys[1 - L::cy[k]] + xs[1 - L::cx[k]]);
        if (EXT != kExtNone && L::cz[k] != 0) {
            // next to a wall the pull from beyond it takes the opposite population leaving the
            // node itself; lanes of one wavefront may differ, so the population's plane is part
            // of the lane offset here
            const bool bb = L::cz[k] == 1 ? bb_lo : bb_hi;
            const unsigned pk = (unsigned)(bb ? opposite<Q>(k) : k) * (unsigned)g.plane + (bb ? own : off);
            pn[k] = io.load(0, (int)pk);
            pe[k] = io.load(Q, (int)pk);
        } else {
            pn[k] = io.load(k, (int)off);
            pe[k] = io.load(Q + k, (int)off);
        }
    }
    double dr, djx, djy, djz, dE, dT, p, phi2;
    bool ok;
    moment_sums<Q>(pn, pe, dr, djx, djy, djz, dE);
    eos_phi2<EXT == kExtTable>(dr, dE, ph, ph.flags, aux, dT, p, phi2, ok);
    if (!ok) {
        atomicOr(aux.err, 1);
        phi2 = 0.0;
    }
    f.store(f.phi(), own, sqrt(phi2));
    f.store(f.rho(), own, dr);
    f.store(f.T(), own, R(dT));
    f.store(f.p(), own, R(p));
    f.store(f.j(0), own, R(djx));
    f.store(f.j(1), own, R(djy));
    f.store(f.j(2), own, R(djz));
}

template <int Q, class S, class R, int EXT>
__global__ void __launch_bounds__(kSplitThreads)
k_split_moments(const S* __restrict__ src, void* __restrict__ scratch, const StepGeom g,
                const Phys ph, const StepAux aux)
{
    split_moments_node<Q, S, R, EXT>(src, scratch, g, ph, aux,
                                     (unsigned)xcd_logical_block(blockIdx.x, gridDim.x) * kSplitThreads + threadIdx.x);
}

// LDS of one workgroup of k_split_collide: a ring of Phi planes on the tile + 2-halo (the force of
// plane zf reads zf - 1 .. zf + 1 while zf + 2 is written; the first five planes of a chunk are
// loaded at once), and rho, T, u*x, u*y on the tile + 1-halo for the planes zf and zf - 1 (written
// by the force stage, read by the collision).
template <class R, int TX, int TY>
struct SplitLds {
    static constexpr int EX = TX + 4, EY = TY + 4, NE = EX * EY;
    static constexpr int FX = TX + 2, FY = TY + 2, NF = FX * FY;
    static constexpr int RING = 8;
    double phi[RING][NE];
    R rho[2][NF], T[2][NF], ux[2][NF], uy[2][NF];
};

constexpr int kSplitTX = 32, kSplitTY = 8;

// Force, energy source, collisions and store of one tile column of z planes, one node per thread
// per plane.  Iteration zf: the force and u* of plane zf (own node; the tile's face neighbours
// by the first threads again, whose u* components normal to the faces div u* needs), then the
// collision of plane zf - 1, with one barrier per iteration.
//
// Loads and stores share one in-order counter, so what an iteration loads is consumed before its
// own stores are issued, and nothing waits for a load behind a store of the same iteration: the
// Maxwell table's cell and the scratch of the next planes are requested first, the pulls last,
// all before the force.  Lanes of a ragged tile beyond the box keep the control flow uniform:
// their pulls and stores carry an offset beyond the buffer, which the hardware drops.
// All threads of the workgroup call it, for tile `lb` (x fastest, then y, then z chunk); a caller
// that runs several tiles puts a barrier between them.
template <int Q, class S, class R, int NMODE, int EXT, bool RED>
__device__ __forceinline__ void split_collide_tile(SplitLds<R, kSplitTX, kSplitTY>& lds,
                                                   const S* __restrict__ src, S* __restrict__ dst,
                                                   const void* __restrict__ scratch, const StepGeom& g,
                                                   const Phys& ph, const StepAux& aux, const int lb,
                                                   const int tid, double (*red)[5] = nullptr)
{
    using L = Lattice<Q>;
    constexpr int TX = kSplitTX, TY = kSplitTY, NTH = kSplitThreads;
    static_assert(TX * TY == NTH, "one node per thread");
    using Lds = SplitLds<R, TX, TY>;
    constexpr int EX = Lds::EX, NE = Lds::NE, FX = Lds::FX, RING = Lds::RING;
    constexpr int NH = 2 * TX + 2 * TY;   // face neighbours of the tile
    constexpr bool WN = NMODE != kTauOne;
    static_assert(NE <= 2 * NTH && NH <= NTH, "slots per thread");
    constexpr unsigned kDropped = 0xfffffffcu;   // beyond every buffer (states are under 4 GB)

    const PopIO<S, kAddrBuf> io(src, dst, g.plane, 2 * Q);
    const unsigned nxy = (unsigned)g.pitch * (unsigned)g.ny;
    const SplitFields<R> m(const_cast<void*>(scratch), nxy * (unsigned)g.nz);
    const int trow = div_uniform(lb, g.inv_ntx), tiz = div_uniform(trow, g.inv_nty);
    const int tix = lb - trow * g.ntx, tiy = trow - tiz * g.nty;
    const int x0 = tix * TX, y0 = tiy * TY, z0 = tiz * g.chunk;
    const int z1 = min(z0 + g.chunk, g.nz);
    const bool has_walls = EXT != kExtNone && ph.walls != 0;
    const bool has_g = EXT != kExtNone && (ph.g[0] != 0.0 || ph.g[1] != 0.0 || ph.g[2] != 0.0);

    // own node
    const int tx = tid % TX, ty = tid / TX;
    const int ox = x0 + tx, oy = y0 + ty;
    const bool own_in = ox < g.nx && oy < g.ny;
    const int gx = wrap_near(ox, g.nx), gy = wrap_near(oy, g.ny);
    const int xs[3] = {wrap_dec(gx, g.nx), gx, wrap_inc(gx, g.nx)};
    const int ys[3] = {wrap_dec(gy, g.ny) * g.pitch, gy * g.pitch, wrap_inc(gy, g.ny) * g.pitch};
    const unsigned oxy = (unsigned)(ys[1] + gx);
    // byte offsets in a plane of the nodes the pulls come from (index 1 - c)
    unsigned pull_xy[3][3];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            pull_xy[b][a] = own_in ? (unsigned)(ys[b] + xs[a]) * (unsigned)sizeof(S) : kDropped;
    const int oe = (tx + 2) + EX * (ty + 2), of = (tx + 1) + FX * (ty + 1);
    // Phi slots of the tile + 2-halo region
    unsigned p_xy[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int s = min(tid + r * NTH, NE - 1);
        p_xy[r] = (unsigned)(wrap_near(x0 - 2 + s % EX, g.nx) + wrap_near(y0 - 2 + s / EX, g.ny) * g.pitch);
    }
    const bool p_two = tid + NTH < NE;
    // face neighbour of the tile: rows below and above, then columns left and right
    const bool halo = tid < NH;
    const bool hxface = tid >= 2 * TX;
    int hx, hy;
    if (!hxface) { hx = tid % TX; hy = tid < TX ? -1 : TY; }
    else { const int r = tid - 2 * TX; hx = (r & 1) ? TX : -1; hy = halo ? r >> 1 : 0; }
    const unsigned h_xy = (unsigned)(wrap_near(x0 + hx, g.nx) + wrap_near(y0 + hy, g.ny) * g.pitch);
    const unsigned hj_xy = h_xy + (hxface ? 0u : m.nodes);   // j_x on the x faces, j_y on the y faces
    const int he = (hx + 2) + EX * (hy + 2), hf = (hx + 1) + FX * (hy + 1);

    const R omega_E = R(ph.omega_E);
    const R keepN = R(1.0 - ph.omega), keepG = R(1.0 - ph.omega_E);
    const R cond_half = R(ph.cond_half);
    const unsigned flags = ph.flags;
    const bool pseudo = (flags & kPseudo) != 0;
    double nsum[RED ? 5 : 1];
    if constexpr (RED) {
#pragma unroll
        for (int q = 0; q < 5; ++q) nsum[q] = 0.0;
    }

    auto zrow = [&](int z) { return (unsigned)wrap_near(z, g.nz) * nxy; };
    auto beyond_wall = [&](int z) { return has_walls && (z < 0 || z >= g.nz); };

    struct Own { double rho; R T, p, jx, jy, jz; };
    struct Face { double rho; R T, j; };
    struct Phi2 { double a, b; };
    auto load_phi = [&](int z) {
        Phi2 v;
        const unsigned zo = zrow(z);
        v.a = m.template load<double>(m.phi(), p_xy[0], zo);
        v.b = m.template load<double>(m.phi(), p_xy[1], zo);
        return v;
    };
    auto put_phi = [&](int z, const Phi2& v) {
        double* s = lds.phi[z & (RING - 1)];
        s[tid] = v.a;
        if (p_two) s[tid + NTH] = v.b;
    };
    auto load_own = [&](int z) {
        const unsigned zo = zrow(z);
        Own o;
        o.rho = m.template load<double>(m.rho(), oxy, zo);
        o.T = m.template load<R>(m.T(), oxy, zo);
        o.p = m.template load<R>(m.p(), oxy, zo);
        o.jx = m.template load<R>(m.j(0), oxy, zo);
        o.jy = m.template load<R>(m.j(1), oxy, zo);
        o.jz = m.template load<R>(m.j(2), oxy, zo);
        return o;
    };
    auto load_face = [&](int z) {
        const unsigned zo = zrow(z);
        Face h;
        h.rho = m.template load<double>(m.rho(), h_xy, zo);
        h.T = m.template load<R>(m.T(), h_xy, zo);
        h.j = m.template load<R>(m.j(0), hj_xy, zo);
        return h;
    };
    // pulls of the own node at plane z (all directions of the energy set; the moving density
    // populations when the collision reads them)
    S pn[Q], pe[Q];
    auto load_pops = [&](int z) {
        const bool bb_lo = has_walls && z == 0, bb_hi = has_walls && z == g.nz - 1;
        const unsigned zo[3] = {zrow(z - 1) * (unsigned)sizeof(S), zrow(z) * (unsigned)sizeof(S),
                                zrow(z + 1) * (unsigned)sizeof(S)};
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            unsigned pk = (unsigned)k, off = zo[1 - L::cz[k]];
            unsigned xy = pull_xy[1 - L::cy[k]][1 - L::cx[k]];
            if (EXT != kExtNone && L::cz[k] != 0) {
                const bool bb = L::cz[k] == 1 ? bb_lo : bb_hi;   // uniform: a plane next to a wall
                pk = bb ? (unsigned)opposite<Q>(k) : pk;
                off = bb ? zo[1] : off;
                xy = bb ? pull_xy[1][1] : xy;
            }
            pe[k] = bufio::load<S>(io.rs, xy, off + ((unsigned)Q + pk) * io.plane_bytes);
            if (WN && k > 0) pn[k] = bufio::load<S>(io.rs, xy, off + pk * io.plane_bytes);
        }
    };

    // force and u* of plane zf: the own node's force into F, u*_z into uz; with `keep` the plane's
    // rho, T, u*x and u*y on the tile and its faces into the LDS planes the collision reads
    auto force_stage = [&](int zf, const Own& o, const Face& h, bool keep, R (&F)[3], R& uz) {
        F[0] = F[1] = F[2] = uz = R(0);
        if (beyond_wall(zf)) return;
        const double* p0 = lds.phi[zf & (RING - 1)];
        const double* pm = (has_walls && zf == 0) ? p0 : lds.phi[(zf - 1) & (RING - 1)];
        const double* pp = (has_walls && zf == g.nz - 1) ? p0 : lds.phi[(zf + 1) & (RING - 1)];
        auto force = [&](int e, double rf, R& ax, R& ay, R& az) {
            double fx, fy, fz;
            force_at<Q>(pm, p0, pp, e, EX, ph.A, ph.inv_alpha, fx, fy, fz);
            if (has_g) {
                fx = fma(rf, ph.g[0], fx);
                fy = fma(rf, ph.g[1], fy);
                fz = fma(rf, ph.g[2], fz);
            }
            ax = R(fx); ay = R(fy); az = R(fz);
        };
        const R rho = R(o.rho);
        force(oe, double(rho), F[0], F[1], F[2]);
        const R inv_rho = R(1) / rho;
        uz = rounded((o.jz + R(0.5) * F[2]) * inv_rho);
        if (!keep) return;
        const int b = zf & 1;
        lds.ux[b][of] = (o.jx + R(0.5) * F[0]) * inv_rho;
        lds.uy[b][of] = (o.jy + R(0.5) * F[1]) * inv_rho;
        lds.rho[b][of] = rho;
        lds.T[b][of] = o.T;
        if (halo) {
            R ax, ay, az;
            const R rh = R(h.rho);
            force(he, double(rh), ax, ay, az);
            const R ih = R(1) / rh;
            const R u = (h.j + R(0.5) * (hxface ? ax : ay)) * ih;
            if (hxface) lds.ux[b][hf] = u;
            else lds.uy[b][hf] = u;
            lds.rho[b][hf] = rh;
            lds.T[b][hf] = h.T;
        }
    };

    // the first planes: Phi of z0 - 2 .. z0 + 2, force of z0 - 1 (for u*_z) and z0
    Own prev, cur;               // scratch of planes zf - 1 and zf
    Face face;
    R Fp[3], uz1, uz2;           // force and u*_z of plane zf - 1, u*_z of plane zf - 2
    R rho2, T2;                  // rho, T of plane zf - 2
    {
        Phi2 v[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) v[q] = load_phi(z0 - 2 + q);
        const Own o = load_own(z0 - 1);
        prev = load_own(z0);
        face = load_face(z0);
        cur = load_own(z0 + 1);
#pragma unroll
        for (int q = 0; q < 5; ++q) put_phi(z0 - 2 + q, v[q]);
        __syncthreads();
        force_stage(z0 - 1, o, face, false, Fp, uz2);
        force_stage(z0, prev, face, true, Fp, uz1);
        rho2 = R(o.rho);
        T2 = o.T;
        if (z0 + 1 < z1) face = load_face(z0 + 1);
        __syncthreads();
    }

    auto iterate = [&](int zf, auto more) {
        constexpr bool MORE = decltype(more)::value;
        const int zc = zf - 1;
        // ---------------- loads: the band's table cell, the scratch of the next planes, the pulls
        double q[8], tcell = 0.0;
        bool band = false;
        if (EXT != kExtTable && (flags & kLatent)) {
            const double Te = (flags & kBaro) ? ph.T0_baro : double(prev.T);
            int j;
            band = band_cell(Te * ph.inv_T_c, aux.tab_s0, aux.tab_inv_ds, j, tcell);
            const double* c = aux.maxwell + 2 * (j - 1);
#pragma unroll
            for (int i = 0; i < 8; ++i) q[i] = c[i];
        }
        Phi2 nphi;
        Own nxt;
        Face nface;
        if constexpr (MORE) {
            nphi = load_phi(zf + 2);
            nxt = load_own(zf + 1);
            nface = load_face(zf + 1);
        }
        load_pops(zc);

        // ---------------- F: force and u* of plane zf
        R F[3], uz;
        force_stage(zf, cur, face, MORE, F, uz);
        if constexpr (MORE) put_phi(zf + 2, nphi);

        // ---------------- C: energy source, collisions, store of plane zf - 1
        const int b = zc & 1;
        const double rho_d = prev.rho;
        const R rho = R(rho_d), T = prev.T, p = prev.p;
        // z neighbours; beyond a wall rho mirrored, u*_z mirrored with the opposite sign, T
        // mirrored or 2 T_wall - T
        R uzm = uz2, uzp = uz, rzm = rho2, rzp = R(cur.rho), tzm = T2, tzp = cur.T;
        if (has_walls) {
            if (zc == 0) {
                uzm = -uz1;
                rzm = rho;
                tzm = (ph.wall_heat & kWallTBottom) ? R(2.0 * ph.T_bottom) - T : T;
            }
            if (zc == g.nz - 1) {
                uzp = -uz1;
                rzp = rho;
                tzp = (ph.wall_heat & kWallTTop) ? R(2.0 * ph.T_top) - T : T;
            }
        }
        R div = R(0.5) * (lds.ux[b][of + 1] - lds.ux[b][of - 1]) +
                R(0.5) * (lds.uy[b][of + FX] - lds.uy[b][of - FX]);
        div += R(0.5) * (uzp - uzm);
        R dE;
        if constexpr (EXT == kExtTable) {
            dE = energy_source<3, R, true>(p, div, rho, T, rzm, lds.rho[b], rzp, tzm, lds.T[b], tzp, of, FX,
                                           cond_half, flags, ph, aux);
        } else {
            dE = work_conduction<3, R>(p, div, rho, rzm, lds.rho[b], rzp, tzm, lds.T[b], tzp, of, FX, cond_half,
                                       flags);
            if (flags & kLatent) {
                double r1, r2;
                band_eval(tcell, q, ph.rho_c, r1, r2);
                if (band) latent_term(dE, r1, r2, rho, div, ph);
            }
        }
        double E_d = 0.0;
#pragma unroll
        for (int k = 0; k < Q; ++k) E_d += double(pe[k]);
        R rn[Q], re[Q];
#pragma unroll
        for (int k = 1; k < Q; ++k) {
            re[k] = R(pe[k]);
            rn[k] = WN ? R(pn[k]) : R(0);
        }
        const R E = R(E_d), inv_rho = R(1) / rho;
        NodeCollision<Q, S, R, WN, NMODE == kMrt> c;
        c.setup(rho, E, prev.jx, prev.jy, prev.jz, Fp[0], Fp[1], Fp[2], inv_rho, dE, keepN, keepG, omega_E,
                pseudo);
        c.mrt_prepare(rn, ph);
        const unsigned zo = zrow(zc) * (unsigned)sizeof(S);
        auto put = [&](int pk, S v) { bufio::store<S>(io.rd, pull_xy[1][1], zo + (unsigned)pk * io.plane_bytes, v); };
        double sx = 0.0, sy = 0.0, sz = 0.0;
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
            if constexpr (RED) {
                const double a = double(out[0]), d = double(out[2]);
                if (L::cx[k] != 0) sx += L::cx[k] > 0 ? a - d : d - a;
                if (L::cy[k] != 0) sy += L::cy[k] > 0 ? a - d : d - a;
                if (L::cz[k] != 0) sz += L::cz[k] > 0 ? a - d : d - a;
            }
        }
        S n0, g0;
        c.rest(rho_d, E_d, dE, n0, g0);
        put(0, n0);
        put(Q, g0);
        if constexpr (RED) {
            if (own_in) {
                nsum[0] += c.sumN + double(n0);
                nsum[1] += sx;
                nsum[2] += sy;
                nsum[3] += sz;
                nsum[4] += c.sumG + double(g0);
            }
        }
        if constexpr (MORE) {
            rho2 = rho;
            T2 = T;
            uz2 = uz1;
            uz1 = uz;
            Fp[0] = F[0]; Fp[1] = F[1]; Fp[2] = F[2];
            prev = cur;
            cur = nxt;
            face = nface;
            __syncthreads();
        }
    };
    for (int zf = z0 + 1; zf < z1; ++zf) iterate(zf, std::true_type{});
    iterate(z1, std::false_type{});

    if constexpr (RED) {
        // the wavefronts' sums by shuffles, then the wavefronts in order
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            double v = nsum[q];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
            if ((tid & 63) == 0) red[tid >> 6][q] = v;
        }
        __syncthreads();
        if (tid < 5) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < NTH / 64; ++w) t += red[w][tid];
            aux.partials[(long long)lb * 5 + tid] = t;
        }
    }
}

template <int Q, class S, class R, int NMODE, int EXT, bool RED>
__global__ void __launch_bounds__(kSplitThreads, sizeof(R) == 4 ? 3 : 2)
k_split_collide(const S* __restrict__ src, S* __restrict__ dst, const void* __restrict__ scratch,
                const StepGeom g, const Phys ph, const StepAux aux)
{
    __shared__ SplitLds<R, kSplitTX, kSplitTY> lds;
    const int lb = xcd_logical_block(blockIdx.x, gridDim.x, g.resident);
    if constexpr (RED) {
        __shared__ double red[kSplitThreads / 64][5];
        split_collide_tile<Q, S, R, NMODE, EXT, true>(lds, src, dst, scratch, g, ph, aux, lb, threadIdx.x, red);
    } else {
        split_collide_tile<Q, S, R, NMODE, EXT, false>(lds, src, dst, scratch, g, ph, aux, lb, threadIdx.x);
    }
}

}  // namespace lbm
