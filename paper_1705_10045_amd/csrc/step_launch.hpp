// Instantiation choice of the fused step (launch_one, launch_step_t), shared by the library's
// plain step launches and the launches that also form the state's totals.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "step_kernel.hpp"

namespace lbm {
namespace step_launch {

// One buffer resource per buffer needs every byte offset of the two population sets in 32 bits.
inline bool fits_buffer(const StepGeom& g, int Q, int storage_bytes)
{
    return (unsigned long long)g.plane * 2ull * Q * storage_bytes < (1ull << 32);
}

// The kernel of an instantiation: held to the registers of WAVES wavefronts per SIMD, or (0) as its
// workgroup size allows.
template <int WAVES, int Q, class S, class R, int TX, int TY, int NTH, bool PIPE, int ADDR, int NMODE,
          bool STASH, int EXT, bool RED>
constexpr auto step_function()
{
    if constexpr (WAVES != 0) return &k_step_waves<WAVES, Q, S, R, TX, TY, NTH, PIPE, ADDR, NMODE, STASH, EXT>;
    else return &k_step<Q, S, R, TX, TY, NTH, PIPE, ADDR, NMODE, STASH, EXT, RED>;
}

// The periodic instantiation, the one with walls and body force when the parameters ask for
// them, or the one that also carries the tabulated equation of state.
template <int Q, class S, class R, int TX, int TY, int NTH, bool PIPE, bool STASH, int ADDR,
          int NMODE, bool RED, int WAVES = 0>
hipError_t launch_one(const void* src, void* dst, const StepGeom& g, const Phys& ph,
                      const StepAux& aux, hipStream_t st)
{
    const unsigned nblk = (unsigned)(g.ntx * g.nty * g.nchunks);
    const bool ext = ph.walls || ph.g[0] != 0.0 || ph.g[1] != 0.0 || ph.g[2] != 0.0;
    if (ph.eos != 0)
        hipLaunchKernelGGL((step_function<WAVES, Q, S, R, TX, TY, NTH, PIPE, ADDR, NMODE, STASH, kExtTable, RED>()),
                           dim3(nblk), dim3(NTH), 0, st, (const S*)src, (S*)dst, g, ph, aux);
    else if (ext)
        hipLaunchKernelGGL((step_function<WAVES, Q, S, R, TX, TY, NTH, PIPE, ADDR, NMODE, STASH, kExtWalls, RED>()),
                           dim3(nblk), dim3(NTH), 0, st, (const S*)src, (S*)dst, g, ph, aux);
    else
        hipLaunchKernelGGL((step_function<WAVES, Q, S, R, TX, TY, NTH, PIPE, ADDR, NMODE, STASH, kExtNone, RED>()),
                           dim3(nblk), dim3(NTH), 0, st, (const S*)src, (S*)dst, g, ph, aux);
    return hipGetLastError();
}

// Picks the instantiation for the run-time facts: the address form the state allows, the
// tau = 1 collision (no re-read of N_k) when 1/tau is exactly 1 with BGK, and the MRT collision
// (which re-reads N_k, with the load order of tau != 1) when asked for.
//   - D2Q9 on the default tiles: below.
//   - FP32 states under 4 GB: one buffer resource per buffer.  Where the variant has the LDS
//     stash, the density prefetch stays on for tau = 1 only (re-reading N_k in the collision
//     leaves no registers for it).
//   - otherwise (FP64, the GLOBAL variant, states of 4 GB and more) global addressing, with the stash
//     where the variant asks for it and without the prefetch: at 512^3 the step is bound by
//     HBM traffic, and the stash saves the collision's second pull of the energy populations
//     (12.6 ms against 14.4 ms for the prefetch alone); not for FP64 with a collision that
//     re-reads N_k (it would spill).
template <int Q, class S, class R, int TX, int TY, int NTH, bool PIPE, bool STASH = false,
          bool GLOBAL = false, bool RED = false>
hipError_t launch_step_t(const void* src, void* dst, const StepGeom& g, const Phys& ph,
                         const StepAux& aux, hipStream_t st)
{
    const bool mrt = ph.collision != 0;
    const bool tau1 = ph.omega == 1.0 && !mrt;
    // D2Q9 on 256 threads: a step of one plane is one serial chain per tile, hidden only by other
    // tiles.  With buffer addressing, and the pulls in the order of their use, the step fits the
    // registers of four tiles per CU for tau = 1 (127, against 144 for FP32 and, with global addressing,
    // 192 for FP64) and of three for MRT (168, against 184) and FP64 (150, against 214) without spills.
    // us per step before and now, one card: FP32 500^2 16.3 and 13.3, 1000^2 51.6 and 49.0, 1400^2 93.0 and
    // 87.5; MRT 1000^2 62.3 and 52.7, 1400^2 116.7 and 96.9; FP64 350^2 13.6 and 10.4, 1000^2 78.9 and
    // 71.5, 1400^2 145.8 and 132.8.  FP32 with tau != 1 holds three either way and is 3% faster in the old order.
    // Two tiles per CU stay where the tiles are two rounds of them (FP64: two to four) with the last at
    // least half full: loads of one round then overlap the arithmetic of another.  The line is fitted to
    // squares, not derived (another card: FP64 500^2 19.3 against 22.1, 600^2 28.9 against 29.8, 700^2 36.5 against
    // 37.0, but 400^2 16.1 against 15.6; FP32 MRT 500^2 15.2 against 15.9, but 700^2 28.6 against 25.1); with it
    // no square from 64^2 to 1400^2 was slower than before.
    constexpr bool kPlane = Q == 9 && NTH == 256 && !GLOBAL && !RED;
    if constexpr (kPlane) {
        const int tiles = g.ntx * g.nty, round = g.resident;
        constexpr bool kWide = sizeof(S) == 8;
        const bool two = tiles > round && tiles <= (kWide ? 4 : 2) * round && (tiles - 1) % round >= round / 2;
        if (fits_buffer(g, Q, sizeof(S))) {
            if (tau1 && !(kWide && two)) return launch_one<Q, S, R, TX, TY, NTH, false, STASH, kAddrBuf, kTauOne, RED, 4>(src, dst, g, ph, aux, st);
            if (mrt && !two) return launch_one<Q, S, R, TX, TY, NTH, false, STASH, kAddrBuf, kMrt, RED, 3>(src, dst, g, ph, aux, st);
            if constexpr (kWide)
                if (!tau1 && !mrt && !two) return launch_one<Q, S, R, TX, TY, NTH, false, STASH, kAddrBuf, kTauAny, RED, 3>(src, dst, g, ph, aux, st);
        }
    }
    if constexpr (sizeof(S) == 4 && !GLOBAL) {
        if (fits_buffer(g, Q, 4)) {
            if constexpr (!kPlane)
                if (tau1) return launch_one<Q, S, R, TX, TY, NTH, PIPE, STASH, kAddrBuf, kTauOne, RED>(src, dst, g, ph, aux, st);
            if (mrt) return launch_one<Q, S, R, TX, TY, NTH, PIPE && !STASH, STASH, kAddrBuf, kMrt, RED>(src, dst, g, ph, aux, st);
            return launch_one<Q, S, R, TX, TY, NTH, PIPE && !STASH, STASH, kAddrBuf, kTauAny, RED>(src, dst, g, ph, aux, st);
        }
    }
    constexpr bool kStashAnyTau = STASH && sizeof(S) == 4;
    if (tau1) return launch_one<Q, S, R, TX, TY, NTH, PIPE && !STASH, STASH, kAddrGlobal, kTauOne, RED>(src, dst, g, ph, aux, st);
    if (mrt) return launch_one<Q, S, R, TX, TY, NTH, PIPE && !kStashAnyTau, kStashAnyTau, kAddrGlobal, kMrt, RED>(src, dst, g, ph, aux, st);
    return launch_one<Q, S, R, TX, TY, NTH, PIPE && !kStashAnyTau, kStashAnyTau, kAddrGlobal, kTauAny, RED>(src, dst, g, ph, aux, st);
}

}  // namespace step_launch
}  // namespace lbm
