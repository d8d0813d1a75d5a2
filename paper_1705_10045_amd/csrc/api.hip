// Host side of the C ABI (include/lbm_mi355x.h): parameter validation, the FP64 Maxwell
// table, device memory, stepping, moments, reductions and checkpoints.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/lbm_mi355x.h"
#include "host_threads.hpp"
#include "kernels.hpp"
#include "lattice.hpp"
#include "physics.hpp"
#include "sim.hpp"

namespace lbm {

static thread_local char g_last_error[512] = "";

void set_error(const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_last_error, sizeof(g_last_error), fmt, ap);
    va_end(ap);
}

void clear_error() { g_last_error[0] = '\0'; }

lbm_status hip_fail(hipError_t e, const char* what)
{
    set_error("%s: %s", what, hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? LBM_ENOMEM : LBM_EDEVICE;
}

lbm_status use_device(int device)
{
    const hipError_t e = hipSetDevice(device);
    return e == hipSuccess ? LBM_OK : hip_fail(e, "hipSetDevice");
}

// ------------------------------------------------------------------------------------------
// Maxwell coexistence table (section 5 band limits), reduced van der Waals fluid.
//
// Equal-area rule in specific volume v = 1/rho: p(v_l) = p(v_g) and
// integral_{v_l}^{v_g} p dv = p (v_g - v_l), with p(v) = 8T/(3v - 1) - 3/v^2 and the
// antiderivative (8T/3) ln(3v - 1) + 3/v.  Solved by Newton's method in (v_l, v_g),
// continued from the critical point (rho = 1 -/+ 2 sqrt(1 - T)) down the temperature grid.
// ------------------------------------------------------------------------------------------
namespace {

double p_of_v(double v, double T) { return 8.0 * T / (3.0 * v - 1.0) - 3.0 / (v * v); }
double dp_of_v(double v, double T)
{
    const double a = 3.0 * v - 1.0;
    return -24.0 * T / (a * a) + 6.0 / (v * v * v);
}
double int_p(double v, double T) { return (8.0 * T / 3.0) * std::log(3.0 * v - 1.0) + 3.0 / v; }

bool solve_coexistence(double T, double& vl, double& vg)
{
    for (int it = 0; it < 100; ++it) {
        const double pl = p_of_v(vl, T), pg = p_of_v(vg, T);
        const double f1 = pl - pg;
        const double f2 = int_p(vg, T) - int_p(vl, T) - pl * (vg - vl);
        const double a11 = dp_of_v(vl, T), a12 = -dp_of_v(vg, T);
        const double a21 = -dp_of_v(vl, T) * (vg - vl), a22 = pg - pl;
        const double det = a11 * a22 - a12 * a21;
        if (det == 0.0 || !std::isfinite(det)) return false;
        const double dl = (f1 * a22 - a12 * f2) / det;
        const double dg = (a11 * f2 - a21 * f1) / det;
        vl -= dl;
        vg -= dg;
        if (!(vl > 1.0 / 3.0) || !(vg > vl)) return false;
        if (std::fabs(dl) < 1e-15 * vl && std::fabs(dg) < 1e-15 * vg) return true;
    }
    return true;
}

struct MaxwellTable {
    std::vector<double> rho;  // interleaved (vapour, liquid) reduced densities
    double s0 = 0.0, ds = 0.0;
    bool ok = false;
};

const MaxwellTable& maxwell_table()
{
    static MaxwellTable tab;
    static std::once_flag once;
    std::call_once(once, [] {
        const int n = kMaxwellPoints;
        tab.rho.assign(2 * n, 0.0);
        tab.s0 = std::sqrt(1.0 - kLatentTmax);
        tab.ds = (std::sqrt(1.0 - kLatentTmin) - tab.s0) / (n - 1);
        double vl = 0, vg = 0, pl1 = 0, pg1 = 0, pl2 = 0, pg2 = 0;  // last two solutions
        bool good = true;
        for (int i = 0; i < n && good; ++i) {
            const double s = tab.s0 + i * tab.ds;
            const double T = 1.0 - s * s;
            if (i == 0) {          // critical-point asymptotics rho = 1 -/+ 2 sqrt(1 - T)
                vl = 1.0 / (1.0 + 2.0 * s);
                vg = 1.0 / (1.0 - 2.0 * s);
            } else if (i == 1) {   // previous solution
                vl = pl1;
                vg = pg1;
            } else {               // linear extrapolation along the branch
                vl = 2.0 * pl1 - pl2;
                vg = 2.0 * pg1 - pg2;
            }
            good = solve_coexistence(T, vl, vg);
            pl2 = pl1; pg2 = pg1;
            pl1 = vl; pg1 = vg;
            tab.rho[2 * i] = 1.0 / vg;
            tab.rho[2 * i + 1] = 1.0 / vl;
        }
        tab.ok = good;
    });
    return tab;
}

// dp/drho at fixed T for the reduced EOS in lattice units.
double dp_drho(double rho, double T, const Phys& ph)
{
    const double rr = rho * ph.inv_rho_c, tr = T * ph.inv_T_c;
    const double a = 3.0 - rr;
    return ph.p_c * ph.inv_rho_c * (24.0 * tr / (a * a) - 6.0 * rr);
}

// Pressure in lattice units of the simulation's EOS (the tabulated one from its host table);
// `inside` false outside a table's grid.
double host_pressure(double rho, double T, const Phys& ph, const double* table, bool& inside)
{
    inside = true;
    if (ph.eos == 0) return vdw_pressure(rho, T, ph);
    return ph.p_c * table_pressure(rho * ph.inv_rho_c, T * ph.inv_T_c, ph, table, inside);
}

// dp/drho at fixed T of the simulation's EOS: analytic for van der Waals, a central
// difference of the interpolant for a table (one-sided next to the grid's ends).
double host_dp_drho(double rho, double T, const Phys& ph, const double* table)
{
    if (ph.eos == 0) return dp_drho(rho, T, ph);
    const double h = 1e-6 * ph.rho_c;
    bool in_lo, in_hi;
    double lo_r = rho - h, hi_r = rho + h;
    double plo = host_pressure(lo_r, T, ph, table, in_lo);
    double phi = host_pressure(hi_r, T, ph, table, in_hi);
    if (!in_lo) { lo_r = rho; plo = host_pressure(rho, T, ph, table, in_lo); }
    if (!in_hi) { hi_r = rho; phi = host_pressure(rho, T, ph, table, in_hi); }
    return (phi - plo) / (hi_r - lo_r);
}

}  // namespace

bool host_band_limits(double Tr, double& rv, double& rl)
{
    const MaxwellTable& t = maxwell_table();
    if (!t.ok || !(Tr >= kLatentTmin && Tr <= kLatentTmax)) return false;
    const double pos = (std::sqrt(1.0 - Tr) - t.s0) / t.ds;
    int j = (int)pos;
    j = j < 1 ? 1 : (j > kMaxwellPoints - 3 ? kMaxwellPoints - 3 : j);
    const double x = pos - j;
    const double l0 = -x * (x - 1.0) * (x - 2.0) / 6.0, l1 = (x + 1.0) * (x - 1.0) * (x - 2.0) / 2.0;
    const double l2 = -(x + 1.0) * x * (x - 2.0) / 2.0, l3 = (x + 1.0) * x * (x - 1.0) / 6.0;
    const double* q = t.rho.data() + 2 * (j - 1);
    rv = l0 * q[0] + l1 * q[2] + l2 * q[4] + l3 * q[6];
    rl = l0 * q[1] + l1 * q[3] + l2 * q[5] + l3 * q[7];
    return true;
}

Phys make_phys(const lbm_params& p)
{
    Phys ph;
    ph.omega = 1.0 / p.tau;
    ph.omega_E = 1.0 / p.tau_E;
    ph.A = p.A;
    ph.inv_alpha = p.lattice == 9 ? 1.0 / Lattice<9>::alpha : 1.0 / Lattice<19>::alpha;
    ph.rho_c = p.rho_c;
    ph.inv_rho_c = 1.0 / p.rho_c;
    ph.inv_T_c = 1.0 / p.T_c;
    ph.p_c = p.p_c;
    ph.c_v = p.c_v;
    ph.inv_c_v = 1.0 / p.c_v;
    ph.cond_half = 0.5 * p.c_v * p.chi;
    ph.rhoQ = p.rhoQ;
    ph.T0_baro = p.T0_baro;
    ph.flags = p.flags;
    ph.walls = p.walls;
    ph.wall_heat = p.walls ? p.wall_heat : 0u;
    ph.T_bottom = p.T_bottom;
    ph.T_top = p.T_top;
    for (int a = 0; a < 3; ++a) ph.g[a] = p.gravity[a];
    ph.collision = p.collision;
    const bool mrt = p.collision == LBM_COLLISION_MRT;
    ph.mrt_de = mrt ? p.s_e - ph.omega : 0.0;
    ph.mrt_deps = mrt ? p.s_eps - ph.omega : 0.0;
    ph.mrt_dq = mrt ? p.s_q - ph.omega : 0.0;
    ph.mrt_dm = mrt ? p.s_m - ph.omega : 0.0;
    ph.eos = p.eos == LBM_EOS_TABLE ? 1 : 0;
    ph.tab_nrho = ph.eos ? p.eos_nrho : 0;
    ph.tab_nT = ph.eos ? p.eos_nT : 0;
    ph.tab_rho_min = p.eos_rho_min;
    ph.tab_rho_max = p.eos_rho_max;
    ph.tab_T_min = p.eos_T_min;
    ph.tab_T_max = p.eos_T_max;
    ph.tab_drho = ph.eos ? (p.eos_rho_max - p.eos_rho_min) / (p.eos_nrho - 1) : 0.0;
    ph.tab_dT = ph.eos ? (p.eos_T_max - p.eos_T_min) / (p.eos_nT - 1) : 0.0;
    return ph;
}

// Elements between consecutive population planes: the node count rounded up to 64 (256 B in
// FP32), plus 64 more, so that the same node of consecutive planes does not sit at the same
// power-of-two alignment (for the power-of-two boxes of the workloads every plane would
// otherwise start at a multiple of 8 MB-512 MB).  Measured 1-2.5% faster at 512^3, neutral at
// 128^3 and 256^3.
long long padded_plane(long long n) { return (n + 63) / 64 * 64 + 64; }

// Elements of one population plane's rows (x rows padded to the row pitch).
long long plane_elements(const lbm_params& p)
{
    return (long long)row_pitch(p.nx, p.storage_bytes) * p.ny * p.nz;
}

size_t state_bytes(const lbm_params& p)
{
    return (size_t)2 * p.lattice * padded_plane(plane_elements(p)) * p.storage_bytes;
}

lbm_status validate_params(const lbm_params* p)
{
    if (!p) { set_error("params is NULL"); return LBM_EINVAL; }
    if (p->lattice != 9 && p->lattice != 19) {
        set_error("lattice must be 9 (D2Q9) or 19 (D3Q19), got %d", p->lattice);
        return LBM_EINVAL;
    }
    if (p->nx < 1 || p->ny < 1 || p->nz < 1) { set_error("box extents must be >= 1"); return LBM_EINVAL; }
    if (p->lattice == 9 && p->nz != 1) { set_error("D2Q9 needs nz == 1"); return LBM_EINVAL; }
    if ((long long)p->nx * p->ny * p->nz >= (1LL << 31)) { set_error("box exceeds 2^31 nodes"); return LBM_EINVAL; }
    if (p->storage_bytes != 4 && p->storage_bytes != 8) { set_error("storage_bytes must be 4 or 8"); return LBM_EINVAL; }
    if (!(p->tau > 0.5) || !(p->tau_E > 0.5)) { set_error("BGK needs tau > 1/2 and tau_E > 1/2"); return LBM_EINVAL; }
    if (!(p->rho_c > 0) || !(p->T_c > 0) || !(p->p_c > 0) || !(p->c_v > 0)) {
        set_error("rho_c, T_c, p_c and c_v must be positive");
        return LBM_EINVAL;
    }
    if (!(p->chi >= 0) || !(p->rhoQ >= 0) || !std::isfinite(p->A)) { set_error("chi, rhoQ must be >= 0 and A finite"); return LBM_EINVAL; }
    const int d = (p->nx > 1) + (p->ny > 1) + (p->lattice == 19 && p->nz > 1);
    if ((p->flags & LBM_CONDUCTION) && !(p->chi < 0.5 / (d < 1 ? 1 : d))) {
        set_error("explicit conduction needs chi < 0.5/d = %g (section 6.1)", 0.5 / (d < 1 ? 1 : d));
        return LBM_EINVAL;
    }
    if ((p->flags & LBM_BAROTROPIC) && !(p->T0_baro > 0)) { set_error("barotropic EOS needs T0_baro > 0"); return LBM_EINVAL; }
    if (p->walls != 0 && p->walls != 1) { set_error("walls must be 0 (periodic) or 1, got %d", p->walls); return LBM_EINVAL; }
    if (p->walls) {
        if (p->lattice != 19 || p->nz < 2) { set_error("walls need D3Q19 and nz >= 2"); return LBM_EINVAL; }
        if (((p->wall_heat & LBM_WALL_T_BOTTOM) && !(p->T_bottom > 0 && std::isfinite(p->T_bottom))) ||
            ((p->wall_heat & LBM_WALL_T_TOP) && !(p->T_top > 0 && std::isfinite(p->T_top)))) {
            set_error("a held wall temperature must be positive and finite");
            return LBM_EINVAL;
        }
        // a held wall face is half a cell from the node next to it, which doubles its conductance
        const double lim = 1.0 / (2 * (d < 1 ? 1 : d) + 1);
        if ((p->flags & LBM_CONDUCTION) && (p->wall_heat & (LBM_WALL_T_BOTTOM | LBM_WALL_T_TOP)) &&
            !(p->chi < lim)) {
            set_error("conduction next to a held wall needs chi < 1/(2d + 1) = %g", lim);
            return LBM_EINVAL;
        }
    }
    for (int a = 0; a < 3; ++a)
        if (!std::isfinite(p->gravity[a])) { set_error("gravity must be finite"); return LBM_EINVAL; }
    if (p->collision != LBM_COLLISION_BGK && p->collision != LBM_COLLISION_MRT) {
        set_error("collision must be LBM_COLLISION_BGK (0) or LBM_COLLISION_MRT (1), got %d", p->collision);
        return LBM_EINVAL;
    }
    if (p->collision == LBM_COLLISION_MRT) {
        const double r[4] = {p->s_e, p->s_eps, p->s_q, p->s_m};
        for (int i = 0; i < 4; ++i)
            if (!(r[i] > 0.0 && r[i] < 2.0)) { set_error("MRT rates must lie in (0, 2)"); return LBM_EINVAL; }
    }
    if (p->eos != LBM_EOS_VDW && p->eos != LBM_EOS_TABLE) {
        set_error("eos must be LBM_EOS_VDW (0) or LBM_EOS_TABLE (1), got %d", p->eos);
        return LBM_EINVAL;
    }
    if (p->eos == LBM_EOS_TABLE) {
        if (!p->eos_p || !p->eos_coex || p->eos_nrho < 4 || p->eos_nT < 2 ||
            (long long)p->eos_nrho * p->eos_nT > (1LL << 26)) {
            set_error("a tabulated EOS needs eos_p and eos_coex, eos_nrho >= 4, eos_nT >= 2 and at most 2^26 points");
            return LBM_EINVAL;
        }
        if (!(p->eos_rho_max > p->eos_rho_min && p->eos_rho_min >= 0.0 && std::isfinite(p->eos_rho_max)) ||
            !(p->eos_T_max > p->eos_T_min && p->eos_T_min > 0.0 && std::isfinite(p->eos_T_max))) {
            set_error("a tabulated EOS needs 0 <= eos_rho_min < eos_rho_max and 0 < eos_T_min < eos_T_max");
            return LBM_EINVAL;
        }
        for (long long i = 0; i < (long long)p->eos_nrho * p->eos_nT; ++i)
            if (!std::isfinite(p->eos_p[i])) { set_error("EOS table value %lld is not finite", i); return LBM_EINVAL; }
        for (int j = 0; j < p->eos_nT; ++j)
            if (!(p->eos_coex[2 * j] <= p->eos_coex[2 * j + 1]) || !std::isfinite(p->eos_coex[2 * j + 1])) {
                set_error("EOS coexistence row %d needs finite rho_1 <= rho_2", j);
                return LBM_EINVAL;
            }
    }
    // the step addresses nodes within one population plane with 32-bit byte offsets
    const long long n = plane_elements(*p);
    if ((unsigned long long)padded_plane(n) * (unsigned long long)p->storage_bytes >= (1ull << 32)) {
        set_error("one population plane of %lld elements exceeds 4 GB", n);
        return LBM_EINVAL;
    }
    if ((p->flags & LBM_LATENT) && !maxwell_table().ok) { set_error("Maxwell table construction failed"); return LBM_EDEVICE; }
    return LBM_OK;
}

namespace {

enum class FieldFault { kNone, kState, kVelocity, kTable, kPhi, kSlope };

// What is wrong with the initial state of node i; dpdr as far as it was formed.
FieldFault field_fault(const lbm_params& p, const Phys& ph, const double* rho0, const double* u0, const double* T0,
                       long long n, long long i, double& dpdr)
{
    const double bound = 1.0 + kTheta;  // (h/dt)^2 + theta, section 3
    const double r = rho0[i], T = T0[i];
    if (!(r > 0) || !(r * ph.inv_rho_c < 3.0) || !(T > 0) || !std::isfinite(T)) return FieldFault::kState;
    if (!std::isfinite(u0[i]) || !std::isfinite(u0[n + i]) || !std::isfinite(u0[2 * n + i])) return FieldFault::kVelocity;
    const double Te = (p.flags & LBM_BAROTROPIC) ? p.T0_baro : T;
    bool inside;
    const double pr = host_pressure(r, Te, ph, p.eos_p, inside);
    if (!inside) return FieldFault::kTable;
    if (!(r * kTheta - pr > 0)) return FieldFault::kPhi;
    dpdr = host_dp_drho(r, Te, ph, p.eos_p);
    return dpdr > bound ? FieldFault::kSlope : FieldFault::kNone;
}

}  // namespace

lbm_status validate_fields(const lbm_params& p, const double* rho0, const double* u0, const double* T0)
{
    if (!rho0 || !u0 || !T0) { set_error("initial fields must not be NULL"); return LBM_EINVAL; }
    const long long n = (long long)p.nx * p.ny * p.nz;
    const Phys ph = make_phys(p);
    // On one core the checks cost more than the upload of the fields (submission of a 96^3 request 3.5 ms,
    // with eight threads 1.9).  A thread is worth its start from some 10 thousand nodes on.  Every thread
    // stops at its first bad node, and the lowest of them is reported.
    const int threads = host_threads(n, 16384);
    std::array<long long, kHostThreads> bad;
    bad.fill(n);
    on_threads(threads, [&](int t) {
        double dpdr;
        const long long end = n * (t + 1) / threads;
        for (long long i = n * t / threads; i < end; ++i)
            if (field_fault(p, ph, rho0, u0, T0, n, i, dpdr) != FieldFault::kNone) {
                bad[t] = i;
                return;
            }
    });
    const long long i = *std::min_element(bad.begin(), bad.end());
    if (i == n) return LBM_OK;
    double dpdr = 0.0;
    const FieldFault fault = field_fault(p, ph, rho0, u0, T0, n, i, dpdr);
    const double Te = (p.flags & LBM_BAROTROPIC) ? p.T0_baro : T0[i];
    if (fault == FieldFault::kState)
        set_error("node %lld: need 0 < rho0 < 3 rho_c and T0 > 0 (rho0 = %g, T0 = %g)", i, rho0[i], T0[i]);
    else if (fault == FieldFault::kVelocity)
        set_error("node %lld: non-finite velocity", i);
    else if (fault == FieldFault::kTable)
        set_error("node %lld: (rho, T) = (%g, %g) outside the EOS table", i, rho0[i], Te);
    else if (fault == FieldFault::kPhi)
        set_error("node %lld: Phi^2 = rho theta - p <= 0 (section 3)", i);
    else
        set_error("node %lld: (dp/drho)_T = %g exceeds the stability bound %g (section 3)", i, dpdr, 1.0 + kTheta);
    return LBM_EINVAL;
}

// Launch geometry: tiles of the selected variant and z chunks sized so that one round of
// workgroups fills the GPU, unless a chunk length is given.
// The launch of the fused step for these parameters, launch variant and z-chunk request
// (0 = automatic) on a device with `cus` compute units; host arithmetic only.
StepGeom plan_geometry(const lbm_params& p, int variant, int chunk_request, int cus, int& tx, int& ty)
{
    int per_cu;
    step_tile(p.lattice, p.storage_bytes, variant, tx, ty, per_cu);
    StepGeom g{};
    g.nx = p.nx; g.ny = p.ny; g.nz = p.nz;
    g.pitch = row_pitch(p.nx, p.storage_bytes);
    g.plane = padded_plane(plane_elements(p));
    g.ntx = (p.nx + tx - 1) / tx;
    g.nty = (p.ny + ty - 1) / ty;
    int chunk = p.nz;
    // workgroups the device holds at once: the launch runs in rounds of this many, and the
    // kernel gives each round a contiguous band of tiles
    g.resident = cus * per_cu;
    if (p.lattice == 19) {
        // z chunks.  Each chunk runs the moment stage on 4 planes outside it (2 on each side),
        // and the launch runs in rounds of `target` workgroups (later ones start as earlier
        // ones retire), so a step takes about ceil(workgroups / target) x (chunk + 4) plane
        // times of one workgroup.  The chunk count minimising that is taken (the fewest
        // chunks among equals; chunks of at least 4 planes): a box whose columns do not fill
        // whole rounds gets more, shorter chunks (288^3: 162 columns, 3 chunks, 486
        // workgroups in two nearly full rounds, instead of 324 in one full and one quarter
        // round), and powers of two keep one round of long chunks.
        const long long cols = (long long)g.ntx * g.nty;
        const long long target = (long long)cus * per_cu;
        const long long maxc = p.nz / 4 > 0 ? p.nz / 4 : 1;
        long long best_cost = -1;
        for (long long nc = 1; nc <= maxc; ++nc) {
            const long long c = (p.nz + nc - 1) / nc;
            const long long chunks = (p.nz + c - 1) / c;
            const long long rounds = (cols * chunks + target - 1) / target;
            const long long cost = rounds * (c + 4);
            if (best_cost < 0 || cost < best_cost) {
                best_cost = cost;
                chunk = (int)c;
            }
        }
        if (chunk_request > 0) chunk = chunk_request < p.nz ? chunk_request : p.nz;
    }
    g.chunk = chunk;
    g.nchunks = (p.nz + chunk - 1) / chunk;
    set_reciprocals(g);
    return g;
}

// Variant lbm_init starts with: 7 (64 x 8 tiles, global addressing) for FP32 D3Q19 states
// beyond one buffer resource's 4 GB where 64-wide tiles leave no more x columns idle than
// 32-wide ones, else 0.
int default_variant(const lbm_params& p)
{
    if (p.lattice != 19 || p.storage_bytes != 4) return 0;
    if (state_bytes(p) < (1ull << 32)) return 0;
    const long long w64 = (p.nx + 63LL) / 64 * 64, w32 = (p.nx + 31LL) / 32 * 32;
    return w64 <= w32 ? 7 : 0;
}

void choose_geometry(lbm_sim* s, int chunk_request)
{
    int tx, ty;
    s->geom = plan_geometry(s->p, s->variant, chunk_request, s->cus, tx, ty);
    s->geom.plane = s->plane;
    s->tile_x = tx;
    s->tile_y = ty;
}

// Tiles and z chunks of the collision launch of the two-launch step (split_kernel.hpp).  Its
// workgroups are small and several run on a CU, so chunks are short: one plane while all tiles
// of all planes run at once (an idle chip is bound by the chain of one workgroup: 32^3 takes
// 10.4 us with chunks of 1, 12.6 with 2, 17.4 with 4), two up to eight rounds (96^3: 85.6, 82.3,
// 84.8 us), then four, whose extra planes no longer matter (160^3: 410, 382, 370 us; 8: 369).
StepGeom split_geometry(const lbm_params& p, int cus)
{
    int tx, ty;
    split_tile(tx, ty);
    StepGeom g{};
    g.nx = p.nx; g.ny = p.ny; g.nz = p.nz;
    g.pitch = row_pitch(p.nx, p.storage_bytes);
    g.plane = padded_plane(plane_elements(p));
    g.ntx = (p.nx + tx - 1) / tx;
    g.nty = (p.ny + ty - 1) / ty;
    const int per_cu = p.storage_bytes == 4 ? 3 : 2;   // by registers: 168 and 256 VGPRs
    const long long tiles = (long long)g.ntx * g.nty * p.nz, round = (long long)cus * per_cu;
    g.resident = (int)round;
    g.chunk = tiles <= round ? 1 : (tiles <= 8 * round ? 2 : 4);
    if (g.chunk > p.nz) g.chunk = p.nz;
    g.nchunks = (p.nz + g.chunk - 1) / g.chunk;
    set_reciprocals(g);
    return g;
}

// The two-launch step covers D3Q19 states under 4 GB (one buffer resource).
bool split_covers(const lbm_params& p) { return p.lattice == 19 && state_bytes(p) < (1ull << 32); }

// Whether the default step of these parameters runs as two launches: where their estimated time
// is at least 5% below that of the fused launch.  Both estimates follow the measured times over
// 18 boxes from 32^3 to 220x180x200 (within 10%, mostly within 5%):
//   - two launches: 5 us and, per lane of the padded 32 x 8 tiles, 92 / 106 / 111 ps for FP32 with
//     tau = 1 / other tau / MRT and 168 / 192 / 196 ps for FP64;
//   - fused: rounds of resident workgroups times (chunk + 4) planes of 9.4 / 9.9 / 10.4 us for
//     FP32 and 11.9 / 10.6 / 11.0 us for FP64, whatever the tiles' idle lanes.
// So small boxes, whose fused launch is a few workgroups or a long chain, and ragged ones go
// through two launches (FP32: 32^3 40.8 -> 10.4 us, 64^3 49.2 -> 24.1, 100^3 142 -> 118,
// 200x150x97 330 -> 303; FP64: 128^3 457 -> 347), and the fused launch keeps the boxes that fill
// its rounds, where it moves fewer bytes (128^3 FP32: 191 against 203 us).
bool split_default(const lbm_params& p, const StepGeom& fused, const StepGeom& split, int cus, int per_cu)
{
    if (!split_covers(p)) return false;
    const int kind = p.collision == LBM_COLLISION_MRT ? 2 : (p.tau == 1.0 ? 0 : 1);
    static const double lane_ps[2][3] = {{92, 106, 111}, {168, 192, 196}};
    static const double plane_us[2][3] = {{9.4, 9.9, 10.4}, {11.9, 10.6, 11.0}};
    const int wide = p.storage_bytes == 8;
    int tx, ty;
    split_tile(tx, ty);
    const double lanes = (double)split.ntx * tx * split.nty * ty * p.nz;
    const double two = 5.0 + 1e-6 * lane_ps[wide][kind] * lanes;
    const long long round = (long long)cus * per_cu;
    const long long rounds = (step_workgroups(fused) + round - 1) / round;
    return two < 0.95 * (double)rounds * (fused.chunk + 4) * plane_us[wide][kind];
}

// Whether the step that forms the totals runs as two launches.  For tau = 1, and for MRT in FP64, it does
// wherever it can: it was the faster form in all of 23 boxes from 48^3 to 200^3 (FP32 1 to 37%: the fused form's
// totals cost its prefetch; FP64 10 to 61%: they cost it registers).  For the other collisions the totals leave
// the two-launch form's collision short of registers, and where the fused launch fills its rounds it is up to
// 16% faster (FP32 tau = 0.8 at 128^3 222 us against 250, 256x256x64 429 against 487).  Their estimates follow
// the measured times of the 23 boxes within 10%:
//   - two launches: 5 us and, per lane of the padded tiles, 111 / 115 ps for FP32 with BGK / MRT and 168 ps for
//     FP64 while two states fit the 256 MB last-level cache, 115 / 123 / 194 ps beyond;
//   - fused: per round 15 us for the halo planes and, per plane, a part for the workgroup and one for the share of
//     its lanes that have nodes.
// Two launches run where they are 3% faster by these: then no box of the 23 was slower than the fused form
// (FP32 tau = 0.8: 64^3 31 us against 56, 80^3 64 against 78; 96^3 104 fused against 107).
bool split_totals(const lbm_params& p, const StepGeom& fused, const StepGeom& split, int cus, int per_cu)
{
    if (!split_covers(p)) return false;
    const bool mrt = p.collision == LBM_COLLISION_MRT, wide = p.storage_bytes == 8;
    if ((p.tau == 1.0 && !mrt) || (wide && mrt)) return true;
    struct Cost { double lane_ps[2], group_us, nodes_us, round_us; };
    static const Cost costs[3] = {{{111, 115}, 9.35, 3.82, 14.8},   // FP32 BGK
                                  {{115, 123}, 9.47, 4.15, 15.9},   // FP32 MRT
                                  {{168, 194}, 8.81, 3.63, 15.1}};  // FP64 BGK
    const Cost& c = costs[wide ? 2 : (mrt ? 1 : 0)];
    int stx, sty, ftx, fty, unused;
    split_tile(stx, sty);
    step_tile(p.lattice, p.storage_bytes, 0, ftx, fty, unused);
    const double lanes = (double)split.ntx * stx * split.nty * sty * p.nz;
    const double two = 5.0 + 1e-6 * c.lane_ps[2 * state_bytes(p) > (256u << 20)] * lanes;
    const long long round = (long long)cus * per_cu;
    const long long rounds = (step_workgroups(fused) + round - 1) / round;
    const double planes = (double)rounds * fused.chunk;
    const double share = (double)p.nx * p.ny * p.nz / (planes * round * ftx * fty);
    return two < 0.97 * (planes * (c.group_us + c.nodes_us * share) + rounds * c.round_us);
}

// The scratch of the two-launch step: a workspace, not state.  False without room for it.
bool ensure_split(lbm_sim* s)
{
    if (s->d_split) return true;
    if (!split_covers(s->p)) return false;
    if (s->split_refused) return false;
    s->split_geom = split_geometry(s->p, s->cus);
    if (hipMalloc(&s->d_split, split_scratch_bytes(s->p.storage_bytes, plane_elements(s->p))) == hipSuccess) {
        s->own_split = true;
        return true;
    }
    (void)hipGetLastError();
    s->d_split = nullptr;
    s->split_refused = true;   // (a refusal costs more than a step gains)
    return false;
}

// Region of a launch of `steps` D2Q9 steps on tx x ty tiles (multi_kernel.hpp).
MultiGeom multi_geometry(const lbm_params& p, int tx, int ty, int steps)
{
    MultiGeom m{};
    m.tx = tx;
    m.ty = ty;
    m.steps = steps;
    m.margin = 3 * steps - 1;
    m.rx = tx + 2 * m.margin;
    m.ry = p.ny == 1 ? 1 : ty + 2 * m.margin;
    m.inv_rx = 1.0 / m.rx;
    return m;
}

// Tiles and steps per launch of the D2Q9 boxes that take several steps per launch; steps = 0 for
// the others.  The tiles have to run in one round, one workgroup per CU (its LDS is up to 129 KB): a region of 704
// nodes, tile and halo, allows that up to about 350^2 and 150,000 nodes in a row.  Among the tiles and step counts
// that do, the one of least time per step is taken, a launch taking about 2 us and each of its steps 2.1 us
// plus 0.21 us per further wavefront of the region (measured over 12 tiles and 1 to 16 steps).  us per step, single
// steps and these: FP64 1000 nodes 6.1 and 2.1, 128^2 7.1 and 4.5, 256^2 7.9 and 6.1, 300^2 9.3 and 8.5; FP32 256^2 7.4
// and 5.6, 350^2 8.5 and 7.8.
MultiGeom plan_multi(const lbm_params& p, int cus)
{
    MultiGeom best{};
    if (p.lattice != 9 || state_bytes(p) >= (1ull << 32)) return best;
    const int nodes = multi_nodes();
    double least = 0.0;
    for (int steps = 1; steps <= 16; ++steps) {
        for (int ty = (p.ny + cus - 1) / cus; ty <= p.ny; ++ty) {
            const long long rows = (p.ny + ty - 1) / ty;
            // the narrowest tile whose columns fit the round
            const int cols = (int)(cus / rows) < p.nx ? (int)(cus / rows) : p.nx;
            const int tx = (p.nx + cols - 1) / cols;
            const MultiGeom m = multi_geometry(p, tx, ty, steps);
            if (m.ry > nodes) break;
            if ((long long)m.rx * m.ry > nodes) continue;
            const int waves = (m.rx * m.ry + 63) / 64;
            const double t = (2.0 + steps * (2.1 + 0.21 * (waves - 1))) / steps;
            if (best.steps == 0 || t < least) {
                best = m;
                least = t;
            }
        }
    }
    // FP64 populations, one step: beyond 9 wavefronts single steps are as fast (350^2 10.2 us either way), and with 9
    // where the tile is narrow, so that its rows are parts of a few lines (20 x 20: 320^2 9.6 us against 9.3,
    // 500x200 10.2 against 9.7; 28 x 14: 304x320 8.6 against 9.1), unless the 32 x 8 tiles of single steps
    // leave more lanes idle (40x2400 8.7 against 11.1)
    if (best.steps == 1 && p.storage_bytes == 8) {
        const int region = best.rx * best.ry;
        const double lanes = ((p.nx + 31LL) / 32 * 32) * (double)((p.ny + 7LL) / 8 * 8);
        if (region > 576 || (region > 512 && best.tx < 24 && (double)p.nx * p.ny > 0.85 * lanes)) return MultiGeom{};
    }
    return best;
}

hipError_t enqueue_multi(lbm_sim* s, int steps)
{
    const MultiGeom m = multi_geometry(s->p, s->multi.tx, s->multi.ty, steps);
    StepGeom g = s->geom;
    g.ntx = (s->p.nx + m.tx - 1) / m.tx;
    g.nty = (s->p.ny + m.ty - 1) / m.ty;
    set_reciprocals(g);
    return launch_multi(s->p.storage_bytes, s->buf[s->cur], s->buf[1 - s->cur], g, m, s->phys, s->aux, s->stream);
}

// The simulation's device memory in one allocation: the two population buffers, the error words, the
// table of the band limits, the partial sums of lbm_reduce and, where the default step is two launches,
// their scratch (without room for that the fused step runs).  For 64^3 this one and its release take
// 105 and 330 us, six by themselves took 195 and 780, beside 2.5 ms for 100 steps.
hipError_t allocate(lbm_sim* s)
{
    int tx, ty, per_cu;
    step_tile(s->p.lattice, s->p.storage_bytes, s->variant, tx, ty, per_cu);
    const StepGeom geom = split_geometry(s->p, s->cus);
    const auto part = [](size_t bytes) { return (bytes + 4095) / 4096 * 4096; };
    // the second buffer begins on a large page as the first, but for states of a few pages, which would
    // hold up to ten times their size (1000 nodes 4.3 MB for 0.4)
    constexpr size_t kLargePage = (size_t)2 << 20;
    const size_t bytes = state_bytes(s->p);
    const size_t state = bytes < 8 * kLargePage ? part(bytes) : (bytes + kLargePage - 1) / kLargePage * kLargePage;
    const size_t err = 2 * state, table = err + part(sizeof(int) * 16);
    const size_t partials = table + part(sizeof(double) * maxwell_table().rho.size());
    const size_t scratch = partials + part(sizeof(double) * (5 * s->red_blocks + 8));
    const size_t more = split_default(s->p, s->geom, geom, s->cus, per_cu)
                            ? split_scratch_bytes(s->p.storage_bytes, plane_elements(s->p)) : 0;
    s->split = more > 0;
    hipError_t e = hipMalloc((void**)&s->memory, scratch + more);
    if (e != hipSuccess && s->split) {
        (void)hipGetLastError();
        s->split = false;
        e = hipMalloc((void**)&s->memory, scratch);
    }
    if (e != hipSuccess) return e;
    s->buf[0] = s->memory;
    s->buf[1] = s->memory + state;
    s->d_err = reinterpret_cast<int*>(s->memory + err);
    s->d_table = reinterpret_cast<double*>(s->memory + table);
    s->d_partials = reinterpret_cast<double*>(s->memory + partials);
    if (s->split) {
        s->split_geom = geom;
        s->d_split = s->memory + scratch;
    }
    return hipSuccess;
}

lbm_status upload_table(lbm_sim* s)
{
    const MaxwellTable& t = maxwell_table();
    hipError_t e = hipMemcpyAsync(s->d_table, t.rho.data(), sizeof(double) * t.rho.size(), hipMemcpyHostToDevice, s->stream);
    if (e != hipSuccess) return hip_fail(e, "upload Maxwell table");
    s->aux.maxwell = s->d_table;
    s->aux.tab_s0 = t.s0;
    s->aux.tab_inv_ds = 1.0 / t.ds;
    return LBM_OK;
}

lbm_status enqueue_steps(lbm_sim* s, int nsteps)
{
    if (!s->aux.err || !s->aux.maxwell || !s->buf[0] || !s->buf[1]) {
        set_error("simulation is not fully initialised (null device pointer)");
        return LBM_EDEVICE;
    }
    const bool multi = s->multi.steps > 0 && !s->launch_set;
    // launches of several steps: even in number for an even number of steps and odd for an odd one, so that
    // the state's buffer follows the step count in every form (a caller's graph of an even number of
    // steps leaves the state where it found it and can be replayed), and of like lengths
    int launches = nsteps;
    if (multi) {
        launches = (nsteps + s->multi.steps - 1) / s->multi.steps;
        launches += (launches ^ nsteps) & 1;
    }
    for (int i = 0, taken = 1; i < nsteps; i += taken, --launches) {
        hipError_t e;
        taken = 1;
        if (multi) {
            taken = (nsteps - i + launches - 1) / launches;
            e = enqueue_multi(s, taken);
        } else if (s->split) {
            e = launch_split_moments(s->p.storage_bytes, s->buf[s->cur], s->d_split, s->split_geom, s->phys,
                                     s->aux, s->stream);
            if (e == hipSuccess)
                e = launch_split_collide(s->p.storage_bytes, s->buf[s->cur], s->buf[1 - s->cur], s->d_split,
                                         s->split_geom, s->phys, s->aux, s->stream);
        } else {
            e = launch_step(s->p.lattice, s->p.storage_bytes, s->variant, s->buf[s->cur],
                            s->buf[1 - s->cur], s->geom, s->phys, s->aux, s->stream);
        }
        if (e != hipSuccess) return hip_fail(e, "step launch");
        s->cur ^= 1;
        s->step += taken;
    }
    return LBM_OK;
}

lbm_status read_error_word(lbm_sim* s)
{
    int h = 0;
    hipError_t e = hipMemcpyAsync(&h, s->d_err, sizeof(int), hipMemcpyDeviceToHost, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return hip_fail(e, "reading the device error word");
    if (h) {
        set_error("a node left the EOS domain (Phi^2 <= 0, rho >= 3 rho_c or non-finite) by step %lld", s->step);
        return LBM_EUNSTABLE;
    }
    return LBM_OK;
}

}  // namespace lbm

using namespace lbm;

extern "C" {

const char* lbm_last_error(void) { return g_last_error; }

size_t lbm_footprint_bytes(const lbm_params* p)
{
    if (!p) return 0;
    size_t tables = sizeof(double) * 2 * kMaxwellPoints + 64;
    if (p->eos == LBM_EOS_TABLE && p->eos_nrho > 0 && p->eos_nT > 0)
        tables += sizeof(double) * ((size_t)p->eos_nrho * p->eos_nT + 2 * (size_t)p->eos_nT);
    return 2 * state_bytes(*p) + tables;
}

int lbm_lattice_info(int Q, int* c, double* w, double* G, double* alpha)
{
    if (Q == 9) {
        for (int k = 0; k < 9; ++k) {
            c[3 * k] = Lattice<9>::cx[k]; c[3 * k + 1] = Lattice<9>::cy[k]; c[3 * k + 2] = Lattice<9>::cz[k];
            w[k] = weight<9>(k); G[k] = force_coef<9>(k);
        }
        *alpha = Lattice<9>::alpha;
        return 2;
    }
    if (Q == 19) {
        for (int k = 0; k < 19; ++k) {
            c[3 * k] = Lattice<19>::cx[k]; c[3 * k + 1] = Lattice<19>::cy[k]; c[3 * k + 2] = Lattice<19>::cz[k];
            w[k] = weight<19>(k); G[k] = force_coef<19>(k);
        }
        *alpha = Lattice<19>::alpha;
        return 3;
    }
    return LBM_EINVAL;
}

lbm_status lbm_coexistence(double Tr, double* rho_v, double* rho_l)
{
    double rv, rl;
    if (!host_band_limits(Tr, rv, rl)) {
        set_error("reduced temperature %g outside the Maxwell table [%g, %g]", Tr, kLatentTmin, kLatentTmax);
        return LBM_EINVAL;
    }
    if (rho_v) *rho_v = rv;
    if (rho_l) *rho_l = rl;
    return LBM_OK;
}

lbm_status lbm_init(const lbm_params* params, const double* rho0, const double* u0, const double* T0,
                    void* stream, lbm_sim** out)
{
    clear_error();
    if (!out) { set_error("out is NULL"); return LBM_EINVAL; }
    *out = nullptr;
    lbm_status st = validate_params(params);
    if (st != LBM_OK) return st;
    st = validate_fields(*params, rho0, u0, T0);
    if (st != LBM_OK) return st;

    lbm_sim* s = new lbm_sim();
    s->p = *params;
    s->phys = make_phys(*params);
    s->n = (long long)params->nx * params->ny * params->nz;
    s->plane = padded_plane(plane_elements(s->p));
    if (hipError_t e = hipGetDevice(&s->device); e != hipSuccess) {
        delete s;
        return hip_fail(e, "hipGetDevice");
    }
    if (hipError_t e = hipDeviceGetAttribute(&s->cus, hipDeviceAttributeMultiprocessorCount, s->device);
        e != hipSuccess || s->cus < 1) {
        delete s;
        return hip_fail(e == hipSuccess ? hipErrorInvalidDevice : e, "compute unit count");
    }
    if (stream) {
        s->stream = (hipStream_t)stream;
        s->own_stream = false;
    } else {
        hipError_t e = hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking);
        if (e != hipSuccess) { delete s; return hip_fail(e, "hipStreamCreate"); }
        s->own_stream = true;
    }
    s->variant = default_variant(s->p);
    choose_geometry(s, 0);
    const size_t bytes = state_bytes(s->p);
    s->red_blocks = reduce_blocks(s->n);
    s->multi = plan_multi(s->p, s->cus);
    hipError_t e = allocate(s);
    if (e != hipSuccess) { lbm_status r = hip_fail(e, "hipMalloc(state)"); lbm_free(s); return r; }
    s->aux.err = s->d_err;
    e = hipMemsetAsync(s->d_err, 0, sizeof(int) * 16, s->stream);
    // zero padding so checkpoints are deterministic
    if (e == hipSuccess) e = hipMemsetAsync(s->buf[0], 0, bytes, s->stream);
    if (e != hipSuccess) { lbm_status r = hip_fail(e, "clear state"); lbm_free(s); return r; }
    st = upload_table(s);
    if (st != LBM_OK) { lbm_free(s); return st; }
    if (s->phys.eos) {
        // the simulation keeps its own device copy of the caller's tables
        const size_t np = (size_t)params->eos_nrho * params->eos_nT, nc = 2 * (size_t)params->eos_nT;
        e = hipMalloc((void**)&s->d_eos_p, sizeof(double) * np);
        if (e == hipSuccess) e = hipMalloc((void**)&s->d_eos_coex, sizeof(double) * nc);
        if (e == hipSuccess) e = hipMemcpy(s->d_eos_p, params->eos_p, sizeof(double) * np, hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(s->d_eos_coex, params->eos_coex, sizeof(double) * nc, hipMemcpyHostToDevice);
        if (e != hipSuccess) { lbm_status r = hip_fail(e, "EOS table upload"); lbm_free(s); return r; }
    }
    s->aux.eos_p = s->d_eos_p;
    s->aux.eos_coex = s->d_eos_coex;
    s->aux.partials = nullptr;   // set by the steps that form the totals
    // the caller's table pointers are not kept
    s->p.eos_p = nullptr;
    s->p.eos_coex = nullptr;

    // the fields (40 B per node) pass through the second buffer (72 B per node at least)
    double* d_fields = static_cast<double*>(s->buf[1]);
    e = hipMemcpyAsync(d_fields, rho0, sizeof(double) * s->n, hipMemcpyHostToDevice, s->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(d_fields + s->n, u0, sizeof(double) * 3 * s->n, hipMemcpyHostToDevice, s->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(d_fields + 4 * s->n, T0, sizeof(double) * s->n, hipMemcpyHostToDevice, s->stream);
    if (e == hipSuccess)
        e = launch_init(s->p.lattice, s->p.storage_bytes, s->buf[0], d_fields, d_fields + s->n, d_fields + 4 * s->n,
                        s->p.nx, s->p.ny, s->p.nz, s->geom.pitch, s->plane, s->p.c_v, s->p.walls, s->stream);
    if (e == hipSuccess) e = hipMemsetAsync(s->buf[1], 0, bytes, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) { lbm_status r = hip_fail(e, "initial state"); lbm_free(s); return r; }
    s->cur = 0;
    s->step = 0;
    *out = s;
    return LBM_OK;
}

lbm_status lbm_step_async(lbm_sim* s, int nsteps)
{
    clear_error();
    if (!s || nsteps < 0) { set_error("bad simulation handle or step count"); return LBM_EINVAL; }
    if (lbm_status sd = use_device(s->device); sd != LBM_OK) return sd;
    return enqueue_steps(s, nsteps);
}

lbm_status lbm_check(lbm_sim* s)
{
    clear_error();
    if (!s) { set_error("simulation is NULL"); return LBM_EINVAL; }
    if (lbm_status sd = use_device(s->device); sd != LBM_OK) return sd;
    return read_error_word(s);
}

lbm_status lbm_step(lbm_sim* s, int nsteps)
{
    lbm_status st = lbm_step_async(s, nsteps);
    if (st != LBM_OK) return st;
    return read_error_word(s);
}

long long lbm_step_count(const lbm_sim* s) { return s ? s->step : -1; }

lbm_status lbm_set_launch(lbm_sim* s, int variant, int chunk)
{
    clear_error();
    if (!s) { set_error("simulation is NULL"); return LBM_EINVAL; }
    if (variant < 0 || variant >= step_variants(s->p.lattice, s->p.storage_bytes) || chunk < 0) {
        set_error("launch variant %d / chunk %d not available for this lattice and storage", variant, chunk);
        return LBM_EINVAL;
    }
    s->variant = variant;
    s->split = false;   // a launch of the fused step was asked for
    s->launch_set = true;
    choose_geometry(s, chunk);
    return LBM_OK;
}

lbm_status lbm_launch_plan(const lbm_params* p, int cus, int info[4])
{
    clear_error();
    if (!p || !info || cus < 1) { set_error("NULL argument or compute-unit count below 1"); return LBM_EINVAL; }
    if (!((p->lattice == 9 && p->nz == 1) || p->lattice == 19) ||
        (p->storage_bytes != 4 && p->storage_bytes != 8) || p->nx < 1 || p->ny < 1 || p->nz < 1) {
        set_error("lattice, storage or shape not supported");
        return LBM_EINVAL;
    }
    int tx, ty;
    const StepGeom g = plan_geometry(*p, default_variant(*p), 0, cus, tx, ty);
    info[0] = tx;
    info[1] = ty;
    info[2] = g.chunk;
    info[3] = g.ntx * g.nty * g.nchunks;
    return LBM_OK;
}

lbm_status lbm_launch_info(const lbm_sim* s, int info[4])
{
    if (!s || !info) { set_error("NULL argument"); return LBM_EINVAL; }
    info[0] = s->tile_x;
    info[1] = s->tile_y;
    info[2] = s->geom.chunk;
    info[3] = s->geom.ntx * s->geom.nty * s->geom.nchunks;
    return LBM_OK;
}

// Scratch of the moment kernels, rho and Phi: that of the two-launch step where there is one (36 bytes per node
// at least, and nothing in it outlives a step), else an allocation that the simulation keeps.
static lbm_status moment_scratch(lbm_sim* s, double** scratch)
{
    if (s->d_split) { *scratch = static_cast<double*>(s->d_split); return LBM_OK; }
    if (!s->d_scratch) {
        hipError_t e = hipMalloc((void**)&s->d_scratch, sizeof(double) * 2 * s->n);
        if (e != hipSuccess) return hip_fail(e, "hipMalloc(moment scratch)");
    }
    *scratch = s->d_scratch;
    return LBM_OK;
}

lbm_status lbm_moments_device(lbm_sim* s, double* rho, double* u_star, double* E, double* T)
{
    clear_error();
    if (!s) { set_error("simulation is NULL"); return LBM_EINVAL; }
    if (lbm_status sd = use_device(s->device); sd != LBM_OK) return sd;
    double* scratch = nullptr;
    lbm_status st = moment_scratch(s, &scratch);
    if (st != LBM_OK) return st;
    hipError_t e = launch_moments(s->p.lattice, s->p.storage_bytes, s->buf[s->cur], scratch, s->p.nx,
                                  s->p.ny, s->p.nz, s->geom.pitch, s->plane, s->phys, s->aux.eos_p, s->d_err, rho,
                                  u_star, E, T, s->stream);
    if (e != hipSuccess) return hip_fail(e, "moments launch");
    return LBM_OK;
}

lbm_status lbm_moments(lbm_sim* s, double* rho, double* u_star, double* E, double* T)
{
    clear_error();
    if (!s) { set_error("simulation is NULL"); return LBM_EINVAL; }
    if (lbm_status sd = use_device(s->device); sd != LBM_OK) return sd;
    const long long n = s->n;
    // scratch and fields (64 B per node) pass through the population buffer that the next step writes (72 B per
    // node at least); its padding is cleared again for that
    double* scr = static_cast<double*>(s->buf[1 - s->cur]);
    double *d_rho = scr + 2 * n, *d_us = scr + 3 * n, *d_E = scr + 6 * n, *d_T = scr + 7 * n;
    hipError_t e = launch_moments(s->p.lattice, s->p.storage_bytes, s->buf[s->cur], scr, s->p.nx, s->p.ny,
                                  s->p.nz, s->geom.pitch, s->plane, s->phys, s->aux.eos_p, s->d_err, rho ? d_rho : nullptr,
                                  u_star ? d_us : nullptr, E ? d_E : nullptr, T ? d_T : nullptr, s->stream);
    if (e == hipSuccess && rho) e = hipMemcpyAsync(rho, d_rho, sizeof(double) * n, hipMemcpyDeviceToHost, s->stream);
    if (e == hipSuccess && u_star) e = hipMemcpyAsync(u_star, d_us, sizeof(double) * 3 * n, hipMemcpyDeviceToHost, s->stream);
    if (e == hipSuccess && E) e = hipMemcpyAsync(E, d_E, sizeof(double) * n, hipMemcpyDeviceToHost, s->stream);
    if (e == hipSuccess && T) e = hipMemcpyAsync(T, d_T, sizeof(double) * n, hipMemcpyDeviceToHost, s->stream);
    if (e == hipSuccess) e = hipMemsetAsync(s->buf[1 - s->cur], 0, state_bytes(s->p), s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return hip_fail(e, "moments");
    return read_error_word(s);
}

lbm_status lbm_reduce(lbm_sim* s, double out[5])
{
    clear_error();
    if (!s || !out) { set_error("NULL argument"); return LBM_EINVAL; }
    if (lbm_status sd = use_device(s->device); sd != LBM_OK) return sd;
    double* d_out = s->d_partials + 5 * s->red_blocks;
    // the padding of the rows is zero (cleared at init, never written by the step)
    hipError_t e = launch_reduce(s->p.lattice, s->p.storage_bytes, s->buf[s->cur], plane_elements(s->p), s->plane,
                                 s->d_partials, s->red_blocks, d_out, s->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(out, d_out, sizeof(double) * 5, hipMemcpyDeviceToHost, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return hip_fail(e, "reduction");
    return LBM_OK;
}

lbm_status lbm_step_reduce(lbm_sim* s, int nsteps, double out[5])
{
    clear_error();
    if (!s || !out || nsteps < 1) {
        set_error("bad simulation handle, NULL output or step count below 1");
        return LBM_EINVAL;
    }
    if (lbm_status sd = use_device(s->device); sd != LBM_OK) return sd;
    lbm_status st = enqueue_steps(s, nsteps - 1);
    if (st != LBM_OK) return st;
    // the last step's partial totals (5 per workgroup) and the totals, grown on demand
    int tx, ty, per_cu;
    step_tile(s->p.lattice, s->p.storage_bytes, s->variant, tx, ty, per_cu);
    const bool split = !s->launch_set &&
                       split_totals(s->p, s->geom, split_geometry(s->p, s->cus), s->cus, per_cu) && ensure_split(s);
    const StepGeom& geom = split ? s->split_geom : s->geom;
    const long long wg = step_workgroups(geom);
    if (5 * wg + 8 > s->step_partials_len) {
        if (s->d_step_partials) {
            hipError_t e = hipFree(s->d_step_partials);
            s->d_step_partials = nullptr;
            s->step_partials_len = 0;
            if (e != hipSuccess) return hip_fail(e, "hipFree(step partials)");
        }
        hipError_t e = hipMalloc((void**)&s->d_step_partials, sizeof(double) * (5 * wg + 8));
        if (e != hipSuccess) return hip_fail(e, "hipMalloc(step partials)");
        s->step_partials_len = 5 * wg + 8;
    }
    double* d_out = s->d_step_partials + 5 * wg;
    StepAux aux = s->aux;
    aux.partials = s->d_step_partials;
    hipError_t e;
    if (split) {
        e = launch_split_moments(s->p.storage_bytes, s->buf[s->cur], s->d_split, geom, s->phys, aux, s->stream);
        if (e == hipSuccess)
            e = launch_split_collide_totals(s->p.storage_bytes, s->buf[s->cur], s->buf[1 - s->cur], s->d_split,
                                            geom, s->phys, aux, d_out, s->stream);
    } else {
        e = launch_step_totals(s->p.lattice, s->p.storage_bytes, s->variant, s->buf[s->cur],
                               s->buf[1 - s->cur], geom, s->phys, aux, d_out, s->stream);
    }
    if (e == hipErrorNotSupported) {
        // a launch variant without the fused form: the plain step, then the separate reduction
        st = enqueue_steps(s, 1);
        if (st != LBM_OK) return st;
        e = launch_reduce(s->p.lattice, s->p.storage_bytes, s->buf[s->cur], plane_elements(s->p), s->plane,
                          s->d_partials, s->red_blocks, d_out, s->stream);
        if (e != hipSuccess) return hip_fail(e, "reduction");
    } else if (e != hipSuccess) {
        return hip_fail(e, "step launch");
    } else {
        s->cur ^= 1;
        s->step += 1;
    }
    e = hipMemcpyAsync(out, d_out, sizeof(double) * 5, hipMemcpyDeviceToHost, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return hip_fail(e, "reading the totals");
    return read_error_word(s);
}

struct CheckpointHeader {
    char magic[8];
    int lattice, nx, ny, nz, storage_bytes, pitch;   // pitch: x row pitch of the layout, in elements
    long long step;
    long long bytes;
};

lbm_status lbm_checkpoint(lbm_sim* s, void* host_buf, size_t cap, size_t* used)
{
    clear_error();
    if (!s || !used) { set_error("NULL argument"); return LBM_EINVAL; }
    const size_t bytes = state_bytes(s->p);
    *used = sizeof(CheckpointHeader) + bytes;
    if (!host_buf) return LBM_OK;
    if (cap < *used) { set_error("checkpoint buffer too small (%zu < %zu)", cap, *used); return LBM_EINVAL; }
    if (lbm_status sd = use_device(s->device); sd != LBM_OK) return sd;
    CheckpointHeader h;
    memset(&h, 0, sizeof(h));
    memcpy(h.magic, "LBMCKPT2", 8);
    h.lattice = s->p.lattice; h.nx = s->p.nx; h.ny = s->p.ny; h.nz = s->p.nz;
    h.storage_bytes = s->p.storage_bytes; h.pitch = s->geom.pitch; h.step = s->step; h.bytes = (long long)bytes;
    memcpy(host_buf, &h, sizeof(h));
    hipError_t e = hipMemcpyAsync((char*)host_buf + sizeof(h), s->buf[s->cur], bytes, hipMemcpyDeviceToHost, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return hip_fail(e, "checkpoint copy");
    return LBM_OK;
}

lbm_status lbm_restore(lbm_sim* s, const void* host_buf, size_t len)
{
    clear_error();
    if (!s || !host_buf) { set_error("NULL argument"); return LBM_EINVAL; }
    CheckpointHeader h;
    if (len < sizeof(h)) { set_error("checkpoint too short"); return LBM_EINVAL; }
    memcpy(&h, host_buf, sizeof(h));
    const size_t bytes = state_bytes(s->p);
    if (memcmp(h.magic, "LBMCKPT2", 8) != 0 || h.lattice != s->p.lattice || h.nx != s->p.nx || h.ny != s->p.ny ||
        h.nz != s->p.nz || h.storage_bytes != s->p.storage_bytes || h.pitch != s->geom.pitch ||
        h.bytes != (long long)bytes ||
        len < sizeof(h) + bytes) {
        set_error("checkpoint does not match this simulation's lattice, shape or storage");
        return LBM_EINVAL;
    }
    if (lbm_status sd = use_device(s->device); sd != LBM_OK) return sd;
    hipError_t e = hipMemcpyAsync(s->buf[s->cur], (const char*)host_buf + sizeof(h), bytes, hipMemcpyHostToDevice, s->stream);
    if (e == hipSuccess) e = hipMemsetAsync(s->d_err, 0, sizeof(int), s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) return hip_fail(e, "restore copy");
    s->step = h.step;
    return LBM_OK;
}

lbm_status lbm_free(lbm_sim* s)
{
    if (!s) return LBM_OK;
    // release everything even if the device reports an error: nothing here can be retried
    (void)hipSetDevice(s->device);
    if (s->stream) (void)hipStreamSynchronize(s->stream);
    if (s->memory) (void)hipFree(s->memory);
    if (s->d_step_partials) (void)hipFree(s->d_step_partials);
    if (s->d_scratch) (void)hipFree(s->d_scratch);
    if (s->d_split && s->own_split) (void)hipFree(s->d_split);
    if (s->d_eos_p) (void)hipFree(s->d_eos_p);
    if (s->d_eos_coex) (void)hipFree(s->d_eos_coex);
    if (s->own_stream && s->stream) (void)hipStreamDestroy(s->stream);
    delete s;
    return LBM_OK;
}

}  // extern "C"
