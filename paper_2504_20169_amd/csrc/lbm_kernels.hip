// HIP kernels (gfx950, wave64) for the thermal LBM with PML and open boundaries, compiled once
// per velocity stencil: LBM_Q = 37 (default; this file), 17 (lbm_kernels_d2q17.hip) or 9
// (lbm_kernels_d2q9.hip), each instance in its own namespace (k37, k17, k9) with its stencil's
// constants in scope.
//
// Every kernel takes an array of run descriptors, so one launch advances one run or a batch of
// uneven runs.  Per step:
//   k_target       (runs with the appendix's PML moments or a CBC (A) side) float64
//                  characteristic targets of the ring
//   k_phase_a      ring blocks: float64 characteristic fill of the 3-deep ring of
//                  characteristic-boundary nodes into G (eqs. PNR / thermal_LODI_macro_evo);
//                  then for the PML Q-region nodes: pull (ring: G) + moments,
//                  Q^{n+1} = Q^n + (fhat^n + fhat^{n+1})/2                      (eq. PMLQ)
//   k_frame        frame nodes (boundary layers, PML, moment strips): pull (ring nodes: G) +
//                  ZG copy, moments, U^{n+1} strip write, BGK + Omega^PML
//                                                             (eqs. PMLCOLL, zg-bc)
//   k_bulk         interior nodes: branch-free pull + moments + BGK             (eq. lbe)
// phase A and the bulk tiles may go out as one grid (k_phase_a_bulk), and a small set's boundary
// launches split a node's populations over four waves (k_frame_split, k_small_step).  Large runs
// take two steps per pass over their interior:
//   k_core         interior nodes: both steps, the level between in LDS
//   k_phase_a, k_frame<STEP_FIRST>    the boundary's first step, into the bands of the level between
//   k_phase_a, k_frame<STEP_SECOND>   its second step, from the bands
//   k_advance      end of a batch of steps: advance the step counters and buffer parities
//                  (the step kernels of sub-step k of a batch use parity par + k)
// The ring blocks come first in their launches (their float64 chains are the longest) and are
// block-uniform, so they never share a wave with frame nodes.  (A separate ring launch lowers
// phase A's registers but measured slower: the ring's latency then adds instead of overlapping.)
// The collision is a per-node projection streaming 2 x q values
// through HBM: no MFMA.  Pulls are coalesced row segments shifted by e_i (each source value is
// read exactly once); descriptors are read through the constant address space (scalar
// loads) and populations through global pointers with one 32-bit byte offset per lane.
//
// Arithmetic is in deviation form: the stored populations are d_i = f_i - fbar_i with
// fbar = feq(rho0, u0, T0), and the equilibrium deviation feq(U) - fbar is evaluated from
// differences of its Hermite coefficients, so float32 storage and arithmetic keep their
// relative precision on the (small) deviations.  With theta = T - 1, a = u.xi, s = |xi|^2,
// b = |u|^2, the fourth-order equilibrium of D2Q37 (eq. feq-4 with the (c^2 - 6) reading) is
//   feq_i = w_i rho H(a, s),
//   H = E0(s) + E2(s) a^2 + a^4/24 + a (O1(s) + a^2/6),
//   E0 = k0 + k2s s + theta^2 s^2/8,  E2 = k2a + theta s/4,  O1 = k1 + theta s/2,
//   k0 = 1 - b/2 - theta + b^2/8 + theta b + theta^2,  k1 = 1 - b/2 - 2 theta,
//   k2a = 1/2 - b/4 - 3 theta/2,  k2s = theta/2 - theta b/4 - theta^2,
// and the third-order equilibrium of D2Q17 (eq. feq-3) drops the fourth-order Hermite term:
//   H = E0(s) + a^2/2 + a (O1(s) + a^2/6),  E0 = k0 + theta s/2,  k0 = 1 - b/2 - theta,
// with O1 and k1 as above; feq(U) - fbar = w (drho H0 + rho dH) with dH = H(U) - H(U0)
// expanded in products of deviations.
// FP64 storage evaluates the same deviation as a polynomial in e (EqPoly).
#include <type_traits>
#include <utility>

#include <hip/hip_ext.h>

#include "lbm_internal.h"

#define GLOBAL __attribute__((address_space(1)))
#define CONSTANT __attribute__((address_space(4)))

#ifndef LBM_Q
#define LBM_Q 37
#endif
#if LBM_Q == 37
#define LBM_LATTICE d2q37
#define LBM_INFO LATTICE_D2Q37
#define LBM_KSET k37
#elif LBM_Q == 17
#define LBM_LATTICE d2q17
#define LBM_INFO LATTICE_D2Q17
#define LBM_KSET k17
#elif LBM_Q == 9
#define LBM_LATTICE d2q9
#define LBM_INFO LATTICE_D2Q9
#define LBM_KSET k9
#else
#error "LBM_Q must be 37, 17 or 9"
#endif

namespace lbm {
namespace LBM_KSET {

using namespace ::lbm::LBM_LATTICE;
constexpr int REACH = reach_of(LBM_INFO);   // longest displacement along an axis
using CRun = const CONSTANT RunDev;

// Index guard of the bounds-checked debug build (compiled with LBM_BOUNDS): an element index i
// outside [0, n) marks the run's descriptor (a vector atomic) and is replaced by 0, so the access
// stays inside its buffer and lbm_check reports the run.  The normal build uses i unchanged.
#ifdef LBM_BOUNDS
__device__ __forceinline__ long long guard(CRun &R, long long i, long long n) {
    if ((unsigned long long)i < (unsigned long long)n) return i;
    GLOBAL unsigned *flag = (GLOBAL unsigned *)(uintptr_t)&R.oob;   // the descriptor, written as global memory
    __hip_atomic_fetch_or(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return 0;
}
#define LBM_GUARD(R, i, n) guard((R), (i), (n))
#define LBM_CHECK(R, i, n) (void)guard((R), (i), (n))   // of an access that cannot leave its buffer
// element `off` bytes past base, inside buffer buf of n elements
#define LBM_AT(R, base, off, buf, n) \
    ((buf) + guard((R), ((base) - (buf)) + (long long)((off) / sizeof(*(buf))), (n)))
// element p of buffer buf of n elements
#define LBM_IN(R, p, buf, n) ((buf) + guard((R), (p) - (buf), (n)))
#else
#define LBM_GUARD(R, i, n) (i)
#define LBM_IN(R, p, buf, n) (p)
#define LBM_CHECK(R, i, n) ((void)0)
#define LBM_AT(R, base, off, buf, n) at((base), (off))
#endif

// ------------------------------------------------------------------------------------------
// helpers
// ------------------------------------------------------------------------------------------
template <int I, int N, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

template <class S> struct Traits;
template <> struct Traits<double> { using C = double; };
template <> struct Traits<float> { using C = float; };
template <> struct Traits<_Float16> { using C = float; };

// element at byte offset `off` from a uniform base
template <class T>
__device__ __forceinline__ const GLOBAL T *at(const GLOBAL T *base, unsigned off) {
    return (const GLOBAL T *)((const GLOBAL char *)base + off);
}
template <class T>
__device__ __forceinline__ GLOBAL T *at(GLOBAL T *base, unsigned off) {
    return (GLOBAL T *)((GLOBAL char *)base + off);
}

__device__ __forceinline__ double cvt_in(double v, double) { return v; }
__device__ __forceinline__ float cvt_in(float v, float) { return v; }
__device__ __forceinline__ float cvt_in(_Float16 v, float inv) { return (float)v * inv; }
__device__ __forceinline__ double cvt_out(double v, double, double *) { return v; }
__device__ __forceinline__ float cvt_out(float v, float, float *) { return v; }
__device__ __forceinline__ _Float16 cvt_out(float v, float sc, _Float16 *) { return (_Float16)(v * sc); }

// Run constants in the compute type.
template <class C> struct K {
    C omega, rho0, u0x, u0y, th0, b0, r0x, r0y, c2Tb0, scale, inv_scale;
    C xx0, xy0, yy0, k2a0, k10;   // FP64: of the mean state, products of v = r u, and k2a, k1
};

template <class C> __device__ __forceinline__ K<C> load_k(CRun &R) {
    K<C> k;
    if constexpr (std::is_same<C, double>::value) {
        k.omega = R.omega; k.rho0 = R.rho0; k.u0x = R.u0x; k.u0y = R.u0y; k.th0 = R.th0;
        k.b0 = R.b0; k.r0x = R.r0x; k.r0y = R.r0y; k.c2Tb0 = 2.0 * R.T0 + R.b0;
        k.scale = R.scale; k.inv_scale = R.inv_scale;
        k.xx0 = R.xx0; k.xy0 = R.xy0; k.yy0 = R.yy0; k.k2a0 = R.k2a0; k.k10 = R.k10;
    } else {
        k.omega = R.omega_f; k.rho0 = R.rho0_f; k.u0x = R.u0x_f; k.u0y = R.u0y_f; k.th0 = R.th0_f;
        k.b0 = R.b0_f; k.r0x = R.r0x_f; k.r0y = R.r0y_f; k.c2Tb0 = 2.0f * R.T0_f + R.b0_f;
        k.scale = R.scale_f; k.inv_scale = R.inv_scale_f;
        k.xx0 = k.xy0 = k.yy0 = k.k2a0 = k.k10 = C(0);   // (not read)
    }
    return k;
}

template <class C> __device__ __forceinline__ C cH0e(CRun &R, int p) {
    if constexpr (std::is_same<C, double>::value) return R.H0e[p]; else return R.H0e_f[p];
}
template <class C> __device__ __forceinline__ C cH0o(CRun &R, int p) {
    if constexpr (std::is_same<C, double>::value) return R.H0o[p]; else return R.H0o_f[p];
}
template <class C> __device__ __forceinline__ C cE2_0(CRun &R, int s) {
    if constexpr (std::is_same<C, double>::value) return R.E2_0[s]; else return R.E2_0_f[s];
}
template <class C> __device__ __forceinline__ C cO1_0(CRun &R, int s) {
    if constexpr (std::is_same<C, double>::value) return R.O1_0[s]; else return R.O1_0_f[s];
}
template <class C> __device__ __forceinline__ C cH0rest(CRun &R) {
    if constexpr (std::is_same<C, double>::value) return R.H0rest; else return R.H0rest_f;
}

// Blocks of one launch are dealt round-robin to the 8 XCDs; remap so that consecutive tiles
// (neighbours sharing cache lines at their edges) run on the same XCD and its L2.
__device__ __forceinline__ int xcd_swizzle(int b, int n) {
    int per = n >> 3, rem = n & 7, xcd = b & 7, loc = b >> 3;
    return xcd < rem ? xcd * (per + 1) + loc : rem * (per + 1) + (xcd - rem) * per + loc;
}

__device__ __forceinline__ int find_run(const int *prefix, int nruns, int b) {
    const CONSTANT int *p = (const CONSTANT int *)prefix;
    int lo = 0, hi = nruns;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (p[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ CRun &run_of(RunDev *const *runs, int j) {
    return *(CRun *)(((RunDev *const CONSTANT *)runs)[j]);
}

// Steps are launched in batches.  A sub-step of a batch sees the run `steps` time steps past its
// descriptor's step counter and works only while that stays below the run's limit; the population
// buffers have then changed roles `flips` times (once per single step, once per two-step pass), so
// its source buffer is par + flips.  k_advance moves the counters at the end of the batch.  Returns
// the population parity, or -1 for a run that is no longer active at the sub-step.
__device__ __forceinline__ int sub_par(CRun &R, Sub k) {
    return R.step + k.steps < R.limit ? ((R.par + k.flips) & 1) : -1;
}
// The moment strips alternate every time step: U[u] holds the level the sub-step starts from.
__device__ __forceinline__ int u_par(CRun &R, Sub k) { return (int)(R.step + k.steps) & 1; }

// Strip numbering of a frame of depths (dxm, dxp, dym, dyp): bottom strip, top strip, left
// strip, right strip.
__device__ __forceinline__ void strip_xy(int Nx, int Ny, int dxm, int dxp, int dym, int dyp, int t,
                                         int &x, int &y) {
    int Fb = dym * Nx, Ft = dyp * Nx, H = Ny - dym - dyp, Fl = H * dxm;
    if (t < Fb) { y = t / Nx; x = t - y * Nx; }
    else if (t < Fb + Ft) { t -= Fb; int r = t / Nx; y = Ny - dyp + r; x = t - r * Nx; }
    else if (t < Fb + Ft + Fl) { t -= Fb + Ft; int r = t / dxm; y = dym + r; x = t - r * dxm; }
    else { t -= Fb + Ft + Fl; int r = t / dxp; y = dym + r; x = Nx - dxp + (t - r * dxp); }
}

__device__ __forceinline__ void ring_xy(CRun &R, int t, int &x, int &y) {
    strip_xy(R.Nx, R.Ny, R.rxm, R.rxp, R.rym, R.ryp, t, x, y);
    x = (int)LBM_GUARD(R, x, R.Nx);
    y = (int)LBM_GUARD(R, y, R.Ny);
}
// Node a of the frame off the ring (annulus numbering, 0 <= a < ann_n); its frame index is
// ann0 + a.
__device__ __forceinline__ void ann_xy(CRun &R, int a, int &x, int &y) {
    strip_xy(R.Nx - R.rxm - R.rxp, R.Ny - R.rym - R.ryp, R.axm, R.axp, R.aym, R.ayp, a, x, y);
    x = (int)LBM_GUARD(R, x + R.rxm, R.Nx);
    y = (int)LBM_GUARD(R, y + R.rym, R.Ny);
}
// Node of frame index t (ring nodes first, then the annulus from ann0; t not in the gap).
__device__ __forceinline__ void frame_xy(CRun &R, int t, int &x, int &y) {
    if (t < R.ring_n) ring_xy(R, t, x, y);
    else ann_xy(R, t - R.ann0, x, y);
}

// Inverse of strip_xy: strip index of (x, y), or -1 outside the strips.
__device__ __forceinline__ int strip_idx(int Nx, int Ny, int dxm, int dxp, int dym, int dyp, int x, int y) {
    if (y < dym) return y * Nx + x;
    if (y >= Ny - dyp) return (dym + y - (Ny - dyp)) * Nx + x;
    int H = Ny - dym - dyp, base = (dym + dyp) * Nx, yy = y - dym;
    if (x < dxm) return base + yy * dxm + x;
    if (x >= Nx - dxp) return base + H * dxm + yy * dxp + (x - (Nx - dxp));
    return -1;
}

__device__ __forceinline__ int ridx(CRun &R, int x, int y) {
    return strip_idx(R.Nx, R.Ny, R.rxm, R.rxp, R.rym, R.ryp, x, y);
}
// Frame index of (x, y) on the grid, or -1 for a node of the fast rectangle.
__device__ __forceinline__ int fidx(CRun &R, int x, int y) {
    if (R.ring_n > 0) {   // (uniform) without a ring the annulus is the whole frame
        const int r = ridx(R, x, y);
        if (r >= 0) return r;
    }
    const int a = strip_idx(R.Nx - R.rxm - R.rxp, R.Ny - R.rym - R.ryp, R.axm, R.axp, R.aym, R.ayp,
                            x - R.rxm, y - R.rym);
    return a < 0 ? -1 : R.ann0 + a;
}

__device__ __forceinline__ bool in_q(CRun &R, int x, int y) {
    return (R.Wxm > 0 && x < R.qd) || (R.Wxp > 0 && x >= R.Nx - R.qd) ||
           (R.Wym > 0 && y < R.qd) || (R.Wyp > 0 && y >= R.Ny - R.qd);
}

// Characteristic-boundary node: within the outer 3 layers of an NRBC side.
__device__ __forceinline__ bool in_ring(CRun &R, int x, int y) {
    return (R.rxm > 0 && x < 3) || (R.rxp > 0 && x >= R.Nx - 3) ||
           (R.rym > 0 && y < 3) || (R.ryp > 0 && y >= R.Ny - 3);
}

// eq. PML_ramp on the Chebyshev ring level.
__device__ __forceinline__ double sigma_at(CRun &R, int x, int y) {
    int lx = x < R.Wxm ? R.Wxm - x : (x >= R.Nx - R.Wxp ? x - (R.Nx - R.Wxp) + 1 : 0);
    int ly = y < R.Wym ? R.Wym - y : (y >= R.Ny - R.Wyp ? y - (R.Ny - R.Wyp) + 1 : 0);
    int l = lx > ly ? lx : ly;
    return l > 0 ? R.sigma_max * (double)(l * l) * R.inv_W2 : 0.0;
}

// ------------------------------------------------------------------------------------------
// moments (eq. macro) in deviation form
// ------------------------------------------------------------------------------------------
template <class C> struct Mom { C drho, dux, duy, dT, rho; };

// Moment sums of populations taken pair by pair (pairs in order): s = sum g, j = sum e g,
// e2 = sum |e|^2 g, then the primitive deviations from them.
template <class C> struct MomAcc { C s, jx, jy, e2; };

template <class C>
__device__ __forceinline__ MomAcc<C> mom_begin(C g0) { return MomAcc<C>{g0, C(0), C(0), C(0)}; }

template <int p, class C>
__device__ __forceinline__ void mom_pair(MomAcc<C> &m, C a, C b) {
    C sp = a + b, dp = a - b;
    m.s += sp;
    if constexpr (PEX[p] == 1) m.jx += dp;
    else if constexpr (PEX[p] == -1) m.jx -= dp;
    else if constexpr (PEX[p] != 0) m.jx += C(PEX[p]) * dp;
    if constexpr (PEY[p] == 1) m.jy += dp;
    else if constexpr (PEY[p] == -1) m.jy -= dp;
    else if constexpr (PEY[p] != 0) m.jy += C(PEY[p]) * dp;
    if constexpr (SHELL_E2[PSH[p]] == 1) m.e2 += sp;
    else m.e2 += C(SHELL_E2[PSH[p]]) * sp;
}

template <class C>
__device__ __forceinline__ Mom<C> mom_end(const MomAcc<C> &a, const K<C> &k) {
    const C s = a.s;
    Mom<C> m;
    m.drho = s;
    m.rho = k.rho0 + s;
    C inv = C(1) / m.rho;
    C Jx = C(LAT_R) * a.jx, Jy = C(LAT_R) * a.jy, E = C(LAT_R2) * a.e2;
    m.dux = (Jx - s * k.u0x) * inv;
    m.duy = (Jy - s * k.u0y) * inv;
    C t = E - s * k.c2Tb0 - C(2) * m.rho * (k.u0x * m.dux + k.u0y * m.duy) -
          m.rho * (m.dux * m.dux + m.duy * m.duy);
    m.dT = C(0.5) * t * inv;
    return m;
}

template <class C>
__device__ __forceinline__ Mom<C> moments(const C (&g)[NQ], const K<C> &k) {
    MomAcc<C> a = mom_begin<C>(g[0]);
    static_for<0, NPAIR>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        mom_pair<p>(a, g[1 + 2 * p], g[2 + 2 * p]);
    });
    return mom_end<C>(a, k);
}

// Moments of populations read by get(i) in groups of PC pairs, each group's reads issued
// together and the groups kept apart, so only one group is held in registers; the same sums
// in the same order as moments().
template <int PC, class C, class Get>
__device__ __forceinline__ Mom<C> moments_streamed(Get &&get, const K<C> &k) {
    MomAcc<C> a = mom_begin<C>(get(std::integral_constant<int, 0>{}));
    static_for<0, (NPAIR + PC - 1) / PC>([&](auto cc) {
        constexpr int P0 = decltype(cc)::value * PC;
        constexpr int P1 = P0 + PC < NPAIR ? P0 + PC : NPAIR;
        C v[2 * (P1 - P0)];
        static_for<0, 2 * (P1 - P0)>([&](auto lc) {
            constexpr int l = decltype(lc)::value;
            v[l] = get(std::integral_constant<int, 1 + 2 * P0 + l>{});
        });
        static_for<P0, P1>([&](auto pc) {
            constexpr int p = decltype(pc)::value;
            mom_pair<p>(a, v[2 * (p - P0)], v[2 * (p - P0) + 1]);
        });
        __builtin_amdgcn_sched_barrier(0);
    });
    return mom_end<C>(a, k);
}

// ------------------------------------------------------------------------------------------
// equilibrium deviation feq(U) - fbar
// ------------------------------------------------------------------------------------------
template <class C> struct Eq {
    C drho, rho, Rdux, Rduy, dT, dk0, dk1, dk2a, dk2s, dth2;
    C dE0, dE2, dO1;   // current shell
};

template <class C>
__device__ __forceinline__ Eq<C> eq_coef(C drho, C dux, C duy, C dT, const K<C> &k) {
    Eq<C> q;
    q.drho = drho;
    q.rho = k.rho0 + drho;
    q.Rdux = C(LAT_R) * dux;
    q.Rduy = C(LAT_R) * duy;
    q.dT = dT;
    C db = dux * (C(2) * k.u0x + dux) + duy * (C(2) * k.u0y + duy);
    if constexpr (ORDER == 4) {
        C ux = k.u0x + dux, uy = k.u0y + duy, th = k.th0 + dT;
        C b = ux * ux + uy * uy;
        C dth2 = dT * (th + k.th0);
        C dthb = dT * b + k.th0 * db;
        C db2 = db * (b + k.b0);
        q.dk0 = -C(0.5) * db - dT + C(0.125) * db2 + dthb + dth2;
        q.dk2a = -C(0.25) * db - C(1.5) * dT;
        q.dk2s = C(0.5) * dT - C(0.25) * dthb - dth2;
        q.dth2 = dth2;
    } else {   // third and second order: k0 = 1 - b/2 - theta, k2a = 1/2, k2s = theta/2
        q.dk0 = -C(0.5) * db - dT;
        q.dk2a = C(0);
        q.dk2s = C(0.5) * dT;
        q.dth2 = C(0);
    }
    // odd part: O1 = k1 + theta c^2/2 with k1 = 1 - b/2 - 2 theta (fourth and third order);
    // the second-order equilibrium's odd part is a alone (O1 = 1)
    if constexpr (ORDER >= 3) q.dk1 = -C(0.5) * db - C(2) * dT;
    else q.dk1 = C(0);
    q.dE0 = q.dE2 = q.dO1 = C(0);
    return q;
}

template <class C>
__device__ __forceinline__ C feq_rest(const Eq<C> &q, CRun &R) {
    return C(SHELL_W[0]) * (q.drho * cH0rest<C>(R) + q.rho * q.dk0);
}

// Shell coefficient deviations (computed once per shell).
template <class C, int sh>
__device__ __forceinline__ void eq_shell(Eq<C> &q) {
    constexpr double sv = LAT_R2 * SHELL_E2[sh];
    if constexpr (ORDER == 4) {
        q.dE0 = q.dk0 + q.dk2s * C(sv) + q.dth2 * C(0.125 * sv * sv);
        q.dE2 = q.dk2a + q.dT * C(0.25 * sv);
    } else {
        q.dE0 = q.dk0 + q.dk2s * C(sv);
        q.dE2 = C(0);
    }
    if constexpr (ORDER >= 3) q.dO1 = q.dk1 + q.dT * C(0.5 * sv);
    else q.dO1 = C(0);
}

// feq - fbar of the pair p: (+e_p, -e_p).
template <class C, int p>
__device__ __forceinline__ void eq_pair(const Eq<C> &q, CRun &R, const K<C> &k, C &fp, C &fm) {
    constexpr int sh = PSH[p];
    constexpr int ex = PEX[p], ey = PEY[p];
    C a0, da;
    if constexpr (ey == 0) { a0 = C(ex) * k.r0x; da = C(ex) * q.Rdux; }
    else if constexpr (ex == 0) { a0 = C(ey) * k.r0y; da = C(ey) * q.Rduy; }
    else { a0 = C(ex) * k.r0x + C(ey) * k.r0y; da = C(ex) * q.Rdux + C(ey) * q.Rduy; }
    const C O1_0 = cO1_0<C>(R, sh);
    C a = a0 + da;
    C A2 = a * a, A02 = a0 * a0;
    C dA2 = da * (a + a0);
    C dEv;
    if constexpr (ORDER == 4)
        dEv = q.dE0 + q.dE2 * A2 + cE2_0<C>(R, sh) * dA2 + dA2 * (A2 + A02) * C(1.0 / 24.0);
    else   // E2 = 1/2 for every shell and state
        dEv = q.dE0 + C(0.5) * dA2;
    C dOd;
    if constexpr (ORDER >= 3)
        dOd = q.dO1 * a + O1_0 * da + da * (A2 + a * a0 + A02) * C(1.0 / 6.0);
    else   // eq. feq-2: the odd part is a itself
        dOd = da;
    C Tev = q.drho * cH0e<C>(R, p) + q.rho * dEv;
    C Tod = q.drho * cH0o<C>(R, p) + q.rho * dOd;
    constexpr double w = SHELL_W[sh];
    fp = C(w) * (Tev + Tod);
    fm = C(w) * (Tev - Tod);
}

// Calls emit(i, feq_i - fbar_i) for i = 0..NQ-1 with compile-time i.
template <class C, class F>
__device__ __forceinline__ void for_each_feq(Eq<C> q, CRun &R, const K<C> &k, F &&emit) {
    emit(std::integral_constant<int, 0>{}, feq_rest<C>(q, R));
    static_for<0, NPAIR>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        if constexpr (p == 0 || PSH[p - 1] != PSH[p]) eq_shell<C, PSH[p]>(q);
        C fp, fm;
        eq_pair<C, p>(q, R, k, fp, fm);
        emit(std::integral_constant<int, 1 + 2 * p>{}, fp);
        emit(std::integral_constant<int, 2 + 2 * p>{}, fm);
    });
}

// Two equilibria in one pass: emit(i, feq_a_i - fbar_i, feq_b_i - fbar_i).
template <class C, class F>
__device__ __forceinline__ void for_each_feq2(Eq<C> qa, Eq<C> qb, CRun &R, const K<C> &k, F &&emit) {
    emit(std::integral_constant<int, 0>{}, feq_rest<C>(qa, R), feq_rest<C>(qb, R));
    static_for<0, NPAIR>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        if constexpr (p == 0 || PSH[p - 1] != PSH[p]) {
            eq_shell<C, PSH[p]>(qa);
            eq_shell<C, PSH[p]>(qb);
        }
        C ap, am, bp, bm;
        eq_pair<C, p>(qa, R, k, ap, am);
        eq_pair<C, p>(qb, R, k, bp, bm);
        emit(std::integral_constant<int, 1 + 2 * p>{}, ap, bp);
        emit(std::integral_constant<int, 2 + 2 * p>{}, am, bm);
    });
}

// Pairs [P0, P1) of two equilibria: emit(i, feq_a_i - fbar_i, feq_b_i - fbar_i); the shell
// coefficients carry over in qa and qb from the pairs before P0 (pairs in order), so a sweep in
// groups gives the values of for_each_feq2.
template <int P0, int P1, class C, class F>
__device__ __forceinline__ void feq2_pairs(Eq<C> &qa, Eq<C> &qb, CRun &R, const K<C> &k, F &&emit) {
    static_for<P0, P1>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        if constexpr (p == 0 || PSH[p - 1] != PSH[p]) {
            eq_shell<C, PSH[p]>(qa);
            eq_shell<C, PSH[p]>(qb);
        }
        C ap, am, bp, bm;
        eq_pair<C, p>(qa, R, k, ap, am);
        eq_pair<C, p>(qb, R, k, bp, bm);
        emit(std::integral_constant<int, 1 + 2 * p>{}, ap, bp);
        emit(std::integral_constant<int, 2 + 2 * p>{}, am, bm);
    });
}

// ------------------------------------------------------------------------------------------
// equilibrium of FP64 storage: the same deviation as a polynomial in e
// ------------------------------------------------------------------------------------------
// rho H is a polynomial in the integer components of e whose coefficients depend on the node
// alone, so a node forms the deviations of its coefficients once (D[rho X] = drho X(U0) + rho dX
// with dX expanded in products of deviations), and a population is a few sums of them with integer
// weights.  Against the form above it takes a quarter fewer operations (FP64 bulk node: 594 vector
// instructions against 760), and 22 mean-state constants in place of two per pair and two per
// shell, which stay in scalar registers across a two-step tile's loop.  FP32 and FP16 storage keep the form above,
// whose rounding their results carry; FP64 results move by 1e-14.
// Duo d holds the pairs 2d and 2d + 1, populations 1 + 4d .. 4 + 4d: (+-a, 0) and (0, +-a) on an
// axis shell, else +-(a, b) and +-(-a, b).
constexpr int NDUO = NPAIR / 2;
static_assert(NPAIR % 2 == 0, "pairs come in duos");
constexpr bool duos_ok() {
    for (int d = 0; d < NDUO; ++d) {
        const int p = 2 * d, a = PEX[p], b = PEY[p];
        if (a < 1 || PSH[p] != PSH[p + 1]) return false;
        if (b == 0 ? (PEX[p + 1] != 0 || PEY[p + 1] != a) : (PEX[p + 1] != -a || PEY[p + 1] != b)) return false;
    }
    return true;
}
static_assert(duos_ok(), "duo order");

// Deviations of the node's polynomial coefficients (enum EqCoef; those an order lacks are neither
// formed nor read).  feq - fbar is linear in them, so the difference or the sum of two equilibria
// is one evaluation of the difference or sum of their coefficients.
template <class C> struct EqPoly { C c[NEQ]; };

// Differences of the node's velocity products from the mean state's, v = r u.
template <class C> struct PolyVel { C rho, dx, dy, vx, vy, dxx, dxy, dyy, db; };

template <class C>
__device__ __forceinline__ PolyVel<C> poly_vel(const Mom<C> &m, const K<C> &k) {
    PolyVel<C> v;
    v.rho = k.rho0 + m.drho;
    v.dx = C(LAT_R) * m.dux;
    v.dy = C(LAT_R) * m.duy;
    v.vx = k.r0x + v.dx;
    v.vy = k.r0y + v.dy;
    v.dxx = v.dx * (v.vx + k.r0x);
    v.dyy = v.dy * (v.vy + k.r0y);
    v.dxy = v.dx * v.vy + k.r0x * v.dy;
    v.db = C(1.0 / LAT_R2) * (v.dxx + v.dyy);
    return v;
}

// The coefficients are D[rho X] = drho X(U0) + rho dX, each with its factor folded into X(U0) (from
// the descriptor) and rho; put(i, D) takes coefficient i.
#define LBM_DEV(i, frho, dX) \
    put(std::integral_constant<int, i>{}, m.drho * R.eq0[i] + (frho) * (dX))

// Coefficients of the populations along x (and the rest's), and those along y need besides.
// O1 = k1 + theta r^2 n/2 with k1 = 1 - b/2 - 2 theta (fourth and third order); the second-order
// equilibrium's odd part is a alone (O1 = 1).
template <class C, class F>
__device__ __forceinline__ void poly_x(CRun &R, const Mom<C> &m, const PolyVel<C> &v, const K<C> &k, F &&put) {
    if constexpr (ORDER == 4) {
        const C xx = k.xx0 + v.dxx, th = k.th0 + m.dT, b = k.b0 + v.db;
        const C dtt = m.dT * (th + k.th0), dtb = m.dT * b + k.th0 * v.db;
        const C dk2a = -C(0.25) * v.db - C(1.5) * m.dT;
        LBM_DEV(E0, v.rho, -C(0.5) * v.db - m.dT + C(0.125) * (v.db * (b + k.b0)) + dtb + dtt);
        LBM_DEV(E1, C(LAT_R2) * v.rho, C(0.5) * m.dT - C(0.25) * dtb - dtt);
        LBM_DEV(E2, C(LAT_R2 * LAT_R2 / 8) * v.rho, dtt);
        LBM_DEV(BXX, v.rho, dk2a * xx + k.k2a0 * v.dxx);
        LBM_DEV(TXX, C(LAT_R2 / 4) * v.rho, m.dT * xx + k.th0 * v.dxx);
        LBM_DEV(Q40, C(1.0 / 24.0) * v.rho, v.dxx * (xx + k.xx0));
    } else {   // third and second order: k0 = 1 - b/2 - theta, k2a = 1/2, k2s = theta/2
        LBM_DEV(E0, v.rho, -C(0.5) * v.db - m.dT);
        LBM_DEV(E1, C(LAT_R2 / 2) * v.rho, m.dT);
        LBM_DEV(BXX, C(0.5) * v.rho, v.dxx);
    }
    if constexpr (ORDER >= 3) {
        const C dk1 = -C(0.5) * v.db - C(2) * m.dT;
        LBM_DEV(LX, v.rho, dk1 * v.vx + k.k10 * v.dx);
        LBM_DEV(MX, C(LAT_R2 / 2) * v.rho, m.dT * v.vx + k.th0 * v.dx);
        LBM_DEV(C30, C(1.0 / 6.0) * v.rho, v.dxx * v.vx + k.xx0 * v.dx);
    } else {
        LBM_DEV(LX, v.rho, v.dx);
    }
}
template <class C, class F>
__device__ __forceinline__ void poly_y(CRun &R, const Mom<C> &m, const PolyVel<C> &v, const K<C> &k, F &&put) {
    if constexpr (ORDER == 4) {
        const C yy = k.yy0 + v.dyy, dk2a = -C(0.25) * v.db - C(1.5) * m.dT;
        LBM_DEV(BYY, v.rho, dk2a * yy + k.k2a0 * v.dyy);
        LBM_DEV(TYY, C(LAT_R2 / 4) * v.rho, m.dT * yy + k.th0 * v.dyy);
        LBM_DEV(Q04, C(1.0 / 24.0) * v.rho, v.dyy * (yy + k.yy0));
    } else {
        LBM_DEV(BYY, C(0.5) * v.rho, v.dyy);
    }
    if constexpr (ORDER >= 3) {
        const C dk1 = -C(0.5) * v.db - C(2) * m.dT;
        LBM_DEV(LY, v.rho, dk1 * v.vy + k.k10 * v.dy);
        LBM_DEV(MY, C(LAT_R2 / 2) * v.rho, m.dT * v.vy + k.th0 * v.dy);
        LBM_DEV(C03, C(1.0 / 6.0) * v.rho, v.dyy * v.vy + k.yy0 * v.dy);
    } else {
        LBM_DEV(LY, v.rho, v.dy);
    }
}

// The others, which only the diagonal populations need.
template <class C, class F>
__device__ __forceinline__ void poly_cross(CRun &R, const Mom<C> &m, const PolyVel<C> &v, const K<C> &k, F &&put) {
    if constexpr (ORDER == 4) {
        const C xx = k.xx0 + v.dxx, yy = k.yy0 + v.dyy, xy = k.xy0 + v.dxy;
        const C dk2a = -C(0.25) * v.db - C(1.5) * m.dT;
        const C o6 = C(1.0 / 6.0) * v.rho;
        LBM_DEV(BXY, C(2) * v.rho, dk2a * xy + k.k2a0 * v.dxy);
        LBM_DEV(TXY, C(LAT_R2 / 2) * v.rho, m.dT * xy + k.th0 * v.dxy);
        LBM_DEV(Q31, o6, v.dxx * xy + k.xx0 * v.dxy);
        LBM_DEV(Q22, C(0.25) * v.rho, v.dxx * yy + k.xx0 * v.dyy);
        LBM_DEV(Q13, o6, v.dxy * yy + k.xy0 * v.dyy);
    } else {
        LBM_DEV(BXY, v.rho, v.dxy);
    }
    if constexpr (ORDER >= 3) {
        const C o2 = C(0.5) * v.rho;
        LBM_DEV(C21, o2, v.dxx * v.vy + k.xx0 * v.dy);
        LBM_DEV(C12, o2, v.dyy * v.vx + k.yy0 * v.dx);
    }
}
#undef LBM_DEV

template <class C, class F>
__device__ __forceinline__ void poly_all(CRun &R, const Mom<C> &m, const K<C> &k, F &&put) {
    const PolyVel<C> v = poly_vel<C>(m, k);
    poly_x<C>(R, m, v, k, put);
    poly_y<C>(R, m, v, k, put);
    poly_cross<C>(R, m, v, k, put);
}
template <class C>
__device__ __forceinline__ EqPoly<C> poly_coef(CRun &R, const Mom<C> &m, const K<C> &k) {
    EqPoly<C> q;
    poly_all<C>(R, m, k, [&](auto ic, C d) { q.c[decltype(ic)::value] = d; });
    return q;
}
// q += sign * the coefficients of m, taken in as they are formed.
template <int sign, class C>
__device__ __forceinline__ void poly_add(EqPoly<C> &q, CRun &R, const Mom<C> &m, const K<C> &k) {
    poly_all<C>(R, m, k, [&](auto ic, C d) { q.c[decltype(ic)::value] += C(sign) * d; });
}

// (feq - fbar) / w of the pair +-a along an axis, from that axis's coefficients.
template <int a, class C>
__device__ __forceinline__ void poly_axis_pair(C e0, C e1, C e2, C bxx, C txx, C q40, C lx, C mx, C c30, C &tp, C &tm) {
    constexpr int aa = a * a;
    C e = e0 + C(aa) * e1;
    if constexpr (ORDER == 4) {
        e += C(aa * aa) * e2;
        bxx += C(aa) * txx;
    }
    e += C(aa) * bxx;
    if constexpr (ORDER == 4) e += C(aa * aa) * q40;
    if constexpr (ORDER >= 3) {
        lx += C(aa) * mx;
        lx += C(aa) * c30;
    }
    tp = e + C(a) * lx;
    tm = e - C(a) * lx;
}
constexpr bool axis_duo(int d) { return PEY[2 * d] == 0; }
template <int d, class C>
__device__ __forceinline__ void poly_pair_x(const EqPoly<C> &q, C &tp, C &tm) {
    poly_axis_pair<PEX[2 * d], C>(q.c[E0], q.c[E1], q.c[E2], q.c[BXX], q.c[TXX], q.c[Q40], q.c[LX], q.c[MX], q.c[C30], tp, tm);
}
template <int d, class C>
__device__ __forceinline__ void poly_pair_y(const EqPoly<C> &q, C &tp, C &tm) {
    poly_axis_pair<PEX[2 * d], C>(q.c[E0], q.c[E1], q.c[E2], q.c[BYY], q.c[TYY], q.c[Q04], q.c[LY], q.c[MY], q.c[C03], tp, tm);
}
// (feq - fbar) / w of the four populations of a diagonal duo d, in population order.
template <int d, class C>
__device__ __forceinline__ void poly_diagonals(const EqPoly<C> &q, C (&t)[4]) {
    constexpr int a = PEX[2 * d], b = PEY[2 * d], n = SHELL_E2[PSH[2 * d]], aa = a * a, bb = b * b;
    C s = q.c[E0] + C(n) * q.c[E1], bxx = q.c[BXX], byy = q.c[BYY], bxy = q.c[BXY], lx = q.c[LX], ly = q.c[LY];
    if constexpr (ORDER == 4) {
        s += C(n * n) * q.c[E2];
        bxx += C(n) * q.c[TXX];
        byy += C(n) * q.c[TYY];
        bxy += C(n) * q.c[TXY];
        bxy += C(aa) * q.c[Q31];
        bxy += C(bb) * q.c[Q13];
    }
    s += C(aa) * bxx;
    s += C(bb) * byy;
    if constexpr (ORDER == 4) {
        s += C(aa * aa) * q.c[Q40];
        s += C(aa * bb) * q.c[Q22];
        s += C(bb * bb) * q.c[Q04];
    }
    if constexpr (ORDER >= 3) {
        lx += C(n) * q.c[MX];
        ly += C(n) * q.c[MY];
        lx += C(aa) * q.c[C30];
        ly += C(bb) * q.c[C03];
        lx += C(bb) * q.c[C12];
        ly += C(aa) * q.c[C21];
    }
    const C ep = s + C(a * b) * bxy, em = s - C(a * b) * bxy;
    const C y = C(b) * ly, op = y + C(a) * lx, om = y - C(a) * lx;
    t[0] = ep + op;
    t[1] = ep - op;
    t[2] = em + om;
    t[3] = em - om;
}

// Weight of population i.
template <int i> constexpr double weight_of() { return SHELL_W[shell_of(i)]; }

// Calls emit(i, (feq_i - fbar_i) / w_i), compile-time i, for pair p (0 or 1) of axis duo d, and for
// the populations of the duos [D0, D1).
template <int d, int p, class C, class F>
__device__ __forceinline__ void poly_axis(const EqPoly<C> &q, F &&emit) {
    C tp, tm;
    if constexpr (p == 0) poly_pair_x<d>(q, tp, tm);
    else poly_pair_y<d>(q, tp, tm);
    emit(std::integral_constant<int, 1 + 4 * d + 2 * p>{}, tp);
    emit(std::integral_constant<int, 2 + 4 * d + 2 * p>{}, tm);
}
template <int D0, int D1, class C, class F>
__device__ __forceinline__ void poly_duos(const EqPoly<C> &q, F &&emit) {
    static_for<D0, D1>([&](auto dc) {
        constexpr int d = decltype(dc)::value;
        if constexpr (axis_duo(d)) {
            poly_axis<d, 0>(q, emit);
            poly_axis<d, 1>(q, emit);
        } else {
            C t[4];
            poly_diagonals<d>(q, t);
            static_for<0, 4>([&](auto lc) {
                constexpr int l = decltype(lc)::value;
                emit(std::integral_constant<int, 1 + 4 * d + l>{}, t[l]);
            });
        }
    });
}

// Calls emit(i, (feq_i - fbar_i) / w_i) for every population of a node of moments m: the rest and
// the x populations first, which need 9 of the 22 coefficients, then the y populations, then the
// diagonals.  In FP64 each stage forms its coefficients only then, from velocity products formed
// afresh: a D2Q37 kernel that holds the 37 populations would pass 128 registers (4 waves per
// SIMD) with all of them beside it.
template <class C>
__device__ __forceinline__ Mom<C> poly_stage(const Mom<C> &m) {
    Mom<C> c = m;
    if constexpr (sizeof(C) == 8) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : "+v"(c.drho), "+v"(c.dux), "+v"(c.duy), "+v"(c.dT));
    }
    return c;
}
template <class C, class F>
__device__ __forceinline__ void for_each_poly(CRun &R, const Mom<C> &m, const K<C> &k, F &&emit) {
    EqPoly<C> q;
    auto put = [&](auto ic, C d) { q.c[decltype(ic)::value] = d; };
    poly_x<C>(R, m, poly_vel<C>(m, k), k, put);
    emit(std::integral_constant<int, 0>{}, q.c[E0]);
    static_for<0, NDUO>([&](auto dc) {
        if constexpr (axis_duo(decltype(dc)::value)) poly_axis<decltype(dc)::value, 0>(q, emit);
    });
    const Mom<C> my = poly_stage<C>(m);
    poly_y<C>(R, my, poly_vel<C>(my, k), k, put);
    static_for<0, NDUO>([&](auto dc) {
        if constexpr (axis_duo(decltype(dc)::value)) poly_axis<decltype(dc)::value, 1>(q, emit);
    });
    const Mom<C> mc = poly_stage<C>(my);
    poly_cross<C>(R, mc, poly_vel<C>(mc, k), k, put);
    static_for<0, NDUO>([&](auto dc) {
        if constexpr (!axis_duo(decltype(dc)::value)) poly_duos<decltype(dc)::value, decltype(dc)::value + 1>(q, emit);
    });
}

// Collision of population i (deviation g): BGK, g + omega (feq - g), and with PML the term
// -2 sigma fhat (s = sigma; with sigma = 0 it leaves BGK's bits).  t: (feq - fbar) / w in FP64
// storage, else feq - fbar.  (feq - g is formed whole: it is small near equilibrium, so the
// relaxation rounds once at the populations' scale.)
template <bool PML, int i, class S, class C>
__device__ __forceinline__ C relax(C g, C t, C omega, C s) {
    if constexpr (std::is_same<S, double>::value) {
        C out = g + omega * (C(weight_of<i>()) * t - g);
        if constexpr (PML) out -= s * (C(2 * weight_of<i>()) * t);
        return out;
    } else {
        C out = g + omega * (t - g);
        if constexpr (PML) out = out - s * (C(2) * t);
        return out;
    }
}

// Collision of a node from its populations; emit(i, out) gets each population as it is done.
template <bool PML, class S, class C, class F>
__device__ __forceinline__ void collide(CRun &R, const K<C> &k, const Mom<C> &m, const C (&g)[NQ], C s, F &&emit) {
    auto one = [&](auto ic, C t) {
        constexpr int i = decltype(ic)::value;
        emit(ic, relax<PML, i, S, C>(g[i], t, k.omega, s));
    };
    if constexpr (std::is_same<S, double>::value)
        for_each_poly<C>(R, m, k, one);
    else
        for_each_feq<C>(eq_coef<C>(m.drho, m.dux, m.duy, m.dT, k), R, k, one);
}
// ------------------------------------------------------------------------------------------
// characteristic boundary (float64 always)
// ------------------------------------------------------------------------------------------
// LODI along the outward normal of `side` for boundary node (x, y): primitive variables
// V = (rho, u_n, u_t, T), A = S^{-1} Lambda S, Lambda = diag(u_n - c, u_n, u_n, u_n + c),
// c = sqrt(2T) (p = rho T, gamma = 2).  Incoming amplitudes are zero (eq. PNR); an outgoing
// amplitude takes the upwind difference over the interval its characteristic crosses in one
// step (nu = lambda/r cells, foot point limited to two cells).  Adds the one-step increment
// dV = -S^{-1} Lbar (eq. thermal_LODI_macro_evo) to Ut in the global frame.
__device__ void lodi_add(CRun &R, const GLOBAL double *Uc, int side, int x, int y, int t,
                         double Ut[4]) {
    const unsigned qp = (unsigned)R.qplane;
    int nx = side == XMIN ? -1 : (side == XMAX ? 1 : 0);
    int ny = side == YMIN ? -1 : (side == YMAX ? 1 : 0);
    double V[3][4];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        int jj = j == 0 ? t : fidx(R, x - j * nx, y - j * ny);
        if (jj < 0) jj = t;
        jj = (int)LBM_GUARD(R, jj, R.qplane);
        double rho = Uc[jj], ux = Uc[qp + jj], uy = Uc[2 * qp + jj], T = Uc[3 * qp + jj];
        V[j][0] = rho;
        V[j][1] = nx ? nx * ux : ny * uy;
        V[j][2] = nx ? uy : ux;
        V[j][3] = T;
    }
    double rho = V[0][0], un = V[0][1], T = V[0][3];
    double c = sqrt(2.0 * T);
    double lam[4] = {un - c, un, un, un + c};
    double L[4][4] = {{T, -rho * c, 0.0, rho}, {T, 0.0, 0.0, -rho}, {0.0, 0.0, 1.0, 0.0},
                      {T, rho * c, 0.0, rho}};
    double D[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double w[3];
#pragma unroll
        for (int j = 0; j < 3; ++j)
            w[j] = L[k][0] * V[j][0] + L[k][1] * V[j][1] + L[k][2] * V[j][2] + L[k][3] * V[j][3];
        if (lam[k] > 0.0) {
            double nu = fmin(lam[k] * (1.0 / LAT_R), 2.0);
            int j0 = nu >= 1.0 ? 1 : 0;
            double phi = nu - j0;
            double wa = j0 ? w[1] : w[0], wb = j0 ? w[2] : w[1];
            double wfoot = (1.0 - phi) * wa + phi * wb;
            D[k] = w[0] - wfoot;
        } else {
            D[k] = 0.0;
        }
    }
    // closed-form S^{-1}: columns (1/4T, -1/2rc, 0, 1/4r), (1/2T, 0, 0, -1/2r), e3,
    // (1/4T, 1/2rc, 0, 1/4r)
    double dR = -((D[0] + D[3]) / (4.0 * T) + D[1] / (2.0 * T));
    double dUn = -(D[3] - D[0]) / (2.0 * rho * c);
    double dUt = -D[2];
    double dTT = -((D[0] + D[3]) / (4.0 * rho) - D[1] / (2.0 * rho));
    Ut[0] += dR;
    Ut[3] += dTT;
    if (nx) { Ut[1] += nx * dUn; Ut[2] += dUt; }
    else    { Ut[2] += ny * dUn; Ut[1] += dUt; }
}

// Characteristic variables of the Euler flux along one direction for primitive variables
// v = (rho, u_along, u_across, T) (p = rho T, gamma = 2, c = sqrt(2T)), rows for the eigenvalues
// u - c, u (entropy), u (shear), u + c, and the inverse map.
__device__ __forceinline__ void char_fwd(double rho, double T, double c, const double (&v)[4], double (&w)[4]) {
    w[0] = T * v[0] - rho * c * v[1] + rho * v[3];
    w[1] = T * v[0] - rho * v[3];
    w[2] = v[2];
    w[3] = T * v[0] + rho * c * v[1] + rho * v[3];
}
__device__ __forceinline__ void char_inv(double rho, double T, double c, const double (&b)[4], double (&v)[4]) {
    v[0] = (b[0] + b[3]) / (4.0 * T) + b[1] / (2.0 * T);
    v[1] = (b[3] - b[0]) / (2.0 * rho * c);
    v[2] = b[2];
    v[3] = (b[0] + b[3]) / (4.0 * rho) - b[1] / (2.0 * rho);
}

// One-step increment, at edge position j (compile-time, 2..4 of 0..6), of the Euler flux along
// the edge: each characteristic variable of the edge direction, eigenvectors frozen at Vn[j],
// moves over the interval its characteristic crosses in one step (foot point at most 2 cells
// away, linear interpolation), written in differences so a state constant along the edge gives
// exactly zero.  Vn and dV in the normal frame (rho, u_n, u_t, T).
template <int J>
__device__ __forceinline__ void edge_advect(const double (&Vn)[7][4], double (&dV)[4]) {
    const double rho = Vn[J][0], ut = Vn[J][2], T = Vn[J][3], c = sqrt(2.0 * T);
    double w[5][4];
#pragma unroll
    for (int m = 0; m < 5; ++m) {
        const double vt[4] = {Vn[J - 2 + m][0], Vn[J - 2 + m][2], Vn[J - 2 + m][1], Vn[J - 2 + m][3]};
        char_fwd(rho, T, c, vt, w[m]);
    }
    const double lam[4] = {ut - c, ut, ut, ut + c};
    double dW[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double nu = lam[k] * (1.0 / LAT_R);
        if (!(nu == nu)) nu = 0.0;
        nu = fmin(fmax(nu, -2.0), 2.0);
        const double a = fabs(nu);
        const bool far = a >= 1.0, fwd = nu > 0.0;      // foot beyond one cell; foot at -nu
        const double phi = far ? a - 1.0 : a;
        const double w1 = fwd ? w[1][k] : w[3][k], w2 = fwd ? w[0][k] : w[4][k];
        const double wa = far ? w1 : w[2][k], wb = far ? w2 : w1;
        dW[k] = -((1.0 - phi) * (w[2][k] - wa) + phi * (w[2][k] - wb));
    }
    double dt[4];
    char_inv(rho, T, c, dW, dt);
    dV[0] = dt[0]; dV[1] = dt[2]; dV[2] = dt[1]; dV[3] = dt[3];
}

// CBC (A) (Sec. 4 eq. thermal_CBC_macro_evo with eq. CBC-Relax of Sec. 5.2) at node (x, y) of
// `side`, a node on no other open side: U_tgt += one step of dU/dt = -S^{-1} (Lbar + T + V) in
// the normal frame, where
//   - outgoing waves keep their LODI amplitude (upwind over the crossed interval, as lodi_add)
//     plus the transverse and viscous parts;
//   - T: the Euler flux along the edge, advected in the edge's characteristics (edge_advect) on
//     the node's own layer;
//   - V: tangential second derivatives only (normal viscous fluxes of an outflow vanish),
//     nu = (tau - 1/2)/r^2 on both velocity components and 2 nu on T (Pr = 1, c_p/c_v = 2),
//     taken of the transverse-advected states at the node and its edge neighbours (advection,
//     then diffusion: the unsplit sum of the two explicit parts is unstable);
//   - eq. CBC-Relax with T and V as right-hand-side terms: an incoming amplitude is
//     (1 - Ma) T_inc + V_inc of them, leaving it Ma T_inc (Ma = |u0| with c_s = 1).
// Edge neighbours beyond an open edge's ends repeat the end node.  Float64 throughout.
__device__ void cbc_a_add(CRun &R, const GLOBAL double *Uc, int side, int x, int y, int t, double Ut[4]) {
    const unsigned qp = (unsigned)R.qplane;
    const int nx = side == XMIN ? -1 : (side == XMAX ? 1 : 0);
    const int ny = side == YMIN ? -1 : (side == YMAX ? 1 : 0);
    const int nt = nx ? R.Ny : R.Nx, ct = nx ? y : x;
    const bool topen = nx ? R.open_y : R.open_x;
    double Vn[7][4];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        int cc = ct + j - 3;
        if (topen) cc = min(max(cc, 0), nt - 1);
        else cc = cc < 0 ? cc + nt : (cc >= nt ? cc - nt : cc);
        int jj = nx ? fidx(R, x, cc) : fidx(R, cc, y);
        if (jj < 0) jj = t;
        jj = (int)LBM_GUARD(R, jj, R.qplane);
        const double ux = Uc[qp + jj], uy = Uc[2 * qp + jj];
        Vn[j][0] = Uc[jj];
        Vn[j][1] = nx ? nx * ux : ny * uy;
        Vn[j][2] = nx ? uy : ux;
        Vn[j][3] = Uc[3 * qp + jj];
    }
    const double rho = Vn[3][0], un = Vn[3][1], T = Vn[3][3], c = sqrt(2.0 * T);
    const double lam[4] = {un - c, un, un, un + c};
    // LODI amplitudes of the outgoing normal characteristics, from x_b, x_b - n, x_b - 2n
    double wn[3][4];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        int jj = k == 0 ? t : fidx(R, x - k * nx, y - k * ny);
        if (jj < 0) jj = t;
        jj = (int)LBM_GUARD(R, jj, R.qplane);
        const double ux = Uc[qp + jj], uy = Uc[2 * qp + jj];
        const double v[4] = {Uc[jj], nx ? nx * ux : ny * uy, nx ? uy : ux, Uc[3 * qp + jj]};
        char_fwd(rho, T, c, v, wn[k]);
    }
    // transverse part at the node and its edge neighbours; viscous part of the advected states
    double dVT[4], dm[4], dp[4];
    edge_advect<2>(Vn, dm);
    edge_advect<3>(Vn, dVT);
    edge_advect<4>(Vn, dp);
    double dVV[4] = {0.0, 0.0, 0.0, 0.0};
    if (!(topen && (ct == 0 || ct == nt - 1))) {
        const double nuv = (1.0 / R.omega - 0.5) * (1.0 / LAT_R2);
#pragma unroll
        for (int m = 1; m < 4; ++m) {
            const double a0 = Vn[2][m] + dm[m], a1 = Vn[3][m] + dVT[m], a2 = Vn[4][m] + dp[m];
            dVV[m] = (m == 3 ? 2.0 * nuv : nuv) * (a2 - 2.0 * a1 + a0);
        }
    }
    double aT[4], aV[4];
    char_fwd(rho, T, c, dVT, aT);
    char_fwd(rho, T, c, dVV, aV);
    const double ma = sqrt(R.b0);
    double dw[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (lam[k] > 0.0) {
            const double nu = fmin(lam[k] * (1.0 / LAT_R), 2.0);
            const bool far = nu >= 1.0;
            const double phi = far ? nu - 1.0 : nu;
            const double wa = far ? wn[1][k] : wn[0][k], wb = far ? wn[2][k] : wn[1][k];
            const double D = (1.0 - phi) * (wn[0][k] - wa) + phi * (wn[0][k] - wb);
            dw[k] = -D + aT[k] + aV[k];
        } else {
            dw[k] = ma * aT[k];
        }
    }
    double d[4];
    char_inv(rho, T, c, dw, d);
    Ut[0] += d[0];
    Ut[3] += d[3];
    if (nx) { Ut[1] += nx * d[1]; Ut[2] += d[2]; }
    else    { Ut[2] += ny * d[1]; Ut[1] += d[2]; }
}

// Where a boundary node's pulls come from: the population buffer (SRC_F), or, in the second step
// of a two-step pass, the bands that hold the level between (SRC_M).
enum { SRC_F = 0, SRC_M = 1 };

__device__ __forceinline__ int clamp_x(CRun &R, int x) { return R.open_x ? min(max(x, 3), R.Nx - 4) : x; }
__device__ __forceinline__ int clamp_y(CRun &R, int y) { return R.open_y ? min(max(y, 3), R.Ny - 4) : y; }

// Row and column of a node in the row band (rows [Ny - bT, Ny), then [0, bB); every column) and in
// the column band (columns [Nx - bR, Nx), then [0, bL); the rows off the y frame strips).
__device__ __forceinline__ int band_row(CRun &R, int y) { return y < R.bB ? R.bT + y : y - (R.Ny - R.bT); }
__device__ __forceinline__ int band_col(CRun &R, int x) { return x < R.bL ? R.bR + x : x - (R.Nx - R.bR); }

// Source of the pulls of node (x, y): x_f = clamp(x, 3, N-4) on open axes (eq. zg-bc copies all q
// populations of x_f to a boundary node; interior frame nodes are their own x_f).  In the bands a
// node whose pulled rows all lie in the row band reads that one, any other the column band; the
// band halves meet at the grid's edge, so a periodic axis needs no wrap across them (only x in the
// row band wraps).
struct Pull {
    int xs, ys, wx;
    unsigned plane, pitch, first;   // SRC_M: strides and first element of the node's band
};

template <int SRC> __device__ __forceinline__ Pull pull_from(CRun &R, int x, int y) {
    Pull n{};
    n.xs = clamp_x(R, x);
    n.ys = clamp_y(R, y);
    if constexpr (SRC == SRC_M) {
        const bool rows = n.ys < R.bB - REACH || n.ys >= R.Ny - (R.bT - REACH);
        n.plane = (unsigned)(rows ? R.m_row : R.l_row);
        n.pitch = NQ * n.plane;
        n.first = rows ? 0u : (unsigned)R.l_first;
        n.wx = rows ? R.Nx : 1 << 30;
        n.ys = rows ? band_row(R, n.ys) : n.ys - R.gym;
        n.xs = rows ? n.xs : band_col(R, n.xs);
    }
    return n;
}

// Pull of population I: the buffer with a single periodic wrap on periodic axes (N >= 3), where
// identical shifts across populations fold to 7 source-row and 7 source-column offsets per node,
// so each population costs one add; or the node's band.
template <int SRC, class S, class C, int I>
__device__ __forceinline__ C pull_one(CRun &R, const GLOBAL S *src, const Pull &n, C inv_scale) {
    int sy = n.ys - ey_of(I), sx = n.xs - ex_of(I);
    if constexpr (SRC == SRC_M) {
        if constexpr (ex_of(I) > 0) sx += sx < 0 ? n.wx : 0;
        if constexpr (ex_of(I) < 0) sx -= sx >= n.wx ? n.wx : 0;
        const unsigned idx = n.first + (unsigned)I * n.plane + (unsigned)sy * n.pitch + (unsigned)sx;
        return cvt_in(src[LBM_GUARD(R, (long long)idx, R.msize)], inv_scale);
    } else {
        const int Nx = R.Nx, Ny = R.Ny;
        if constexpr (ey_of(I) > 0) sy += sy < 0 ? Ny : 0;
        if constexpr (ey_of(I) < 0) sy -= sy >= Ny ? Ny : 0;
        if constexpr (ex_of(I) > 0) sx += sx < 0 ? Nx : 0;
        if constexpr (ex_of(I) < 0) sx -= sx >= Nx ? Nx : 0;
        return cvt_in(src[LBM_GUARD(R, (long long)I * R.plane + (long long)sy * R.pitch + sx, R.fsize)], inv_scale);
    }
}

template <int SRC, class S>
__device__ __forceinline__ const GLOBAL S *pull_base(CRun &R, int par) {
    return (const GLOBAL S *)(SRC == SRC_M ? R.M : R.f[par]);
}

template <int SRC, class S, class C>
__device__ __forceinline__ void gather_clamped(CRun &R, const GLOBAL S *src, int x, int y,
                                               C inv_scale, C (&g)[NQ]) {
    const Pull n = pull_from<SRC>(R, x, y);
    static_for<0, NQ>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        g[i] = pull_one<SRC, S, C, i>(R, src, n, inv_scale);
    });
}

// Non-equilibrium extrapolation into G (ring index tt): G <- feq(U_tgt) + g(x_f) - feq(U(x_f)),
// in float64, g the pulled populations of x_f (deviation form).  Two sweeps keep it in few
// registers: the moments of the pull first, then the fill a few pairs at a time from a second
// pull of the same values (cache hits).
template <int SRC, class S, class C>
__device__ __forceinline__ void nrbc_fill(CRun &R, const GLOBAL S *src, int x, int y, C inv_scale,
                                          const double (&Ut)[4], int tt) {
    K<double> kd = load_k<double>(R);
    Mom<double> mf;
    {
        const Pull n = pull_from<SRC>(R, x, y);
        mf = moments_streamed<6, double>(
            [&](auto ic) { return (double)pull_one<SRC, S, C, decltype(ic)::value>(R, src, n, inv_scale); }, kd);
    }
    __builtin_amdgcn_sched_barrier(0);
    constexpr bool POLY = std::is_same<S, double>::value;
    Eq<double> ef, et;
    EqPoly<double> e;
    if constexpr (POLY) {   // feq(U_tgt) - feq(U(x_f)): one evaluation of the difference of their coefficients
        e = poly_coef<double>(R, Mom<double>{Ut[0] - R.rho0, Ut[1] - R.u0x, Ut[2] - R.u0y, Ut[3] - R.T0, 0.0}, kd);
        __builtin_amdgcn_sched_barrier(0);
        poly_add<-1, double>(e, R, mf, kd);
        __builtin_amdgcn_sched_barrier(0);
    } else {
        ef = eq_coef<double>(mf.drho, mf.dux, mf.duy, mf.dT, kd);
        et = eq_coef<double>(Ut[0] - R.rho0, Ut[1] - R.u0x, Ut[2] - R.u0y, Ut[3] - R.T0, kd);
    }
    Pull n = pull_from<SRC>(R, x, y);
    // recompute the addresses of the second pull instead of keeping those of the first live
    asm volatile("" : "+v"(n.xs), "+v"(n.ys));
    GLOBAL C *G = (GLOBAL C *)R.G;
    const unsigned rp = (unsigned)R.rplane;
    {
        const C g0 = pull_one<SRC, S, C, 0>(R, src, n, inv_scale);
        if constexpr (POLY) G[tt] = (C)((double)g0 + SHELL_W[0] * e.c[E0]);
        else G[tt] = (C)((double)g0 + (feq_rest<double>(et, R) - feq_rest<double>(ef, R)));
    }
    constexpr int PC = POLY ? 4 : 3;   // pairs per sweep group
    static_for<0, (NPAIR + PC - 1) / PC>([&](auto cc) {
        constexpr int P0 = decltype(cc)::value * PC;
        constexpr int P1 = P0 + PC < NPAIR ? P0 + PC : NPAIR;
        C gv[2 * (P1 - P0)];
        static_for<0, 2 * (P1 - P0)>([&](auto lc) {
            constexpr int l = decltype(lc)::value;
            gv[l] = pull_one<SRC, S, C, 1 + 2 * P0 + l>(R, src, n, inv_scale);
        });
        if constexpr (POLY)
            poly_duos<P0 / 2, P1 / 2>(e, [&](auto ic, double t) {
                constexpr int i = decltype(ic)::value;
                G[i * rp + tt] = (C)((double)gv[i - 1 - 2 * P0] + weight_of<i>() * t);
            });
        else
            feq2_pairs<P0, P1>(et, ef, R, kd, [&](auto ic, double ft, double ff) {
                constexpr int i = decltype(ic)::value;
                G[i * rp + tt] = (C)((double)gv[i - 1 - 2 * P0] + (ft - ff));
            });
        __builtin_amdgcn_sched_barrier(0);
    });
}

// grad Q stencil of a frame node (frame index t): d/dalpha Q = cs*Q(x) + c0*Q(j0) + c1*Q(j1),
// central (0, 1/2, -1/2 at x+1, x-1), one-sided at the outermost layer of an open axis (outward
// normal s: s*(3/2, -2, 1/2) at x, x-s, x-2s) (eqs. FD-dx-center, FD-dx-bw).  Offsets are byte
// offsets into one Q plane; a neighbour outside the frame falls back to the node itself (such
// nodes lie off the layer, where sigma = 0).
template <class C> struct QStencil {
    unsigned ot, ox0, ox1, oy0, oy1;
    C cxs, cx0, cx1, cys, cy0, cy1;
};

template <class C>
__device__ __forceinline__ QStencil<C> q_stencil(CRun &R, int x, int y, int t) {
    QStencil<C> q;
    int jx0, jx1, jy0, jy1;
    if (R.open_x && x == 0) {
        jx0 = fidx(R, 1, y); jx1 = fidx(R, 2, y);
        q.cxs = C(-1.5); q.cx0 = C(2); q.cx1 = C(-0.5);
    } else if (R.open_x && x == R.Nx - 1) {
        jx0 = fidx(R, x - 1, y); jx1 = fidx(R, x - 2, y);
        q.cxs = C(1.5); q.cx0 = C(-2); q.cx1 = C(0.5);
    } else {
        int xp = x + 1, xm = x - 1;
        if (xp >= R.Nx) xp -= R.Nx;
        if (xm < 0) xm += R.Nx;
        jx0 = fidx(R, xp, y); jx1 = fidx(R, xm, y);
        q.cxs = C(0); q.cx0 = C(0.5); q.cx1 = C(-0.5);
    }
    if (R.open_y && y == 0) {
        jy0 = fidx(R, x, 1); jy1 = fidx(R, x, 2);
        q.cys = C(-1.5); q.cy0 = C(2); q.cy1 = C(-0.5);
    } else if (R.open_y && y == R.Ny - 1) {
        jy0 = fidx(R, x, y - 1); jy1 = fidx(R, x, y - 2);
        q.cys = C(1.5); q.cy0 = C(-2); q.cy1 = C(0.5);
    } else {
        int yp = y + 1, ym = y - 1;
        if (yp >= R.Ny) yp -= R.Ny;
        if (ym < 0) ym += R.Ny;
        jy0 = fidx(R, x, yp); jy1 = fidx(R, x, ym);
        q.cys = C(0); q.cy0 = C(0.5); q.cy1 = C(-0.5);
    }
    q.ox0 = (unsigned)LBM_GUARD(R, jx0 < 0 ? t : jx0, R.qplane) * (unsigned)sizeof(C);
    q.ox1 = (unsigned)LBM_GUARD(R, jx1 < 0 ? t : jx1, R.qplane) * (unsigned)sizeof(C);
    q.oy0 = (unsigned)LBM_GUARD(R, jy0 < 0 ? t : jy0, R.qplane) * (unsigned)sizeof(C);
    q.oy1 = (unsigned)LBM_GUARD(R, jy1 < 0 ? t : jy1, R.qplane) * (unsigned)sizeof(C);
    q.ot = (unsigned)LBM_GUARD(R, t, R.qplane) * (unsigned)sizeof(C);
    return q;
}

// The rest of the PML term of population i, -sigma (e.grad Q + sigma Q), added to h; v: Q at the node,
// its x neighbours and its y neighbours.
template <int i, class C>
__device__ __forceinline__ C pml_gradient(const QStencil<C> &q, const C (&v)[5], C h, C s) {
    C gq = C(0);
    if constexpr (ex_of(i) != 0) gq += C(ex_of(i)) * (q.cxs * v[0] + q.cx0 * v[1] + q.cx1 * v[2]);
    if constexpr (ey_of(i) != 0) gq += C(ey_of(i)) * (q.cys * v[0] + q.cy0 * v[3] + q.cy1 * v[4]);
    return h - s * (gq + s * v[0]);
}

// Appendix (eq. NSF-CHAR-PML): with a PML the macroscopic equations carry source terms built
// from the auxiliary moments; with phi = (1, xi_x, xi_y, |xi|^2/2) the selected parts
// I = sum phi_i e_i . grad Q_i (bit 0), II = 2 sum phi_i fhat_i (bit 1) and
// III = sigma sum phi_i Q_i (bit 2) move the characteristic target over one step by
// s = +sigma (I + II + III) (the appendix's signs) in conserved variables (rho, rho u,
// rho (|u|^2/2 + T)), converted to (rho, u, T) at U^n by the chain rule.  The quadrature carries
// the conserved moments of feq exactly, so II = 2 (U^n - Ubar) in conserved form.  Q and U of
// level n; float64 arithmetic; the population loop is left rolled (few nodes, low pressure).
template <class C>
__device__ __forceinline__ void pml_moments(CRun &R, int x, int y, int t, const GLOBAL double *Uc,
                                            double (&dU)[4]) {
    dU[0] = dU[1] = dU[2] = dU[3] = 0.0;
    const double sg = sigma_at(R, x, y);
    if (!(sg > 0.0)) return;
    const unsigned qp = (unsigned)R.qplane, flags = (unsigned)R.pml_terms;
    const double rho = Uc[t], ux = Uc[qp + t], uy = Uc[2 * qp + t], T = Uc[3 * qp + t];
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    if (flags & 5u) {
        const QStencil<C> qs = q_stencil<C>(R, x, y, t);
        const GLOBAL C *Q = (const GLOBAL C *)R.Q;
#pragma unroll 1
        for (int i = 0; i < NQ; ++i) {
            const int ex = ex_of(i), ey = ey_of(i);
            const GLOBAL C *Qi = Q + (long long)i * qp;
            const double Qt = (double)*at(Qi, qs.ot);
            double a = 0.0;
            if (flags & 1u) {
                if (ex != 0)
                    a += ex * ((double)qs.cxs * Qt + (double)qs.cx0 * (double)*at(Qi, qs.ox0) +
                               (double)qs.cx1 * (double)*at(Qi, qs.ox1));
                if (ey != 0)
                    a += ey * ((double)qs.cys * Qt + (double)qs.cy0 * (double)*at(Qi, qs.oy0) +
                               (double)qs.cy1 * (double)*at(Qi, qs.oy1));
            }
            if (flags & 4u) a += sg * Qt;
            const double xx = LAT_R * ex, yy = LAT_R * ey;
            s0 += a;
            s1 += xx * a;
            s2 += yy * a;
            s3 += (0.5 * (xx * xx + yy * yy)) * a;
        }
    }
    if (flags & 2u) {
        const double b0 = R.rho0, bx = R.u0x, by = R.u0y, bT = R.T0;
        s0 += 2.0 * (rho - b0);
        s1 += 2.0 * (rho * ux - b0 * bx);
        s2 += 2.0 * (rho * uy - b0 * by);
        s3 += 2.0 * (rho * (0.5 * (ux * ux + uy * uy) + T) - b0 * (0.5 * (bx * bx + by * by) + bT));
    }
    s0 *= sg; s1 *= sg; s2 *= sg; s3 *= sg;
    dU[0] = s0;
    dU[1] = (s1 - ux * s0) / rho;
    dU[2] = (s2 - uy * s0) / rho;
    dU[3] = (s3 - ux * s1 - uy * s2 + (0.5 * (ux * ux + uy * uy) - T) * s0) / rho;
}

// Blocks of a run's boundary launches: the characteristic ring first (ring numbering, RING_BLOCK
// nodes per block), then the frame off the ring (annulus numbering, FRAME_BLOCK nodes per block),
// both counts padded to multiples of 8.  frame_start maps a frame block to its first annulus
// index, XCD by XCD.
__device__ __forceinline__ int ring_blocks(CRun &R) { return ring_block_count(R.ring_n); }
__device__ __forceinline__ int frame_start(CRun &R, int fblock) {
    return xcd_swizzle(fblock, frame_block_count(R.ann_n)) * FRAME_BLOCK;
}

// Characteristic targets of the ring, formed ahead of phase A for runs that select the appendix's
// PML moments or have a CBC (A) side: U_tgt = U^n(x_b) plus, for each characteristic side the
// node lies on, the CBC (A) increment (a node on that side only) or the LODI increment (corners
// add both normals), plus the PML moments; stored to P (4 planes of the ring numbering,
// float64).
template <class S>
__global__ __launch_bounds__(256) void k_target(RunDev *const *__restrict__ runs,
                                                const int *__restrict__ prefix, int nruns, Sub ks) {
    using C = typename Traits<S>::C;
    const int b = blockIdx.x;
    const int j = find_run(prefix, nruns, b);
    CRun &R = run_of(runs, j);
    const int par = sub_par(R, ks);
    if (par < 0 || !R.tgt_pre) return;
    if ((int)threadIdx.x >= RING_BLOCK) return;
    const int tt = (b - ((const CONSTANT int *)prefix)[j]) * RING_BLOCK + (int)threadIdx.x;
    if (tt >= R.ring_n) return;
    int x, y;
    ring_xy(R, tt, x, y);
    const int t = (int)LBM_GUARD(R, tt, R.rplane);   // a ring node's frame index is its ring index
    const GLOBAL double *Uc = (const GLOBAL double *)R.U[u_par(R, ks)];
    const unsigned qp = (unsigned)R.qplane;
    double Ut[4] = {Uc[t], Uc[qp + t], Uc[2 * qp + t], Uc[3 * qp + t]};
    // open sides whose boundary layers hold the node: CBC (A) applies on one side only, corners
    // take the LODI target of each characteristic normal
    bool on[4];
    int n_open = 0;
    for (int s = 0; s < 4; ++s) {
        on[s] = s == XMIN ? x < 3 : s == XMAX ? x >= R.Nx - 3 : s == YMIN ? y < 3 : y >= R.Ny - 3;
        on[s] = on[s] && R.bc[s] != BC_PERIODIC;
        n_open += on[s];
    }
    for (int s = 0; s < 4; ++s) {
        if (!on[s]) continue;
        if (R.bc[s] == BC_NRBC_A && n_open == 1) cbc_a_add(R, Uc, s, x, y, t, Ut);
        else if (is_char_bc(R.bc[s])) lodi_add(R, Uc, s, x, y, t, Ut);
    }
    if (R.pml_terms) {
        double dU[4];
        pml_moments<C>(R, x, y, t, Uc, dU);
        for (int k = 0; k < 4; ++k) Ut[k] += dU[k];
    }
    GLOBAL double *P = (GLOBAL double *)R.P;
    const unsigned rp = (unsigned)R.rplane;
#pragma unroll
    for (int k = 0; k < 4; ++k) P[k * rp + tt] = Ut[k];
}

// Ring node of characteristic sides: U_tgt = U(x_b) of the last completed level plus the LODI
// increment of each NRBC side the node lies on (corners add both normals) or, for runs that form
// their targets ahead, the target of k_target; then the clamped pull of x_f and the
// non-equilibrium extrapolation into G (ring index tt), where the Q update, the frame kernel and
// the moment export read it.
__device__ __forceinline__ void ring_target(CRun &R, const GLOBAL double *Uc, int x, int y, int t, double (&Ut)[4]) {
    const unsigned qp = (unsigned)R.qplane;
    const bool pre = R.tgt_pre != 0;
    const GLOBAL double *Ub = pre ? (const GLOBAL double *)R.P : Uc;
    const unsigned sb = pre ? (unsigned)R.rplane : qp;
#pragma unroll
    for (int c = 0; c < 4; ++c) Ut[c] = Ub[c * sb + (unsigned)t];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        bool on = s == XMIN ? x < 3 : s == XMAX ? x >= R.Nx - 3 : s == YMIN ? y < 3 : y >= R.Ny - 3;
        // (runs with a CBC (A) side always form their targets ahead: pre is set)
        if (on && !pre && R.bc[s] == BC_NRBC) lodi_add(R, Uc, s, x, y, t, Ut);
    }
}
template <int SRC, class S, class C>
__device__ __forceinline__ void nrbc_node(CRun &R, int par, int up, int x, int y, int t, C inv_scale) {
    double Ut[4];
    ring_target(R, (const GLOBAL double *)R.U[up], x, y, t, Ut);
    nrbc_fill<SRC, S, C>(R, pull_base<SRC, S>(R, par), x, y, inv_scale, Ut, t);
}

// ------------------------------------------------------------------------------------------
// step kernels
// ------------------------------------------------------------------------------------------
// Bulk tile b (logical, after the XCD remap) of a launch set.
template <class S, int TX>
__device__ __forceinline__ void bulk_tile(RunDev *const *__restrict__ runs,
                                          const int *__restrict__ prefix, int nruns, Sub ks, int b) {
    using C = typename Traits<S>::C;
    constexpr int TY = 256 / TX;
    constexpr int TI = TX == 64 ? 0 : (TX == 128 ? 1 : 2);
    const int j = find_run(prefix, nruns, b);
    CRun &R = run_of(runs, j);
    const int par = sub_par(R, ks);
    if (par < 0) return;
    const int tb = b - ((const CONSTANT int *)prefix)[j];
    const int ty = tb / R.tiles_x[TI], tx = tb - ty * R.tiles_x[TI];
    const int x = (R.fx0 / TX) * TX + tx * TX + (int)(threadIdx.x % TX);
    const int y = R.fy0 + ty * TY + (int)(threadIdx.x / TX);
    if (x < R.fx0 || x >= R.fx1 || y >= R.fy1) return;
    const K<C> k = load_k<C>(R);
    const GLOBAL S *src = (const GLOBAL S *)R.f[par];
    GLOBAL S *dst = (GLOBAL S *)R.f[par ^ 1];
    const long long plane = R.plane;
    const int pitch = R.pitch;
    // uniform base at the tile's first row; per-lane 32-bit byte offset inside the tile
    const int y0 = R.fy0 + ty * TY;
    const GLOBAL S *src0 = src + (long long)y0 * pitch;
    GLOBAL S *dst0 = dst + (long long)y0 * pitch;
    const unsigned off = (unsigned)((y - y0) * pitch + x) * (unsigned)sizeof(S);
    C g[NQ];
    static_for<0, NQ>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        const GLOBAL S *base = src0 + ((long long)i * plane - (ey_of(i) * pitch + ex_of(i)));
        g[i] = cvt_in(*LBM_AT(R, base, off, src, R.fsize), k.inv_scale);
    });
    const Mom<C> m = moments<C>(g, k);
    collide<false, S, C>(R, k, m, g, C(0), [&](auto ic, C out) {
        constexpr int i = decltype(ic)::value;
        // FP64/FP32: streaming store (the next reads of these lines are a step away); FP16 rows
        // of a wave are single cache lines and measure faster as ordinary stores
        if constexpr (sizeof(S) >= 4)
            __builtin_nontemporal_store(cvt_out(out, k.scale, (S *)nullptr),
                                        LBM_AT(R, dst0 + (long long)i * plane, off, dst, R.fsize));
        else
            *LBM_AT(R, dst0 + (long long)i * plane, off, dst, R.fsize) = cvt_out(out, k.scale, (S *)nullptr);
    });
}

template <class S, int TX>
__global__ __launch_bounds__(256) void k_bulk(RunDev *const *__restrict__ runs,
                                              const int *__restrict__ prefix, int nruns, Sub ks) {
    bulk_tile<S, TX>(runs, prefix, nruns, ks, xcd_swizzle(blockIdx.x, gridDim.x));
}

// Collision of a frame node (frame index t) from its post-stream, post-boundary populations g:
// BGK plus, on PML nodes, -sigma (e.grad Q + 2 fhat + sigma Q) (eq. PMLCOLL) with grad Q central
// and one-sided at the outermost layer of an open axis (eqs. FD-dx-*); the moments go to U.
// The BGK part and -2 sigma fhat are formed first, in place of g; Q at the node and its
// neighbours is then read a few populations at a time, every read of a group issued before its
// first use (the pointers are restrict-qualified so later groups may be read ahead of earlier
// stores): a handful of memory round trips per node instead of one per population.
// With BANDS (first step of a two-step pass) the node is written to the bands instead of a buffer:
// dnode in its band, and dnode2 if `two`, where it lies in both.
template <class S, class C, bool BANDS, bool STREAM, class Stride>
__device__ __forceinline__ void frame_collide(CRun &R, const K<C> &k, const C (&g)[NQ], int x, int y,
                                              int t, const GLOBAL C *__restrict__ Q,
                                              GLOBAL S *__restrict__ dnode, Stride plane,
                                              GLOBAL S *__restrict__ dnode2, Stride plane2, bool two,
                                              GLOBAL double *__restrict__ Un) {
    // FP64 streams to a buffer, which is next read a whole step later (frame launch, streaming /
    // ordinary stores: 1088^2 40.0 / 39.5 us, 4224^2 295 / 298); FP32 and FP16 do so in small sets
    // (1088^2 FP32 25.1 / 22.6, FP16 20.8 / 18.5, 4224^2 FP32 181 / 161; frame_streams has the
    // line).  The bands are read by the next kernel.
    auto put = [&](auto ic, C out) {
        constexpr int i = decltype(ic)::value;
        const S v = cvt_out(out, k.scale, (S *)nullptr);
        if constexpr (BANDS) {
            *LBM_IN(R, dnode + (Stride)i * plane, (GLOBAL S *)R.M, R.msize) = v;
            if (two) *LBM_IN(R, dnode2 + (Stride)i * plane2, (GLOBAL S *)R.M, R.msize) = v;
        } else {
            if constexpr (STREAM) __builtin_nontemporal_store(v, dnode + (long long)i * plane);
            else dnode[(long long)i * plane] = v;
        }
    };
    const unsigned qp = (unsigned)R.qplane;
    const Mom<C> m = moments<C>(g, k);
    if (R.has_q) {
        const QStencil<C> qs = q_stencil<C>(R, x, y, t);
        const unsigned ot = qs.ot, ox0 = qs.ox0, ox1 = qs.ox1, oy0 = qs.oy0, oy1 = qs.oy1;
        // sigma = 0 off the layer: the PML terms are then -0 * (finite) and leave BGK's bits
        const C s = (C)(R.W > 0 ? sigma_at(R, x, y) : 0.0);
        C h[NQ];
        collide<true, S, C>(R, k, m, g, s, [&](auto ic, C out) { h[decltype(ic)::value] = out; });
        constexpr int CH = sizeof(C) == 8 ? 4 : 12;   // populations per group of Q reads
        static_for<0, (NQ + CH - 1) / CH>([&](auto cc) {
            constexpr int c0 = decltype(cc)::value * CH;
            constexpr int c1 = c0 + CH < NQ ? c0 + CH : NQ;
            C v[c1 - c0][5];
            static_for<c0, c1>([&](auto ic) {
                constexpr int i = decltype(ic)::value, l = i - c0;
                const GLOBAL C *Qi = Q + (long long)i * qp;
                v[l][0] = *at(Qi, ot);
                if constexpr (ex_of(i) != 0) { v[l][1] = *at(Qi, ox0); v[l][2] = *at(Qi, ox1); }
                if constexpr (ey_of(i) != 0) { v[l][3] = *at(Qi, oy0); v[l][4] = *at(Qi, oy1); }
            });
            static_for<c0, c1>([&](auto ic) {
                constexpr int i = decltype(ic)::value, l = i - c0;
                put(ic, pml_gradient<i>(qs, v[l], h[i], s));
            });
        });
    } else {
        collide<false, S, C>(R, k, m, g, C(0), put);
    }
    Un[t] = R.rho0 + (double)m.drho;
    Un[qp + t] = R.u0x + (double)m.dux;
    Un[2 * qp + t] = R.u0y + (double)m.duy;
    Un[3 * qp + t] = R.T0 + (double)m.dT;
}

// Barrier that orders LDS accesses only: loads from memory stay in flight across it.
__device__ __forceinline__ void core_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Second step of a two-step pass on shell node ts (strip numbering of the REACH interior layers
// next to the frame): pull from the bands, BGK, into buffer `to`.
template <class S, class C>
__device__ __forceinline__ void shell_node(CRun &R, int to, const K<C> &k, int ts) {
    int x, y;
    strip_xy(R.fx1 - R.fx0, R.fy1 - R.fy0, REACH, REACH, REACH, REACH, ts, x, y);
    x = (int)LBM_GUARD(R, x + R.fx0, R.Nx);
    y = (int)LBM_GUARD(R, y + R.fy0, R.Ny);
    C g[NQ];
    gather_clamped<SRC_M, S, C>(R, (const GLOBAL S *)R.M, x, y, k.inv_scale, g);
    const Mom<C> m = moments<C>(g, k);
    GLOBAL S *dnode = (GLOBAL S *)R.f[to] + (long long)y * R.pitch + x;
    collide<false, S, C>(R, k, m, g, C(0), [&](auto ic, C out) {
        constexpr int i = decltype(ic)::value;
        dnode[(long long)i * R.plane] = cvt_out(out, k.scale, (S *)nullptr);
    });
}

// Two steps of the interior in one pass over memory.  A block sweeps a strip of CORE_X columns up
// H rows, CORE_R rows per turn, one row per wave: it forms the level between (n+1) of its row from
// the buffer, puts it in LDS, and forms level n+2 of the row REACH below from LDS.  Population i of
// a row is pulled D = e_y + REACH rows after it is formed, by the wave D further on: in the same
// turn or one of the next two.  Wave w keeps its row in slot w of every population, so a slot is
// written anew each turn; the waves that still need the row it held read it ahead of the turn's
// writes.  A turn is then: read the populations that come from earlier turns, barrier, form and
// write the row, barrier, read the others, form level n+2.  The next turn's loads go out between
// the two halves.  Only a row pulled two turns later (w + D >= 2 CORE_R) needs a second slot, used
// in turn with the first.
// That is 159 rows of LDS for D2Q37, 79.6 KiB in FP64, so a compute unit holds two tiles: the
// halves of one stream while the other computes.  (With e_y + REACH + CORE_R slots per
// population and one barrier a turn, one tile fits a unit; with 8 rows a turn, one tile of 8
// waves: its waves then load, compute and store together, and the times add: 169 and 177 us for
// the 1088^2 FP64 interior.)
// The tiles cover the interior off its outer REACH layers; level n+1 of the layers the frame and
// the shell pull from (depth < 2 REACH) goes to the bands.
constexpr int core_delay(int i) { return ey_of(i) + REACH; }
constexpr int core_base(int i) {   // first element of population i
    int n = 0;
    for (int j = 0; j < i; ++j) n += CORE_R + (core_delay(j) > CORE_R ? core_delay(j) - CORE_R : 0);
    return CORE_PAD + n * CORE_X;
}
static_assert(core_base(NQ) + CORE_PAD == core_lds_rows(LBM_INFO) * CORE_X + 2 * CORE_PAD, "LDS size");
static_assert(2 * REACH <= 2 * CORE_R - 2, "a row is pulled at most two turns later");
// Slot of wave w's row, of a turn of parity `odd`, in a population of delay D.
template <int D> __device__ __forceinline__ int core_slot(int w, int odd) {
    if constexpr (D > CORE_R) return w + D >= 2 * CORE_R && odd ? w + D - CORE_R : w;
    else return w;
}

// Rows of populations through a buffer resource: population i of a grid row sits i population rows
// past the row's start (the row layout), so an access is one scalar multiple of the population
// row's size, one per-lane offset and an immediate, and no 64-bit address per population: with
// those the FP32 tile spilled 81 scalar registers, which hold the equilibrium's constants now.  (What
// still spills: D2Q37 FP64 43 scalar registers, FP32 21 and 6 vector registers, 28 bytes a lane.)
// The resource ends with the rows it covers.
template <class S> struct Rows {
    __amdgpu_buffer_rsrc_t r;
    int row;          // bytes of a population row
};
template <class S>
__device__ __forceinline__ Rows<S> rows_at(GLOBAL S *first, int plane, int nrows) {
    int row = plane * (int)sizeof(S);
    asm volatile("" : "+s"(row));   // its multiples are formed at each use, not kept across the loop
    return {__builtin_amdgcn_make_buffer_rsrc((S *)first, 0, nrows * NQ * row, 0x00020000), row};
}
// element `dx` + off / sizeof(S) of population i of grid row k of the rows
template <int i, int k, int dx, class S>
__device__ __forceinline__ S row_load(const Rows<S> &a, unsigned off) {
    const int so = (k * NQ + i) * a.row;
    if constexpr (sizeof(S) == 8)
        return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(a.r, off + dx * 8, so, 0));
    else if constexpr (sizeof(S) == 4)
        return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(a.r, off + dx * 4, so, 0));
    else
        return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b16(a.r, off + dx * 2, so, 0));
}
// streaming store (the next reads of these lines are a pass away)
template <int i, class S>
__device__ __forceinline__ void row_store(const Rows<S> &a, unsigned off, S v) {
    const int so = i * a.row;
    if constexpr (sizeof(S) == 8) {
        typedef unsigned v2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(v2, v), a.r, off, so, 2);
    } else if constexpr (sizeof(S) == 4)
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), a.r, off, so, 2);
    else
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), a.r, off, so, 2);
}

template <class S>
__global__ __launch_bounds__(CORE_X *CORE_R, core_waves(LBM_INFO, (int)sizeof(S))) void k_core(RunDev *const *__restrict__ runs,
                                                         const int *__restrict__ prefix, int nruns,
                                                         Sub ks, int H) {
    using C = typename Traits<S>::C;
    __shared__ S lds[core_lds_rows(LBM_INFO) * CORE_X + 2 * CORE_PAD];
    const int b = xcd_swizzle(blockIdx.x, gridDim.x);
    const int j = find_run(prefix, nruns, b);
    CRun &R = run_of(runs, j);
    const int par = sub_par(R, ks);
    if (par < 0) return;
    const int tb = b - ((const CONSTANT int *)prefix)[j];
    const int chunk = tb / R.core_strips, strip = tb - chunk * R.core_strips;
    const int lane = (int)threadIdx.x & (CORE_X - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / CORE_X);
    const int r0 = R.fy0 + REACH + chunk * H, r1 = min(r0 + H, R.fy1 - REACH);
    constexpr int OUT = core_out(REACH, (int)sizeof(S));
    const int xs = core_x0(R.fx0, REACH, (int)sizeof(S)) + strip * OUT - REACH;   // first column of level n+1
    const int x = min(max(xs + lane, R.fx0), R.fx1 - 1);   // (lanes past the interior repeat its edge)
    const bool out2 = lane >= REACH && lane < REACH + OUT && xs + lane >= R.fx0 + REACH && xs + lane < R.fx1 - REACH;
    const K<C> k = load_k<C>(R);
    GLOBAL S *src = (GLOBAL S *)R.f[par];
    GLOBAL S *dst = (GLOBAL S *)R.f[par ^ 1];
    const int plane = (int)R.plane, pitch = NQ * plane;
    const unsigned off = (unsigned)x * (unsigned)sizeof(S), offl = off - REACH * (unsigned)sizeof(S);
    // columns and rows of level n+1 this block writes to the bands
    const int ox0 = strip == 0 ? R.fx0 : xs + REACH;
    const int ox1 = strip == R.core_strips - 1 ? R.fx1 : xs + REACH + OUT;
    const bool own_x = xs + lane >= ox0 && xs + lane < ox1;
    const int oy0 = chunk == 0 ? R.fy0 : r0, oy1 = r1 == R.fy1 - REACH ? R.fy1 : r1;
    const bool band_x = xs + lane < R.bL || xs + lane >= R.Nx - R.bR;
    const bool edge_strip = xs < R.bL || xs + CORE_X > R.Nx - R.bR;

    int y = r0 - REACH + w;
    const int yl = r1 + REACH;
    S gs[NQ];
    auto load = [&](int yy) {
        const Rows<S> a = rows_at<S>(src + (long long)(yy - REACH) * pitch, plane, 2 * REACH + 1);
        static_for<0, NQ>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            LBM_CHECK(R, (long long)(yy - ey_of(i)) * pitch + (long long)i * plane + x - ex_of(i), R.fsize);
            gs[i] = row_load<i, REACH - ey_of(i), REACH - ex_of(i)>(a, offl);
        });
    };
    if (y < yl) load(y);
    // FP32: the uniform pair terms (e_p . u0 and its square) are formed afresh at each use: kept
    // across the loop they take 36 registers
    auto fresh = [](K<C> c) {
        if constexpr (sizeof(C) == 4) asm volatile("" : "+s"(c.r0x), "+s"(c.r0y));
        return c;
    };
    const int turns = (r1 - r0 + 2 * REACH + CORE_R - 1) / CORE_R;
    for (int it = 0; it < turns; ++it, y += CORE_R) {
        const int r = y - REACH;
        const bool second = r >= r0 && r < r1;
        S h[NQ];
        const int odd = it & 1;
        // the populations of delay D, from this turn's rows (D <= w), the last turn's or, of the same
        // parity as this turn's, those of the turn before it
        auto read = [&](auto dc) {
            constexpr int D = decltype(dc)::value;
            const int from = core_slot<D>((w - D) & (CORE_R - 1), odd) * CORE_X + lane;
            static_for<0, NQ>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                if constexpr (core_delay(i) == D) h[i] = lds[core_base(i) + from - ex_of(i)];
            });
        };
        int mine[2 * REACH + 1];   // this row's place by delay
        static_for<0, 2 * REACH + 1>([&](auto dc) {
            constexpr int D = decltype(dc)::value;
            mine[D] = core_slot<D>(w, odd) * CORE_X + lane;
        });
        if (second)
            static_for<1, 2 * REACH + 1>([&](auto dc) {
                if (w < decltype(dc)::value) read(dc);
            });
        core_barrier();
        if (y < yl) {
            C g[NQ];
            static_for<0, NQ>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                g[i] = cvt_in(gs[i], k.inv_scale);
            });
            const Mom<C> m = moments<C>(g, k);
            collide<false, S, C>(R, fresh(k), m, g, C(0), [&](auto ic, C out) {
                constexpr int i = decltype(ic)::value;
                lds[core_base(i) + mine[core_delay(i)]] = cvt_out(out, k.scale, (S *)nullptr);
            });
            // the row's part in the bands, read back from LDS (this lane's own writes)
            const bool rows = y < R.bB || y >= R.Ny - R.bT;
            if ((rows || edge_strip) && y >= oy0 && y < oy1) {
                GLOBAL S *M = (GLOBAL S *)R.M;
                auto copy = [&](unsigned first, int stride) {
                    static_for<0, NQ>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        M[LBM_GUARD(R, first + (unsigned)(i * stride), R.msize)] = lds[core_base(i) + mine[core_delay(i)]];
                    });
                };
                if (rows && own_x) copy((unsigned)band_row(R, y) * (unsigned)(NQ * R.m_row) + (unsigned)x, R.m_row);
                if (own_x && band_x)
                    copy((unsigned)R.l_first + (unsigned)(y - R.gym) * (unsigned)(NQ * R.l_row) +
                             (unsigned)band_col(R, x), R.l_row);
            }
        }
        core_barrier();
        if (y + CORE_R < yl) load(y + CORE_R);
        if (second) {
            static_for<0, 2 * REACH + 1>([&](auto dc) {
                if (w >= decltype(dc)::value) read(dc);
            });
            C g[NQ];
            static_for<0, NQ>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                g[i] = cvt_in(h[i], k.inv_scale);
            });
            const Mom<C> m = moments<C>(g, k);
            const Rows<S> a = rows_at<S>(dst + (long long)r * pitch, plane, 1);
            if (out2)
                collide<false, S, C>(R, fresh(k), m, g, C(0), [&](auto ic, C out) {
                    constexpr int i = decltype(ic)::value;
                    LBM_CHECK(R, (long long)r * pitch + (long long)i * plane + x, R.fsize);
                    row_store<i, S>(a, off, cvt_out(out, k.scale, (S *)nullptr));
                });
        }
    }
}

// Phase B of a step on the frame: ring blocks take the post-boundary populations phase A stored
// in G; the frame blocks, which cover the frame off the ring, pull (periodic wrap, or eq.
// zg-bc's copy of x_f = clamp(x, 3, N-4) on open axes).  STEP: a single step, from buffer to
// buffer; the first step of a two-step pass, from the buffer to the bands; the second, from the
// bands to the other buffer, with the shell blocks after the frame blocks: the REACH layers of
// interior nodes next to the frame, which the two-step tiles leave out because their second step
// reads frame nodes of the first.
enum { STEP_ONE = 0, STEP_FIRST = 1, STEP_SECOND = 2 };

template <class S, int STEP, bool STREAM>
__global__ __launch_bounds__(256) void k_frame(RunDev *const *__restrict__ runs,
                                               const int *__restrict__ prefix, int nruns, Sub ks) {
    using C = typename Traits<S>::C;
    constexpr int SRC = STEP == STEP_SECOND ? SRC_M : SRC_F;
    const int b = blockIdx.x;
    const int j = find_run(prefix, nruns, b);
    CRun &R = run_of(runs, j);
    const int par = sub_par(R, ks);
    if (par < 0) return;
    const int tb = b - ((const CONSTANT int *)prefix)[j];
    const int rb = ring_blocks(R);
    const K<C> k = load_k<C>(R);
    int x, y, t;
    C g[NQ];
    if (tb < rb) {
        if ((int)threadIdx.x >= RING_BLOCK) return;
        const int tt = tb * RING_BLOCK + (int)threadIdx.x;
        if (tt >= R.ring_n) return;
        ring_xy(R, tt, x, y);
        t = (int)LBM_GUARD(R, tt, R.rplane);
        const GLOBAL C *G = (const GLOBAL C *)R.G;
        const unsigned rp = (unsigned)R.rplane;
#pragma unroll
        for (int i = 0; i < NQ; ++i) g[i] = G[i * rp + t];
    } else {
        const int fb = frame_block_count(R.ann_n);
        if (STEP == STEP_SECOND && tb - rb >= fb) {
            const int ts = (tb - rb - fb) * FRAME_BLOCK + (int)threadIdx.x;
            if (ts >= R.shell_n) return;
            shell_node<S, C>(R, par ^ 1, k, ts);
            return;
        }
        const int ta = frame_start(R, tb - rb) + (int)threadIdx.x;
        if (ta >= R.ann_n) return;
        ann_xy(R, ta, x, y);
        t = (int)LBM_GUARD(R, R.ann0 + ta, R.qplane);
        gather_clamped<SRC, S, C>(R, pull_base<SRC, S>(R, par), x, y, k.inv_scale, g);
    }
    const GLOBAL C *Q = (const GLOBAL C *)R.Q;
    GLOBAL double *Un = (GLOBAL double *)R.U[u_par(R, ks) ^ 1];
    if constexpr (STEP == STEP_FIRST) {
        // the rows of the y strips (and as far as they are pulled) in the row band, the columns of
        // the x strips in the column band off the y strips; near the corners in both
        GLOBAL S *M = (GLOBAL S *)R.M;
        const bool rows = y < R.bB || y >= R.Ny - R.bT;
        const bool cols = (x < R.bL || x >= R.Nx - R.bR) && y >= R.gym && y < R.Ny - R.gyp;
        const unsigned ra = (unsigned)band_row(R, y) * (unsigned)(NQ * R.m_row) + (unsigned)x;
        const unsigned ca = (unsigned)R.l_first + (unsigned)(y - R.gym) * (unsigned)(NQ * R.l_row) +
                            (unsigned)band_col(R, x);
        const unsigned pa = (unsigned)(rows ? R.m_row : R.l_row);
        frame_collide<S, C, true, STREAM, unsigned>(R, k, g, x, y, t, Q, M + (rows ? ra : ca), pa, M + ca,
                                            (unsigned)R.l_row, rows && cols, Un);
    } else {
        frame_collide<S, C, false, STREAM, long long>(R, k, g, x, y, t, Q,
                                              (GLOBAL S *)R.f[par ^ 1] + (long long)y * R.pitch + x,
                                              R.plane, (GLOBAL S *)nullptr, 0, false, Un);
    }
}

#if LBM_Q >= 17   // D2Q9 has fewer duos than waves
// Kernels whose 4 waves share 64 nodes: wave W of a block has the duos [D0, D1) of each node's
// populations (and wave 0 the rest population), kept in registers in the order of index(), the rest
// population first.  What a wave needs of all populations (the moments) it sums from LDS, where
// the waves lay their own.  Only the steps on a wave's own populations are compiled per wave
// (by_wave); all else is one code, so that the four waves fetch the same instructions.
template <int W> struct Share {
    static constexpr int D0 = NDUO * W / 4, D1 = NDUO * (W + 1) / 4;
    static constexpr bool REST = W == 0;
    static constexpr int N = 4 * (D1 - D0) + REST;
    static constexpr int index(int l) { return REST && l == 0 ? 0 : 1 + 4 * D0 + l - REST; }
    static constexpr int local(int i) { return i == 0 ? 0 : i - 1 - 4 * D0 + REST; }
};
constexpr int SHARE = 4 * ((NDUO + 3) / 4) > Share<0>::N ? 4 * ((NDUO + 3) / 4) : Share<0>::N;   // the most of a wave

template <class F> __device__ __forceinline__ void by_wave(int w, F &&f) {
    if (w == 0) f(Share<0>{});
    else if (w == 1) f(Share<1>{});
    else if (w == 2) f(Share<2>{});
    else f(Share<3>{});
}
template <class H, class C> __device__ __forceinline__ void share_put(C *lds, int lane, const C (&v)[SHARE]) {
    static_for<0, H::N>([&](auto lc) { lds[H::index(decltype(lc)::value) * SPLIT_BLOCK + lane] = v[decltype(lc)::value]; });
}
// A wave's populations of the equilibrium of one state, or of two: emit(i, t, ...), t as in relax().
template <class H, class C, class F>
__device__ __forceinline__ void share_eq(CRun &R, const K<C> &, const EqPoly<C> &q, F &&emit) {
    if constexpr (H::REST) emit(std::integral_constant<int, 0>{}, q.c[E0]);
    poly_duos<H::D0, H::D1>(q, emit);
}
template <class H, class C, class F>
__device__ __forceinline__ void share_eq(CRun &R, const K<C> &k, Eq<C> q, F &&emit) {
    if constexpr (H::REST) emit(std::integral_constant<int, 0>{}, feq_rest<C>(q, R));
    static_for<2 * H::D0, 2 * H::D1>([&](auto pc) {
        constexpr int p = decltype(pc)::value;
        if constexpr (p == 2 * H::D0 || PSH[p - 1] != PSH[p]) eq_shell<C, PSH[p]>(q);
        C fp, fm;
        eq_pair<C, p>(q, R, k, fp, fm);
        emit(std::integral_constant<int, 1 + 2 * p>{}, fp);
        emit(std::integral_constant<int, 2 + 2 * p>{}, fm);
    });
}
template <class H, class C, class F>
__device__ __forceinline__ void share_eq2(CRun &R, const K<C> &k, Eq<C> qa, Eq<C> qb, F &&emit) {
    if constexpr (H::REST) emit(std::integral_constant<int, 0>{}, feq_rest<C>(qa, R), feq_rest<C>(qb, R));
    if constexpr (H::D0 > 0 && PSH[2 * H::D0 - 1] == PSH[2 * H::D0]) {   // (feq2_pairs sets a shell at its first pair)
        eq_shell<C, PSH[2 * H::D0]>(qa);
        eq_shell<C, PSH[2 * H::D0]>(qb);
    }
    feq2_pairs<2 * H::D0, 2 * H::D1>(qa, qb, R, k, emit);
}

// The single step on the frame where its nodes leave the device idle: the waves of a block share the
// nodes, each pulling and colliding its populations with every Q it needs in flight at once; the
// sums are those of moments() in order, so the bits are those of k_frame.  There a lone wave
// issues at half rate and waits most of its time, so a node's chain of loads and arithmetic is what
// the launch takes.  By k_frame and here, us, D2Q37: FP64 120^2 13.2, 8.1; 190^2 13.4, 9.5; 340^2
// 15.0, 13.3; FP32 140^2 10.2, 7.7; 490^2 13.4, 12.4; FP16 140^2 9.9, 7.7; 490^2 12.2, 11.4.  D2Q17:
// FP64 340^2 9.3, 8.0; 490^2 10.7, 10.3; FP32 340^2 8.2, 7.1; 880^2 10.5, 10.3; FP16 490^2 8.2, 7.7.
template <class S>
__global__ __launch_bounds__(256) void k_frame_split(RunDev *const *__restrict__ runs,
                                                     const int *__restrict__ prefix, int nruns, Sub ks) {
    using C = typename Traits<S>::C;
    __shared__ C lds[NQ * SPLIT_BLOCK];
    const int b = blockIdx.x;
    const int j = find_run(prefix, nruns, b);
    CRun &R = run_of(runs, j);
    const int par = sub_par(R, ks);
    if (par < 0) return;
    const int tb = b - ((const CONSTANT int *)prefix)[j];
    const int rb = ring_blocks(R);
    const bool ring = tb < rb;
    const int lane = (int)threadIdx.x & (SPLIT_BLOCK - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / SPLIT_BLOCK);
    const int n = (ring ? tb : tb - rb) * SPLIT_BLOCK + lane, count = ring ? R.ring_n : R.ann_n;
    if (n - lane >= count) return;
    const int nn = min(n, count - 1);          // every wave of the block meets its barriers
    int x, y, t;
    if (ring) {
        ring_xy(R, nn, x, y);
        t = (int)LBM_GUARD(R, nn, R.rplane);
    } else {
        ann_xy(R, nn, x, y);
        t = (int)LBM_GUARD(R, R.ann0 + nn, R.qplane);
    }
    const K<C> k = load_k<C>(R);
    const GLOBAL S *src = (const GLOBAL S *)R.f[par];
    const Pull from = pull_from<SRC_F>(R, x, y);
    const GLOBAL C *__restrict__ Q = (const GLOBAL C *)R.Q, *__restrict__ G = (const GLOBAL C *)R.G;
    GLOBAL S *__restrict__ dnode = (GLOBAL S *)R.f[par ^ 1] + (long long)y * R.pitch + x;
    const unsigned qp = (unsigned)R.qplane, rp = (unsigned)R.rplane;
    QStencil<C> qs{};
    C s = C(0);
    if (R.has_q) {
        qs = q_stencil<C>(R, x, y, t);
        s = (C)(R.W > 0 ? sigma_at(R, x, y) : 0.0);
    }
    C g[SHARE], v[SHARE][5];
    by_wave(w, [&](auto h) {
        using H = decltype(h);
        if (ring)
            static_for<0, H::N>([&](auto lc) { g[decltype(lc)::value] = G[H::index(decltype(lc)::value) * rp + t]; });
        else
            static_for<0, H::N>([&](auto lc) {
                constexpr int l = decltype(lc)::value;
                g[l] = pull_one<SRC_F, S, C, H::index(l)>(R, src, from, k.inv_scale);
            });
        if (R.has_q)
            static_for<0, H::N>([&](auto lc) {
                constexpr int l = decltype(lc)::value, i = H::index(l);
                const GLOBAL C *Qi = Q + (long long)i * qp;
                v[l][0] = *at(Qi, qs.ot);
                if constexpr (ex_of(i) != 0) { v[l][1] = *at(Qi, qs.ox0); v[l][2] = *at(Qi, qs.ox1); }
                if constexpr (ey_of(i) != 0) { v[l][3] = *at(Qi, qs.oy0); v[l][4] = *at(Qi, qs.oy1); }
            });
        share_put<H>(lds, lane, g);
    });
    core_barrier();
    const Mom<C> m = moments_streamed<NPAIR, C>(
        [&](auto ic) { return lds[decltype(ic)::value * SPLIT_BLOCK + lane]; }, k);
    if (n >= count) return;
    const auto eq = [&] {
        if constexpr (std::is_same<S, double>::value) return poly_coef<C>(R, m, k);
        else return eq_coef<C>(m.drho, m.dux, m.duy, m.dT, k);
    }();
    by_wave(w, [&](auto h) {
        using H = decltype(h);
        auto put = [&](auto ic, C out) {
            const S o = cvt_out(out, k.scale, (S *)nullptr);
            dnode[(long long)decltype(ic)::value * R.plane] = o;
        };
        if (R.has_q)
            share_eq<H>(R, k, eq, [&](auto ic, C f) {
                constexpr int i = decltype(ic)::value, l = H::local(i);
                put(ic, pml_gradient<i>(qs, v[l], relax<true, i, S, C>(g[l], f, k.omega, s), s));
            });
        else
            share_eq<H>(R, k, eq, [&](auto ic, C f) {
                constexpr int i = decltype(ic)::value;
                put(ic, relax<false, i, S, C>(g[H::local(i)], f, k.omega, C(0)));
            });
        if constexpr (H::REST) {
            GLOBAL double *Un = (GLOBAL double *)R.U[u_par(R, ks) ^ 1];
            Un[t] = R.rho0 + (double)m.drho;
            Un[qp + t] = R.u0x + (double)m.dux;
            Un[2 * qp + t] = R.u0y + (double)m.duy;
            Un[3 * qp + t] = R.T0 + (double)m.dT;
        }
    });
}
#endif

// PML auxiliary update Q += (fhat^n + fhat^{n+1}) / 2 at frame node t (eq. PMLQ, trapezoid rule),
// fhat^n from the moment strip of the last level, fhat^{n+1} from m, the moments of g^{n+1}.  Q is
// read a few pairs at a time (each group's reads issued together, the groups kept apart), so the
// update runs in few registers.
template <class C>
__device__ __forceinline__ void q_update(CRun &R, int up, const K<C> &k0, const Mom<C> &m, int t) {
    constexpr bool POLY = sizeof(C) == 8;   // FP64 storage
    // the uniform pair terms (e_p . u0 and its square) are formed afresh here: shared with the
    // ring fill's, they would stay live across it
    K<C> k = k0;
    if constexpr (!POLY) asm volatile("" : "+s"(k.r0x), "+s"(k.r0y));
    const GLOBAL double *Uc = (const GLOBAL double *)R.U[up];
    const unsigned qp = (unsigned)R.qplane;
    GLOBAL C *Q = (GLOBAL C *)R.Q;
    const double r0 = Uc[t], ux0 = Uc[qp + t], uy0 = Uc[2 * qp + t], T0 = Uc[3 * qp + t];
    const unsigned ot = (unsigned)LBM_GUARD(R, t, R.qplane) * (unsigned)sizeof(C);
    const Mom<C> m0{(C)(r0 - R.rho0), (C)(ux0 - R.u0x), (C)(uy0 - R.u0y), (C)(T0 - R.T0), C(0)};
    Eq<C> q1, q0;
    EqPoly<C> e;
    if constexpr (POLY) {   // fhat^n + fhat^{n+1}: one evaluation of the sum of their coefficients
        e = poly_coef<C>(R, m0, k);
        __builtin_amdgcn_sched_barrier(0);
        poly_add<1, C>(e, R, m, k);
        __builtin_amdgcn_sched_barrier(0);
    } else {
        q1 = eq_coef<C>(m.drho, m.dux, m.duy, m.dT, k);
        q0 = eq_coef<C>(m0.drho, m0.dux, m0.duy, m0.dT, k);
    }
    {
        const C q = *at(Q, ot);
        if constexpr (POLY) *at(Q, ot) = q + C(0.5 * SHELL_W[0]) * e.c[E0];
        else *at(Q, ot) = q + C(0.5) * (feq_rest<C>(q0, R) + feq_rest<C>(q1, R));
    }
    constexpr int PC = 4;   // pairs per group of Q reads
    static_for<0, (NPAIR + PC - 1) / PC>([&](auto cc) {
        constexpr int P0 = decltype(cc)::value * PC;
        constexpr int P1 = P0 + PC < NPAIR ? P0 + PC : NPAIR;
        C Qv[2 * (P1 - P0)];
        static_for<0, 2 * (P1 - P0)>([&](auto lc) {
            constexpr int l = decltype(lc)::value;
            Qv[l] = *at(Q + (long long)(1 + 2 * P0 + l) * qp, ot);
        });
        if constexpr (POLY)
            poly_duos<P0 / 2, P1 / 2>(e, [&](auto ic, C f) {
                constexpr int i = decltype(ic)::value;
                *at(Q + (long long)i * qp, ot) = Qv[i - 1 - 2 * P0] + C(0.5 * weight_of<i>()) * f;
            });
        else
            feq2_pairs<P0, P1>(q1, q0, R, k, [&](auto ic, C fe1, C fe0) {
                constexpr int i = decltype(ic)::value;
                *at(Q + (long long)i * qp, ot) = Qv[i - 1 - 2 * P0] + C(0.5) * (fe0 + fe1);
            });
        __builtin_amdgcn_sched_barrier(0);
    });
}

// Block b of the phase-A class: ring blocks form the characteristic fill of the ring (into G)
// and, on PML nodes, update Q from it; frame blocks update Q of the PML nodes off the ring from
// their pull.
template <class S, int SRC>
__device__ __forceinline__ void phase_a_block(RunDev *const *__restrict__ runs,
                                              const int *__restrict__ prefix, int nruns, Sub ks, int b) {
    using C = typename Traits<S>::C;
    const int j = find_run(prefix, nruns, b);
    CRun &R = run_of(runs, j);
    const int par = sub_par(R, ks);
    if (par < 0) return;
    const int up = u_par(R, ks);
    const int tb = b - ((const CONSTANT int *)prefix)[j];
    const int rb = ring_blocks(R);
    const K<C> k = load_k<C>(R);
    int x, y, t;
    Mom<C> m;
    if (tb < rb) {
        if ((int)threadIdx.x >= RING_BLOCK) return;
        const int tt = tb * RING_BLOCK + (int)threadIdx.x;
        if (tt >= R.ring_n) return;
        ring_xy(R, tt, x, y);
        t = (int)LBM_GUARD(R, tt, R.rplane);
        nrbc_node<SRC, S, C>(R, par, up, x, y, t, k.inv_scale);
        if (!R.has_q || !in_q(R, x, y)) return;
        // the moments of the filled populations, read back from G (this thread's own stores);
        // the opaque index makes the reads form their addresses afresh rather than keep those
        // of the stores live
        int tr = t;
        asm volatile("" : "+v"(tr) : : "memory");
        const GLOBAL C *G = (const GLOBAL C *)R.G;
        const unsigned rp = (unsigned)R.rplane;
        m = moments_streamed<6, C>([&](auto ic) { return G[decltype(ic)::value * rp + tr]; }, k);
    } else {
        const int ta = frame_start(R, tb - rb) + (int)threadIdx.x;
        if (!R.has_q || ta >= R.ann_n) return;
        ann_xy(R, ta, x, y);
        if (!in_q(R, x, y)) return;
        t = (int)LBM_GUARD(R, R.ann0 + ta, R.qplane);
        C g[NQ];
        gather_clamped<SRC, S, C>(R, pull_base<SRC, S>(R, par), x, y, k.inv_scale, g);
        m = moments<C>(g, k);
    }
    __builtin_amdgcn_sched_barrier(0);
    q_update<C>(R, up, k, m, t);
}

#if LBM_Q >= 17
// Phase A of block b where its nodes leave the device idle: as k_frame_split, the 4 waves of a block
// share 64 nodes, each pulling, filling and updating its populations, and what every wave needs
// of all of them (the moments of the pull, then of the fill) is summed from LDS in the order of
// moments(), so the bits are those of phase_a_block.  There a lone wave's groups of loads (the pull
// twice, the fill read back, Q) take some 25 trips to memory one after the other, here four.  What
// bounds it now is the FP64 arithmetic of the moments and of the two equilibria, which every wave
// forms.  The fused launch by phase_a_block and here, us, D2Q37: FP64 120^2 12.8, 10.6; 190^2 13.8,
// 12.5; 340^2 22.0, 20.4; FP32 140^2 14.7, 11.6; 490^2 24.1, 21.1; FP16 140^2 16.7, 11.9; 490^2
// 21.7, 16.0.  D2Q17: FP64 340^2 12.7, 11.5; 490^2 18.6, 17.8; FP32 340^2 10.0, 9.5; 640^2 16.7,
// 15.2; FP16 490^2 12.2, 11.5.
template <class S, int SRC>
__device__ __forceinline__ void phase_a_split(RunDev *const *__restrict__ runs, const int *__restrict__ prefix,
                                              int nruns, Sub ks, int b, typename Traits<S>::C *lds) {
    using C = typename Traits<S>::C;
    constexpr bool POLY = std::is_same<S, double>::value;
    const int j = find_run(prefix, nruns, b);
    CRun &R = run_of(runs, j);
    const int par = sub_par(R, ks);
    if (par < 0) return;
    const int up = u_par(R, ks);
    const int tb = b - ((const CONSTANT int *)prefix)[j];
    const int rb = ring_blocks(R);
    const bool ring = tb < rb;
    const int lane = (int)threadIdx.x & (SPLIT_BLOCK - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / SPLIT_BLOCK);
    const int n = (ring ? tb : tb - rb) * SPLIT_BLOCK + lane, count = ring ? R.ring_n : R.ann_n;
    if (n - lane >= count || (!ring && !R.has_q)) return;
    const int nn = min(n, count - 1);
    int x, y, t;
    if (ring) {
        ring_xy(R, nn, x, y);
        t = (int)LBM_GUARD(R, nn, R.rplane);
    } else {
        ann_xy(R, nn, x, y);
        t = (int)LBM_GUARD(R, R.ann0 + nn, R.qplane);
    }
    const bool on = n < count, upd = on && R.has_q && in_q(R, x, y);
    if (!ring && __builtin_amdgcn_ballot_w64(upd) == 0) return;   // the same nodes in every wave
    const K<C> k = load_k<C>(R);
    const GLOBAL S *src = pull_base<SRC, S>(R, par);
    const Pull from = pull_from<SRC>(R, x, y);
    GLOBAL C *Q = (GLOBAL C *)R.Q;
    GLOBAL C *G = (GLOBAL C *)R.G;
    const GLOBAL double *Uc = (const GLOBAL double *)R.U[up];
    const unsigned qp = (unsigned)R.qplane, rp = (unsigned)R.rplane;
    const unsigned ot = (unsigned)t * (unsigned)sizeof(C);
    C g[SHARE], q[SHARE];
    double u[4] = {};
    by_wave(w, [&](auto h) {
        using H = decltype(h);
        static_for<0, H::N>([&](auto lc) {
            constexpr int l = decltype(lc)::value;
            g[l] = pull_one<SRC, S, C, H::index(l)>(R, src, from, k.inv_scale);
        });
        if (R.has_q)
            static_for<0, H::N>([&](auto lc) {
                q[decltype(lc)::value] = *at(Q + (long long)H::index(decltype(lc)::value) * qp, ot);
            });
        share_put<H>(lds, lane, g);
    });
    if (R.has_q)
        for (int c = 0; c < 4; ++c) u[c] = Uc[c * qp + t];
    auto pulled = [&](auto ic) { return lds[decltype(ic)::value * SPLIT_BLOCK + lane]; };
    if (ring) {
        double Ut[4];
        ring_target(R, Uc, x, y, t, Ut);
        core_barrier();
        const K<double> kd = load_k<double>(R);
        const Mom<double> mf = moments_streamed<6, double>([&](auto ic) { return (double)pulled(ic); }, kd);
        const Mom<double> mt{Ut[0] - R.rho0, Ut[1] - R.u0x, Ut[2] - R.u0y, Ut[3] - R.T0, 0.0};
        if constexpr (POLY) {
            EqPoly<double> e = poly_coef<double>(R, mt, kd);
            poly_add<-1, double>(e, R, mf, kd);
            core_barrier();   // every wave has read the pull
            by_wave(w, [&](auto h) {
                using H = decltype(h);
                share_eq<H>(R, kd, e, [&](auto ic, double f) {
                    constexpr int i = decltype(ic)::value, l = H::local(i);
                    g[l] = (C)((double)g[l] + weight_of<i>() * f);
                    if (on) G[i * rp + t] = g[l];
                });
                share_put<H>(lds, lane, g);
            });
        } else {
            const Eq<double> ef = eq_coef<double>(mf.drho, mf.dux, mf.duy, mf.dT, kd);
            const Eq<double> et = eq_coef<double>(mt.drho, mt.dux, mt.duy, mt.dT, kd);
            core_barrier();
            by_wave(w, [&](auto h) {
                using H = decltype(h);
                share_eq2<H>(R, kd, et, ef, [&](auto ic, double ft, double ff) {
                    constexpr int i = decltype(ic)::value, l = H::local(i);
                    g[l] = (C)((double)g[l] + (ft - ff));
                    if (on) G[i * rp + t] = g[l];
                });
                share_put<H>(lds, lane, g);
            });
        }
        if (!R.has_q) return;
    }
    core_barrier();
    const Mom<C> m = moments_streamed<6, C>(pulled, k);
    if (!upd) return;
    const Mom<C> m0{(C)(u[0] - R.rho0), (C)(u[1] - R.u0x), (C)(u[2] - R.u0y), (C)(u[3] - R.T0), C(0)};
    if constexpr (POLY) {
        EqPoly<C> e = poly_coef<C>(R, m0, k);
        poly_add<1, C>(e, R, m, k);
        by_wave(w, [&](auto h) {
            using H = decltype(h);
            share_eq<H>(R, k, e, [&](auto ic, C f) {
                constexpr int i = decltype(ic)::value;
                *at(Q + (long long)i * qp, ot) = q[H::local(i)] + C(0.5 * weight_of<i>()) * f;
            });
        });
    } else {
        const Eq<C> q1 = eq_coef<C>(m.drho, m.dux, m.duy, m.dT, k);
        const Eq<C> q0 = eq_coef<C>(m0.drho, m0.dux, m0.duy, m0.dT, k);
        by_wave(w, [&](auto h) {
            using H = decltype(h);
            share_eq2<H>(R, k, q1, q0, [&](auto ic, C fe1, C fe0) {
                constexpr int i = decltype(ic)::value;
                *at(Q + (long long)i * qp, ot) = q[H::local(i)] + C(0.5) * (fe0 + fe1);
            });
        });
    }
}
#endif

// Phase A of a step (eq. PMLQ on the Q region; the characteristic fill of the ring).
template <class S, int SRC>
__global__ __launch_bounds__(256) void k_phase_a(RunDev *const *__restrict__ runs,
                                                 const int *__restrict__ prefix, int nruns, Sub ks) {
    phase_a_block<S, SRC>(runs, prefix, nruns, ks, blockIdx.x);
}

// Phase A and the bulk tiles of a step in one launch: h bulk tiles, the nA phase-A blocks, then
// the other nB - h bulk tiles.  The latency-bound phase-A waves run beside streaming tiles; the
// tiles after them keep them off the grid's tail, the tiles before them evict less of what the
// frame kernel then reads.  nA and h are multiples of 8, so every block keeps its XCD map.  Both
// paths share one register budget, held at 4 waves per SIMD (128 VGPRs) by the low-register
// boundary code, the branch-light block dispatch and the occupancy target.
template <class S, int TX>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_phase_a_bulk(RunDev *const *__restrict__ runs,
                                                      const int *__restrict__ preA, int nA,
                                                      const int *__restrict__ preB, int nB, int h,
                                                      int nruns, Sub ks) {
    const int b = blockIdx.x;
    const int pa = b - h;   // blocks [h, h + nA) are phase A; the tiles before and after them
    if ((unsigned)pa < (unsigned)nA) phase_a_block<S, SRC_F>(runs, preA, nruns, ks, pa);
    else bulk_tile<S, TX>(runs, preB, nruns, ks, xcd_swizzle(pa < 0 ? b : b - nA, nB));
}

#if LBM_Q >= 17
// The same grid for small sets, with the phase-A blocks of phase_a_split.  Its waves run alone or in
// twos on a SIMD and take up to 256 VGPRs (at 128 they spill: 340^2 D2Q37 FP64 29.2 us against 20.4).
template <class S, int TX>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_small_step(RunDev *const *__restrict__ runs,
                                                      const int *__restrict__ preA, int nA,
                                                      const int *__restrict__ preB, int nB, int h,
                                                      int nruns, Sub ks) {
    __shared__ typename Traits<S>::C lds[NQ * SPLIT_BLOCK];
    const int b = blockIdx.x;
    const int pa = b - h;
    if ((unsigned)pa < (unsigned)nA) phase_a_split<S, SRC_F>(runs, preA, nruns, ks, pa, lds);
    else bulk_tile<S, TX>(runs, preB, nruns, ks, xcd_swizzle(pa < 0 ? b : b - nA, nB));
}
#endif

// End of a batch of n steps in which the population buffers changed roles `flips` times: each run
// advances by the sub-steps it was active for, min(n, limit - step).  A run's limit never falls
// inside a two-step pass, so a run that stopped within the batch stopped among single steps after
// it, or the batch holds none.
__global__ void k_advance(RunDev *const *runs, int nruns, int n, int flips) {
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nruns) return;
    RunDev *R = runs[j];
    long long a = R->limit - R->step;
    a = a < 0 ? 0 : (a > n ? n : a);
    R->step += a;
    R->par ^= (int)(a == n ? flips : a) & 1;
}

// Debug canary: before the step kernels of sub-step ks, every buffer that a step writes in full
// -- the destination populations, the new moment strips, and the ring's characteristic fill G
// and targets P -- is filled with NaN in its own type.  A node or component that the step leaves
// unwritten and a later kernel reads then carries NaN into the result.  A two-step pass fills the
// destination buffer and the bands before its first step, U, G and P before each.
enum { POISON_ONE = 0, POISON_FIRST = 1, POISON_SECOND = 2 };
template <class S>
__global__ __launch_bounds__(256) void k_poison(RunDev *const *runs, Sub ks, int what) {
    using C = typename Traits<S>::C;
    CRun &R = run_of(runs, blockIdx.y);
    const int par = sub_par(R, ks);
    if (par < 0) return;
    const long long t0 = (long long)blockIdx.x * 256 + threadIdx.x, st = (long long)gridDim.x * 256;
    const S ns = (S)__builtin_nanf("");
    if (what != POISON_SECOND) {
        GLOBAL S *f = (GLOBAL S *)R.f[par ^ 1];
        for (long long i = t0; i < R.fsize; i += st) f[i] = ns;
    }
    if (what == POISON_FIRST) {
        GLOBAL S *M = (GLOBAL S *)R.M;
        for (long long i = t0; i < R.msize; i += st) M[i] = ns;
    }
    GLOBAL double *U = (GLOBAL double *)R.U[u_par(R, ks) ^ 1];
    for (long long i = t0; i < 4 * R.qplane; i += st) U[i] = __builtin_nan("");
    if (R.ring_n > 0 && R.G) {
        GLOBAL C *G = (GLOBAL C *)R.G;
        for (long long i = t0; i < (long long)NQ * R.rplane; i += st) G[i] = (C)__builtin_nanf("");
    }
    if (R.ring_n > 0 && R.P) {
        GLOBAL double *P = (GLOBAL double *)R.P;
        for (long long i = t0; i < 4 * R.rplane; i += st) P[i] = __builtin_nan("");
    }
}

__global__ void k_set_limit(RunDev *run, long long limit) {
    if (threadIdx.x == 0) run->limit = limit;
}

__global__ void k_set_limits(RunDev *const *runs, const long long *limits, int n) {
    int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < n) runs[j]->limit = limits[j];
}

// ------------------------------------------------------------------------------------------
// init, export, checks, reductions
// ------------------------------------------------------------------------------------------
template <class S>
__global__ __launch_bounds__(256) void k_init(RunDev *Rw, const double *rho, const double *ux,
                                              const double *uy, const double *T, float *absmax) {
    using C = typename Traits<S>::C;
    CRun &R = *(CRun *)Rw;
    __shared__ float red[256];
    const int n = blockIdx.x * 256 + threadIdx.x;
    const int nn = R.Nx * R.Ny;
    float mx = 0.0f;
    if (n < nn) {
        const int y = n / R.Nx, x = n - y * R.Nx;
        const K<C> k = load_k<C>(R);
        const Mom<C> m{(C)(rho[n] - R.rho0), (C)(ux[n] - R.u0x), (C)(uy[n] - R.u0y), (C)(T[n] - R.T0), C(0)};
        GLOBAL S *dst = (GLOBAL S *)R.f[0];
        const long long idx = (long long)y * R.pitch + x, plane = R.plane;
        auto take = [&](auto ic, C fe) {
            constexpr int i = decltype(ic)::value;
            if (absmax) mx = fmaxf(mx, fabsf((float)fe));
            else dst[(long long)i * plane + idx] = cvt_out(fe, k.scale, (S *)nullptr);
        };
        if constexpr (std::is_same<S, double>::value)
            for_each_poly<C>(R, m, k, [&](auto ic, C t) { take(ic, C(weight_of<decltype(ic)::value>()) * t); });
        else
            for_each_feq<C>(eq_coef<C>(m.drho, m.dux, m.duy, m.dT, k), R, k, take);
        if (!absmax) {
            int t = fidx(R, x, y);
            if (t >= 0) {
                const long long qp = R.qplane;
                for (int c = 0; c < 2; ++c) {
                    GLOBAL double *U = (GLOBAL double *)R.U[c];
                    U[t] = rho[n];
                    U[qp + t] = ux[n];
                    U[2 * qp + t] = uy[n];
                    U[3 * qp + t] = T[n];
                }
            }
        }
    }
    if (absmax) {
        red[threadIdx.x] = mx;
        __syncthreads();
        for (int s = 128; s > 0; s >>= 1) {
            if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
            __syncthreads();
        }
        if (threadIdx.x == 0) absmax[blockIdx.x] = red[0];
    }
}

// Moments of node (x, y) at the current step (post-stream, post-boundary): re-pull from the
// previous buffer with the previous moment strips; after 0 steps, moments of f*(0).
template <class S, class C>
__device__ __forceinline__ Mom<C> state_moments(CRun &R, int x, int y, const K<C> &k) {
    C g[NQ];
    if (R.step == 0) {
        const GLOBAL S *src = (const GLOBAL S *)R.f[R.par];
        const long long idx = (long long)y * R.pitch + x;
#pragma unroll
        for (int i = 0; i < NQ; ++i) g[i] = cvt_in(src[(long long)i * R.plane + idx], k.inv_scale);
    } else {
        const GLOBAL S *src = (const GLOBAL S *)R.f[R.par ^ 1];
        if (in_ring(R, x, y)) {   // ring: G, refreshed by the caller for this level
            const GLOBAL C *G = (const GLOBAL C *)R.G;
            const unsigned rp = (unsigned)R.rplane, r = (unsigned)ridx(R, x, y);
#pragma unroll
            for (int i = 0; i < NQ; ++i) g[i] = G[i * rp + r];
        } else {
            gather_clamped<SRC_F, S, C>(R, src, x, y, k.inv_scale, g);
        }
    }
    return moments<C>(g, k);
}

template <class S>
__global__ __launch_bounds__(256) void k_moments(RunDev *Rw, double *rho, double *ux, double *uy,
                                                 double *T) {
    using C = typename Traits<S>::C;
    CRun &R = *(CRun *)Rw;
    const int n = blockIdx.x * 256 + threadIdx.x;
    if (n >= R.Nx * R.Ny) return;
    const int y = n / R.Nx, x = n - y * R.Nx;
    const K<C> k = load_k<C>(R);
    Mom<C> m = state_moments<S, C>(R, x, y, k);
    if (rho) rho[n] = R.rho0 + (double)m.drho;
    if (ux) ux[n] = R.u0x + (double)m.dux;
    if (uy) uy[n] = R.u0y + (double)m.duy;
    if (T) T[n] = R.T0 + (double)m.dT;
}

// Populations and PML field to float64 planes of the whole grid, one population per block row: a
// thread that goes through the populations leaves a small grid's copy to a few lone waves (104^2
// D2Q37 FP64: 16.8 and 12.4 us, by rows 3.8 and 3.5).
template <class S>
__global__ __launch_bounds__(256) void k_export_f(RunDev *Rw, const double *fbar, double *out) {
    using C = typename Traits<S>::C;
    CRun &R = *(CRun *)Rw;
    const int n = blockIdx.x * 256 + threadIdx.x;
    const int nn = R.Nx * R.Ny;
    if (n >= nn) return;
    const int y = n / R.Nx, x = n - y * R.Nx;
    const K<C> k = load_k<C>(R);
    const GLOBAL S *src = (const GLOBAL S *)R.f[R.par];
    const long long idx = (long long)y * R.pitch + x;
    const int i = blockIdx.y;
    out[(long long)i * nn + n] = fbar[i] + (double)cvt_in(src[(long long)i * R.plane + idx], k.inv_scale);
}

template <class S>
__global__ __launch_bounds__(256) void k_export_q(RunDev *Rw, double *out) {
    using C = typename Traits<S>::C;
    CRun &R = *(CRun *)Rw;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= R.ann0 + R.ann_n || (t >= R.ring_n && t < R.ann0)) return;   // past the end; the gap
    int x, y;
    frame_xy(R, t, x, y);
    const long long nn = (long long)R.Nx * R.Ny;
    const GLOBAL C *Q = (const GLOBAL C *)R.Q;
    const int i = blockIdx.y;
    out[i * nn + (long long)y * R.Nx + x] = (double)Q[i * R.qplane + t];
}

template <class S>
__global__ __launch_bounds__(256) void k_check(RunDev *Rw, int *flag) {
    using C = typename Traits<S>::C;
    CRun &R = *(CRun *)Rw;
    const int n = blockIdx.x * 256 + threadIdx.x;
#ifdef LBM_BOUNDS
    if (n == 0 && R.oob) atomicOr(flag, 2);   // an index out of range since the run was set up
#endif
    if (n >= R.Nx * R.Ny) return;
    const int y = n / R.Nx, x = n - y * R.Nx;
    const K<C> k = load_k<C>(R);
    const GLOBAL S *src = (const GLOBAL S *)R.f[R.par];
    const long long idx = (long long)y * R.pitch + x;
    C g[NQ];
    bool bad = false;
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        g[i] = cvt_in(src[(long long)i * R.plane + idx], k.inv_scale);
        bad |= !isfinite((double)g[i]);
    }
    Mom<C> m = moments<C>(g, k);
    double rho = R.rho0 + (double)m.drho, T = R.T0 + (double)m.dT;
    bad |= !(rho > 0.0) || !(T > 0.0) || !isfinite(rho) || !isfinite(T);
    if (bad) atomicOr(flag, 1);
}

// Reflection-error sums of one bulk row per block, fixed order (strided per thread, then a
// tree in LDS): partials[3*row + z].
__global__ __launch_bounds__(256) void k_err_rows(const double *rho, const double *ux,
                                                  const double *T, int Nx, int x0, int y0, int lx,
                                                  const double *rr, const double *ru,
                                                  const double *rt, double *partials) {
    __shared__ double red[3][256];
    const int row = blockIdx.x;
    double s[3] = {0.0, 0.0, 0.0};
    for (int xb = threadIdx.x; xb < lx; xb += 256) {
        long long n = (long long)(row + y0) * Nx + (xb + x0), m = (long long)row * lx + xb;
        double a = (rho[n] - rr[m]) / rr[m], b = (ux[n] - ru[m]) / ru[m], c = (T[n] - rt[m]) / rt[m];
        s[0] += a * a; s[1] += b * b; s[2] += c * c;
    }
    for (int z = 0; z < 3; ++z) red[z][threadIdx.x] = s[z];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int z = 0; z < 3; ++z) red[z][threadIdx.x] += red[z][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 3) partials[3 * row + threadIdx.x] = red[threadIdx.x][0];
}

// The reflection-error sums of k_err_rows taken straight from the run's state (the moments of
// state_moments, formed as k_moments writes them): the same values, the same order, so the same
// bits as k_moments followed by k_err_rows.  One bulk row per block; refs are bulk-sized.
template <class S>
__global__ __launch_bounds__(256) void k_err_rows_state(RunDev *Rw, int x0, int y0, int lx,
                                                        const double *rr, const double *ru,
                                                        const double *rt, double *partials) {
    using C = typename Traits<S>::C;
    CRun &R = *(CRun *)Rw;
    __shared__ double red[3][256];
    const int row = blockIdx.x;
    const K<C> k = load_k<C>(R);
    double s[3] = {0.0, 0.0, 0.0};
    for (int xb = threadIdx.x; xb < lx; xb += 256) {
        const Mom<C> m = state_moments<S, C>(R, xb + x0, row + y0, k);
        const double rho = R.rho0 + (double)m.drho, ux = R.u0x + (double)m.dux, T = R.T0 + (double)m.dT;
        const long long q = (long long)row * lx + xb;
        double a = (rho - rr[q]) / rr[q], b = (ux - ru[q]) / ru[q], c = (T - rt[q]) / rt[q];
        s[0] += a * a; s[1] += b * b; s[2] += c * c;
    }
    for (int z = 0; z < 3; ++z) red[z][threadIdx.x] = s[z];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int z = 0; z < 3; ++z) red[z][threadIdx.x] += red[z][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 3) partials[3 * row + threadIdx.x] = red[threadIdx.x][0];
}

__global__ __launch_bounds__(256) void k_err_final(const double *partials, int nrows, double *out) {
    __shared__ double red[3][256];
    double s[3] = {0.0, 0.0, 0.0};
    for (int r = threadIdx.x; r < nrows; r += 256)
        for (int z = 0; z < 3; ++z) s[z] += partials[3 * r + z];
    for (int z = 0; z < 3; ++z) red[z][threadIdx.x] = s[z];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int z = 0; z < 3; ++z) red[z][threadIdx.x] += red[z][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x < 3) out[threadIdx.x] = sqrt(red[threadIdx.x][0]);
}

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------
#define LBM_DISPATCH(storage, ...)                                                          \
    switch (storage) {                                                                      \
    case ST_F64: { using S = double; __VA_ARGS__; break; }                                  \
    case ST_F32: { using S = float; __VA_ARGS__; break; }                                   \
    default: { using S = _Float16; __VA_ARGS__; break; }                                    \
    }

static inline int blocks_for(long long n) { return (int)((n + 255) / 256); }

static hipError_t launch_phase_a(const LaunchSet &L, int storage, Sub ks, hipStream_t s) {
    if (L.blocks[CLS_A] > 0)
        LBM_DISPATCH(storage, hipLaunchKernelGGL((k_phase_a<S, SRC_F>), dim3(L.blocks[CLS_A]), dim3(256), 0, s,
                                                 L.runs, L.prefix[CLS_A], L.nruns, ks));
    return hipGetLastError();
}

static hipError_t launch_target(const LaunchSet &L, int storage, Sub ks, hipStream_t s) {
    if (L.blocks[CLS_TGT] > 0)
        LBM_DISPATCH(storage, hipLaunchKernelGGL((k_target<S>), dim3(L.blocks[CLS_TGT]), dim3(256), 0, s,
                                                 L.runs, L.prefix[CLS_TGT], L.nruns, ks));
    return hipGetLastError();
}

static hipError_t launch_frame(const LaunchSet &L, int storage, Sub ks, hipStream_t s, hipEvent_t a,
                               hipEvent_t b) {
#if LBM_Q >= 17
    if (const int nb4 = L.blocks[CLS_SPLIT]; nb4 > 0 && L.split_small) {
        const int *pre = L.prefix[CLS_SPLIT];
        LBM_DISPATCH(storage, if (a) hipExtLaunchKernelGGL((k_frame_split<S>), dim3(nb4), dim3(256), 0, s, a, b, 0,
                                                           L.runs, pre, L.nruns, ks);
                              else hipLaunchKernelGGL((k_frame_split<S>), dim3(nb4), dim3(256), 0, s, L.runs, pre,
                                                      L.nruns, ks));
        return hipGetLastError();
    }
#endif
    const int nb = L.blocks[CLS_FRAME];
    if (nb <= 0) return hipSuccess;
    const int *pre = L.prefix[CLS_FRAME];
#define LBM_FRAME(STREAM)                                                                                  \
    do {                                                                                                   \
        if (a) hipExtLaunchKernelGGL((k_frame<S, STEP_ONE, STREAM>), dim3(nb), dim3(256), 0, s, a, b, 0,   \
                                     L.runs, pre, L.nruns, ks);                                            \
        else hipLaunchKernelGGL((k_frame<S, STEP_ONE, STREAM>), dim3(nb), dim3(256), 0, s, L.runs, pre,    \
                                L.nruns, ks);                                                              \
    } while (0)
    if (L.stream_frame) {
        LBM_DISPATCH(storage, LBM_FRAME(true));
    } else {
        LBM_DISPATCH(storage, LBM_FRAME(sizeof(S) == 8));
    }
#undef LBM_FRAME
    return hipGetLastError();
}

static hipError_t launch_bulk(const LaunchSet &L, int storage, int tx, Sub ks, hipStream_t s,
                              hipEvent_t a, hipEvent_t b) {
    const int nb = L.blocks[CLS_BULK];
    if (nb <= 0) return hipSuccess;
    const int *pre = L.prefix[CLS_BULK];
    // events attached to the dispatch itself (no separate event packets around the kernel)
#define LBM_BULK(TXV)                                                                              \
    LBM_DISPATCH(storage, if (a) hipExtLaunchKernelGGL((k_bulk<S, TXV>), dim3(nb), dim3(256), 0, s, \
                                                       a, b, 0, L.runs, pre, L.nruns, ks);        \
                          else hipLaunchKernelGGL((k_bulk<S, TXV>), dim3(nb), dim3(256), 0, s,     \
                                                  L.runs, pre, L.nruns, ks))
    switch (tx) {
    case 64: LBM_BULK(64); break;
    case 128: LBM_BULK(128); break;
    default: LBM_BULK(256); break;
    }
#undef LBM_BULK
    return hipGetLastError();
}

static hipError_t launch_phase_a_bulk(const LaunchSet &L, int storage, int tx, Sub ks, hipStream_t s,
                                      hipEvent_t a, hipEvent_t b) {
    const bool split = NQ >= 17 && L.split_small;
    const int nA = L.blocks[split ? CLS_A_SPLIT : CLS_A], nB = L.blocks[CLS_BULK];
    if (nA + nB <= 0) return hipSuccess;
    // Bulk tiles ahead of the phase-A blocks (by default).  On large grids, where the tiles
    // outnumber the phase-A blocks eightfold or more, all of them: phase A's latency then hides
    // in the grid's tail, 0.1-3% faster at 4224^2 (D2Q37 NRBC FP32 1158.7 against 1171.3 us per
    // step, FP16 707.9 against 722.5; D2Q17 ZG FP16 303.6 against 313.1; D2Q9 ZG FP64 510.1
    // against 523.3).  Otherwise half of them for D2Q37 in FP64, where the half after phase A
    // still outlasts its latency (1088^2 NRBC + PML: 178.5 against 185.5 us per step), and none
    // for the rest, where the shorter tiles would leave phase A on the tail (FP32 98.8 against
    // 97.1 us, FP16 66.6 against 62.0, D2Q9 FP64 47.1 against 46.5).  With split phase-A blocks all
    // of them in FP64 (D2Q37 at 190^2: 12.5 us, with half 13.9; D2Q17 at 340^2: 11.5, with none
    // 13.2) and none in FP32 and FP16, at any ratio (us per step with none and all: NRBC 500^2 with 4
    // cells FP32 31.0, 33.9, 1000^2 72.4, 77.5; ZG 700^2 with 4 cells 42.5, 42.5).
    const int h = L.split >= 0 ? (nB * L.split / 8) & ~7
                  : split ? (storage == ST_F64 ? nB & ~7 : 0)
                  : nB >= 8 * nA ? nB & ~7
                  : (NQ == 37 && storage == ST_F64) ? (nB / 2) & ~7 : 0;
    const int *pa = L.prefix[split ? CLS_A_SPLIT : CLS_A], *pb = L.prefix[CLS_BULK];
#define LBM_PAB(KERNEL, TXV)                                                                               \
    LBM_DISPATCH(storage, if (a) hipExtLaunchKernelGGL((KERNEL<S, TXV>), dim3(nA + nB), dim3(256), \
                                                       0, s, a, b, 0, L.runs, pa, nA, pb, nB, h,   \
                                                       L.nruns, ks);                               \
                          else hipLaunchKernelGGL((KERNEL<S, TXV>), dim3(nA + nB), dim3(256), \
                                                  0, s, L.runs, pa, nA, pb, nB, h, L.nruns, ks))
#if LBM_Q >= 17
    if (split) {
        switch (tx) {
        case 64: LBM_PAB(k_small_step, 64); break;
        case 128: LBM_PAB(k_small_step, 128); break;
        default: LBM_PAB(k_small_step, 256); break;
        }
        return hipGetLastError();
    }
#endif
    switch (tx) {
    case 64: LBM_PAB(k_phase_a_bulk, 64); break;
    case 128: LBM_PAB(k_phase_a_bulk, 128); break;
    default: LBM_PAB(k_phase_a_bulk, 256); break;
    }
#undef LBM_PAB
    return hipGetLastError();
}

static hipError_t poison(const LaunchSet &L, int storage, Sub ks, int what, hipStream_t s) {
    if (L.nruns <= 0) return hipSuccess;
    LBM_DISPATCH(storage, hipLaunchKernelGGL((k_poison<S>), dim3(1024, L.nruns), dim3(256), 0, s, L.runs,
                                             ks, what));
    return hipGetLastError();
}
static hipError_t launch_poison(const LaunchSet &L, int storage, Sub ks, hipStream_t s) {
    return poison(L, storage, ks, POISON_ONE, s);
}

// Two steps of every run in one pass over its interior: the interior's two steps, then the boundary
// chain of the first step (characteristic fill and Q update, the frame into the bands) and of the
// second, from the bands.  The tiles hold nearly all of a compute unit's LDS and registers, so the
// chain does not run beside them; it comes after them so that it finds its own bands, Q and G in
// the Infinity Cache (1088^2 FP64: frame launches 41.2 and 39.8 us before, 37.5 and 39.3 after).
template <class S>
static hipError_t two_steps(const LaunchSet &L, int storage, Sub k1, hipStream_t s) {
    const Sub k2{k1.steps + 1, k1.flips};
    const dim3 tb(256), nA(L.blocks[CLS_A]);
    hipError_t e = L.poison ? poison(L, storage, k1, POISON_FIRST, s) : hipSuccess;
    hipLaunchKernelGGL((k_core<S>), dim3(L.blocks[CLS_CORE]), dim3(CORE_X * CORE_R), 0, s, L.runs,
                       L.prefix[CLS_CORE], L.nruns, k1, L.core_rows);
    if (e == hipSuccess) e = launch_target(L, storage, k1, s);
    if (nA.x > 0)
        hipLaunchKernelGGL((k_phase_a<S, SRC_F>), nA, tb, 0, s, L.runs, L.prefix[CLS_A], L.nruns, k1);
    hipLaunchKernelGGL((k_frame<S, STEP_FIRST, false>), dim3(L.blocks[CLS_FRAME]), tb, 0, s, L.runs,
                       L.prefix[CLS_FRAME], L.nruns, k1);
    if (e == hipSuccess && L.poison) e = poison(L, storage, k2, POISON_SECOND, s);
    if (e == hipSuccess) e = launch_target(L, storage, k2, s);
    if (nA.x > 0)
        hipLaunchKernelGGL((k_phase_a<S, SRC_M>), nA, tb, 0, s, L.runs, L.prefix[CLS_A], L.nruns, k2);
    hipLaunchKernelGGL((k_frame<S, STEP_SECOND, sizeof(S) == 8>), dim3(L.blocks[CLS_FRAME2]), tb, 0, s, L.runs,
                       L.prefix[CLS_FRAME2], L.nruns, k2);
    return e != hipSuccess ? e : hipGetLastError();
}
static hipError_t launch_two_steps(const LaunchSet &L, int storage, Sub k1, hipStream_t s) {
    switch (storage) {
    case ST_F64: return two_steps<double>(L, storage, k1, s);
    case ST_F32: return two_steps<float>(L, storage, k1, s);
    default: return hipErrorInvalidValue;   // FP16 is never paired
    }
}

static hipError_t launch_advance(const LaunchSet &L, int n, int flips, hipStream_t s) {
    hipLaunchKernelGGL(k_advance, dim3((L.nruns + 255) / 256), dim3(256), 0, s, L.runs, L.nruns, n, flips);
    return hipGetLastError();
}

static hipError_t launch_set_limit(RunDev *run, long long limit, hipStream_t s) {
    hipLaunchKernelGGL(k_set_limit, dim3(1), dim3(64), 0, s, run, limit);
    return hipGetLastError();
}

static hipError_t launch_set_limits(RunDev *const *runs, const long long *limits, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_set_limits, dim3((n + 255) / 256), dim3(256), 0, s, runs, limits, n);
    return hipGetLastError();
}

static hipError_t launch_init(RunDev *run, int storage, int Nx, int Ny, const double *rho,
                       const double *ux, const double *uy, const double *T, float *absmax,
                       hipStream_t s) {
    int nb = blocks_for((long long)Nx * Ny);
    LBM_DISPATCH(storage, hipLaunchKernelGGL((k_init<S>), dim3(nb), dim3(256), 0, s, run, rho, ux, uy,
                                             T, absmax));
    return hipGetLastError();
}

static hipError_t launch_moments(RunDev *run, int storage, int Nx, int Ny, double *rho, double *ux,
                          double *uy, double *T, hipStream_t s) {
    int nb = blocks_for((long long)Nx * Ny);
    LBM_DISPATCH(storage, hipLaunchKernelGGL((k_moments<S>), dim3(nb), dim3(256), 0, s, run, rho, ux,
                                             uy, T));
    return hipGetLastError();
}

static hipError_t launch_export_f(RunDev *run, int storage, int Nx, int Ny, const double *fbar,
                           double *out, hipStream_t s) {
    int nb = blocks_for((long long)Nx * Ny);
    LBM_DISPATCH(storage, hipLaunchKernelGGL((k_export_f<S>), dim3(nb, NQ), dim3(256), 0, s, run, fbar,
                                             out));
    return hipGetLastError();
}

static hipError_t launch_export_q(RunDev *run, int storage, int nt, double *out, hipStream_t s) {
    if (nt <= 0) return hipSuccess;
    int nb = blocks_for(nt);
    LBM_DISPATCH(storage, hipLaunchKernelGGL((k_export_q<S>), dim3(nb, NQ), dim3(256), 0, s, run, out));
    return hipGetLastError();
}

static hipError_t launch_check(RunDev *run, int storage, int Nx, int Ny, int *flag, hipStream_t s) {
    int nb = blocks_for((long long)Nx * Ny);
    LBM_DISPATCH(storage, hipLaunchKernelGGL((k_check<S>), dim3(nb), dim3(256), 0, s, run, flag));
    return hipGetLastError();
}

static hipError_t launch_err_rows(const double *rho, const double *ux, const double *T, int Nx, int x0,
                           int y0, int lx, int ly, const double *rr, const double *ru,
                           const double *rt, double *partials, hipStream_t s) {
    if (ly <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_err_rows, dim3(ly), dim3(256), 0, s, rho, ux, T, Nx, x0, y0, lx, rr, ru, rt,
                       partials);
    return hipGetLastError();
}

static hipError_t launch_err_rows_state(RunDev *run, int storage, int x0, int y0, int lx, int ly,
                                        const double *rr, const double *ru, const double *rt,
                                        double *partials, hipStream_t s) {
    if (ly <= 0) return hipSuccess;
    LBM_DISPATCH(storage, hipLaunchKernelGGL((k_err_rows_state<S>), dim3(ly), dim3(256), 0, s, run, x0, y0,
                                             lx, rr, ru, rt, partials));
    return hipGetLastError();
}

static hipError_t launch_err_final(const double *partials, int nrows, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_err_final, dim3(1), dim3(256), 0, s, partials, nrows, out);
    return hipGetLastError();
}

// host-side table (the device pass has no host functions to point at)
#ifndef __HIP_DEVICE_COMPILE__
const KernelSet kernels = {NQ, launch_phase_a, launch_frame, launch_target, launch_phase_a_bulk, launch_bulk,
                           launch_advance, launch_set_limit, launch_set_limits, launch_init,
                           launch_moments, launch_export_f, launch_export_q, launch_check,
                           launch_err_rows, launch_err_rows_state, launch_err_final, launch_poison, launch_two_steps};
#endif

}  // namespace LBM_KSET
}  // namespace lbm
