// Output stages shared by the FP64 finalize kernels of the grid engine and by the launches
// that store their outputs themselves (device code): what is stored for store slot c of
// particle i, given `sum(o)`, the FP64 sum over all j of the pipeline's output o.
#pragma once

#include "nbody_internal.h"

namespace nbody {

// Forces and potentials: slots 0, 1, 2 are the acceleration components (optionally
// followed by the leapfrog's second kick v += h a), slot 3 the potential (optionally
// with the j == i term -m_i / eps, formed in FP64).  Slot c stores output c.
struct ForceOut {
    using Args = FinalizeArgs;
    static constexpr int kOutputs = kForceOutputs;
    // Store slots: 4, or 3 without the last output (no potential).
    static constexpr int stores(bool full) { return full ? 4 : 3; }
    template <class Sum>
    static __device__ __forceinline__ void put(const Args &a, int i, int c, Sum sum) {
        double r = sum(c);
        if (c == 3) {
            if (a.include_self) r -= (double)a.m[i] / (double)a.eps;
            a.pot[i] = r;
            return;
        }
        store(a, c * (size_t)a.n + i, r);
    }
    // Acceleration component r at flat index q, with what follows it in a leapfrog step;
    // returns the drifted coordinate (0 without a drift).
    static __device__ __forceinline__ double store(const Args &a, size_t q, double r) {
        a.acc[q] = r;
        if (!a.kick_v) return 0.0;
        double v = a.kick_v[q] + a.kick_h * r;
        double x = 0.0;
        if (a.drift_x) {
            v = v + a.kick_h * r;
            x = a.drift_from[q] + a.drift_dt * v;
            a.drift_x[q] = x;
            if (a.checkpoint) a.checkpoint[q] = x;
        }
        a.kick_v[q] = v;
        return x;
    }
};

// Force, jerk and potential: slots 0-2 the acceleration, 3-5 the jerk, 6 the potential
// (optionally with the j == i term -m_i / eps, formed in FP64).  Slot c stores output c.
struct JerkOut {
    using Args = JerkFinalizeArgs;
    static constexpr int kOutputs = kJerkOutputs;
    // Store slots: 7, or 6 without the last output (no potential).
    static constexpr int stores(bool full) { return full ? 7 : 6; }
    template <class Sum>
    static __device__ __forceinline__ void put(const Args &a, int i, int c, Sum sum) {
        const size_t n = (size_t)a.n;
        if (a.x) {
            if (c < 3) step(a, c * n + i, sum(c), sum(c + 3));
            return;
        }
        double r = sum(c);
        if (c == 6) {
            if (a.include_self) r -= (double)a.m[i] / (double)a.eps;
            a.pot[i] = r;
        } else if (c < 3) {
            a.acc[c * n + i] = r;
        } else {
            a.jerk[(c - 3) * n + i] = r;
        }
    }
    // The corrector of flat index q, v' = v + (a + a1) dt/2 + (j - j1) dt^2/12 and x' = x +
    // (v + v') dt/2 + (a - a1) dt^2/12, then (a, j) <- (a1, j1) and the next step's predictor,
    // x_p = x + v dt + a dt^2/2 + j dt^3/6 and v_p = v + a dt + j dt^2/2 (returned).
    static __device__ __forceinline__ double2 step(const Args &a, size_t q, double an, double jn) {
        const double dt = a.dt;
        const double dt2 = dt * dt;
        const double a0 = a.acc[q], j0 = a.jerk[q], v0 = a.v[q];
        const double vn = v0 + (a0 + an) * dt / 2.0 + (j0 - jn) * dt2 / 12.0;
        const double xn = a.x[q] + (v0 + vn) * dt / 2.0 + (a0 - an) * dt2 / 12.0;
        a.x[q] = xn;
        a.v[q] = vn;
        a.acc[q] = an;
        a.jerk[q] = jn;
        double2 p = make_double2(0.0, 0.0);
        if (a.xp) {
            p.x = xn + vn * dt + an * dt2 / 2.0 + jn * dt2 * dt / 6.0;
            p.y = vn + an * dt + jn * dt2 / 2.0;
            a.xp[q] = p.x;
            a.vp[q] = p.y;
        }
        return p;
    }
};

// Adjoint: slots 0, 1, 2 are dL/dx_i = sum(c) - g_i,c * sum(3) (g_i the particle's own
// cotangent, as the FP32 value the pair kernel sees), slot 3 dL/dm_i = -sum(4); with
// accumulate set both are added to what the arrays hold.
struct VjpOut {
    using Args = VjpFinalizeArgs;
    static constexpr int kOutputs = kVjpOutputs;
    // Store slots: 4, or 3 without the mass gradient.
    static constexpr int stores(bool full) { return full ? 4 : 3; }
    template <class Sum>
    static __device__ __forceinline__ void put(const Args &a, int i, int c, Sum sum) {
        if (c < 3) {
            const double gk = (double)(float)a.ga[(size_t)c * a.n + i];
            const double r = sum(c) - gk * sum(3);
            const size_t q = (size_t)c * a.n + i;
            const double g = a.accumulate ? a.grad_pos[q] + r : r;
            a.grad_pos[q] = g;
            if (a.vbar) {
                const double vb = a.vbar[q] + a.step_dt * g;
                a.vbar[q] = vb;
                a.abar[q] = a.step_h * vb;
            }
            return;
        }
        const double gm = -sum(4);
        a.grad_mass[i] = a.accumulate ? a.grad_mass[i] + gm : gm;
    }
};

}  // namespace nbody
