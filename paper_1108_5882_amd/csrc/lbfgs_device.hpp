// Device L-BFGS for many independent fits (one wave per fit), advanced once
// per evaluation so that the whole iteration (evaluate every fit's trial
// point, then update every fit) stays on the device.
//
// Each fit minimises its NLL over the real vector x = (Re V_0, Im V_0, ...)
// (minimisers work on real parameters, Berger Section 4).  State machine per
// fit, entered after its trial point xt was evaluated (f_t, g_t):
//   phase 0 (start):  accept xt, choose a direction.
//   phase 1 (search): Armijo test f_t <= f + c1 alpha g.d.  Accepted: the pair
//     s = xt - x, y = g_t - g enters the history if s.y > 0, the point moves
//     and a new direction is chosen.  Rejected: alpha halves and the trial
//     point moves back along the same direction.
//   direction: d = -H g by the two-loop recursion over the last m pairs with
//     H0 = (s.y / y.y) of the newest pair (Nocedal & Wright, Alg. 7.4); if it
//     is not a descent direction the history is dropped and d = -g.  The first
//     trial step of a fresh history moves x by 1% of |x| (alpha = 0.01 |x| / |d|).
//   stop: status 1 when an accepted step changes f by at most ftol (1 + |f|),
//     status 2 when the step underflows.
//
// Everything a wave needs sits in its registers: lane i holds parameters i and
// i + 64, and the history's pairs, newest first, are all loaded at once.  Dot
// products add their terms in index order (deterministic; a fit from
// single-precision sums magnifies the last bit of a trial point).  Bound by
// latency: one round of loads for the state, one for the history, about 20 dot
// products.  As launches of their own: 24 fits of up to 48 waves 9.3 us per update,
// 32 starts of 8 waves 6.2 us; 13.2 and 14.1 us when a block of 128 threads walked
// the history in memory with three barriers per dot product.
//
// Polar mode (the other representation Section 4 discusses): parameters
// (|V_a|, arg V_a) per wave.  The gradient in them follows from the one in
// (Re V_a, Im V_a) by the chain rule, d/d|V| = cos(phi) d/dRe + sin(phi) d/dIm,
// d/dphi = |V| (-sin(phi) d/dRe + cos(phi) d/dIm).  arg V_0 is held at 0 (the
// likelihood does not change under a global phase, so fixing it removes a flat
// direction).  The lower bound |V_a| >= rmin is kept by projecting every trial
// point onto it, dropping direction components that push a magnitude at the
// bound further down, and testing the Armijo condition along the projected
// step, f_t <= f + c1 g.(x_t - x).  Phases are periodic: after each accepted
// step they are wrapped into [-pi, pi] (the history keeps the step taken).
#pragma once

#include "internal.hpp"

namespace pwa {

constexpr int kLbfgsHist = 8;        // pairs kept
constexpr int kLbfgsPer = 2;         // parameters per lane
static_assert(kLbfgsHist <= kLbfgsMaxHist && 64 * kLbfgsPer >= kLbfgsMaxN, "L-BFGS sizes");

// A vector of the fit's parameters: lane i holds elements i and i + 64 (zeros past n).
struct LbVec {
    double e[kLbfgsPer];
};

__device__ __forceinline__ LbVec lb_load(const double *p, int n, int lane) {
    LbVec v;
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) v.e[u] = lane + 64 * u < n ? p[lane + 64 * u] : 0.0;
    return v;
}
__device__ __forceinline__ void lb_store(double *p, const LbVec &v, int n, int lane) {
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u)
        if (lane + 64 * u < n) p[lane + 64 * u] = v.e[u];
}
// a + s b
__device__ __forceinline__ LbVec lb_axpy(const LbVec &a, double s, const LbVec &b) {
    LbVec v;
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) v.e[u] = a.e[u] + s * b.e[u];
    return v;
}
// Products in LDS, added in index order by every lane (a wave's LDS operations
// complete in order; the fences only keep the compiler's order).  p: 64 kLbfgsPer
// doubles of LDS of this wave.  The loops stay rolled beyond 16 terms: an update runs
// some 20 of these once each, and its time follows the size of the code it fetches.
__device__ __forceinline__ double lb_dot(const LbVec &a, const LbVec &b, int n, double *p) {
    const int lane = threadIdx.x & 63;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) p[lane + 64 * u] = a.e[u] * b.e[u];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    double s = 0.0;
    int i = 0;
#pragma clang loop unroll(disable)
    for (; i + 16 <= n; i += 16) {
        double v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = p[i + j];
#pragma unroll
        for (int j = 0; j < 16; ++j) s += v[j];
    }
#pragma clang loop unroll(disable)
    for (; i < n; i += 2) {                               // n is even
        s += p[i];
        s += p[i + 1];
    }
    return s;
}
__device__ __forceinline__ double lb_maxabs(const LbVec &a) {
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) s = fmax(s, fabs(a.e[u]));
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) s = fmax(s, __shfl_xor(s, off));
    return s;
}
// the other element of each (even, odd) pair
__device__ __forceinline__ LbVec lb_pair(const LbVec &a) {
    LbVec v;
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) v.e[u] = __shfl_xor(a.e[u], 1);
    return v;
}

// Polar mode: the trial point projected onto |V_a| >= rmin (arg V_0 stays 0), and
// the V it stands for.
__device__ __forceinline__ void lb_polar_trial(LbVec &xt, LbVec &vt, double rmin, int lane) {
    const LbVec o = lb_pair(xt);
    const bool odd = lane & 1;
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) {
        const bool first = lane < 2 && u == 0;
        const double r = fmax(odd ? o.e[u] : xt.e[u], rmin);
        const double ph = first ? 0.0 : odd ? xt.e[u] : o.e[u];
        xt.e[u] = odd ? ph : r;
        vt.e[u] = odd ? r * sin(ph) : r * cos(ph);
    }
}

// A fit's state in the registers of one wave.
struct LbRegs {
    LbVec xt, x, g, d, vt;
    LbVec S[kLbfgsHist], Y[kLbfgsHist];               // the history, newest pair first
    double rho[kLbfgsHist];
    double f, alpha, gtd;
    int status, phase, head, count;
};

// Loads the state (n parameters) by one whole wave.
__device__ __forceinline__ void lbfgs_load(LbRegs &r, const LbfgsState *st, int n, bool polar) {
    constexpr int m = kLbfgsHist;
    const int lane = threadIdx.x & 63;
    r.xt = lb_load(st->xt, n, lane);
    r.x = lb_load(st->x, n, lane);
    r.g = lb_load(st->g, n, lane);
    r.d = lb_load(st->d, n, lane);
    r.vt = LbVec{};
    if (polar) r.vt = lb_load(st->vt, n, lane);
    r.status = st->status;
    r.phase = st->phase;
    r.head = st->head;
    r.count = st->count;
    r.f = st->f;
    r.alpha = st->alpha;
    r.gtd = st->gtd;
#pragma unroll
    for (int t = 0; t < m; ++t) {
        const int i = (r.head - 1 - t + 2 * m) % m;
        r.S[t] = lb_load(st->S[i], n, lane);
        r.Y[t] = lb_load(st->Y[i], n, lane);
        r.rho[t] = st->rho[i];
    }
}

// Advances the fit's state after its trial point was evaluated: ft its NLL, gt its
// gradient in (Re V_a, Im V_a).  Called by the wave that holds the state, with 64
// kLbfgsPer doubles of LDS of its own (prod).  Returns the vector the next
// evaluation reads (the trial point, or the V it stands for).
__device__ __forceinline__ LbVec lbfgs_advance(LbfgsState *st, LbRegs &r, int n, double ft, LbVec gt, double c1,
                                               double ftol, bool polar, double rmin, double *prod) {
    constexpr int m = kLbfgsHist;
    const int lane = threadIdx.x & 63;
    const bool odd = lane & 1;
    LbVec &xt = r.xt, &x = r.x, &g = r.g, &d = r.d, &vt = r.vt;
    LbVec(&S)[m] = r.S;
    LbVec(&Y)[m] = r.Y;
    double(&rho)[m] = r.rho;
    double &f = r.f, &alpha = r.alpha, &gtd = r.gtd;
    int &count = r.count;
    const int phase = r.phase, head = r.head;
    if (r.status != 0) return polar ? vt : xt;
    if (polar) {
        // gradient in (|V_a|, arg V_a) at the trial point (arg V_0 held fixed)
        const LbVec xo = lb_pair(xt), go = lb_pair(gt);
#pragma unroll
        for (int u = 0; u < kLbfgsPer; ++u) {
            const double mag = odd ? xo.e[u] : xt.e[u], ph = odd ? xt.e[u] : xo.e[u];
            const double gre = odd ? go.e[u] : gt.e[u], gim = odd ? gt.e[u] : go.e[u];
            const double c = cos(ph), sn = sin(ph);
            gt.e[u] = odd ? (lane == 1 && u == 0 ? 0.0 : mag * fma(c, gim, -(sn * gre))) : fma(c, gre, sn * gim);
        }
    }

    // the trial point from x, alpha and d; in polar mode also the slope of the
    // projected step, which the Armijo test uses
    auto trial = [&]() {
        xt = lb_axpy(x, alpha, d);
        if (polar) {
            lb_polar_trial(xt, vt, rmin, lane);
            gtd = lb_dot(g, lb_axpy(xt, -1.0, x), n, prod);
        }
    };
    auto stop = [&](int code) {
        xt = x;
        if (polar) lb_polar_trial(xt, vt, rmin, lane);
        lb_store(st->xt, xt, n, lane);
        if (polar) lb_store(st->vt, vt, n, lane);
        if (lane == 0) st->status = code;
        return polar ? vt : xt;
    };
    if (phase == 0) {
        x = xt;
        g = gt;
        f = ft;
    } else if (isfinite(ft) && ft <= f + c1 * (polar ? gtd : alpha * gtd)) {
        // accepted: the pair s = xt - x, y = g_t - g goes to the slot at head
        const LbVec s = lb_axpy(xt, -1.0, x), y = lb_axpy(gt, -1.0, g);
        lb_store(st->S[head], s, n, lane);
        lb_store(st->Y[head], y, n, lane);
        const double sy = lb_dot(s, y, n, prod);
        if (sy > 0.0) {
#pragma unroll
            for (int t = m - 1; t > 0; --t) {
                S[t] = S[t - 1];
                Y[t] = Y[t - 1];
                rho[t] = rho[t - 1];
            }
            S[0] = s;
            Y[0] = y;
            rho[0] = 1.0 / sy;
            count = count < m ? count + 1 : m;
            if (lane == 0) {
                st->rho[head] = rho[0];
                st->head = (head + 1) % m;
            }
        } else {
            // the pair is not counted; in a full history its slot is the oldest pair's
            S[m - 1] = s;
            Y[m - 1] = y;
        }
        const double fold = f;
        x = xt;
        g = gt;
        f = ft;
        if (polar && odd) {
            // periodic phases back into [-pi, pi]
#pragma unroll
            for (int u = 0; u < kLbfgsPer; ++u) x.e[u] = remainder(x.e[u], 6.283185307179586476925286766559);
        }
        if (lane == 0) {
            st->f = f;
            st->iter += 1;
            st->count = count;
        }
        lb_store(st->x, x, n, lane);
        lb_store(st->g, g, n, lane);
        if (fabs(fold - ft) <= ftol * (1.0 + fabs(ft))) return stop(1);
    } else {
        alpha *= 0.5;
        const double dmax = lb_maxabs(d), xmax = lb_maxabs(x);
        if (lane == 0) st->alpha = alpha;
        if (alpha * dmax <= 1e-15 * (1.0 + xmax)) return stop(2);
        trial();
        lb_store(st->xt, xt, n, lane);
        if (polar) lb_store(st->vt, vt, n, lane);
        if (lane == 0) {
            st->nbacktrack += 1;
            st->gtd = gtd;
        }
        return polar ? vt : xt;
    }

    // d = -H g by the two-loop recursion; steepest descent when the result is not a
    // descent direction
    LbVec q = g;
    double a[m];
#pragma unroll
    for (int t = 0; t < m; ++t)                           // newest to oldest
        if (t < count) {
            a[t] = rho[t] * lb_dot(S[t], q, n, prod);
            q = lb_axpy(q, -a[t], Y[t]);
        }
    if (count > 0) {
        const double gamma = lb_dot(S[0], Y[0], n, prod) / lb_dot(Y[0], Y[0], n, prod);
#pragma unroll
        for (int u = 0; u < kLbfgsPer; ++u) q.e[u] *= gamma;
    }
#pragma unroll
    for (int t = m - 1; t >= 0; --t)                      // oldest to newest
        if (t < count) q = lb_axpy(q, a[t] - rho[t] * lb_dot(Y[t], q, n, prod), S[t]);
#pragma unroll
    for (int u = 0; u < kLbfgsPer; ++u) d.e[u] = -q.e[u];
    gtd = lb_dot(g, d, n, prod);
    if (!(gtd < 0.0)) {
        count = 0;
#pragma unroll
        for (int u = 0; u < kLbfgsPer; ++u) d.e[u] = -g.e[u];
        gtd = lb_dot(g, d, n, prod);
    }
    bool flat = false;
    if (polar) {
        // no component that pushes a magnitude at its bound further down
#pragma unroll
        for (int u = 0; u < kLbfgsPer; ++u)
            if (!odd && x.e[u] <= rmin && d.e[u] < 0.0) d.e[u] = 0.0;
        gtd = lb_dot(g, d, n, prod);
        if (!(gtd < 0.0)) {
            count = 0;
#pragma unroll
            for (int u = 0; u < kLbfgsPer; ++u) d.e[u] = !odd && x.e[u] <= rmin && g.e[u] > 0.0 ? 0.0 : -g.e[u];
            gtd = lb_dot(g, d, n, prod);
            flat = !(gtd < 0.0);                          // stationary on the bound
        }
    }
    lb_store(st->d, d, n, lane);
    if (phase == 0) {
        lb_store(st->x, x, n, lane);
        lb_store(st->g, g, n, lane);
        if (lane == 0) st->f = f;
    }
    if (lane == 0) st->count = count;
    if (flat) return stop(1);
    alpha = 1.0;
    if (count == 0) {                                     // empty history, or reset to steepest descent
        const double xn = sqrt(lb_dot(x, x, n, prod)), dn = sqrt(lb_dot(d, d, n, prod));
        alpha = dn > 0.0 ? 0.01 * (xn > 0.0 ? xn : 1.0) / dn : 0.0;
    }
    trial();
    lb_store(st->xt, xt, n, lane);
    if (polar) lb_store(st->vt, vt, n, lane);
    if (lane == 0) {
        st->gtd = gtd;
        st->alpha = alpha;
        st->phase = 1;
    }
    return polar ? vt : xt;
}

}  // namespace pwa
