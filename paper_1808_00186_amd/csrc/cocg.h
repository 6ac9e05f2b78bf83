// The state of one column of the mixed-precision COCG, its stop rules and its
// scalar steps, shared by the kernels of block.hip (one kernel per phase) and
// resident.hip (the whole inner solve in one kernel). Plain arithmetic only, so
// that a test compiles it for the host and compares the two statements of the
// rules.
#pragma once
#include "cplx.h"

namespace petgem {

namespace {

__device__ __forceinline__ float2 f2(float x, float y) { return make_float2(x, y); }

__device__ __forceinline__ float2 cmulf(float2 a, float2 b) {
    return f2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

__device__ __forceinline__ bool cfinite(double2 a) { return isfinite(a.x) && isfinite(a.y); }
__device__ __forceinline__ bool czero(double2 a) { return a.x == 0.0 && a.y == 0.0; }

// c ? a : b by value (the operator selects an address, which keeps a state
// that lives in registers in memory)
__device__ __forceinline__ double2 pick(bool c, double2 a, double2 b) {
    return make_double2(c ? a.x : b.x, c ? a.y : b.y);
}

struct ColState {
    double2 rho, alpha, beta;
    double rn2;        // inner |r|^2 (relative to the normalised start)
    double rn2_0;      // |r|^2 at the start of the inner solve the tolerance is relative to (1, or the
                       // split residual's of an Eisenstat solve)
    double rn2_best;   // least inner |r|^2 of the current refinement step
    double scale;      // |r64| of the current refinement step
    double bnorm;      // |b|
    double rnorm64;    // true residual norm
    double tol_abs;    // rtol |b|
    double inner_tol2; // squared inner tolerance of the current refinement step
    double inner_rtol; // requested inner tolerance
    int active;        // inner iteration running
    int outer;         // not yet converged in double precision
    int breakdown;
    int iters;         // inner iterations (all refinement steps)
    int kin;           // inner iterations of the current refinement step
    int stepped;       // this iteration's alpha was applied to r (set at the beta step)
    int k_best;        // inner iteration of rn2_best
    int stalled;       // inner steps ended by the stagnation guard (all refinement steps)
    // symmetric QMR (sqmr): the quasi-minimal-residual smoothing of the iterate
    double tau2;       // tau^2, the smoothed residual's estimate (same norm as rn2)
    double cq;         // c^2 of the latest beta step: x_Q = (1 - c^2) x_Q + c^2 x
    double tmark;      // tau^2 (COCG: |r|^2) at the last halving of tau (|r|)
    int sqmr;          // this solve is SQMR
    int k_mark;        // inner iteration of tmark (COCG)
    int restarts;      // of the directions in this inner solve
    int it_start;      // iters at the start of this inner solve
    int k_prev;        // inner iterations of the one before (0: this is the first)
};

// Stagnation guard of the inner COCG, which has no minimisation property: a
// column whose inner |r|^2 has not improved on its best of this refinement
// step for twice the iterations the best took plus kStallIters stops its
// inner solve; the refinement step applies its correction and the next step
// restarts from the true residual. Without it one column of a 32-source block
// on the 6.9M-DOF marine mesh, after a last-bit change of its starting scale,
// wandered at inner |r| ~ 1 for 18,000 iterations instead of converging.
// (A guard that also stopped a column on a 1000-fold rise of |r|, with 500
// instead of 3000 iterations, fired on ordinary spikes of converging columns:
// their corrections raised the true residual 50-fold and the block needed
// 4-6 refinement steps instead of 3.)
constexpr int kStallIters = 3000;
__device__ __forceinline__ bool stalled_now(ColState& S, double r2) {
    if (r2 < S.rn2_best) {
        S.rn2_best = r2;
        S.k_best = S.kin;
        return false;
    }
    return S.kin - S.k_best > 2 * S.k_best + kStallIters;
}

// The last refinement step of a column solves its correction only as far as
// the target needs, with a factor 0.3 to spare (res_step). A column whose
// inner |r| hovers just above that target without a new best for half the
// iterations its best took (at least kRelaxIters) gives the margin up: it
// stops once |r| is within the target without the factor. (With a quarter,
// columns that were still converging gave the margin up, missed rtol and
// needed a fourth refinement step.) (On the
// 6.9M-unknown survey one 0.25 Hz column reached 1.04 times its target of
// 2.2e-2 at iteration 576 of its third step, then wandered for 4,000
// iterations until the guard above stopped it.)
constexpr int kRelaxIters = 100;
// In any refinement step, a column whose |r| has had no new best for as many
// iterations as its best took (at least kPlateauIters) stops at the first
// iterate whose |r| is at most 0.1 of the step's start: its correction
// still reduces the true residual tenfold, and the next refinement step
// restarts from it. (The same 0.25 Hz survey had a column reach 1.4 times the
// inner target 3e-5 at iteration 365 of its first step and wander between
// 2e-4 and 7e-3 until the guard stopped it at 4,096.) A plateau as long as
// the whole descent before it does not occur in a column that still
// converges.
constexpr int kPlateauIters = 200;
__device__ __forceinline__ bool plateau_now(const ColState& S, double r2) {
    const bool last_step = S.inner_tol2 > S.inner_rtol * S.inner_rtol;   // that one has its own rule
    return !last_step && S.kin - S.k_best >= max(kPlateauIters, S.k_best) && r2 <= 0.01 * S.rn2_0;
}
// A column that wanders: its |r| has not halved for as many iterations as the
// whole refinement step before took (at least kWanderIters). Its directions
// have lost their conjugacy; it restarts in place, with p = z, from the residual
// it has, at most kWanderStarts times an inner solve. The rules above and below
// miss it while the best |r| creeps down: one of 96 3,032-unknown models, |r^T z|
// a millionth of |r|^2 at the start of its third step, stayed between 0.1 and 9 for
// 19,000 iterations.
// The measure is the step before because a column that converges has long
// plateaus too, the longer the larger the mesh and the lower the frequency: over
// 180 inner solves of 3,000 to 80,000 unknowns at 0.25 to 1.3 Hz (a mirror of this
// recurrence) the longest one was 465 iterations, and at most 0.47 of the step
// before; a wandering one went 22 of them. (Eight times the average
// halving so far, at least 200, fired on 21 of the 180 and made their columns up to
// 29 % slower, 172 columns by 2 %, where this changes none of them.) The first step
// has no measure and keeps to the stagnation guard.
constexpr int kWanderIters = 200, kWanderStarts = 4;
__device__ __forceinline__ bool wander_test(const ColState& S) {   // since the last halving
    return (S.k_prev > 0) & (S.restarts < kWanderStarts) & (S.kin - S.k_mark >= max(kWanderIters, S.k_prev));
}
__device__ __forceinline__ bool wander_now(ColState& S, double r2) {
    if (r2 < 0.25 * S.tmark) {
        S.tmark = r2;
        S.k_mark = S.kin;
        return false;
    }
    if (!wander_test(S)) return false;
    S.tmark = r2;
    S.k_mark = S.kin;
    S.restarts += 1;
    return true;
}
__device__ __forceinline__ bool relaxed_now(const ColState& S, double r2) {
    const bool last_step = S.inner_tol2 > S.inner_rtol * S.inner_rtol;
    return last_step && r2 <= S.inner_tol2 * S.rn2_0 / (0.3 * 0.3) &&
           S.kin - S.k_best >= max(kRelaxIters, S.k_best / 2);
}

// The scalar step of SQMR (Section 5.3 names SQMR with SOR as the paper's
// single-process solver). Its recurrence is COCG's (rho, beta as in
// step_beta); the quasi-minimal-residual smoothing of the iterate takes, from
// the new residual norm |r|^2 = r2, theta^2 = r2 / tau^2, c^2 = 1 / (1 +
// theta^2) and tau^2 <- tau^2 theta^2 c^2, and the smoothed iterate is
// x_Q = (1 - c^2) x_Q + c^2 x (written by the update kernels). tau falls
// monotonically, so the inner solve stops once tau is within the target, or
// once tau has not halved for as many iterations as its last halving took
// (at least kPlateauIters). tau bounds the smoothed residual only when the
// residuals are orthogonal; COCG's are orthogonal in the bilinear form, not
// in the Euclidean one, and where the unsmoothed residual diverges tau still
// falls while the smoothed residual does not (a refinement step then gains
// nothing).
__device__ __forceinline__ void sqmr_beta(ColState& S, double2 rz, double r2) {
    S.iters += 1;
    S.kin += 1;
    S.rn2 = r2;
    if (!isfinite(r2) || !cfinite(rz)) {
        S.active = 0;
        S.breakdown = 1;
        return;
    }
    const double th2 = S.tau2 > 0.0 ? r2 / S.tau2 : 0.0;
    const double c2 = 1.0 / (1.0 + th2);
    S.tau2 = S.tau2 * th2 * c2;
    S.cq = c2;
    S.rn2_best = S.tau2;
    if (S.tau2 <= S.inner_tol2 * S.rn2_0) {
        S.active = 0;
        return;
    }
    if (S.tau2 <= 0.25 * S.tmark) {
        S.tmark = S.tau2;
        S.k_best = S.kin;
    } else if (S.kin - S.k_best >= max(kPlateauIters, S.k_best)) {
        S.active = 0;
        S.stalled += 1;
        return;
    }
    if (czero(S.rho)) {
        S.active = 0;
        S.breakdown = 1;
        return;
    }
    S.beta = cdiv(rz, S.rho);
    S.rho = rz;
}

// convergence test on |r|^2 and beta = rho' / rho for an active column
// (counting the update that produced r)
__device__ __forceinline__ void step_beta(ColState& S, double2 rz, double r2) {
    S.iters += 1;
    S.kin += 1;
    S.rn2 = r2;
    if (!isfinite(r2) || !cfinite(rz)) {
        S.active = 0;
        S.breakdown = 1;
    } else if (r2 <= S.inner_tol2 * S.rn2_0) {
        S.active = 0;
    } else if (stalled_now(S, r2)) {
        S.active = 0;
        S.stalled += 1;
    } else if (relaxed_now(S, r2)) {
        S.active = 0;
    } else if (plateau_now(S, r2)) {
        S.active = 0;
        S.stalled += 1;
    } else if (czero(S.rho)) {
        S.active = 0;
        S.breakdown = 1;
    } else {
        S.beta = wander_now(S, r2) ? make_double2(0.0, 0.0) : cdiv(rz, S.rho);
        S.rho = rz;
    }
}

// The scalar step of the fused step for one column, from the five sums t:
// the product's p^T q, q^T D^-1 r, q^T D^-1 q and the previous step's r^T z,
// |r|^2. kin == 0 (just started): rho and |r|^2 are the state's own;
// otherwise the convergence test (with the stagnation guard) runs first.
__device__ __forceinline__ void fused_scalars(ColState& S, const double2* t) {
    // alpha = rho / p^T q and beta = next / rho with the next
    // rho = rho - 2 alpha q^T D^-1 r + alpha^2 q^T D^-1 q; since alpha / rho is
    // 1 / p^T q, beta = 1 + (alpha q^T D^-1 q - 2 q^T D^-1 r) / p^T q. Ahead of
    // the tests: one thread runs this, and its latency is that of the chain
    const double2 pq = t[0], rz = t[3], rho = pick(S.kin > 0, rz, S.rho);
    const double i2 = 1.0 / (pq.x * pq.x + pq.y * pq.y);
    const double2 ip = make_double2(pq.x * i2, -pq.y * i2);
    const double2 al = cmul(rho, ip);
    const double2 be = cadd(make_double2(1.0, 0.0), cmul(csub(cmul(al, t[2]), cscale(t[1], 2.0)), ip));
    // the r left by the previous step: finite, converged, stalled_now,
    // relaxed_now, plateau_now, wander_now in this order (without branches,
    // for the same reason)
    const double r2 = t[4].x;
    const bool on = S.active && S.kin > 0;
    const bool bad = !(isfinite(r2) & cfinite(rz)), conv = r2 <= S.inner_tol2;
    const bool better = on & !bad & !conv & (r2 < S.rn2_best);
    const double best = better ? r2 : S.rn2_best;
    const int kb = better ? S.kin : S.k_best, since = S.kin - kb;
    const bool last_step = S.inner_tol2 > S.inner_rtol * S.inner_rtol;
    const bool stall = !better & (since > 2 * kb + kStallIters);
    const bool relax = last_step & (r2 <= S.inner_tol2 * S.rn2_0 / (0.3 * 0.3)) & (since >= max(kRelaxIters, kb / 2));
    const bool plateau = !last_step & (since >= max(kPlateauIters, kb)) & (r2 <= 0.01 * S.rn2_0);
    const bool zero = czero(rz);
    const bool stop = on & (bad | conv | stall | relax | plateau | zero);
    const bool mark = on & !stop & (r2 < 0.25 * S.tmark);
    const bool wander = on & !stop & !mark & wander_test(S);
    const bool go = (S.active != 0) & !stop;
    const bool ok = go & cfinite(pq) & !czero(pq) & cfinite(be);
    S.rn2 = on ? r2 : S.rn2;
    S.rn2_best = best;
    S.k_best = kb;
    S.tmark = mark | wander ? r2 : S.tmark;
    S.k_mark = mark | wander ? S.kin : S.k_mark;
    S.restarts += wander;
    S.stalled += on & !bad & !conv & (stall | (!relax & plateau));
    S.breakdown |= (on & (bad | (!conv & !stall & !relax & !plateau & zero))) | (go & !ok);
    S.rho = pick(on & !stop, rz, S.rho);
    S.active = ok;
    S.alpha = pick(ok, al, S.alpha);
    S.beta = pick(ok, pick(wander, make_double2(0.0, 0.0), be), S.beta);
    S.iters += ok;
    S.kin += ok;
}

}  // namespace

}  // namespace petgem
