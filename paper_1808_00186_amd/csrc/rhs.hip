// Right-hand side (Section 3, eq. 9 with the primary field of Appendix A)
// and receiver interpolation (Section 3, eq. 8; Section 2, eq. 4).
//
// k_rhs_elem: one thread per tetrahedron; elements with sigma = sigma_bg
//   write zeros, the others evaluate the dipole field at the 4 points of the
//   degree-2 rule and integrate it against the 6 edge basis functions.
// k_rhs_gather: one thread per DOF sums its incident element entries in
//   increasing element order (deterministic, no atomics).
//   Both take up to kRhsJobs jobs (sources of one system, or systems of a
//   batch) in one launch, a row of blocks each: one at a time they leave the
//   chip partly idle (9 sources on 56,000 elements took 18 launches of 5 to
//   9 us each) and pay a kernel boundary per launch. A job is one source, or
//   two of one system with their entries side by side: the gather is bound by
//   its requests, which then fetch 32 bytes each (26.1 -> 20.5 us a source on
//   750,000 elements). The element kernel is bound by its double-precision
//   arithmetic.
// k_receivers: one thread per receiver evaluates the 6 basis functions of its
//   element at the receiver and adds the primary field.
// k_receivers_h: the magnetic field H = curl E / (i w mu0) (Faraday's law of
//   Section 2 with e^{-iwt}): the curl of the secondary field is constant in
//   an element, sum_i e_i 2 s_i l_i grad lambda_a x grad lambda_b, and the
//   primary part is the dipole's analytic H.
#include <algorithm>

#include "device.h"
#include "internal.h"

namespace petgem {

namespace {

constexpr int kE0[6] = {0, 0, 0, 1, 3, 2};
constexpr int kE1[6] = {1, 2, 3, 2, 1, 3};

struct SrcParams {
    double pos[3];
    double dir[3];
    double kappa;   // sqrt(w mu0 sigma_bg / 2)
    double pref;    // moment / (4 pi sigma_bg)
    double hpref;   // moment / (4 pi)
    double inv_wmu; // 1 / (w mu0)
};

// One or two right-hand sides of a system: sources, staging and outputs.
struct RhsJob {
    int T, n, stride, fresh;      // fresh: the staging holds no zeros yet where dsigma = 0
    const double* xyz;
    const int4* tets;
    const double* sigma;
    double sigma_bg, r_min;
    SrcParams sp[2];
    double wmu[2];
    double2* Rst;                 // [6][T][sources]
    int* flag;
    const int32_t *iptr, *islot;
    double2* b[2];
};
struct RhsJobs {                  // by value: 2.5 KB of kernel arguments
    RhsJob j[kRhsJobs];
};

SrcParams make_src(const petgem_source& s, double sigma_bg) {
    SrcParams p;
    for (int k = 0; k < 3; ++k) { p.pos[k] = s.pos[k]; p.dir[k] = s.dir[k]; }
    const double w = 2.0 * kPi * s.freq_hz;
    p.kappa = sqrt(w * kMu0 * sigma_bg * 0.5);
    p.pref = s.moment / (4.0 * kPi * sigma_bg);
    p.hpref = s.moment / (4.0 * kPi);
    p.inv_wmu = 1.0 / (w * kMu0);
    return p;
}

// 177 registers, two waves per SIMD; (256, 3) spills. Sums by vertex instead of
// by point and rsqrt instead of sqrt and a division take 136 registers and a
// quarter less time, but leave a larger error against exact arithmetic.
__global__ void __launch_bounds__(256)
k_rhs_elem(RhsJobs jobs, int ns) {
    const int c = (int)blockIdx.y % ns;
    const RhsJob& job = jobs.j[blockIdx.y / ns];
    const int T = job.T;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= T) return;
    double2* __restrict__ Rst = job.Rst + c;
    const double r_min = job.r_min;
    const double ds = job.sigma[t] - job.sigma_bg;
    if (ds == 0.0) {
        if (!job.fresh) return;
#pragma unroll
        for (int i = 0; i < 6; ++i) Rst[((size_t)i * T + t) * ns] = make_double2(0.0, 0.0);
        return;
    }
    TetGeom G;
    tet_geometry(job.xyz, job.tets[t], G);
    // 4-point degree-2 rule: barycentric (a,b,b,b) and permutations, weights V/4
    const double qa = 0.58541019662496845446;   // (5 + 3 sqrt 5) / 20
    const double qb = 0.13819660112501051518;   // (5 - sqrt 5) / 20
    const SrcParams& sp = job.sp[c];
    double2 R[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) R[i] = make_double2(0.0, 0.0);
    bool singular = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        double lam[4] = {qb, qb, qb, qb};
        lam[q] = qa;
        double x[3];
#pragma unroll
        for (int k = 0; k < 3; ++k)
            x[k] = lam[0] * G.X[0][k] + lam[1] * G.X[1][k] + lam[2] * G.X[2][k] + lam[3] * G.X[3][k];
        double d0 = x[0] - sp.pos[0], d1 = x[1] - sp.pos[1], d2 = x[2] - sp.pos[2];
        if (d0 * d0 + d1 * d1 + d2 * d2 <= r_min * r_min) singular = true;
        double2 E[3];
        dipole_E(x, sp.pos, sp.dir, sp.kappa, sp.pref, E);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const int a = kE0[i], b = kE1[i];
            double n0 = G.sl[i] * (lam[a] * G.g[b][0] - lam[b] * G.g[a][0]);
            double n1 = G.sl[i] * (lam[a] * G.g[b][1] - lam[b] * G.g[a][1]);
            double n2 = G.sl[i] * (lam[a] * G.g[b][2] - lam[b] * G.g[a][2]);
            R[i].x += n0 * E[0].x + n1 * E[1].x + n2 * E[2].x;
            R[i].y += n0 * E[0].y + n1 * E[1].y + n2 * E[2].y;
        }
    }
    if (singular) atomicOr(job.flag, 1);
    // i w mu0 dsigma (V/4) R  ->  multiply by i: (x, y) -> (-y, x)
    const double f = job.wmu[c] * ds * G.vol * 0.25;
#pragma unroll
    for (int i = 0; i < 6; ++i) Rst[((size_t)i * T + t) * ns] = make_double2(-f * R[i].y, f * R[i].x);
}

template <int NS>
__global__ void __launch_bounds__(256)
k_rhs_gather(RhsJobs jobs) {
    const RhsJob& job = jobs.j[blockIdx.y];
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= job.n) return;
    const int T = job.T;
    const int32_t* __restrict__ iptr = job.iptr;
    const int32_t* __restrict__ islot = job.islot;
    const double2* __restrict__ Rst = job.Rst;
    double2 acc[NS];
#pragma unroll
    for (int c = 0; c < NS; ++c) acc[c] = make_double2(0.0, 0.0);
    const int32_t k1 = iptr[r + 1];
    // four incidences, then their entries, in flight at a time; the sum keeps
    // the list order
    for (int32_t k = iptr[r]; k < k1; k += 4) {
        int32_t sl[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) sl[q] = k + q < k1 ? islot[k + q] : -1;
        double2 v[4][NS];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int32_t t = sl[q] / 6, i = sl[q] - 6 * t;
#pragma unroll
            for (int c = 0; c < NS; ++c)
                v[q][c] = sl[q] >= 0 ? Rst[((size_t)i * T + t) * NS + c] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (sl[q] >= 0)
#pragma unroll
                for (int c = 0; c < NS; ++c) acc[c] = cadd(acc[c], v[q][c]);
    }
#pragma unroll
    for (int c = 0; c < NS; ++c) job.b[c][(size_t)r * job.stride] = acc[c];
}

__global__ void k_receivers(int n_rx, const double* __restrict__ rxyz, const int32_t* __restrict__ rtet,
                            const int32_t* __restrict__ rdof, const double* __restrict__ xyz,
                            const int4* __restrict__ tets, const double2* __restrict__ x,
                            SrcParams sp, double2* __restrict__ E, double2* __restrict__ Es) {
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rx) return;
    TetGeom G;
    tet_geometry(xyz, tets[rtet[r]], G);
    const double p[3] = {rxyz[3 * r], rxyz[3 * r + 1], rxyz[3 * r + 2]};
    double lam[4];
    lam[1] = lam[2] = lam[3] = 0.0;
#pragma unroll
    for (int v = 1; v < 4; ++v)
#pragma unroll
        for (int k = 0; k < 3; ++k) lam[v] += G.g[v][k] * (p[k] - G.X[0][k]);
    lam[0] = 1.0 - lam[1] - lam[2] - lam[3];
    double2 es[3] = {make_double2(0, 0), make_double2(0, 0), make_double2(0, 0)};
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        int d = rdof[6 * r + i];
        if (d < 0) continue;
        double2 v = x[d];
        const int a = kE0[i], b = kE1[i];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            double nk = G.sl[i] * (lam[a] * G.g[b][k] - lam[b] * G.g[a][k]);
            es[k].x += nk * v.x;
            es[k].y += nk * v.y;
        }
    }
    double2 ep[3];
    dipole_E(p, sp.pos, sp.dir, sp.kappa, sp.pref, ep);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        E[3 * r + k] = cadd(ep[k], es[k]);
        if (Es) Es[3 * r + k] = es[k];
    }
}

__global__ void k_receivers_h(int n_rx, const double* __restrict__ rxyz, const int32_t* __restrict__ rtet,
                              const int32_t* __restrict__ rdof, const double* __restrict__ xyz,
                              const int4* __restrict__ tets, const double2* __restrict__ x,
                              SrcParams sp, double2* __restrict__ H, double2* __restrict__ Hs) {
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rx) return;
    TetGeom G;
    tet_geometry(xyz, tets[rtet[r]], G);
    double2 cs[3] = {make_double2(0, 0), make_double2(0, 0), make_double2(0, 0)};
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        int d = rdof[6 * r + i];
        if (d < 0) continue;
        const double2 v = x[d];
        const int a = kE0[i], b = kE1[i];
        // curl N_i = 2 s_i l_i grad lambda_a x grad lambda_b
        const double c0 = 2.0 * G.sl[i] * (G.g[a][1] * G.g[b][2] - G.g[a][2] * G.g[b][1]);
        const double c1 = 2.0 * G.sl[i] * (G.g[a][2] * G.g[b][0] - G.g[a][0] * G.g[b][2]);
        const double c2 = 2.0 * G.sl[i] * (G.g[a][0] * G.g[b][1] - G.g[a][1] * G.g[b][0]);
        cs[0].x += c0 * v.x; cs[0].y += c0 * v.y;
        cs[1].x += c1 * v.x; cs[1].y += c1 * v.y;
        cs[2].x += c2 * v.x; cs[2].y += c2 * v.y;
    }
    const double p[3] = {rxyz[3 * r], rxyz[3 * r + 1], rxyz[3 * r + 2]};
    double2 hp[3];
    dipole_H(p, sp.pos, sp.dir, sp.kappa, sp.hpref, hp);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        // curl E_s / (i w mu0) = -i curl E_s / (w mu0): (x, y) -> (y, -x) / (w mu0)
        const double2 hs = make_double2(cs[k].y * sp.inv_wmu, -cs[k].x * sp.inv_wmu);
        H[3 * r + k] = cadd(hp[k], hs);
        if (Hs) Hs[3 * r + k] = hs;
    }
}

}  // namespace

// The element staging and the singular-source flag of every right-hand side
// are where the task says (the system's buffers, or the scratch of the
// allocation-free entry point). Tasks run in order, kRhsJobs to a launch, or
// fewer where the next one has another number of sources or shares its
// staging with one of them (a batch may name a system twice).
int launch_rhs_tasks(const RhsTask* tasks, int n, hipStream_t s) {
    for (int k0 = 0, nj = 0; k0 < n; k0 += nj) {
        const int ns = tasks[k0].ns;
        auto apart = [&](int k) {
            for (int q = k0; q < k; ++q)
                if (tasks[q].Rst == tasks[k].Rst) return false;
            return tasks[k].ns == ns;
        };
        for (nj = 1; nj < kRhsJobs && k0 + nj < n && apart(k0 + nj);) ++nj;
        RhsJobs jobs{};
        int most_t = 0, most_n = 0;
        for (int k = 0; k < nj; ++k) {
            const RhsTask& t = tasks[k0 + k];
            const petgem_system* sys = t.sys;
            RhsJob& j = jobs.j[k];
            j.n = sys->n_dof;
            j.T = sys->n_tets;
            j.stride = t.stride;
            j.fresh = t.fresh;
            j.xyz = sys->xyz;
            j.tets = reinterpret_cast<const int4*>(sys->tets);
            j.sigma = sys->sigma;
            j.sigma_bg = sys->sigma_bg;
            j.r_min = 1e-9 * sys->h_mean;
            for (int c = 0; c < ns; ++c) {
                j.sp[c] = make_src(t.src[c], sys->sigma_bg);
                j.wmu[c] = 2.0 * kPi * t.src[c].freq_hz * kMu0;
                j.b[c] = t.b + c * t.step;
            }
            j.Rst = t.Rst;
            j.flag = t.flag;
            j.iptr = sys->iptr;
            j.islot = sys->islot;
            most_n = std::max(most_n, j.n);
            if (!sys->layers.on) most_t = std::max(most_t, j.T);
        }
        const dim3 ge(ceil_div(most_t, 256), nj * ns), gg(ceil_div(most_n, 256), nj);
        if (most_t > 0) {
            RhsJobs whole = jobs;
            for (int k = 0; k < nj; ++k)
                if (tasks[k0 + k].sys->layers.on) whole.j[k].T = 0;
            hipLaunchKernelGGL(k_rhs_elem, ge, dim3(256), 0, s, whole, ns);
            PG_HIP(hipGetLastError());
        }
        for (int k = 0, m = 0; k < nj; k += m) {   // the layered sources of a system together
            const RhsTask& t = tasks[k0 + k];
            for (m = 1; k + m < nj && tasks[k0 + k + m].sys == t.sys;) ++m;
            if (!t.sys->layers.on) continue;
            petgem_source src[2 * kRhsJobs];
            double2* Rst[2 * kRhsJobs];
            int fresh = 0;
            for (int c = 0; c < m * ns; ++c) {
                const RhsTask& u = tasks[k0 + k + c / ns];
                src[c] = u.src[c % ns];
                Rst[c] = u.Rst + c % ns;
                fresh |= u.fresh;
            }
            PG_TRY(launch_rhs_layered(t.sys, src, Rst, m * ns, ns, fresh, t.flag, s));
        }
        if (ns == 2) hipLaunchKernelGGL(k_rhs_gather<2>, gg, dim3(256), 0, s, jobs);
        else hipLaunchKernelGGL(k_rhs_gather<1>, gg, dim3(256), 0, s, jobs);
        PG_HIP(hipGetLastError());
    }
    return PETGEM_OK;
}

// Staging of one system's right-hand sides side by side: a pair, and as many
// as fill a launch while they stay within kRhsStage (the Infinity Cache holds 256 MB,
// and the gather should find what the elements wrote there).
constexpr size_t kRhsStage = (size_t)128 << 20;
int rhs_staging(petgem_system* sys, int n_src, int* copies) {
    const size_t one = (size_t)6 * sys->n_tets;
    const int fit = (int)std::max<size_t>(2, kRhsStage / (one * sizeof(double2)));
    const int want = sys->rst_one ? 1 : std::min(std::min(n_src, 2 * kRhsJobs), fit);
    if (sys->rst_copies < want) {
        dfree(sys->Rst);
        sys->spare.back(sys->rst_held);
        sys->rst_copies = 0;
        // more than one source's is spare; without room for it one does
        const int64_t more = (int64_t)((want - 1) * one * sizeof(double2));
        if (want > 1 && sys->spare.room(more)) {
            const int rc = dalloc(&sys->Rst, one * want);
            if (rc != PETGEM_OK && rc != PETGEM_OUT_OF_MEMORY) return rc;
        }
        if (sys->Rst) {
            sys->rst_copies = want;
            sys->rst_held = more;
            sys->spare.used += more;
        } else {
            sys->rst_one = want > 1;
            PG_TRY(dalloc(&sys->Rst, one));
            sys->rst_copies = 1;
        }
    }
    *copies = std::min(want, sys->rst_copies);
    return PETGEM_OK;
}

// Right-hand sides of n_src sources of one system into b + k * step with the
// given row stride, staged in `copies` buffers from Rst on: two sources to a
// task where two buffers are there.
int launch_rhs_into(petgem_system* sys, const petgem_source* src, int n_src, double2* b, size_t step, int stride,
                    double2* Rst, int copies, int* flag, hipStream_t s) {
    const size_t one = (size_t)6 * sys->n_tets;
    copies = std::min(copies, 2 * kRhsJobs);
    // the layered sources' elements run in one launch however they are staged,
    // and a launch holds kRhsJobs tasks of the same number of sources
    const bool pairs = copies > 1 && !sys->layers.on;
    if (pairs) copies &= ~1;     // a pair keeps its two buffers from one round to the next
    for (int k0 = 0; k0 < n_src; k0 += copies) {
        RhsTask t[2 * kRhsJobs];
        const int nc = std::min(copies, n_src - k0);
        int nt = 0;
        for (int k = 0; k < nc;) {
            // a single last source finds no zeros of its own layout
            const int ns = pairs && k + 1 < nc ? 2 : 1;
            t[nt++] = RhsTask{sys, src + k0 + k, ns, b + (size_t)(k0 + k) * step, step, stride,
                              k0 == 0 || (ns == 1 && pairs), Rst + (size_t)k * one, flag};
            k += ns;
        }
        PG_TRY(launch_rhs_tasks(t, nt, s));
    }
    return PETGEM_OK;
}

int launch_rhs(petgem_system* sys, const petgem_source* src, int n_src, double2* b, size_t step, int stride,
               hipStream_t s) {
    int copies = 0;
    PG_TRY(rhs_staging(sys, n_src, &copies));
    return launch_rhs_into(sys, src, n_src, b, step, stride, sys->Rst, copies, sys->dflag, s);
}

int launch_receivers(const petgem_solution* sol, int32_t n_rx, double2* E, double2* Es,
                     hipStream_t s, bool magnetic) {
    const petgem_system* sys = sol->sys;
    if (sol->layers.on && magnetic) {
        set_error("the magnetic field over a layered background is not provided");
        return PETGEM_INVALID_ARG;
    }
    for (int32_t k = 0; k < sol->n_src; ++k) {
        SrcParams sp = make_src(sol->src[k], sol->sigma_bg);
        if (sol->layers.on) {
            PG_TRY(launch_receivers_layered(sol, k, n_rx, E + (size_t)k * n_rx * 3,
                                            Es ? Es + (size_t)k * n_rx * 3 : nullptr, s));
            continue;
        }
        if (magnetic) {
            hipLaunchKernelGGL(k_receivers_h, dim3(ceil_div(n_rx, 64)), dim3(64), 0, s, n_rx,
                               sys->rxc.xyz, sys->rxc.tet, sys->rxc.dof, sys->xyz,
                               reinterpret_cast<const int4*>(sys->tets),
                               sol->x + (size_t)k * sys->n_dof, sp, E + (size_t)k * n_rx * 3,
                               Es ? Es + (size_t)k * n_rx * 3 : nullptr);
            PG_HIP(hipGetLastError());
            continue;
        }
        hipLaunchKernelGGL(k_receivers, dim3(ceil_div(n_rx, 64)), dim3(64), 0, s, n_rx,
                           sys->rxc.xyz, sys->rxc.tet, sys->rxc.dof, sys->xyz,
                           reinterpret_cast<const int4*>(sys->tets),
                           sol->x + (size_t)k * sys->n_dof, sp, E + (size_t)k * n_rx * 3,
                           Es ? Es + (size_t)k * n_rx * 3 : nullptr);
        PG_HIP(hipGetLastError());
    }
    return PETGEM_OK;
}

}  // namespace petgem
