// Right-hand side and receiver fields over a layered background of two
// half-spaces (the layered primary field; see the comment below). The
// whole-space case is in rhs.hip.
#include <algorithm>
#include <cmath>

#include "device.h"
#include "internal.h"

namespace petgem {

namespace {

constexpr int kLE0[6] = {0, 0, 0, 1, 3, 2};
constexpr int kLE1[6] = {1, 2, 3, 2, 1, 3};

struct LSrc {
    double pos[3];
    double dir[3];
    double w;      // angular frequency
    double mom;    // moment I dS
};

// The sources of one launch and where their entries go: Rst[c] + (i T + t) ns.
constexpr int kLSrcs = 2 * kRhsJobs;
struct LTargets {
    int n, ns, fresh;             // fresh: zeros are still to be written where dsigma = 0
    LSrc src[kLSrcs];
    double2* Rst[kLSrcs];
};

// ------------------------------------------------- layered background
// Primary field of the dipole over two half-spaces (sigma_1 above z0, holding
// the source; sigma_2 below), from the TE / TM split of the whole-space field
// at the flat interface (Section 2: the primary field is that of the
// background model). With kappa the horizontal wavenumber,
// u_j = sqrt(kappa^2 - i w mu0 sigma_j) (Re u_j > 0),
//   r_TE = (u1 - u2)/(u1 + u2),   r_TM = (s2 u1 - s1 u2)/(s2 u1 + s1 u2),
//   t_TE = 2 u1/(u1 + u2),        t_TM = 2 s1 u1/(s2 u1 + s1 u2),
// and Hankel transforms in the horizontal offset rho at angle phi, c = m/(8 pi s1):
// above: E = E_whole-space(s1) + E_r with Z = (z - z0) + (zs - z0),
//   A_n = int k1^2 r_TE/u1 e^{-u1 Z} J_n k dk,  B_n = int u1 r_TM e^{-u1 Z} J_n k dk,
//   E1 = int r_TM e^{-u1 Z} J_1 k^2 dk,        V0 = int r_TM k^3/u1 e^{-u1 Z} J_0 dk;
//   x dipole: (c (A0 + B0 + cos2phi (A2 - B2)), c sin2phi (A2 - B2), -2c cos phi E1),
//   y dipole: (c sin2phi (A2 - B2), c (A0 + B0 - cos2phi (A2 - B2)), -2c sin phi E1),
//   z dipole: (2c cos phi E1, 2c sin phi E1, 2c V0);
// below, with e = exp(u2 (z - z0) - u1 (zs - z0)): the same with t for r,
//   TA_n = int k1^2 t_TE/u1 e J_n k dk, TB_n = int u2 t_TM e J_n k dk,
//   TE1 = int t_TM e J_1 k^2 dk, VE1 = int t_TM u2/u1 e J_1 k^2 dk, VV0 = int t_TM k^3/u1 e J_0 dk;
//   x dipole: (c (TA0 - TB0 + cos2phi (TA2 + TB2)), c sin2phi (TA2 + TB2), -2c cos phi TE1),
//   y dipole: (c sin2phi (TA2 + TB2), c (TA0 - TB0 - cos2phi (TA2 + TB2)), -2c sin phi TE1),
//   z dipole: (-2c cos phi VE1, -2c sin phi VE1, 2c VV0).
// Quadrature: 16-point Gauss-Legendre panels over [0, kmax], kmax = 50 /
// (decay length) (the exponential below e^-50 there), panels of width
// min(0.2 min|k_j|, pi / (2.5 rho)) up to 10 max|k_j| and min(pi / (2.5 rho),
// (kmax - that) / 48) beyond; the 64 lanes of a wavefront share the nodes
// and the sums are reduced by shuffles in a fixed order.
struct GL16 {
    double x[16], w[16];   // nodes and weights on [-1, 1]
};

// u = sqrt(k^2 - i b) (principal branch), b > 0, and |u|^-2: with n = k^4 + b^2
// and its reciprocal square root i, |u|^2 = n i and |u|^-2 = i
__device__ __forceinline__ double2 vert(double k2, double b, double& inv2) {
    const double n = k2 * k2 + b * b;
    inv2 = rsqrt(n);
    const double h = 0.5 * (n * inv2 + k2), ih = rsqrt(h);
    return make_double2(h * ih, -0.5 * b * ih);
}

__device__ __forceinline__ double2 cexp_(double2 z) {
    double s, c;
    sincos(z.y, &s, &c);
    const double e = exp(z.x);
    return make_double2(e * c, e * s);
}

// E_p at x; called by all 64 lanes of a wavefront with the same x, every
// lane gets the result.
__device__ void layered_E(const double x[3], const LSrc& sp, const Layers L, const GL16& gl, double2 E[3]) {
    const int lane = threadIdx.x & 63;
    const double w = sp.w;
    const double dx = x[0] - sp.pos[0], dy = x[1] - sp.pos[1];
    const double rho = sqrt(dx * dx + dy * dy);
    const double cph = rho > 0.0 ? dx / rho : 1.0, sph = rho > 0.0 ? dy / rho : 0.0;
    const double c2 = cph * cph - sph * sph, s2 = 2.0 * sph * cph;
    const double z = x[2] - L.z0, zs = sp.pos[2] - L.z0;
    const bool upper = z >= 0.0;
    const double dec = upper ? z + zs : zs - z;
    const double kmax = 50.0 / dec;
    const double s1 = L.s_up, s2s = L.s_dn;
    const double2 k1s = make_double2(0.0, w * kMu0 * s1), k2s = make_double2(0.0, w * kMu0 * s2s);
    const double ka1 = sqrt(w * kMu0 * s1), ka2 = sqrt(w * kMu0 * s2s);
    const double per = rho > 0.0 ? kPi / (2.5 * rho) : 1e300;
    const double kA = fmin(10.0 * fmax(ka1, ka2), kmax);
    const int nA = (int)ceil(kA / fmin(0.2 * fmin(ka1, ka2), per));
    const double hA = kA / nA;
    const int nB = kmax > kA ? (int)ceil((kmax - kA) / fmin(per, (kmax - kA) / 48.0)) : 0;
    const double hB = nB > 0 ? (kmax - kA) / nB : 0.0;
    const int N = 16 * (nA + nB);
    double2 I[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) I[j] = make_double2(0.0, 0.0);
    for (int n = lane; n < N; n += 64) {
        const int pnl = n >> 4, q = n & 15;
        const double a = pnl < nA ? pnl * hA : kA + (pnl - nA) * hB;
        const double h = pnl < nA ? hA : hB;
        const double kap = a + 0.5 * h * (1.0 + gl.x[q]);
        const double wt = 0.5 * h * gl.w[q];
        const double k2 = kap * kap;
        double i1, i2;
        const double2 u1 = vert(k2, k1s.y, i1), u2 = vert(k2, k2s.y, i2);
        const double2 iu1 = make_double2(u1.x * i1, -u1.y * i1);
        const double xr = kap * rho;
        const double j0v = j0(xr), j1v = j1(xr);
        const double j2v = xr > 1e-6 ? 2.0 * j1v / xr - j0v : 0.125 * xr * xr;
        // the two denominators u1 + u2 and s2 u1 + s1 u2 by one division
        const double2 sum = cadd(u1, u2), den = cadd(cscale(u1, s2s), cscale(u2, s1));
        const double na = cabs2(sum), nb = cabs2(den), iab = 1.0 / (na * nb);
        const double2 isum = cscale(cconj(sum), iab * nb), iden = cscale(cconj(den), iab * na);
        if (upper) {
            // (u1 - u2) / (u1 + u2) = (u1^2 - u2^2) / (u1 + u2)^2
            const double2 rte = cmul(make_double2(0.0, k2s.y - k1s.y), cmul(isum, isum));
            const double2 rtm = cmul(csub(cscale(u1, s2s), cscale(u2, s1)), iden);
            const double2 ex = cexp_(cscale(u1, -(z + zs)));
            const double2 fa = cscale(cmul(cmul(k1s, cmul(rte, iu1)), ex), kap * wt);
            const double2 fb = cscale(cmul(cmul(u1, rtm), ex), kap * wt);
            I[0] = cadd(I[0], cscale(fa, j0v));
            I[1] = cadd(I[1], cscale(fa, j2v));
            I[2] = cadd(I[2], cscale(fb, j0v));
            I[3] = cadd(I[3], cscale(fb, j2v));
            I[4] = cadd(I[4], cscale(cmul(rtm, ex), j1v * k2 * wt));
            I[5] = cadd(I[5], cscale(cmul(cmul(rtm, iu1), ex), k2 * kap * j0v * wt));
        } else {
            const double2 tte = cmul(cscale(u1, 2.0), isum);
            const double2 ttm = cmul(cscale(u1, 2.0 * s1), iden);
            const double2 ex = cexp_(csub(cscale(u2, z), cscale(u1, zs)));
            const double2 fa = cscale(cmul(cmul(k1s, cmul(tte, iu1)), ex), kap * wt);
            const double2 fb = cscale(cmul(cmul(u2, ttm), ex), kap * wt);
            I[0] = cadd(I[0], cscale(fa, j0v));
            I[1] = cadd(I[1], cscale(fa, j2v));
            I[2] = cadd(I[2], cscale(fb, j0v));
            I[3] = cadd(I[3], cscale(fb, j2v));
            const double2 te = cmul(ttm, ex);
            I[4] = cadd(I[4], cscale(te, j1v * k2 * wt));
            I[5] = cadd(I[5], cscale(cmul(cmul(te, u2), iu1), j1v * k2 * wt));
            I[6] = cadd(I[6], cscale(cmul(te, iu1), k2 * kap * j0v * wt));
        }
    }
#pragma unroll
    for (int j = 0; j < 7; ++j) { I[j].x = wave_sum(I[j].x); I[j].y = wave_sum(I[j].y); }
    const double c = sp.mom / (8.0 * kPi * s1);
    const double* p = sp.dir;
    double2 hx[3], hy[3], vz[3];
    if (upper) {
        const double2 S0 = cadd(I[0], I[2]), D2 = csub(I[1], I[3]);
        hx[0] = cscale(cadd(S0, cscale(D2, c2)), c); hx[1] = cscale(D2, c * s2); hx[2] = cscale(I[4], -2.0 * c * cph);
        hy[0] = cscale(D2, c * s2); hy[1] = cscale(csub(S0, cscale(D2, c2)), c); hy[2] = cscale(I[4], -2.0 * c * sph);
        vz[0] = cscale(I[4], 2.0 * c * cph); vz[1] = cscale(I[4], 2.0 * c * sph); vz[2] = cscale(I[5], 2.0 * c);
        double2 Ew[3];
        dipole_E(x, sp.pos, sp.dir, sqrt(0.5 * w * kMu0 * s1), sp.mom / (4.0 * kPi * s1), Ew);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            E[k] = cadd(Ew[k], cadd(cadd(cscale(hx[k], p[0]), cscale(hy[k], p[1])), cscale(vz[k], p[2])));
    } else {
        const double2 S0 = csub(I[0], I[2]), D2 = cadd(I[1], I[3]);
        hx[0] = cscale(cadd(S0, cscale(D2, c2)), c); hx[1] = cscale(D2, c * s2); hx[2] = cscale(I[4], -2.0 * c * cph);
        hy[0] = cscale(D2, c * s2); hy[1] = cscale(csub(S0, cscale(D2, c2)), c); hy[2] = cscale(I[4], -2.0 * c * sph);
        vz[0] = cscale(I[5], -2.0 * c * cph); vz[1] = cscale(I[5], -2.0 * c * sph); vz[2] = cscale(I[6], 2.0 * c);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            E[k] = cadd(cadd(cscale(hx[k], p[0]), cscale(hy[k], p[1])), cscale(vz[k], p[2]));
    }
}

// Right-hand side: dsigma_q = sigma_e - sigma_b(z_q) at each point of the
// 4-point rule (weights V/4), the layered E_p where it is non-zero; entries
// i w mu0 (V/4) sum_q dsigma_q N_i . E_p into Rst[i][t] (element-major planes,
// as the whole-space kernel).
// The Hankel transforms are all of the work (bound by double-precision
// arithmetic), and few elements have any: k_layered_hot lists them and writes
// the zeros of the others, then a block takes a listed element and source, a
// wavefront for each of its four points. One wavefront per element, the points
// in turn and one launch per source, left most of the chip idle: 337 us a
// source for some 400 elements with dsigma != 0; now 320 us for five sources.
constexpr double kQa = 0.58541019662496845446, kQb = 0.13819660112501051518;   // (5 + 3 sqrt 5)/20, (5 - sqrt 5)/20

__device__ __forceinline__ double dsigma_at(const double* __restrict__ xyz, int4 v, int q, double sigma, const Layers& L) {
    const int id[4] = {v.x, v.y, v.z, v.w};
    double zq = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) zq += (k == q ? kQa : kQb) * xyz[3 * (size_t)id[k] + 2];
    return sigma - (zq >= L.z0 ? L.s_up : L.s_dn);
}

__global__ void k_layered_clear(int* count) {
    if (threadIdx.x == 0) *count = 0;
}

__global__ void __launch_bounds__(256)
k_layered_hot(int T, const double* __restrict__ xyz, const int4* __restrict__ tets, const double* __restrict__ sigma,
              Layers L, LTargets out, int* __restrict__ list, int* __restrict__ count) {
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= T) return;
    bool any = false;
#pragma unroll
    for (int q = 0; q < 4; ++q) any = any || dsigma_at(xyz, tets[t], q, sigma[t], L) != 0.0;
    if (any) {
        list[atomicAdd(count, 1)] = t;   // in any order: every element has its own entries
        return;
    }
    for (int c = 0; c < out.n && out.fresh; ++c)
#pragma unroll
        for (int i = 0; i < 6; ++i) out.Rst[c][((size_t)i * T + t) * out.ns] = make_double2(0.0, 0.0);
}

__global__ void __launch_bounds__(256, 2)
k_rhs_layered(int T, const double* __restrict__ xyz, const int4* __restrict__ tets, const double* __restrict__ sigma,
              Layers L, LTargets out, GL16 gl, double r_min, const int* __restrict__ list,
              const int* __restrict__ count, int* __restrict__ flag) {
    __shared__ double2 Eq[4][3];
    const LSrc& sp = out.src[blockIdx.y];
    double2* __restrict__ Rst = out.Rst[blockIdx.y];
    const int nhot = *count, q = threadIdx.x >> 6;
    for (int h = blockIdx.x; h < nhot; h += gridDim.x) {
        const int t = list[h];
        const double ds = dsigma_at(xyz, tets[t], q, sigma[t], L);   // the same in every lane of the wave
        double2 E[3] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
        if (ds != 0.0) {
            const int4 v = tets[t];
            const int id[4] = {v.x, v.y, v.z, v.w};
            double x[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                x[k] = 0.0;
#pragma unroll
                for (int p = 0; p < 4; ++p) x[k] += (p == q ? kQa : kQb) * xyz[3 * (size_t)id[p] + k];
            }
            const double d0 = x[0] - sp.pos[0], d1 = x[1] - sp.pos[1], d2 = x[2] - sp.pos[2];
            if (d0 * d0 + d1 * d1 + d2 * d2 <= r_min * r_min && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
            layered_E(x, sp, L, gl, E);
        }
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int k = 0; k < 3; ++k) Eq[q][k] = cscale(E[k], ds);
        __syncthreads();
        if (threadIdx.x < 6) {
            TetGeom G;   // only now: the transforms need the registers
            tet_geometry(xyz, tets[t], G);
            // i w mu0 (V/4) R  ->  multiply by i: (x, y) -> (-y, x)
            const double f = sp.w * kMu0 * G.vol * 0.25;
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                if ((int)threadIdx.x != i) continue;
                const int a = kLE0[i], b = kLE1[i];
                double2 R = make_double2(0.0, 0.0);
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const double la = a == p ? kQa : kQb, lb = b == p ? kQa : kQb;
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const double nk = G.sl[i] * (la * G.g[b][k] - lb * G.g[a][k]);
                        R.x += nk * Eq[p][k].x;
                        R.y += nk * Eq[p][k].y;
                    }
                }
                Rst[((size_t)i * T + t) * out.ns] = make_double2(-f * R.y, f * R.x);
            }
        }
        __syncthreads();   // Eq is read before the next element writes it
    }
}

// Receivers: one wavefront per receiver (the layered E_p), lane 0 adds the
// interpolated secondary field (eq. 8).
__global__ void __launch_bounds__(64)
k_receivers_layered(int n_rx, const double* __restrict__ rxyz, const int32_t* __restrict__ rtet,
                    const int32_t* __restrict__ rdof, const double* __restrict__ xyz, const int4* __restrict__ tets,
                    const double2* __restrict__ x, Layers L, LSrc sp, GL16 gl, double2* __restrict__ E,
                    double2* __restrict__ Es) {
    const int r = blockIdx.x;
    const double p[3] = {rxyz[3 * r], rxyz[3 * r + 1], rxyz[3 * r + 2]};
    double2 ep[3];
    layered_E(p, sp, L, gl, ep);
    if (threadIdx.x != 0) return;
    TetGeom G;
    tet_geometry(xyz, tets[rtet[r]], G);
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
        const int d = rdof[6 * r + i];
        if (d < 0) continue;
        const double2 v = x[d];
        const int a = kLE0[i], b = kLE1[i];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double nk = G.sl[i] * (lam[a] * G.g[b][k] - lam[b] * G.g[a][k]);
            es[k].x += nk * v.x;
            es[k].y += nk * v.y;
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        E[3 * r + k] = cadd(ep[k], es[k]);
        if (Es) Es[3 * r + k] = es[k];
    }
}

// Gauss-Legendre nodes and weights on [-1, 1]: Newton on P_16 from
// Chebyshev-like guesses, P_n and its derivative by the three-term recurrence.
GL16 make_gl16() {
    GL16 g;
    const int n = 16;
    for (int i = 0; i < n; ++i) {
        double x = std::cos(kPi * (i + 0.75) / (n + 0.5));
        double dp = 1.0;
        for (int it = 0; it < 100; ++it) {
            double p0 = 1.0, p1 = x;
            for (int k = 2; k <= n; ++k) {
                const double p2 = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            dp = n * (x * p1 - p0) / (x * x - 1.0);
            const double step = p1 / dp;
            x -= step;
            if (std::fabs(step) < 1e-16) break;
        }
        g.x[i] = x;
        g.w[i] = 2.0 / ((1.0 - x * x) * dp * dp);
    }
    return g;
}

const GL16& gl16() {
    static const GL16 g = make_gl16();
    return g;
}

LSrc make_lsrc(const petgem_source& s) {
    LSrc p;
    for (int k = 0; k < 3; ++k) { p.pos[k] = s.pos[k]; p.dir[k] = s.dir[k]; }
    p.w = 2.0 * kPi * s.freq_hz;
    p.mom = s.moment;
    return p;
}

}  // namespace

int launch_rhs_layered(petgem_system* sys, const petgem_source* src, double2* const* Rst, int n, int ns, int fresh,
                       int* flag, hipStream_t s) {
    LTargets out{};
    for (int c = 0; c < n; ++c) {
        if (!(src[c].pos[2] > sys->layers.z0)) {
            set_error("layered background: the source must lie above the interface");
            return PETGEM_INVALID_ARG;
        }
        out.src[c] = make_lsrc(src[c]);
        out.Rst[c] = Rst[c];
    }
    out.n = n;
    out.ns = ns;
    out.fresh = fresh;
    hipLaunchKernelGGL(k_layered_clear, dim3(1), dim3(64), 0, s, sys->hot);
    hipLaunchKernelGGL(k_layered_hot, dim3(ceil_div(sys->n_tets, 256)), dim3(256), 0, s, sys->n_tets, sys->xyz,
                       reinterpret_cast<const int4*>(sys->tets), sys->sigma, sys->layers, out, sys->hot + 1, sys->hot);
    hipLaunchKernelGGL(k_rhs_layered, dim3(std::min(sys->n_tets, 4096), n), dim3(256), 0, s, sys->n_tets, sys->xyz,
                       reinterpret_cast<const int4*>(sys->tets), sys->sigma, sys->layers, out, gl16(),
                       1e-9 * sys->h_mean, sys->hot + 1, sys->hot, flag);
    PG_HIP(hipGetLastError());
    return PETGEM_OK;
}

int launch_receivers_layered(const petgem_solution* sol, int k, int32_t n_rx, double2* E, double2* Es,
                             hipStream_t s) {
    const petgem_system* sys = sol->sys;
    hipLaunchKernelGGL(k_receivers_layered, dim3(n_rx), dim3(64), 0, s, n_rx, sys->rxc.xyz, sys->rxc.tet,
                       sys->rxc.dof, sys->xyz, reinterpret_cast<const int4*>(sys->tets),
                       sol->x + (size_t)k * sys->n_dof, sol->layers, make_lsrc(sol->src[k]), gl16(), E, Es);
    PG_HIP(hipGetLastError());
    return PETGEM_OK;
}

}  // namespace petgem
