// Element matrices and deterministic global assembly (Section 3, eq. 9;
// Section 4; Appendix B, eqs. B.13-B.15).
//
// k_elem_km: one thread per tetrahedron computes the 21 unique entries of the
//   symmetric 6x6 curl-curl matrix K^e and of sigma_e M^e in closed form and
//   stores them as pairs {K^e, sigma_e M^e}, structure-of-arrays ([21][T]):
//   the writes here are coalesced and the gather fetches both values of a
//   contribution with one 16-byte load (two arrays: twice the gathers, and
//   the gathers bound it). It also keeps the conductivities it used.
// k_gather: one thread per nonzero sums its element contributions in
//   increasing element order (fixed lists built on the host), so the assembled
//   values are bitwise reproducible and bitwise symmetric, without atomics.
//   The threads of the diagonal also write it to its own arrays.
#include "device.h"
#include "internal.h"

namespace petgem {

namespace {

constexpr int kE0[6] = {0, 0, 0, 1, 3, 2};
constexpr int kE1[6] = {1, 2, 3, 2, 1, 3};

__global__ void __launch_bounds__(256)
k_elem_km(int T, const double* __restrict__ xyz, const int4* __restrict__ tets,
          const double* __restrict__ sigma, double* __restrict__ sigma_kept, double2* __restrict__ st) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    TetGeom G;
    tet_geometry(xyz, tets[t], G);
    // curl N_i = 2 s_i l_i grad(lambda_a) x grad(lambda_b)
    double C[6][3];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const double* ga = G.g[kE0[i]];
        const double* gb = G.g[kE1[i]];
        double f = 2.0 * G.sl[i];
        C[i][0] = f * (ga[1] * gb[2] - ga[2] * gb[1]);
        C[i][1] = f * (ga[2] * gb[0] - ga[0] * gb[2]);
        C[i][2] = f * (ga[0] * gb[1] - ga[1] * gb[0]);
    }
    // g_pq = grad lambda_p . grad lambda_q
    double gg[4][4];
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int q = p; q < 4; ++q) {
            double v = G.g[p][0] * G.g[q][0] + G.g[p][1] * G.g[q][1] + G.g[p][2] * G.g[q][2];
            gg[p][q] = v;
            gg[q][p] = v;
        }
    const double V = G.vol;
    const double sg = sigma[t], sV = sg * V * (1.0 / 20.0);
    if (sigma_kept != sigma) sigma_kept[t] = sg;
    int k = 0;
#pragma unroll
    for (int i = 0; i < 6; ++i) {
#pragma unroll
        for (int j = i; j < 6; ++j, ++k) {
            double kij = V * (C[i][0] * C[j][0] + C[i][1] * C[j][1] + C[i][2] * C[j][2]);
            // int lambda_p lambda_q = V (1 + delta_pq) / 20
            const int a = kE0[i], b = kE1[i], c = kE0[j], d = kE1[j];
            double m = (1.0 + (a == c)) * gg[b][d] - (1.0 + (a == d)) * gg[b][c]
                     - (1.0 + (b == c)) * gg[a][d] + (1.0 + (b == d)) * gg[a][c];
            st[(size_t)k * T + t] = make_double2(kij, sV * G.sl[i] * G.sl[j] * m);
        }
    }
}

// Packed entries (i, i) of an element matrix: a bit for each.
constexpr unsigned kDiagEntries = 1u << 0 | 1u << 6 | 1u << 11 | 1u << 15 | 1u << 18 | 1u << 20;

__global__ void __launch_bounds__(256)
k_gather(int64_t nnz, int T, const int32_t* __restrict__ cptr, const int32_t* __restrict__ cidx,
         const int32_t* __restrict__ col, const double2* __restrict__ st, double* __restrict__ K,
         double* __restrict__ Ms, double* __restrict__ Kd, double* __restrict__ Msd) {
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nnz) return;
    double sk = 0.0, sm = 0.0;
    const int32_t c0 = cptr[k], c1 = cptr[k + 1];
    int32_t first = 0;
    // four contribution indices, then their values, in flight at a time; the
    // sums keep the list order
    for (int32_t c = c0; c < c1; c += 4) {
        int32_t idx[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) idx[q] = c + q < c1 ? cidx[c + q] : -1;
        if (c == c0) first = idx[0];
        double2 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = idx[q] >= 0 ? st[idx[q]] : make_double2(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (idx[q] >= 0) {
                sk += v[q].x;
                sm += v[q].y;
            }
    }
    K[k] = sk;
    Ms[k] = sm;
    // a nonzero that gathers diagonal element entries is its row's diagonal
    if (kDiagEntries >> ((unsigned)first / (unsigned)T) & 1u) {
        const int32_t r = col[k];
        Kd[r] = sk;
        Msd[r] = sm;
    }
}

// D = diag(A) = Kd - i w mu0 Msd and its inverse.
__global__ void k_jacobi(int n, double wmu, const double* __restrict__ Kd,
                         const double* __restrict__ Msd, double2* __restrict__ dvec,
                         double2* __restrict__ dinv) {
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n) return;
    double2 d = make_double2(Kd[r], -wmu * Msd[r]);
    dvec[r] = d;
    dinv[r] = cdiv(make_double2(1.0, 0.0), d);
}

// Ahat_k = (K_k - i w mu0 Ms_k) / D_col(k): the right-Jacobi-preconditioned
// operator A D^{-1} of the double-precision GMRES. A thread per nonzero (one
// per row reads and writes with a row's stride between lanes: 778 us for 13.8M
// nonzeros).
__global__ void __launch_bounds__(256)
k_ahat(int64_t nnz, double wmu, const int32_t* __restrict__ col, const double* __restrict__ K,
       const double* __restrict__ Ms, const double2* __restrict__ dinv, double2* __restrict__ Ahat) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k < nnz) Ahat[k] = cmul(make_double2(K[k], -wmu * Ms[k]), dinv[col[k]]);
}

// y = A x = K x - i w mu0 M_sigma x on the assembled matrices, eight lanes to
// a row (16 nonzeros on average), two nonzeros of each in flight: 20 bytes a
// nonzero, where forming A D^{-1} first moves another 36 of them.
__global__ void __launch_bounds__(256)
k_spmv_km(int n, double wmu, const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
          const double* __restrict__ K, const double* __restrict__ Ms, const double2* __restrict__ x,
          double2* __restrict__ y) {
    constexpr int G = 8;
    const int row = (xcd_block(blockIdx.x, gridDim.x) * 256 + (int)threadIdx.x) / G;
    const int lane = threadIdx.x & (G - 1);
    if (row >= n) return;
    double2 ak = make_double2(0.0, 0.0), am = ak;
    const int32_t e = rp[row + 1];
    for (int32_t k0 = rp[row] + lane; k0 < e; k0 += 2 * G) {
        const int32_t k1 = k0 + G;
        const bool two = k1 < e;
        const int32_t c0 = col[k0], c1 = two ? col[k1] : c0;
        const double a0 = K[k0], m0 = Ms[k0], a1 = two ? K[k1] : 0.0, m1 = two ? Ms[k1] : 0.0;
        const double2 v0 = x[c0], v1 = two ? x[c1] : make_double2(0.0, 0.0);
        ak.x += a0 * v0.x; ak.y += a0 * v0.y; am.x += m0 * v0.x; am.y += m0 * v0.y;
        ak.x += a1 * v1.x; ak.y += a1 * v1.y; am.x += m1 * v1.x; am.y += m1 * v1.y;
    }
    double2 v = make_double2(ak.x + wmu * am.y, ak.y - wmu * am.x);
    // over the eight lanes of the row
    v.x = sum8(v.x);
    v.y = sum8(v.y);
    if (lane == 0) y[row] = v;
}

__global__ void k_to_f32(int64_t n, const double* __restrict__ a, const double* __restrict__ b,
                         float* __restrict__ a32, float* __restrict__ b32) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    a32[i] = (float)a[i];
    b32[i] = (float)b[i];
}

}  // namespace

int launch_assembly(petgem_system* sys, const double* sigma, hipStream_t s) {
    const int T = sys->n_tets;
    hipLaunchKernelGGL(k_elem_km, dim3(ceil_div(T, 256)), dim3(256), 0, s, T, sys->xyz,
                       reinterpret_cast<const int4*>(sys->tets), sigma, sys->sigma, sys->KMst);
    PG_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_gather, dim3(ceil_div(sys->nnz, 256)), dim3(256), 0, s, sys->nnz, T, sys->cptr, sys->cidx,
                       sys->col, sys->KMst, sys->K, sys->Ms, sys->Kd, sys->Msd);
    PG_HIP(hipGetLastError());
    sys->cached_freq = sys->diag_freq = -1.0;   // operators derived from K, Ms are stale
    sys->have32 = false;
    for (Resident& L : sys->res) {
        L.values = false;
        L.a_freq = -1.0;
    }
    return PETGEM_OK;
}

int launch_diag(petgem_system* sys, double freq, hipStream_t s) {
    if (sys->diag_freq == freq) return PETGEM_OK;
    const int n = sys->n_dof;
    if (!sys->dvec) PG_TRY(dalloc(&sys->dvec, n));
    if (!sys->dinv) PG_TRY(dalloc(&sys->dinv, n));
    hipLaunchKernelGGL(k_jacobi, dim3(ceil_div(n, 256)), dim3(256), 0, s, n, 2.0 * kPi * freq * kMu0, sys->Kd,
                       sys->Msd, sys->dvec, sys->dinv);
    PG_HIP(hipGetLastError());
    sys->diag_freq = freq;
    return PETGEM_OK;
}

int launch_freq_prep(petgem_system* sys, double freq, hipStream_t s) {
    PG_TRY(launch_diag(sys, freq, s));
    if (sys->cached_freq == freq) return PETGEM_OK;
    if (!sys->Ahat) PG_TRY(dalloc(&sys->Ahat, sys->nnz));
    hipLaunchKernelGGL(k_ahat, dim3(ceil_div(sys->nnz, 256)), dim3(256), 0, s, sys->nnz, 2.0 * kPi * freq * kMu0,
                       sys->col, sys->K, sys->Ms, sys->dinv, sys->Ahat);
    PG_HIP(hipGetLastError());
    sys->cached_freq = freq;
    return PETGEM_OK;
}

int launch_spmv(petgem_system* sys, double freq, const double2* x, double2* y, hipStream_t s) {
    const int n = sys->n_dof;
    // a block writes y while others still read x: vectors that overlap are
    // multiplied from a copy
    const uintptr_t a = reinterpret_cast<uintptr_t>(x), b = reinterpret_cast<uintptr_t>(y);
    if (a < b + sizeof(double2) * n && b < a + sizeof(double2) * n) {
        if (!sys->xtmp) PG_TRY(dalloc(&sys->xtmp, (size_t)n));
        PG_HIP(hipMemcpyAsync(sys->xtmp, x, sizeof(double2) * n, hipMemcpyDeviceToDevice, s));
        x = sys->xtmp;
    }
    hipLaunchKernelGGL(k_spmv_km, dim3(ceil_div((int64_t)n * 8, 256)), dim3(256), 0, s, n, 2.0 * kPi * freq * kMu0,
                       sys->row_ptr, sys->col, sys->K, sys->Ms, x, y);
    PG_HIP(hipGetLastError());
    sys->tune_freq = freq;
    return PETGEM_OK;
}

int ensure_fp32(petgem_system* sys, hipStream_t s) {
    if (sys->have32) return PETGEM_OK;
    if (!sys->K32) {
        PG_TRY(dalloc(&sys->K32, sys->nnz));
        PG_TRY(dalloc(&sys->Ms32, sys->nnz));
    }
    hipLaunchKernelGGL(k_to_f32, dim3(ceil_div(sys->nnz, 256)), dim3(256), 0, s, sys->nnz, sys->K,
                       sys->Ms, sys->K32, sys->Ms32);
    PG_HIP(hipGetLastError());
    sys->have32 = true;
    sys->sell32.values = false;
    sys->ssor32.values = false;
    return PETGEM_OK;
}

}  // namespace petgem
