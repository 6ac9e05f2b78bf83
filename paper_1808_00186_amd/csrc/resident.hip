// Krylov solves in one launch: the inner complex64 COCG of the mixed-precision
// solve with the operator resident in the register files, instead of two to
// five kernels per iteration, and the plain GMRES (at the end of the file).
//
// What it replaces and why. An iteration of the kernel-per-phase form streams
// the operator (12 B a nonzero) and five vectors through the Infinity Cache
// and pays two to three kernel boundaries; on a 434k-DOF mesh that is 28 us,
// on a 3k-DOF mesh 14 us, nearly all of it launch latency and drain. The
// chip's 256 compute units hold 128 MB of registers and 40 MB of LDS, more
// than the operator of that mesh (70 MB with 16-bit column indices), so each
// workgroup takes a run of up to 2,048 consecutive rows (spatially compact:
// the rows are in Morton order), loads its entries into registers once per
// inner solve, and keeps r, x, D^-1 and p in LDS. Per iteration only the
// search direction at the rows' outer neighbours (the halo) and nine partial
// sums travel between workgroups.
//
// The recurrence is the fused step's (fused_scalars in cocg.h): the product
// q = A p with the sums p^T q, q^T D^-1 r, q^T D^-1 q, then r -= alpha q,
// z = D^-1 r, x += alpha p, p = z + beta p with the sums r^T z, |r|^2 that the
// next step's convergence test uses. D^-1 is kept in double.
//
// Exchange between workgroups of one domain (the workgroups of one mesh and
// column), all through agent-scope atomic loads and stores of 64-bit words,
// which bypass the non-coherent L2s of the XCDs, and without a fence:
// A word that is not yet written holds all ones (a NaN no finite recurrence
// produces), so a word validates itself and the reader polls the data, not a
// flag. Each array has three copies used in turn, and publishing copy k goes
// with clearing one's words of copy k+1. Its last readers are done by then: a
// workgroup publishes the sums of step k after it has read everybody's of
// step k-1, which they publish after they have read those of step k-2 and the
// p of step k-1. The clearing stores are waited for before the next sums are
// published, and nobody polls that copy before having seen those.
//   * p: the rows' new search direction, gathered by the neighbours. (Writing
//     each row into the halos that need it, to be read in order, measured
//     0.4 us slower a step on 6 workgroups and equal on 251: the step is bound
//     by the latency of the exchange, not by its bytes.)
//   * sums: nine doubles of every workgroup. Up to 32 workgroups read each
//     other's; beyond that the first of every 32 sums its group's and writes
//     the result once for each group to read.
//     Everybody reading everybody's took 7.9 us a step at 251 workgroups (the
//     polls of one small array queue at its memory channels), two levels
//     through one array 5.8 us, this 4.3 us.
// Every wait is bounded (kResSpin polls, or the caller's); one that runs out raises the
// launch's abort flag, every workgroup then leaves, and the host solves again
// with the kernel-per-phase form. All workgroups of a launch are resident
// together: at most one per compute unit, launched cooperatively.
// Sums are taken in a fixed order (lanes, waves, workgroups), so results do
// not depend on timing, and every workgroup computes the same scalars.
#include <algorithm>
#include <vector>

#include "cocg.h"
#include "device.h"
#include "internal.h"

namespace petgem {

namespace {

typedef unsigned long long u64;

constexpr int kResT = 512;          // threads of a workgroup
constexpr int kResW = kResT / kWave;
constexpr int kResK = 4;            // rows of a thread
constexpr int kResRows = kResT * kResK;
constexpr int kResCh = 18;          // chunks of 4 entries of a thread: 72 entries, 180 of 256 registers
constexpr int kResMaxG = 256;       // workgroups of a domain: 8 groups of 32
constexpr int kResV = 9;            // doubles summed per step
constexpr int kResLds = 160 * 1024 - 2048;
constexpr int kResSpin = 1 << 21;   // polls of one wait (default), about a second
constexpr u64 kResEmpty = ~0ull;

constexpr int kResHaloLds = kResMaxG * kResRows / 32 * 8;   // k_res_halo: two words for 32 rows of the largest mesh

// The 64-row slice of wave w that its row slot k takes: slices are sorted by
// row length, and alternating the direction evens out the waves' entries.
__host__ __device__ constexpr int res_slice(int w, int k) { return k * kResW + ((k & 1) ? kResW - 1 - w : w); }

// Words of one copy of the sums: an area for the workgroups of each group,
// and beyond one group an area for the groups' sums in each group.
constexpr int kResArea = 544;       // words from one area to the next (4 KB and 256 B: other memory channels)
__host__ __device__ constexpr size_t res_words(int G) {
    return (size_t)kResArea * (G > 32 ? 2 * ((G + 31) / 32) : 1);
}

// One domain: G workgroups from logical block block0 on, columns c0, c0 +
// cstep, ... of a block of C columns.
struct ResDom {
    int block0, G, n, rw, rwcap, hcap, hmax, C, c0, cstep;
    const int32_t *rows, *wend, *halo, *nh, *rp;
    const uint2* idx;
    const float4 *K, *M;
    float4 *Kw, *Mw;                  // the same arrays, for k_res_vals
    const double *K64, *M64;
    const double *Kd, *Md, *wmu;
    const double2* R64;
    float2* Xi;
    ColState* st;
    u64 *words, *pex;
};

__device__ __forceinline__ void put(u64* p, u64 v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 get(const u64* p) {
    return __hip_atomic_load(const_cast<u64*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool aborted(const int* flag) {
    return __hip_atomic_load(const_cast<int*>(flag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}
__device__ __forceinline__ u64 bits(float2 v) {
    return (u64)__float_as_uint(v.x) | ((u64)__float_as_uint(v.y) << 32);
}
__device__ __forceinline__ float2 unbits(u64 v) {
    return f2(__uint_as_float((unsigned)v), __uint_as_float((unsigned)(v >> 32)));
}

// The thread's number, not known to be the same as before: what follows from
// it (LDS and exchange addresses) would otherwise be kept in registers across
// the iterations, which the operator needs.
__device__ __forceinline__ int fresh_thread() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// N words once all are written; false when the wait ran out. Words with no
// address (null) are zero.
template <int N>
__device__ __forceinline__ bool wait_words(const u64* const* a, int polls, const int* abort, u64* v) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = a[i] ? get(a[i]) : 0ull;
#pragma unroll
    for (int i = 0; i < N; ++i)
        for (int spin = 0; v[i] == kResEmpty; ++spin) {
            if (spin >= polls || ((spin & 1023) == 1023 && aborted(abort))) return false;
            v[i] = get(a[i]);
        }
    return true;
}

// ------------------------------------------------------------ the layout
// One layout to build; its G workgroups are blocks block0 .. of both kernels,
// so the layouts of a whole batch are two launches (one at a time, 200 small
// meshes took 20 ms: eight workgroups do not fill the chip).
struct ResLay {
    int block0, n, rw, rwcap, hmax;
    const int32_t *rp, *col;
    int32_t *rows, *wend, *halo, *nh, *pos;
    uint2* idx;
    int* stat;
};

// Workgroup g takes rows [g rw, g rw + rw), ordered by length (longest first,
// then by index). wend[g][wave][k]: the chunk at which the wave's row slot k
// ends. stat[0]: most chunks of a wave.
__global__ void __launch_bounds__(1024)
k_res_sort(const ResLay* __restrict__ lays, const int* __restrict__ blk) {
    const ResLay& y = lays[blk[blockIdx.x]];
    const int n = y.n, rw = y.rw, rwcap = y.rwcap;
    const int32_t* __restrict__ rp = y.rp;
    int32_t* __restrict__ rows = y.rows;
    int32_t* __restrict__ wend = y.wend;
    int32_t* __restrict__ pos = y.pos;
    int* __restrict__ stat = y.stat;
    // lengths as 16 bits, eight to a read: the ranks of 1,516 rows in 20 us, not 86
    __shared__ __align__(16) uint16_t len[kResRows];
    __shared__ int slen[kResRows];
    const int g = (int)blockIdx.x - y.block0, r0 = g * rw, R = min(n - r0, rw), t = threadIdx.x;
    for (int i = t; i < kResRows; i += 1024) len[i] = i < R ? (uint16_t)min(rp[r0 + i + 1] - rp[r0 + i], 0xffff) : 0;
    for (int s = R + t; s < rwcap; s += 1024) rows[(size_t)g * rwcap + s] = -1;
    __syncthreads();
    for (int i = t; i < R; i += 1024) {
        const int l = len[i];
        int rank = 0;
        for (int j = 0; j < R; j += 8) {   // rows past R have length 0 and never rank before
            const uint4 v = *reinterpret_cast<const uint4*>(len + j);
            const unsigned w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int lj = (int)((w[u / 2] >> (16 * (u & 1))) & 0xffffu);
                rank += (lj > l) || (lj == l && j + u < i);
            }
        }
        slen[rank] = l;
        rows[(size_t)g * rwcap + rank] = r0 + i;
        pos[r0 + i] = g * rwcap + rank;
    }
    __syncthreads();
    if (t < kResW) {
        int end = 0;
        for (int k = 0; k < kResK; ++k) {
            const int s = res_slice(t, k) * 64;
            if (s < R) end += (slen[s] + 3) / 4;
            wend[((size_t)g * kResW + t) * kResK + k] = end;
        }
        atomicMax(&stat[0], end);
    }
}

// The halo of workgroup g (the distinct columns outside its rows, ascending,
// as positions in the exchange array) and the 16-bit LDS offset of every
// entry (8 bytes a row: own rows first, then the halo from rwcap on). A bitmap of all rows
// finds the distinct columns. stat[1]: most halo rows of a workgroup.
__global__ void __launch_bounds__(1024)
k_res_halo(const ResLay* __restrict__ lays, const int* __restrict__ blk) {
    const ResLay& y = lays[blk[blockIdx.x]];
    const int n = y.n, rw = y.rw, rwcap = y.rwcap, hmax = y.hmax;
    const int32_t *__restrict__ rp = y.rp, *__restrict__ col = y.col;
    const int32_t *__restrict__ rows = y.rows, *__restrict__ wend = y.wend, *__restrict__ pos = y.pos;
    int32_t *__restrict__ halo = y.halo, *__restrict__ nh = y.nh;
    uint2* __restrict__ idx = y.idx;
    int* __restrict__ stat = y.stat;
    extern __shared__ unsigned lds_u[];
    __shared__ int scan[1024];
    const int nw = (n + 31) / 32, t = threadIdx.x;
    unsigned* bm = lds_u;
    unsigned* pre = lds_u + nw;
    const int g = (int)blockIdx.x - y.block0, r0 = g * rw, R = min(n - r0, rw);
    for (int i = t; i < nw; i += 1024) bm[i] = 0u;
    __syncthreads();
    const int e0 = rp[r0], e1 = rp[r0 + R];
    for (int e = e0 + t; e < e1; e += 1024) {
        const int c = col[e];
        if (c < r0 || c >= r0 + R) atomicOr(&bm[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    const int per = (nw + 1023) / 1024, w0 = min(t * per, nw), w1 = min(w0 + per, nw);
    int mine = 0;
    for (int i = w0; i < w1; ++i) mine += __popc(bm[i]);
    scan[t] = mine;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int v = t >= d ? scan[t - d] : 0;
        __syncthreads();
        scan[t] += v;
        __syncthreads();
    }
    const int total = scan[1023];
    int run = scan[t] - mine;
    for (int i = w0; i < w1; ++i) {
        pre[i] = (unsigned)run;
        for (unsigned m = bm[i]; m; m &= m - 1, ++run)
            if (run < hmax) halo[(size_t)g * hmax + run] = pos[i * 32 + __ffs(m) - 1];
    }
    if (t == 0) {
        nh[g] = min(total, hmax);
        atomicMax(&stat[1], total);
    }
    __syncthreads();
    if (total > hmax) return;   // this layout is not used
    const int wave = (t >> 6) & (kResW - 1), lane = t & 63;
    if (t >= kResT) return;
    const size_t base = ((size_t)g * kResW + wave) * kResCh * 64 + lane;
    int ch = 0;
    for (int k = 0; k < kResK; ++k) {
        const int end = min(wend[((size_t)g * kResW + wave) * kResK + k], kResCh);
        const int s = res_slice(wave, k) * 64 + lane;
        const int row = s < R ? rows[(size_t)g * rwcap + s] : -1;
        const int b = row >= 0 ? rp[row] : 0, l = row >= 0 ? rp[row + 1] - b : 0;
        for (int q = 0; ch < end; ++ch, q += 4) {
            unsigned v[4];
            for (int u = 0; u < 4; ++u) {
                unsigned o = s < rwcap ? (unsigned)s : 0u;   // padding: the row itself, with zero values
                if (q + u < l) {
                    const int c = col[b + q + u];
                    o = (c >= r0 && c < r0 + R) ? (unsigned)(pos[c] - g * rwcap)
                                                : (unsigned)rwcap + pre[c >> 5] + __popc(bm[c >> 5] & ((1u << (c & 31)) - 1u));
                }
                v[u] = o;
            }
            idx[base + (size_t)ch * 64] = make_uint2(8u * (v[0] | (v[1] << 16)), 8u * (v[2] | (v[3] << 16)));
        }
    }
}

// The complex64 operator's values in the order the registers take them, from
// the assembled doubles: one wave per (workgroup, wave) of every domain.
__global__ void __launch_bounds__(256)
k_res_vals(const ResDom* __restrict__ doms, const int* __restrict__ blk_dom) {
    const int lb = blockIdx.x / 2;
    const ResDom& d = doms[blk_dom[lb]];
    const int g = lb - d.block0;
    const int wave = (blockIdx.x & 1) * 4 + ((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int R = min(d.n - g * d.rw, d.rw);
    const size_t base = ((size_t)g * kResW + wave) * kResCh * 64 + lane;
    int ch = 0;
    for (int k = 0; k < kResK; ++k) {
        const int end = d.wend[((size_t)g * kResW + wave) * kResK + k];
        const int s = res_slice(wave, k) * 64 + lane;
        const int row = s < R ? d.rows[(size_t)g * d.rwcap + s] : -1;
        const int b = row >= 0 ? d.rp[row] : 0, l = row >= 0 ? d.rp[row + 1] - b : 0;
        for (int q = 0; ch < end; ++ch, q += 4) {
            float kv[4], mv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                kv[u] = q + u < l ? (float)d.K64[b + q + u] : 0.f;
                mv[u] = q + u < l ? (float)d.M64[b + q + u] : 0.f;
            }
            d.Kw[base + (size_t)ch * 64] = make_float4(kv[0], kv[1], kv[2], kv[3]);
            d.Mw[base + (size_t)ch * 64] = make_float4(mv[0], mv[1], mv[2], mv[3]);
        }
    }
}

__global__ void k_res_clear(size_t n_words, u64* __restrict__ words, size_t n_pex, u64* __restrict__ pex,
                            int* __restrict__ abort) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n_words) words[i] = kResEmpty;
    if (i < n_pex) pex[i] = kResEmpty;
    if (i == 0) *abort = 0;
}

// ------------------------------------------------------------ the solve
__global__ void __launch_bounds__(kResT)
k_res_cocg(const ResDom* __restrict__ doms, const int* __restrict__ blk_dom, int max_inner, int polls,
           int* __restrict__ abort) {
    extern __shared__ double2 lds_d[];
    __shared__ double wsum[kResW][kResV];
    __shared__ double tot[kResV + 1];
    __shared__ ColState S;
    __shared__ float4 step;      // alpha, beta
    __shared__ int live, fail1, fail2;
    const int lb = xcd_block(blockIdx.x, gridDim.x);
    const ResDom d = doms[blk_dom[lb]];
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int G = d.G, g = lb - d.block0, rwcap = d.rwcap;
    const int R = min(d.n - g * d.rw, d.rw);
    // p first (own rows, then the halo): its entries' indices are byte offsets
    float2* const pl = reinterpret_cast<float2*>(lds_d);
    double2* const dl = reinterpret_cast<double2*>(pl + rwcap + d.hcap);   // D^-1
    float2* const xl = reinterpret_cast<float2*>(dl + rwcap);
    float2* const yl = xl + rwcap;
    float2* const rl = yl + rwcap;
    int* const hl = reinterpret_cast<int*>(rl + rwcap);                  // places of the halo
    const int nh = d.nh[g];
    for (int h = t; h < nh; h += kResT) hl[h] = d.halo[(size_t)g * d.hmax + h];
    if (t == 0) { fail1 = 0; fail2 = 0; }
    // the operator into registers
    int end[kResK], sb[kResK];
#pragma unroll
    for (int k = 0; k < kResK; ++k) {
        end[k] = __builtin_amdgcn_readfirstlane(d.wend[((size_t)g * kResW + wave) * kResK + k]);
        sb[k] = res_slice(wave, k) * 64;
    }
    const int nch = end[kResK - 1];
    float4 kv[kResCh], mv[kResCh];
    uint2 ix[kResCh];
    {
        const size_t base = ((size_t)g * kResW + wave) * kResCh * 64 + lane;
#pragma unroll
        for (int c = 0; c < kResCh; ++c) {
            if (c < nch) {
                kv[c] = d.K[base + (size_t)c * 64];
                mv[c] = d.M[base + (size_t)c * 64];
                ix[c] = d.idx[base + (size_t)c * 64];
            } else {
                kv[c] = mv[c] = make_float4(0.f, 0.f, 0.f, 0.f);
                ix[c] = make_uint2(0u, 0u);
            }
        }
    }
    const int ng = (G + 31) / 32, gr = g >> 5;           // groups of 32 workgroups; this one's
    const size_t wstride = res_words(G), pstride = (size_t)G * rwcap;
    unsigned ep = 0;      // sums published next (copy ep % 3)
    unsigned xc = 0;      // p published next (copy xc % 3)
    auto publish = [&](int s, float2 p) {
        put(d.pex + (xc % 3) * pstride + (size_t)g * rwcap + s, bits(p));
        put(d.pex + ((xc + 1) % 3) * pstride + (size_t)g * rwcap + s, kResEmpty);
    };
    __syncthreads();
    for (int c = d.c0; c < d.C; c += d.cstep) {
        if (!d.st[c].outer) continue;
        const int t = fresh_thread(), lane = t & 63;
        const double scale = d.st[c].scale, wmu_d = d.wmu[c];
        const float wmu = (float)wmu_d;
        const double inv_s = scale > 0.0 ? 1.0 / scale : 0.0;
        if (t < (int)(sizeof(ColState) / 8))
            reinterpret_cast<double*>(&S)[t] = reinterpret_cast<const double*>(d.st + c)[t];
        double rz0 = 0.0, rz1 = 0.0, rr = 0.0;
        // r = r64 / |r64|, x = 0, p = z = D^-1 r
#pragma unroll
        for (int k = 0; k < kResK; ++k) {
            const int s = sb[k] + lane;
            if (s < R) {
                const int row = d.rows[(size_t)g * rwcap + s];
                const double2 v = d.R64[(size_t)row * d.C + c];
                const double dr = d.Kd[row], di = -wmu_d * d.Md[row];
                const double inv = 1.0 / (dr * dr + di * di);
                const double2 dv = make_double2(dr * inv, -di * inv);
                const float2 r = f2((float)(v.x * inv_s), (float)(v.y * inv_s));
                const float2 z = f2((float)(r.x * dv.x - r.y * dv.y), (float)(r.x * dv.y + r.y * dv.x));
                dl[s] = dv;
                rl[s] = r;
                xl[s] = f2(0.f, 0.f);
                pl[s] = z;
                if (G > 1) publish(s, z);
                rz0 += (double)r.x * z.x - (double)r.y * z.y;
                rz1 += (double)r.x * z.y + (double)r.y * z.x;
                rr += (double)r.x * r.x + (double)r.y * r.y;
            }
        }
        bool first = true;
        while (true) {
            const int t = fresh_thread(), lane = t & 63;
            // the next step's sums are cleared, then the halo of p comes in
            if (G > 1) {
                u64* const wn = d.words + (size_t)((ep + 1) % 3) * wstride;
                if (t < kResV) put((ng > 1 ? wn + (size_t)(ng + gr) * kResArea : wn) + t * 32 + (g & 31), kResEmpty);
                if (ng > 1 && (g & 31) == 0 && t < kResV * 32 && (t & 31) < ng)
                    put(wn + (size_t)(t & 31) * kResArea + (t >> 5) * 8 + gr, kResEmpty);
            }
            if (nh > 0) {
                const u64* const px = d.pex + (xc % 3) * pstride;
                bool bad = false;
                for (int h0 = t; h0 < nh; h0 += 4 * kResT) {
                    const u64* ad[4];
                    u64 v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) ad[u] = h0 + u * kResT < nh ? px + hl[h0 + u * kResT] : nullptr;
                    if (!wait_words<4>(ad, polls, abort, v)) bad = true;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (ad[u]) pl[rwcap + h0 + u * kResT] = unbits(v[u]);
                }
                if (bad) fail2 = 1;
            }
            ++xc;
            __syncthreads();
            if (fail2) break;
            // ---- q = A p over the register-held entries; a row slot's sum is
            //      stored when its last chunk is done
            {
                float2 ak = f2(0.f, 0.f), am = f2(0.f, 0.f);
                int slot = 0, stop = end[0], so = sb[0];
                float2 xv[2][4];
                const char* const pb = reinterpret_cast<const char*>(lds_d);
                auto fetch = [&](uint2 i, float2* x) {
                    x[0] = *reinterpret_cast<const float2*>(pb + (i.x & 0xffffu));
                    x[1] = *reinterpret_cast<const float2*>(pb + (i.x >> 16));
                    x[2] = *reinterpret_cast<const float2*>(pb + (i.y & 0xffffu));
                    x[3] = *reinterpret_cast<const float2*>(pb + (i.y >> 16));
                };
                // keep the packed indices packed: unpacked once ahead of the
                // iterations they would take 72 more registers
#pragma unroll
                for (int ch = 0; ch < kResCh; ++ch) asm volatile("" : "+v"(ix[ch].x), "+v"(ix[ch].y));
                fetch(ix[0], xv[0]);
                fetch(ix[1], xv[1]);
#pragma unroll
                for (int ch = 0; ch < kResCh; ++ch) {
                    if (ch < nch) {
                        const float4 a = kv[ch], b = mv[ch];
                        float2* const x = xv[ch & 1];
                        ak.x += a.x * x[0].x; ak.y += a.x * x[0].y; am.x += b.x * x[0].x; am.y += b.x * x[0].y;
                        ak.x += a.y * x[1].x; ak.y += a.y * x[1].y; am.x += b.y * x[1].x; am.y += b.y * x[1].y;
                        ak.x += a.z * x[2].x; ak.y += a.z * x[2].y; am.x += b.z * x[2].x; am.y += b.z * x[2].y;
                        ak.x += a.w * x[3].x; ak.y += a.w * x[3].y; am.x += b.w * x[3].x; am.y += b.w * x[3].y;
                        if (ch + 2 < kResCh) fetch(ix[ch + 2 < kResCh ? ch + 2 : 0], x);
                        if (ch + 1 == stop) {
                            if (so + lane < rwcap) yl[so + lane] = f2(ak.x + wmu * am.y, ak.y - wmu * am.x);
                            ak = f2(0.f, 0.f);
                            am = f2(0.f, 0.f);
                            ++slot;
                            stop = slot == 1 ? end[1] : slot == 2 ? end[2] : end[3];
                            so = slot == 1 ? sb[1] : slot == 2 ? sb[2] : sb[3];
                        }
                    }
                }
            }
            // ---- the nine sums
            double v[kResV] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, rz0, rz1, rr};
#pragma unroll
            for (int k = 0; k < kResK; ++k) {
                const int s = sb[k] + lane;
                if (s < R) {
                    const float2 y = yl[s], p = pl[s], r = rl[s];
                    const double2 dv = dl[s];
                    const float2 zr = f2((float)(r.x * dv.x - r.y * dv.y), (float)(r.x * dv.y + r.y * dv.x));
                    const float2 zq = f2((float)(y.x * dv.x - y.y * dv.y), (float)(y.x * dv.y + y.y * dv.x));
                    v[0] += (double)p.x * y.x - (double)p.y * y.y;
                    v[1] += (double)p.x * y.y + (double)p.y * y.x;
                    v[2] += (double)y.x * zr.x - (double)y.y * zr.y;
                    v[3] += (double)y.x * zr.y + (double)y.y * zr.x;
                    v[4] += (double)y.x * zq.x - (double)y.y * zq.y;
                    v[5] += (double)y.x * zq.y + (double)y.y * zq.x;
                }
            }
            // over the wave: at each of the first three steps a lane keeps
            // half of the eight values, so value j ends in lanes 8j .. 8j + 7
            // after ten additions instead of 48; the ninth by itself
            {
                const double a0 = swap32_add(v[0], v[4]), a1 = swap32_add(v[1], v[5]), a2 = swap32_add(v[2], v[6]),
                             a3 = swap32_add(v[3], v[7]);
                const double b0 = swap16_add(a0, a2), b1 = swap16_add(a1, a3);
                const double e = sum8(swap8_add(b0, b1, (lane & 8) != 0));
                const double f = sum32(v[8]);
                const double h = swap32_add(f, f);
                if ((lane & 7) == 0) wsum[wave][lane >> 3] = e;
                if (lane == 0) wsum[wave][8] = h;
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the cleared words are out before the sums are
            __syncthreads();
            // this step's copy of the domain's words: the groups' sums, one
            // copy for each reading group, then the workgroups' by group
            u64* const w2 = d.words + (size_t)(ep % 3) * wstride;
            u64* const w1 = ng > 1 ? w2 + (size_t)(ng + gr) * kResArea : w2;
            if (t < kResV) {
                double a = wsum[0][t];
#pragma unroll
                for (int w = 1; w < kResW; ++w) a += wsum[w][t];
                if (G == 1) tot[t] = a;
                else put(w1 + t * 32 + (g & 31), (u64)__double_as_longlong(a));
            }
            // a value to every 32 lanes, a workgroup of the group to each
            if (G > 1 && t < kResV * 32 && (ng == 1 || (g & 31) == 0)) {
                const int q = t & 31;
                const u64* ad[1] = {32 * gr + q < G ? w1 + t : nullptr};
                u64 x[1];
                if (!wait_words<1>(ad, polls, abort, x)) fail1 = 1;
                const double a = sum32(__longlong_as_double((long long)x[0]));
                if (ng == 1) {
                    if (q == 0) tot[t >> 5] = a;
                } else if (q < ng) {   // the group's sum, to every group
                    put(w2 + (size_t)q * kResArea + (t >> 5) * 8 + gr, (u64)__double_as_longlong(a));
                }
            }
            if (ng > 1 && t < kResV * 8) {
                const u64* ad[1] = {(t & 7) < ng ? w2 + (size_t)gr * kResArea + t : nullptr};
                u64 x[1];
                if (!wait_words<1>(ad, polls, abort, x)) fail1 = 1;
                const double a = sum8(__longlong_as_double((long long)x[0]));
                if ((t & 7) == 0) tot[t >> 3] = a;
            }
            ++ep;
            __syncthreads();
            if (fail1) break;
            if (t == 0) {
                const double2 sums[5] = {make_double2(tot[0], tot[1]), make_double2(tot[2], tot[3]),
                                         make_double2(tot[4], tot[5]), make_double2(tot[6], tot[7]),
                                         make_double2(tot[8], 0.0)};
                // on the state in LDS: a copy in registers would push the operator out of them
                if (first) {
                    S.rho = sums[3];
                    S.rn2 = S.rn2_best = S.tau2 = S.tmark = sums[4].x;
                    S.rn2_0 = 1.0;
                    S.k_best = S.k_mark = S.restarts = S.kin = 0;
                    S.k_prev = S.iters - S.it_start;
                    S.it_start = S.iters;
                    S.beta = make_double2(0.0, 0.0);
                    S.active = S.outer && cfinite(sums[3]) && !czero(sums[3]);
                    S.breakdown = S.stepped = 0;
                    S.cq = 0.0;
                }
                if (S.kin >= max_inner) S.active = 0;
                fused_scalars(S, sums);
                live = S.active;
                step = make_float4((float)S.alpha.x, (float)S.alpha.y, (float)S.beta.x, (float)S.beta.y);
            }
            first = false;
            __syncthreads();
            if (!live) break;
            // ---- r, x, p
            const float4 ab = step;
            rz0 = rz1 = rr = 0.0;
#pragma unroll
            for (int k = 0; k < kResK; ++k) {
                const int s = sb[k] + lane;
                if (s < R) {
                    const float2 q = yl[s], p = pl[s], x = xl[s];
                    float2 r = rl[s];
                    const double2 dv = dl[s];
                    r.x -= ab.x * q.x - ab.y * q.y;
                    r.y -= ab.x * q.y + ab.y * q.x;
                    const float2 z = f2((float)(r.x * dv.x - r.y * dv.y), (float)(r.x * dv.y + r.y * dv.x));
                    rl[s] = r;
                    xl[s] = f2(x.x + ab.x * p.x - ab.y * p.y, x.y + ab.x * p.y + ab.y * p.x);
                    const float2 pn = f2(z.x + ab.z * p.x - ab.w * p.y, z.y + ab.z * p.y + ab.w * p.x);
                    pl[s] = pn;
                    if (G > 1) publish(s, pn);
                    rz0 += (double)r.x * z.x - (double)r.y * z.y;
                    rz1 += (double)r.x * z.y + (double)r.y * z.x;
                    rr += (double)r.x * r.x + (double)r.y * r.y;
                }
            }
        }
        if (fail1 || fail2) {   // a wait ran out: every workgroup leaves
            if (threadIdx.x == 0) __hip_atomic_store(abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        const int te = fresh_thread();
#pragma unroll
        for (int k = 0; k < kResK; ++k) {
            const int s = sb[k] + (te & 63);
            if (s < R) d.Xi[(size_t)d.rows[(size_t)g * rwcap + s] * d.C + c] = xl[s];
        }
        if (g == 0 && te < (int)(sizeof(ColState) / 8))
            reinterpret_cast<double*>(d.st + c)[te] = reinterpret_cast<const double*>(&S)[te];
        __syncthreads();
    }
}

// ------------------------------------------------ the plain GMRES, resident
// Right-Jacobi GMRES(m) in double precision (krylov.hip describes the method
// and holds the kernel-per-phase form) with all its cycles in one launch, over
// the same layout and exchange. A step of that form is seven launches, three
// of them normally empty: 26 us on 3k unknowns, of which little is work.
// The basis and the operator (A D^-1, complex128 in the layout's order) stay
// in memory: a workgroup reads only its own rows of them, so they come
// through its caches; v_j with its halo, w and the iterate are in LDS.
//   step j: w = Ahat v_j; c_k = v_k^H w, |w|^2 (one exchange of 2 j + 3
//   doubles); v_{j+1} = (w - sum c_k v_k) / beta with beta by Pythagoras,
//   after a second pass where that is unreliable (kGmEta, kGmDrop); one thread
//   of every workgroup runs the Givens recurrence while v_{j+1} travels.
// A solve to 1e-12 of 3k unknowns took 12.6 ms with the kernels and takes 5.5
// (11.7 us a step); of 434k unknowns 108 and 77 ms, 70 us a step, in which the
// 378 MB of operator and basis of an average step go by at 5.4 TB/s.
constexpr int kGmMax = 31;                    // longest restart: 2 m + 1 sums in 64
constexpr int kGmVals = 64;
constexpr int kGmArea = kGmVals * 32 + 32;    // words from one area to the next

struct GmArgs {
    int G, n, rw, rwcap, hcap, hmax, m, max_iter, polls;
    double rtol;
    const int32_t *rows, *wend, *halo, *nh;
    const uint2* idx;
    const double2 *A, *b;
    double2 *u, *V;
    u64 *words, *pex;
    int* abort;
    GmOut* out;
};

// Ahat = A D^-1 in the layout's order, one wave per (workgroup, wave).
__global__ void __launch_bounds__(256)
k_gm_vals(int n, int rw, int rwcap, double wmu, const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
          const int32_t* __restrict__ rows, const int32_t* __restrict__ wend, const double* __restrict__ K,
          const double* __restrict__ Ms, const double2* __restrict__ dinv, double2* __restrict__ A) {
    const int g = blockIdx.x / 2, wave = (blockIdx.x & 1) * 4 + ((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int R = min(n - g * rw, rw);
    const size_t base = ((size_t)g * kResW + wave) * kResCh * 256 + lane;
    int ch = 0;
    for (int k = 0; k < kResK; ++k) {
        const int end = wend[((size_t)g * kResW + wave) * kResK + k];
        const int s = res_slice(wave, k) * 64 + lane;
        const int row = s < R ? rows[(size_t)g * rwcap + s] : -1;
        const int b = row >= 0 ? rp[row] : 0, l = row >= 0 ? rp[row + 1] - b : 0;
        for (int q = 0; ch < end; ++ch, q += 4)
#pragma unroll
            for (int u = 0; u < 4; ++u)
                A[base + (size_t)ch * 256 + u * 64] =
                    q + u < l ? cmul(make_double2(K[b + q + u], -wmu * Ms[b + q + u]), dinv[col[b + q + u]])
                              : make_double2(0.0, 0.0);
    }
}

__host__ __device__ constexpr size_t gm_words(int G) {
    return (size_t)kGmArea * (G > 32 ? 2 * ((G + 31) / 32) : 1);
}

// RK rows to a thread (at most kResT RK rows to a workgroup); the passes over
// the basis take kQ vectors at a time, 16 loads of a thread in flight.
template <int RK>
__global__ void __launch_bounds__(kResT)
k_gm_solve(GmArgs a) {
    constexpr int kQ = 16 / RK;
    extern __shared__ double2 lds_d[];
    __shared__ double wsum[kResW][kGmVals];
    __shared__ double tot[kGmVals];
    __shared__ double2 coef[kGmMax + 1], hsave[kGmMax + 1], col[kGmMax + 2], cs[kGmMax], gv[kGmMax + 1],
        yv[kGmMax + 1];
    __shared__ double sn[kGmMax];
    __shared__ double scale_s, beta_s, tol_s, rnorm_s;
    __shared__ int action, done, nonfinite, mdone, fail1, fail2;
    const int g = xcd_block(blockIdx.x, gridDim.x);
    const int G = a.G, m = a.m, rwcap = a.rwcap, R = min(a.n - g * a.rw, a.rw);
    const int ng = (G + 31) / 32, gr = g >> 5, lanes1 = G <= 8 ? 8 : 32;
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    double2* const z = lds_d;                           // own rows, then the halo
    double2* const yl = z + rwcap + a.hcap;
    double2* const ul = yl + rwcap;
    double2* const H = ul + rwcap;                      // [m][m + 1]
    int* const hl = reinterpret_cast<int*>(H + (size_t)m * (m + 1));
    const int nh = a.nh[g];
    for (int h = t; h < nh; h += kResT) hl[h] = a.halo[(size_t)g * a.hmax + h];
    if (t == 0) { fail1 = 0; fail2 = 0; nonfinite = 0; }
    int end[RK], sb[RK];
#pragma unroll
    for (int k = 0; k < RK; ++k) {   // (a workgroup of at most kResT RK rows has no more row slots)
        end[k] = __builtin_amdgcn_readfirstlane(a.wend[((size_t)g * kResW + wave) * kResK + k]);
        sb[k] = res_slice(wave, k) * 64;
    }
    const size_t ldv = (size_t)G * rwcap, mine = (size_t)g * rwcap;
    const size_t wstride = gm_words(G), pstride = 2 * ldv;
    unsigned ep = 0, xc = 0;
    bool failed = false;

    // own rows of z to the neighbours
    auto publish = [&]() {
#pragma unroll
        for (int k = 0; k < RK; ++k) {
            const int s = sb[k] + lane;
            if (s < R && G > 1) {
                u64* const p = a.pex + (xc % 3) * pstride + 2 * (mine + s);
                u64* const q = a.pex + ((xc + 1) % 3) * pstride + 2 * (mine + s);
                put(p, (u64)__double_as_longlong(z[s].x));
                put(p + 1, (u64)__double_as_longlong(z[s].y));
                put(q, kResEmpty);
                put(q + 1, kResEmpty);
            }
        }
        ++xc;
    };
    // yl = Ahat z; four chunks of the operator on their way ahead of their use,
    // the first of them while the halo is awaited
    const int nch = end[RK - 1];
    // (until_done: nothing more once the Givens recurrence has said so)
    auto multiply = [&](bool until_done) {
        const size_t base = ((size_t)g * kResW + wave) * kResCh;
        uint2 ib[4];
        double2 ab[4][4];
        auto fetch = [&](int c, int u) {
            if (c >= nch) return;
            ib[u] = a.idx[(base + c) * 64 + lane];
#pragma unroll
            for (int q = 0; q < 4; ++q) ab[u][q] = a.A[(base + c) * 256 + q * 64 + lane];
        };
#pragma unroll
        for (int u = 0; u < 4; ++u) fetch(u, u);
        if (nh > 0) {
            const u64* const px = a.pex + ((xc - 1) % 3) * pstride;
            bool bad = false;
            for (int h0 = t; h0 < nh; h0 += 2 * kResT) {
                const int h1 = h0 + kResT;
                const u64* const p0 = px + 2 * (size_t)hl[h0];
                const u64* const p1 = h1 < nh ? px + 2 * (size_t)hl[h1] : nullptr;
                const u64* ad[4] = {p0, p0 + 1, p1, p1 ? p1 + 1 : nullptr};
                u64 v[4];
                if (!wait_words<4>(ad, a.polls, a.abort, v)) bad = true;
                z[rwcap + h0] = make_double2(__longlong_as_double((long long)v[0]), __longlong_as_double((long long)v[1]));
                if (p1)
                    z[rwcap + h1] = make_double2(__longlong_as_double((long long)v[2]), __longlong_as_double((long long)v[3]));
            }
            if (bad) fail2 = 1;
        }
        __syncthreads();
        failed = failed || fail2;
        if (failed || (until_done && done)) return;
        const char* const zb = reinterpret_cast<const char*>(lds_d);
        double2 y = make_double2(0.0, 0.0);
        int slot = 0, stop = end[0], so = sb[0];
        for (int c0 = 0; c0 < nch; c0 += 4) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (c0 + u >= nch) continue;
                const uint2 i = ib[u];
                const unsigned o[4] = {i.x & 0xffffu, i.x >> 16, i.y & 0xffffu, i.y >> 16};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double2 x = *reinterpret_cast<const double2*>(zb + 2 * o[q]);
                    y.x += ab[u][q].x * x.x - ab[u][q].y * x.y;
                    y.y += ab[u][q].x * x.y + ab[u][q].y * x.x;
                }
                fetch(c0 + 4 + u, u);
                if (c0 + u + 1 == stop) {
                    yl[so + lane] = y;
                    y = make_double2(0.0, 0.0);
                    ++slot;
#pragma unroll
                    for (int k = 1; k < RK; ++k)
                        if (slot == k) {
                            stop = end[k];
                            so = sb[k];
                        }
                }
            }
        }
    };
    // tot[0 .. nv - 1]: the waves' sums over all workgroups
    auto exchange = [&](int nv) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // cleared words are out before new ones are
        __syncthreads();
        u64* const w2 = a.words + (size_t)(ep % 3) * wstride;
        u64* const w1 = ng > 1 ? w2 + (size_t)(ng + gr) * kGmArea : w2;
        if (t < nv) {
            double v = wsum[0][t];
#pragma unroll
            for (int w = 1; w < kResW; ++w) v += wsum[w][t];
            if (G == 1) tot[t] = v;
            else put(w1 + t * lanes1 + (g & 31), (u64)__double_as_longlong(v));
        }
        if (lanes1 == 8) {   // up to eight workgroups: eight lanes to a value, all values at once
            const u64* ad[1] = {t < nv * 8 && (t & 7) < G ? w1 + t : nullptr};
            u64 x[1];
            if (G > 1 && !wait_words<1>(ad, a.polls, a.abort, x)) fail1 = 1;
            const double v = sum8(__longlong_as_double((long long)x[0]));
            if (G > 1 && t < nv * 8 && (t & 7) == 0) tot[t >> 3] = v;
        } else if (ng == 1 || (g & 31) == 0) {
            const int q = t & 31;
            const u64* ad[4];
            u64 x[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) ad[r] = 32 * gr + q < G && t + r * kResT < nv * 32 ? w1 + t + r * kResT : nullptr;
            if (!wait_words<4>(ad, a.polls, a.abort, x)) fail1 = 1;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double v = sum32(__longlong_as_double((long long)x[r]));
                const int j = (t + r * kResT) >> 5;
                if (j >= nv) continue;
                if (ng == 1) {
                    if (q == 0) tot[j] = v;
                } else if (q < ng) {
                    put(w2 + (size_t)q * kGmArea + j * 8 + gr, (u64)__double_as_longlong(v));
                }
            }
        }
        if (ng > 1) {
            const u64* ad[1] = {t < nv * 8 && (t & 7) < ng ? w2 + (size_t)gr * kGmArea + t : nullptr};
            u64 x[1];
            if (!wait_words<1>(ad, a.polls, a.abort, x)) fail1 = 1;
            const double v = sum8(__longlong_as_double((long long)x[0]));
            if (t < nv * 8 && (t & 7) == 0) tot[t >> 3] = v;
        }
        if (G > 1) {   // the copy of the step before is read by all: clear it for the step after next
            u64* const c2 = a.words + (size_t)((ep + 2) % 3) * wstride;
            if (t < kGmVals) put((ng > 1 ? c2 + (size_t)(ng + gr) * kGmArea : c2) + t * lanes1 + (g & 31), kResEmpty);
            if (ng > 1 && (g & 31) == 0 && (t & 7) < ng)
                put(c2 + (size_t)(t & 7) * kGmArea + (t >> 3) * 8 + gr, kResEmpty);
        }
        ++ep;
        __syncthreads();
        failed = failed || fail1;
    };
    auto wave_total = [&](double v) {
        v = sum32(v);
        return swap32_add(v, v);
    };

    // u = 0 or the given iterate; r = b - Ahat u, rnorm
    auto residual = [&]() {
#pragma unroll
        for (int k = 0; k < RK; ++k) {
            const int s = sb[k] + lane;
            if (s < R) z[s] = ul[s];
        }
        publish();
        multiply(false);
        if (failed) return;
        double nn = 0.0;
#pragma unroll
        for (int k = 0; k < RK; ++k) {
            const int s = sb[k] + lane;
            if (s < R) {
                const double2 r = csub(a.b[a.rows[mine + s]], yl[s]);
                yl[s] = r;
                nn += cabs2(r);
            }
        }
        nn = wave_total(nn);
        if (lane == 0) wsum[wave][0] = nn;
        exchange(1);
    };
#pragma unroll
    for (int k = 0; k < RK; ++k) {
        const int s = sb[k] + lane;
        if (s < R) ul[s] = make_double2(0.0, 0.0);
    }
    residual();
    if (t == 0) {
        tol_s = a.rtol * sqrt(tot[0]);
        if (g == 0) a.out->bnorm = sqrt(tot[0]);
    }
    int iters = 0, cycles = 0, status = PETGEM_OK;
    while (!failed) {
        const double r2 = tot[0], rn = sqrt(r2);
        if (t == 0) {
            rnorm_s = rn;
            nonfinite = nonfinite || !isfinite(r2);
            done = 0;
            mdone = 0;
            gv[0] = make_double2(rn, 0.0);
        }
        __syncthreads();
        if (nonfinite) { status = PETGEM_NONFINITE; break; }
        if (rn <= tol_s || rn == 0.0) break;
        if (iters >= a.max_iter) { status = PETGEM_NOT_CONVERGED; break; }
        // v_0 = r / |r|
#pragma unroll
        for (int k = 0; k < RK; ++k) {
            const int s = sb[k] + lane;
            if (s < R) {
                const double2 v = cscale(yl[s], 1.0 / rn);
                z[s] = v;
                a.V[mine + s] = v;
            }
        }
        publish();
        for (int j = 0; j < m; ++j) {
            multiply(true);
            if (failed || done) break;
            for (int pass = 0; pass < 2; ++pass) {
                double2 w[RK];
                double nn = 0.0;
#pragma unroll
                for (int k = 0; k < RK; ++k) {
                    const int s = sb[k] + lane;
                    w[k] = s < R ? yl[s] : make_double2(0.0, 0.0);
                    nn += cabs2(w[k]);
                }
                nn = wave_total(nn);
                if (lane == 0) wsum[wave][2 * (j + 1)] = nn;
                for (int k0 = 0; k0 <= j; k0 += kQ) {
                    double2 acc[kQ], v[kQ][RK];
#pragma unroll
                    for (int q = 0; q < kQ; ++q)
#pragma unroll
                        for (int k = 0; k < RK; ++k) {
                            const int s = sb[k] + lane;
                            v[q][k] = s < R && k0 + q <= j ? a.V[(size_t)(k0 + q) * ldv + mine + s]
                                                           : make_double2(0.0, 0.0);
                        }
#pragma unroll
                    for (int q = 0; q < kQ; ++q) {
                        acc[q] = make_double2(0.0, 0.0);
#pragma unroll
                        for (int k = 0; k < RK; ++k) acc[q] = cadd(acc[q], cmulc(v[q][k], w[k]));
                    }
#pragma unroll
                    for (int q = 0; q < kQ; q += 4) {
                        if (k0 + q > j) continue;
                        const double b0 = swap16_add(swap32_add(acc[q].x, acc[q + 2].x),
                                                     swap32_add(acc[q + 1].x, acc[q + 3].x));
                        const double b1 = swap16_add(swap32_add(acc[q].y, acc[q + 2].y),
                                                     swap32_add(acc[q + 1].y, acc[q + 3].y));
                        const double e = sum8(swap8_add(b0, b1, (lane & 8) != 0));
                        const int i = 2 * (k0 + q) + (lane >> 3);
                        if ((lane & 7) == 0 && i < 2 * (j + 1)) wsum[wave][i] = e;
                    }
                }
                exchange(2 * (j + 1) + 1);
                if (failed) break;
                if (wave == 0) {
                    const bool has = lane <= j;
                    const double2 c = has ? make_double2(tot[2 * lane], tot[2 * lane + 1]) : make_double2(0.0, 0.0);
                    if (has) coef[lane] = c;
                    const double hh = sum32(cabs2(c)), nrm2 = tot[2 * (j + 1)];   // j < 32: the lower half-wave
                    if (has) {
                        col[lane] = pass == 0 ? c : cadd(hsave[lane], c);
                        if (pass == 0) hsave[lane] = c;
                    }
                    if (lane == 0) {
                        const double b2 = nrm2 - hh;
                        if (!isfinite(nrm2) || !isfinite(hh)) {
                            nonfinite = 1;
                            action = 0;
                        } else if (pass == 0 && (b2 <= kGmEta * nrm2 ||
                                                 cabs2(gv[j]) <= kGmDrop * kGmDrop * rnorm_s * rnorm_s)) {
                            action = 2;
                            scale_s = 1.0;
                        } else {
                            const double be = b2 > 0.0 ? sqrt(b2) : 0.0;
                            action = 1;
                            beta_s = be;
                            scale_s = be > 0.0 ? 1.0 / be : 0.0;
                        }
                    }
                }
                __syncthreads();
                const int act = action;
                if (act == 0) break;
                const double sc = scale_s;
                for (int k0 = 0; k0 <= j; k0 += kQ) {
                    double2 v[kQ][RK];
#pragma unroll
                    for (int q = 0; q < kQ; ++q)
#pragma unroll
                        for (int k = 0; k < RK; ++k) {
                            const int s = sb[k] + lane;
                            v[q][k] = s < R && k0 + q <= j ? a.V[(size_t)(k0 + q) * ldv + mine + s]
                                                           : make_double2(0.0, 0.0);
                        }
#pragma unroll
                    for (int q = 0; q < kQ; ++q) {
                        const double2 h = k0 + q <= j ? coef[k0 + q] : make_double2(0.0, 0.0);
#pragma unroll
                        for (int k = 0; k < RK; ++k) w[k] = csub(w[k], cmul(h, v[q][k]));
                    }
                }
#pragma unroll
                for (int k = 0; k < RK; ++k) {
                    const int s = sb[k] + lane;
                    if (s < R) {
                        const double2 v = cscale(w[k], sc);
                        if (act == 2) {
                            yl[s] = v;
                        } else {
                            z[s] = v;
                            a.V[(size_t)(j + 1) * ldv + mine + s] = v;
                        }
                    }
                }
                if (act == 1) break;
                __syncthreads();   // coef is read before the second pass writes it
            }
            if (failed || nonfinite) break;
            if (j + 1 < m) publish();
            // the previous rotations on the new column, then the new one, by a
            // thread whose wave has the least of the halo to read; the others
            // go on, and see `done` when the halo has come in. s is real, so
            // the chain from one rotation to the next is a multiply-add
            if (t == kResT - kWave) {
                const double be = beta_s;
                double2* const Hj = H + (size_t)j * (m + 1);
                double2 x = col[0];
                for (int i0 = 0; i0 < j; i0 += 8) {
                    double2 c[8], y[8], o[8];
                    double r[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int i = min(i0 + u, j - 1);
                        c[u] = cs[i];
                        r[u] = sn[i];
                        y[u] = col[i + 1];
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const double2 cy = cmul(c[u], y[u]);
                        o[u] = cadd(cmulc(c[u], x), cscale(y[u], r[u]));
                        if (i0 + u < j) x = csub(cy, cscale(x, r[u]));
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (i0 + u < j) Hj[i0 + u] = o[u];
                }
                const double den = sqrt(cabs2(x) + be * be), iden = den > 0.0 ? 1.0 / den : 0.0;
                const double2 c = den > 0.0 ? cscale(x, iden) : make_double2(1.0, 0.0);
                const double s1 = den > 0.0 ? be * iden : 0.0;
                cs[j] = c;
                sn[j] = s1;
                Hj[j] = make_double2(den, 0.0);
                const double2 gj = gv[j], g1 = cscale(gj, -s1);
                gv[j + 1] = g1;
                gv[j] = cmulc(c, gj);
                mdone = j + 1;
                if (sqrt(cabs2(g1)) <= tol_s || be <= 1e-300) done = 1;
            }
        }
        if (failed) break;
        __syncthreads();
        if (done && mdone < m) {
            // v_{mdone} went out and nobody read it: an exchange separates it
            // from the iterate that goes out next
            exchange(1);
            if (failed) break;
        }
        // back substitution on the first half-wave: lane i holds y_i
        const int md = mdone;
        if (wave == 0) {
            double2 s = lane < md ? gv[lane] : make_double2(0.0, 0.0);
            const double2 inv = lane < md ? cdiv(make_double2(1.0, 0.0), H[(size_t)lane * (m + 1) + lane])
                                          : make_double2(0.0, 0.0);
            for (int i = md - 1; i >= 0; --i) {
                const double2 yi = cmul(s, inv);
                const double2 y = make_double2(__shfl(yi.x, i), __shfl(yi.y, i));
                if (lane == i) s = y;
                else if (lane < i) s = csub(s, cmul(H[(size_t)i * (m + 1) + lane], y));
            }
            if (lane < md) yv[lane] = s;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < RK; ++k) {
            const int s = sb[k] + lane;
            if (s < R) {
                double2 u = ul[s];
                for (int q = 0; q < md; ++q) u = cadd(u, cmul(yv[q], a.V[(size_t)q * ldv + mine + s]));
                ul[s] = u;
            }
        }
        iters += md;
        ++cycles;
        residual();
        if (!failed && md == 0 && !nonfinite) {   // no progress; the new residual is the last word on it
            if (t == 0) rnorm_s = sqrt(tot[0]);
            status = sqrt(tot[0]) <= tol_s ? PETGEM_OK : PETGEM_NOT_CONVERGED;
            __syncthreads();
            break;
        }
    }
    if (failed) {
        if (t == 0) __hip_atomic_store(a.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
#pragma unroll
    for (int k = 0; k < RK; ++k) {
        const int s = sb[k] + lane;
        if (s < R) a.u[a.rows[mine + s]] = ul[s];
    }
    if (g == 0 && t == 0) {
        a.out->rnorm = rnorm_s;
        a.out->iters = iters;
        a.out->cycles = cycles;
        a.out->status = status;
    }
}

}  // namespace

// ------------------------------------------------------------ host side
void Resident::release(Spare& spare) {
    dfree(pattern); dfree(K); dfree(A);
    spare.back(held);
    rows = wend = halo = nh = nullptr;
    idx = nullptr;
    M = nullptr;
    a_freq = -1.0;
    G = 0;
    state = 0;
    values = false;
}

int ResWork::room(size_t bytes) {
    if (!host) PG_HIP(hipHostMalloc(reinterpret_cast<void**>(&host), sizeof(GmHost)));
    if ((size_t)held >= bytes) return PETGEM_OK;
    give_back();
    return spare->take(&buf, bytes, held);
}

void ResWork::give_back() {
    dfree(buf);
    if (spare) spare->back(held);
}

void ResWork::release() {
    give_back();
    if (host) (void)hipHostFree(host);
    host = nullptr;
}

void release_spare(petgem_system* sys) {
    for (Resident& L : sys->res) L.release(sys->spare);
    for (ResWork* w : {&sys->gres, block_res(sys->bw)})
        if (w) {
            w->give_back();
            w->skip = 0;
        }
    if (sys->rst_held > 0) {
        dfree(sys->Rst);
        sys->spare.back(sys->rst_held);
        sys->rst_copies = 0;
    }
    sys->rst_one = false;
}

namespace {

size_t res_lds(const Resident& L) { return (size_t)48 * L.rwcap + (size_t)12 * L.hcap; }

// Rows of a workgroup: about `target`, in whole 64-row slices, on at most ncu
// workgroups; 0 when the mesh is too large.
int res_rows(int n, int target, int ncu) {
    const int G = std::min(std::min(ncu, kResMaxG), ceil_div(n, target));
    const int rw = ceil_div(ceil_div(n, G), 64) * 64;
    return rw <= kResRows ? rw : 0;
}

// Parts of one device allocation, each at a multiple of 256 bytes; with a null
// base it only adds up the size.
struct Carve {
    char* base = nullptr;
    size_t size = 0;
    template <class T>
    T* part(size_t count) {
        T* p = base ? reinterpret_cast<T*>(base + size) : nullptr;
        size += (count * sizeof(T) + 255) / 256 * 256;
        return p;
    }
};

// A layout and the split it is wanted for.
struct ResWant {
    petgem_system* sys;
    Resident* L;
    int rw;                       // rows per workgroup
};

// Builds the layouts that are not there yet (once per mesh and split; the
// pattern does not change). state: 1 usable, -1 the mesh does not fit. All of
// them together take two launches, a temporary allocation and a readback, and each
// an allocation: with two launches, ten allocations, two copies and a wait for each
// the first solve of a batch of 200 small meshes took 76 ms, with these 37
// (kernel by kernel 49; 11 once the layouts are there).
int res_build(const std::vector<ResWant>& want, hipStream_t s) {
    std::vector<ResWant> todo;
    for (const ResWant& w : want) {
        if (w.L->state != 0 && w.L->rw == w.rw) continue;   // (a mesh named twice: 2, set below)
        w.L->release(w.sys->spare);
        w.L->rw = w.rw;
        w.L->state = w.rw == 0 ? -1 : 2;
        if (w.rw != 0) todo.push_back(w);
    }
    if (todo.empty()) return PETGEM_OK;
    const size_t nt = todo.size();
    char* tmp = nullptr;
    std::vector<int> got(2 * nt, 0);
    auto hmax_of = [](int rw) { return std::min((kResLds - 48 * rw) / 12, 65536 / 8 - rw) / 64 * 64; };
    auto go = [&]() -> int {
        std::vector<ResLay> lays(nt);
        std::vector<int> blk;
        size_t rows = 0;
        int most = 0;
        for (size_t k = 0; k < nt; ++k) {
            petgem_system* sys = todo[k].sys;
            Resident& L = *todo[k].L;
            const int n = sys->n_dof, rw = L.rw, hmax = hmax_of(rw);
            L.rwcap = rw;
            L.G = ceil_div(n, rw);
            auto parts = [&](Carve& p) {
                L.rows = p.part<int32_t>((size_t)L.G * rw);
                L.wend = p.part<int32_t>((size_t)L.G * kResW * kResK);
                L.halo = p.part<int32_t>((size_t)L.G * hmax);
                L.nh = p.part<int32_t>((size_t)L.G);
                L.idx = p.part<uint64_t>((size_t)L.G * kResW * kResCh * 64);
            };
            Carve need;
            parts(need);
            PG_TRY(sys->spare.take(&L.pattern, need.size, L.held));
            Carve have{L.pattern};
            parts(have);
            lays[k] = ResLay{(int)blk.size(), n, rw, rw, hmax, sys->row_ptr, sys->col, L.rows, L.wend, L.halo, L.nh,
                             nullptr, reinterpret_cast<uint2*>(L.idx), nullptr};
            blk.insert(blk.end(), (size_t)L.G, (int)k);
            rows += (size_t)n;
            most = std::max(most, n);
        }
        int *pos = nullptr, *stat = nullptr, *blk_d = nullptr;
        ResLay* lays_d = nullptr;
        auto parts = [&](Carve& p) {
            pos = p.part<int>(rows);
            stat = p.part<int>(2 * nt);
            blk_d = p.part<int>(blk.size());
            lays_d = p.part<ResLay>(nt);
        };
        Carve need;
        parts(need);
        PG_TRY(dalloc(&tmp, need.size));
        Carve have{tmp};
        parts(have);
        for (size_t k = 0, r = 0; k < nt; r += (size_t)lays[k].n, ++k) {
            lays[k].pos = pos + r;
            lays[k].stat = stat + 2 * k;
        }
        PG_HIP(hipMemcpyAsync(stat, got.data(), sizeof(int) * got.size(), hipMemcpyHostToDevice, s));
        PG_HIP(hipMemcpyAsync(blk_d, blk.data(), sizeof(int) * blk.size(), hipMemcpyHostToDevice, s));
        PG_HIP(hipMemcpyAsync(lays_d, lays.data(), sizeof(ResLay) * nt, hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(k_res_sort, dim3(blk.size()), dim3(1024), 0, s, lays_d, blk_d);
        const size_t lds = (size_t)2 * ceil_div(most, 32) * sizeof(unsigned);
        PG_HIP(allow_lds(k_res_halo, kResHaloLds));
        hipLaunchKernelGGL(k_res_halo, dim3(blk.size()), dim3(1024), lds, s, lays_d, blk_d);
        PG_HIP(hipGetLastError());
        PG_HIP(hipMemcpyAsync(got.data(), stat, sizeof(int) * got.size(), hipMemcpyDeviceToHost, s));
        PG_HIP(hipStreamSynchronize(s));
        return PETGEM_OK;
    };
    const int rc = go();
    dfree(tmp);
    for (size_t k = 0; k < nt; ++k) {
        Resident& L = *todo[k].L;
        const int rw = L.rw, hmax = hmax_of(rw);
        if (rc == PETGEM_OK && got[2 * k] <= kResCh && got[2 * k + 1] <= hmax) {
            L.hmax = hmax;
            L.hcap = (got[2 * k + 1] + 63) / 64 * 64;
            L.state = 1;
        } else {   // too many entries or outer neighbours; or an error, and it may be tried again
            L.release(todo[k].sys->spare);
            L.rw = rw;
            L.state = rc == PETGEM_OK ? -1 : 0;
        }
    }
    return rc;
}

}  // namespace

// Rows of a workgroup in the finer and the coarser split of a mesh. A step of
// one solve took 5.7 to 5.8 us with 256 to 512 rows and 6.4 with 768 to 1,024
// on 3k to 6k unknowns, 7.6, 7.5, 7.8, 8.2, 7.9 us with 256, 384, 512, 768 and
// 1,024 on 61k; the coarser split lets more domains be resident at once.
constexpr int kResFine = 512, kResCoarse = 1536;

// Out of memory in a plan: what it took is given back, and the workspace's next
// solves run kernel by kernel without building layouts in vain before each.
static int without_room(ResWork& W, petgem_system* sys) {
    for (Resident& L : sys->res) L.release(sys->spare);
    W.give_back();
    W.skip = kResSkip;
    return PETGEM_OK;
}
// whether the form is tried at all, with the polls its waits may take
static bool res_try(ResWork& W, const petgem_system* sys) {
    W.polls = sys->wait_polls > 0 ? sys->wait_polls : kResSpin;
    if (W.skip == 0) return true;
    --W.skip;
    return false;
}

static int res_plan_(ResWork& W, const std::vector<ResItem>& items, const ResVectors& v, hipStream_t s, bool* fits) {
    int dev = 0, ncu = 0, coop = 0;
    PG_HIP(hipGetDevice(&dev));
    PG_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    PG_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    if (!coop) return PETGEM_OK;
    int64_t fine = 0;
    for (const ResItem& it : items) {
        if (!res_rows(it.sys->n_dof, kResCoarse, ncu)) return PETGEM_OK;
        fine += (int64_t)it.C * ceil_div(it.sys->n_dof, kResFine);
    }
    const int which = fine <= ncu ? 0 : 1;
    std::vector<Resident*> L(items.size());
    std::vector<ResWant> want(items.size());
    for (size_t k = 0; k < items.size(); ++k) {
        petgem_system* sys = items[k].sys;
        L[k] = &sys->res[which];
        want[k] = ResWant{sys, L[k], res_rows(sys->n_dof, which ? kResCoarse : kResFine, ncu)};
    }
    PG_TRY(res_build(want, s));
    for (const Resident* l : L)
        if (l->state != 1) return PETGEM_OK;
    bool stale = false;
    for (const ResWant& w : want) {
        Resident* l = w.L;
        const size_t ent = (size_t)l->G * kResW * kResCh * 64;
        if (!l->K) PG_TRY(w.sys->spare.take(&l->K, 8 * ent, l->held));
        l->M = l->K + 4 * ent;
        stale = stale || !l->values;
    }
    // rounds of domains that are resident together, the largest first
    std::vector<size_t> order(items.size());
    for (size_t k = 0; k < order.size(); ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return L[a]->G > L[b]->G; });
    struct Round { int used = 0; std::vector<size_t> who; };
    std::vector<Round> rounds;
    for (size_t k : order) {
        size_t r = 0;
        while (r < rounds.size() && rounds[r].used + L[k]->G > ncu) ++r;
        if (r == rounds.size()) rounds.emplace_back();
        rounds[r].used += L[k]->G;
        rounds[r].who.push_back(k);
    }
    std::vector<ResDom> doms;
    std::vector<int> blk;
    W.rounds.clear();
    size_t nw = 0, np = 0;
    std::vector<std::pair<size_t, size_t>> off;
    for (const Round& r : rounds) {
        ResWork::Round out;
        out.blk0 = (int)blk.size();
        out.lds = 0;
        int b = 0;
        for (size_t k : r.who) {
            const ResItem& it = items[k];
            const Resident& l = *L[k];
            // several columns of one mesh: as many domains as fit beside each other
            const int D = items.size() == 1 ? std::max(1, std::min(it.C, ncu / l.G)) : 1;
            for (int q = 0; q < D; ++q) {
                ResDom d{};
                d.block0 = b;
                d.G = l.G;
                d.n = it.sys->n_dof;
                d.rw = l.rw;
                d.rwcap = l.rwcap;
                d.hcap = l.hcap;
                d.hmax = l.hmax;
                d.C = it.C;
                d.c0 = q;
                d.cstep = D;
                d.rows = l.rows;
                d.wend = l.wend;
                d.halo = l.halo;
                d.nh = l.nh;
                d.rp = it.sys->row_ptr;
                d.idx = reinterpret_cast<const uint2*>(l.idx);
                d.K = d.Kw = reinterpret_cast<float4*>(l.K);
                d.M = d.Mw = reinterpret_cast<float4*>(l.M);
                d.K64 = it.sys->K;
                d.M64 = it.sys->Ms;
                d.Kd = it.sys->Kd;
                d.Md = it.sys->Msd;
                d.wmu = v.wmu + (size_t)it.seg * it.C;
                d.R64 = v.R64 + it.row_off * it.C;
                d.Xi = v.Xi + it.row_off * it.C;
                d.st = static_cast<ColState*>(v.st) + (size_t)it.seg * it.C;
                off.emplace_back(nw, np);
                nw += 3 * res_words(l.G);
                np += (size_t)3 * l.G * l.rwcap;
                for (int g = 0; g < l.G; ++g) blk.push_back((int)doms.size());
                doms.push_back(d);
                b += l.G;
            }
            out.lds = std::max(out.lds, res_lds(l));
        }
        out.nblk = b;
        W.rounds.push_back(out);
    }
    auto parts = [&](Carve& c) {
        W.abort = c.part<int>(1);
        W.doms = c.part<char>(doms.size() * sizeof(ResDom));
        W.blk = c.part<int>(blk.size());
        W.words = c.part<u64>(nw);
        W.pex = c.part<u64>(np);
    };
    Carve need;
    parts(need);
    PG_TRY(W.room(need.size));
    Carve have{W.buf};
    parts(have);
    W.n_words = nw;
    W.n_pex = np;
    for (size_t k = 0; k < doms.size(); ++k) {
        doms[k].words = W.words + off[k].first;
        doms[k].pex = W.pex + off[k].second;
    }
    PG_HIP(hipMemcpyAsync(W.doms, doms.data(), doms.size() * sizeof(ResDom), hipMemcpyHostToDevice, s));
    PG_HIP(hipMemcpyAsync(W.blk, blk.data(), blk.size() * sizeof(int), hipMemcpyHostToDevice, s));
    PG_HIP(hipStreamSynchronize(s));   // the tables are read from host vectors
    if (stale) {
        for (const ResWork::Round& r : W.rounds) {
            // one mesh: its first domain's workgroups cover the whole layout
            const int nb = items.size() == 1 ? L[0]->G : r.nblk;
            hipLaunchKernelGGL(k_res_vals, dim3(2 * nb), dim3(256), 0, s, reinterpret_cast<const ResDom*>(W.doms),
                               W.blk + r.blk0);
        }
        PG_HIP(hipGetLastError());
        for (Resident* l : L) l->values = true;
    }
    *fits = true;
    return PETGEM_OK;
}

int res_plan(ResWork& W, const std::vector<ResItem>& items, const ResVectors& v, hipStream_t s, bool* fits) {
    *fits = false;
    W.spare = &items[0].sys->spare;   // whose workspace it is
    if (!res_try(W, items[0].sys)) return PETGEM_OK;
    const int rc = res_plan_(W, items, v, s, fits);
    if (rc != PETGEM_OUT_OF_MEMORY) return rc;
    for (const ResItem& it : items) (void)without_room(W, it.sys);
    return PETGEM_OK;
}

// The workgroups of a launch have to be resident together; a device that has
// fewer compute units for it than it said refuses.
static int launched(hipError_t e) {
    if (e == hipErrorCooperativeLaunchTooLarge) {
        (void)hipGetLastError();
        return kResAborted;
    }
    PG_HIP(e);
    return PETGEM_OK;
}

// Dynamic LDS of k_gm_solve; its static part and this fill a compute unit's.
constexpr int kGmLds = 160 * 1024 - 9216;
static size_t gm_lds(const Resident& L, int restart) {
    return (size_t)16 * (L.rwcap + L.hcap) + (size_t)32 * L.rwcap + (size_t)16 * restart * (restart + 1) +
           (size_t)4 * L.hcap;
}

// Lays the mesh out and makes room for the plain GMRES of one source in one
// launch; *fits false: the mesh or the restart does not fit (and nothing was
// done that such a solve would have to pay for), or there is no room.
static int gm_plan_(petgem_system* sys, ResWork& W, int restart, hipStream_t s, bool* fits) {
    const int n = sys->n_dof;
    int dev = 0, ncu = 0, coop = 0;
    PG_HIP(hipGetDevice(&dev));
    PG_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    PG_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    const int which = ceil_div(n, kResFine) <= ncu ? 0 : 1, rw = res_rows(n, which ? kResCoarse : kResFine, ncu);
    if (restart > kGmMax || !coop || rw == 0) return PETGEM_OK;
    Resident& L = sys->res[which];
    PG_TRY(res_build({ResWant{sys, &L, rw}}, s));
    if (L.state != 1 || gm_lds(L, restart) > (size_t)kGmLds) return PETGEM_OK;
    if (!L.A) PG_TRY(sys->spare.take(&L.A, (size_t)L.G * kResW * kResCh * 256, L.held));
    const size_t ldv = (size_t)L.G * L.rwcap;
    W.L = &L;
    W.n_words = 3 * gm_words(L.G);
    W.n_pex = 6 * ldv;
    auto parts = [&](Carve& c) {
        W.abort = c.part<int>(1);
        W.out = c.part<GmOut>(1);
        W.words = c.part<u64>(W.n_words);
        W.pex = c.part<u64>(W.n_pex);
        W.V = c.part<double2>((size_t)(restart + 1) * ldv);
        W.b = c.part<double2>((size_t)n);
        W.u = c.part<double2>((size_t)n);
    };
    Carve need;
    parts(need);
    PG_TRY(W.room(need.size));
    Carve have{W.buf};
    parts(have);
    *fits = true;
    return PETGEM_OK;
}

int gm_plan(petgem_system* sys, ResWork& W, int restart, hipStream_t s, bool* fits) {
    *fits = false;
    W.spare = &sys->spare;
    if (!res_try(W, sys)) return PETGEM_OK;
    const int rc = gm_plan_(sys, W, restart, s, fits);
    return rc == PETGEM_OUT_OF_MEMORY ? without_room(W, sys) : rc;
}

// The whole plain GMRES of the source whose right-hand side is in W.b, from a
// zero guess, after gm_plan; D^-1 (sys->dinv) is current.
int gm_run(petgem_system* sys, ResWork& W, double freq, int restart, int max_iter, double rtol, hipStream_t s) {
    Resident& L = *W.L;
    const int n = sys->n_dof;
    if (L.a_freq != freq) {
        hipLaunchKernelGGL(k_gm_vals, dim3(2 * L.G), dim3(256), 0, s, n, L.rw, L.rwcap, 2.0 * kPi * freq * kMu0,
                           sys->row_ptr, sys->col, L.rows, L.wend, sys->K, sys->Ms, sys->dinv, L.A);
        PG_HIP(hipGetLastError());
        L.a_freq = freq;
    }
    const size_t m = std::max(W.n_words, W.n_pex);
    hipLaunchKernelGGL(k_res_clear, dim3(ceil_div(m, 256)), dim3(256), 0, s, W.n_words, W.words, W.n_pex, W.pex,
                       W.abort);
    PG_HIP(hipGetLastError());
    GmArgs a{};
    a.G = L.G;
    a.n = n;
    a.rw = L.rw;
    a.rwcap = L.rwcap;
    a.hcap = L.hcap;
    a.hmax = L.hmax;
    a.m = restart;
    a.max_iter = max_iter;
    a.polls = W.polls;
    a.rtol = rtol;
    a.rows = L.rows;
    a.wend = L.wend;
    a.halo = L.halo;
    a.nh = L.nh;
    a.idx = reinterpret_cast<const uint2*>(L.idx);
    a.A = L.A;
    a.b = W.b;
    a.u = W.u;
    a.V = W.V;
    a.words = W.words;
    a.pex = W.pex;
    a.abort = W.abort;
    a.out = W.out;
    void* args[1] = {&a};
    // the finer split has at most 512 rows to a workgroup, the coarser one more than 1,024
    const void* fn = L.rw <= kResT ? reinterpret_cast<const void*>(k_gm_solve<1>)
                                   : reinterpret_cast<const void*>(k_gm_solve<4>);
    const size_t lds = gm_lds(L, restart);
    PG_HIP(allow_lds(fn, kGmLds));
    return launched(hipLaunchCooperativeKernel(fn, dim3(L.G), dim3(kResT), args, (unsigned)lds, s));
}

int res_run(ResWork& W, int max_inner, hipStream_t s) {
    const size_t m = std::max(W.n_words, W.n_pex);
    hipLaunchKernelGGL(k_res_clear, dim3(ceil_div(m, 256)), dim3(256), 0, s, W.n_words, W.words, W.n_pex, W.pex,
                       W.abort);
    PG_HIP(hipGetLastError());
    PG_HIP(allow_lds(k_res_cocg, kResLds));
    for (const ResWork::Round& r : W.rounds) {
        const ResDom* doms = reinterpret_cast<const ResDom*>(W.doms);
        const int* blk = W.blk + r.blk0;
        int polls = W.polls;
        int* abort = W.abort;
        void* args[5] = {&doms, &blk, &max_inner, &polls, &abort};
        PG_TRY(launched(hipLaunchCooperativeKernel(reinterpret_cast<const void*>(k_res_cocg), dim3(r.nblk), dim3(kResT),
                                                   args, (unsigned)r.lds, s)));
    }
    return PETGEM_OK;
}

}  // namespace petgem
