// Internal declarations of the HIP library: the system and solution handles,
// device-side helpers and the kernel launchers shared by the .hip units.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/petgem.h"
#include "mesh.h"

namespace petgem {

constexpr double kPi = 3.14159265358979323846;
constexpr double kMu0 = 4.0e-7 * kPi;
constexpr int kMaxRestart = 64;
// GMRES, both forms: an Arnoldi step takes a second Gram-Schmidt pass when
// beta^2 <= kGmEta |w|^2 (cancellation), and once the cycle has brought its residual
// down by kGmDrop. One pass loses orthogonality as 1e-16 times the square of
// that reduction; beyond 1e7 (a loss of 1e-2) the estimate of the residual no longer
// follows it. Steps of six roundings of b, with the first rule alone and with both
// (in a mirror): 26 unknowns to 1e-9 in one cycle 17 to 27, and 17; 3,000 to 1e-8 with
// restart 60 53 to 59, and 52; 600 to 1e-12 with restart 64 64 to 159, and 44. 1e-6
// takes the same steps and more second passes, 3e-8 leaves them uneven. A cycle of a
// larger mesh brings its residual down by 1e1 to 1e3, and its steps are as before.
constexpr double kGmEta = 1e-2, kGmDrop = 1e-7;

void set_error(const std::string& msg);

// ---------------------------------------------------------------- errors
#define PG_HIP(call)                                                          \
    do {                                                                      \
        hipError_t e_ = (call);                                               \
        if (e_ != hipSuccess) {                                               \
            ::petgem::set_error(std::string(#call) + ": " + hipGetErrorString(e_)); \
            return e_ == hipErrorOutOfMemory ? PETGEM_OUT_OF_MEMORY : PETGEM_HIP_ERROR; \
        }                                                                     \
    } while (0)

#define PG_TRY(call)                      \
    do {                                  \
        int rc_ = (call);                 \
        if (rc_ != PETGEM_OK) return rc_; \
    } while (0)

template <class T>
inline int dalloc(T** p, size_t count) {
    *p = nullptr;
    if (count == 0) return PETGEM_OK;
    hipError_t e = hipMalloc(reinterpret_cast<void**>(p), count * sizeof(T));
    if (e != hipSuccess) {
        (void)hipGetLastError();   // else the next launch's check would report it
        set_error(std::string("hipMalloc of ") + std::to_string(count * sizeof(T)) + " bytes: " +
                  hipGetErrorString(e));
        return e == hipErrorOutOfMemory ? PETGEM_OUT_OF_MEMORY : PETGEM_HIP_ERROR;
    }
    return PETGEM_OK;
}
template <class T>
inline void dfree(T*& p) {
    if (p) (void)hipFree(p);
    p = nullptr;
}

// Device memory of a system that only makes it faster: the layouts and buffers
// of the one-launch solves, right-hand side staging beyond one source's. A caller may
// bound it (petgem_set_spare_limit); beyond that, as where the device has no more, the
// forms that do without are taken.
struct Spare {
    int64_t limit = -1;           // -1: none
    int64_t used = 0;
    bool room(int64_t bytes) const { return limit < 0 || bytes <= limit - used; }
    template <class T>
    int take(T** p, size_t count, int64_t& held) {
        *p = nullptr;
        const int64_t bytes = (int64_t)(count * sizeof(T));
        if (!room(bytes)) {
            set_error("beyond the limit of spare device memory");
            return PETGEM_OUT_OF_MEMORY;
        }
        PG_TRY(dalloc(p, count));
        used += bytes;
        held += bytes;
        return PETGEM_OK;
    }
    void back(int64_t& held) {
        used -= held;
        held = 0;
    }
};

// Sliced-ELLPACK copy of the complex64 operator (the pattern and the real K,
// M_sigma values): slices of 64 rows, stored column-major inside a slice so a
// wavefront reads one entry of each of its 64 rows per load; rows are padded
// to the slice's longest with zero values that point at the row itself.
// Inside every 256-row tile the rows are ordered by length (longest first,
// then by index) before they are cut into slices, so that a slice holds rows
// of like length: on a 434k-DOF marine mesh this takes the padding from 18.6 % of the
// nonzeros to 6.7 %. row[] maps each slice lane back to its matrix row.
struct Sell {
    int nsl = 0;
    int64_t elems = 0;
    int32_t* ptr = nullptr;   // [nsl + 1] first element of each slice
    int32_t* w = nullptr;     // [nsl] slice width
    int32_t* row = nullptr;   // [nsl * 64] matrix row of each slice lane
    int32_t* col = nullptr;   // [elems]
    float* K = nullptr;       // [elems]
    float* M = nullptr;       // [elems]
    bool values = false;      // K, M current
    void release() {
        dfree(ptr); dfree(w); dfree(row); dfree(col); dfree(K); dfree(M);
        nsl = 0;
        elems = 0;
        values = false;
    }
};

// Multicolour split of the complex64 operator for the SSOR preconditioner:
// the DOFs coloured so that no two of a colour share a matrix entry, rows
// listed colour by colour (in DOF order within a colour), and for each listed
// row its entries coupling to earlier colours (L) and to later colours (U),
// the diagonal left out. pos: the entry's position in the CSR arrays, from
// which the values are gathered again whenever K32, Ms32 change.
struct Ssor {
    int nc = 0;                        // colours
    std::vector<int32_t> cptr;         // host [nc + 1] listed rows of each colour
    std::vector<int32_t> color_h;      // host [n] colour of each DOF
    int32_t* row = nullptr;            // [n] DOF of each listed row
    int32_t *lrp = nullptr, *lcol = nullptr, *lpos = nullptr;   // [n + 1], [nl], [nl]
    int32_t *urp = nullptr, *ucol = nullptr, *upos = nullptr;   // [n + 1], [nu], [nu]
    float *lK = nullptr, *lM = nullptr, *uK = nullptr, *uM = nullptr;
    double2* dg = nullptr;             // [n] {Kd, Md} of each listed row (read contiguously by the sweeps)
    int64_t nl = 0, nu = 0;
    bool values = false;               // lK .. uM, dg current
    void release() {
        dfree(row); dfree(lrp); dfree(lcol); dfree(lpos); dfree(urp); dfree(ucol); dfree(upos);
        dfree(lK); dfree(lM); dfree(uK); dfree(uM); dfree(dg);
        nc = 0; nl = nu = 0; values = false;
        cptr.clear(); color_h.clear();
    }
};

// A mesh's operator laid out for the resident COCG (resident.hip): G
// workgroups of rw consecutive rows each, their rows ordered by length, the
// entries in the order the registers take them (chunks of four per lane, LDS
// indices of 16 bits) and each workgroup's outer neighbours.
struct Resident {
    int state = 0;                // 0 not built, 1 usable, -1 the mesh does not fit
    int G = 0, rw = 0, rwcap = 0; // workgroups; rows of each; their LDS slots
    int hcap = 0, hmax = 0;       // most outer neighbours of a workgroup; stride of halo
    char* pattern = nullptr;      // one allocation that holds the next five
    int32_t* rows = nullptr;      // [G][rwcap] matrix row of each slot (-1: none)
    int32_t* wend = nullptr;      // [G][8][4] chunks of a wave's row slots, cumulative
    int32_t* halo = nullptr;      // [G][hmax] exchange place of each outer neighbour
    int32_t* nh = nullptr;        // [G]
    uint64_t* idx = nullptr;      // [G][8][chunks][64] four LDS indices
    float* K = nullptr;           // [G][8][chunks][64][4], then M (built when the COCG first needs them)
    float* M = nullptr;
    bool values = false;          // K, M current
    double2* A = nullptr;         // [G][8][chunks][4][64] A D^-1 of the plain GMRES at a_freq
    double a_freq = -1.0;
    int64_t held = 0;             // bytes of all of it
    void release(Spare& spare);
};

// Background of the primary field: the whole space sigma_bg, or two
// half-spaces meeting at z = z0 (s_up above, holding the sources).
struct Layers {
    int on = 0;
    double z0 = 0.0, s_up = 1.0, s_dn = 1.0;
};

// ------------------------------------------------------- GMRES control block
// Small device-resident state of one GMRES cycle: the Hessenberg column in
// progress, Givens rotations, the least-squares right-hand side g and flags
// that let every later kernel of the cycle exit early once it has converged.
struct GmresCtl {
    double2 H[(kMaxRestart + 1) * kMaxRestart];  // column-major, ld = kMaxRestart+1
    double2 cs[kMaxRestart], sn[kMaxRestart];
    double2 g[kMaxRestart + 1];
    double2 h[kMaxRestart + 1];                   // coefficients of the current pass
    double2 y[kMaxRestart];
    double nrm2;        // |w|^2 of the current pass
    double scale;       // multiplier applied by the update kernel
    double tol_abs;     // rtol * |b|
    double rnorm;       // true residual norm at the start of the cycle
    int done;           // cycle finished (converged estimate or breakdown)
    int reorth;         // second Gram-Schmidt pass requested
    int mdone;          // Arnoldi steps completed in this cycle
    int nonfinite;
};

struct GmresWork {
    int n = 0, m = 0, nb_dot = 0;
    double2* V = nullptr;        // (m+1) x n basis
    double2* u = nullptr;        // scaled iterate D x
    double2* b = nullptr;        // right-hand side of the current source
    double* partial = nullptr;   // [(m+2)][nb_dot] complex partial sums
    GmresCtl* ctl = nullptr;
    GmresCtl* ctl_host = nullptr;  // pinned mirror for the per-cycle readback
    hipGraphExec_t graph = nullptr;  // one captured cycle
    hipStream_t graph_stream = nullptr;
    void release();
};

// ------------------------------------------------------- resident COCG
struct GmOut {                    // what a resident GMRES reports
    double bnorm, rnorm;
    int iters, cycles, status, pad;
};
struct GmHost {
    GmOut out;
    int abort, flag;
};
// Solves that run kernel by kernel after one without room for the one-launch
// form, or one in which a wait of it ran out: either is likely to come again
// (a wait that runs out costs about a second), and may pass.
constexpr int kResSkip = 64;
constexpr int kResAborted = 1;    // a launch that the device refuses, or whose wait ran out
// Device tables and exchange buffers of one solve's resident launches, in one
// allocation that a plan lays out.
struct ResWork {
    struct Round { int blk0 = 0, nblk = 0; size_t lds = 0; };
    std::vector<Round> rounds;    // one launch each
    int skip = 0;                 // solves that run kernel by kernel before this form is tried again
    int polls = 0;                // of one wait
    Spare* spare = nullptr;       // of the system that holds it
    char* buf = nullptr;
    int64_t held = 0;             // its bytes
    char* doms = nullptr;
    int* blk = nullptr;           // domain of each logical block
    unsigned long long *words = nullptr, *pex = nullptr;
    size_t n_words = 0, n_pex = 0;
    int* abort = nullptr;
    Resident* L = nullptr;        // GMRES: the layout of the plan
    double2* V = nullptr;         // basis, in the layout's order
    double2 *b = nullptr, *u = nullptr;
    GmOut* out = nullptr;
    GmHost* host = nullptr;       // pinned; the COCG uses its abort only
    int room(size_t bytes);       // buf of at least so many
    void give_back();             // buf
    void release();
};
// One mesh of a solve: its rows start at row_off of the block vectors, its C
// columns have the states and frequencies from seg * C on.
struct ResItem {
    petgem_system* sys;
    size_t row_off;
    int seg, C;
};
struct ResVectors {
    const double2* R64;
    float2* Xi;
    void* st;                     // ColState
    const double* wmu;
};

// ------------------------------------------------------- multi-RHS workspace
struct BlockWork;   // defined in block.hip
void release_block_work(BlockWork*& w);

struct ReceiverCache {
    std::vector<double> rx;     // host copy of the located coordinates
    int32_t n_rx = 0;
    int32_t* tet = nullptr;     // device [n_rx]
    int32_t* dof = nullptr;     // device [n_rx][6]
    double* xyz = nullptr;      // device [n_rx][3]
    void release() { dfree(tet); dfree(dof); dfree(xyz); n_rx = 0; rx.clear(); }
};

}  // namespace petgem

struct petgem_system {
    int device = 0;
    int32_t n_nodes = 0, n_tets = 0, n_dof = 0, n_edges = 0;
    int64_t nnz = 0;
    double h_mean = 0.0;
    double sigma_bg = 1.0;
    petgem::Layers layers;                // layered background (layers.on) of the primary field
    double setup_seconds = 0.0;
    // host copies kept for receivers and accessors
    std::vector<double> xyz_h;
    std::vector<int32_t> tets_h;
    std::vector<int32_t> elem_dof_h;      // [T][6] DOF or -1
    std::vector<int32_t> dof_nodes_h;     // [n_dof][2]
    std::vector<int32_t> row_ptr_h;       // kept for host-side tools
    // device topology
    double* xyz = nullptr;                // [N][3]
    int32_t* tets = nullptr;              // [T][4]
    double* sigma = nullptr;              // [T]
    int32_t* row_ptr = nullptr;           // [n+1]
    int32_t* col = nullptr;               // [nnz]
    int32_t* cptr = nullptr;              // [nnz+1]
    int32_t* cidx = nullptr;              // contributions
    int32_t* iptr = nullptr;              // [n+1]
    int32_t* islot = nullptr;             // incidence slots
    // assembled real matrices (frequency independent)
    double2* KMst = nullptr;              // [21][T] staging: {K^e, sigma_e M^e} entries
    double* K = nullptr;                  // [nnz]
    double* Ms = nullptr;                 // [nnz]
    double* Kd = nullptr;                 // [n]
    double* Msd = nullptr;                // [n]
    // single-precision copies for the mixed-precision path
    float* K32 = nullptr;
    float* Ms32 = nullptr;
    bool have32 = false;
    petgem::Sell sell32;     // sliced-ELLPACK copy of K32 / Ms32 (built on first use)
    petgem::Resident res[2]; // finer and coarser split for the resident COCG (built on first use)
    petgem::Ssor ssor32;     // multicolour L / U split of K32 / Ms32 (built on first SSOR use)
    // frequency-specific operator of the FP64 GMRES: Ahat = A D^{-1}
    double cached_freq = -1.0;            // of Ahat
    double diag_freq = -1.0;              // of dvec, dinv
    double2* Ahat = nullptr;              // [nnz]
    double2* dvec = nullptr;              // [n] D = diag(A)
    double2* dinv = nullptr;              // [n]
    // right-hand-side staging and error flag
    double2* Rst = nullptr;               // [rst_copies][6][T]
    int rst_copies = 0;
    int* hot = nullptr;                   // layered background: count, then the elements with dsigma != 0
    int* dflag = nullptr;                 // device error flags
    double2* xtmp = nullptr;              // [n] copy of the operand of a product that overlaps its result
    // voxel grid of the learned initial guess (cached at first use)
    int32_t* vox_tet = nullptr;           // [32^3] element containing each voxel centre
    int32_t* vox_dof = nullptr;           // [32^3][6]
    double* dof_mid = nullptr;            // [n][3] edge midpoints
    double* dof_tan = nullptr;            // [n][3] unit tangents (lo -> hi)
    double vox_lo[3] = {0.0, 0.0, 0.0};
    double vox_h = 0.0, vox_L = 0.0;
    int spmv_group = 8;                   // lanes per CSR row (autotuned)
    bool spmv_tuned = false;
    double tune_freq = 0.0;               // of the latest double-precision product or solve that did not tune
    float spmv_tune_ms[3] = {0.f, 0.f, 0.f};  // measured 4/8/16-lane SpMV times
    int wait_polls = 0;                   // polls of one wait of a one-launch solve (0: the default)
    petgem::Spare spare;
    int64_t rst_held = 0;                 // of it, in Rst
    bool rst_one = false;                 // no room for more than one source's staging
    petgem::GmresWork gw;
    petgem::ResWork gres;                 // tables and exchange buffers of the resident GMRES
    petgem::BlockWork* bw = nullptr;
    petgem::ReceiverCache rxc;
};

struct petgem_solution {
    petgem_system* sys = nullptr;
    int32_t n_src = 0;
    double2* x = nullptr;                 // [n_src][n_dof]
    std::vector<petgem_source> src;
    double sigma_bg = 1.0;
    petgem::Layers layers;                // the background the solve used
};

namespace petgem {

// Launchers implemented in the .hip units; all ordered on `s`.
// sigma: device [n_tets], kept in sys->sigma by the launch
int launch_assembly(petgem_system* sys, const double* sigma, hipStream_t s);
int launch_diag(petgem_system* sys, double freq, hipStream_t s);
int launch_freq_prep(petgem_system* sys, double freq, hipStream_t s);
// allocation-free scratch of this device (looked up once per device) and the
// right-hand side that uses it
int noalloc_scratch(int dev, char** out);
int rhs_noalloc(petgem_system* sys, const petgem_source* src, int32_t n_src, double2* b, hipStream_t s);
// one or two right-hand sides (src[0 .. ns - 1] into b + c * step); fresh: the
// staging holds nothing of these conductivities yet
constexpr int kRhsJobs = 8;       // tasks of a launch
struct RhsTask {
    petgem_system* sys;
    const petgem_source* src;
    int ns;
    double2* b;
    size_t step;
    int stride, fresh;
    double2* Rst;                 // [6][n_tets][ns]
    int* flag;
};
int launch_rhs_tasks(const RhsTask* tasks, int n, hipStream_t s);
int rhs_staging(petgem_system* sys, int n_src, int* copies);
int launch_rhs_into(petgem_system* sys, const petgem_source* src, int n_src, double2* b, size_t step, int stride,
                    double2* Rst, int copies, int* flag, hipStream_t s);
// time per round of a graph-replayed kernel boundary (mode 0) or of a grid
// barrier in one cooperative kernel (mode 1), probe.hip
int sync_probe(int32_t rounds, int32_t mode, int32_t* blocks_out, float* us_per_round, hipStream_t s);
// layered background (layered.hip)
// entries of n <= 2 kRhsJobs sources, source c's into Rst[c][(i n_tets + t) ns]
int launch_rhs_layered(petgem_system* sys, const petgem_source* src, double2* const* Rst, int n, int ns, int fresh,
                       int* flag, hipStream_t s);
int launch_receivers_layered(const petgem_solution* sol, int k, int32_t n_rx, double2* E, double2* Es,
                             hipStream_t s);
int launch_rhs(petgem_system* sys, const petgem_source* src, int n_src, double2* b, size_t step, int stride,
               hipStream_t s);
int tune_spmv(petgem_system* sys, hipStream_t s);
// y = A(freq) x, double precision
int launch_spmv(petgem_system* sys, double freq, const double2* x, double2* y, hipStream_t s);
int launch_receivers(const petgem_solution* sol, int32_t n_rx, double2* E, double2* Es,
                     hipStream_t s, bool magnetic = false);
int gmres_solve(petgem_system* sys, const petgem_source& src, const petgem_opts& o,
                const double2* x0, double2* x_out, hipStream_t s, petgem_stats* st);
int block_solve(petgem_system* sys, const petgem_source* src, int32_t n_src,
                const petgem_opts& o, const double2* x0, double2* x_out, hipStream_t s,
                petgem_stats* st);
int batch_solve(petgem_system* const* systems, const petgem_source* src, int32_t n_sys,
                const petgem_opts& o, const void* const* x0, petgem_solution** sols, hipStream_t s,
                petgem_stats* st);
int ensure_fp32(petgem_system* sys, hipStream_t s);
// gives back all spare memory of a system and lets it be tried again
void release_spare(petgem_system* sys);
ResWork* block_res(BlockWork* w);   // null: no workspace
// Resident COCG: lays the meshes out and fills the launch tables (*fits false:
// some mesh is too large, use the kernel-per-phase form); then one inner solve
// of every column whose state is `outer`, at most max_inner iterations. After
// it *W.abort is non-zero if a wait ran out.
int res_plan(ResWork& W, const std::vector<ResItem>& items, const ResVectors& v, hipStream_t s, bool* fits);
int res_run(ResWork& W, int max_inner, hipStream_t s);
// The plain GMRES in one launch: room for it, then the solve of W.b into W.u, W.out
int gm_plan(petgem_system* sys, ResWork& W, int restart, hipStream_t s, bool* fits);
int gm_run(petgem_system* sys, ResWork& W, double freq, int restart, int max_iter, double rtol, hipStream_t s);
// the multicolour split of the operator (pattern built once, values gathered
// again after every reassembly); ssor_apply: z = M^-1 r of one complex64
// column at one frequency (device vectors of n_dof)
int ensure_ssor(petgem_system* sys, hipStream_t s);
int ssor_apply1(petgem_system* sys, double freq, double omega, const float2* r, float2* z, hipStream_t s);
// complex64 SpMM shapes the autotuner times for C columns (codes as the
// spmv_shape statistic); returns the count, writes at most cap codes
int spmm_candidate_codes(int C, bool sliced, int32_t* out, int cap);

// Lets a kernel be launched with up to `bytes` of dynamic LDS on the current
// device: ahead of each launch (0.14 us), since the library keeps no record of
// devices, and with the same number at each, so that threads that launch the
// same kernel for different sizes do not lower each other's.
template <class F>
inline hipError_t allow_lds(F kernel, int bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// Grid helpers
inline int ceil_div(int64_t a, int64_t b) { return int((a + b - 1) / b); }

}  // namespace petgem
