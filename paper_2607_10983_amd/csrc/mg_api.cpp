// Host side of the C ABI declared in include/mg.h: parameter validation,
// hierarchy allocation, Chebyshev schedules, coarsest-level solver setup and
// the outer defect-correction loop.  All device work is issued on the
// context's stream through the launchers of kernels.hip.
#include "mg.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "flat_row.h"
#include "geometry_bwd.h"
#include "host_slots.h"
#include "kernels.h"
#include "pcg_row.h"
#include "setup.h"
#include "tail.h"
#include "var_row.h"
#include "var_tail.h"
#include "var_visit.h"
#include "visit.h"

#include <type_traits>

using namespace mg;

namespace {

struct Level {
    int n = 0;
    size_t N = 0;
    double h = 0, ih2 = 0;
    void* x[3] = {nullptr, nullptr, nullptr};  // inner iterates; x[2] only where two-step kernels run
    void* b = nullptr;                // inner right-hand side / restricted residual
    void* coeff = nullptr;            // inner-precision coefficients (6 N), nullptr for 7-point
    double lmax = 2.0;                // Gershgorin bound of D^-1 M
    int cur = 0;                      // which x holds the current iterate
    bool x1 = false;                  // x[0] already holds the first step from zero for the current b
    // smoothing schedule: step k computes x + a_k (x - x_prev) + c_k D^-1 (b - M x)
    std::vector<double> a, c;
};

struct TimingPair {
    hipEvent_t start, stop;
};

// Integer results of the setup kernels: bounds per level (bits of a double),
// invalid cells per level from 16, invalid entries of the coarsest inverse at
// 32, its elimination steps that met an indefinite block at 33.
constexpr int kSetupSlots = 34;

}  // namespace

struct mg_ctx {
    mg_params p{};
    hipStream_t stream = nullptr;
    bool other_streams = false;  // work may be left on a stream it had before
    int device = 0;
    bool var = false;
    bool inner_double = true;   // inner V-cycle in double (MG_FP64) or float
    std::vector<Level> lev;
    // fine-level coefficients used by the outer residual
    void* coeff_outer = nullptr;
    bool coeff_outer_double = true;
    void* mem = nullptr;        // the context's device memory when it owns it
    u64* slots = nullptr;       // integer results of the setup kernels
    double* phi_tmp = nullptr;  // second buffer for the phi update
    double* partials = nullptr;
    int nparts = 0;        // partial sums written by launch_block_sums on the fine grid
    int nparts_outer = 0;  // partial sums written by launch_outer_residual
    double* dscal = nullptr;    // device scalars
    double* hscal = nullptr;    // pinned host mirror
    // The outer sums wait to be finished by the next pass from zero on level 0
    // (an extra block of that kernel) instead of a finalize launch.
    bool pending_sums = false;
    bool fuse_sums = true;
    double* Q = nullptr;        // coarsest seven-point basis and eigenvalues
    double* lam1 = nullptr;
    double* G = nullptr;        // coarsest variable-coefficient pseudo-inverse
    int tail_start = -1;        // first level run by the single-workgroup tail kernel, -1 = none
    bool x1_ready = false;      // the outer residual already wrote level 0's first smoothing step
    int x1_buf = 0;             // ... into this level-0 iterate buffer
    // The coarse sub-cycle (levels 1 .. coarsest) touches only context-owned
    // buffers with fixed arguments, so it can be captured once into a HIP graph
    // and replayed with one launch per V-cycle (MG_OPT_GRAPH).
    bool use_graph = false;
    bool capturing = false;
    hipStream_t cap_stream = nullptr;
    hipGraph_t coarse_graph = nullptr;
    hipGraphExec_t coarse_exec = nullptr;
    int coarse_cur = 0;
    hipEvent_t norm_ev = nullptr;  // completion of a scalar readback (conjugate gradients)
    // The outer sums need no event: the block
    // that writes them to the pinned mirror makes them visible at system
    // scope and then writes sums_seq to hscal[kHostFlagSlot], which the host
    // polls.  An event there cost a 5.6 us stall between the pass from zero
    // and the next kernel at 256^3 (4.6 us without its system-scope release).
    double sums_seq = 0.0;
    bool scal_flag = false;  // the pending readback is the flag, not norm_ev
    double mean_seq = 0.0;   // number of the last readback of the sum of b
    bool use_pairs = true;         // last two steps of a smoothing pass in one two-step kernel
    bool use_visits = true;        // fused visits of the 32^3 and 64^3 levels
    bool use_tail = true;          // levels of at most 16^3 points in one workgroup
    // conjugate-gradient state (allocated by the first mg_solve_pcg)
    double* pcg_r = nullptr;
    double* pcg_p[2] = {nullptr, nullptr};
    double* pcg_q = nullptr;
    double* pcg_s = nullptr;
    double* pcg_partials = nullptr;
    double* scratch = nullptr;  // double scratch for the single-step entry points
    size_t scratch_elems = 0;
    std::string err;
    // timing of the fine-level smoothing kernel
    int timing = 0;  // mask of timed kernel kinds (MG_TIME_STEP, MG_TIME_PAIR, MG_TIME_TRIPLE)
    std::vector<TimingPair> events;
    size_t events_used = 0;
    int timed_launches = 0;
    double timed_ms = 0.0;
    double timed_bytes = 0.0;
};

namespace {

const char* kStatus[] = {"MG_OK",
                         "MG_ERR_INVALID: invalid argument",
                         "MG_ERR_INVALID_COEFF: coefficient field not finite or with a non-positive diagonal component",
                         "MG_ERR_NOMEM: device allocation failed",
                         "MG_ERR_HIP: HIP runtime error",
                         "MG_ERR_NONFINITE: NaN or Inf encountered",
                         "MG_ERR_NOT_CONVERGED: tolerance not reached"};

mg_status fail(mg_ctx* ctx, mg_status s, const std::string& msg) {
    if (ctx) ctx->err = msg;
    return s;
}

#define HIPCHK(ctx, ...)                                                                           \
    do {                                                                                           \
        hipError_t e_ = (__VA_ARGS__);                                                             \
        if (e_ != hipSuccess)                                                                      \
            return fail((ctx), MG_ERR_HIP, std::string(#__VA_ARGS__) + ": " + hipGetErrorString(e_)); \
    } while (0)

bool is_pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }

mg_status dalloc(mg_ctx* ctx, void** p, size_t bytes) {
    *p = nullptr;
    if (bytes == 0) return MG_OK;
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) {
        *p = nullptr;
        (void)hipGetLastError();
        return fail(ctx, MG_ERR_NOMEM, "hipMalloc of " + std::to_string(bytes) + " bytes failed");
    }
    return MG_OK;
}

void dfree(void* p) {
    if (p) (void)hipFree(p);
}

int coarsest_n(const mg_params& p) { return p.n >> (p.levels - 1); }

// Chebyshev schedule on [lmax/alpha, lmax] (three-term recurrence, x_prev form).
void make_schedule(const mg_params& p, Level& L) {
    L.a.clear();
    L.c.clear();
    if (p.smoother == MG_JACOBI) {
        for (int k = 0; k < p.jacobi_sweeps; ++k) {
            L.a.push_back(0.0);
            L.c.push_back(p.jacobi_omega);
        }
        return;
    }
    const double lmin = L.lmax / p.cheb_alpha;
    const double theta = 0.5 * (L.lmax + lmin), delta = 0.5 * (L.lmax - lmin), sigma = theta / delta;
    double rho = 1.0 / sigma;
    L.a.push_back(0.0);
    L.c.push_back(1.0 / theta);
    for (int k = 1; k < p.cheb_degree; ++k) {
        const double rn = 1.0 / (2.0 * sigma - rho);
        L.a.push_back(rn * rho);
        L.c.push_back(2.0 * rn / delta);
        rho = rn;
    }
}

// Real orthonormal Fourier basis of the periodic second difference on nc points.
void flat_basis(int nc, double hc, std::vector<double>& Q, std::vector<double>& lam) {
    Q.assign((size_t)nc * nc, 0.0);
    lam.assign(nc, 0.0);
    const double pi = std::acos(-1.0);
    auto eig = [&](int m) { double s = std::sin(pi * m / nc); return -4.0 * s * s / (hc * hc); };
    for (int j = 0; j < nc; ++j) Q[j + nc * 0] = 1.0 / std::sqrt((double)nc);
    lam[0] = 0.0;
    for (int m = 1; m < nc / 2; ++m) {
        for (int j = 0; j < nc; ++j) {
            Q[j + nc * (2 * m - 1)] = std::sqrt(2.0 / nc) * std::cos(2.0 * pi * m * j / nc);
            Q[j + nc * (2 * m)] = std::sqrt(2.0 / nc) * std::sin(2.0 * pi * m * j / nc);
        }
        lam[2 * m - 1] = lam[2 * m] = eig(m);
    }
    for (int j = 0; j < nc; ++j) Q[j + nc * (nc - 1)] = (j % 2 ? -1.0 : 1.0) / std::sqrt((double)nc);
    lam[nc - 1] = eig(nc / 2);
}

// Dense matrix of the 19-point operator on the coarsest level (host, double).
void assemble_dense(int n, double ih2, const std::vector<double>& C, std::vector<double>& M) {
    const int N = n * n * n;
    M.assign((size_t)N * N, 0.0);
    auto id = [n](int x, int y, int z) { return (((z % n + n) % n) * n + ((y % n + n) % n)) * n + ((x % n + n) % n); };
    auto cc = [&](int c, int x, int y, int z) { return C[(size_t)c * N + id(x, y, z)]; };
    for (int z = 0; z < n; ++z)
        for (int y = 0; y < n; ++y)
            for (int x = 0; x < n; ++x) {
                const int i = id(x, y, z);
                const int p[3] = {x, y, z};
                for (int a = 0; a < 3; ++a)
                    for (int s = -1; s <= 1; s += 2) {
                        int q[3] = {p[0], p[1], p[2]};
                        q[a] += s;
                        const double cf = 0.5 * (cc(a, x, y, z) + cc(a, q[0], q[1], q[2]));
                        M[(size_t)i * N + id(q[0], q[1], q[2])] += cf * ih2;
                        M[(size_t)i * N + i] -= cf * ih2;
                    }
                const int pa[3] = {0, 0, 1}, pb[3] = {1, 2, 2};
                for (int k = 0; k < 3; ++k) {
                    const int a = pa[k], b = pb[k], comp = 3 + k;
                    for (int sa = -1; sa <= 1; sa += 2)
                        for (int sb = -1; sb <= 1; sb += 2) {
                            int qa[3] = {p[0], p[1], p[2]}, qb[3] = {p[0], p[1], p[2]}, q[3] = {p[0], p[1], p[2]};
                            qa[a] += sa;
                            qb[b] += sb;
                            q[a] += sa;
                            q[b] += sb;
                            const double v = sa * sb * (cc(comp, qa[0], qa[1], qa[2]) + cc(comp, qb[0], qb[1], qb[2])) * 0.25 * ih2;
                            M[(size_t)i * N + id(q[0], q[1], q[2])] += v;
                        }
                }
            }
}

// Zero-mean pseudo-inverse of a symmetric M with null space span(1):
// B = M - s 11^T / N is regular, and G = P B^-1 P with P = I - 11^T / N.
// Eliminated with partial pivoting, so M need not be semidefinite.
bool pseudo_inverse(int N, const std::vector<double>& M, std::vector<double>& G) {
    double s = 0.0;
    for (int i = 0; i < N; ++i) s += std::fabs(M[(size_t)i * N + i]);
    s /= N;
    std::vector<double> A((size_t)N * 2 * N, 0.0);
    for (int i = 0; i < N; ++i) {
        for (int j = 0; j < N; ++j) A[(size_t)i * 2 * N + j] = M[(size_t)i * N + j] - s / N;
        A[(size_t)i * 2 * N + N + i] = 1.0;
    }
    const int W = 2 * N;
    for (int col = 0; col < N; ++col) {  // Gauss-Jordan with partial pivoting
        int piv = col;
        for (int r = col + 1; r < N; ++r)
            if (std::fabs(A[(size_t)r * W + col]) > std::fabs(A[(size_t)piv * W + col])) piv = r;
        if (A[(size_t)piv * W + col] == 0.0) return false;
        if (piv != col)
            for (int j = 0; j < W; ++j) std::swap(A[(size_t)piv * W + j], A[(size_t)col * W + j]);
        const double inv = 1.0 / A[(size_t)col * W + col];
        for (int j = 0; j < W; ++j) A[(size_t)col * W + j] *= inv;
        for (int r = 0; r < N; ++r) {
            if (r == col) continue;
            const double f = A[(size_t)r * W + col];
            if (f == 0.0) continue;
            for (int j = 0; j < W; ++j) A[(size_t)r * W + j] -= f * A[(size_t)col * W + j];
        }
    }
    std::vector<double> Bi((size_t)N * N);
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) Bi[(size_t)i * N + j] = A[(size_t)i * W + N + j];
    // G = P Bi P
    std::vector<double> rm(N, 0.0), cm(N, 0.0);
    double tm = 0.0;
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) {
            rm[i] += Bi[(size_t)i * N + j] / N;
            cm[j] += Bi[(size_t)i * N + j] / N;
        }
    for (int i = 0; i < N; ++i) tm += rm[i] / N;
    G.assign((size_t)N * N, 0.0);
    for (int i = 0; i < N; ++i)
        for (int j = 0; j < N; ++j) G[(size_t)i * N + j] = Bi[(size_t)i * N + j] - rm[i] - cm[j] + tm;
    return true;
}

// Carves a context's fields out of one block of device memory; with a null
// base it only adds up the sizes.
struct Arena {
    char* base;
    size_t used = 0;
    void* take(size_t bytes) {
        const size_t at = used;
        used += (bytes + 255) & ~(size_t)255;
        return base ? base + at : nullptr;
    }
    double* doubles(size_t count) { return (double*)take(count * sizeof(double)); }
};

// The contexts' pinned host mirrors.  Portable, so a slot serves a context on
// any device; coherent: the finalize kernels write the outer sums into it
// directly.  Never destroyed: contexts may be, after the library's statics.
HostSlots& host_slots() {
    static HostSlots* slots = new HostSlots(
        [](double** page, size_t bytes) {
            return (int)hipHostMalloc((void**)page, bytes, hipHostMallocCoherent | hipHostMallocPortable);
        },
        [](double* page) { (void)hipHostFree(page); });
    return *slots;
}

template <typename T>
OpDesc<T> op_of(const Level& L) {
    return OpDesc<T>{L.n, L.ih2, (const T*)L.coeff};
}

// ---- fine-level smoothing kernel timing ----------------------------------------------
// The event pair travels with the kernel's own dispatch (hipExtLaunchKernel),
// so the elapsed time is the kernel's execution time, as a profiler sees it.
mg_status time_events(mg_ctx* c, bool fine, int kind, hipEvent_t* ev0, hipEvent_t* ev1) {
    *ev0 = *ev1 = nullptr;
    if (!(c->timing & kind) || !fine) return MG_OK;
    if (c->events_used == c->events.size()) {
        TimingPair tp;
        // timing only: no system-scope release (an L2 writeback of every XCD,
        // 4-6 us of stall around the timed kernel)
        HIPCHK(c, hipEventCreateWithFlags(&tp.start, hipEventDisableSystemFence));
        HIPCHK(c, hipEventCreateWithFlags(&tp.stop, hipEventDisableSystemFence));
        c->events.push_back(tp);
    }
    *ev0 = c->events[c->events_used].start;
    *ev1 = c->events[c->events_used].stop;
    return MG_OK;
}
mg_status time_end(mg_ctx* c, bool fine, int kind, double bytes) {
    if (!(c->timing & kind) || !fine) return MG_OK;
    c->events_used++;
    c->timed_launches++;
    c->timed_bytes += bytes;
    if (c->events_used >= 16384) {  // harvest to bound the pool
        HIPCHK(c, hipStreamSynchronize(c->stream));
        for (size_t i = 0; i < c->events_used; ++i) {
            float ms = 0.f;
            HIPCHK(c, hipEventElapsedTime(&ms, c->events[i].start, c->events[i].stop));
            c->timed_ms += ms;
        }
        c->events_used = 0;
    }
    return MG_OK;
}

// ---- inner V-cycle ----------------------------------------------------------------------
// One smoothing pass on level l in inner precision T.  from_zero: the iterate is 0.
// index of an iterate buffer other than `cur` among x[0], x[1]
inline int other(int cur) { return cur == 0 ? 1 : 0; }

// The outer residual kernel can write level 0's first smoothing step (when
// level 0 is not itself run by the tail kernel).
inline bool x1_fusable(const mg_ctx* c) { return c->tail_start != 0 && c->lev.size() > 1; }

// Level l (not the coarsest, not run by the tail kernel) is visited by the
// fused visit kernels: seven-point operator, 32^3 points or, in a float
// hierarchy, 64^3; pre (post) selects the visit before (after) the coarse
// correction.
inline bool visit_level(const mg_ctx* c, int l, bool pre) {
    if (!(c->use_visits && !c->var && c->p.smoother == MG_CHEBYSHEV && l + 1 < (int)c->lev.size() &&
          l != c->tail_start))
        return false;
    const int n = c->lev[l].n, v = (int)c->lev[l].a.size();
    const size_t elem = c->inner_double ? sizeof(double) : sizeof(float);
    return pre ? visit_pre_applies(n, v, elem) : visit_post_applies(n, v, elem);
}

// 19-point levels of 32^3 points: pre- and post-visits in one launch each.
inline bool var_visit_level(const mg_ctx* c, int l) {
    return c->use_visits && c->var && l + 1 < (int)c->lev.size() && l != c->tail_start &&
           var_visit_applies(c->lev[l].n, (int)c->lev[l].a.size(),
                             c->inner_double ? sizeof(double) : sizeof(float));
}

// Level l's pass from zero can start from a first step written by the
// restriction that produces its right-hand side (19-point levels smoothed by
// separate kernels or visits).
inline bool first_step_level(const mg_ctx* c, int l) {
    return c->var && l > 0 && l + 1 < (int)c->lev.size() && l != c->tail_start;
}

// Level l's post-smoothing pass (three Chebyshev steps) runs fused with the
// prolongation before it.
inline bool post_fused(const mg_ctx* c, int l, size_t elem) {
    const Level& L = c->lev[l];
    return c->p.smoother == MG_CHEBYSHEV && L.a.size() == 3 && c->use_pairs && !c->var &&
           triple_pro_applies(L.n, elem);
}

// Level l's post-smoothing pass (Chebyshev, at least two steps) starts with a
// pair that forms x + P e itself: rows over 1 KB, where the three-step kernels
// do not run.  With an odd number of steps the last one is then a single step
// whose x_prev the pair wrote: 8.1 fields instead of 9.1 for the prolongation,
// a step and a pair (512^3 mixed, degree 3: 2.45 -> 2.32 ms per cycle).
inline bool post_pair_fused(const mg_ctx* c, int l, size_t elem) {
    const Level& L = c->lev[l];
    return c->p.smoother == MG_CHEBYSHEV && L.a.size() >= 2 && c->use_pairs && !c->var && L.x[2] != nullptr &&
           pair_pro_applies(L.n, elem);
}

// Level l's post-smoothing pass starts with a 19-point step that forms x + P e
// itself; a Chebyshev pass of several steps keeps that iterate, as the next
// step's x_prev, in the third buffer.  Not where the whole pass runs in pairs
// on rows of 1 KB: at 256^3 float the prolongation and a pair take 27 + 197 us,
// this step and a single one 141 + 127 to 137 (128^3: 5 + 30 and 17 + 15).
inline bool post_step_fused(const mg_ctx* c, int l, size_t elem) {
    const Level& L = c->lev[l];
    const bool cheb = c->p.smoother == MG_CHEBYSHEV;
    const size_t v = L.a.size();
    const bool paired = var_pair_applies(L.n, elem) && (size_t)L.n * elem >= 1024 && (cheb ? v == 2 : v % 2 == 0);
    return c->use_pairs && c->var && var_pro_applies(L.n, elem) && !paired &&
           (!cheb || v == 1 || L.x[2] != nullptr);
}

// Level l runs its pass from zero as one three-step kernel (first step formed
// from b on the fly): seven-point operator, two-step kernels available, and
// at least three steps per pass.
inline bool from_zero_triple(const mg_ctx* c, int l) {
    return c->use_pairs && !c->var && c->lev[l].x[2] != nullptr && c->lev[l].a.size() >= 3;
}

// pro_e (not from zero): the pass starts from x + P pro_e, formed by its first
// pair (post_pair_fused) or step (post_step_fused), instead of a prolongation
// launch.
template <typename T>
mg_status smooth_level(mg_ctx* c, int l, bool from_zero, const T* pro_e = nullptr) {
    Level& L = c->lev[l];
    const OpDesc<T> op = op_of<T>(L);
    int cur = L.cur;
    int prev = -1;  // buffer of x_{k-1}, -1 when x_{k-1} = 0 or not needed
    const bool cheb = c->p.smoother == MG_CHEBYSHEV;
    const bool fine = (l == 0);
    const double fbytes = (double)L.N * sizeof(T);
    const double cbytes = c->var ? 6.0 * (double)L.N * sizeof(T) : 0.0;
    T* bufs[3] = {(T*)L.x[0], (T*)L.x[1], (T*)L.x[2]};
    const int v = (int)L.a.size();
    // the last two steps of the pass run as one two-step kernel where it exists
    const bool pairs = c->use_pairs && L.x[2] != nullptr && !c->var;
    // 19-point: the last two Chebyshev steps of the pass run as one kernel, Jacobi steps two by two
    // (no x_prev, so no third buffer)
    const bool vpairs = c->use_pairs && c->var && var_pair_applies(L.n, sizeof(T)) && (!cheb || L.x[2] != nullptr);
    bool prev_b = false;  // x_{k-1} is the pointwise first step c0 D^-1 b, formed by the next kernel
    for (int k = 0; k < v; ++k) {
        double bytes = 0.0;
        if (k == 0 && from_zero && l == 0 && c->x1_ready) {  // formed by the outer residual kernel
            c->x1_ready = false;
            cur = c->x1_buf;
            prev = -1;
            continue;
        }
        if (k == 0 && from_zero && L.x1) {  // formed by the restriction above
            L.x1 = false;
            cur = 0;
            prev = -1;
            continue;
        }
        // Steps pair up from the end of the pass: an even number of remaining
        // steps runs as two-step kernels.  A pair that is not the last one also
        // writes its first step (the next pair's x_prev); that needs two free
        // buffers, i.e. no x_prev of its own.
        const int rem = v - k;
        const bool has_prev = cheb && prev >= 0;
        const bool need_y1 = cheb && rem > 2;
        // a pass from zero of degree 4: steps 0 and 1 from b alone (b -> x_2),
        // then steps 2 and 3 as a pair whose x_prev = x_1 is formed from b
        // (b, x_2 -> x_4): 5 field passes instead of 7 for steps 0-2 in one
        // kernel (b -> x_3, x_2) and step 3 on its own
        const bool fromb = k == 0 && from_zero && cheb && v == 4 && from_zero_triple(c, l);
        const bool triple = k == 0 && from_zero && from_zero_triple(c, l) && !fromb;
        // a pass of three steps that does not start from zero: one three-step kernel
        const bool triple3 = k == 0 && !from_zero && cheb && v == 3 && c->use_pairs && !c->var &&
                             triple_kernels_apply(L.n, sizeof(T));
        // a pass that prolongs on the fly starts with a pair whatever its degree
        const bool pro_pair = k == 0 && pro_e != nullptr && pairs && rem >= 2 && post_pair_fused(c, l, sizeof(T));
        const bool pair = pro_pair || (pairs && rem >= 2 && rem % 2 == 0 && !(k == 0 && from_zero) &&
                                       !(need_y1 && has_prev));
        const bool vpro = k == 0 && pro_e != nullptr && post_step_fused(c, l, sizeof(T));
        const bool vpair = vpairs && !vpro && (rem == 2 || (!cheb && rem % 2 == 0)) && !(k == 0 && from_zero);
        if (k == 0 && pro_e != nullptr && !pair && !vpro) return MG_ERR_INVALID;
        const int kind = triple3                               ? MG_TIME_TRIPLE
                         : (pair || triple || vpair) && !fromb ? MG_TIME_PAIR
                                                               : MG_TIME_STEP;
        hipEvent_t ev0, ev1;
        mg_status st = time_events(c, fine, kind, &ev0, &ev1);
        if (st != MG_OK) return st;
        if (fromb) {
            const int out = 1;
            const double D = -6.0 * L.ih2;
            HIPCHK(c, launch_smooth_fromb_row<T>(L.n, L.ih2, (const T*)L.b, bufs[out], L.a[1], L.c[1] / D,
                                                 L.c[0] / D, c->stream, ev0, ev1));
            bytes = 2.0 * fbytes;  // b; x_2
            prev = -1;
            prev_b = true;
            cur = out;
            k = 1;  // two steps done
        } else if (triple3) {
            const int out = other(cur);
            const double D = -6.0 * L.ih2;
            HIPCHK(c, launch_smooth_triple_row<T>(L.n, L.ih2, bufs[cur], (const T*)L.b, bufs[out], L.a[0],
                                                  L.c[0] / D, L.a[1], L.c[1] / D, L.a[2], L.c[2] / D, c->stream, ev0,
                                                  ev1));
            bytes = 3.0 * fbytes;  // x, b; x_3
            prev = -1;
            cur = out;
            k = 2;  // three steps done
        } else if (triple) {
            // steps 0, 1, 2 of the pass from zero: reads b, writes x_3 (and x_2
            // when a fourth step needs it as x_prev)
            const bool y1 = cheb && v > 3;
            const int out = 0, mid = y1 ? 1 : -1;
            const double D = -6.0 * L.ih2;
            // on level 0 the pending outer sums are finished by an extra block
            const bool sums = l == 0 && c->pending_sums;
            const SumsJob job{c->partials, c->nparts_outer, 3, c->dscal, 1, c->hscal, sums ? c->sums_seq + 1.0 : 0.0};
            HIPCHK(c, launch_smooth_pair_row<T>(L.n, L.ih2, nullptr, nullptr, (const T*)L.b, bufs[out],
                                                mid >= 0 ? bufs[mid] : nullptr, L.a[1], L.c[1] / D, L.a[2],
                                                L.c[2] / D, c->stream, ev0, ev1, 1, L.c[0] / D,
                                                sums ? &job : nullptr));
            if (sums) {
                c->sums_seq += 1.0;
                c->scal_flag = true;
                c->pending_sums = false;
            }
            bytes = (2.0 + (mid >= 0 ? 1.0 : 0.0)) * fbytes;  // b; x_3 [, x_2]
            prev = mid;
            cur = out;
            k = 2;  // three steps done
        } else if (vpro) {  // x, e -> x_1 and, where the next step needs it, x_0 = x + P e
            const int out = other(cur);
            const int keep = cheb && v > 1 ? 3 - cur - out : -1;
            HIPCHK(c, launch_var_pro<T, T>(L.n, L.ih2, op.coeff, bufs[cur], pro_e, (const T*)L.b, bufs[out],
                                           keep >= 0 ? bufs[keep] : nullptr, L.a[0], L.c[0], c->stream, ev0, ev1));
            bytes = (3.0 + 1.0 / 8.0 + (keep >= 0 ? 1.0 : 0.0)) * fbytes + cbytes;  // x, e, b, C; x_1, [x_0]
            prev = keep;
            cur = out;
        } else if (vpair) {  // x, x_prev -> y2 in the third buffer (the kernel reads both on halo rows)
            const T* xp = has_prev ? bufs[prev] : nullptr;
            const int out = has_prev ? 3 - cur - prev : other(cur);
            HIPCHK(c, launch_var_smooth_pair<T, T>(L.n, L.ih2, op.coeff, bufs[cur], xp, (const T*)L.b, bufs[out],
                                                   L.a[k], L.c[k], L.a[k + 1], L.c[k + 1], c->stream, ev0, ev1));
            bytes = (3.0 + (xp ? 1.0 : 0.0)) * fbytes + cbytes;  // x, [x_prev], b, C; y2
            prev = -1;
            cur = out;
            ++k;  // the pair's second step
        } else if (pair) {
            const T* xp = has_prev ? bufs[prev] : nullptr;
            int out, mid = -1;
            if (has_prev) {
                out = 3 - cur - prev;
            } else {
                const int f1 = cur == 0 ? 1 : 0;
                const int f2 = 3 - cur - f1;
                out = need_y1 ? f2 : f1;
                mid = need_y1 ? f1 : -1;
            }
            const double D = -6.0 * L.ih2;  // c / D rounded as in the single-step launch
            // after a step from b, level 0 finishes the pending outer sums here
            const bool sums = prev_b && l == 0 && c->pending_sums;
            const T* ec = k == 0 ? pro_e : nullptr;  // x0 = x + P e formed by this pair
            const SumsJob job{c->partials, c->nparts_outer, 3, c->dscal, 1, c->hscal, sums ? c->sums_seq + 1.0 : 0.0};
            HIPCHK(c, launch_smooth_pair_row<T>(L.n, L.ih2, bufs[cur], xp, (const T*)L.b, bufs[out],
                                                mid >= 0 ? bufs[mid] : nullptr, L.a[k], L.c[k] / D, L.a[k + 1],
                                                L.c[k + 1] / D, c->stream, ev0, ev1, prev_b ? 2 : 0, L.c[0] / D,
                                                sums ? &job : nullptr, ec));
            if (sums) {
                c->sums_seq += 1.0;
                c->scal_flag = true;
                c->pending_sums = false;
            }
            // x, [x_prev], b; y2, [y1]; [e once per coarse point]
            bytes = (3.0 + (xp ? 1.0 : 0.0) + (mid >= 0 ? 1.0 : 0.0) + (ec ? 1.0 / 8.0 : 0.0)) * fbytes;
            prev_b = false;
            prev = mid;
            cur = out;
            ++k;  // the pair's second step
        } else if (k == 0 && from_zero) {
            cur = 0;
            prev = -1;
            HIPCHK(c, launch_smooth_step<T, T>(op, nullptr, nullptr, (const T*)L.b, bufs[0], 0.0, L.c[0], c->stream,
                                               ev0, ev1));
            bytes = 2.0 * fbytes + cbytes;  // read b (and C for D), write x
        } else {
            const T* xp = (cheb && prev >= 0) ? bufs[prev] : nullptr;
            const int out = (cheb && prev >= 0) ? prev : other(cur);
            HIPCHK(c, launch_smooth_step<T, T>(op, bufs[cur], xp, (const T*)L.b, bufs[out], L.a[k], L.c[k],
                                               c->stream, ev0, ev1));
            bytes = (xp ? 4.0 : 3.0) * fbytes + cbytes;  // read x, [x_prev], b (, C); write out
            prev = cur;
            cur = out;
        }
        st = time_end(c, fine, kind, bytes);
        if (st != MG_OK) return st;
    }
    L.cur = cur;
    return MG_OK;
}

template <typename T>
mg_status coarse_level(mg_ctx* c, int l) {
    Level& L = c->lev[l];
    L.cur = 0;
    if (!c->var)
        HIPCHK(c, launch_coarse_flat<T>(L.n, c->Q, c->lam1, (const T*)L.b, (T*)L.x[0], c->stream));
    else
        HIPCHK(c, launch_coarse_dense<T>((int)L.N, c->G, (const T*)L.b, (T*)L.x[0], c->stream));
    return MG_OK;
}

// The pending outer sums as a job for the kernel about to be launched, which
// then finishes them; count 0 when none are pending.
SumsJob take_sums(mg_ctx* c) {
    if (!c->pending_sums) return SumsJob{};
    c->pending_sums = false;
    c->scal_flag = true;
    c->sums_seq += 1.0;
    return SumsJob{c->partials, c->nparts_outer, 3, c->dscal, 1, c->hscal, c->sums_seq};
}

// The variable-coefficient levels from l0 down in one workgroup.
template <typename T>
mg_status var_tail_cycle(mg_ctx* c, int l0) {
    VarTailArgs<T> a{};
    a.sums = take_sums(c);
    a.nlev = (int)c->lev.size() - l0;
    a.sched.cheb = c->p.smoother == MG_CHEBYSHEV ? 1 : 0;
    a.sched.steps = (int)c->lev[l0].a.size();
    for (int k = 0; k < a.nlev; ++k) {
        const Level& Lv = c->lev[l0 + k];
        a.n[k] = Lv.n;
        a.ih2[k] = Lv.ih2;
        a.C[k] = (const T*)Lv.coeff;
        for (int j = 0; j < a.sched.steps; ++j) {
            a.sched.a[k][j] = Lv.a[j];
            a.sched.c[k][j] = Lv.c[j];
        }
    }
    a.b = (const T*)c->lev[l0].b;
    a.x = (T*)c->lev[l0].x[0];
    a.G = c->G;
    HIPCHK(c, launch_var_tail<T>(a, c->stream));
    c->lev[l0].cur = 0;
    return MG_OK;
}

template <typename T>
mg_status tail_cycle(mg_ctx* c, int l0) {
    if (c->var) return var_tail_cycle<T>(c, l0);
    TailArgs<T> a{};
    const int L = (int)c->lev.size();
    a.nlev = L - l0;
    const bool cheb = c->p.smoother == MG_CHEBYSHEV;
    a.sched.cheb = cheb ? 1 : 0;
    a.sched.steps = (int)c->lev[l0].a.size();
    for (int k = 0; k < a.nlev; ++k) {
        const Level& Lv = c->lev[l0 + k];
        a.n[k] = Lv.n;
        a.ih2[k] = Lv.ih2;
        for (int j = 0; j < a.sched.steps; ++j) {
            a.sched.a[k][j] = Lv.a[j];
            a.sched.c[k][j] = Lv.c[j];
        }
    }
    a.b = (const T*)c->lev[l0].b;
    a.x = (T*)c->lev[l0].x[0];
    a.Q = c->Q;
    a.lam1 = c->lam1;
    a.sums = take_sums(c);
    HIPCHK(c, launch_tail<T>(a, c->stream));
    c->lev[l0].cur = 0;
    return MG_OK;
}

template <typename T>
mg_status vcycle_from_zero(mg_ctx* c, int l);

// r_{l+1} = R(b_l - M_l x_l) into level l+1's right-hand side; the buffer of
// the previous iterate is free here and serves as residual scratch.  cycle: a
// V-cycle on level l + 1 follows, whose first step may be formed here.
template <typename T>
mg_status residual_restrict_level(mg_ctx* c, int l, bool cycle = false) {
    Level& L = c->lev[l];
    Level& Lc = c->lev[l + 1];
    const bool fine = (l == 0);
    hipEvent_t ev0, ev1;
    mg_status st = time_events(c, fine, MG_TIME_TRANSFER, &ev0, &ev1);
    if (st != MG_OK) return st;
    FirstStep<T> first;
    if (cycle && first_step_level(c, l + 1)) {
        first.C = (const T*)Lc.coeff;
        first.x1 = (T*)Lc.x[0];
        first.c0 = Lc.c[0];
        Lc.x1 = true;
    }
    HIPCHK(c, launch_residual_restrict<T, T>(op_of<T>(L), (const T*)L.x[L.cur], (const T*)L.b, (T*)Lc.b,
                                             (T*)L.x[other(L.cur)], c->stream, ev0, ev1, first));
    // x, b [, C] read, r_{l+1} written; 19-point rows without the fused pass: the timed
    // one forms the fine residual (x, b, C read, r written) and a second one restricts it
    const double N = (double)L.N, s = sizeof(T);
    const double bytes = !c->var                         ? N * (2.0 + 1.0 / 8.0) * s
                         : var_rr_applies(L.n, sizeof(T)) ? N * (2.0 + 6.0 + 1.0 / 8.0) * s
                                                          : N * (3.0 + 6.0) * s;
    return time_end(c, fine, MG_TIME_TRANSFER, bytes);
}

// Up-leg of level l: x_l += P e_{l+1}, then the post-smoothing pass (one
// kernel for both where the prolongation is fused into the three-step pass).
template <typename T>
mg_status post_level(mg_ctx* c, int l) {
    Level& L = c->lev[l];
    Level& Lc = c->lev[l + 1];
    const bool fine = (l == 0);
    hipEvent_t ev0, ev1;
    mg_status st;
    if (post_fused(c, l, sizeof(T))) {  // prolongation and the three-step post-smoothing pass in one kernel
        if ((st = time_events(c, fine, MG_TIME_TRIPLE, &ev0, &ev1)) != MG_OK) return st;
        const double D = -6.0 * L.ih2;  // c / D rounded as in the single-step launch
        const int out = other(L.cur);
        HIPCHK(c, launch_prolong_triple_row<T>(L.n, L.ih2, (const T*)L.x[L.cur], (const T*)Lc.x[Lc.cur],
                                               (const T*)L.b, (T*)L.x[out], L.a[0], L.c[0] / D, L.a[1],
                                               L.c[1] / D, L.a[2], L.c[2] / D, c->stream, ev0, ev1));
        L.cur = out;
        // x, b read, x_3 written, e read once per coarse point
        return time_end(c, fine, MG_TIME_TRIPLE, (3.0 + 1.0 / 8.0) * (double)L.N * sizeof(T));
    }
    // the prolongation runs inside the pass's first pair or step
    if (post_pair_fused(c, l, sizeof(T)) || post_step_fused(c, l, sizeof(T)))
        return smooth_level<T>(c, l, false, (const T*)Lc.x[Lc.cur]);
    if ((st = time_events(c, fine, MG_TIME_TRANSFER, &ev0, &ev1)) != MG_OK) return st;
    HIPCHK(c, launch_prolong_add<T>(L.n, (const T*)Lc.x[Lc.cur], (T*)L.x[L.cur], c->stream, ev0, ev1));
    if ((st = time_end(c, fine, MG_TIME_TRANSFER, (2.0 + 1.0 / 8.0) * (double)L.N * sizeof(T))) != MG_OK) return st;
    return smooth_level<T>(c, l, false);
}

// The first step from zero of a 19-point visit level, where the kernel that
// wrote the right-hand side did not form it.
template <typename T>
mg_status ensure_first_step(mg_ctx* c, int l) {
    Level& L = c->lev[l];
    if (L.x1) return MG_OK;
    HIPCHK(c, launch_smooth_step<T, T>(op_of<T>(L), nullptr, nullptr, (const T*)L.b, (T*)L.x[0], 0.0, L.c[0],
                                       c->stream));
    L.x1 = true;
    return MG_OK;
}

// Down-leg of a 19-point visit level.
template <typename T>
mg_status var_visit_pre(mg_ctx* c, int l) {
    Level& L = c->lev[l];
    Level& Lc = c->lev[l + 1];
    int in = 0;
    if (l == 0 && c->x1_ready) {
        in = c->x1_buf;
        c->x1_ready = false;
    } else {
        const mg_status st = ensure_first_step<T>(c, l);
        if (st != MG_OK) return st;
    }
    L.x1 = false;
    const bool first = first_step_level(c, l + 1);
    const int out = other(in);
    HIPCHK(c, launch_var_visit_pre<T>(L.n, L.ih2, (const T*)L.coeff, (const T*)L.x[in], (const T*)L.b, (T*)L.x[out],
                                      (T*)Lc.b, (const T*)Lc.coeff, first ? (T*)Lc.x[0] : nullptr,
                                      Lc.c.empty() ? 0.0 : Lc.c[0], L.a.data(), L.c.data(), (int)L.a.size(),
                                      c->p.smoother == MG_CHEBYSHEV, c->stream));
    Lc.x1 = first;
    L.cur = out;
    return MG_OK;
}

// Capture V(0, b_1) on level 1 and below into c->coarse_exec.
template <typename T>
mg_status capture_coarse(mg_ctx* c) {
    if (!c->cap_stream) HIPCHK(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
    hipStream_t saved = c->stream;
    c->stream = c->cap_stream;
    c->capturing = true;
    HIPCHK(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal));
    mg_status st = vcycle_from_zero<T>(c, 1);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
    c->capturing = false;
    c->stream = saved;
    if (st != MG_OK) {
        if (e == hipSuccess && g) (void)hipGraphDestroy(g);
        return st;
    }
    HIPCHK(c, e);
    c->coarse_graph = g;
    HIPCHK(c, hipGraphInstantiate(&c->coarse_exec, g, nullptr, nullptr, 0));
    c->coarse_cur = c->lev[1].cur;
    return MG_OK;
}

// x_l = V(0, b_l)
template <typename T>
mg_status vcycle_from_zero(mg_ctx* c, int l) {
    const int last = (int)c->lev.size() - 1;
    if (l == 1 && last >= 2 && c->use_graph && !c->capturing) {
        if (first_step_level(c, 1)) {  // the captured cycle starts from the first step
            mg_status st = ensure_first_step<T>(c, 1);
            if (st != MG_OK) return st;
        }
        if (!c->coarse_exec) {
            mg_status st = capture_coarse<T>(c);
            if (st != MG_OK) return st;
        }
        HIPCHK(c, hipGraphLaunch(c->coarse_exec, c->stream));
        c->lev[1].cur = c->coarse_cur;
        c->lev[1].x1 = false;
        return MG_OK;
    }
    if (l == c->tail_start) return tail_cycle<T>(c, l);
    if (l == last) return coarse_level<T>(c, l);
    Level& L = c->lev[l];
    Level& Lc = c->lev[l + 1];
    mg_status st = MG_OK;
    const int v = (int)L.a.size();
    if (visit_level(c, l, true)) {  // one launch before the coarse level
        if (l == 0) c->x1_ready = false;
        HIPCHK(c, launch_visit_pre<T>(L.n, L.ih2, (const T*)L.b, (T*)L.x[0], (T*)Lc.b, L.a.data(), L.c.data(), v,
                                      c->stream));
        L.cur = 0;
    } else if (var_visit_level(c, l)) {
        if ((st = var_visit_pre<T>(c, l)) != MG_OK) return st;
    } else {
        if ((st = smooth_level<T>(c, l, true)) != MG_OK) return st;
        if ((st = residual_restrict_level<T>(c, l, true)) != MG_OK) return st;
    }
    if ((st = vcycle_from_zero<T>(c, l + 1)) != MG_OK) return st;
    if (visit_level(c, l, false)) {  // and one after it
        const int nx = other(L.cur);
        HIPCHK(c, launch_visit_post<T>(L.n, L.ih2, (const T*)L.x[L.cur], (const T*)Lc.x[Lc.cur], (const T*)L.b,
                                       (T*)L.x[nx], L.a.data(), L.c.data(), v, c->stream));
        L.cur = nx;
        return MG_OK;
    }
    if (var_visit_level(c, l)) {
        const int nx = other(L.cur);
        HIPCHK(c, launch_var_visit_post<T>(L.n, L.ih2, (const T*)L.coeff, (const T*)L.x[L.cur],
                                           (const T*)Lc.x[Lc.cur], (const T*)L.b, (T*)L.x[nx], L.a.data(),
                                           L.c.data(), v, c->p.smoother == MG_CHEBYSHEV, c->stream));
        L.cur = nx;
        return MG_OK;
    }
    return post_level<T>(c, l);
}

// ---- outer residual dispatch ---------------------------------------------------------------
// r = (b - mean b) - M phi (phi = phi_in + e when e != null); per-block r^2 sums into partials.
// The sum of b is in device slot 0 (device_sum).
// With next_cycle set, the kernel also writes the first smoothing step of the
// V-cycle that follows (x = c0 D^-1 r on level 0).
mg_status outer_residual(mg_ctx* c, const double* phi_in, const void* e, double* phi_out, const double* b,
                         bool next_cycle = false) {
    Level& L = c->lev[0];
    const int n = L.n;
    const double ih2 = L.ih2;
    const bool x1 = next_cycle && x1_fusable(c) && !from_zero_triple(c, 0) &&
                    !visit_level(c, 0, true);
    const double c0 = L.c.empty() ? 0.0 : L.c[0];
    // x1 goes to a buffer other than the one holding e (the previous cycle's result)
    const int xb = other(L.cur);
    hipEvent_t ev0, ev1;
    mg_status st = time_events(c, true, MG_TIME_OUTER, &ev0, &ev1);
    if (st != MG_OK) return st;
    hipError_t err;
    const Mean bmean{c->dscal, 1.0 / (double)L.N};  // the sum of b is in slot 0
    if (c->p.precision == MG_FP64) {
        OpDesc<double> op{n, ih2, (const double*)c->coeff_outer};
        err = launch_outer_residual<double, double, double, double>(op, phi_in, (const double*)e, phi_out, b, bmean,
                                                                    (double*)L.b, x1 ? (double*)L.x[xb] : nullptr, c0,
                                                                    c->partials, c->stream, ev0, ev1);
    } else if (c->p.precision == MG_MIXED) {
        float* x1p = x1 ? (float*)L.x[xb] : nullptr;
        if (c->coeff_outer_double) {
            OpDesc<double> op{n, ih2, (const double*)c->coeff_outer};
            err = launch_outer_residual<double, float, float, double>(op, phi_in, (const float*)e, phi_out, b, bmean,
                                                                      (float*)L.b, x1p, c0, c->partials, c->stream,
                                                                      ev0, ev1);
        } else {
            OpDesc<float> op{n, ih2, (const float*)c->coeff_outer};
            err = launch_outer_residual<double, float, float, float>(op, phi_in, (const float*)e, phi_out, b, bmean,
                                                                     (float*)L.b, x1p, c0, c->partials, c->stream,
                                                                     ev0, ev1);
        }
    } else {
        OpDesc<float> op{n, ih2, (const float*)c->coeff_outer};
        err = launch_outer_residual<float, float, float, float>(op, phi_in, (const float*)e, phi_out, b, bmean,
                                                                (float*)L.b, x1 ? (float*)L.x[xb] : nullptr, c0,
                                                                c->partials, c->stream, ev0, ev1);
    }
    HIPCHK(c, err);
    c->x1_ready = x1;
    c->x1_buf = xb;
    // phi (and e, phi_out) and b in their storage types, r (and x1) in the inner type, C once
    const double si = c->inner_double ? 8.0 : 4.0;
    const double sc = c->var ? 6.0 * (c->coeff_outer_double ? 8.0 : 4.0) : 0.0;
    const double per_pt = 8.0 + 8.0 + si + (e ? si + 8.0 : 0.0) + (x1 ? si : 0.0) + sc;
    return time_end(c, true, MG_TIME_OUTER, per_pt * (double)L.N);
}

mg_status read_scalars(mg_ctx* c, int count) {
    HIPCHK(c, hipMemcpyAsync(c->hscal, c->dscal, sizeof(double) * count, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return MG_OK;
}

mg_status inner_vcycle(mg_ctx* c) {
    return c->inner_double ? vcycle_from_zero<double>(c, 0) : vcycle_from_zero<float>(c, 0);
}

const void* inner_e(mg_ctx* c) { return c->lev[0].x[c->lev[0].cur]; }

mg_status check_ctx(mg_ctx* c) { return c ? MG_OK : MG_ERR_INVALID; }

template <typename F>
hipError_t with_op(mg_ctx* c, int level, F f) {
    const Level& L = c->lev[level];
    if (!c->var || c->inner_double) return f(OpDesc<double>{L.n, L.ih2, (const double*)L.coeff});
    return f(OpDesc<float>{L.n, L.ih2, (const float*)L.coeff});
}

}  // namespace

// =============================================================================================
// C ABI
// =============================================================================================
extern "C" {

const char* mg_status_string(mg_status s) {
    if ((int)s < 0 || (int)s > 6) return "unknown mg_status";
    return kStatus[(int)s];
}

const char* mg_last_error(const mg_ctx* ctx) { return ctx ? ctx->err.c_str() : ""; }

mg_status mg_params_default(mg_params* p, int n) {
    if (!p) return MG_ERR_INVALID;
    p->n = n;
    int lg = 0;
    while ((1 << lg) < n) ++lg;
    p->levels = lg - 1 > 1 ? lg - 1 : 1;
    p->cheb_degree = 3;
    p->cheb_alpha = 8.0;
    p->h = n > 0 ? 1.0 / n : 0.0;
    p->precision = MG_MIXED;
    p->smoother = MG_CHEBYSHEV;
    p->jacobi_omega = 2.0 / 3.0;
    p->jacobi_sweeps = 2;
    p->options = 0;
    return MG_OK;
}

mg_status mg_validate_params(const mg_params* p) {
    if (!p) return MG_ERR_INVALID;
    if (!is_pow2(p->n) || p->n < 8 || p->n > 2048) return MG_ERR_INVALID;
    if (p->levels < 1 || p->levels > 12) return MG_ERR_INVALID;
    const int nc = coarsest_n(*p);
    if (nc < 4 || nc > 16) return MG_ERR_INVALID;
    if (p->cheb_degree < 1 || p->cheb_degree > 8) return MG_ERR_INVALID;
    if (!(p->cheb_alpha > 1.0) || !std::isfinite(p->cheb_alpha)) return MG_ERR_INVALID;
    if (!(p->h > 0.0) || !std::isfinite(p->h)) return MG_ERR_INVALID;
    if (p->precision < MG_FP64 || p->precision > MG_FP32) return MG_ERR_INVALID;
    if (p->smoother != MG_CHEBYSHEV && p->smoother != MG_JACOBI) return MG_ERR_INVALID;
    if ((p->options & ~MG_OPT_ALL) != 0) return MG_ERR_INVALID;
    if (p->smoother == MG_JACOBI) {
        if (!(p->jacobi_omega > 0.0 && p->jacobi_omega < 2.0)) return MG_ERR_INVALID;
        if (p->jacobi_sweeps < 1 || p->jacobi_sweeps > 16) return MG_ERR_INVALID;
    }
    return MG_OK;
}

mg_status mg_destroy(mg_ctx* c) {
    if (!c) return MG_OK;
    if (c->stream && !c->other_streams) {
        (void)hipStreamSynchronize(c->stream);
    } else {  // the earlier streams may be gone by now: wait for the device
        int dev = c->device;
        (void)hipGetDevice(&dev);
        if (dev != c->device) (void)hipSetDevice(c->device);
        (void)hipDeviceSynchronize();
        if (dev != c->device) (void)hipSetDevice(dev);
    }
    dfree(c->mem);
    if (c->hscal) host_slots().back(c->hscal);
    dfree(c->scratch);
    dfree(c->pcg_r);
    dfree(c->pcg_p[0]);
    dfree(c->pcg_p[1]);
    dfree(c->pcg_q);
    dfree(c->pcg_s);
    dfree(c->pcg_partials);
    for (auto& e : c->events) {
        (void)hipEventDestroy(e.start);
        (void)hipEventDestroy(e.stop);
    }
    if (c->coarse_exec) (void)hipGraphExecDestroy(c->coarse_exec);
    if (c->coarse_graph) (void)hipGraphDestroy(c->coarse_graph);
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    if (c->norm_ev) (void)hipEventDestroy(c->norm_ev);
    delete c;
    return MG_OK;
}

}  // extern "C"

namespace {

// What the hierarchy is built from.
bool var_source(int source) { return source != MG_SOURCE_FLAT; }

// Device memory that only the setup uses.
struct SetupMem {
    double* c64[12] = {};  // coefficients of each level in double, where the level itself does not keep them
    double* psi[12] = {};  // restricted deformation potentials
    double* dense = nullptr;
};

// Places every field of the context in `keep` and every temporary of its
// setup in `tmp` (sizes only when their bases are null).
void layout(mg_ctx* c, int source, Arena& keep, Arena& tmp, SetupMem& sm) {
    const mg_params& p = c->p;
    const size_t Tsz = c->inner_double ? sizeof(double) : sizeof(float);
    c->lev.resize(p.levels);
    for (int l = 0; l < p.levels; ++l) {
        Level& L = c->lev[l];
        L.n = p.n >> l;
        L.N = (size_t)L.n * L.n * L.n;
        L.h = p.h * (double)(1 << l);
        L.ih2 = 1.0 / (L.h * L.h);
        L.x[0] = keep.take(L.N * Tsz);
        L.x[1] = keep.take(L.N * Tsz);
        const bool third =
            c->use_pairs && (c->var ? (var_pair_applies(L.n, Tsz) || var_pro_applies(L.n, Tsz)) &&
                                          p.smoother == MG_CHEBYSHEV && p.cheb_degree >= 2
                                    : pair_kernels_apply(L.n, Tsz));
        L.x[2] = third ? keep.take(L.N * Tsz) : nullptr;
        L.b = keep.take(L.N * Tsz);
        L.coeff = c->var ? keep.take(6 * L.N * Tsz) : nullptr;
    }
    const size_t N0 = c->lev[0].N;
    const int nc = c->lev.back().n;
    const size_t Nc = c->lev.back().N;
    c->phi_tmp = keep.doubles(N0);
    c->nparts = stencil_blocks(p.n);
    c->nparts_outer = outer_blocks(p.n, !c->var, p.precision != MG_FP32);
    // three arrays: the outer kernels write three partial sums per block
    c->partials = keep.doubles(3 * (size_t)(c->nparts > c->nparts_outer ? c->nparts : c->nparts_outer));
    c->dscal = keep.doubles(16);
    if (!c->var) {
        c->Q = keep.doubles((size_t)nc * nc);
        c->lam1 = keep.doubles(nc);
        return;
    }
    c->slots = (u64*)keep.take(kSetupSlots * sizeof(u64));
    c->G = keep.doubles(Nc * Nc);
    // the outer residual of a mixed solve uses the coefficients in double where they came in double
    c->coeff_outer_double = c->inner_double || (p.precision == MG_MIXED && source != MG_SOURCE_COEFF_F32);
    if (c->coeff_outer_double && !c->inner_double) c->coeff_outer = keep.take(6 * N0 * sizeof(double));
    else c->coeff_outer = c->lev[0].coeff;
    for (int l = 0; l < p.levels; ++l) {
        const size_t N = c->lev[l].N;
        if (c->inner_double) sm.c64[l] = (double*)c->lev[l].coeff;
        else if (l == 0 && c->coeff_outer_double) sm.c64[l] = (double*)c->coeff_outer;
        else if (l > 0 || source == MG_SOURCE_PSI || p.levels == 1) sm.c64[l] = tmp.doubles(6 * N);
        if (source == MG_SOURCE_PSI && l > 0) sm.psi[l] = tmp.doubles(N);
    }
    sm.dense = tmp.doubles(dense_work(nc));
}

// Coefficients of every level, their checks and bounds, the coarsest inverse:
// all enqueued, then one readback.
mg_status setup_var(mg_ctx* c, int source, const void* field, const SetupMem& sm) {
    const mg_params& p = c->p;
    hipStream_t s = c->stream;
    const int levels = p.levels;
    u64* lmax = c->slots;
    u64* bad = c->slots + 16;
    HIPCHK(c, launch_clear_slots(c->slots, kSetupSlots, s));
    auto inner_copy = [&](int l) { return c->inner_double ? nullptr : (float*)c->lev[l].coeff; };
    if (source == MG_SOURCE_PSI) {
        const double* psi = (const double*)field;
        for (int l = 0; l < levels; ++l) {
            const Level& L = c->lev[l];
            if (l > 0) {
                HIPCHK(c, launch_restrict_fields<double>(c->lev[l - 1].n, psi, sm.psi[l], nullptr, 1, s));
                psi = sm.psi[l];
            }
            HIPCHK(c, launch_geometry_fields(L.n, L.ih2, psi, sm.c64[l], inner_copy(l), nullptr, bad + l, s));
            if (l + 1 < levels) HIPCHK(c, launch_bound<double>(L.n, sm.c64[l], lmax + l, s));
        }
    } else {
        const Level& L0 = c->lev[0];
        // the double copy of level 0 that the outer residual (or a one-level hierarchy) needs
        double* outer = c->inner_double ? nullptr : sm.c64[0];
        auto from = [&](auto* src) -> hipError_t {
            typedef std::remove_const_t<std::remove_pointer_t<decltype(src)>> TS;
            hipError_t e = c->inner_double ? launch_coeff_copy<TS, double>(L0.N, src, (double*)L0.coeff, outer, bad, s)
                                           : launch_coeff_copy<TS, float>(L0.N, src, (float*)L0.coeff, outer, bad, s);
            if (levels == 1 || e != hipSuccess) return e;
            if ((e = launch_bound<TS>(L0.n, src, lmax, s)) != hipSuccess) return e;
            return launch_restrict_fields<TS>(L0.n, src, sm.c64[1], inner_copy(1), 6, s);
        };
        HIPCHK(c, source == MG_SOURCE_COEFF_F64 ? from((const double*)field) : from((const float*)field));
        for (int l = 1; l + 1 < levels; ++l) {
            HIPCHK(c, launch_bound<double>(c->lev[l].n, sm.c64[l], lmax + l, s));
            HIPCHK(c, launch_restrict_fields<double>(c->lev[l].n, sm.c64[l], sm.c64[l + 1], inner_copy(l + 1), 6, s));
        }
    }
    const Level& Lc = c->lev.back();
    HIPCHK(c, launch_dense_inverse(Lc.n, Lc.ih2, sm.c64[levels - 1], c->G, sm.dense, bad + 16, bad + 17, s));
    static_assert(16 + kSetupSlots <= kHostDoubles && sizeof(u64) == sizeof(double), "the slots fit the host mirror");
    u64* host = reinterpret_cast<u64*>(c->hscal + 16);
    HIPCHK(c, hipMemcpyAsync(host, c->slots, kSetupSlots * sizeof(u64), hipMemcpyDeviceToHost, s));
    HIPCHK(c, hipStreamSynchronize(s));
    for (int l = 0; l < levels; ++l) {
        if (host[16 + l] == 0) continue;
        const std::string cells = std::to_string((long long)host[16 + l]) + " cells ";
        return fail(c, MG_ERR_INVALID_COEFF,
                    source == MG_SOURCE_PSI
                        ? cells + "of level " + std::to_string(l) +
                              " with a folded mesh (non-finite or non-positive diagonal coefficients)"
                        : cells + "with non-finite or non-positive diagonal coefficients");
    }
    if (host[32] != 0 || host[33] != 0) {  // not definite (coefficients that are not): invert with pivoting
        std::vector<double> C(6 * Lc.N), M, G;
        HIPCHK(c, hipMemcpyAsync(C.data(), sm.c64[levels - 1], C.size() * sizeof(double), hipMemcpyDeviceToHost, s));
        HIPCHK(c, hipStreamSynchronize(s));
        assemble_dense(Lc.n, Lc.ih2, C, M);
        if (!pseudo_inverse((int)Lc.N, M, G))
            return fail(c, MG_ERR_INVALID_COEFF, "coarsest operator is singular beyond its constant null space");
        HIPCHK(c, hipMemcpyAsync(c->G, G.data(), G.size() * sizeof(double), hipMemcpyHostToDevice, s));
        HIPCHK(c, hipStreamSynchronize(s));
    }
    for (int l = 0; l + 1 < levels; ++l) std::memcpy(&c->lev[l].lmax, &host[l], sizeof(double));
    // levels of at most 16^3 points run in one kernel (coarsest 4^3, or 8^3 with enough steps)
    const int steps = p.smoother == MG_JACOBI ? p.jacobi_sweeps : p.cheb_degree;
    if (c->use_tail && steps <= kTailMaxSteps) {
        int l0 = levels - 1;
        while (l0 > 0 && c->lev[l0 - 1].n <= 16) --l0;
        if (var_tail_applies(c->lev[l0].n, Lc.n, levels - l0, l0, steps, c->inner_double ? sizeof(double) : sizeof(float)))
            c->tail_start = l0;
    }
    return MG_OK;
}

mg_status setup_flat(mg_ctx* c) {
    const mg_params& p = c->p;
    Level& Lc = c->lev.back();
    std::vector<double> Q, lam;
    flat_basis(Lc.n, Lc.h, Q, lam);
    HIPCHK(c, hipMemcpyAsync(c->Q, Q.data(), Q.size() * sizeof(double), hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipMemcpyAsync(c->lam1, lam.data(), lam.size() * sizeof(double), hipMemcpyHostToDevice, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    // levels of at most 16^3 points down to a coarsest of at most 8^3 run in one kernel
    const int steps = p.smoother == MG_JACOBI ? p.jacobi_sweeps : p.cheb_degree;
    if (Lc.n <= 8 && steps <= kTailMaxSteps && c->use_tail) {
        int l0 = p.levels - 1;
        while (l0 > 0 && c->lev[l0 - 1].n <= 16 && p.levels - (l0 - 1) <= kTailMaxLevels) --l0;
        if (p.levels - l0 >= 2) c->tail_start = l0;
    }
    return MG_OK;
}

// Parameters the context's memory depends on.
mg_status describe(mg_ctx* c, int source) {
    const mg_params& p = c->p;
    c->var = var_source(source);
    c->inner_double = p.precision == MG_FP64;
    if (c->var && coarsest_n(p) > 8)
        return fail(c, MG_ERR_INVALID, "variable-coefficient coarsest level must have at most 8^3 points");
    // reference switches of this context (mg_params.options)
    c->use_pairs = (p.options & MG_OPT_NO_PAIR) == 0;
    c->use_visits = (p.options & MG_OPT_NO_VISIT) == 0;
    c->fuse_sums = (p.options & MG_OPT_NO_FUSED_SUMS) == 0;
    c->use_tail = (p.options & MG_OPT_NO_TAIL) == 0;
    // replaying the coarse sub-cycle from a HIP graph measured slower than eager
    // launches on this platform; MG_OPT_GRAPH keeps it available
    c->use_graph = (p.options & MG_OPT_GRAPH) != 0;
    return MG_OK;
}

// keep / setup: the caller's memory, or null to allocate it here (one block
// for the context, one for its setup, freed before the return).
mg_status create_impl(mg_ctx* c, int source, const void* field, void* keep, size_t keep_bytes, void* setup,
                      size_t setup_bytes) {
    mg_status st = describe(c, source);
    if (st != MG_OK) return st;
    SetupMem sm;
    Arena need_keep{nullptr}, need_tmp{nullptr};
    layout(c, source, need_keep, need_tmp, sm);
    void* own_tmp = nullptr;
    if (keep) {
        if (keep_bytes < need_keep.used || setup_bytes < need_tmp.used || (need_tmp.used && !setup))
            return fail(c, MG_ERR_INVALID, "workspace too small");
    } else {
        if ((st = dalloc(c, &c->mem, need_keep.used)) != MG_OK) return st;
        keep = c->mem;
        if ((st = dalloc(c, &own_tmp, need_tmp.used)) != MG_OK) return st;
        setup = own_tmp;
    }
    Arena A{(char*)keep}, B{(char*)setup};
    layout(c, source, A, B, sm);
    const hipError_t e = (hipError_t)host_slots().take(&c->hscal);
    if (e != hipSuccess) {
        c->hscal = nullptr;
        st = fail(c, MG_ERR_HIP, std::string("pinned host memory: ") + hipGetErrorString(e));
    } else {
        c->hscal[kHostFlagSlot] = 0.0;
        c->hscal[kHostMeanSlot] = 0.0;
        st = c->var ? setup_var(c, source, field, sm) : setup_flat(c);
    }
    if (own_tmp) {
        (void)hipStreamSynchronize(c->stream);
        dfree(own_tmp);
    }
    if (st != MG_OK) return st;
    for (auto& L : c->lev) make_schedule(c->p, L);
    return MG_OK;
}

mg_status create(const mg_params* p, int source, const void* field, void* keep, size_t keep_bytes, void* setup,
                 size_t setup_bytes, void* stream, mg_ctx** out, const char* where) {
    mg_ctx* c = new (std::nothrow) mg_ctx();
    if (!c) return MG_ERR_NOMEM;
    c->p = *p;
    c->stream = (hipStream_t)stream;
    (void)hipGetDevice(&c->device);
    mg_status st;
    try {
        st = create_impl(c, source, field, keep, keep_bytes, setup, setup_bytes);
    } catch (const std::bad_alloc&) {
        st = MG_ERR_NOMEM;
    }
    if (st != MG_OK) {
        std::fprintf(stderr, "%s: %s\n", where, c->err.c_str());
        mg_destroy(c);
        return st;
    }
    *out = c;
    return MG_OK;
}

bool valid_source(int source) { return source >= MG_SOURCE_FLAT && source <= MG_SOURCE_PSI; }

}  // namespace

extern "C" {

mg_status mg_create(const mg_params* p, const void* coeff, int coeff_dtype, void* stream, mg_ctx** out) {
    if (!out) return MG_ERR_INVALID;
    *out = nullptr;
    if (mg_validate_params(p) != MG_OK) return MG_ERR_INVALID;
    if (coeff && coeff_dtype != MG_DTYPE_F32 && coeff_dtype != MG_DTYPE_F64) return MG_ERR_INVALID;
    const int source = !coeff                          ? MG_SOURCE_FLAT
                       : coeff_dtype == MG_DTYPE_F32 ? MG_SOURCE_COEFF_F32
                                                       : MG_SOURCE_COEFF_F64;
    return create(p, source, coeff, nullptr, 0, nullptr, 0, stream, out, "mg_create");
}

mg_status mg_create_psi(const mg_params* p, const double* psi, void* stream, mg_ctx** out) {
    if (!out) return MG_ERR_INVALID;
    *out = nullptr;
    if (!psi || mg_validate_params(p) != MG_OK) return MG_ERR_INVALID;
    return create(p, MG_SOURCE_PSI, psi, nullptr, 0, nullptr, 0, stream, out, "mg_create_psi");
}

mg_status mg_workspace_bytes(const mg_params* p, int source, size_t* keep_bytes, size_t* setup_bytes) {
    if (!keep_bytes || !setup_bytes || !valid_source(source) || mg_validate_params(p) != MG_OK) return MG_ERR_INVALID;
    try {
        mg_ctx c;
        c.p = *p;
        const mg_status st = describe(&c, source);
        if (st != MG_OK) return st;
        SetupMem sm;
        Arena A{nullptr}, B{nullptr};
        layout(&c, source, A, B, sm);
        *keep_bytes = A.used;
        *setup_bytes = B.used;
    } catch (const std::bad_alloc&) {
        return MG_ERR_NOMEM;
    }
    return MG_OK;
}

mg_status mg_create_in(const mg_params* p, int source, const void* field, void* keep, size_t keep_bytes, void* setup,
                       size_t setup_bytes, void* stream, mg_ctx** out) {
    if (!out) return MG_ERR_INVALID;
    *out = nullptr;
    if (!valid_source(source) || mg_validate_params(p) != MG_OK || !keep || ((uintptr_t)keep & 15) != 0 ||
        ((uintptr_t)setup & 15) != 0 || var_source(source) != (field != nullptr))
        return MG_ERR_INVALID;
    return create(p, source, field, keep, keep_bytes, setup, setup_bytes, stream, out, "mg_create_in");
}

mg_status mg_set_stream(mg_ctx* c, void* stream) {
    if (!c) return MG_ERR_INVALID;
    if (c->stream != (hipStream_t)stream) c->other_streams = true;
    c->stream = (hipStream_t)stream;
    return MG_OK;
}

// sum of (u - shift)^pw into dscal[slot]; to_host: also into the host mirror,
// for wait_mean
static mg_status device_sum(mg_ctx* c, const double* u, double shift, int pw, int slot, bool to_host = false) {
    HIPCHK(c, launch_block_sums(c->p.n, u, shift, pw, c->partials, c->stream));
    if (to_host) c->mean_seq += 1.0;
    HIPCHK(c, launch_finalize_sum(c->partials, c->nparts, c->dscal, slot, c->stream, to_host ? c->hscal : nullptr,
                                  c->mean_seq));
    return MG_OK;
}

// Readback of device scalars through an event, so the host can enqueue more
// work before it waits for the values.
static mg_status post_scalars(mg_ctx* c, int count) {
    HIPCHK(c, hipMemcpyAsync(c->hscal, c->dscal, sizeof(double) * count, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipEventRecord(c->norm_ev, c->stream));
    c->scal_flag = false;
    return MG_OK;
}
// The three outer sums (slots 1..3), finalized straight into the pinned host
// mirror as well; its flag slot marks when the host may read them.
static mg_status post_outer_sums(mg_ctx* c) {
    c->sums_seq += 1.0;
    c->scal_flag = true;
    HIPCHK(c, launch_finalize_sums(c->partials, c->nparts_outer, 3, c->dscal, 1, c->stream, c->hscal, c->sums_seq));
    return MG_OK;
}
// Level 0's inner V-cycle starts with the pass-from-zero kernel, which can
// finish the outer sums in an extra block.
static bool sums_in_pass_from_zero(const mg_ctx* c) {
    return c->fuse_sums && c->lev.size() > 1 && c->tail_start != 0 && !visit_level(c, 0, true) &&
           from_zero_triple(c, 0);
}
// The single-workgroup tail of the V-cycle that follows can finish them in a
// second block (not inside a captured graph, whose arguments are fixed).  The
// host gets them in the middle of the cycle, with the up-leg still to run
// while it enqueues the next one; a launch of their own took 6 us a cycle and
// its event another 5.
static bool sums_in_tail(const mg_ctx* c) {
    return c->fuse_sums && c->tail_start >= 0 && (!c->use_graph || c->tail_start == 0);
}
// Outer residual of the solve loop and its three sums.  When a V-cycle is
// enqueued right after it (cycle_follows) and has a kernel that can finish
// them (the pass from zero, or the tail), the sums are left pending for it;
// flush_sums finishes them otherwise.
static mg_status outer_with_sums(mg_ctx* c, const double* phi_in, const void* e, double* phi_out, const double* b,
                                 bool cycle_follows) {
    mg_status st = outer_residual(c, phi_in, e, phi_out, b, true);
    if (st != MG_OK) return st;
    if (cycle_follows && (sums_in_pass_from_zero(c) || sums_in_tail(c))) {
        c->pending_sums = true;
        return MG_OK;
    }
    return post_outer_sums(c);
}
static mg_status flush_sums(mg_ctx* c) {
    if (!c->pending_sums) return MG_OK;
    c->pending_sums = false;
    return post_outer_sums(c);
}
// Waits until slot of the pinned mirror holds seq.  The slot is polled; only
// after 50 ms of waiting is the stream asked whether it still runs: a stream
// query enqueues a marker, which costs a 5.8 us stall in front of the next
// kernel.
static mg_status poll_host(mg_ctx* c, int slot, double seq) {
    const volatile double* flag = c->hscal + slot;
    auto last = std::chrono::steady_clock::now();
    for (unsigned i = 1;; ++i) {
        if (*flag == seq) break;
        if ((i & 4095) != 0) continue;
        const auto now = std::chrono::steady_clock::now();
        if (now - last < std::chrono::milliseconds(50)) continue;
        last = now;
        const hipError_t e = hipStreamQuery(c->stream);
        if (e != hipSuccess && e != hipErrorNotReady) HIPCHK(c, e);
        if (e == hipSuccess && *flag != seq) return fail(c, MG_ERR_HIP, "host flag not raised");
    }
    std::atomic_thread_fence(std::memory_order_acquire);
    return MG_OK;
}
static mg_status wait_scalars(mg_ctx* c) {
    if (!c->scal_flag) {
        HIPCHK(c, hipEventSynchronize(c->norm_ev));
        return MG_OK;
    }
    c->scal_flag = false;
    return poll_host(c, kHostFlagSlot, c->sums_seq);
}
// the sum of b (device_sum with to_host) in hscal[0]
static mg_status wait_mean(mg_ctx* c) { return poll_host(c, kHostMeanSlot, c->mean_seq); }

static mg_status solve_impl(mg_ctx* c, double* phi, const double* b, double tol, int max_cycles,
                            mg_solve_info* info) {
    const size_t N0 = c->lev[0].N;
    const double invN = 1.0 / (double)N0;
    mg_status st;
    // the outer kernels read the sum of b on the device; the host checks it
    // with the first norms, before anything is written to phi
    if ((st = device_sum(c, b, 0.0, 1, 0, true)) != MG_OK) return st;
    // the outer kernel also sums (b - bmean)^2 (slot 1) and phi (slot 3) beside r^2 (slot 2)
    // Look-ahead: the next V-cycle depends only on device data (the residual
    // just formed), so it is enqueued before the host waits for the norm; it
    // is skipped when the measured contraction predicts convergence.  A
    // look-ahead cycle that turns out unneeded only wrote hierarchy buffers.
    c->pending_sums = false;
    bool ahead = max_cycles > 0;
    if ((st = outer_with_sums(c, phi, nullptr, nullptr, b, ahead)) != MG_OK) return st;
    if (ahead && (st = inner_vcycle(c)) != MG_OK) return st;
    if ((st = flush_sums(c)) != MG_OK) return st;
    if ((st = wait_mean(c)) != MG_OK) return st;
    if (!std::isfinite(c->hscal[0] * invN)) {
        (void)hipStreamSynchronize(c->stream);
        c->x1_ready = false;
        return fail(c, MG_ERR_NONFINITE, "source contains NaN or Inf");
    }
    if ((st = wait_scalars(c)) != MG_OK) return st;
    const double nb = std::sqrt(c->hscal[1]);
    if (info) {
        info->cycles = 0;
        info->rel_res0 = info->rel_res = 0.0;
    }
    if (nb == 0.0) {
        HIPCHK(c, launch_fill<double>(N0, 0.0, phi, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        c->x1_ready = false;
        if (info && info->history && info->history_cap > 0) info->history[0] = 0.0;
        return MG_OK;
    }
    double rel = std::sqrt(c->hscal[2]) / nb;
    if (!std::isfinite(rel)) {
        (void)hipStreamSynchronize(c->stream);
        c->x1_ready = false;
        return fail(c, MG_ERR_NONFINITE, "initial residual is not finite (NaN/Inf in phi?)");
    }
    if (info) {
        info->rel_res0 = rel;
        if (info->history && info->history_cap > 0) info->history[0] = rel;
    }
    double* cur = phi;
    double* other = c->phi_tmp;
    int cycles = 0;
    double prev1 = INFINITY, prev2 = INFINITY;
    double rho = 0.3;  // running estimate of the per-cycle residual reduction
    mg_status result = MG_OK;
    while (rel > tol && cycles < max_cycles) {
        if (!ahead && (st = inner_vcycle(c)) != MG_OK) return st;
        ahead = cycles + 1 < max_cycles && rho * rel > tol;
        if ((st = outer_with_sums(c, cur, inner_e(c), other, b, ahead)) != MG_OK) return st;
        std::swap(cur, other);
        if (ahead && (st = inner_vcycle(c)) != MG_OK) return st;
        if ((st = flush_sums(c)) != MG_OK) return st;
        if ((st = wait_scalars(c)) != MG_OK) return st;
        prev2 = prev1;
        prev1 = rel;
        rel = std::sqrt(c->hscal[2]) / nb;
        ++cycles;
        if (prev1 > 0.0 && std::isfinite(rel)) rho = std::min(1.0, std::max(1e-3, rel / prev1));
        if (info && info->history && cycles < info->history_cap) info->history[cycles] = rel;
        if (!std::isfinite(rel)) {
            result = fail(c, MG_ERR_NONFINITE, "residual became non-finite");
            break;
        }
        // stagnation at the rounding floor: no decrease over two consecutive cycles
        if (rel >= 0.999 * prev1 && prev1 >= 0.999 * prev2) break;
    }
    if (result == MG_OK && rel > tol) {
        result = MG_ERR_NOT_CONVERGED;
        c->err = "relative residual " + std::to_string(rel) + " > tol after " + std::to_string(cycles) + " cycles";
    }
    c->x1_ready = false;
    // gauge: phi <- cur - mean(cur); the sum of cur came with the last norm
    HIPCHK(c, launch_shift(N0, cur, c->hscal[3] * invN, phi, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (info) {
        info->cycles = cycles;
        info->rel_res = rel;
    }
    return result;
}

mg_status mg_solve(mg_ctx* c, double* phi, const double* b, double tol, int max_cycles, mg_solve_info* info) {
    if (!c || !phi || !b || max_cycles < 0 || !(tol >= 0.0)) return fail(c, MG_ERR_INVALID, "invalid solve arguments");
    if (phi == b) return fail(c, MG_ERR_INVALID, "phi and b must not alias");
    return solve_impl(c, phi, b, tol, max_cycles, info);
}

mg_status mg_solve_adjoint(mg_ctx* c, double* lam, const double* phibar, double tol, int max_cycles,
                           mg_solve_info* info) {
    if (!c || !lam || !phibar || max_cycles < 0 || !(tol >= 0.0))
        return fail(c, MG_ERR_INVALID, "invalid adjoint-solve arguments");
    if (lam == phibar) return fail(c, MG_ERR_INVALID, "lam and phibar must not alias");
    // M = M^T: the adjoint system is the forward system with the cotangent as source.
    return solve_impl(c, lam, phibar, tol, max_cycles, info);
}

// A fixed number of defect-correction cycles with no host wait between them:
// every outer kernel is followed by the next inner V-cycle at once, and the
// outer sums are read once, after the last update.
mg_status mg_cycles(mg_ctx* c, double* phi, const double* b, int cycles, double* rel_res_out) {
    if (!c || !phi || !b || cycles < 0) return fail(c, MG_ERR_INVALID, "invalid cycles arguments");
    if (phi == b) return fail(c, MG_ERR_INVALID, "phi and b must not alias");
    const size_t N0 = c->lev[0].N;
    const double invN = 1.0 / (double)N0;
    mg_status st;
    if ((st = device_sum(c, b, 0.0, 1, 0, true)) != MG_OK) return st;
    c->pending_sums = false;
    double* cur = phi;
    double* other = c->phi_tmp;
    for (int k = 0; k <= cycles; ++k) {
        // the last cycle's norms only are read: the others are not finished at all
        const bool follows = k < cycles;
        if (k == 0) st = outer_residual(c, phi, nullptr, nullptr, b, true);
        else st = outer_residual(c, cur, inner_e(c), other, b, true);
        if (st != MG_OK) return st;
        if (k > 0) std::swap(cur, other);
        if (follows && (st = inner_vcycle(c)) != MG_OK) return st;
        // the mean of b, before phi is overwritten; the first cycle is running
        if (k == 0) {
            if ((st = wait_mean(c)) != MG_OK) return st;
            if (!std::isfinite(c->hscal[0] * invN)) {
                (void)hipStreamSynchronize(c->stream);
                c->x1_ready = false;
                return fail(c, MG_ERR_NONFINITE, "source contains NaN or Inf");
            }
        }
    }
    if ((st = post_outer_sums(c)) != MG_OK) return st;
    c->scal_flag = false;
    // gauge from the sums on the device, so that one wait serves it and the norms
    HIPCHK(c, launch_gauge(N0, cur, c->dscal, invN, phi, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->x1_ready = false;
    const double nb = std::sqrt(c->hscal[1]);
    const double rel = nb > 0.0 ? std::sqrt(c->hscal[2]) / nb : 0.0;
    if (rel_res_out) *rel_res_out = rel;
    if (!std::isfinite(rel)) return fail(c, MG_ERR_NONFINITE, "residual is not finite");
    return MG_OK;
}

}  // extern "C"

namespace {

// The seven-point passes on rows form q = M p where they use it, and a double
// hierarchy's right-hand side serves as r.
inline bool pcg_rows(const mg_ctx* c) { return !c->var && pcg_row_applies(c->lev[0].n); }

mg_status ensure_pcg(mg_ctx* c) {
    if (!c->norm_ev) HIPCHK(c, hipEventCreateWithFlags(&c->norm_ev, hipEventDisableTiming));
    const int n = c->lev[0].n;
    const size_t bytes = c->lev[0].N * sizeof(double);
    const size_t parts = pcg_rows(c) ? 3 * (size_t)pcg_row_blocks(n) : 2 * (size_t)pcg_blocks(n);
    mg_status st = MG_OK;
    auto need = [&](double*& p, size_t size) {
        if (st == MG_OK && !p) st = dalloc(c, (void**)&p, size);
    };
    if (!c->inner_double) need(c->pcg_r, bytes);
    need(c->pcg_p[0], bytes);
    need(c->pcg_p[1], bytes);
    if (!pcg_rows(c)) need(c->pcg_q, bytes);
    need(c->pcg_s, kPcgSlots * sizeof(double));
    need(c->pcg_partials, parts * sizeof(double));
    return st;
}

// Multigrid-preconditioned CG.  TI: type of the hierarchy (preconditioner
// input r_in = level 0's right-hand side, output z = level 0's iterate);
// TC: type of the fine coefficients used for q = M p.
template <typename TI, typename TC>
mg_status pcg_impl(mg_ctx* c, double* phi, const double* b, double tol, int max_iter, mg_solve_info* info) {
    Level& L0 = c->lev[0];
    const int n = L0.n;
    const size_t N0 = L0.N;
    const double invN = 1.0 / (double)N0;
    const OpDesc<TC> op{n, L0.ih2, (const TC*)c->coeff_outer};
    TI* rin = (TI*)L0.b;
    double* r = c->inner_double ? (double*)L0.b : c->pcg_r;
    double* q = c->pcg_q;
    double* S = c->pcg_s;
    double* part = c->pcg_partials;
    const bool rows = pcg_rows(c);
    const int nb = rows ? pcg_row_blocks(n) : pcg_blocks(n);
    mg_status st;
    c->x1_ready = false;
    c->pending_sums = false;
    if ((st = device_sum(c, b, 0.0, 1, 0, true)) != MG_OK) return st;
    double bmean = 0.0;
    if (!rows) {  // the row passes read the sum on the device
        if ((st = wait_mean(c)) != MG_OK) return st;
        bmean = c->hscal[0] * invN;
        if (!std::isfinite(bmean)) return fail(c, MG_ERR_NONFINITE, "source contains NaN or Inf");
        if ((st = device_sum(c, b, bmean, 2, 1)) != MG_OK) return st;
    }
    // r, r_in and the sums of slots 1 .. 3 on their way to the host (slot 3, of phi, from the row passes)
    auto true_residual = [&]() -> mg_status {
        if (rows) {
            HIPCHK(c, launch_pcg_row_residual<TI>(n, L0.ih2, phi, b, Mean{c->dscal, invN}, r, rin, part, c->stream));
            c->sums_seq += 1.0;
            c->scal_flag = true;
            HIPCHK(c, launch_finalize_sums(part, nb, 3, c->dscal, 1, c->stream, c->hscal, c->sums_seq));
            return MG_OK;
        }
        HIPCHK(c, (launch_pcg_residual<TI, TC>(op, phi, b, bmean, r, rin, part, c->stream)));
        HIPCHK(c, launch_finalize_sum(part, nb, c->dscal, 2, c->stream));
        return post_scalars(c, 3);
    };
    if ((st = true_residual()) != MG_OK) return st;
    bool ahead = max_iter > 0;  // look-ahead preconditioner application, as in the defect-correction loop
    if (ahead && (st = inner_vcycle(c)) != MG_OK) return st;
    if (rows) {
        if ((st = wait_mean(c)) != MG_OK) return st;
        if (!std::isfinite(c->hscal[0] * invN)) {
            (void)hipStreamSynchronize(c->stream);
            return fail(c, MG_ERR_NONFINITE, "source contains NaN or Inf");
        }
    }
    if ((st = wait_scalars(c)) != MG_OK) return st;
    const double nbn = std::sqrt(c->hscal[1]);
    if (info) {
        info->cycles = 0;
        info->rel_res0 = info->rel_res = 0.0;
    }
    if (nbn == 0.0) {
        HIPCHK(c, launch_fill<double>(N0, 0.0, phi, c->stream));
        HIPCHK(c, hipStreamSynchronize(c->stream));
        if (info && info->history && info->history_cap > 0) info->history[0] = 0.0;
        return MG_OK;
    }
    double rel = std::sqrt(c->hscal[2]) / nbn;
    if (!std::isfinite(rel)) {
        (void)hipStreamSynchronize(c->stream);
        return fail(c, MG_ERR_NONFINITE, "initial residual is not finite (NaN/Inf in phi?)");
    }
    if (info) {
        info->rel_res0 = rel;
        if (info->history && info->history_cap > 0) info->history[0] = rel;
    }
    int its = 0, pc = 0;
    bool restart = true;
    double rho = 0.3, last_true = rel, true_rel = rel;
    bool true_current = true;  // true_rel belongs to the current iterate
    mg_status result = MG_OK;
    while (rel > tol && its < max_iter) {
        if (!ahead && (st = inner_vcycle(c)) != MG_OK) return st;
        const TI* z = (const TI*)inner_e(c);
        double* p_old = c->pcg_p[pc];
        double* p_new = c->pcg_p[1 - pc];
        if (rows) {
            const double* p_prev = restart ? nullptr : p_old;
            HIPCHK(c, launch_pcg_row_dots<TI>(n, L0.ih2, r, z, p_prev, part, c->stream));
            HIPCHK(c, launch_pcg_scalars(part, nb, S, kPcgBeta, restart, c->stream));
            HIPCHK(c, launch_pcg_row_direction<TI>(n, L0.ih2, z, p_prev, p_new, S, part, c->stream));
            HIPCHK(c, launch_pcg_scalars(part, nb, S, kPcgAlpha, false, c->stream));
            HIPCHK(c, launch_pcg_row_update<TI>(n, L0.ih2, phi, p_new, r, rin, S, part, c->stream));
        } else {
            HIPCHK(c, launch_pcg_dots<TI>(n, r, z, restart ? nullptr : q, part, c->stream));
            HIPCHK(c, launch_pcg_scalars(part, nb, S, kPcgBeta, restart, c->stream));
            HIPCHK(c, (launch_pcg_direction<TI, TC>(op, z, p_old, p_new, q, S, restart, part, c->stream)));
            HIPCHK(c, launch_pcg_scalars(part, nb, S, kPcgAlpha, false, c->stream));
            HIPCHK(c, launch_pcg_update<TI>(n, phi, p_new, r, q, rin, S, part, c->stream));
        }
        c->sums_seq += 1.0;
        c->scal_flag = true;
        HIPCHK(c, launch_finalize_sums(part, nb, 1, S, kPcgRr, c->stream, c->hscal, c->sums_seq));
        pc = 1 - pc;
        restart = false;
        true_current = false;
        ahead = its + 1 < max_iter && rho * rel > tol;
        if (ahead && (st = inner_vcycle(c)) != MG_OK) return st;
        if ((st = wait_scalars(c)) != MG_OK) return st;
        const double prev = rel;
        rel = std::sqrt(c->hscal[kPcgRr]) / nbn;
        ++its;
        if (prev > 0.0 && std::isfinite(rel)) rho = std::min(1.0, std::max(1e-3, rel / prev));
        if (info && info->history && its < info->history_cap) info->history[its] = rel;
        if (!std::isfinite(rel)) {
            result = fail(c, MG_ERR_NONFINITE, "residual became non-finite");
            break;
        }
        if (rel <= tol) {
            // the recursive residual met tol: confirm with the true residual
            if ((st = true_residual()) != MG_OK) return st;
            if ((st = wait_scalars(c)) != MG_OK) return st;
            true_rel = std::sqrt(c->hscal[2]) / nbn;
            true_current = true;
            if (true_rel > tol && its < max_iter) {
                if (true_rel >= 0.999 * last_true) {  // no progress since the last restart: rounding floor
                    rel = true_rel;
                    break;
                }
                last_true = true_rel;
                rel = true_rel;
                if (info && info->history && its < info->history_cap) info->history[its] = rel;
                restart = true;  // r and r_in now hold the true residual
                ahead = false;
            }
        }
    }
    if (!true_current && result == MG_OK) {
        if ((st = true_residual()) != MG_OK) return st;
        if ((st = wait_scalars(c)) != MG_OK) return st;
        true_rel = std::sqrt(c->hscal[2]) / nbn;
    }
    if (result == MG_OK && true_rel > tol) {
        result = MG_ERR_NOT_CONVERGED;
        c->err = "relative residual " + std::to_string(true_rel) + " > tol after " + std::to_string(its) +
                 " iterations";
    }
    // gauge: phi <- phi - mean(phi), from the sum on the device
    if (!rows || (!true_current && result != MG_OK)) {
        if ((st = device_sum(c, phi, 0.0, 1, 3)) != MG_OK) return st;
    }
    HIPCHK(c, launch_gauge(N0, phi, c->dscal, invN, phi, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (info) {
        info->cycles = its;
        info->rel_res = true_rel;
    }
    return result;
}

}  // namespace

extern "C" {

mg_status mg_solve_pcg(mg_ctx* c, double* phi, const double* b, double tol, int max_iter, mg_solve_info* info) {
    if (!c || !phi || !b || max_iter < 0 || !(tol >= 0.0)) return fail(c, MG_ERR_INVALID, "invalid solve arguments");
    if (phi == b) return fail(c, MG_ERR_INVALID, "phi and b must not alias");
    mg_status st;
    if ((st = ensure_pcg(c)) != MG_OK) return st;
    const bool cd = !c->var || c->coeff_outer_double;
    if (c->inner_double) return cd ? pcg_impl<double, double>(c, phi, b, tol, max_iter, info)
                                   : pcg_impl<double, float>(c, phi, b, tol, max_iter, info);
    return cd ? pcg_impl<float, double>(c, phi, b, tol, max_iter, info)
              : pcg_impl<float, float>(c, phi, b, tol, max_iter, info);
}

mg_status mg_predict(int n, int kind, const double* phi1, const double* phi2, const double* phi3, double growth,
                     double* out, void* stream) {
    if (!is_pow2(n) || n < 4 || n > 2048 || !phi1 || !out) return MG_ERR_INVALID;
    double c1, c2 = 0.0, c3 = 0.0;
    switch (kind) {
        case MG_PREDICT_RECYCLE: c1 = 1.0; break;
        case MG_PREDICT_GROWTH:
            if (!std::isfinite(growth)) return MG_ERR_INVALID;
            c1 = growth;
            break;
        case MG_PREDICT_LINEAR:
            if (!phi2) return MG_ERR_INVALID;
            c1 = 2.0; c2 = -1.0;
            break;
        case MG_PREDICT_QUADRATIC:
            if (!phi2 || !phi3) return MG_ERR_INVALID;
            c1 = 3.0; c2 = -3.0; c3 = 1.0;
            break;
        default: return MG_ERR_INVALID;
    }
    const size_t N = (size_t)n * n * n;
    return launch_combine3(N, c1, phi1, c2, phi2, c3, phi3, out, (hipStream_t)stream) == hipSuccess ? MG_OK
                                                                                                   : MG_ERR_HIP;
}

mg_status mg_accel(int n, double h, const double* phi, const double* psi, double scale, void* a_out, int dtype,
                   void* stream) {
    if (!is_pow2(n) || n < 4 || n > 2048 || !(h > 0) || !phi || !a_out || !std::isfinite(scale))
        return MG_ERR_INVALID;
    hipError_t e;
    if (dtype == MG_DTYPE_F64) e = launch_accel<double>(n, h, phi, psi, scale, (double*)a_out, (hipStream_t)stream);
    else if (dtype == MG_DTYPE_F32) e = launch_accel<float>(n, h, phi, psi, scale, (float*)a_out, (hipStream_t)stream);
    else return MG_ERR_INVALID;
    return e == hipSuccess ? MG_OK : MG_ERR_HIP;
}

mg_status mg_vcycle(mg_ctx* c, double* phi, const double* b, double* rel_res_out) {
    if (!c || !phi || !b) return fail(c, MG_ERR_INVALID, "invalid vcycle arguments");
    if (phi == b) return fail(c, MG_ERR_INVALID, "phi and b must not alias");
    const size_t N0 = c->lev[0].N;
    const double invN = 1.0 / (double)N0;
    mg_status st;
    c->pending_sums = false;
    if ((st = device_sum(c, b, 0.0, 1, 0)) != MG_OK) return st;
    if ((st = outer_residual(c, phi, nullptr, nullptr, b, true)) != MG_OK) return st;
    if ((st = inner_vcycle(c)) != MG_OK) return st;
    const void* e = inner_e(c);
    if (c->inner_double) HIPCHK(c, launch_add<double>(N0, phi, (const double*)e, phi, c->stream));
    else HIPCHK(c, launch_add<float>(N0, phi, (const float*)e, phi, c->stream));
    if (rel_res_out) {
        if ((st = outer_residual(c, phi, nullptr, nullptr, b)) != MG_OK) return st;
        HIPCHK(c, launch_finalize_sums(c->partials, c->nparts_outer, 3, c->dscal, 1, c->stream));
        if ((st = read_scalars(c, 3)) != MG_OK) return st;
        const double nb = std::sqrt(c->hscal[1]);
        *rel_res_out = nb > 0 ? std::sqrt(c->hscal[2]) / nb : 0.0;
    }
    return MG_OK;
}

mg_status mg_coeff_grad(mg_ctx* c, const double* lam, const double* phi, void* cbar, int cbar_dtype) {
    if (!c || !lam || !phi || !cbar) return fail(c, MG_ERR_INVALID, "invalid coeff_grad arguments");
    if (!c->var) return fail(c, MG_ERR_INVALID, "coefficient gradient needs a variable-coefficient context");
    const Level& L = c->lev[0];
    if (cbar_dtype == MG_DTYPE_F64)
        HIPCHK(c, launch_coeff_grad<double>(L.n, L.ih2, lam, phi, (double*)cbar, c->stream));
    else if (cbar_dtype == MG_DTYPE_F32)
        HIPCHK(c, launch_coeff_grad<float>(L.n, L.ih2, lam, phi, (float*)cbar, c->stream));
    else
        return fail(c, MG_ERR_INVALID, "cbar_dtype must be MG_DTYPE_F32 or MG_DTYPE_F64");
    return MG_OK;
}

mg_status mg_geometry(int n, double h, const double* psi, void* C_out, int dtype, double* sqrtg_out, void* stream) {
    if (!is_pow2(n) || n < 4 || n > 2048 || !(h > 0) || !psi || !C_out) return MG_ERR_INVALID;
    const double ih2 = 1.0 / (h * h);
    hipError_t e;
    hipStream_t s = (hipStream_t)stream;
    if (dtype == MG_DTYPE_F64)
        e = launch_geometry_fields(n, ih2, psi, (double*)C_out, nullptr, sqrtg_out, nullptr, s);
    else if (dtype == MG_DTYPE_F32)
        e = launch_geometry_fields(n, ih2, psi, nullptr, (float*)C_out, sqrtg_out, nullptr, s);
    else
        return MG_ERR_INVALID;
    return e == hipSuccess ? MG_OK : MG_ERR_HIP;
}

mg_status mg_geometry_bwd(int n, double h, const double* psi, const double* Cbar, const double* sqrtgbar,
                          double* psibar, void* stream) {
    if (!is_pow2(n) || n < 4 || n > 2048 || !(h > 0) || !psi || !Cbar || !psibar) return MG_ERR_INVALID;
    const double ih2 = 1.0 / (h * h);
    const size_t N = (size_t)n * n * n;
    hipStream_t s = (hipStream_t)stream;
    if (!geometry_bwd_overlaps(N, psi, Cbar, sqrtgbar, psibar))
        return launch_geometry_bwd(n, ih2, psi, Cbar, sqrtgbar, psibar, s) == hipSuccess ? MG_OK : MG_ERR_HIP;
    // the result replaces an input that other blocks still read: through a temporary
    double* tmp = nullptr;
    if (hipMalloc((void**)&tmp, N * sizeof(double)) != hipSuccess) {
        (void)hipGetLastError();
        return MG_ERR_NOMEM;
    }
    hipError_t e = launch_geometry_bwd(n, ih2, psi, Cbar, sqrtgbar, tmp, s);
    if (e == hipSuccess) e = launch_shift(N, tmp, 0.0, psibar, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(tmp);
    return e == hipSuccess ? MG_OK : MG_ERR_HIP;
}

// ---- single steps (double arithmetic on caller fields) ---------------------------------------
static mg_status level_check(mg_ctx* c, int level, bool need_coarser) {
    if (!c) return MG_ERR_INVALID;
    if (level < 0 || level >= (int)c->lev.size()) return fail(c, MG_ERR_INVALID, "level out of range");
    if (need_coarser && level + 1 >= (int)c->lev.size()) return fail(c, MG_ERR_INVALID, "no coarser level");
    return MG_OK;
}

static mg_status ensure_scratch(mg_ctx* c, size_t elems) {
    if (c->scratch_elems >= elems) return MG_OK;
    dfree(c->scratch);
    c->scratch = nullptr;
    c->scratch_elems = 0;
    mg_status st = dalloc(c, (void**)&c->scratch, elems * sizeof(double));
    if (st == MG_OK) c->scratch_elems = elems;
    return st;
}

mg_status mg_apply(mg_ctx* c, int level, const double* u, double* out) {
    mg_status st = level_check(c, level, false);
    if (st != MG_OK) return st;
    if (!u || !out || u == out) return fail(c, MG_ERR_INVALID, "invalid apply arguments");
    HIPCHK(c, with_op(c, level, [&](auto op) { return launch_apply<double>(op, u, out, c->stream); }));
    return MG_OK;
}

mg_status mg_smooth(mg_ctx* c, int level, double* x, const double* b) {
    mg_status st = level_check(c, level, false);
    if (st != MG_OK) return st;
    if (!x || !b || x == b) return fail(c, MG_ERR_INVALID, "invalid smooth arguments");
    const Level& L = c->lev[level];
    if ((st = ensure_scratch(c, L.N)) != MG_OK) return st;
    double* bufs[2] = {x, c->scratch};
    const bool cheb = c->p.smoother == MG_CHEBYSHEV;
    int cur = 0, prev = -1;
    for (size_t k = 0; k < L.a.size(); ++k) {
        const bool use_prev = cheb && prev >= 0;
        const double* xp = use_prev ? bufs[prev] : nullptr;
        const int out = use_prev ? prev : 1 - cur;
        HIPCHK(c, with_op(c, level, [&](auto op) {
                   return launch_smooth_step<double>(op, bufs[cur], xp, b, bufs[out], L.a[k], L.c[k], c->stream);
               }));
        prev = cur;
        cur = out;
    }
    if (cur != 0) HIPCHK(c, hipMemcpyAsync(x, bufs[cur], L.N * sizeof(double), hipMemcpyDeviceToDevice, c->stream));
    return MG_OK;
}

mg_status mg_residual_restrict(mg_ctx* c, int level, const double* x, const double* b, double* coarse) {
    mg_status st = level_check(c, level, true);
    if (st != MG_OK) return st;
    if (!b || !coarse) return fail(c, MG_ERR_INVALID, "invalid residual_restrict arguments");
    if ((st = ensure_scratch(c, c->lev[level].N)) != MG_OK) return st;
    HIPCHK(c, with_op(c, level, [&](auto op) {
               return launch_residual_restrict<double>(op, x, b, coarse, c->scratch, c->stream);
           }));
    return MG_OK;
}

mg_status mg_prolong_add(mg_ctx* c, int level, const double* e, double* x) {
    mg_status st = level_check(c, level, true);
    if (st != MG_OK) return st;
    if (!e || !x) return fail(c, MG_ERR_INVALID, "invalid prolong arguments");
    HIPCHK(c, launch_prolong_add<double>(c->lev[level].n, e, x, c->stream));
    return MG_OK;
}

mg_status mg_coarse_solve(mg_ctx* c, const double* r, double* e) {
    if (!c || !r || !e || r == e) return fail(c, MG_ERR_INVALID, "invalid coarse_solve arguments");
    const Level& L = c->lev.back();
    if (!c->var) HIPCHK(c, launch_coarse_flat<double>(L.n, c->Q, c->lam1, r, e, c->stream));
    else HIPCHK(c, launch_coarse_dense<double>((int)L.N, c->G, r, e, c->stream));
    return MG_OK;
}

}  // extern "C"

namespace {

// One V-cycle step of level l in the inner type T on the context's buffers;
// the caller's double fields are rounded to T on entry and out is widened.
template <typename T>
mg_status inner_step_impl(mg_ctx* c, int step, int l, const double* x, const double* e, const double* b,
                          double* out) {
    Level& L = c->lev[l];
    Level* Lc = l + 1 < (int)c->lev.size() ? &c->lev[l + 1] : nullptr;
    hipStream_t s = c->stream;
    c->x1_ready = false;
    for (Level& Lv : c->lev) Lv.x1 = false;
    c->pending_sums = false;
    auto in = [&](size_t count, const double* src, void* dst) -> hipError_t {
        return launch_convert<T, double>(count, src, (T*)dst, s);
    };
    const T* res = nullptr;
    size_t count = L.N;
    mg_status st = MG_OK;
    switch (step) {
        case MG_STEP_SMOOTH:
            HIPCHK(c, in(L.N, x, L.x[0]));
            HIPCHK(c, in(L.N, b, L.b));
            L.cur = 0;
            st = smooth_level<T>(c, l, false);
            res = (const T*)L.x[L.cur];
            break;
        case MG_STEP_SMOOTH_ZERO:
            HIPCHK(c, in(L.N, b, L.b));
            st = smooth_level<T>(c, l, true);
            res = (const T*)L.x[L.cur];
            break;
        case MG_STEP_PROLONG_SMOOTH:
            HIPCHK(c, in(L.N, x, L.x[0]));
            HIPCHK(c, in(Lc->N, e, Lc->x[0]));
            HIPCHK(c, in(L.N, b, L.b));
            L.cur = 0;
            Lc->cur = 0;
            st = post_level<T>(c, l);
            res = (const T*)L.x[L.cur];
            break;
        case MG_STEP_RESIDUAL_RESTRICT:
            HIPCHK(c, in(L.N, x, L.x[0]));
            HIPCHK(c, in(L.N, b, L.b));
            L.cur = 0;
            st = residual_restrict_level<T>(c, l);
            res = (const T*)Lc->b;
            count = Lc->N;
            break;
        case MG_STEP_PROLONG:
            HIPCHK(c, in(L.N, x, L.x[0]));
            HIPCHK(c, in(Lc->N, e, Lc->x[0]));
            HIPCHK(c, launch_prolong_add<T>(L.n, (const T*)Lc->x[0], (T*)L.x[0], s));
            L.cur = 0;
            res = (const T*)L.x[0];
            break;
        case MG_STEP_VCYCLE:
            HIPCHK(c, in(L.N, b, L.b));
            st = vcycle_from_zero<T>(c, l);
            res = (const T*)L.x[L.cur];
            break;
        default:
            return fail(c, MG_ERR_INVALID, "unknown step");
    }
    if (st != MG_OK) return st;
    HIPCHK(c, (launch_convert<double, T>(count, res, out, s)));
    return MG_OK;
}

}  // namespace

extern "C" {

mg_status mg_inner_step(mg_ctx* c, int step, int level, const double* x, const double* e, const double* b,
                        double* out) {
    if (!c) return MG_ERR_INVALID;
    if (step < MG_STEP_SMOOTH || step > MG_STEP_VCYCLE) return fail(c, MG_ERR_INVALID, "unknown step");
    const bool coarser = step == MG_STEP_PROLONG_SMOOTH || step == MG_STEP_RESIDUAL_RESTRICT || step == MG_STEP_PROLONG;
    mg_status st = level_check(c, level, coarser);
    if (st != MG_OK) return st;
    const bool need_x = step == MG_STEP_SMOOTH || step == MG_STEP_PROLONG_SMOOTH ||
                        step == MG_STEP_RESIDUAL_RESTRICT || step == MG_STEP_PROLONG;
    const bool need_e = step == MG_STEP_PROLONG_SMOOTH || step == MG_STEP_PROLONG;
    const bool need_b = step != MG_STEP_PROLONG;
    if (!out || (need_x && !x) || (need_e && !e) || (need_b && !b))
        return fail(c, MG_ERR_INVALID, "missing field for this step");
    return c->inner_double ? inner_step_impl<double>(c, step, level, x, e, b, out)
                           : inner_step_impl<float>(c, step, level, x, e, b, out);
}

mg_status mg_level_lmax(const mg_ctx* c, double* out) {
    if (!c || !out) return MG_ERR_INVALID;
    for (size_t l = 0; l < c->lev.size(); ++l) out[l] = c->lev[l].lmax;
    return MG_OK;
}

mg_status mg_enable_kernel_timing(mg_ctx* c, int enable) {
    if (!c) return MG_ERR_INVALID;
    const int all = MG_TIME_STEP | MG_TIME_PAIR | MG_TIME_TRIPLE | MG_TIME_OUTER | MG_TIME_TRANSFER;
    if (enable < 0 || enable > all) return fail(c, MG_ERR_INVALID, "timing mask out of range");
    c->timing = enable;
    c->events_used = 0;
    c->timed_launches = 0;
    c->timed_ms = 0.0;
    c->timed_bytes = 0.0;
    return MG_OK;
}

mg_status mg_kernel_timing(mg_ctx* c, int* launches, double* total_ms, double* alg_bytes) {
    if (!c || !launches || !total_ms || !alg_bytes) return MG_ERR_INVALID;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    for (size_t i = 0; i < c->events_used; ++i) {
        float ms = 0.f;
        HIPCHK(c, hipEventElapsedTime(&ms, c->events[i].start, c->events[i].stop));
        c->timed_ms += ms;
    }
    c->events_used = 0;
    *launches = c->timed_launches;
    *total_ms = c->timed_ms;
    *alg_bytes = c->timed_bytes;
    c->timed_launches = 0;
    c->timed_ms = 0.0;
    c->timed_bytes = 0.0;
    return MG_OK;
}

}  // extern "C"
