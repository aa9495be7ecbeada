// gfx950 kernels of the matrix-free multigrid V-cycle.
//
// Every stencil kernel streams a periodic n^3 field (x fastest) with one
// thread per (x, y) column marching `nz` planes in z; wave64 rows run along
// the contiguous x axis so loads and stores are coalesced, and neighbour
// values are served from the vector L1 / L2 caches.  Reductions are
// per-block LDS trees in a fixed order followed by a single-block pass over
// the partials, so every result is bitwise reproducible run to run.
#include "kernels.h"
#include "flat_row.h"
#include "var_row.h"

#include "launch.h"
#include "stencil.h"
#include "sums.h"

#include <cmath>
#include <cstdint>
#include <type_traits>

namespace mg {
namespace {

// =====================================================================================
// smoothing step
// =====================================================================================
template <typename T, typename TC, bool HASX, bool HASPREV>
__global__ __launch_bounds__(kThreads) void k_smooth(int n, T ih2, const TC* __restrict__ C,
                                                     const T* __restrict__ x, const T* xprev,
                                                     const T* __restrict__ b, T* out, T a, T c,
                                                     int nz) {
    const Grid g{n, n - 1};
    const size_t N = (size_t)n * n * n;
    const int xi = blockIdx.x * blockDim.x + threadIdx.x;
    const int yi = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * nz;
    const Plain<T, T> u{x};
    const T dflat = T(-6) * ih2;
    for (int z = z0; z < z0 + nz; ++z) {
        const size_t i = g(xi, yi, z);
        const T bi = b[i];
        T val;
        if constexpr (HASX) {
            const T uc = x[i];
            T Mu, D;
            if (C == nullptr) {
                Mu = flat_Mu<T>(u, g, xi, yi, z, uc, ih2);
                D = dflat;
            } else {
                var_Mu<T, TC>(u, C, N, g, xi, yi, z, uc, ih2, Mu, D);
            }
            T xp = T(0);
            if constexpr (HASPREV) xp = xprev[i];
            // seven-point: c arrives as c / D (as in the row kernels)
            val = C == nullptr ? step_pt<T>(uc, xp, bi, Mu, a, c) : uc + a * (uc - xp) + c * (bi - Mu) / D;
        } else {
            val = C == nullptr ? c * bi : c * bi / var_diag<T, TC>(C, N, g, xi, yi, z, ih2);
        }
        out[i] = val;
    }
}

// =====================================================================================
// residual + full weighting
// =====================================================================================
template <typename T, typename TC, bool HASX>
__global__ __launch_bounds__(kThreads) void k_resid_restrict(int n, T ih2, const TC* __restrict__ C,
                                                             const T* __restrict__ x,
                                                             const T* __restrict__ b,
                                                             T* __restrict__ coarse, int nz) {
    const int nc = n >> 1;
    const Grid g{n, n - 1};
    const Grid gc{nc, nc - 1};
    const size_t N = (size_t)n * n * n;
    const int X = blockIdx.x * blockDim.x + threadIdx.x;
    const int Y = blockIdx.y * blockDim.y + threadIdx.y;
    const int Z0 = blockIdx.z * nz;
    const Plain<T, T> u{x};
    const T w1[3] = {T(0.25), T(0.5), T(0.25)};
    for (int Z = Z0; Z < Z0 + nz; ++Z) {
        T acc = T(0);
        for (int dz = -1; dz <= 1; ++dz) {
            T accy = T(0);
            for (int dy = -1; dy <= 1; ++dy) {
                T accx = T(0);
                for (int dx = -1; dx <= 1; ++dx) {
                    const int fx = 2 * X + dx, fy = 2 * Y + dy, fz = 2 * Z + dz;
                    const size_t i = g(fx, fy, fz);
                    T r = b[i];
                    if constexpr (HASX) {
                        const T uc = x[i];
                        T Mu, D;
                        if (C == nullptr) {
                            Mu = flat_Mu<T>(u, g, fx, fy, fz, uc, ih2);
                        } else {
                            var_Mu<T, TC>(u, C, N, g, fx, fy, fz, uc, ih2, Mu, D);
                        }
                        r -= Mu;
                    }
                    accx += w1[dx + 1] * r;
                }
                accy += w1[dy + 1] * accx;
            }
            acc += w1[dz + 1] * accy;
        }
        coarse[gc(X, Y, Z)] = acc;
    }
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_restrict(int n, const T* __restrict__ fine,
                                                       T* __restrict__ coarse, int nz,
                                                       const T* __restrict__ cC, T* cx1, T cc0, T cih2) {
    const int nc = n >> 1;
    const Grid g{n, n - 1};
    const Grid gc{nc, nc - 1};
    const int X = blockIdx.x * blockDim.x + threadIdx.x;
    const int Y = blockIdx.y * blockDim.y + threadIdx.y;
    const int Z0 = blockIdx.z * nz;
    for (int Z = Z0; Z < Z0 + nz; ++Z) {
        T v[3][3][3];
        for (int dz = 0; dz < 3; ++dz)
            for (int dy = 0; dy < 3; ++dy)
                for (int dx = 0; dx < 3; ++dx) v[dz][dy][dx] = fine[g(2 * X + dx - 1, 2 * Y + dy - 1, 2 * Z + dz - 1)];
        const T w = fw_pt<T>(v);
        const size_t i = gc(X, Y, Z);
        coarse[i] = w;
        // the coarse level's first step from zero needs its own right-hand side
        // point only, and saves that level a launch (about 4 us)
        if (cx1) cx1[i] = cc0 * w / var_diag<T, T>(cC, (size_t)nc * nc * nc, gc, X, Y, Z, cih2);
    }
}

// =====================================================================================
// trilinear prolongation + correction
// =====================================================================================
template <typename T>
__global__ __launch_bounds__(kThreads) void k_prolong_add(int n, const T* __restrict__ e, T* x, int nz) {
    const int nc = n >> 1;
    const Grid g{n, n - 1};
    const Grid gc{nc, nc - 1};
    const int xi = blockIdx.x * blockDim.x + threadIdx.x;
    const int yi = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * nz;
    auto ec = [&](int X, int Y, int Z) { return e[gc(X, Y, Z)]; };
    for (int z = z0; z < z0 + nz; ++z) {
        // interpolate along x on the (up to) 4 coarse lines, then y, then z
        const T p = prolong_pt<T>(ec, xi, yi, z);
        const size_t i = g(xi, yi, z);
        x[i] = add_pt<T>(x[i], p);
    }
}

// =====================================================================================
// operator application
// =====================================================================================
// out = M x, or out = b - M x when b is given
template <typename T, typename TC>
__global__ __launch_bounds__(kThreads) void k_apply(int n, T ih2, const TC* __restrict__ C,
                                                    const T* __restrict__ x, const T* __restrict__ b,
                                                    T* __restrict__ out, int nz) {
    const Grid g{n, n - 1};
    const size_t N = (size_t)n * n * n;
    const int xi = blockIdx.x * blockDim.x + threadIdx.x;
    const int yi = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * nz;
    const Plain<T, T> u{x};
    for (int z = z0; z < z0 + nz; ++z) {
        const size_t i = g(xi, yi, z);
        const T uc = x[i];
        T Mu, D;
        if (C == nullptr) {
            Mu = flat_Mu<T>(u, g, xi, yi, z, uc, ih2);
        } else {
            var_Mu<T, TC>(u, C, N, g, xi, yi, z, uc, ih2, Mu, D);
        }
        out[i] = b ? b[i] - Mu : Mu;
    }
}

// =====================================================================================
// outer defect correction: optional phi update, residual in TA, sum of r^2
// =====================================================================================
template <typename TA, typename TR, typename TE, typename TC, bool UPDATE>
__global__ __launch_bounds__(kThreads) void k_outer_residual(int n, TA ih2, const TC* __restrict__ C,
                                                             const double* __restrict__ phi_in,
                                                             const TE* __restrict__ e,
                                                             double* __restrict__ phi_out,
                                                             const double* __restrict__ b, Mean bm,
                                                             TR* __restrict__ r, TR* __restrict__ x1, TA c0,
                                                             double* partials, int nz) {
    const double bmean = bm.get();
    __shared__ double sh[3 * kThreads];
    const Grid g{n, n - 1};
    const size_t N = (size_t)n * n * n;
    const int xi = blockIdx.x * blockDim.x + threadIdx.x;
    const int yi = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * nz;
    double ss = 0.0, sb = 0.0, sp = 0.0;
    for (int z = z0; z < z0 + nz; ++z) {
        const size_t i = g(xi, yi, z);
        TA Mu, D, uc;
        if constexpr (UPDATE) {
            const double pn = phi_in[i] + (double)e[i];
            phi_out[i] = pn;
            sp += pn;
            uc = (TA)pn;
            const PlusE<TA, TE> u{phi_in, e};
            if (C == nullptr) Mu = flat_Mu<TA>(u, g, xi, yi, z, uc, ih2);
            else var_Mu<TA, TC>(u, C, N, g, xi, yi, z, uc, ih2, Mu, D);
        } else {
            sp += phi_in[i];
            uc = (TA)phi_in[i];
            const Plain<TA, double> u{phi_in};
            if (C == nullptr) Mu = flat_Mu<TA>(u, g, xi, yi, z, uc, ih2);
            else var_Mu<TA, TC>(u, C, N, g, xi, yi, z, uc, ih2, Mu, D);
        }
        const double bq = b[i] - bmean;
        const TA ri = (TA)bq - Mu;
        r[i] = (TR)ri;
        if (x1) {  // first smoothing step from zero, rounded as the smoothing kernels round it
            if (C == nullptr) x1[i] = (TR)c0 * (TR)ri;  // seven-point: c0 arrives as c0 / D
            else x1[i] = (TR)(c0 * (TA)(TR)ri / D);
        }
        ss += (double)ri * (double)ri;
        sb += bq * bq;
    }
    // three partial sums, arrays of the block count: sum (b - bmean)^2, sum r^2, sum phi
    const int nb = gridDim.x * gridDim.y * gridDim.z;
    double t[3] = {sb, ss, sp};
    block_sums<3>(t, sh);
    if (lin_tid() == 0) {
        partials[lin_bid()] = t[0];
        partials[nb + lin_bid()] = t[1];
        partials[2 * nb + lin_bid()] = t[2];
    }
}

// =====================================================================================
// reductions
// =====================================================================================
__global__ __launch_bounds__(kThreads) void k_block_sums(int n, const double* __restrict__ u, double shift, int p,
                                                         double* partials, int nz) {
    __shared__ double sh[kThreads];
    const Grid g{n, n - 1};
    const int xi = blockIdx.x * blockDim.x + threadIdx.x;
    const int yi = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * nz;
    double s = 0.0;
    // unrolled so that several planes' loads are in flight (39 -> 35 us at 256^3);
    // the sum keeps its z order
#pragma unroll 8
    for (int z = z0; z < z0 + nz; ++z) {
        const double v = u[g(xi, yi, z)] - shift;
        s += p == 2 ? v * v : v;
    }
    const double tot = block_sum(s, sh);
    if (lin_tid() == 0) partials[lin_bid()] = tot;
}

__global__ __launch_bounds__(1024) void k_finalize(const double* __restrict__ partials, int count, double* out,
                                                   int slot, double* host_out, double seq) {
    __shared__ double sh[1024];
    const int tid = threadIdx.x;
    double v = 0.0;
    for (int i = tid; i < count; i += 1024) v += partials[i];
    const double r = block_sum(v, sh);
    if (tid == 0) {
        out[slot] = r;
        if (host_out) {  // pinned host mirror, then the flag the host polls
            host_out[slot] = r;
            __threadfence_system();
            *reinterpret_cast<volatile double*>(host_out + kHostMeanSlot) = seq;
            __threadfence_system();
        }
    }
}

// out[slot + k] = sum of partials[k * count .. (k + 1) * count), k < arrays
// (host_out: pinned host mirror, no separate copy)
__global__ __launch_bounds__(kSumLanes) void k_finalize_multi(SumsJob job) {
    __shared__ double sh[kSumLanes];
    finish_sums(job, sh);
}

// =====================================================================================
// elementwise
// =====================================================================================
__global__ void k_shift(size_t count, const double* src, double shift, double* dst) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i] - shift;
}
// dst = src - mean(src), or zero where the source norm (sums[1]) is zero; the
// sum of src is sums[3]
__global__ __launch_bounds__(kThreads) void k_gauge(size_t pairs, const double2* src, const double* sums, double inv,
                                                    double2* dst) {
    const bool zero = sums[1] == 0.0;
    const double shift = sums[3] * inv;
    // four pairs in flight per thread: 8 us at 128^3 where one value per thread took 17.5
    const size_t stride = (size_t)gridDim.x * kThreads;
    for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < pairs; i += 4 * stride) {
        double2 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i + k * stride < pairs) v[k] = src[i + k * stride];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (i + k * stride < pairs)
                dst[i + k * stride] = zero ? make_double2(0.0, 0.0) : make_double2(v[k].x - shift, v[k].y - shift);
    }
}
template <typename T>
__global__ void k_add(size_t count, const double* src, const T* e, double* dst) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i] + (double)e[i];
}
template <typename TD, typename TS>
__global__ void k_convert(size_t count, const TS* src, TD* dst) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = (TD)src[i];
}
template <typename T>
__global__ void k_fill(size_t count, T v, T* dst) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = v;
}
dim3 ew_grid(size_t count) {
    size_t b = (count + kThreads - 1) / kThreads;
    if (b > 65536) b = 65536;
    if (b == 0) b = 1;
    return dim3((unsigned)b);
}

// =====================================================================================
// coarsest level
// =====================================================================================
// Separable exact solve of the seven-point system: three 1-D basis changes,
// division by the eigenvalue, three inverse basis changes, all in double.
// Every basis change is a set of independent lines (NC^2 lines of NC points
// along one axis): one thread holds a whole line in registers, forms all NC
// outputs and writes them back over the line, so each value crosses LDS once
// per change and the basis matrix, the same for every line, is read with
// uniform loads.  The z change, the division and the inverse z change run on
// the same line in one pass.  LDS rows are padded to NC + 1 values and planes
// to NC (NC + 1), so the lanes of a wave fall on different banks along every
// axis.  Each output is the same sum, in the same order, as a plain basis
// change (acc = 0, then q_j v_j added for j = 0 .. NC-1).  NC (4, 8 or 16) is
// a compile-time constant, so every loop unrolls.  One workgroup of
// coarse_threads(NC) threads (one per line).
constexpr int coarse_threads(int nc) { return nc * nc < 64 ? 64 : nc * nc; }
template <typename T, int NC>
__global__ __launch_bounds__(coarse_threads(NC)) void k_coarse_flat(const double* __restrict__ Q,
                                                                    const double* __restrict__ lam1,
                                                                    const T* __restrict__ r, T* __restrict__ e) {
    constexpr int N = NC * NC * NC;
    constexpr int RP = NC + 1, PP = NC * RP;  // padded row and plane pitches
    constexpr int LINES = NC * NC, NT = coarse_threads(NC);
    __shared__ double A[NC * PP];
    const int tid = threadIdx.x;
    auto at = [](int x, int y, int z) { return x + RP * y + PP * z; };
    for (int i = tid; i < N; i += NT) A[at(i & (NC - 1), (i / NC) & (NC - 1), i / (NC * NC))] = (double)r[i];
    __syncthreads();
    // q[j + NC*k] = basis vector k at point j.  Forward: c_k = sum_j q[j,k] v_j;
    // inverse: v_k = sum_j q[k,j] c_j.  The line's values are all in registers
    // before output k is stored over point k (the thread owns the line), and
    // f(k, c_k) is what is stored.
    auto change = [&](const double(&v)[NC], int base, int stride, bool forward, auto f) {
#pragma unroll 4
        for (int k = 0; k < NC; ++k) {
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const double w = forward ? Q[j + NC * k] : Q[k + NC * j];
                acc += w * v[j];
            }
            A[base + k * stride] = f(k, acc);
        }
    };
    auto load = [&](double(&v)[NC], int base, int stride) {
#pragma unroll
        for (int j = 0; j < NC; ++j) v[j] = A[base + j * stride];
    };
    auto same = [](int, double c) { return c; };
    const int u = tid & (NC - 1), w = tid / NC;  // line tid: the two other coordinates
    const int bx = at(0, u, w), by = at(u, 0, w), bz = at(u, w, 0);
    double v[NC];
    // forward x and y changes
    if (tid < LINES) {
        load(v, bx, 1);
        change(v, bx, 1, true, same);
    }
    __syncthreads();
    if (tid < LINES) {
        load(v, by, RP);
        change(v, by, RP, true, same);
    }
    __syncthreads();
    // z line of wavenumbers (kx, ky) = (u, w): forward change divided by the
    // eigenvalue (the constant mode set to zero), then the inverse change
    if (tid < LINES) {
        const double lxy = lam1[u] + lam1[w];
        load(v, bz, PP);
        change(v, bz, PP, true, [&](int k, double c) {
            const double l = lxy + lam1[k];
            return (u == 0 && w == 0 && k == 0) ? 0.0 : c / l;
        });
        load(v, bz, PP);
        change(v, bz, PP, false, same);
    }
    __syncthreads();
    // inverse y and x changes
    if (tid < LINES) {
        load(v, by, RP);
        change(v, by, RP, false, same);
    }
    __syncthreads();
    if (tid < LINES) {
        load(v, bx, 1);
        change(v, bx, 1, false, same);
    }
    __syncthreads();
    for (int i = tid; i < N; i += NT) e[i] = (T)A[at(i & (NC - 1), (i / NC) & (NC - 1), i / (NC * NC))];
}

// The same solve on 16^3 points: each pass is a product of the 16 x 16 basis
// with 16 columns of 16 lines, so it runs on the FP64 matrix unit, a 16 x 16
// tile of lines per wave (four 16x16x4 products) with the basis held in
// registers.  One thread per line fetched its 256 weights per pass through the
// scalar cache and took 14.6 us per launch; this takes 10.8.
typedef double v4d __attribute__((ext_vector_type(4)));
template <typename T>
__global__ __launch_bounds__(1024) void k_coarse_flat16(const double* __restrict__ Q,
                                                        const double* __restrict__ lam1,
                                                        const T* __restrict__ r, T* __restrict__ e) {
    constexpr int RP = 17, PP = 16 * RP;  // padded row and plane pitches
    __shared__ double A[16 * PP];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // operand layout of the product: lane holds line c and point 4 s + k of
    // step s, the basis element (row c, column 4 s + k), and of the result
    // rows 4 i + k (i = 0 .. 3) of line c
    const int c = lane & 15, k = lane >> 4;
    double qf[4], qi[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        qf[s] = Q[4 * s + k + 16 * c];
        qi[s] = Q[c + 16 * (4 * s + k)];
    }
    auto product = [&](const double(&q)[4], const double(&v)[4]) {
        v4d d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) d = __builtin_amdgcn_mfma_f64_16x16x4f64(q[s], v[s], d, 0, 0, 0);
        return d;
    };
    // line c of the wave's tile, point j: x lines and y lines of plane z = w,
    // z lines of plane y = w
    auto ax = [&](int j) { return j + RP * c + PP * w; };
    auto ay = [&](int j) { return c + RP * j + PP * w; };
    auto az = [&](int j) { return c + RP * w + PP * j; };
    auto pass = [&](const double(&q)[4], auto at) {
        double v[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = A[at(4 * s + k)];
        return product(q, v);
    };
    auto put = [&](const v4d& d, auto at) {
#pragma unroll
        for (int i = 0; i < 4; ++i) A[at(4 * i + k)] = d[i];
        __syncthreads();
    };
    {
        double v[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) v[s] = (double)r[(w * 16 + c) * 16 + 4 * s + k];
        put(product(qf, v), ax);
    }
    put(pass(qf, ay), ay);
    {  // z line of wavenumbers (c, w): divided by the eigenvalue, the constant mode set to zero
        const double lxy = lam1[c] + lam1[w];
        v4d d = pass(qf, az);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int kz = 4 * i + k;
            d[i] = (c == 0 && w == 0 && kz == 0) ? 0.0 : d[i] / (lxy + lam1[kz]);
        }
        put(d, az);
    }
    put(pass(qi, az), az);
    put(pass(qi, ay), ay);
    const v4d d = pass(qi, ax);
#pragma unroll
    for (int i = 0; i < 4; ++i) e[(w * 16 + c) * 16 + 4 * i + k] = (T)d[i];
}

// e = G r, 8 rows per block, 32 lanes per row, fixed-order sums.
template <typename T>
__global__ __launch_bounds__(256) void k_coarse_dense(int N, const double* __restrict__ G, const T* __restrict__ r,
                                                      T* __restrict__ e) {
    __shared__ double sh[256];
    const int row = blockIdx.x * 8 + (threadIdx.x >> 5);
    const int lane = threadIdx.x & 31;
    double acc = 0.0;
    if (row < N)
        for (int j = lane; j < N; j += 32) acc += G[(size_t)row * N + j] * (double)r[j];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 16; s > 0; s >>= 1) {
        if (lane < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (lane == 0 && row < N) e[row] = (T)sh[threadIdx.x];
}

// =====================================================================================
// coefficient gradient (operator VJP)
// =====================================================================================
template <typename TO>
__global__ __launch_bounds__(kThreads) void k_coeff_grad(int n, double ih2, const double* __restrict__ lam,
                                                         const double* __restrict__ phi, TO* __restrict__ out,
                                                         int nz) {
    const Grid g{n, n - 1};
    const size_t N = (size_t)n * n * n;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * nz;
    for (int z = z0; z < z0 + nz; ++z) {
        const size_t i = g(x, y, z);
        const double l0 = lam[i], p0 = phi[i];
        double lp[3], lm[3], pp[3], pm[3];
        const int d[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
        for (int a = 0; a < 3; ++a) {
            const size_t ip = g(x + d[a][0], y + d[a][1], z + d[a][2]);
            const size_t im = g(x - d[a][0], y - d[a][1], z - d[a][2]);
            lp[a] = lam[ip];
            lm[a] = lam[im];
            pp[a] = phi[ip];
            pm[a] = phi[im];
            const double gp = (lp[a] - l0) * (pp[a] - p0);
            const double gm = (l0 - lm[a]) * (p0 - pm[a]);
            out[a * N + i] = (TO)(0.5 * (gp + gm) * ih2);
        }
        const int pa[3] = {0, 0, 1}, pb[3] = {1, 2, 2};
        for (int p = 0; p < 3; ++p) {
            const int a = pa[p], b = pb[p];
            const double dla = lp[a] - lm[a], dlb = lp[b] - lm[b];
            const double dpa = pp[a] - pm[a], dpb = pp[b] - pm[b];
            out[(3 + p) * N + i] = (TO)((dla * dpb + dlb * dpa) * 0.25 * ih2);
        }
    }
}

}  // namespace

// =====================================================================================
// launchers
// =====================================================================================
int stencil_blocks(int n) {
    Shape s = stencil_shape(n);
    return (int)(s.grid.x * s.grid.y * s.grid.z);
}

int outer_blocks(int n, bool flat, bool double_arith) {
    if (flat) return row_kernels_apply(n) ? row_outer_blocks(n, double_arith) : stencil_blocks(n);
    return var_row_kernels_apply(n) ? var_row_blocks(n) : stencil_blocks(n);
}

template <typename T, typename TC>
hipError_t launch_smooth_step(const OpDesc<TC>& op, const T* x, const T* xprev, const T* b, T* out, double a,
                              double c, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    if (op.coeff == nullptr && row_kernels_apply(op.n))
        return launch_smooth_row<T>(op.n, op.ih2, x, xprev, b, out, a, c / (-6.0 * op.ih2), s, ev0, ev1);
    if (op.coeff != nullptr && var_row_kernels_apply(op.n))
        return launch_var_smooth_row<T, TC>(op.n, op.ih2, op.coeff, x, xprev, b, out, a, c, s, ev0, ev1);
    Shape sh = stencil_shape(op.n);
    if (op.coeff == nullptr) c = c / (-6.0 * op.ih2);  // the seven-point kernel takes c / D
    if (x == nullptr)
        MG_LAUNCH((k_smooth<T, TC, false, false>), sh.grid, sh.block, s, ev0, ev1, op.n, (T)op.ih2, op.coeff, x,
                           xprev, b, out, (T)a, (T)c, sh.nz);
    else if (xprev == nullptr)
        MG_LAUNCH((k_smooth<T, TC, true, false>), sh.grid, sh.block, s, ev0, ev1, op.n, (T)op.ih2, op.coeff, x,
                           xprev, b, out, (T)a, (T)c, sh.nz);
    else
        MG_LAUNCH((k_smooth<T, TC, true, true>), sh.grid, sh.block, s, ev0, ev1, op.n, (T)op.ih2, op.coeff, x,
                           xprev, b, out, (T)a, (T)c, sh.nz);
    return hipGetLastError();
}

template <typename T, typename TC>
hipError_t launch_residual_restrict(const OpDesc<TC>& op, const T* x, const T* b, T* coarse, T* scratch,
                                    hipStream_t s, hipEvent_t ev0, hipEvent_t ev1, const FirstStep<T>& first) {
    if (op.coeff == nullptr && x != nullptr && row_kernels_apply(op.n))
        return launch_rr_row<T>(op.n, op.ih2, x, b, coarse, s, ev0, ev1);
    if (op.coeff != nullptr && x != nullptr && var_rr_applies(op.n, sizeof(T)))
        return launch_var_rr<T, TC>(op.n, op.ih2, op.coeff, x, b, coarse, first.C, first.x1, first.c0, s, ev0, ev1);
    if (scratch != nullptr && x != nullptr) {
        if (op.coeff != nullptr && var_row_kernels_apply(op.n)) {
            hipError_t e = launch_var_resid_row<T, TC>(op.n, op.ih2, op.coeff, x, b, scratch, s, ev0, ev1);
            if (e != hipSuccess) return e;
        } else {
            Shape sf = stencil_shape(op.n);
            hipLaunchKernelGGL((k_apply<T, TC>), sf.grid, sf.block, 0, s, op.n, (T)op.ih2, op.coeff, x, b, scratch,
                               sf.nz);
        }
        Shape sc = stencil_shape(op.n / 2);
        hipLaunchKernelGGL((k_restrict<T>), sc.grid, sc.block, 0, s, op.n, (const T*)scratch, coarse, sc.nz, first.C,
                           first.x1, (T)first.c0, (T)(op.ih2 / 4.0));
        return hipGetLastError();
    }
    Shape sh = stencil_shape(op.n / 2);
    if (x)
        hipLaunchKernelGGL((k_resid_restrict<T, TC, true>), sh.grid, sh.block, 0, s, op.n, (T)op.ih2, op.coeff, x, b,
                           coarse, sh.nz);
    else
        hipLaunchKernelGGL((k_resid_restrict<T, TC, false>), sh.grid, sh.block, 0, s, op.n, (T)op.ih2, op.coeff, x, b,
                           coarse, sh.nz);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_prolong_add(int n, const T* e, T* x, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    if (row_kernels_apply(n)) return launch_prolong_row<T>(n, e, x, s, ev0, ev1);
    Shape sh = stencil_shape(n);
    MG_LAUNCH((k_prolong_add<T>), sh.grid, sh.block, s, ev0, ev1, n, e, x, sh.nz);
    return hipGetLastError();
}

template <typename T, typename TC>
hipError_t launch_apply(const OpDesc<TC>& op, const T* u, T* out, hipStream_t s) {
    if (op.coeff != nullptr && var_row_kernels_apply(op.n))
        return launch_var_resid_row<T, TC>(op.n, op.ih2, op.coeff, u, (const T*)nullptr, out, s);
    Shape sh = stencil_shape(op.n);
    hipLaunchKernelGGL((k_apply<T, TC>), sh.grid, sh.block, 0, s, op.n, (T)op.ih2, op.coeff, u, (const T*)nullptr,
                       out, sh.nz);
    return hipGetLastError();
}

template <typename TA, typename TR, typename TE, typename TC>
hipError_t launch_outer_residual(const OpDesc<TC>& op, const double* phi_in, const TE* e, double* phi_out,
                                 const double* b, Mean bmean, TR* r, TR* x1, double c0, double* partials,
                                 hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    if (op.coeff == nullptr && row_kernels_apply(op.n))
        return launch_outer_row<TA, TR, TE>(op.n, op.ih2, phi_in, e, phi_out, b, bmean, r, x1,
                                            c0 / (-6.0 * op.ih2), partials, s, ev0, ev1);
    if (op.coeff != nullptr && var_row_kernels_apply(op.n))
        return launch_var_outer_row<TA, TR, TE, TC>(op.n, op.ih2, op.coeff, phi_in, e, phi_out, b, bmean, r, x1, c0,
                                                    partials, s, ev0, ev1);
    Shape sh = stencil_shape(op.n);
    if (op.coeff == nullptr) c0 = c0 / (-6.0 * op.ih2);
    if (e)
        MG_LAUNCH((k_outer_residual<TA, TR, TE, TC, true>), sh.grid, sh.block, s, ev0, ev1, op.n, (TA)op.ih2,
                  op.coeff, phi_in, e, phi_out, b, bmean, r, x1, (TA)c0, partials, sh.nz);
    else
        MG_LAUNCH((k_outer_residual<TA, TR, TE, TC, false>), sh.grid, sh.block, s, ev0, ev1, op.n, (TA)op.ih2,
                  op.coeff, phi_in, e, phi_out, b, bmean, r, x1, (TA)c0, partials, sh.nz);
    return hipGetLastError();
}

hipError_t launch_block_sums(int n, const double* u, double shift, int p, double* partials, hipStream_t s) {
    Shape sh = stencil_shape(n);
    hipLaunchKernelGGL(k_block_sums, sh.grid, sh.block, 0, s, n, u, shift, p, partials, sh.nz);
    return hipGetLastError();
}
hipError_t launch_finalize_sum(const double* partials, int count, double* out, int slot, hipStream_t s,
                               double* host_out, double seq) {
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(1024), 0, s, partials, count, out, slot, host_out, seq);
    return hipGetLastError();
}
hipError_t launch_finalize_sums(const double* partials, int count, int arrays, double* out, int slot,
                                hipStream_t s, double* host_out, double seq) {
    const SumsJob job{partials, count, arrays, out, slot, host_out, seq};
    hipLaunchKernelGGL(k_finalize_multi, dim3(1), dim3(kSumLanes), 0, s, job);
    return hipGetLastError();
}
hipError_t launch_shift(size_t count, const double* src, double shift, double* dst, hipStream_t s) {
    hipLaunchKernelGGL(k_shift, ew_grid(count), dim3(kThreads), 0, s, count, src, shift, dst);
    return hipGetLastError();
}
hipError_t launch_gauge(size_t count, const double* src, const double* sums, double inv, double* dst, hipStream_t s) {
    const size_t pairs = count / 2, per = 4 * (size_t)kThreads;  // n^3 is even
    const size_t blocks = (pairs + per - 1) / per;
    hipLaunchKernelGGL(k_gauge, dim3((unsigned)(blocks < 1 ? 1 : blocks > 16384 ? 16384 : blocks)), dim3(kThreads), 0,
                       s, pairs, reinterpret_cast<const double2*>(src), sums, inv, reinterpret_cast<double2*>(dst));
    return hipGetLastError();
}
template <typename T>
hipError_t launch_add(size_t count, const double* src, const T* e, double* dst, hipStream_t s) {
    hipLaunchKernelGGL((k_add<T>), ew_grid(count), dim3(kThreads), 0, s, count, src, e, dst);
    return hipGetLastError();
}
template <typename TD, typename TS>
hipError_t launch_convert(size_t count, const TS* src, TD* dst, hipStream_t s) {
    hipLaunchKernelGGL((k_convert<TD, TS>), ew_grid(count), dim3(kThreads), 0, s, count, src, dst);
    return hipGetLastError();
}
template <typename T>
hipError_t launch_fill(size_t count, T value, T* dst, hipStream_t s) {
    hipLaunchKernelGGL((k_fill<T>), ew_grid(count), dim3(kThreads), 0, s, count, value, dst);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_coarse_flat(int nc, const double* Q, const double* lam1, const T* r, T* e, hipStream_t s) {
    switch (nc) {
        case 4: hipLaunchKernelGGL((k_coarse_flat<T, 4>), dim3(1), dim3(coarse_threads(4)), 0, s, Q, lam1, r, e); break;
        case 8: hipLaunchKernelGGL((k_coarse_flat<T, 8>), dim3(1), dim3(coarse_threads(8)), 0, s, Q, lam1, r, e); break;
        case 16:
            hipLaunchKernelGGL((k_coarse_flat16<T>), dim3(1), dim3(1024), 0, s, Q, lam1, r, e);
            break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template <typename T>
hipError_t launch_coarse_dense(int N, const double* G, const T* r, T* e, hipStream_t s) {
    hipLaunchKernelGGL((k_coarse_dense<T>), dim3((N + 7) / 8), dim3(256), 0, s, N, G, r, e);
    return hipGetLastError();
}

template <typename TO>
hipError_t launch_coeff_grad(int n, double ih2, const double* lam, const double* phi, TO* cbar, hipStream_t s) {
    Shape sh = stencil_shape(n);
    hipLaunchKernelGGL((k_coeff_grad<TO>), sh.grid, sh.block, 0, s, n, ih2, lam, phi, cbar, sh.nz);
    return hipGetLastError();
}
// ---- explicit instantiations ------------------------------------------------------
#define INST_T_TC(T, TC)                                                                                         \
    template hipError_t launch_smooth_step<T, TC>(const OpDesc<TC>&, const T*, const T*, const T*, T*, double,   \
                                                  double, hipStream_t, hipEvent_t, hipEvent_t);                  \
    template hipError_t launch_residual_restrict<T, TC>(const OpDesc<TC>&, const T*, const T*, T*, T*, hipStream_t, \
                                                        hipEvent_t, hipEvent_t, const FirstStep<T>&);             \
    template hipError_t launch_apply<T, TC>(const OpDesc<TC>&, const T*, T*, hipStream_t);
INST_T_TC(float, float)
INST_T_TC(double, double)
INST_T_TC(double, float)
INST_T_TC(float, double)

#define INST_T(T)                                                                                  \
    template hipError_t launch_prolong_add<T>(int, const T*, T*, hipStream_t, hipEvent_t, hipEvent_t); \
    template hipError_t launch_add<T>(size_t, const double*, const T*, double*, hipStream_t);      \
    template hipError_t launch_fill<T>(size_t, T, T*, hipStream_t);                                \
    template hipError_t launch_coarse_flat<T>(int, const double*, const double*, const T*, T*, hipStream_t); \
    template hipError_t launch_coarse_dense<T>(int, const double*, const T*, T*, hipStream_t);     \
    template hipError_t launch_coeff_grad<T>(int, double, const double*, const double*, T*, hipStream_t);
INST_T(float)
INST_T(double)

template hipError_t launch_convert<float, double>(size_t, const double*, float*, hipStream_t);
template hipError_t launch_convert<double, float>(size_t, const float*, double*, hipStream_t);
template hipError_t launch_convert<double, double>(size_t, const double*, double*, hipStream_t);
template hipError_t launch_convert<float, float>(size_t, const float*, float*, hipStream_t);

#define INST_OUTER(TA, TR, TE, TC)                                                                                \
    template hipError_t launch_outer_residual<TA, TR, TE, TC>(const OpDesc<TC>&, const double*, const TE*, double*, \
                                                              const double*, Mean, TR*, TR*, double, double*,     \
                                                              hipStream_t, hipEvent_t, hipEvent_t);
INST_OUTER(double, double, double, double)
INST_OUTER(double, double, double, float)
INST_OUTER(double, float, float, float)
INST_OUTER(double, float, float, double)
INST_OUTER(float, float, float, float)
INST_OUTER(float, float, float, double)

}  // namespace mg
