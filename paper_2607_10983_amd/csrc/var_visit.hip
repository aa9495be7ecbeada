// Fused visits of the 32^3 level of a variable-coefficient hierarchy.
//
// A visit of that level with v smoothing steps took 2 v + 3 launches, each of
// them bound by its launch (about 4 us) and by one trip to L2, not by its
// work.  Here it takes two.  A workgroup owns a tile of 8 x 4 x 4 fine points
// and keeps the tile with a halo as wide as the visit needs in LDS: two copies
// of the iterate and the six coefficient fields.  Every application of the
// operator shrinks the valid region by one point per side, so neighbouring
// tiles compute their common halo twice and never wait for each other:
//
//   pre:  x_2 .. x_v from x_1 (written by the kernel that produced b), the
//         residual, its full weighting; writes x_v on the tile, the 4 x 2 x 2
//         coarse right-hand side and the coarse level's own first step;
//   post: x_0 = x + P e, then v steps; writes x_v on the tile.
//
// The tile is small on purpose.  At 32^3 it gives one workgroup per CU: the
// redundant points (10 to 14 applications per point of a visit instead of 3)
// cost less than leaving CUs idle, and the halo'd coefficients still fit LDS,
// from which one application reads its 19 iterate and 21 coefficient values at
// constant offsets.
//
// Measured at 32^3, degree 3: 9.0 + 7.0 us in float and 9.4 + 9.0 us in double
// (tiles of 8 x 8 x 4 points, 128 workgroups: 10.5 + 8.3 and 11.5 + 10.5), in
// place of nine launches of 38 to 41 us.  The 64^3 level keeps its separate
// kernels: 1024 tiles of 8 x 8 x 4 are four rounds of the chip's LDS, and the
// visits took 27.5 + 26.4 us in float and 45.5 + 44.0 us in double, against
// about 37 and 55 us for the launches.
//
// The point formula is that of var_Mu and k_smooth (stencil.h, kernels.hip).
#include "var_visit.h"

#include "row.h"
#include "stencil.h"

namespace mg {
namespace {

constexpr int kTX = 8, kTY = 4, kTZ = 4;  // tile
constexpr int kThrV = 512;

struct VisitSteps {
    double a[kVarVisitMaxSteps], c[kVarVisitMaxSteps];
};

// Region of the tile grown by LO points below and HI points above on each
// axis, DX x DY x DZ points, x fastest.
template <int LO, int HI>
struct Region {
    static constexpr int DX = kTX + LO + HI, DY = kTY + LO + HI, DZ = kTZ + LO + HI;
    static constexpr int P = DX * DY * DZ, SY = DX, SZ = DX * DY;
};

// Points of region R with the outer `S` layers removed, numbered by q: the
// linear index in R.
template <typename R, int S>
__device__ __forceinline__ int inner_index(int q) {
    constexpr int X = R::DX - 2 * S, Y = R::DY - 2 * S;
    const int k = q / (X * Y), rem = q - k * (X * Y);
    const int j = rem / X, i = rem - j * X;
    return ((k + S) * R::DY + (j + S)) * R::DX + (i + S);
}
template <typename R, int S>
struct Inner {
    static constexpr int P = (R::DX - 2 * S) * (R::DY - 2 * S) * (R::DZ - 2 * S);
    static constexpr int K = (P + kThrV - 1) / kThrV;  // points per thread
};

// global index of region point p of the tile at (tx, ty, tz), region origin LO below
template <typename R, int LO>
__device__ __forceinline__ int global_index(int p, int tx, int ty, int tz, int n, int lg) {
    const int k = p / R::SZ, rem = p - k * R::SZ;
    const int j = rem / R::DX, i = rem - j * R::DX;
    const int m = n - 1;
    return ((((tz - LO + k) & m) << lg | ((ty - LO + j) & m)) << lg) | ((tx - LO + i) & m);
}

// M u and D at region point p; C: six fields of R::P values
template <typename T, typename R>
__device__ __forceinline__ void Mu_at(const T* u, const T* C, int p, T ih2, T& Mu, T& D) {
    constexpr int SX = 1, SY = R::SY, SZ = R::SZ, P = R::P;
    const T uc = u[p];
    T acc, dsum, cross;
    {
        const T c0 = C[p];
        const T fp = T(0.5) * (c0 + C[p + SX]), fm = T(0.5) * (c0 + C[p - SX]);
        acc = fp * (u[p + SX] - uc) - fm * (uc - u[p - SX]);
        dsum = fp + fm;
    }
    {
        const T* Cy = C + P;
        const T c0 = Cy[p];
        const T fp = T(0.5) * (c0 + Cy[p + SY]), fm = T(0.5) * (c0 + Cy[p - SY]);
        acc += fp * (u[p + SY] - uc) - fm * (uc - u[p - SY]);
        dsum += fp + fm;
    }
    {
        const T* Cz = C + 2 * P;
        const T c0 = Cz[p];
        const T fp = T(0.5) * (c0 + Cz[p + SZ]), fm = T(0.5) * (c0 + Cz[p - SZ]);
        acc += fp * (u[p + SZ] - uc) - fm * (uc - u[p - SZ]);
        dsum += fp + fm;
    }
    {
        const T* K = C + 3 * P;
        const T upp = u[p + SX + SY], upm = u[p + SX - SY], ump = u[p - SX + SY], umm = u[p - SX - SY];
        cross = K[p + SX] * (upp - upm) - K[p - SX] * (ump - umm);
        cross += K[p + SY] * (upp - ump) - K[p - SY] * (upm - umm);
    }
    {
        const T* K = C + 4 * P;
        const T upp = u[p + SX + SZ], upm = u[p + SX - SZ], ump = u[p - SX + SZ], umm = u[p - SX - SZ];
        cross += K[p + SX] * (upp - upm) - K[p - SX] * (ump - umm);
        cross += K[p + SZ] * (upp - ump) - K[p - SZ] * (upm - umm);
    }
    {
        const T* K = C + 5 * P;
        const T upp = u[p + SY + SZ], upm = u[p + SY - SZ], ump = u[p - SY + SZ], umm = u[p - SY - SZ];
        cross += K[p + SY] * (upp - upm) - K[p - SY] * (ump - umm);
        cross += K[p + SZ] * (upp - ump) - K[p - SZ] * (upm - umm);
    }
    Mu = (acc + T(0.25) * cross) * ih2;
    D = -dsum * ih2;
}

// One smoothing step on the points S layers inside R: out = step(u); out holds
// the previous iterate there (prev) and is overwritten in place.
template <typename T, typename R, int LO, int S>
__device__ __forceinline__ void smooth_region(const T* u, T* out, const T* C, const T* __restrict__ b, int tx, int ty,
                                              int tz, int n, int lg, T ih2, T a, T c, bool prev) {
    constexpr int P = Inner<R, S>::P, K = Inner<R, S>::K;
    T bv[K];
    int pi[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = threadIdx.x + k * kThrV;
        pi[k] = inner_index<R, S>(q < P ? q : P - 1);
        bv[k] = b[global_index<R, LO>(pi[k], tx, ty, tz, n, lg)];
    }
    __syncthreads();  // u is complete
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = threadIdx.x + k * kThrV;
        if (q < P) {
            const int p = pi[k];
            T Mu, D;
            Mu_at<T, R>(u, C, p, ih2, Mu, D);
            const T xc = u[p];
            const T xp = prev ? out[p] : T(0);
            out[p] = xc + a * (xc - xp) + c * (bv[k] - Mu) / D;
        }
    }
}

// the six coefficient fields and one more field of region R into LDS, all
// loads of a thread in flight together
template <typename T, typename R, int LO>
__device__ __forceinline__ void stage(const T* __restrict__ C, size_t N, T* sC, int tx, int ty, int tz, int n, int lg) {
    constexpr int K = (R::P + kThrV - 1) / kThrV;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = threadIdx.x + k * kThrV;
        const int gi = global_index<R, LO>(q < R::P ? q : R::P - 1, tx, ty, tz, n, lg);
        T v[6];
#pragma unroll
        for (int f = 0; f < 6; ++f) v[f] = C[f * N + gi];
        if (q < R::P) {
#pragma unroll
            for (int f = 0; f < 6; ++f) sC[f * R::P + q] = v[f];
        }
    }
}

__device__ __forceinline__ void tile_of(int lb, int n, int& tx, int& ty, int& tz) {
    const int nx = n / kTX, ny = n / kTY;
    tx = (lb % nx) * kTX;
    ty = (lb / nx % ny) * kTY;
    tz = lb / (nx * ny) * kTZ;
}

// smoothing steps K .. V-1 of a pass, step K on the points S layers inside R;
// returns with the last iterate in buf[..] (index returned)
template <typename T, typename R, int LO, int V, int K, int S>
__device__ __forceinline__ void steps_from(T* u, T* w, const T* C, const T* b, int tx, int ty, int tz, int n, int lg,
                                           T ih2, const VisitSteps& st, bool cheb, bool prev) {
    if constexpr (K < V) {
        smooth_region<T, R, LO, S>(u, w, C, b, tx, ty, tz, n, lg, ih2, (T)st.a[K], (T)st.c[K], prev);
        steps_from<T, R, LO, V, K + 1, S + 1>(w, u, C, b, tx, ty, tz, n, lg, ih2, st, cheb, cheb);
    }
}

template <typename T, int V>
__global__ __launch_bounds__(kThrV) void k_var_visit_pre(int n, int lg, T ih2, const T* __restrict__ C,
                                                         const T* __restrict__ x1, const T* __restrict__ b,
                                                         T* __restrict__ xout, T* __restrict__ cb,
                                                         const T* __restrict__ cC, T* __restrict__ cx1, T cc0,
                                                         T cih2, VisitSteps st, bool cheb) {
    // the residual is needed on [-1, tile), x_v one point further, x_1 another V - 1
    constexpr int LO = V + 1, HI = V;
    using R = Region<LO, HI>;
    __shared__ T lds[8 * R::P];
    T* sC = lds;
    T* u0 = lds + 6 * R::P;
    T* u1 = lds + 7 * R::P;
    const size_t N = (size_t)n * n * n;
    int tx, ty, tz;
    tile_of(xcd_logical(blockIdx.x, gridDim.x), n, tx, ty, tz);
    {
        constexpr int K = (R::P + kThrV - 1) / kThrV;
        T v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int q = threadIdx.x + k * kThrV;
            v[k] = x1[global_index<R, LO>(q < R::P ? q : R::P - 1, tx, ty, tz, n, lg)];
        }
        stage<T, R, LO>(C, N, sC, tx, ty, tz, n, lg);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int q = threadIdx.x + k * kThrV;
            if (q < R::P) u0[q] = v[k];
        }
    }
    steps_from<T, R, LO, V, 1, 1>(u0, u1, sC, b, tx, ty, tz, n, lg, ih2, st, cheb, false);
    T* u = (V - 1) & 1 ? u1 : u0;  // x_v
    T* r = (V - 1) & 1 ? u0 : u1;  // free
    // residual on the points V layers inside R: (T + 1)^3 points from -1
    constexpr int S = V;
    {
        constexpr int P = Inner<R, S>::P, K = Inner<R, S>::K;
        T bv[K];
        int pi[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int q = threadIdx.x + k * kThrV;
            pi[k] = inner_index<R, S>(q < P ? q : P - 1);
            bv[k] = b[global_index<R, LO>(pi[k], tx, ty, tz, n, lg)];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int q = threadIdx.x + k * kThrV;
            if (q < P) {
                T Mu, D;
                Mu_at<T, R>(u, sC, pi[k], ih2, Mu, D);
                r[pi[k]] = bv[k] - Mu;
            }
        }
    }
    // the smoothed iterate on the tile (256 points)
    if (threadIdx.x < kTX * kTY * kTZ) {
        const int i = threadIdx.x % kTX, j = threadIdx.x / kTX % kTY, k = threadIdx.x / (kTX * kTY);
        xout[(((size_t)(tz + k) << lg | (ty + j)) << lg) | (tx + i)] = u[((k + LO) * R::DY + j + LO) * R::DX + i + LO];
    }
    __syncthreads();
    constexpr int NCX = kTX / 2, NCY = kTY / 2, NCZ = kTZ / 2;
    if (threadIdx.x < NCX * NCY * NCZ) {
        const int I = threadIdx.x % NCX, J = threadIdx.x / NCX % NCY, K = threadIdx.x / (NCX * NCY);
        const int p = ((2 * K + LO) * R::DY + 2 * J + LO) * R::DX + 2 * I + LO;
        T v[3][3][3];
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) v[dz][dy][dx] = r[p + (dz - 1) * R::SZ + (dy - 1) * R::SY + dx - 1];
        const T w = fw_pt<T>(v);
        const int nc = n >> 1, X = tx / 2 + I, Y = ty / 2 + J, Z = tz / 2 + K;
        const size_t ci = ((size_t)Z * nc + Y) * nc + X;
        cb[ci] = w;
        if (cx1) cx1[ci] = cc0 * w / var_diag<T, T>(cC, (size_t)nc * nc * nc, Grid{nc, nc - 1}, X, Y, Z, cih2);
    }
}

template <typename T, int V>
__global__ __launch_bounds__(kThrV) void k_var_visit_post(int n, int lg, T ih2, const T* __restrict__ C,
                                                          const T* __restrict__ x, const T* __restrict__ e,
                                                          const T* __restrict__ b, T* __restrict__ xout,
                                                          VisitSteps st, bool cheb) {
    constexpr int LO = V;
    using R = Region<V, V>;
    // coarse points under the region, from ((tx - V) >> 1): one more than half the width, rounded up
    constexpr int EX = (R::DX + 1) / 2 + 1, EY = (R::DY + 1) / 2 + 1, EZ = (R::DZ + 1) / 2 + 1, EP = EX * EY * EZ;
    __shared__ T lds[8 * R::P];
    static_assert(EP <= R::P, "the staged coarse field fits the second iterate");
    T* sC = lds;
    T* u0 = lds + 6 * R::P;
    T* u1 = lds + 7 * R::P;
    T* se = u1;  // until the first step
    const size_t N = (size_t)n * n * n;
    int tx, ty, tz;
    tile_of(xcd_logical(blockIdx.x, gridDim.x), n, tx, ty, tz);
    const int nc = n >> 1, X0 = (tx - V) >> 1, Y0 = (ty - V) >> 1, Z0 = (tz - V) >> 1;
    constexpr int K = (R::P + kThrV - 1) / kThrV, KE = (EP + kThrV - 1) / kThrV;
    T v[K], ev[KE];
#pragma unroll
    for (int k = 0; k < KE; ++k) {
        const int q = threadIdx.x + k * kThrV, p = q < EP ? q : EP - 1;
        const int I = p % EX, J = p / EX % EY, Q = p / (EX * EY);
        ev[k] = e[((size_t)((Z0 + Q) & (nc - 1)) * nc + ((Y0 + J) & (nc - 1))) * nc + ((X0 + I) & (nc - 1))];
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = threadIdx.x + k * kThrV;
        v[k] = x[global_index<R, LO>(q < R::P ? q : R::P - 1, tx, ty, tz, n, lg)];
    }
    stage<T, R, LO>(C, N, sC, tx, ty, tz, n, lg);
#pragma unroll
    for (int k = 0; k < KE; ++k) {
        const int q = threadIdx.x + k * kThrV;
        if (q < EP) se[q] = ev[k];
    }
    __syncthreads();
    auto ec = [&](int X, int Y, int Z) { return se[((Z - Z0) * EY + (Y - Y0)) * EX + (X - X0)]; };
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int q = threadIdx.x + k * kThrV;
        if (q < R::P) {
            const int kk = q / R::SZ, rem = q - kk * R::SZ, j = rem / R::DX, i = rem - j * R::DX;
            u0[q] = add_pt<T>(v[k], prolong_pt<T>(ec, tx - V + i, ty - V + j, tz - V + kk));
        }
    }
    steps_from<T, R, LO, V, 0, 1>(u0, u1, sC, b, tx, ty, tz, n, lg, ih2, st, cheb, false);
    const T* u = V & 1 ? u1 : u0;
    __syncthreads();
    if (threadIdx.x < kTX * kTY * kTZ) {
        const int i = threadIdx.x % kTX, j = threadIdx.x / kTX % kTY, k = threadIdx.x / (kTX * kTY);
        xout[(((size_t)(tz + k) << lg | (ty + j)) << lg) | (tx + i)] = u[((k + LO) * R::DY + j + LO) * R::DX + i + LO];
    }
}

template <int V>
constexpr size_t pre_lds(size_t elem) { return 8 * (size_t)Region<V + 1, V>::P * elem; }
constexpr size_t kLdsMax = 160 * 1024;

VisitSteps visit_steps(const double* a, const double* c, int steps) {
    VisitSteps st{};
    for (int k = 0; k < steps; ++k) {
        st.a[k] = a[k];
        st.c[k] = c[k];
    }
    return st;
}
int log2i(int n) {
    int lg = 0;
    while ((1 << lg) < n) ++lg;
    return lg;
}

}  // namespace

bool var_visit_applies(int n, int steps, size_t elem) {
    if (n != 32) return false;
    // the pre visit has the larger halo
    switch (steps) {
        case 1: return pre_lds<1>(elem) <= kLdsMax;
        case 2: return pre_lds<2>(elem) <= kLdsMax;
        case 3: return pre_lds<3>(elem) <= kLdsMax;
        case 4: return pre_lds<4>(elem) <= kLdsMax;
        default: return false;
    }
}

#define DISPATCH_STEPS(steps, ...)                                                                  \
    switch (steps) {                                                                                \
        case 1: { constexpr int V = 1; __VA_ARGS__; break; }                                        \
        case 2: { constexpr int V = 2; __VA_ARGS__; break; }                                        \
        case 3: { constexpr int V = 3; __VA_ARGS__; break; }                                        \
        case 4: { constexpr int V = 4; if constexpr (pre_lds<V>(sizeof(T)) <= kLdsMax) __VA_ARGS__; break; } \
        default: return hipErrorInvalidValue;                                                       \
    }

template <typename T>
hipError_t launch_var_visit_pre(int n, double ih2, const T* C, const T* x1, const T* b, T* xout, T* cb, const T* cC,
                                T* cx1, double cc0, const double* a, const double* c, int steps, bool cheb,
                                hipStream_t s) {
    if (!var_visit_applies(n, steps, sizeof(T)) || x1 == xout) return hipErrorInvalidValue;
    const VisitSteps st = visit_steps(a, c, steps);
    const dim3 grid((n / kTX) * (n / kTY) * (n / kTZ));
    DISPATCH_STEPS(steps, {
        hipLaunchKernelGGL((k_var_visit_pre<T, V>), grid, dim3(kThrV), 0, s, n, log2i(n), (T)ih2, C, x1, b, xout, cb,
                           cC, cx1, (T)cc0, (T)(ih2 / 4.0), st, cheb);
    })
    return hipGetLastError();
}

template <typename T>
hipError_t launch_var_visit_post(int n, double ih2, const T* C, const T* x, const T* e, const T* b, T* xout,
                                 const double* a, const double* c, int steps, bool cheb, hipStream_t s) {
    if (!var_visit_applies(n, steps, sizeof(T)) || x == xout) return hipErrorInvalidValue;
    const VisitSteps st = visit_steps(a, c, steps);
    const dim3 grid((n / kTX) * (n / kTY) * (n / kTZ));
    DISPATCH_STEPS(steps, {
        hipLaunchKernelGGL((k_var_visit_post<T, V>), grid, dim3(kThrV), 0, s, n, log2i(n), (T)ih2, C, x, e, b, xout,
                           st, cheb);
    })
    return hipGetLastError();
}

#define INST_VISIT(T)                                                                                               \
    template hipError_t launch_var_visit_pre<T>(int, double, const T*, const T*, const T*, T*, T*, const T*, T*,    \
                                                double, const double*, const double*, int, bool, hipStream_t);      \
    template hipError_t launch_var_visit_post<T>(int, double, const T*, const T*, const T*, const T*, T*,           \
                                                 const double*, const double*, int, bool, hipStream_t);
INST_VISIT(float)
INST_VISIT(double)

}  // namespace mg
