// Single-workgroup V-cycle tail for the seven-point hierarchy.
//
// Levels with at most 16^3 points are far too small to fill the chip; one
// kernel launch per smoothing step there costs more in launch latency than in
// work.  This kernel runs the whole remaining V-cycle from a small level down
// to the coarsest and back up inside ONE workgroup of 1024 threads, its phases
// separated by workgroup barriers.
//
// A phase is bound by the LDS and the barrier of one CU, so the fields stay in
// registers: a thread owns 4 consecutive x points of the 16^3 level (x, x_prev
// and b there) and one point of the 8^3 level, and publishes only the iterate
// of each step, in two alternating copies (one barrier per step).  The x
// neighbours of a 16^3 segment come from the other lanes of its quad.  The
// residual is weighted in x before it is published, and the prolongation reads
// its coarse rows without branches.  The coarsest level's exact solve
// (separable real Fourier basis) runs in double, a 4^3 one inside one wave.
//
// Degree 3, 16^3 to 4^3: 8.7 us per launch in float and 11.7 in double, against
// 19 and 25.8 with every field in LDS and each point reading its neighbours, b
// and x_prev from there.
#include "tail.h"

#include "row.h"

namespace mg {
namespace {

constexpr int kTailThreads = 1024;

// value of the next (+1) or previous (-1) lane of the quad, wrapping inside it
template <int D>
__device__ __forceinline__ int quad_rot32(int v) {
    // quad_perm selectors [1,2,3,0] and [3,0,1,2]
    return __builtin_amdgcn_update_dpp(0, v, D > 0 ? 0x39 : 0x93, 0xF, 0xF, false);
}
template <int D, typename T>
__device__ __forceinline__ T quad_rot(T v) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, quad_rot32<D>(__builtin_bit_cast(int, v)));
    } else {
        v2i h = __builtin_bit_cast(v2i, v);
        h.x = quad_rot32<D>(h.x);
        h.y = quad_rot32<D>(h.y);
        return __builtin_bit_cast(T, h);
    }
}

// A copy of the 16^3 level, segment i (points 4 i .. 4 i + 3) in 16-byte
// pieces with piece j of all segments together, so that the lanes of a wave
// access consecutive addresses in both types.
template <typename T>
struct Copy16 {
    static constexpr int P = 16 / (int)sizeof(T), J = 4 / P;
    T v[4096];
    __device__ __forceinline__ void put(int i, const T (&s)[4]) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            v4i t;
            __builtin_memcpy(&t, &s[j * P], 16);
            *reinterpret_cast<v4i*>(v + (j * 1024 + i) * P) = t;
        }
    }
    __device__ __forceinline__ void get(T (&s)[4], int i) const {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const v4i t = *reinterpret_cast<const v4i*>(v + (j * 1024 + i) * P);
            __builtin_memcpy(&s[j * P], &t, 16);
        }
    }
};

template <typename T>
struct Shared {
    __align__(16) Copy16<T> f[2];  // 16^3 iterate or, weighted in x, its residual
    __align__(16) T g[2][512];     // 8^3 iterate or residual
    T h[2][64];                    // 4^3 right-hand side and solution
    double sA[512], sB[512], q[64], lam[8];
};

// the thread's share of a level: the 16^3 level
template <typename T>
struct Seg {
    T x[4], b[4];
};

// M x on the segment from the published copy
template <typename T>
__device__ __forceinline__ void M16(const Copy16<T>& f, const T (&x)[4], T ih2, T (&Mx)[4]) {
    const int i = threadIdx.x, r = i & ~63;  // a wave holds a plane, a quad a row
    T ym[4], yp[4], zm[4], zp[4];
    f.get(ym, r | ((i - 4) & 63));
    f.get(yp, r | ((i + 4) & 63));
    f.get(zm, (i - 64) & 1023);
    f.get(zp, (i + 64) & 1023);
    const T lft = quad_rot<-1>(x[3]), rgt = quad_rot<1>(x[0]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        T s = (e > 0 ? x[e - 1] : lft) + (e < 3 ? x[e + 1] : rgt);
        s += ym[e] + yp[e];
        s += zm[e] + zp[e];
        Mx[e] = (s - T(6) * x[e]) * ih2;
    }
}
template <typename T>
__device__ __forceinline__ T M8(const T* g, T x, T ih2) {
    const int i = threadIdx.x;
    T s = g[(i & ~7) | ((i - 1) & 7)] + g[(i & ~7) | ((i + 1) & 7)];
    s += g[(i & ~56) | ((i - 8) & 56)] + g[(i & ~56) | ((i + 8) & 56)];
    s += g[(i - 64) & 511] + g[(i + 64) & 511];
    return (s - T(6) * x) * ih2;
}

// A smoothing pass on the thread's segment of the 16^3 level (tail level l);
// w: the copy the next publication goes to.
template <typename T>
__device__ __forceinline__ void smooth16(const TailArgs<T>& A, Shared<T>& S, int l, Seg<T>& u, int& w, bool from_zero) {
    const T ih2 = (T)A.ih2[l], dinv = T(1) / (T(-6) * ih2);
    T p[4] = {T(0), T(0), T(0), T(0)};
    int k = 0;
    if (from_zero) {
        const T c = (T)A.sched.c[l][0];
#pragma unroll
        for (int e = 0; e < 4; ++e) u.x[e] = c * dinv * u.b[e];
        k = 1;
    }
    for (; k < A.sched.steps; ++k) {
        const T a = (T)A.sched.a[l][k], c = (T)A.sched.c[l][k];
        S.f[w].put(threadIdx.x, u.x);
        __syncthreads();
        T Mx[4];
        M16<T>(S.f[w], u.x, ih2, Mx);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const T x = u.x[e];
            u.x[e] = x + a * (x - p[e]) + c * dinv * (u.b[e] - Mx[e]);
            if (A.sched.cheb) p[e] = x;
        }
        w ^= 1;
    }
}
// The same on the thread's point of the 8^3 level (threads 0 .. 511; the
// others pass the barriers only).
template <typename T>
__device__ __forceinline__ void smooth8(const TailArgs<T>& A, Shared<T>& S, int l, T& x, T b, int& w, bool from_zero) {
    const bool on = threadIdx.x < 512;
    const T ih2 = (T)A.ih2[l], dinv = T(1) / (T(-6) * ih2);
    T p = T(0);
    int k = 0;
    if (from_zero) {
        x = (T)A.sched.c[l][0] * dinv * b;
        k = 1;
    }
    for (; k < A.sched.steps; ++k) {
        const T a = (T)A.sched.a[l][k], c = (T)A.sched.c[l][k];
        if (on) S.g[w][threadIdx.x] = x;
        __syncthreads();
        if (on) {
            const T y = x;
            x = y + a * (y - p) + c * dinv * (b - M8<T>(S.g[w], y, ih2));
            if (A.sched.cheb) p = y;
        }
        w ^= 1;
    }
}

// residual on 16^3, full weighting: returns b of the thread's 8^3 point
template <typename T>
__device__ __forceinline__ T restrict16(const TailArgs<T>& A, Shared<T>& S, int l, const Seg<T>& u, int& w) {
    const int i = threadIdx.x;
    T Mx[4], r[4];
    S.f[w].put(i, u.x);
    __syncthreads();
    M16<T>(S.f[w], u.x, (T)A.ih2[l], Mx);
    w ^= 1;
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = u.b[e] - Mx[e];
    const T lft = quad_rot<-1>(r[3]);
    T* v = S.f[w].v;  // [z][y][X], weighted in x
    v[2 * i] = T(0.25) * lft + T(0.5) * r[0] + T(0.25) * r[1];
    v[2 * i + 1] = T(0.25) * r[1] + T(0.5) * r[2] + T(0.25) * r[3];
    __syncthreads();
    w ^= 1;
    T acc = T(0);
    if (i < 512) {
        const int X = i & 7, y0 = 2 * ((i >> 3) & 7), z0 = 2 * (i >> 6);
#pragma unroll
        for (int dz = -1; dz <= 1; ++dz) {
            T ay = T(0);
#pragma unroll
            for (int dy = -1; dy <= 1; ++dy)
                ay += (dy == 0 ? T(0.5) : T(0.25)) * v[(((z0 + dz) & 15) * 16 + ((y0 + dy) & 15)) * 8 + X];
            acc += (dz == 0 ? T(0.5) : T(0.25)) * ay;
        }
    }
    return acc;
}
// residual on 8^3, full weighting into S.h[0][i] by thread i < 64
template <typename T>
__device__ __forceinline__ void restrict8(const TailArgs<T>& A, Shared<T>& S, int l, T x, T b, int& w) {
    const int i = threadIdx.x;
    if (i < 512) S.g[w][i] = x;
    __syncthreads();
    const T r = i < 512 ? b - M8<T>(S.g[w], x, (T)A.ih2[l]) : T(0);
    w ^= 1;
    if (i < 512) S.g[w][i] = r;
    __syncthreads();
    if (i < 64) {
        const T* g = S.g[w];
        const int x0 = 2 * (i & 3), y0 = 2 * ((i >> 2) & 3), z0 = 2 * (i >> 4);
        T acc = T(0);
#pragma unroll
        for (int dz = -1; dz <= 1; ++dz) {
            T ay = T(0);
#pragma unroll
            for (int dy = -1; dy <= 1; ++dy) {
                const T* row = g + (((z0 + dz) & 7) * 8 + ((y0 + dy) & 7)) * 8;
                const T ax = T(0.25) * row[(x0 - 1) & 7] + T(0.5) * row[x0] + T(0.25) * row[x0 + 1];
                ay += (dy == 0 ? T(0.5) : T(0.25)) * ax;
            }
            acc += (dz == 0 ? T(0.5) : T(0.25)) * ay;
        }
        S.h[0][i] = acc;
    }
    w ^= 1;
}

// The interpolation weight of a fine point and the sum over its coarse points
// in the order z, y, x, each product exact (a power of two): the terms of an
// even coordinate's second point are zero instead of branches.
template <typename T>
__device__ __forceinline__ T weight(bool ox, bool oy, bool oz) {
    return (ox ? T(0.5) : T(1)) * (oy ? T(0.5) : T(1)) * (oz ? T(0.5) : T(1));
}
template <typename T>
__device__ __forceinline__ T interp(const T (&r)[4][2], bool ox, bool oy, bool oz) {
    const T w = weight<T>(ox, oy, oz);
    const bool on[4] = {true, oy, oz, oy && oz};
    T v = T(0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {  // rows (Y, Z), (Y + 1, Z), (Y, Z + 1), (Y + 1, Z + 1)
        v += on[k] ? w * r[k][0] : T(0);
        v += on[k] && ox ? w * r[k][1] : T(0);
    }
    return v;
}
// P e at the thread's 8^3 point, e of 4^3 points
template <typename T>
__device__ __forceinline__ T prolong8(const T* e) {
    const int i = threadIdx.x, x = i & 7, y = (i >> 3) & 7, z = (i >> 6) & 7;
    const int X = x >> 1, Y = y >> 1, Z = z >> 1, X1 = (X + 1) & 3, Y1 = (Y + 1) & 3, Z1 = (Z + 1) & 3;
    const int row[4] = {Z * 16 + Y * 4, Z * 16 + Y1 * 4, Z1 * 16 + Y * 4, Z1 * 16 + Y1 * 4};
    T r[4][2];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        r[k][0] = e[row[k] + X];
        r[k][1] = e[row[k] + X1];
    }
    return interp<T>(r, x & 1, y & 1, z & 1);
}
// x += P e on the thread's 16^3 segment, e of 8^3 points: coarse points X, X + 1
// of each row, X + 2 from the next lane of the quad
template <typename T>
__device__ __forceinline__ void prolong16(T (&x)[4], const T* e) {
    const int i = threadIdx.x, X = 2 * (i & 3), y = (i >> 2) & 15, z = i >> 6;
    const bool oy = y & 1, oz = z & 1;
    const int Y = y >> 1, Z = z >> 1, Y1 = (Y + 1) & 7, Z1 = (Z + 1) & 7;
    const int row[4] = {Z * 64 + Y * 8, Z * 64 + Y1 * 8, Z1 * 64 + Y * 8, Z1 * 64 + Y1 * 8};
    T lo[4][2], hi[4][2];  // (X, X + 1) and (X + 1, X + 2)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        lo[k][0] = e[row[k] + X];
        lo[k][1] = hi[k][0] = e[row[k] + X + 1];
        hi[k][1] = quad_rot<1>(lo[k][0]);
    }
    x[0] = x[0] + interp<T>(lo, false, oy, oz);
    x[1] = x[1] + interp<T>(lo, true, oy, oz);
    x[2] = x[2] + interp<T>(hi, false, oy, oz);
    x[3] = x[3] + interp<T>(hi, true, oy, oz);
}

// Exact zero-mean solve on the coarsest level (NC^3 points) in double with the
// separable basis: three forward passes, the division by the eigenvalue sums,
// three backward passes.  The basis q and eigenvalues lam are in LDS.
template <typename T, int NC>
__device__ void coarsest(const T* bl, T* xl, double* sA, double* sB, const double* q, const double* lam) {
    constexpr int N = NC * NC * NC;
    const int tid = threadIdx.x;
    for (int i = tid; i < N; i += kTailThreads) sA[i] = (double)bl[i];
    __syncthreads();
    auto pass = [&](const double* src, double* dst, int axis, bool forward) {
        for (int i = tid; i < N; i += kTailThreads) {
            const int x = i % NC, y = (i / NC) % NC, z = i / (NC * NC);
            const int k = axis == 0 ? x : axis == 1 ? y : z;
            const int stride = axis == 0 ? 1 : axis == 1 ? NC : NC * NC;
            const int base = i - k * stride;
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < NC; ++j) acc += (forward ? q[j + NC * k] : q[k + NC * j]) * src[base + j * stride];
            dst[i] = acc;
        }
        __syncthreads();
    };
    pass(sA, sB, 0, true);
    pass(sB, sA, 1, true);
    pass(sA, sB, 2, true);
    for (int i = tid; i < N; i += kTailThreads) {
        const int x = i % NC, y = (i / NC) % NC, z = i / (NC * NC);
        sB[i] = (x == 0 && y == 0 && z == 0) ? 0.0 : sB[i] / (lam[x] + lam[y] + lam[z]);
    }
    __syncthreads();
    pass(sB, sA, 2, false);
    pass(sA, sB, 1, false);
    pass(sB, sA, 0, false);
    for (int i = tid; i < N; i += kTailThreads) xl[i] = (T)sA[i];
    __syncthreads();
}

// The same solve on a 4^3 coarsest level by one wave: lane i owns point
// i = x + 4 y + 16 z and takes the other points of its line from their lanes
// by cross-lane moves, so the six passes need no workgroup barrier.  Same
// sums in the same order as the workgroup version.
template <typename T>
__device__ void coarsest4(const T* bl, T* xl, const double* q, const double* lam) {
    constexpr int NC = 4;
    if (threadIdx.x < 64) {
        const int i = threadIdx.x, x = i & 3, y = (i >> 2) & 3, z = i >> 4;
        auto pass = [&](double u, int axis, bool forward) {
            const int k = axis == 0 ? x : axis == 1 ? y : z;
            const int stride = axis == 0 ? 1 : axis == 1 ? NC : NC * NC;
            const int base = i - k * stride;
            double acc = 0.0;
#pragma unroll
            for (int j = 0; j < NC; ++j)
                acc += (forward ? q[j + NC * k] : q[k + NC * j]) * __shfl(u, base + j * stride, 64);
            return acc;
        };
        double v = (double)bl[i];
        v = pass(v, 0, true);
        v = pass(v, 1, true);
        v = pass(v, 2, true);
        v = (x == 0 && y == 0 && z == 0) ? 0.0 : v / (lam[x] + lam[y] + lam[z]);
        v = pass(v, 2, false);
        v = pass(v, 1, false);
        v = pass(v, 0, false);
        xl[i] = (T)v;
    }
    __syncthreads();
}

// HAS16: the first tail level has 16^3 points (else 8^3); CST: points per side
// of the coarsest level.
template <typename T, bool HAS16, int CST>
__global__ __launch_bounds__(kTailThreads) void k_tail(TailArgs<T> A) {
    __shared__ Shared<T> S;
    static_assert(sizeof(S.f) >= kSumLanes * sizeof(double), "the sums fit the tail's LDS");
    if (blockIdx.x == 1) {  // the outer sums, beside the tail
        finish_sums(A.sums, reinterpret_cast<double*>(&S));
        return;
    }
    constexpr bool HAS8 = CST == 4;
    constexpr int l8 = HAS16 ? 1 : 0;
    static_assert(HAS16 || HAS8, "at least one level above the coarsest");
    const int i = threadIdx.x;
    Seg<T> u;
    T x8 = T(0), b8 = T(0);
    int w16 = 0, w8 = 0;
    if constexpr (HAS16) {
        ldrow<T, 4>(u.b, A.b + 4 * i);
    } else {
        if (i < 512) b8 = A.b[i];
    }
    if (i < CST * CST) S.q[i] = A.Q[i];
    if (i < CST) S.lam[i] = A.lam1[i];
    if constexpr (HAS16) {
        smooth16<T>(A, S, 0, u, w16, true);
        b8 = restrict16<T>(A, S, 0, u, w16);
    }
    T* e8 = S.g[0];  // solution of the 8^3 level
    if constexpr (HAS8) {
        smooth8<T>(A, S, l8, x8, b8, w8, true);
        restrict8<T>(A, S, l8, x8, b8, w8);  // lane i of the first wave wrote what it reads next
        coarsest4<T>(S.h[0], S.h[1], S.q, S.lam);
        if (i < 512) x8 = x8 + prolong8<T>(S.h[1]);
        smooth8<T>(A, S, l8, x8, b8, w8, false);
        if constexpr (HAS16) {
            // the copy the last step did not read
            e8 = S.g[w8];
            if (i < 512) e8[i] = x8;
            __syncthreads();
        } else {
            if (i < 512) A.x[i] = x8;
        }
    } else {
        if (i < 512) S.g[1][i] = b8;
        __syncthreads();
        coarsest<T, 8>(S.g[1], e8, S.sA, S.sB, S.q, S.lam);
    }
    if constexpr (HAS16) {
        prolong16<T>(u.x, e8);
        smooth16<T>(A, S, 0, u, w16, false);
        strow<T, 4>(A.x + 4 * i, u.x);
    }
}

}  // namespace

template <typename T>
hipError_t launch_tail(const TailArgs<T>& args, hipStream_t s) {
    // levels of 16^3 or 8^3 points down to a coarsest of 8^3 or 4^3, halving each time
    if (args.nlev < 2 || args.nlev > kTailMaxLevels) return hipErrorInvalidValue;
    for (int l = 0; l < args.nlev; ++l) {
        const int nl = args.n[l];
        const bool coarsest = l == args.nlev - 1;
        if (coarsest ? (nl != 8 && nl != 4) : (nl != 16 && nl != 8)) return hipErrorInvalidValue;
        if (l > 0 && nl * 2 != args.n[l - 1]) return hipErrorInvalidValue;
    }
    const dim3 grid(args.sums.count > 0 ? 2 : 1), block(kTailThreads);
    if (args.n[0] == 8) hipLaunchKernelGGL((k_tail<T, false, 4>), grid, block, 0, s, args);
    else if (args.n[args.nlev - 1] == 8) hipLaunchKernelGGL((k_tail<T, true, 8>), grid, block, 0, s, args);
    else hipLaunchKernelGGL((k_tail<T, true, 4>), grid, block, 0, s, args);
    return hipGetLastError();
}

template hipError_t launch_tail<float>(const TailArgs<float>&, hipStream_t);
template hipError_t launch_tail<double>(const TailArgs<double>&, hipStream_t);

}  // namespace mg
