// Row helpers of the seven-point kernels (flat_row.hip, pair_tile.hip): the
// stencil and the smoothing step on a row with their rounding written out, and
// the rows of a coarse correction that a kernel prolongs on the fly.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>

#include "fma.h"
#include "row.h"

namespace mg {
namespace {

// Element i (0 <= i < 64 VEC) of a row copy written by lds_strow.
template <typename T, int VEC>
__device__ __forceinline__ T lds_elem(const T* row, int i) {
    constexpr int B = VEC * (int)sizeof(T);
    if constexpr (B <= 16) {
        return row[i];
    } else {
        constexpr int P = 16 / (int)sizeof(T);
        const int l = i / VEC, e = i - l * VEC;
        return row[((e / P) * 64 + l) * P + e % P];
    }
}

template <typename T, int VEC>
__device__ __forceinline__ void copyrow(T (&d)[VEC], const T (&s)[VEC]) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) d[e] = s[e];
}

// M x on one row: c = centre row, ym/yp = rows y-1/y+1, zm/zp = planes z-1/z+1.
// The rounding of the stencil and of the smoothing step below is written out
// (no contraction left to the compiler), so every kernel that applies a step
// -- single or fused -- produces the same bits.
template <typename T, int VEC>
__device__ __forceinline__ void flat7_row(const T (&c)[VEC], const T (&ym)[VEC], const T (&yp)[VEC],
                                          const T (&zm)[VEC], const T (&zp)[VEC], T ih2, T (&Mx)[VEC]) {
#pragma clang fp contract(off)
    const T lft = lane_rot(c[VEC - 1], -1);
    const T rgt = lane_rot(c[0], 1);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const T l = e > 0 ? c[e - 1] : lft;
        const T r = e < VEC - 1 ? c[e + 1] : rgt;
        const T s = ((l + r) + (ym[e] + yp[e])) + (zm[e] + zp[e]);
        Mx[e] = fma_rn(T(-6), c[e], s) * ih2;
    }
}

// flat7_row for a row split into segments held by several waves: the
// x-neighbours beyond the segment (lane 0's left, lane 63's right) are the
// lane's halo value hx instead of the wrapped-around lanes of its own wave.
// Same arithmetic as flat7_row.
template <typename T, int VEC, int S>
__device__ __forceinline__ void flat7_row_seg(const T (&c)[VEC], const T (&ym)[VEC], const T (&yp)[VEC],
                                              const T (&zm)[VEC], const T (&zp)[VEC], T ih2, T (&Mx)[VEC], T hx) {
#pragma clang fp contract(off)
    T lft = lane_rot(c[VEC - 1], -1);
    T rgt = lane_rot(c[0], 1);
    if constexpr (S > 1) {
        const int lane = threadIdx.x & 63;
        if (lane == 0) lft = hx;
        if (lane == 63) rgt = hx;
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const T l = e > 0 ? c[e - 1] : lft;
        const T r = e < VEC - 1 ? c[e + 1] : rgt;
        const T s = ((l + r) + (ym[e] + yp[e])) + (zm[e] + zp[e]);
        Mx[e] = fma_rn(T(-6), c[e], s) * ih2;
    }
}

// Element of a full row (length S * 64 * VEC) that lane `lane` of the wave
// holding segment `seg` needs beyond its segment: the one before the segment
// for the lower half of the wave (lane 0 uses it), the one after it for the
// upper half (lane 63 uses it).  Periodic in x.
template <int VEC, int S>
__device__ __forceinline__ int seg_halo(int seg, int lane) {
    constexpr int NR = 64 * VEC, NF = NR * S;
    return lane < 32 ? (seg * NR - 1) & (NF - 1) : ((seg + 1) * NR) & (NF - 1);
}

// The coarse rows the trilinear prolongation of fine row (y, z) reads (VEC >= 2):
// (Y, Z), and (Y+1, Z), (Y, Z+1), (Y+1, Z+1) where y, z are odd; loaded raw so
// that a prefetch is not waited for until the values are combined.
// VEC == 1 (64^3): lane l holds fine x = l, i.e. coarse X = l / 2, and reads
// the coarse values X and X + 1 of each row itself.
template <typename T, int VEC>
struct CoarseRows {
    T t00[VEC / 2], t01[VEC / 2], t10[VEC / 2], t11[VEC / 2];
};
template <typename T>
struct CoarseRows<T, 1> {
    T a, a1, b0, b1, c0, c1, d0, d1;  // rows (Y, Z), (Y+1, Z), (Y, Z+1), (Y+1, Z+1) at X, X + 1
};
template <typename T, int VEC>
__device__ __forceinline__ void coarse_load(CoarseRows<T, VEC>& c, const T* e, const RowGrid& gc, int y, int z,
                                            int lane) {
    const int Y = y >> 1, Z = z >> 1, oy = y & 1, oz = z & 1;
    if constexpr (VEC == 1) {
        const int X = lane >> 1, ox = lane & 1, m = gc.mask;
        const T* r0 = e + gc.row(Y, Z);
        c.a = r0[X & m];
        if (ox) c.a1 = r0[(X + 1) & m];
        if (oy) {
            const T* r1 = e + gc.row(Y + 1, Z);
            c.b0 = r1[X & m];
            if (ox) c.b1 = r1[(X + 1) & m];
        }
        if (oz) {
            const T* r2 = e + gc.row(Y, Z + 1);
            c.c0 = r2[X & m];
            if (ox) c.c1 = r2[(X + 1) & m];
            if (oy) {
                const T* r3 = e + gc.row(Y + 1, Z + 1);
                c.d0 = r3[X & m];
                if (ox) c.d1 = r3[(X + 1) & m];
            }
        }
    } else {
        constexpr int CV = VEC / 2;
        const size_t off = (size_t)lane * CV;
        ldrow<T, CV>(c.t00, e + gc.row(Y, Z) + off);
        if (oy) ldrow<T, CV>(c.t01, e + gc.row(Y + 1, Z) + off);
        if (oz) ldrow<T, CV>(c.t10, e + gc.row(Y, Z + 1) + off);
        if (oy && oz) ldrow<T, CV>(c.t11, e + gc.row(Y + 1, Z + 1) + off);
    }
}
// xv += P e on fine row (y, z): interpolate in y, then z, then x (the x + 1
// coarse value from the next lane).  Rounding written out: every kernel that
// prolongs (the prolongation kernel, the fused post-smoothing pass) gets the
// same bits.
template <typename T, int VEC>
__device__ __forceinline__ void prolong_add(T (&xv)[VEC], const CoarseRows<T, VEC>& c, int y, int z) {
#pragma clang fp contract(off)
    const int oy = y & 1, oz = z & 1;
    if constexpr (VEC == 1) {  // interpolate in x, then y, then z
        const int ox = threadIdx.x & 1;
        T v = ox ? T(0.5) * (c.a + c.a1) : c.a;
        if (oy) v = T(0.5) * (v + (ox ? T(0.5) * (c.b0 + c.b1) : c.b0));
        if (oz) {
            T u = ox ? T(0.5) * (c.c0 + c.c1) : c.c0;
            if (oy) u = T(0.5) * (u + (ox ? T(0.5) * (c.d0 + c.d1) : c.d0));
            v = T(0.5) * (v + u);
        }
        xv[0] = xv[0] + v;
    } else {
        constexpr int CV = VEC / 2, CW = CV + 1;
        T w[CW];
        auto seg = [&](const T (&t)[CV], int q) { return q < CV ? t[q] : lane_rot(t[0], 1); };
#pragma unroll
        for (int q = 0; q < CW; ++q) {
            const T r00 = seg(c.t00, q);
            T a0 = r00;
            if (oy) a0 = T(0.5) * (r00 + seg(c.t01, q));
            if (oz) {
                const T r10 = seg(c.t10, q);
                const T a1 = oy ? T(0.5) * (r10 + seg(c.t11, q)) : r10;
                a0 = T(0.5) * (a0 + a1);
            }
            w[q] = a0;
        }
#pragma unroll
        for (int q = 0; q < CV; ++q) {
            xv[2 * q] = xv[2 * q] + w[q];
            xv[2 * q + 1] = xv[2 * q + 1] + T(0.5) * (w[q] + w[q + 1]);
        }
    }
}

// The coarse rows of fine row (y, z) for a row split into S segments of
// 64 VEC points, one per wave (VEC >= 2): the segment's VEC / 2 coarse values
// per lane of each row, and the first coarse value after the segment
// (periodic), which lane 63 needs where an unsplit row takes it from the
// next lane.
template <typename T, int VEC>
struct CoarseSeg {
    CoarseRows<T, VEC> r;
    T h00, h01, h10, h11;
};
template <typename T, int VEC>
__device__ __forceinline__ void coarse_load_seg(CoarseSeg<T, VEC>& c, const T* e, const RowGrid& gc, int y, int z,
                                                int seg, int lane) {
    constexpr int CV = VEC / 2, NC = 32 * VEC;  // coarse values per lane and per segment
    const int Y = y >> 1, Z = z >> 1, oy = y & 1, oz = z & 1;
    const size_t off = (size_t)seg * NC + (size_t)lane * CV;
    const int hx = ((seg + 1) * NC) & gc.mask;
    const T* r0 = e + gc.row(Y, Z);
    ldrow<T, CV>(c.r.t00, r0 + off);
    c.h00 = r0[hx];
    if (oy) {
        const T* r1 = e + gc.row(Y + 1, Z);
        ldrow<T, CV>(c.r.t01, r1 + off);
        c.h01 = r1[hx];
    }
    if (oz) {
        const T* r2 = e + gc.row(Y, Z + 1);
        ldrow<T, CV>(c.r.t10, r2 + off);
        c.h10 = r2[hx];
    }
    if (oy && oz) {
        const T* r3 = e + gc.row(Y + 1, Z + 1);
        ldrow<T, CV>(c.r.t11, r3 + off);
        c.h11 = r3[hx];
    }
}
// prolong_add for a segment: the same interpolation and rounding, with lane
// 63's coarse value after the segment taken from the halo.
template <typename T, int VEC>
__device__ __forceinline__ void prolong_add_seg(T (&xv)[VEC], const CoarseSeg<T, VEC>& c, int y, int z) {
#pragma clang fp contract(off)
    static_assert(VEC >= 2, "two fine points per lane at least");
    const int oy = y & 1, oz = z & 1;
    const bool last = (threadIdx.x & 63) == 63;
    constexpr int CV = VEC / 2, CW = CV + 1;
    T w[CW];
    auto seg = [&](const T (&t)[CV], T h, int q) {
        if (q < CV) return t[q];
        const T r = lane_rot(t[0], 1);
        return last ? h : r;
    };
#pragma unroll
    for (int q = 0; q < CW; ++q) {
        const T r00 = seg(c.r.t00, c.h00, q);
        T a0 = r00;
        if (oy) a0 = T(0.5) * (r00 + seg(c.r.t01, c.h01, q));
        if (oz) {
            const T r10 = seg(c.r.t10, c.h10, q);
            const T a1 = oy ? T(0.5) * (r10 + seg(c.r.t11, c.h11, q)) : r10;
            a0 = T(0.5) * (a0 + a1);
        }
        w[q] = a0;
    }
#pragma unroll
    for (int q = 0; q < CV; ++q) {
        xv[2 * q] = xv[2 * q] + w[q];
        xv[2 * q + 1] = xv[2 * q + 1] + T(0.5) * (w[q] + w[q + 1]);
    }
}

// One smoothing step at a point: x + a (x - xp) + cd (b - M x).
template <typename T>
__device__ __forceinline__ T cheb_step(T x, T xp, T b, T Mx, T a, T cd) {
#pragma clang fp contract(off)
    return fma_rn(cd, b - Mx, fma_rn(a, x - xp, x));
}

// The pointwise first step of a pass from zero, x = cd0 r (cd0 = c0 / D),
// formed in T; with FROMB false, r itself.
template <typename T, bool FROMB>
__device__ __forceinline__ T first_step(T r, T cd0) {
    if constexpr (FROMB) return cd0 * r;
    return r;
}

}  // namespace
}  // namespace mg
