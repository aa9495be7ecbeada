// Single-workgroup V-cycle tail for variable-coefficient hierarchies.
//
// The 19-point levels of 16^3 points and fewer are launch-bound: a visit of
// v steps took 2 v + 3 launches of about 4 us each, whatever the level's
// size.  This kernel runs the whole sub-cycle from the first such level down
// to the dense coarsest solve and back up in one workgroup.
//
// What bounds it is the LDS traffic and the vector instructions of one CU, so
// the layout keeps everything that is not shared between points out of LDS:
//   - 16^3: a thread owns segments of four consecutive x points for the whole
//     kernel.  Their iterate, previous iterate, right-hand side, face
//     coefficients and inverse diagonal stay in registers; LDS holds only the
//     published iterate, read as 16-byte pieces of the 8 neighbour rows.
//   - 8^3: one point per thread, the same way.
//   - the tangential coefficients around a segment are loaded once: into
//     registers in float (40 of the 128 a thread of a 1024-thread block may
//     use), into LDS in double (96 KB), where they do not fit.
// Measured (16^3, 8^3, dense 4^3, degree 3; one launch): 18.6 us in float,
// 27.5 us in double, in place of 19 launches of 74 us (19.2 and 28.5 with the
// residual weighted from 27 reads, the prolongation point by point and the
// coarsest operator loaded where it is applied).  Reading the x
// neighbours as single LDS values at the segments' stride (bank conflicts)
// took 21 and 53 us, and an earlier form that re-read the coefficients from
// L2 in each application was as slow as the launches.  256^3 mixed solve
// 13.5 -> 13.0 ms, 64^3 moving-mesh step 2.5 -> 2.0 ms.
//
// The point formula is that of var_Mu (stencil.h) with the x parts of the
// tangential terms collected; the step multiplies by 1/D where the separate
// kernels divide by D.
#include "var_tail.h"

#include "row.h"

namespace mg {
namespace {

constexpr int kSegs = 1024;  // segments of four points of the 16^3 level
// Float: one segment per thread.  Double: two, in half as many threads, whose
// 256 registers hold the state (128 spilled 53 of them and took 46 us).
template <typename T>
constexpr int tail_threads() { return sizeof(T) == 4 ? kSegs : kSegs / 2; }
constexpr int kP16 = 4096, kP8 = 512, kP4 = 64;

// ---- 16^3: four consecutive x points per thread --------------------------------------
// Thread t holds points 4 (t & 3) .. + 3 of row (y, z) = ((t >> 2) & 15, t >> 6).
// A published field is stored in 16-byte pieces with piece j of every thread
// together, so each 16-byte LDS access of a wave covers consecutive addresses
// (with the plain layout the 32-byte stride of a double segment used half the
// banks).  The x neighbours beyond a segment belong to the next lane of the
// row's four: a rotation inside a quad, one DPP move, instead of an LDS read
// at a 16- or 32-byte stride (a four-way bank conflict).
template <typename T>
struct Seg {
    static constexpr int W = 16 / sizeof(T);  // values per piece
    static constexpr int J = 4 / W;           // pieces per segment
    // LDS element of point i = x + 16 y + 256 z
    __device__ static __forceinline__ int at(int i) {
        if constexpr (J == 1) return i;
        else return ((i >> 1) & 1) * (kP16 / 2) + (i >> 2) * 2 + (i & 1);
    }
};
template <typename T>
__device__ __forceinline__ void get4(T (&v)[4], const T* f, int t) {
    if constexpr (sizeof(T) == 4) {
        const float4 a = *reinterpret_cast<const float4*>(f + 4 * t);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    } else {
        const double2 a = *reinterpret_cast<const double2*>(f + 2 * t);
        const double2 b = *reinterpret_cast<const double2*>(f + kP16 / 2 + 2 * t);
        v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    }
}
template <typename T>
__device__ __forceinline__ void set4(T* f, int t, const T (&v)[4]) {
    if constexpr (sizeof(T) == 4) {
        *reinterpret_cast<float4*>(f + 4 * t) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
        *reinterpret_cast<double2*>(f + 2 * t) = make_double2(v[0], v[1]);
        *reinterpret_cast<double2*>(f + kP16 / 2 + 2 * t) = make_double2(v[2], v[3]);
    }
}
// the segment of thread t in a global field (plain layout)
template <typename T>
__device__ __forceinline__ void gget4(T (&v)[4], const T* f, int t) {
    if constexpr (sizeof(T) == 4) {
        get4<T>(v, f, t);
    } else {
        const double2 a = *reinterpret_cast<const double2*>(f + 4 * t);
        const double2 b = *reinterpret_cast<const double2*>(f + 4 * t + 2);
        v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    }
}
template <typename T>
__device__ __forceinline__ void gset4(T* f, int t, const T (&v)[4]) {
    if constexpr (sizeof(T) == 4) {
        set4<T>(f, t, v);
    } else {
        *reinterpret_cast<double2*>(f + 4 * t) = make_double2(v[0], v[1]);
        *reinterpret_cast<double2*>(f + 4 * t + 2) = make_double2(v[2], v[3]);
    }
}

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
// d[e] = v[e + 1] - v[e - 1]
template <typename T>
__device__ __forceinline__ void xdiff(T (&d)[4], const T (&v)[4]) {
    const T l = quad_rot<-1>(v[3]), r = quad_rot<1>(v[0]);
    d[0] = v[1] - l;
    d[1] = v[2] - v[0];
    d[2] = v[3] - v[1];
    d[3] = r - v[2];
}

// threads holding the neighbour segments: (y +- 1, z), (y, z +- 1), the corners
struct Pos16 {
    int p0, m0, op, om, pp, pm, mp, mm;
    __device__ __forceinline__ Pos16(int t) {
        const int q = t & 3, y = (t >> 2) & 15, z = t >> 6;
        const int yp = ((y + 1) & 15) << 2 | q, ym = ((y - 1) & 15) << 2 | q, yo = y << 2 | q;
        const int zp = ((z + 1) & 15) << 6, zm = ((z - 1) & 15) << 6, zo = z << 6;
        p0 = zo | yp; m0 = zo | ym; op = zp | yo; om = zm | yo;
        pp = zp | yp; pm = zm | yp; mp = zp | ym; mm = zm | ym;
    }
};

template <typename T>
struct Faces16 {
    T x[5], ym[4], yp[4], zm[4], zp[4], dinv[4];
};
template <typename T>
__device__ __forceinline__ void faces16(Faces16<T>& f, const T* C, const Pos16& p, int t, T ih2) {
    T q[4], c[4];
    gget4<T>(c, C, t);
    const T l = quad_rot<-1>(c[3]), r = quad_rot<1>(c[0]);
    f.x[0] = T(0.5) * (l + c[0]);
    f.x[4] = T(0.5) * (c[3] + r);
#pragma unroll
    for (int e = 1; e < 4; ++e) f.x[e] = T(0.5) * (c[e - 1] + c[e]);
    gget4<T>(c, C + kP16, t);
    gget4<T>(q, C + kP16, p.p0);
#pragma unroll
    for (int e = 0; e < 4; ++e) f.yp[e] = T(0.5) * (c[e] + q[e]);
    gget4<T>(q, C + kP16, p.m0);
#pragma unroll
    for (int e = 0; e < 4; ++e) f.ym[e] = T(0.5) * (c[e] + q[e]);
    gget4<T>(c, C + 2 * kP16, t);
    gget4<T>(q, C + 2 * kP16, p.op);
#pragma unroll
    for (int e = 0; e < 4; ++e) f.zp[e] = T(0.5) * (c[e] + q[e]);
    gget4<T>(q, C + 2 * kP16, p.om);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        f.zm[e] = T(0.5) * (c[e] + q[e]);
        const T d = ((f.x[e + 1] + f.x[e]) + (f.yp[e] + f.ym[e])) + (f.zp[e] + f.zm[e]);
        f.dinv[e] = T(1) / (-d * ih2);
    }
}

// The tangential coefficients an application reads: C^{xy} on the own row and
// at y +- 1, C^{xz} on the own row and at z +- 1, C^{yz} at y +- 1 and z +- 1.
enum Cross { XY0, XYP, XYM, XZ0, XZP, XZM, YZYP, YZYM, YZZP, YZZM, kCross };
template <typename T>
struct RegCross16 {  // in registers
    T v[kCross][4];
    __device__ __forceinline__ void load(const T* Cxy, const T* Cxz, const T* Cyz, const Pos16& p, int t) {
        gget4<T>(v[XY0], Cxy, t);
        gget4<T>(v[XYP], Cxy, p.p0);
        gget4<T>(v[XYM], Cxy, p.m0);
        gget4<T>(v[XZ0], Cxz, t);
        gget4<T>(v[XZP], Cxz, p.op);
        gget4<T>(v[XZM], Cxz, p.om);
        gget4<T>(v[YZYP], Cyz, p.p0);
        gget4<T>(v[YZYM], Cyz, p.m0);
        gget4<T>(v[YZZP], Cyz, p.op);
        gget4<T>(v[YZZM], Cyz, p.om);
    }
    template <int K>
    __device__ __forceinline__ void get(T (&o)[4], int) const {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = v[K][e];
    }
};
template <typename T>
struct LdsCross16 {  // in LDS, the three fields one after the other
    const T* f;
    template <int K>
    __device__ __forceinline__ void get(T (&o)[4], int t) const {
        get4<T>(o, f + (K < XZ0 ? 0 : K < YZYP ? kP16 : 2 * kP16), t);
    }
};

// M u at the thread's four points; c = u there, u = the published field.  The
// x part of the tangential terms is taken as the central difference of
// g = C^{xy} (u_{y+1} - u_{y-1}) + C^{xz} (u_{z+1} - u_{z-1}).
template <typename T, typename X>
__device__ __forceinline__ void Mu16(const T* u, const Pos16& p, int t, const T (&c)[4], const Faces16<T>& f,
                                     const X& cross, T ih2, T (&Mu)[4]) {
    constexpr bool SPLIT = sizeof(T) == 8;  // keep the blocks' loads apart: registers
    T acc[4], cr[4], g[4];
    {
        const T l = quad_rot<-1>(c[3]), r = quad_rot<1>(c[0]);
        T q[5];  // fluxes through the five x faces
        q[0] = f.x[0] * (c[0] - l);
        q[4] = f.x[4] * (r - c[3]);
#pragma unroll
        for (int e = 1; e < 4; ++e) q[e] = f.x[e] * (c[e] - c[e - 1]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = q[e + 1] - q[e];
    }
    {   // y faces, C^{xy}
        T vp[4], vm[4], k[4], d[4];
        get4<T>(vp, u, p.p0);
        get4<T>(vm, u, p.m0);
        cross.template get<XY0>(k, t);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc[e] += f.yp[e] * (vp[e] - c[e]) - f.ym[e] * (c[e] - vm[e]);
            g[e] = k[e] * (vp[e] - vm[e]);
        }
        xdiff<T>(d, vp);
        cross.template get<XYP>(k, p.p0);
#pragma unroll
        for (int e = 0; e < 4; ++e) cr[e] = k[e] * d[e];
        xdiff<T>(d, vm);
        cross.template get<XYM>(k, p.m0);
#pragma unroll
        for (int e = 0; e < 4; ++e) cr[e] -= k[e] * d[e];
    }
    if constexpr (SPLIT) __builtin_amdgcn_sched_barrier(0);
    {   // z faces, C^{xz}
        T vp[4], vm[4], k[4], d[4];
        get4<T>(vp, u, p.op);
        get4<T>(vm, u, p.om);
        cross.template get<XZ0>(k, t);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc[e] += f.zp[e] * (vp[e] - c[e]) - f.zm[e] * (c[e] - vm[e]);
            g[e] += k[e] * (vp[e] - vm[e]);
        }
        xdiff<T>(d, vp);
        cross.template get<XZP>(k, p.op);
#pragma unroll
        for (int e = 0; e < 4; ++e) cr[e] += k[e] * d[e];
        xdiff<T>(d, vm);
        cross.template get<XZM>(k, p.om);
#pragma unroll
        for (int e = 0; e < 4; ++e) cr[e] -= k[e] * d[e];
        xdiff<T>(d, g);
#pragma unroll
        for (int e = 0; e < 4; ++e) cr[e] += d[e];
    }
    if constexpr (SPLIT) __builtin_amdgcn_sched_barrier(0);
    {   // C^{yz}
        T pp[4], pm[4], mp[4], mm[4], k[4];
        get4<T>(pp, u, p.pp);
        get4<T>(pm, u, p.pm);
        get4<T>(mp, u, p.mp);
        get4<T>(mm, u, p.mm);
        cross.template get<YZYP>(k, p.p0);
#pragma unroll
        for (int e = 0; e < 4; ++e) cr[e] += k[e] * (pp[e] - pm[e]);
        cross.template get<YZYM>(k, p.m0);
#pragma unroll
        for (int e = 0; e < 4; ++e) cr[e] -= k[e] * (mp[e] - mm[e]);
        cross.template get<YZZP>(k, p.op);
#pragma unroll
        for (int e = 0; e < 4; ++e) cr[e] += k[e] * (pp[e] - mp[e]);
        cross.template get<YZZM>(k, p.om);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            cr[e] -= k[e] * (pm[e] - mm[e]);
            Mu[e] = (acc[e] + T(0.25) * cr[e]) * ih2;
        }
    }
}

// ---- 8^3: one point per thread of the first 512 ----------------------------------------
struct Pos8 {
    int i, xm, xp, ym, yp, zm, zp;                                          // the point and its face neighbours
    int xpyp, xpym, xmyp, xmym, xpzp, xpzm, xmzp, xmzm, ypzp, ypzm, ymzp, ymzm;  // edge neighbours
    __device__ __forceinline__ Pos8(int t) {
        const int x = t & 7, y = (t >> 3) & 7, z = (t >> 6) & 7;
        auto at = [](int xx, int yy, int zz) { return ((zz & 7) * 8 + (yy & 7)) * 8 + (xx & 7); };
        i = at(x, y, z);
        xm = at(x - 1, y, z); xp = at(x + 1, y, z);
        ym = at(x, y - 1, z); yp = at(x, y + 1, z);
        zm = at(x, y, z - 1); zp = at(x, y, z + 1);
        xpyp = at(x + 1, y + 1, z); xpym = at(x + 1, y - 1, z); xmyp = at(x - 1, y + 1, z); xmym = at(x - 1, y - 1, z);
        xpzp = at(x + 1, y, z + 1); xpzm = at(x + 1, y, z - 1); xmzp = at(x - 1, y, z + 1); xmzm = at(x - 1, y, z - 1);
        ypzp = at(x, y + 1, z + 1); ypzm = at(x, y + 1, z - 1); ymzp = at(x, y - 1, z + 1); ymzm = at(x, y - 1, z - 1);
    }
};
template <typename T>
struct Faces8 {
    T xm, xp, ym, yp, zm, zp, dinv;
};
template <typename T>
struct Cross8 {
    T xy[4], xz[4], yz[4];  // at +a, -a, +b, -b of the pair (a, b)
    __device__ __forceinline__ void load(const T* Cxy, const T* Cxz, const T* Cyz, const Pos8& p) {
        xy[0] = Cxy[p.xp]; xy[1] = Cxy[p.xm]; xy[2] = Cxy[p.yp]; xy[3] = Cxy[p.ym];
        xz[0] = Cxz[p.xp]; xz[1] = Cxz[p.xm]; xz[2] = Cxz[p.zp]; xz[3] = Cxz[p.zm];
        yz[0] = Cyz[p.yp]; yz[1] = Cyz[p.ym]; yz[2] = Cyz[p.zp]; yz[3] = Cyz[p.zm];
    }
};
template <typename T>
__device__ __forceinline__ void faces8(Faces8<T>& f, const T* C, const Pos8& p, T ih2) {
    const T cx = C[p.i], cy = C[kP8 + p.i], cz = C[2 * kP8 + p.i];
    f.xm = T(0.5) * (cx + C[p.xm]);
    f.xp = T(0.5) * (cx + C[p.xp]);
    f.ym = T(0.5) * (cy + C[kP8 + p.ym]);
    f.yp = T(0.5) * (cy + C[kP8 + p.yp]);
    f.zm = T(0.5) * (cz + C[2 * kP8 + p.zm]);
    f.zp = T(0.5) * (cz + C[2 * kP8 + p.zp]);
    f.dinv = T(1) / (-(((f.xp + f.xm) + (f.yp + f.ym)) + (f.zp + f.zm)) * ih2);
}
template <typename T>
__device__ __forceinline__ T Mu8(const T* u, const Pos8& p, T c, const Faces8<T>& f, const Cross8<T>& k, T ih2) {
    T acc = f.xp * (u[p.xp] - c) - f.xm * (c - u[p.xm]);
    acc += f.yp * (u[p.yp] - c) - f.ym * (c - u[p.ym]);
    acc += f.zp * (u[p.zp] - c) - f.zm * (c - u[p.zm]);
    T cr;
    {
        const T pp = u[p.xpyp], pm = u[p.xpym], mp = u[p.xmyp], mm = u[p.xmym];
        cr = k.xy[0] * (pp - pm) - k.xy[1] * (mp - mm);
        cr += k.xy[2] * (pp - mp) - k.xy[3] * (pm - mm);
    }
    {
        const T pp = u[p.xpzp], pm = u[p.xpzm], mp = u[p.xmzp], mm = u[p.xmzm];
        cr += k.xz[0] * (pp - pm) - k.xz[1] * (mp - mm);
        cr += k.xz[2] * (pp - mp) - k.xz[3] * (pm - mm);
    }
    {
        const T pp = u[p.ypzp], pm = u[p.ypzm], mp = u[p.ymzp], mm = u[p.ymzm];
        cr += k.yz[0] * (pp - pm) - k.yz[1] * (mp - mm);
        cr += k.yz[2] * (pp - mp) - k.yz[3] * (pm - mm);
    }
    return (acc + T(0.25) * cr) * ih2;
}

// full weighting of the fine field r (2 M points per side) at coarse point i
template <typename T, int M>
__device__ __forceinline__ T weigh(const T* f, int i) {
    constexpr int N = 2 * M;
    auto r = [&](int j) { return f[j]; };
    const int X = i % M, Y = (i / M) % M, Z = i / (M * M);
    T acc = T(0);
#pragma unroll
    for (int dz = -1; dz <= 1; ++dz) {
        T ay = T(0);
#pragma unroll
        for (int dy = -1; dy <= 1; ++dy) {
            const int row = (((2 * Z + dz) & (N - 1)) * N + ((2 * Y + dy) & (N - 1))) * N;
            const T ax = T(0.25) * r(row + ((2 * X - 1) & (N - 1))) + T(0.5) * r(row + 2 * X) +
                         T(0.25) * r(row + 2 * X + 1);
            ay += (dy == 0 ? T(0.5) : T(0.25)) * ax;
        }
        acc += (dz == 0 ? T(0.5) : T(0.25)) * ay;
    }
    return acc;
}

// trilinear interpolation of the coarse field e (M points per side) at fine (x, y, z)
template <typename T, int M>
__device__ __forceinline__ T interp(const T* e, int x, int y, int z) {
    const int X = x >> 1, Y = y >> 1, Z = z >> 1, ox = x & 1, oy = y & 1, oz = z & 1;
    auto line = [&](int YY, int ZZ) {
        const T* p = e + ((ZZ & (M - 1)) * M + (YY & (M - 1))) * M;
        return T(0.5) * (p[X] + p[(X + ox) & (M - 1)]);
    };
    auto plane = [&](int ZZ) { return T(0.5) * (line(Y, ZZ) + line(Y + oy, ZZ)); };
    return T(0.5) * (plane(Z) + plane(Z + oz));
}

// LDS: the published 16^3 iterate (two buffers in float: one barrier a step;
// one in double), then the fields below.
template <typename T>
struct Lds {
    static constexpr bool kReg = sizeof(T) == 4;  // tangential coefficients in registers
    static constexpr int kX16 = kReg ? 2 * kP16 : kP16;
    T x16[kX16];
    T c16[kReg ? 4 : 3 * kP16];
    T x8[2 * kP8];
    T b8[kP8];
    T c8[kReg ? 6 * kP8 : 4];
    T x4[kP4];
    T b4[kP4];
};

template <typename T, bool HAS16, bool DENSE8>
__global__ __launch_bounds__(tail_threads<T>()) void k_var_tail(VarTailArgs<T> A) {
    constexpr bool REG = Lds<T>::kReg;
    constexpr int NT = tail_threads<T>(), NS = kSegs / NT;  // segments of 16^3 per thread
    __shared__ __align__(16) Lds<T> S;
    if (blockIdx.x == 1) {  // the outer sums, beside the tail
        static_assert(sizeof(S.x16) >= kSumLanes * sizeof(double), "the sums fit the tail's LDS");
        finish_sums(A.sums, reinterpret_cast<double*>(S.x16));
        return;
    }
    const int t = threadIdx.x;
    const int steps = A.sched.steps;
    const bool cheb = A.sched.cheb != 0;
    constexpr int L8 = HAS16 ? 1 : 0;  // tail level of 8^3 points
    // Row starts and neighbour indices are formed again in each application
    // from a thread index the compiler cannot see through: kept for the whole
    // kernel they would take the registers of the coefficients.
    auto tid = [&](int s = 0) {
        int v = t + s * NT;
        asm volatile("" : "+v"(v));
        return v;
    };
    T b16[NS][4] = {}, x[NS][4] = {}, xp[NS][4] = {};
    Faces16<T> f16[NS];
    RegCross16<T> k16;
    T b8v = T(0), x8v = T(0), xp8 = T(0);
    Faces8<T> f8;
    Cross8<T> k8;
    const T h16 = HAS16 ? (T)A.ih2[0] : T(0), h8 = (T)A.ih2[L8];
    // everything that the kernel reads from global memory, in flight together
    if constexpr (HAS16) {
        const T* C = A.C[0];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int v = tid(s);
            gget4<T>(b16[s], A.b, v);
            const Pos16 p16(v);
            faces16<T>(f16[s], C, p16, v, h16);
            if constexpr (REG) {
                k16.load(C + 3 * kP16, C + 4 * kP16, C + 5 * kP16, p16, v);
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    T q[4];
                    gget4<T>(q, C + (3 + k) * kP16, v);
                    set4<T>(S.c16 + k * kP16, v, q);
                }
            }
        }
    }
    // the 8^3 level's coefficients wait in LDS in float; in double (no room)
    // they are loaded when the cycle reaches the level
    if constexpr (!DENSE8) {
        if (REG && t < kP8) {
#pragma unroll
            for (int k = 0; k < 6; ++k) S.c8[k * kP8 + t] = A.C[L8][k * kP8 + t];
        }
    }
    // published iterate of the 16^3 level: buf is the one holding it
    int buf = 0;
    auto x16 = [&](int k) { return S.x16 + (REG ? k * kP16 : 0); };
    auto publish16 = [&](const T (&v)[NS][4]) {  // into the free buffer; readable after the barrier
        if constexpr (REG) buf ^= 1;
        else __syncthreads();
#pragma unroll
        for (int s = 0; s < NS; ++s) set4<T>(x16(buf), t + s * NT, v[s]);
        __syncthreads();
    };
    auto M16 = [&](int s, T (&Mu)[4]) {
        const int v = tid(s);
        const Pos16 p16(v);
        if constexpr (REG) Mu16<T>(x16(buf), p16, v, x[s], f16[s], k16, h16, Mu);
        else Mu16<T>(x16(buf), p16, v, x[s], f16[s], LdsCross16<T>{S.c16}, h16, Mu);
        if constexpr (NS > 1) __builtin_amdgcn_sched_barrier(0);
    };
    auto step16 = [&](int k, bool prev) {
        const T a = (T)A.sched.a[0][k], c = (T)A.sched.c[0][k];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            T Mu[4];
            M16(s, Mu);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const T pv = prev ? xp[s][e] : T(0);
                const T n = x[s][e] + a * (x[s][e] - pv) + c * (b16[s][e] - Mu[e]) * f16[s].dinv[e];
                xp[s][e] = x[s][e];
                x[s][e] = n;
            }
        }
    };
    int buf8 = 0;
    auto publish8 = [&](T v) {
        buf8 ^= 1;
        if (t < kP8) S.x8[buf8 * kP8 + t] = v;
        __syncthreads();
    };
    auto M8 = [&]() {
        const T* u = S.x8 + buf8 * kP8;
        const Pos8 p8(tid());
        return Mu8<T>(u, p8, x8v, f8, k8, h8);
    };
    auto step8 = [&](int k, bool prev) {
        const T a = (T)A.sched.a[L8][k], c = (T)A.sched.c[L8][k];
        if (t < kP8) {
            const T n = x8v + a * (x8v - (prev ? xp8 : T(0))) + c * (b8v - M8()) * f8.dinv;
            xp8 = x8v;
            x8v = n;
        }
    };

    // ---------------- down leg
    if constexpr (HAS16) {
        const T c0 = (T)A.sched.c[0][0];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[s][e] = c0 * b16[s][e] * f16[s].dinv[e];
        publish16(x);
        for (int k = 1; k < steps; ++k) {
            step16(k, cheb && k > 1);
            publish16(x);
        }
        T r[NS][4];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            M16(s, r[s]);
#pragma unroll
            for (int e = 0; e < 4; ++e) r[s][e] = b16[s][e] - r[s][e];
        }
        // weighted in x before it is published: [z][y][X], half the values and
        // 9 reads per coarse point instead of 27
        if constexpr (REG) buf ^= 1;
        else __syncthreads();
        T* h = x16(buf);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const T l = quad_rot<-1>(r[s][3]);
            const int v = 2 * (t + s * NT);
            h[v] = T(0.25) * l + T(0.5) * r[s][0] + T(0.25) * r[s][1];
            h[v + 1] = T(0.25) * r[s][1] + T(0.5) * r[s][2] + T(0.25) * r[s][3];
        }
        __syncthreads();
        if (t < kP8) {
            const int X = t & 7, y0 = 2 * ((t >> 3) & 7), z0 = 2 * (t >> 6);
            T acc = T(0);
#pragma unroll
            for (int dz = -1; dz <= 1; ++dz) {
                T ay = T(0);
#pragma unroll
                for (int dy = -1; dy <= 1; ++dy)
                    ay += (dy == 0 ? T(0.5) : T(0.25)) * h[(((z0 + dz) & 15) * 16 + ((y0 + dy) & 15)) * 8 + X];
                acc += (dz == 0 ? T(0.5) : T(0.25)) * ay;
            }
            b8v = acc;
            if constexpr (DENSE8) S.b8[t] = b8v;
        }
    }
    if constexpr (!DENSE8) {
        if constexpr (!HAS16) {
            __syncthreads();
            if (t < kP8) b8v = A.b[t];
        }
        if (t < kP8) {
            const T* C = REG ? S.c8 : A.C[L8];
            const Pos8 p8(tid());
            faces8<T>(f8, C, p8, h8);
            k8.load(C + 3 * kP8, C + 4 * kP8, C + 5 * kP8, p8);
            x8v = (T)A.sched.c[L8][0] * b8v * f8.dinv;
        }
        // the coarsest level's operator, for the end of this leg: each wave forms
        // NR consecutive rows, one column per lane
        constexpr int NR = kP4 / (NT / 64);
        const int w = t >> 6, lane = t & 63;
        double gr[NR];
#pragma unroll
        for (int j = 0; j < NR; ++j) gr[j] = A.G[(NR * w + j) * kP4 + lane];
        publish8(x8v);
        for (int k = 1; k < steps; ++k) {
            step8(k, cheb && k > 1);
            publish8(x8v);
        }
        T r8 = T(0);
        if (t < kP8) r8 = b8v - M8();
        publish8(r8);
        if (t < kP4) S.b4[t] = weigh<T, 4>(S.x8 + buf8 * kP8, t);
        __syncthreads();
        // coarsest: e = G b
        const double rb = (double)S.b4[lane];
        double acc[NR];
#pragma unroll
        for (int j = 0; j < NR; ++j) acc[j] = gr[j] * rb;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
#pragma unroll
            for (int j = 0; j < NR; ++j) acc[j] += __shfl_xor(acc[j], o, 64);
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (lane == j) S.x4[NR * w + j] = (T)acc[j];
        __syncthreads();
        // ---------------- up leg
        if (t < kP8) x8v += interp<T, 4>(S.x4, t & 7, (t >> 3) & 7, t >> 6);
        publish8(x8v);
        for (int k = 0; k < steps; ++k) {
            step8(k, cheb && k > 0);
            if (HAS16 || k + 1 < steps) publish8(x8v);
        }
        if constexpr (!HAS16) {
            if (t < kP8) A.x[t] = x8v;
        }
    } else {
        // coarsest 8^3: G is symmetric, so a thread sums (its part of) column i
        // and the loads of a wave are consecutive
        constexpr int PARTS = NT / kP8, JP = kP8 / PARTS;
        __syncthreads();
        const int i = t & (kP8 - 1), j0 = (t / kP8) * JP;
        const double* g = A.G + (size_t)j0 * kP8 + i;
        double acc = 0.0;
#pragma unroll 16
        for (int j = 0; j < JP; ++j) acc += g[(size_t)j * kP8] * (double)S.b8[j0 + j];
        if constexpr (PARTS > 1) {
            double* part = reinterpret_cast<double*>(S.x16);  // free: the residual was consumed before the barrier
            if (t >= kP8) part[i] = acc;
            __syncthreads();
            if (t < kP8) acc += part[i];
        }
        if (t < kP8) S.x8[buf8 * kP8 + t] = (T)acc;
        __syncthreads();
    }
    if constexpr (HAS16) {
        const T* e = S.x8 + buf8 * kP8;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            // the segment's coarse points 2 q, 2 q + 1, and 2 q + 2 from the next lane
            const int v = t + s * NT, X = 2 * (v & 3), y = (v >> 2) & 15, z = v >> 6;
            const int Y = y >> 1, Z = z >> 1, Y1 = (Y + (y & 1)) & 7, Z1 = (Z + (z & 1)) & 7;
            T a[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                auto at = [&](int yy, int zz) { return e[zz * 64 + yy * 8 + X + j]; };
                a[j] = T(0.5) * (T(0.5) * (at(Y, Z) + at(Y1, Z)) + T(0.5) * (at(Y, Z1) + at(Y1, Z1)));
            }
            const T a2 = quad_rot<1>(a[0]);
            x[s][0] += a[0];
            x[s][1] += T(0.5) * (a[0] + a[1]);
            x[s][2] += a[1];
            x[s][3] += T(0.5) * (a[1] + a2);
        }
        publish16(x);
        for (int k = 0; k < steps; ++k) {
            step16(k, cheb && k > 0);
            if (k + 1 < steps) publish16(x);
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) gset4<T>(A.x, t + s * NT, x[s]);
    }
}

}  // namespace

template <typename T>
hipError_t launch_var_tail(const VarTailArgs<T>& a, hipStream_t s) {
    if (a.nlev < 2 || a.nlev > 3 || a.sched.steps < 1 || a.sched.steps > kTailMaxSteps) return hipErrorInvalidValue;
    const bool dense8 = a.nlev == 2 && a.n[0] == 16 && a.n[1] == 8;
    if (!dense8 && !(a.n[a.nlev - 1] == 4 && var_tail_dense4(a.n[0], a.nlev))) return hipErrorInvalidValue;
    const dim3 grid(a.sums.count > 0 ? 2 : 1);
    if (a.n[0] == 8) hipLaunchKernelGGL((k_var_tail<T, false, false>), grid, dim3(tail_threads<T>()), 0, s, a);
    else if (a.n[a.nlev - 1] == 4) hipLaunchKernelGGL((k_var_tail<T, true, false>), grid, dim3(tail_threads<T>()), 0, s, a);
    else hipLaunchKernelGGL((k_var_tail<T, true, true>), grid, dim3(tail_threads<T>()), 0, s, a);
    return hipGetLastError();
}

template hipError_t launch_var_tail<float>(const VarTailArgs<float>&, hipStream_t);
template hipError_t launch_var_tail<double>(const VarTailArgs<double>&, hipStream_t);

}  // namespace mg
