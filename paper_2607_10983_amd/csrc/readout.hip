// Initial guesses for the next solve and the force readout after a solve.
//
// combine3: the predictors of successive solves are linear combinations of
// earlier solutions (recycling, growth scaling, linear and quadratic
// extrapolation), one streaming pass of 8 bytes per term plus 8 written.
//
// accel: the acceleration -s J^-1 grad phi with the fourth-order central
// difference (u_{-2} - 8 u_{-1} + 8 u_{+1} - u_{+2}) / (12 h) along each axis
// and J = I + Hess psi from the same second-order stencils as the geometry.
// One pass reads phi (and psi) once from HBM.  From 64 points per side a wave
// holds 64 VEC consecutive points of an x-row (VEC at most 4, so longer rows
// are several segments), takes the x-neighbours by rotating cross-lane moves
// (beyond a segment's ends from two extra values of its first and last lane)
// and the z-neighbours from a register queue of its own rows as it marches a
// chunk of planes.  On the uniform mesh the y-neighbour rows are shared by a
// block of eight rows through LDS; on the curvilinear one they come from the
// caches.  Smaller grids use one thread per (x, y) column.
//
// The pass is bound by its 20 (float) or 32 (double) bytes a point: 565 us at
// 512^3 and 3.93 ms at 1024^3 in float (4.7 and 5.5 TB/s).  Whole rows of 8
// and 16 values per lane with cached y-neighbours took 1163 us and 12.1 ms.
#include "kernels.h"
#include "row.h"
#include "stencil.h"

namespace mg {
namespace {

__global__ void k_combine3(size_t count, double c1, const double* phi1, double c2, const double* phi2,
                           double c3, const double* phi3, double* out) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x) {
        double v = c1 * phi1[i];
        if (c2 != 0.0) v += c2 * phi2[i];
        if (c3 != 0.0) v += c3 * phi3[i];
        out[i] = v;
    }
}

__device__ __forceinline__ double d4(const double* __restrict__ u, const Grid& g, int x, int y, int z, int dx,
                                     int dy, int dz, double i12h) {
    return (u[g(x - 2 * dx, y - 2 * dy, z - 2 * dz)] - 8.0 * u[g(x - dx, y - dy, z - dz)] +
            8.0 * u[g(x + dx, y + dy, z + dz)] - u[g(x + 2 * dx, y + 2 * dy, z + 2 * dz)]) *
           i12h;
}

template <typename TO, bool CURV>
__global__ __launch_bounds__(kThreads) void k_accel(int n, double ih2, double i12h, const double* __restrict__ phi,
                                                    const double* __restrict__ psi, double scale,
                                                    TO* __restrict__ a, int nz) {
    const Grid g{n, n - 1};
    const size_t N = (size_t)n * n * n;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * nz;
    for (int z = z0; z < z0 + nz; ++z) {
        const size_t i = g(x, y, z);
        double gx = d4(phi, g, x, y, z, 1, 0, 0, i12h);
        double gy = d4(phi, g, x, y, z, 0, 1, 0, i12h);
        double gz = d4(phi, g, x, y, z, 0, 0, 1, i12h);
        if constexpr (CURV) {
            double H[6];
            hess_at(psi, g, x, y, z, ih2, H);
            H[0] += 1.0; H[1] += 1.0; H[2] += 1.0;
            Sym3 J, K;
            sym_from6(H, J);
            (void)inv3(J, K);
            const double ax = K.m[0][0] * gx + K.m[0][1] * gy + K.m[0][2] * gz;
            const double ay = K.m[1][0] * gx + K.m[1][1] * gy + K.m[1][2] * gz;
            const double az = K.m[2][0] * gx + K.m[2][1] * gy + K.m[2][2] * gz;
            gx = ax; gy = ay; gz = az;
        }
        a[i] = (TO)(-scale * gx);
        a[N + i] = (TO)(-scale * gy);
        a[2 * N + i] = (TO)(-scale * gz);
    }
}

// ---- row-wave force readout ------------------------------------------------------
constexpr int kAccelWaves = 4;

// The two values before a segment (lane 0) or after it (lane 63).
template <int VEC>
__device__ __forceinline__ void ld_ends(double (&h)[2], const double* row, int x, int lane, int n) {
    h[0] = h[1] = 0.0;
    if (lane == 0) {
        h[0] = row[(x - 2) & (n - 1)];
        h[1] = row[(x - 1) & (n - 1)];
    }
    if (lane == 63) {
        h[0] = row[(x + VEC) & (n - 1)];
        h[1] = row[(x + VEC + 1) & (n - 1)];
    }
}
// u shifted by -2, -1, +1, +2 in x along a row held VEC per lane; h: the
// values beyond the segment's ends where a row has several segments.
template <int VEC, bool MULTI>
__device__ __forceinline__ void xshifts(const double (&u)[VEC], const double (&h)[2], int lane, double (&m2)[VEC],
                                        double (&m1)[VEC], double (&p1)[VEC], double (&p2)[VEC]) {
    if constexpr (VEC == 1) {
        m1[0] = lane_rot(u[0], -1);
        m2[0] = lane_rot(m1[0], -1);
        p1[0] = lane_rot(u[0], 1);
        p2[0] = lane_rot(p1[0], 1);
    } else {
        double l1 = lane_rot(u[VEC - 1], -1), l2 = lane_rot(u[VEC - 2], -1);
        double r1 = lane_rot(u[0], 1), r2 = lane_rot(u[1], 1);
        if constexpr (MULTI) {
            if (lane == 0) { l2 = h[0]; l1 = h[1]; }
            if (lane == 63) { r1 = h[0]; r2 = h[1]; }
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            m1[e] = e >= 1 ? u[e - 1] : l1;
            m2[e] = e >= 2 ? u[e - 2] : (e == 1 ? l1 : l2);
            p1[e] = e + 1 < VEC ? u[e + 1] : r1;
            p2[e] = e + 2 < VEC ? u[e + 2] : (e + 1 < VEC ? r1 : r2);
        }
    }
}

// Uniform mesh.  A block of W waves holds one segment of rows y0 .. y0+W-1;
// every wave publishes its row of the current plane, the first and last two
// waves also the block's four halo rows, all loaded a plane ahead.  Two LDS
// planes, one barrier per plane.
constexpr int kAccelRows = 8;
template <typename TO, int VEC, bool MULTI>
__global__ __launch_bounds__(64 * kAccelRows) void k_accel_lds(int side, double i12h, const double* __restrict__ phi,
                                                               double scale, TO* __restrict__ a, int nz, int per) {
    constexpr int W = kAccelRows, NS = 64 * VEC;
    __shared__ double rows[2][W + 4][NS];
    const int n = MULTI ? side : NS;
    const int segs = MULTI ? n / NS : 1, m = n - 1;
    const size_t N = (size_t)n * n * n;
    const int lb = xcd_logical(blockIdx.x, gridDim.x);
    const int w = wave_id(), lane = threadIdx.x & 63;
    const int bp = lb % per, z0 = lb / per * nz;
    const int y0 = bp / segs * W, y = y0 + w;
    const int x = (bp % segs) * NS + lane * VEC;
    auto row = [&](int yy, int z) { return phi + ((size_t)(z & m) * n + (yy & m)) * n; };
    const bool edge = w < 2 || w >= W - 2;
    const int yh = w < 2 ? y0 - 2 + w : y0 + 2 + w, hs = w < 2 ? w : w + 4;  // halo row and its LDS slot
    double q[6][VEC], hr[VEC], hn[VEC], ends[2], endn[2];
#pragma unroll
    for (int k = 0; k < 5; ++k) ldrow<double, VEC>(q[k], row(y, z0 - 2 + k) + x);
    if (edge) ldrow<double, VEC>(hr, row(yh, z0) + x);
    if constexpr (MULTI) ld_ends<VEC>(ends, row(y, z0), x, lane, n);
    for (int k = 0; k < nz; ++k) {
        const int z = z0 + k;
        if (k + 1 < nz) {  // rows of the next planes, one iteration early
            ldrow<double, VEC>(q[5], row(y, z + 3) + x);
            if (edge) ldrow<double, VEC>(hn, row(yh, z + 1) + x);
            if constexpr (MULTI) ld_ends<VEC>(endn, row(y, z + 1), x, lane, n);
        }
        double (*pl)[NS] = rows[z & 1];
        lds_strow<double, VEC>(pl[w + 2], lane, q[2]);
        if (edge) lds_strow<double, VEC>(pl[hs], lane, hr);
        __syncthreads();
        double m2[VEC], m1[VEC], p1[VEC], p2[VEC];
        TO ox[VEC], oy[VEC], oz[VEC];
        xshifts<VEC, MULTI>(q[2], ends, lane, m2, m1, p1, p2);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const double gx = (m2[e] - 8.0 * m1[e] + 8.0 * p1[e] - p2[e]) * i12h;
            const double gz = (q[0][e] - 8.0 * q[1][e] + 8.0 * q[3][e] - q[4][e]) * i12h;
            ox[e] = (TO)(-scale * gx);
            oz[e] = (TO)(-scale * gz);
        }
        lds_ldrow<double, VEC>(m2, pl[w], lane);
        lds_ldrow<double, VEC>(m1, pl[w + 1], lane);
        lds_ldrow<double, VEC>(p1, pl[w + 3], lane);
        lds_ldrow<double, VEC>(p2, pl[w + 4], lane);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const double gy = (m2[e] - 8.0 * m1[e] + 8.0 * p1[e] - p2[e]) * i12h;
            oy[e] = (TO)(-scale * gy);
        }
        const size_t r = ((size_t)z * n + y) * n + x;
        strow<TO, VEC>(a + r, ox);
        strow<TO, VEC>(a + N + r, oy);
        strow<TO, VEC>(a + 2 * N + r, oz);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
#pragma unroll
            for (int j = 0; j < 5; ++j) q[j][e] = q[j + 1][e];
            hr[e] = hn[e];
        }
        ends[0] = endn[0];
        ends[1] = endn[1];
    }
}

// A row of psi: VEC values per lane and, in h, the one before (lane 0) or
// after (lane 63) a segment.
template <int VEC, bool MULTI>
__device__ __forceinline__ void ld_seg(double (&v)[VEC], double& h, const double* row, int x, int lane, int n) {
    ldrow<double, VEC>(v, row + x);
    if constexpr (MULTI) {
        h = 0.0;
        if (lane == 0) h = row[(x - 1) & (n - 1)];
        if (lane == 63) h = row[(x + VEC) & (n - 1)];
    }
}
// u shifted by -1 and +1 in x.
template <int VEC, bool MULTI>
__device__ __forceinline__ void xshift1(const double (&u)[VEC], double h, int lane, double (&m1)[VEC],
                                        double (&p1)[VEC]) {
    double l1 = lane_rot(u[VEC - 1], -1), r1 = lane_rot(u[0], 1);
    if constexpr (MULTI) {
        if (lane == 0) l1 = h;
        if (lane == 63) r1 = h;
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        m1[e] = e >= 1 ? u[e - 1] : l1;
        p1[e] = e + 1 < VEC ? u[e + 1] : r1;
    }
}

// Curvilinear mesh.
template <typename TO, int VEC, bool MULTI>
__global__ __launch_bounds__(64 * kAccelWaves) void k_accel_row(int side, double ih2, double i12h,
                                                                const double* __restrict__ phi,
                                                                const double* __restrict__ psi, double scale,
                                                                TO* __restrict__ a, int nz, int per) {
    constexpr int NS = 64 * VEC;
    // a compile-time size for 64^3 (8.1 -> 7.6 us in float); where a lane holds
    // more values it cost registers (256^3 float 157 -> 192)
    const int n = VEC > 1 ? side : NS;
    const int segs = MULTI ? n / NS : 1, m = n - 1;
    const size_t N = (size_t)n * n * n;
    const int lb = xcd_logical(blockIdx.x, gridDim.x);
    const int wv = lb % per * kAccelWaves + wave_id();
    const int y = wv / segs, z0 = lb / per * nz;
    const int lane = threadIdx.x & 63;
    const int x = (wv % segs) * NS + lane * VEC;
    auto off = [&](int dy, int z) { return ((size_t)(z & m) * n + ((y + dy) & m)) * n; };
    // phi rows of this wave at planes z-2 .. z+2, psi rows at z-1 .. z+1
    double q0[VEC], q1[VEC], q2[VEC], q3[VEC], q4[VEC];
    double s0[VEC], s1[VEC], s2[VEC], h0 = 0, h1 = 0, h2 = 0;
    ldrow<double, VEC>(q0, phi + off(0, z0 - 2) + x);
    ldrow<double, VEC>(q1, phi + off(0, z0 - 1) + x);
    ldrow<double, VEC>(q2, phi + off(0, z0) + x);
    ldrow<double, VEC>(q3, phi + off(0, z0 + 1) + x);
    ld_seg<VEC, MULTI>(s0, h0, psi + off(0, z0 - 1), x, lane, n);
    ld_seg<VEC, MULTI>(s1, h1, psi + off(0, z0), x, lane, n);
    for (int k = 0; k < nz; ++k) {
        const int z = z0 + k;
        double ym2[VEC], ym1[VEC], yp1[VEC], yp2[VEC], ends[2] = {0.0, 0.0};
        ldrow<double, VEC>(q4, phi + off(0, z + 2) + x);
        ldrow<double, VEC>(ym2, phi + off(-2, z) + x);
        ldrow<double, VEC>(ym1, phi + off(-1, z) + x);
        ldrow<double, VEC>(yp1, phi + off(1, z) + x);
        ldrow<double, VEC>(yp2, phi + off(2, z) + x);
        if constexpr (MULTI) ld_ends<VEC>(ends, phi + off(0, z), x, lane, n);
        double m2[VEC], m1[VEC], p1[VEC], p2[VEC];
        xshifts<VEC, MULTI>(q2, ends, lane, m2, m1, p1, p2);
        double gx[VEC], gy[VEC], gz[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            gx[e] = (m2[e] - 8.0 * m1[e] + 8.0 * p1[e] - p2[e]) * i12h;
            gy[e] = (ym2[e] - 8.0 * ym1[e] + 8.0 * yp1[e] - yp2[e]) * i12h;
            gz[e] = (q0[e] - 8.0 * q1[e] + 8.0 * q3[e] - q4[e]) * i12h;
        }
        double tm[VEC], tp[VEC], um[VEC], up[VEC], wm[VEC], wp[VEC], htm = 0, htp = 0;
        ld_seg<VEC, MULTI>(s2, h2, psi + off(0, z + 1), x, lane, n);
        ld_seg<VEC, MULTI>(tm, htm, psi + off(-1, z), x, lane, n);
        ld_seg<VEC, MULTI>(tp, htp, psi + off(1, z), x, lane, n);
        ldrow<double, VEC>(um, psi + off(-1, z - 1) + x);
        ldrow<double, VEC>(up, psi + off(1, z - 1) + x);
        ldrow<double, VEC>(wm, psi + off(-1, z + 1) + x);
        ldrow<double, VEC>(wp, psi + off(1, z + 1) + x);
        double cm[VEC], cp[VEC], tmm[VEC], tmp[VEC], tpm[VEC], tpp[VEC], lm[VEC], lp[VEC], hm[VEC], hp[VEC];
        xshift1<VEC, MULTI>(s1, h1, lane, cm, cp);
        xshift1<VEC, MULTI>(tm, htm, lane, tmm, tmp);
        xshift1<VEC, MULTI>(tp, htp, lane, tpm, tpp);
        xshift1<VEC, MULTI>(s0, h0, lane, lm, lp);
        xshift1<VEC, MULTI>(s2, h2, lane, hm, hp);
        TO ox[VEC], oy[VEC], oz[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const double c = s1[e];
            double H[6];
            H[0] = (cp[e] - 2.0 * c + cm[e]) * ih2;
            H[1] = (tp[e] - 2.0 * c + tm[e]) * ih2;
            H[2] = (s2[e] - 2.0 * c + s0[e]) * ih2;
            H[3] = (tpp[e] - tmp[e] - tpm[e] + tmm[e]) * 0.25 * ih2;
            H[4] = (hp[e] - lp[e] - hm[e] + lm[e]) * 0.25 * ih2;
            H[5] = (wp[e] - up[e] - wm[e] + um[e]) * 0.25 * ih2;
            H[0] += 1.0; H[1] += 1.0; H[2] += 1.0;
            Sym3 J, K;
            sym_from6(H, J);
            (void)inv3(J, K);
            ox[e] = (TO)(-scale * (K.m[0][0] * gx[e] + K.m[0][1] * gy[e] + K.m[0][2] * gz[e]));
            oy[e] = (TO)(-scale * (K.m[1][0] * gx[e] + K.m[1][1] * gy[e] + K.m[1][2] * gz[e]));
            oz[e] = (TO)(-scale * (K.m[2][0] * gx[e] + K.m[2][1] * gy[e] + K.m[2][2] * gz[e]));
        }
        const size_t r = off(0, z) + x;
        strow<TO, VEC>(a + r, ox);
        strow<TO, VEC>(a + N + r, oy);
        strow<TO, VEC>(a + 2 * N + r, oz);
        h0 = h1;
        h1 = h2;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            q0[e] = q1[e]; q1[e] = q2[e]; q2[e] = q3[e]; q3[e] = q4[e];
            s0[e] = s1[e]; s1[e] = s2[e];
        }
    }
}

}  // namespace

hipError_t launch_combine3(size_t count, double c1, const double* phi1, double c2, const double* phi2,
                           double c3, const double* phi3, double* out, hipStream_t s) {
    size_t blocks = (count + kThreads - 1) / kThreads;
    if (blocks > 65536) blocks = 65536;
    if (blocks == 0) blocks = 1;
    hipLaunchKernelGGL(k_combine3, dim3((unsigned)blocks), dim3(kThreads), 0, s, count, c1, phi1, c2, phi2, c3,
                       phi3, out);
    return hipGetLastError();
}

template <typename TO>
hipError_t launch_accel(int n, double h, const double* phi, const double* psi, double scale, TO* a,
                        hipStream_t s) {
    const double ih2 = 1.0 / (h * h), i12h = 1.0 / (12.0 * h);
    if (n >= 64) {
        // segments of VEC = min(n / 64, 4) values per lane; z chunks that give two
        // LDS blocks of eight rows per CU, or about 1024 blocks of four in chunks of
        // at least 8 planes.  The LDS blocks go down to 2 planes: with at least 8
        // the uniform 64^3 readout took 7.0 us in double and 6.2 in float against 4.5
        // and 3.9, 128^3 (4 planes) in float 9.8 against 9.0.
        const int vec = n / 64 < 4 ? n / 64 : 4, rows = psi ? kAccelWaves : kAccelRows;
        const int per = n / (64 * vec) * n / rows;
        int nz = n;
        while (nz > (psi ? 8 : 2) && (long)per * (n / nz) < (psi ? 1024 : 512)) nz >>= 1;
        const dim3 grid(per * (n / nz)), block(64 * rows);
#define MG_ACCEL(VEC, MULTI)                                                                                       \
    do {                                                                                                           \
        if (psi) hipLaunchKernelGGL((k_accel_row<TO, VEC, MULTI>), grid, block, 0, s, n, ih2, i12h, phi, psi,      \
                                    scale, a, nz, per);                                                            \
        else hipLaunchKernelGGL((k_accel_lds<TO, VEC, MULTI>), grid, block, 0, s, n, i12h, phi, scale, a, nz, per); \
    } while (0)
        if (n == 64) MG_ACCEL(1, false);
        else if (n == 128) MG_ACCEL(2, false);
        else if (n == 256) MG_ACCEL(4, false);
        else MG_ACCEL(4, true);
#undef MG_ACCEL
        return hipGetLastError();
    }
    const Shape sh = stencil_shape(n);
    if (psi)
        hipLaunchKernelGGL((k_accel<TO, true>), sh.grid, sh.block, 0, s, n, ih2, i12h, phi, psi, scale, a, sh.nz);
    else
        hipLaunchKernelGGL((k_accel<TO, false>), sh.grid, sh.block, 0, s, n, ih2, i12h, phi, psi, scale, a, sh.nz);
    return hipGetLastError();
}

template hipError_t launch_accel<float>(int, double, const double*, const double*, double, float*, hipStream_t);
template hipError_t launch_accel<double>(int, double, const double*, const double*, double, double*, hipStream_t);

}  // namespace mg
