// Setup of a variable-coefficient hierarchy on the device.
//
// A moving mesh gets a new context every step, so its setup is on the path of
// every solve.  Each pass here is bound by the coefficients it reads and
// writes (24 or 48 bytes a point), so the passes are few: one copies and
// checks the caller's fields, one bounds the spectrum, one restricts all six
// fields to the next level (in double, with the float copy of a mixed
// hierarchy written beside it).  Counts and bounds go to integer slots by
// atomics (order-independent), so the host reads all levels' results once, at
// the end, instead of waiting per level.  The coarsest dense inverse of a
// definite operator, which the host computed, is a blocked Gauss-Jordan
// elimination in a few launches.
// Creating a 64^3 context takes 0.17 ms with a 4^3 coarsest level and 0.6 ms
// with 8^3; a 256^3 step (geometry in both precisions 283 us, 4.7 TB/s; bounds
// 211 us in double, 3.8 TB/s) 0.7 ms.
//
// Row kernels (levels of 64^3 and more) hold 64 VEC consecutive x points of a
// row per wave; the values beyond a segment come from the neighbouring lanes,
// or, where a row has more than one segment, from one extra element loaded by
// the first and the last lane.
#include "setup.h"

#include "row.h"
#include "stencil.h"

#include <cmath>
#include <cstdint>
#include <type_traits>

namespace mg {
namespace {

constexpr int kRowWaves = 4;

__global__ void k_clear_slots(u64* slots, int count) {
    if ((int)threadIdx.x < count) slots[threadIdx.x] = 0;
}

// add a per-thread count to a slot, one atomic per wave that has any
__device__ __forceinline__ void wave_add(u64* slot, unsigned v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0 && v) atomicAdd(slot, (u64)v);
}
// Maximum of a block of whole waves into a slot (non-negative doubles order
// like their bits).  Atomics on one address take about 10 ns each, so a block
// issues at most one, and none when the slot already holds as much.
__device__ __forceinline__ void block_slot_max(u64* slot, double m) {
    __shared__ double wm[16];
    const int t = threadIdx.x + blockDim.x * threadIdx.y, waves = blockDim.x * blockDim.y / 64;
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    if ((t & 63) == 0) wm[t >> 6] = m;
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < waves; ++w) m = fmax(m, wm[w]);
        const u64 bits = __builtin_bit_cast(u64, m);
        if (m > 0.0 && bits > __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(slot, bits);
    }
}

__device__ __forceinline__ bool cell_ok(const double (&c)[6]) {
    bool ok = true;
#pragma unroll
    for (int k = 0; k < 6; ++k) ok = ok && isfinite(c[k]) && (k >= 3 || c[k] > 0.0);
    return ok;
}

// ---- copy and check ----------------------------------------------------------------
template <typename TS, typename TI, bool OUTER>
__global__ __launch_bounds__(kThreads) void k_coeff_copy(size_t n3, const TS* __restrict__ src, TI* __restrict__ inner,
                                                         double* __restrict__ outer, u64* bad) {
    // two points per thread and iteration: 8- or 16-byte accesses
    typedef TS S2 __attribute__((ext_vector_type(2)));
    typedef TI I2 __attribute__((ext_vector_type(2)));
    typedef double D2 __attribute__((ext_vector_type(2)));
    unsigned nbad = 0;
    for (size_t i = blockIdx.x * (size_t)kThreads + threadIdx.x; i < n3 / 2; i += (size_t)gridDim.x * kThreads) {
        S2 v[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) v[k] = *(reinterpret_cast<const S2*>(src + k * n3) + i);
        double a[6], b[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            a[k] = (double)v[k].x;
            b[k] = (double)v[k].y;
            const I2 w = {(TI)v[k].x, (TI)v[k].y};
            *(reinterpret_cast<I2*>(inner + k * n3) + i) = w;
            if constexpr (OUTER) {
                const D2 d = {a[k], b[k]};
                *(reinterpret_cast<D2*>(outer + k * n3) + i) = d;
            }
        }
        nbad += (cell_ok(a) ? 0u : 1u) + (cell_ok(b) ? 0u : 1u);
    }
    wave_add(bad, nbad);
}

// ---- Gershgorin bound ----------------------------------------------------------------
// c0 and the neighbours of each component at one point -> 1 + sum |M_ij| / |M_ii|
struct BoundPt {
    double xx, xxp, xxm, yy, yyp, yym, zz, zzp, zzm;   // diagonal components at the point and along their axis
    double xyxp, xyxm, xyyp, xyym, xzxp, xzxm, xzzp, xzzm, yzyp, yzym, yzzp, yzzm;
    __device__ __forceinline__ double value() const {
        double face = 0.0;
        face += 0.5 * (xx + xxp) + 0.5 * (xx + xxm);
        face += 0.5 * (yy + yyp) + 0.5 * (yy + yym);
        face += 0.5 * (zz + zzp) + 0.5 * (zz + zzm);
        double edge = 0.0;
        auto pair = [&](double ap, double am, double bp, double bm) {
            edge += fabs(am + bm) * 0.25;
            edge += fabs(am + bp) * 0.25;
            edge += fabs(ap + bm) * 0.25;
            edge += fabs(ap + bp) * 0.25;
        };
        pair(xyxp, xyxm, xyyp, xyym);
        pair(xzxp, xzxm, xzzp, xzzm);
        pair(yzyp, yzym, yzzp, yzzm);
        return 1.0 + (face + edge) / face;
    }
};

template <typename TC>
__global__ __launch_bounds__(kThreads) void k_bound(int n, const TC* __restrict__ C, u64* lmax, int nz) {
    const Grid g{n, n - 1};
    const size_t N = (size_t)n * n * n;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * nz;
    double m = 0.0;
    for (int z = z0; z < z0 + nz; ++z) {
        auto at = [&](int c, int dx, int dy, int dz) { return (double)C[c * N + g(x + dx, y + dy, z + dz)]; };
        const BoundPt p{at(0, 0, 0, 0),  at(0, 1, 0, 0),  at(0, -1, 0, 0), at(1, 0, 0, 0),  at(1, 0, 1, 0),
                        at(1, 0, -1, 0), at(2, 0, 0, 0),  at(2, 0, 0, 1),  at(2, 0, 0, -1), at(3, 1, 0, 0),
                        at(3, -1, 0, 0), at(3, 0, 1, 0),  at(3, 0, -1, 0), at(4, 1, 0, 0),  at(4, -1, 0, 0),
                        at(4, 0, 0, 1),  at(4, 0, 0, -1), at(5, 0, 1, 0),  at(5, 0, -1, 0), at(5, 0, 0, 1),
                        at(5, 0, 0, -1)};
        m = fmax(m, p.value());
    }
    block_slot_max(lmax, m);
}

// A row segment of one field: VEC values per lane, `hl` (lane 0) and `hr`
// (lane 63) the values beyond it when the row has several segments.
template <typename T, int VEC, bool MULTI>
struct SegRow {
    T v[VEC];
    T h;
    __device__ __forceinline__ void load(const T* row, int x, int lane, int n) {
        ldrow<T, VEC>(v, row + x);
        if constexpr (MULTI) {
            h = T(0);
            if (lane == 0) h = row[(x - 1) & (n - 1)];
            if (lane == 63) h = row[(x + VEC) & (n - 1)];
        }
    }
    // p[e] = v[e + 1], m[e] = v[e - 1]
    __device__ __forceinline__ void shifts(T (&p)[VEC], T (&m)[VEC], int lane) const {
        T r = lane_rot(v[0], 1), l = lane_rot(v[VEC - 1], -1);
        if constexpr (MULTI) {
            if (lane == 63) r = h;
            if (lane == 0) l = h;
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            p[e] = e < VEC - 1 ? v[e + 1] : r;
            m[e] = e > 0 ? v[e - 1] : l;
        }
    }
};
template <int VEC>
struct RowPos {
    int x, y, z0, lane, n;
    __device__ __forceinline__ RowPos(int lb, int n_, int nz) : n(n_) {
        const int segs = n / (64 * VEC), nyb = n * segs / kRowWaves;
        const int wv = (lb % nyb) * kRowWaves + wave_id();
        lane = threadIdx.x & 63;
        y = wv / segs;
        x = (wv % segs) * 64 * VEC + lane * VEC;
        z0 = lb / nyb * nz;
    }
    __device__ __forceinline__ size_t row(int dy, int z) const {
        const int m = n - 1;
        return ((size_t)(z & m) * n + ((y + dy) & m)) * n;
    }
};
constexpr int kRowVecMax = 4;
inline int row_vec(int n, int most = kRowVecMax) { return n / 64 < most ? n / 64 : most; }
inline void row_shape(int n, int target, int& nz, int& blocks, int vec) {
    const int per = n / (64 * vec) * n / kRowWaves;  // blocks of a plane
    nz = n;
    while (nz > 4 && (long)per * (n / nz) < target) nz >>= 1;
    blocks = per * (n / nz);
}

// The z rows of C^{zz}, C^{xz}, C^{yz} travel in a register queue, so each row
// of the wave's own y is read once per chunk.
template <typename TC, int VEC, bool MULTI>
__global__ __launch_bounds__(64 * kRowWaves) void k_bound_row(int n, const TC* __restrict__ C, u64* lmax, int nz) {
    const RowPos<VEC> p(xcd_logical(blockIdx.x, gridDim.x), n, nz);
    const size_t N = (size_t)n * n * n;
    const int lane = p.lane;
    typedef SegRow<TC, VEC, MULTI> Row;
    Row xz[3];
    TC zz[3][VEC], yz[3][VEC];
    auto queue = [&](int k, int z) {
        const size_t r = p.row(0, z);
        ldrow<TC, VEC>(zz[k], C + 2 * N + r + p.x);
        xz[k].load(C + 4 * N + r, p.x, lane, n);
        ldrow<TC, VEC>(yz[k], C + 5 * N + r + p.x);
    };
    queue(0, p.z0 - 1);
    queue(1, p.z0);
    double m = 0.0;
    for (int k = 0; k < nz; ++k) {
        const int z = p.z0 + k;
        queue(2, z + 1);
        Row xx, xy;
        TC yy[VEC], yyp[VEC], yym[VEC], xyp[VEC], xym[VEC], yzp[VEC], yzm[VEC];
        const size_t r0 = p.row(0, z), rp = p.row(1, z) + p.x, rm = p.row(-1, z) + p.x;
        xx.load(C + r0, p.x, lane, n);
        ldrow<TC, VEC>(yy, C + N + r0 + p.x);
        ldrow<TC, VEC>(yyp, C + N + rp);
        ldrow<TC, VEC>(yym, C + N + rm);
        xy.load(C + 3 * N + r0, p.x, lane, n);
        ldrow<TC, VEC>(xyp, C + 3 * N + rp);
        ldrow<TC, VEC>(xym, C + 3 * N + rm);
        ldrow<TC, VEC>(yzp, C + 5 * N + rp);
        ldrow<TC, VEC>(yzm, C + 5 * N + rm);
        TC xxp[VEC], xxm[VEC], xyxp[VEC], xyxm[VEC], xzxp[VEC], xzxm[VEC];
        xx.shifts(xxp, xxm, lane);
        xy.shifts(xyxp, xyxm, lane);
        xz[1].shifts(xzxp, xzxm, lane);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const BoundPt q{(double)xx.v[e],  (double)xxp[e],     (double)xxm[e],     (double)yy[e],    (double)yyp[e],
                            (double)yym[e],   (double)zz[1][e],   (double)zz[2][e],   (double)zz[0][e], (double)xyxp[e],
                            (double)xyxm[e],  (double)xyp[e],     (double)xym[e],     (double)xzxp[e],  (double)xzxm[e],
                            (double)xz[2].v[e], (double)xz[0].v[e], (double)yzp[e],   (double)yzm[e],   (double)yz[2][e],
                            (double)yz[0][e]};
            m = fmax(m, q.value());
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            xz[j] = xz[j + 1];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                zz[j][e] = zz[j + 1][e];
                yz[j][e] = yz[j + 1][e];
            }
        }
    }
    block_slot_max(lmax, m);
}

// ---- restriction of coefficient fields -------------------------------------------------
template <typename TS>
__global__ __launch_bounds__(kThreads) void k_restrict_fields(int n, const TS* __restrict__ src,
                                                              double* __restrict__ dst, float* __restrict__ copy,
                                                              int nz, int chunks) {
    const int nc = n >> 1;
    const Grid g{n, n - 1};
    const Grid gc{nc, nc - 1};
    const int X = blockIdx.x * blockDim.x + threadIdx.x;
    const int Y = blockIdx.y * blockDim.y + threadIdx.y;
    const int comp = blockIdx.z / chunks, Z0 = (blockIdx.z % chunks) * nz;
    const TS* f = src + comp * (size_t)n * n * n;
    const size_t o = comp * (size_t)nc * nc * nc;
    for (int Z = Z0; Z < Z0 + nz; ++Z) {
        double v[3][3][3];
        for (int dz = 0; dz < 3; ++dz)
            for (int dy = 0; dy < 3; ++dy)
                for (int dx = 0; dx < 3; ++dx)
                    v[dz][dy][dx] = (double)f[g(2 * X + dx - 1, 2 * Y + dy - 1, 2 * Z + dz - 1)];
        const double w = fw_pt<double>(v);
        const size_t i = o + gc(X, Y, Z);
        dst[i] = w;
        if (copy) copy[i] = (float)w;
    }
}

// One wave per 64 coarse points of a row: a lane loads its two fine values of
// each of the six new rows of a coarse plane; the weighted plane 2 Z + 1 is
// kept as the next plane's 2 Z - 1.  Sums in the order of fw_pt.  The gather
// form above read 27 values per point (56 us per field at 256^3).
template <typename TS>
__global__ __launch_bounds__(64 * kRowWaves) void k_restrict_fields_row(int n, const TS* __restrict__ src,
                                                                        double* __restrict__ dst,
                                                                        float* __restrict__ copy, int nz, int per) {
#pragma clang fp contract(off)
    typedef TS S2 __attribute__((ext_vector_type(2)));
    const int nc = n >> 1, m = n - 1, segs = nc / 64;
    const int lb = xcd_logical(blockIdx.x, gridDim.x);
    const int wv = (lb % per) * kRowWaves + wave_id();
    const int chunk = lb / per;
    const int chunks = nc / nz;
    const int comp = chunk / chunks, Z0 = (chunk % chunks) * nz;
    const int Y = wv / segs, seg = wv % segs;
    const int lane = threadIdx.x & 63;
    const int X = seg * 64 + lane;
    const TS* f = src + comp * (size_t)n * n * n;
    const size_t o = comp * (size_t)nc * nc * nc;
    auto plane = [&](int z) {  // x- and y-weighted fine plane z
        double ax[3];
        S2 v[3];
        TS h[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const TS* row = f + ((size_t)(z & m) * n + ((2 * Y + d - 1) & m)) * n;
            v[d] = *reinterpret_cast<const S2*>(row + 2 * X);
            h[d] = TS(0);
            if (segs > 1 && lane == 0) h[d] = row[(2 * X - 1) & m];
        }
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            TS l = lane_rot((TS)v[d].y, -1);
            if (segs > 1 && lane == 0) l = h[d];
            ax[d] = (0.25 * (double)l + 0.5 * (double)v[d].x) + 0.25 * (double)v[d].y;
        }
        return (0.25 * ax[0] + 0.5 * ax[1]) + 0.25 * ax[2];
    };
    double lo = plane(2 * Z0 - 1);
    for (int Z = Z0; Z < Z0 + nz; ++Z) {
        const double c = plane(2 * Z), hi = plane(2 * Z + 1);
        const double w = (0.25 * lo + 0.5 * c) + 0.25 * hi;
        lo = hi;
        const size_t i = o + ((size_t)Z * nc + Y) * nc + X;
        dst[i] = w;
        if (copy) copy[i] = (float)w;
    }
}

// ---- geometry ------------------------------------------------------------------------
// C = det(J) J^-1 J^-T and det J of J = I + H
__device__ __forceinline__ double metric(double (&H)[6], double (&C)[6]) {
    H[0] += 1.0; H[1] += 1.0; H[2] += 1.0;
    Sym3 J, K, K2;
    sym_from6(H, J);
    const double det = inv3(J, K);
    mul3(K, K, K2);  // J symmetric: J^-1 J^-T = K K
    C[0] = det * K2.m[0][0];
    C[1] = det * K2.m[1][1];
    C[2] = det * K2.m[2][2];
    C[3] = det * K2.m[0][1];
    C[4] = det * K2.m[0][2];
    C[5] = det * K2.m[1][2];
    return det;
}

template <bool D, bool F>
__global__ __launch_bounds__(kThreads) void k_geometry_fields(int n, double ih2, const double* __restrict__ psi,
                                                              double* __restrict__ Cd, float* __restrict__ Cf,
                                                              double* __restrict__ sqrtg, u64* bad, int nz) {
    const Grid g{n, n - 1};
    const size_t N = (size_t)n * n * n;
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    const int y = blockIdx.y * blockDim.y + threadIdx.y;
    const int z0 = blockIdx.z * nz;
    unsigned nbad = 0;
    for (int z = z0; z < z0 + nz; ++z) {
        double H[6], C[6];
        hess_at(psi, g, x, y, z, ih2, H);
        const double det = metric(H, C);
        const size_t i = g(x, y, z);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            if constexpr (D) Cd[k * N + i] = C[k];
            if constexpr (F) Cf[k * N + i] = (float)C[k];
        }
        if (sqrtg) sqrtg[i] = det;
        nbad += cell_ok(C) ? 0u : 1u;
    }
    if (bad && nbad) atomicAdd(bad, (u64)nbad);  // blocks of the smallest levels are not whole waves
}

// Rows of 64^3 and more: the 3 x 3 (y, z) rows of psi around the wave's row in
// a register queue.  Bound by the 24 to 80 bytes a point it writes; one thread
// per column (19 loads a point through the vector caches) ran at 2.85 TB/s.
template <int VEC, bool MULTI, bool D, bool F>
__global__ __launch_bounds__(64 * kRowWaves) void k_geometry_row(int n, double ih2, const double* __restrict__ psi,
                                                                 double* __restrict__ Cd, float* __restrict__ Cf,
                                                                 double* __restrict__ sqrtg, u64* bad, int nz) {
    const RowPos<VEC> p(xcd_logical(blockIdx.x, gridDim.x), n, nz);
    const size_t N = (size_t)n * n * n;
    const int lane = p.lane;
    typedef SegRow<double, VEC, MULTI> Row;
    Row q[3][3];  // [dy + 1][dz + 1]
    auto plane = [&](int k, int z) {
#pragma unroll
        for (int d = 0; d < 3; ++d) q[d][k].load(psi + p.row(d - 1, z), p.x, lane, n);
    };
    plane(0, p.z0 - 1);
    plane(1, p.z0);
    unsigned nbad = 0;
    for (int k = 0; k < nz; ++k) {
        const int z = p.z0 + k;
        plane(2, z + 1);
        double cp[VEC], cm[VEC], ypp[VEC], ypm[VEC], ymp[VEC], ymm[VEC], zpp[VEC], zpm[VEC], zmp[VEC], zmm[VEC];
        q[1][1].shifts(cp, cm, lane);
        q[2][1].shifts(ypp, ypm, lane);  // psi(y + 1, x +- 1)
        q[0][1].shifts(ymp, ymm, lane);
        q[1][2].shifts(zpp, zpm, lane);  // psi(z + 1, x +- 1)
        q[1][0].shifts(zmp, zmm, lane);
        double out[6][VEC], det[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const double c = q[1][1].v[e];
            double H[6], C[6];
            H[0] = (cp[e] - 2.0 * c + cm[e]) * ih2;
            H[1] = (q[2][1].v[e] - 2.0 * c + q[0][1].v[e]) * ih2;
            H[2] = (q[1][2].v[e] - 2.0 * c + q[1][0].v[e]) * ih2;
            H[3] = (ypp[e] - ymp[e] - ypm[e] + ymm[e]) * 0.25 * ih2;
            H[4] = (zpp[e] - zmp[e] - zpm[e] + zmm[e]) * 0.25 * ih2;
            H[5] = (q[2][2].v[e] - q[2][0].v[e] - q[0][2].v[e] + q[0][0].v[e]) * 0.25 * ih2;
            det[e] = metric(H, C);
#pragma unroll
            for (int f = 0; f < 6; ++f) out[f][e] = C[f];
            nbad += cell_ok(C) ? 0u : 1u;
        }
        const size_t r = p.row(0, z) + p.x;
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            if constexpr (D) strow<double, VEC>(Cd + f * N + r, out[f]);
            if constexpr (F) {
                float o[VEC];
#pragma unroll
                for (int e = 0; e < VEC; ++e) o[e] = (float)out[f][e];
                strow<float, VEC>(Cf + f * N + r, o);
            }
        }
        if (sqrtg) strow<double, VEC>(sqrtg + r, det);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            q[d][0] = q[d][1];
            q[d][1] = q[d][2];
        }
    }
    if (bad) wave_add(bad, nbad);
}

// ---- coarsest dense inverse -----------------------------------------------------------
// Row i of A = M - (s / N) 1 1^T, s the mean of |diag M|.  One block per row.
__global__ __launch_bounds__(kThreads) void k_dense_assemble(int n, double ih2, const double* __restrict__ C,
                                                             double* __restrict__ A) {
    __shared__ double sh[kThreads];
    const int N = n * n * n, i = blockIdx.x;
    const Grid g{n, n - 1};
    double s = 0.0;
    for (int j = threadIdx.x; j < N; j += kThreads)
        s += fabs(var_diag<double, double>(C, N, g, j % n, j / n % n, j / (n * n), ih2));
    const double shift = block_sum(s, sh) / N / N;
    for (int j = threadIdx.x; j < N; j += kThreads) A[(size_t)i * N + j] = -shift;
    __syncthreads();
    const int x = i % n, y = i / n % n, z = i / (n * n);
    double* row = A + (size_t)i * N;
    auto cc = [&](int c, int dx, int dy, int dz) { return C[(size_t)c * N + g(x + dx, y + dy, z + dz)]; };
    // every neighbour is a different entry (n >= 4)
    const int t = threadIdx.x;
    if (t == 0) row[i] += var_diag<double, double>(C, N, g, x, y, z, ih2);
    if (t >= 1 && t <= 6) {
        const int a = (t - 1) >> 1, d = (t & 1) ? 1 : -1;
        const int dx = a == 0 ? d : 0, dy = a == 1 ? d : 0, dz = a == 2 ? d : 0;
        row[g(x + dx, y + dy, z + dz)] += 0.5 * (cc(a, 0, 0, 0) + cc(a, dx, dy, dz)) * ih2;
    }
    if (t >= 64 && t < 76) {
        const int k = (t - 64) >> 2, sa = (t & 1) ? 1 : -1, sb = (t & 2) ? 1 : -1;
        const int a = k == 2 ? 1 : 0, b = k == 0 ? 1 : 2;
        const int ax = a == 0 ? sa : 0, ay = a == 1 ? sa : 0, by = b == 1 ? sb : 0, bz = b == 2 ? sb : 0;
        row[g(x + ax, y + ay + by, z + bz)] += sa * sb * (cc(3 + k, ax, ay, 0) + cc(3 + k, 0, by, bz)) * 0.25 * ih2;
    }
}

// One step of the in-place block inversion, out of place: with the diagonal
// block K (kB rows) and P = A_KK^-1,
//   A_KJ <- P A_KJ,  A_IK <- -A_IK P,  A_IJ <- A_IJ - A_IK P A_KJ,  A_KK <- P.
// Each block forms P and its part of P A_KJ itself and updates one 64 x 64
// tile.  P is eliminated by one wave with a column of A_KK per lane in
// registers; the pivot column comes by scalar broadcasts.  A step takes 30 us
// (bound by the serial pivots), two for 4^3 and 16 for 8^3.
// There is no pivoting: A is negative definite where C is positive definite,
// and then none is needed.  The coefficients are only checked for positive
// diagonal components, so the premise is checked here.  The pivots of a
// symmetric matrix have the signs of its eigenvalues: a step that meets one
// that is positive counts itself in *indefinite, and the caller inverts such a
// matrix with pivoting (a zero or NaN pivot leaves values that are not finite).
constexpr int kB = 32, kT = 64;
__device__ __forceinline__ double lane_bcast(double v, int lane) {
    v2i h = __builtin_bit_cast(v2i, v);
    h.x = __builtin_amdgcn_readlane(h.x, lane);
    h.y = __builtin_amdgcn_readlane(h.y, lane);
    return __builtin_bit_cast(double, h);
}
__global__ __launch_bounds__(kThreads) void k_dense_step(int N, int k, const double* __restrict__ in,
                                                         double* __restrict__ out, u64* indefinite) {
    __shared__ double P[kB][kB + 1], L[kT][kB + 1], U[kB][kT + 1], W[kB][kT + 1];
    const int t = threadIdx.x, k0 = k * kB, I = blockIdx.y * kT, J = blockIdx.x * kT;
    for (int e = t; e < kT * kB; e += kThreads) L[e / kB][e % kB] = in[(size_t)(I + e / kB) * N + k0 + e % kB];
    for (int e = t; e < kB * kT; e += kThreads) U[e / kT][e % kT] = in[(size_t)(k0 + e / kT) * N + J + e % kT];
    if (t < 64) {  // lanes 32 .. 63 repeat the columns of lanes 0 .. 31
        const int j = t & (kB - 1);
        double a[kB];
#pragma unroll
        for (int i = 0; i < kB; ++i) a[i] = in[(size_t)(k0 + i) * N + k0 + j];
        // The pivot row is always a[0]: every update moves its row down by one,
        // so after kB pivots the rows are back in order and the loop needs no
        // unrolling.
        double inv = 1.0 / lane_bcast(a[0], 0);
        int signs = -1;  // of the pivots, and-ed: by the scalar unit, off the serial chain
#pragma unroll 1
        for (int p = 0; p < kB; ++p) {
            const bool own = j == p;
            signs &= __builtin_amdgcn_readlane(__builtin_bit_cast(v2i, a[0]).y, p);
            const double r = own ? inv : a[0] * inv;
            a[0] = (own ? 0.0 : a[1]) - lane_bcast(a[1], p) * r;
            // the next pivot's reciprocal, beside the other rows' updates
            inv = 1.0 / lane_bcast(a[0], (p + 1) & (kB - 1));
#pragma unroll
            for (int i = 2; i < kB; ++i) {
                const double f = lane_bcast(a[i], p);
                a[i - 1] = (own ? 0.0 : a[i]) - f * r;
            }
            a[kB - 1] = r;
        }
        if (t < kB) {
#pragma unroll
            for (int i = 0; i < kB; ++i) P[i][j] = a[i];
        }
        if (t == 0 && signs >= 0 && blockIdx.x + blockIdx.y == 0) atomicAdd(indefinite, (u64)1);
    }
    __syncthreads();
    {   // W = P U, or P itself in the diagonal block's columns: 8 columns per thread
        const int i = t >> 3, j0 = (t & 7) * 8;
        double w[8] = {};
#pragma unroll 4
        for (int q = 0; q < kB; ++q) {
            const double p = P[i][q];
#pragma unroll
            for (int j = 0; j < 8; ++j) w[j] += p * U[q][j0 + j];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int jk = J + j0 + j - k0;
            W[i][j0 + j] = jk >= 0 && jk < kB ? P[i][jk] : w[j];
        }
    }
    __syncthreads();
    // 4 x 4 values of the tile per thread
    const int i0 = (t >> 4) * 4, j0 = (t & 15) * 4;
    double v[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int jk = J + j0 + j - k0;
            v[i][j] = jk >= 0 && jk < kB ? 0.0 : in[(size_t)(I + i0 + i) * N + J + j0 + j];
        }
#pragma unroll 4
    for (int q = 0; q < kB; ++q) {
        double l[4], w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            l[i] = L[i0 + i][q];
            w[i] = W[q][j0 + i];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[i][j] -= l[i] * w[j];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int ik = I + i0 + i - k0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            out[(size_t)(I + i0 + i) * N + J + j0 + j] = ik >= 0 && ik < kB ? W[ik][j0 + j] : v[i][j];
    }
}

// means of the rows and columns of B
__global__ __launch_bounds__(kThreads) void k_dense_means(int N, const double* __restrict__ B, double* __restrict__ rm,
                                                          double* __restrict__ cm) {
    __shared__ double sh[kThreads];
    double r = 0.0, c = 0.0;
    for (int j = threadIdx.x; j < N; j += kThreads) {
        r += B[(size_t)blockIdx.x * N + j];
        c += B[(size_t)j * N + blockIdx.x];
    }
    const double tr = block_sum(r, sh), tc = block_sum(c, sh);
    if (threadIdx.x == 0) {
        rm[blockIdx.x] = tr / N;
        cm[blockIdx.x] = tc / N;
    }
}
// G = P B P with P = I - 1 1^T / N
__global__ __launch_bounds__(kThreads) void k_dense_project(int N, const double* __restrict__ B,
                                                            const double* __restrict__ rm,
                                                            const double* __restrict__ cm, double* __restrict__ G,
                                                            u64* bad) {
    __shared__ double sh[kThreads];
    double s = 0.0;
    for (int j = threadIdx.x; j < N; j += kThreads) s += rm[j];
    const double tm = block_sum(s, sh) / N;
    unsigned nbad = 0;
    for (int j = threadIdx.x; j < N; j += kThreads) {
        const size_t o = (size_t)blockIdx.x * N + j;
        const double v = B[o] - rm[blockIdx.x] - cm[j] + tm;
        G[o] = v;
        nbad += isfinite(v) ? 0u : 1u;
    }
    wave_add(bad, nbad);
}

}  // namespace

// =====================================================================================
// launchers
// =====================================================================================
hipError_t launch_clear_slots(u64* slots, int count, hipStream_t s) {
    if (count > 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_clear_slots, dim3(1), dim3(64), 0, s, slots, count);
    return hipGetLastError();
}

template <typename TS, typename TI>
hipError_t launch_coeff_copy(size_t n3, const TS* src, TI* inner, double* outer, u64* bad, hipStream_t s) {
    size_t blocks = (n3 / 2 + kThreads - 1) / kThreads;
    if (blocks > 8192) blocks = 8192;
    if (outer)
        hipLaunchKernelGGL((k_coeff_copy<TS, TI, true>), dim3((unsigned)blocks), dim3(kThreads), 0, s, n3, src, inner,
                           outer, bad);
    else
        hipLaunchKernelGGL((k_coeff_copy<TS, TI, false>), dim3((unsigned)blocks), dim3(kThreads), 0, s, n3, src, inner,
                           outer, bad);
    return hipGetLastError();
}

// row kernels for n >= 64, VEC = min(n / 64, 4)
#define ROW_VEC(n, ...)                                                                     \
    if ((n) == 64) { constexpr int VEC = 1; constexpr bool MULTI = false; __VA_ARGS__; }    \
    else if ((n) == 128) { constexpr int VEC = 2; constexpr bool MULTI = false; __VA_ARGS__; } \
    else if ((n) == 256) { constexpr int VEC = 4; constexpr bool MULTI = false; __VA_ARGS__; } \
    else { constexpr int VEC = 4; constexpr bool MULTI = true; __VA_ARGS__; }

template <typename TC>
hipError_t launch_bound(int n, const TC* C, u64* lmax, hipStream_t s) {
    if (n >= 64) {
        // 16 bytes of a row per lane: wider double rows left 3 waves per SIMD
        // (256^3: 299 us)
        int nz, blocks;
        if (sizeof(TC) == 8 && n > 128) {
            row_shape(n, 1024, nz, blocks, 2);
            hipLaunchKernelGGL((k_bound_row<TC, 2, true>), dim3(blocks), dim3(64 * kRowWaves), 0, s, n, C, lmax, nz);
            return hipGetLastError();
        }
        row_shape(n, 1024, nz, blocks, row_vec(n));
        ROW_VEC(n, hipLaunchKernelGGL((k_bound_row<TC, VEC, MULTI>), dim3(blocks), dim3(64 * kRowWaves), 0, s, n, C,
                                      lmax, nz))
        return hipGetLastError();
    }
    const Shape sh = stencil_shape(n);
    hipLaunchKernelGGL((k_bound<TC>), sh.grid, sh.block, 0, s, n, C, lmax, sh.nz);
    return hipGetLastError();
}

template <typename TS>
hipError_t launch_restrict_fields(int n, const TS* src, double* dst, float* copy, int ncomp, hipStream_t s) {
    const int nc = n / 2;
    if (nc >= 64) {
        const int per = nc * (nc / 64) / kRowWaves;
        int nz = nc;
        while (nz > 4 && (long)per * (nc / nz) * ncomp < 2048) nz >>= 1;
        hipLaunchKernelGGL((k_restrict_fields_row<TS>), dim3(per * (nc / nz) * ncomp), dim3(64 * kRowWaves), 0, s, n,
                           src, dst, copy, nz, per);
        return hipGetLastError();
    }
    Shape sh = stencil_shape(nc);
    const int chunks = sh.grid.z;
    sh.grid.z *= ncomp;
    hipLaunchKernelGGL((k_restrict_fields<TS>), sh.grid, sh.block, 0, s, n, src, dst, copy, sh.nz, chunks);
    return hipGetLastError();
}

hipError_t launch_geometry_fields(int n, double ih2, const double* psi, double* Cd, float* Cf, double* sqrtg, u64* bad,
                                  hipStream_t s) {
    if (!Cd && !Cf) return hipErrorInvalidValue;
    if (n >= 64) {
        int nz, blocks;
        row_shape(n, 1024, nz, blocks, row_vec(n));
        ROW_VEC(n, {
            const dim3 grid(blocks), block(64 * kRowWaves);
            if (Cd && Cf)
                hipLaunchKernelGGL((k_geometry_row<VEC, MULTI, true, true>), grid, block, 0, s, n, ih2, psi, Cd, Cf,
                                   sqrtg, bad, nz);
            else if (Cd)
                hipLaunchKernelGGL((k_geometry_row<VEC, MULTI, true, false>), grid, block, 0, s, n, ih2, psi, Cd, Cf,
                                   sqrtg, bad, nz);
            else
                hipLaunchKernelGGL((k_geometry_row<VEC, MULTI, false, true>), grid, block, 0, s, n, ih2, psi, Cd, Cf,
                                   sqrtg, bad, nz);
        })
        return hipGetLastError();
    }
    const Shape sh = stencil_shape(n);
    if (Cd && Cf)
        hipLaunchKernelGGL((k_geometry_fields<true, true>), sh.grid, sh.block, 0, s, n, ih2, psi, Cd, Cf, sqrtg, bad,
                           sh.nz);
    else if (Cd)
        hipLaunchKernelGGL((k_geometry_fields<true, false>), sh.grid, sh.block, 0, s, n, ih2, psi, Cd, Cf, sqrtg, bad,
                           sh.nz);
    else
        hipLaunchKernelGGL((k_geometry_fields<false, true>), sh.grid, sh.block, 0, s, n, ih2, psi, Cd, Cf, sqrtg, bad,
                           sh.nz);
    return hipGetLastError();
}

hipError_t launch_dense_inverse(int n, double ih2, const double* C, double* G, double* work, u64* bad,
                                u64* indefinite, hipStream_t s) {
    const int N = n * n * n;
    if (N % kT != 0) return hipErrorInvalidValue;
    double* a = work;
    double* b = work + (size_t)N * N;
    double* rm = work + 2 * (size_t)N * N;
    double* cm = rm + N;
    hipLaunchKernelGGL(k_dense_assemble, dim3(N), dim3(kThreads), 0, s, n, ih2, C, a);
    for (int k = 0; k < N / kB; ++k) {
        hipLaunchKernelGGL(k_dense_step, dim3(N / kT, N / kT), dim3(kThreads), 0, s, N, k, (const double*)a, b,
                           indefinite);
        double* q = a;
        a = b;
        b = q;
    }
    hipLaunchKernelGGL(k_dense_means, dim3(N), dim3(kThreads), 0, s, N, (const double*)a, rm, cm);
    hipLaunchKernelGGL(k_dense_project, dim3(N), dim3(kThreads), 0, s, N, (const double*)a, (const double*)rm,
                       (const double*)cm, G, bad);
    return hipGetLastError();
}

template hipError_t launch_coeff_copy<float, float>(size_t, const float*, float*, double*, u64*, hipStream_t);
template hipError_t launch_coeff_copy<float, double>(size_t, const float*, double*, double*, u64*, hipStream_t);
template hipError_t launch_coeff_copy<double, float>(size_t, const double*, float*, double*, u64*, hipStream_t);
template hipError_t launch_coeff_copy<double, double>(size_t, const double*, double*, double*, u64*, hipStream_t);
template hipError_t launch_bound<float>(int, const float*, u64*, hipStream_t);
template hipError_t launch_bound<double>(int, const double*, u64*, hipStream_t);
template hipError_t launch_restrict_fields<float>(int, const float*, double*, float*, int, hipStream_t);
template hipError_t launch_restrict_fields<double>(int, const double*, double*, float*, int, hipStream_t);

}  // namespace mg
