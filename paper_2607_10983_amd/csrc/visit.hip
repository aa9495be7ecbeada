// Fused level visits for the 32^3 and 64^3 levels of the seven-point hierarchy.
//
// A visit of such a level with v smoothing steps takes 2 v + 3 launches, each
// of them bound by its launch and by one trip to L2, not by its work.  Here it
// takes two:
//
//   pre:  x_1 = c_0 D^-1 b (pointwise), v - 1 further steps, r = b - M x_v,
//         coarse rhs = R r; writes x_v on the tile and the coarse points of it;
//   post: x_0 = x + P e, v steps; writes x_v on the tile.
//
// A workgroup owns a tile and keeps it with a halo as wide as the visit needs
// in LDS (b and two copies of the iterate).  Every application of the operator
// shrinks the valid region by one point per side, so neighbouring tiles
// compute their common halo twice and never wait for each other.
//
// This is the paper's fused wide-halo level visit (one exchange per visit
// instead of one per step), used here to save launches instead of exchanges.
// Every point formula is the shared one of the unfused kernels (stencil.h,
// fma.h), so the result is bitwise that of the separate smoothing, residual,
// restriction and prolongation kernels.
#include "visit.h"

#include "fma.h"
#include "row.h"
#include "stencil.h"

namespace mg {
namespace {

// ---- the 32^3 level: tiles of 8 x 4 x 4 points ------------------------------------
// One tile per CU: what sets the time of a visit is how many points a thread
// handles one after the other.  Degree 3 in float: 3.9 + 4.4 us (pre, post),
// degree 4 in double 5.7 + 6.0 us, where the 8 or 10 launches take 38 us and
// more; with 8 x 8 x 4 tiles (128 workgroups) 4.4 + 4.2 and 6.5 + 6.6 us, with
// whole planes (16 workgroups of 1024 threads, float) 5.1 + 8.5 us.
constexpr int kN = 32;
constexpr int kTX = 8, kTY = 4, kTZ = 4;
constexpr int kThr = 512;

template <typename T>
struct VisitCoef {
    T a[kVisitMaxDegree], cd[kVisitMaxDegree];  // step k: x + a_k (x - x_prev) + cd_k (b - M x)
};

// The tile grown by LO points below and HI points above on each axis, x fastest.
template <int LO, int HI>
struct Region {
    static constexpr int DX = kTX + LO + HI, DY = kTY + LO + HI, DZ = kTZ + LO + HI;
    static constexpr int P = DX * DY * DZ, SY = DX, SZ = DX * DY;
    static constexpr int K = (P + kThr - 1) / kThr;  // points per thread
};

// Point q of the box of X x Y x Z points at (ox, oy, oz) of a region, as its
// index there.
template <typename R, int X, int Y>
__device__ __forceinline__ int box_index(int q, int ox, int oy, int oz) {
    const int k = q / (X * Y), rem = q - k * (X * Y);
    const int j = rem / X, i = rem - j * X;
    return (k + oz) * R::SZ + (j + oy) * R::SY + (i + ox);
}

struct Tile {
    int x, y, z;
};
__device__ __forceinline__ Tile tile_of(int lb) {
    constexpr int nx = kN / kTX, ny = kN / kTY;
    return Tile{lb % nx * kTX, lb / nx % ny * kTY, lb / (nx * ny) * kTZ};
}

// global index of region point p, the region starting LO points below the tile
template <typename R, int LO>
__device__ __forceinline__ int global_index(int p, const Tile& t) {
    const int k = p / R::SZ, rem = p - k * R::SZ;
    const int j = rem / R::DX, i = rem - j * R::DX;
    return (((t.z - LO + k) & (kN - 1)) * kN + ((t.y - LO + j) & (kN - 1))) * kN + ((t.x - LO + i) & (kN - 1));
}

template <typename T, typename R>
__device__ __forceinline__ T M_at(const T* u, int p, T ih2) {
    return flat7_pt<T>(u[p - 1], u[p + 1], u[p - R::SY], u[p + R::SY], u[p - R::SZ], u[p + R::SZ], u[p], ih2);
}

// Steps K .. V - 1 of a pass, step K on the points S layers inside R.  u is
// the current iterate; w holds the previous one (HASP), which the step reads
// only where it writes.  Returns the stack of x_V.
template <typename T, typename R, int V, int K, int S, bool HASP>
__device__ __forceinline__ T* steps_from(T* u, T* w, const T* sb, T ih2, const VisitCoef<T>& coef) {
    if constexpr (K < V) {
        constexpr int X = R::DX - 2 * S, Y = R::DY - 2 * S, Z = R::DZ - 2 * S, P = X * Y * Z;
#pragma unroll
        for (int q0 = 0; q0 < P; q0 += kThr) {
            const int q = q0 + threadIdx.x;
            if (q < P) {
                const int p = box_index<R, X, Y>(q, S, S, S);
                const T xp = HASP ? w[p] : T(0);
                w[p] = step_pt<T>(u[p], xp, sb[p], M_at<T, R>(u, p, ih2), coef.a[K], coef.cd[K]);
            }
        }
        __syncthreads();
        return steps_from<T, R, V, K + 1, S + 1, true>(w, u, sb, ih2, coef);
    } else {
        return u;
    }
}

// x_v of the tile (LO points inside the region) to memory
template <typename T, typename R, int LO>
__device__ __forceinline__ void store_tile(const T* u, T* __restrict__ xout, const Tile& t) {
    if (threadIdx.x < kTX * kTY * kTZ) {
        const int p = box_index<R, kTX, kTY>(threadIdx.x, LO, LO, LO);
        xout[global_index<R, LO>(p, t)] = u[p];
    }
}

template <typename T, int V>
__global__ __launch_bounds__(kThr) void k_visit_pre(const T* __restrict__ b, T* __restrict__ xout,
                                                    T* __restrict__ coarse_b, T ih2, VisitCoef<T> coef) {
    // the residual is needed one point below the tile, x_v one point further
    // and x_1 another V - 1
    constexpr int LO = V + 1, HI = V;
    using R = Region<LO, HI>;
    __shared__ T sb[R::P], su[R::P], sw[R::P];
    const Tile t = tile_of(xcd_logical(blockIdx.x, gridDim.x));
    T bv[R::K];
#pragma unroll
    for (int k = 0; k < R::K; ++k) {
        const int q = threadIdx.x + k * kThr;
        bv[k] = b[global_index<R, LO>(q < R::P ? q : R::P - 1, t)];
    }
#pragma unroll
    for (int k = 0; k < R::K; ++k) {
        const int q = threadIdx.x + k * kThr;
        if (q < R::P) {
            sb[q] = bv[k];
            su[q] = coef.cd[0] * bv[k];
        }
    }
    __syncthreads();
    T* u = steps_from<T, R, V, 1, 1, false>(su, sw, sb, ih2, coef);
    store_tile<T, R, LO>(u, xout, t);
    T* r = u == su ? sw : su;
    constexpr int X = kTX + 1, Y = kTY + 1, Z = kTZ + 1;
#pragma unroll
    for (int q0 = 0; q0 < X * Y * Z; q0 += kThr) {
        const int q = q0 + threadIdx.x;
        if (q < X * Y * Z) {
            const int p = box_index<R, X, Y>(q, LO - 1, LO - 1, LO - 1);
            r[p] = sb[p] - M_at<T, R>(u, p, ih2);
        }
    }
    __syncthreads();
    constexpr int CX = kTX / 2, CY = kTY / 2, CZ = kTZ / 2, M = kN / 2;
    if (threadIdx.x < CX * CY * CZ) {
        const int i = threadIdx.x % CX, j = threadIdx.x / CX % CY, k = threadIdx.x / (CX * CY);
        const T* c = r + (LO + 2 * k) * R::SZ + (LO + 2 * j) * R::SY + (LO + 2 * i);
        T vv[3][3][3];
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
#pragma unroll
            for (int dy = 0; dy < 3; ++dy)
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) vv[dz][dy][dx] = c[(dz - 1) * R::SZ + (dy - 1) * R::SY + (dx - 1)];
        coarse_b[((t.z / 2 + k) * M + t.y / 2 + j) * M + t.x / 2 + i] = fw_pt<T>(vv);
    }
}

template <typename T, int V>
__global__ __launch_bounds__(kThr) void k_visit_post(const T* __restrict__ xin, const T* __restrict__ e,
                                                     const T* __restrict__ b, T* __restrict__ xout, T ih2,
                                                     VisitCoef<T> coef) {
    using R = Region<V, V>;  // x_0
    // the coarse points under R and one more above, from H below the tile's
    constexpr int H = (V + 1) / 2, M = kN / 2;
    constexpr int CX = kTX / 2 + 2 * H + 1, CY = kTY / 2 + 2 * H + 1, CZ = kTZ / 2 + 2 * H + 1, CP = CX * CY * CZ;
    constexpr int CK = (CP + kThr - 1) / kThr;
    __shared__ T sb[R::P], su[R::P], sw[R::P], se[CP];
    const Tile t = tile_of(xcd_logical(blockIdx.x, gridDim.x));
    const int cx = t.x / 2 - H, cy = t.y / 2 - H, cz = t.z / 2 - H;
    T ev[CK], bv[R::K], xv[R::K];
#pragma unroll
    for (int j = 0; j < CK; ++j) {
        const int q = threadIdx.x + j * kThr < CP ? threadIdx.x + j * kThr : CP - 1;
        const int k = q / (CX * CY), rem = q - k * (CX * CY);
        const int y = rem / CX, x = rem - y * CX;
        ev[j] = e[(((cz + k) & (M - 1)) * M + ((cy + y) & (M - 1))) * M + ((cx + x) & (M - 1))];
    }
#pragma unroll
    for (int k = 0; k < R::K; ++k) {
        const int q = threadIdx.x + k * kThr;
        const int gi = global_index<R, V>(q < R::P ? q : R::P - 1, t);
        bv[k] = b[gi];
        xv[k] = xin[gi];
    }
#pragma unroll
    for (int j = 0; j < CK; ++j)
        if (threadIdx.x + j * kThr < CP) se[threadIdx.x + j * kThr] = ev[j];
    __syncthreads();
    // coarse value at (X, Y, Z), unwrapped, within the staged points
    auto ec = [&](int X, int Y, int Z) { return se[((Z - cz) * CY + (Y - cy)) * CX + (X - cx)]; };
#pragma unroll
    for (int k = 0; k < R::K; ++k) {
        const int q = threadIdx.x + k * kThr;
        if (q < R::P) {
            const int z = q / R::SZ, rem = q - z * R::SZ;
            const int y = rem / R::DX, x = rem - y * R::DX;
            sb[q] = bv[k];
            su[q] = add_pt<T>(xv[k], prolong_pt<T>(ec, t.x - V + x, t.y - V + y, t.z - V + z));
        }
    }
    __syncthreads();
    store_tile<T, R, V>(steps_from<T, R, V, 0, 1, false>(su, sw, sb, ih2, coef), xout, t);
}

// step coefficients in the kernels' precision, c_k / D rounded as in the
// single-step launches
template <typename T>
VisitCoef<T> visit_coef(double ih2, const double* a, const double* c, int degree) {
    VisitCoef<T> coef{};
    const double D = -6.0 * ih2;
    for (int k = 0; k < degree; ++k) {
        coef.a[k] = (T)a[k];
        coef.cd[k] = (T)(c[k] / D);
    }
    return coef;
}

// ---- the 64^3 level: tiles of 64 x 8 fine rows -------------------------------------
// Float only.  A workgroup owns coarse plane Z and fine rows y0 .. y0+7 (y0 = 8 t, tile t
// of 8); it keeps the rows y0-4 .. y0+11 (16 x 64 = one point per thread) of
// every plane it needs, and the valid rows shrink by one per side per step
// like the planes.  Point formulas are those of the row kernels of this size:
// the stencil and step of flat7_row / cheb_step (same operation order), the
// restriction in y, then x, then z with fw3 rounding (k_rr_row), the
// prolongation in x, then y, then z (k_prolong_row for one point per lane).
constexpr int kN64 = 64, kTR64 = 8, kHY = 4, kTR = kTR64 + 2 * kHY;  // 16 tile rows
constexpr int kP = kN64 * kTR;  // tile points per plane = threads per workgroup
constexpr int kDeg64Pre = kHY - 1;  // the pre visit's halo covers at most three steps
// b and two iterate stacks, and the three residual planes of the pre visit
// (nine planes of x_1) or the coarse points of the post visit (ten of x_0)
constexpr int kLdsFloats = 32 * kP;

__device__ __forceinline__ int wrap64(int i) { return i & (kN64 - 1); }

// seven-point stencil at (x, row r) of plane p of a tile stack (r +- 1 inside the tile)
__device__ __forceinline__ float M_tile(const float* st, int p, int x, int r, float ih2) {
    const float* c = st + p * kP;
    const float* m = c - kP;
    const float* q = c + kP;
    return flat7_pt<float>(c[r * kN64 + wrap64(x - 1)], c[r * kN64 + wrap64(x + 1)], c[(r - 1) * kN64 + x],
                           c[(r + 1) * kN64 + x], m[r * kN64 + x], q[r * kN64 + x], c[r * kN64 + x], ih2);
}

template <int V>
__global__ __launch_bounds__(kP) void k_visit64_pre(const float* __restrict__ b, float* __restrict__ xout,
                                                    float* __restrict__ coarse_b, float ih2, VisitCoef<float> coef) {
    constexpr int NP = 2 * V + 3;  // planes z0 - 1 - V .. z0 + 1 + V
    __shared__ float lds[kLdsFloats];
    const int t = threadIdx.x;
    const int x = t & (kN64 - 1), r = t >> 6;
    const int Z = blockIdx.x >> 3, tile = blockIdx.x & 7;
    const int z0 = 2 * Z, y0 = kTR64 * tile;
    const int y = wrap64(y0 - kHY + r);
    const int lo = z0 - 1 - V;
    float* sb = lds;
    float* buf[2] = {lds + NP * kP, lds + 2 * NP * kP};
    float* rs = lds + 3 * NP * kP;  // residual on planes z0 - 1 .. z0 + 1
    static_assert(3 * NP * kP + 3 * kP <= kLdsFloats, "pre visit stacks exceed LDS");
    static_assert(V + 1 <= kHY, "the tile halo covers the steps, the residual and the restriction");
    float bv[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) bv[p] = b[((size_t)wrap64(lo + p) * kN64 + y) * kN64 + x];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        sb[p * kP + t] = bv[p];
        buf[0][p * kP + t] = coef.cd[0] * bv[p];
    }
    __syncthreads();
    int cur = 0, prv = -1;
#pragma unroll
    for (int k = 1; k < V; ++k) {  // x_{k+1} on rows k .. 15-k, planes k .. NP-1-k
        const int out = prv >= 0 ? prv : 1;
        if (r >= k && r <= kTR - 1 - k) {
#pragma unroll
            for (int p = k; p <= NP - 1 - k; ++p) {
                const float xc = buf[cur][p * kP + t];
                const float xp = prv >= 0 ? buf[prv][p * kP + t] : 0.0f;
                const float Mx = M_tile(buf[cur], p, x, r, ih2);
                buf[out][p * kP + t] = step_pt<float>(xc, xp, sb[p * kP + t], Mx, coef.a[k], coef.cd[k]);
            }
        }
        __syncthreads();
        prv = cur;
        cur = out;
    }
    // residual on rows 3 .. 11 (fine rows y0-1 .. y0+7), planes V .. V+2
    if (r >= kHY - 1 && r <= kHY + kTR64 - 1) {
#pragma unroll
        for (int p = V; p <= V + 2; ++p) rs[(p - V) * kP + t] = sb[p * kP + t] - M_tile(buf[cur], p, x, r, ih2);
    }
    // the smoothed iterate on the owned rows and planes
    if (r >= kHY && r < kHY + kTR64) {
#pragma unroll
        for (int p = V + 1; p <= V + 2; ++p) xout[((size_t)(lo + p) * kN64 + y) * kN64 + x] = buf[cur][p * kP + t];
    }
    __syncthreads();
    // full weighting onto the tile's 4 coarse rows of coarse plane Z: y, then x, then z
    if (t < (kN64 / 2) * (kTR64 / 2)) {
        const int X = t & (kN64 / 2 - 1), Yl = t >> 5;
        const float* rr = rs;
        float sz[3];
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
            float sx[3];
#pragma unroll
            for (int dx = 0; dx < 3; ++dx) {
                const int xx = wrap64(2 * X + dx - 1);
                const float* col = rr + dz * kP + xx;
                const int r0 = kHY - 1 + 2 * Yl;  // tile row of fine row 2Y - 1
                sx[dx] = fw3<float>(col[r0 * kN64], col[(r0 + 1) * kN64], col[(r0 + 2) * kN64]);
            }
            sz[dz] = fw3<float>(sx[0], sx[1], sx[2]);
        }
        const int Y = y0 / 2 + Yl;
        coarse_b[((size_t)Z * (kN64 / 2) + Y) * (kN64 / 2) + X] = fw3<float>(sz[0], sz[1], sz[2]);
    }
}

template <int V>
__global__ __launch_bounds__(kP) void k_visit64_post(const float* __restrict__ xin, const float* __restrict__ e,
                                                     const float* __restrict__ b, float* __restrict__ xout,
                                                     float ih2, VisitCoef<float> coef) {
    constexpr int NP = 2 * V + 2;              // planes z0 - V .. z0 + 1 + V
    constexpr int NC = 2 * ((V + 1) / 2) + 2;  // coarse planes the prolongation reads
    constexpr int nc = kN64 / 2;
    constexpr int CR = kTR / 2 + 2;            // coarse rows staged: (y0-4)/2 - 1 .. (y0+11)/2 + 1
    __shared__ float lds[kLdsFloats];
    const int t = threadIdx.x;
    const int x = t & (kN64 - 1), r = t >> 6;
    const int Z = blockIdx.x >> 3, tile = blockIdx.x & 7;
    const int z0 = 2 * Z, y0 = kTR64 * tile;
    const int yu = y0 - kHY + r;  // unwrapped fine row (parity and coarse row as for the wrapped one)
    const int y = wrap64(yu);
    const int lo = z0 - V;
    const int zlo = Z - (V + 1) / 2, ylo = (y0 - kHY) / 2 - 1;  // first staged coarse plane / row
    float* sb = lds;
    float* buf[2] = {lds + NP * kP, lds + 2 * NP * kP};
    float* se = lds + 3 * NP * kP;  // coarse planes zlo .. zlo+NC-1, rows ylo .. ylo+CR-1
    static_assert(3 * NP * kP + NC * CR * nc <= kLdsFloats, "post visit stacks exceed LDS");
    static_assert(V <= kHY, "the tile halo covers the steps");
    constexpr int NE = (NC * CR * nc + kP - 1) / kP;
    float ev[NE], bv[NP], xv[NP];
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        const int q = j * kP + t;
        if (q < NC * CR * nc) {
            const int zc = q / (CR * nc), rc = (q / nc) % CR, xc = q % nc;
            ev[j] = e[((size_t)((zlo + zc) & (nc - 1)) * nc + ((ylo + rc) & (nc - 1))) * nc + xc];
        }
    }
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const size_t gi = ((size_t)wrap64(lo + p) * kN64 + y) * kN64 + x;
        bv[p] = b[gi];
        xv[p] = xin[gi];
    }
#pragma unroll
    for (int j = 0; j < NE; ++j)
        if (j * kP + t < NC * CR * nc) se[j * kP + t] = ev[j];
    __syncthreads();
    // coarse value at (X, Y, Zc): Y, Zc unwrapped within the staged block, X periodic
    auto ec = [&](int X, int Y, int Zc) { return se[((Zc - zlo) * CR + (Y - ylo)) * nc + (X & (nc - 1))]; };
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        sb[p * kP + t] = bv[p];
        buf[0][p * kP + t] = add_pt<float>(xv[p], prolong_pt<float>(ec, x, yu, lo + p));
    }
    __syncthreads();
    int cur = 0, prv = -1;
#pragma unroll
    for (int k = 0; k < V; ++k) {  // x_{k+1} on rows k+1 .. 14-k, planes k+1 .. NP-2-k
        const int out = prv >= 0 ? prv : 1;
        if (r >= k + 1 && r <= kTR - 2 - k) {
#pragma unroll
            for (int p = k + 1; p <= NP - 2 - k; ++p) {
                const float xc = buf[cur][p * kP + t];
                const float xp = prv >= 0 ? buf[prv][p * kP + t] : 0.0f;
                const float Mx = M_tile(buf[cur], p, x, r, ih2);
                buf[out][p * kP + t] = step_pt<float>(xc, xp, sb[p * kP + t], Mx, coef.a[k], coef.cd[k]);
            }
        }
        __syncthreads();
        prv = cur;
        cur = out;
    }
    if (r >= kHY && r < kHY + kTR64) {
#pragma unroll
        for (int p = V; p <= V + 1; ++p) xout[((size_t)(lo + p) * kN64 + y) * kN64 + x] = buf[cur][p * kP + t];
    }
}

}  // namespace

// 32^3 in both types, 64^3 in float (tiles of 8 x 8 x 4 points took 7.1 + 9.5
// us there, 64 x 8 rows 5.2 + 6.5; in double, degree 4, two tiles per CU took longer
// than the six launches they replace: 20 us more per cycle).
bool visit_pre_applies(int n, int degree, size_t elem) {
    return degree >= 1 &&
           ((n == kN && degree <= kVisitMaxDegree) || (n == kN64 && elem == sizeof(float) && degree <= kDeg64Pre));
}
bool visit_post_applies(int n, int degree, size_t elem) {
    return degree >= 1 && degree <= kVisitMaxDegree && (n == kN || (n == kN64 && elem == sizeof(float)));
}

template <typename T>
hipError_t launch_visit_pre(int n, double ih2, const T* b, T* xout, T* coarse_b, const double* a, const double* c,
                            int degree, hipStream_t s) {
    if (!visit_pre_applies(n, degree, sizeof(T))) return hipErrorInvalidValue;
    const VisitCoef<T> coef = visit_coef<T>(ih2, a, c, degree);
    if constexpr (sizeof(T) == sizeof(float)) {
        if (n == kN64) {
            const dim3 grid((kN64 / 2) * (kN64 / kTR64)), block(kP);
            switch (degree) {
                case 1: hipLaunchKernelGGL(k_visit64_pre<1>, grid, block, 0, s, b, xout, coarse_b, (T)ih2, coef); break;
                case 2: hipLaunchKernelGGL(k_visit64_pre<2>, grid, block, 0, s, b, xout, coarse_b, (T)ih2, coef); break;
                default: hipLaunchKernelGGL(k_visit64_pre<3>, grid, block, 0, s, b, xout, coarse_b, (T)ih2, coef); break;
            }
            return hipGetLastError();
        }
    }
    const dim3 grid((kN / kTX) * (kN / kTY) * (kN / kTZ)), block(kThr);
    switch (degree) {
        case 1: hipLaunchKernelGGL((k_visit_pre<T, 1>), grid, block, 0, s, b, xout, coarse_b, (T)ih2, coef); break;
        case 2: hipLaunchKernelGGL((k_visit_pre<T, 2>), grid, block, 0, s, b, xout, coarse_b, (T)ih2, coef); break;
        case 3: hipLaunchKernelGGL((k_visit_pre<T, 3>), grid, block, 0, s, b, xout, coarse_b, (T)ih2, coef); break;
        default: hipLaunchKernelGGL((k_visit_pre<T, 4>), grid, block, 0, s, b, xout, coarse_b, (T)ih2, coef); break;
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_visit_post(int n, double ih2, const T* xin, const T* e, const T* b, T* xout, const double* a,
                             const double* c, int degree, hipStream_t s) {
    if (!visit_post_applies(n, degree, sizeof(T)) || xout == xin) return hipErrorInvalidValue;
    const VisitCoef<T> coef = visit_coef<T>(ih2, a, c, degree);
    if constexpr (sizeof(T) == sizeof(float)) {
        if (n == kN64) {
            const dim3 grid((kN64 / 2) * (kN64 / kTR64)), block(kP);
            switch (degree) {
                case 1: hipLaunchKernelGGL(k_visit64_post<1>, grid, block, 0, s, xin, e, b, xout, (T)ih2, coef); break;
                case 2: hipLaunchKernelGGL(k_visit64_post<2>, grid, block, 0, s, xin, e, b, xout, (T)ih2, coef); break;
                case 3: hipLaunchKernelGGL(k_visit64_post<3>, grid, block, 0, s, xin, e, b, xout, (T)ih2, coef); break;
                default: hipLaunchKernelGGL(k_visit64_post<4>, grid, block, 0, s, xin, e, b, xout, (T)ih2, coef); break;
            }
            return hipGetLastError();
        }
    }
    const dim3 grid((kN / kTX) * (kN / kTY) * (kN / kTZ)), block(kThr);
    switch (degree) {
        case 1: hipLaunchKernelGGL((k_visit_post<T, 1>), grid, block, 0, s, xin, e, b, xout, (T)ih2, coef); break;
        case 2: hipLaunchKernelGGL((k_visit_post<T, 2>), grid, block, 0, s, xin, e, b, xout, (T)ih2, coef); break;
        case 3: hipLaunchKernelGGL((k_visit_post<T, 3>), grid, block, 0, s, xin, e, b, xout, (T)ih2, coef); break;
        default: hipLaunchKernelGGL((k_visit_post<T, 4>), grid, block, 0, s, xin, e, b, xout, (T)ih2, coef); break;
    }
    return hipGetLastError();
}

#define MG_VISIT_INST(T)                                                                                             \
    template hipError_t launch_visit_pre<T>(int, double, const T*, T*, T*, const double*, const double*, int,        \
                                            hipStream_t);                                                            \
    template hipError_t launch_visit_post<T>(int, double, const T*, const T*, const T*, T*, const double*,           \
                                             const double*, int, hipStream_t);
MG_VISIT_INST(float)
MG_VISIT_INST(double)
#undef MG_VISIT_INST

}  // namespace mg
