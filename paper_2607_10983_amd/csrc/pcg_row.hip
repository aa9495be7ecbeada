// The passes of the preconditioned conjugate-gradient solve (pcg.hip) for the
// seven-point operator on rows of 64 points and more.
//
// The passes are bound by the fields they move, so q = M p is not stored: the
// stencil is formed again from p where q is used, and a double hierarchy's
// right-hand side is r itself.
//
//   dots       (r, z), (z, M p_prev)                 reads r, z, p
//   direction  p = z + beta p_prev, (p, M p)         reads z, p_prev; writes p
//   update     phi += alpha p, r -= alpha M p, (r, r) reads phi, p, r; writes phi, r [, r_in]
//
// 11 fields of 8 bytes per iteration in double instead of 14 with q and a
// copy of r.  256^3 double against the passes that store q: direction 211 ->
// 78 us (5.2 TB/s), update 168 -> 130 (5.2), dots 82 -> 95 (4.2), residual
// with its three sums 159 + 27 -> 85.
//
// A block owns an x tile of 64 VEC points of kWaves consecutive rows and
// marches a chunk of planes: a wave keeps its row of u (the field under the
// stencil) at z - 1, z and z + 1 in registers and publishes the centre row in
// LDS, the edge waves the rows outside the block; the rows of the next plane
// are loaded a whole plane ahead.  A tile shorter than the row takes its x
// neighbours from one value beside each end.
#include "pcg_row.h"

#include "flat_rows.h"
#include "kernels.h"

#include <type_traits>

namespace mg {
namespace {

constexpr int kWaves = 8;      // rows of a block
constexpr int kMaxVec = 4;     // 2 KB of doubles per row tile
static_assert(64 * kMaxVec <= 256, "a tile fits the shortest row that is split into tiles");
constexpr int kMinPlanes = 8;  // shortest chunk
constexpr int kTargetBlocks = 1024;

enum Pass { RESIDUAL, DOTS, DIRECTION, UPDATE };

template <int NS>
__device__ __forceinline__ void store_sums(double (&v)[NS], double* partials, int nb) {
    __shared__ double sh[NS][kWaves];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
        if (lane == 0) sh[k][w] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < NS) {
        double t = 0.0;
        for (int i = 0; i < kWaves; ++i) t += sh[threadIdx.x][i];
        partials[(size_t)threadIdx.x * nb + blockIdx.x] = t;
    }
}

// PREV: there is a p_prev (not in the first iteration after a restart).
template <Pass P, bool PREV, typename TI, int VEC, bool SPLIT>
__global__ __launch_bounds__(64 * kWaves) void k_pcg_row(int n, double ih2, const double* u, const TI* zv,
                                                         const double* b, double* out, double* r, TI* rin, Mean mean,
                                                         const double* scal, double* partials, int nz, int nyb) {
    constexpr int NR = 64 * VEC, S = SPLIT ? 2 : 1;
    constexpr bool HASZ = P == DIRECTION;        // u is z + beta p_prev
    constexpr bool HASU = !HASZ || PREV;
    constexpr bool SAME = std::is_same<TI, double>::value;  // r_in is r
    constexpr int NS = P == RESIDUAL ? 3 : P == DOTS ? 2 : 1;
    __shared__ double rows[2][kWaves + 2][NR];
    const RowGrid g{n, n - 1};
    const int lb = xcd_logical(blockIdx.x, gridDim.x);
    const int tiles = n / NR;
    const int tx = lb % tiles * NR, yb = lb / tiles % nyb, zc = lb / (tiles * nyb);
    const int w = wave_id(), lane = threadIdx.x & 63;
    const int y = yb * kWaves + w, z0 = zc * nz;
    const bool lo = w == 0, hi = w == kWaves - 1;
    const int yh = lo ? y - 1 : y + 1;  // row outside the block (edge waves)
    const size_t off = (size_t)tx + (size_t)lane * VEC;
    const int hx = lane < 32 ? (tx - 1) & g.mask : (tx + NR) & g.mask;
    double beta = 0.0, alpha = 0.0, bmean = 0.0;
    if constexpr (P == DIRECTION && PREV) beta = scal[kPcgBeta];
    if constexpr (P == UPDATE) alpha = scal[kPcgAlpha];
    if constexpr (P == RESIDUAL) bmean = mean.get();

    struct Row {  // a row of u as loaded
        double a[VEC], ah;
        TI z[VEC], zh;
    };
    auto load = [&](Row& q, int yy, int z, bool halo) {
        const size_t i = g.row(yy, z);
        if constexpr (HASU) ldrow<double, VEC>(q.a, u + i + off);
        if constexpr (HASZ) ldrow<TI, VEC>(q.z, zv + i + off);
        if (SPLIT && halo) {
            if constexpr (HASU) q.ah = u[i + hx];
            if constexpr (HASZ) q.zh = zv[i + hx];
        }
    };
    auto form = [&](double (&v)[VEC], double& h, const Row& q, bool halo) {
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            v[e] = !HASZ ? q.a[e] : PREV ? fma_rn(beta, q.a[e], (double)q.z[e]) : (double)q.z[e];
        if (SPLIT && halo) h = !HASZ ? q.ah : PREV ? fma_rn(beta, q.ah, (double)q.zh) : (double)q.zh;
    };
    // rows used with the stencil's result at the same point
    struct Aux {
        double a[VEC], r[VEC];
        TI z[VEC];
    };
    auto load_aux = [&](Aux& q, int z) {
        const size_t i = g.row(y, z) + off;
        if constexpr (P == RESIDUAL) ldrow<double, VEC>(q.a, b + i);
        if constexpr (P == UPDATE) ldrow<double, VEC>(q.a, out + i);
        if constexpr (P == UPDATE || P == DOTS) ldrow<double, VEC>(q.r, r + i);
        if constexpr (P == DOTS) ldrow<TI, VEC>(q.z, zv + i);
    };

    double zm[VEC], c[VEC], zp[VEC], h[VEC] = {}, hc = 0.0, hp = 0.0, unused;
    Aux ax;
    {
        Row q;
        load(q, y, z0 - 1, false);
        form(zm, unused, q, false);
        load(q, y, z0, true);
        form(c, hc, q, true);
        load(q, y, z0 + 1, true);
        form(zp, hp, q, true);
        if (lo || hi) {
            load(q, yh, z0, false);
            form(h, unused, q, false);
        }
        load_aux(ax, z0);
    }
    double sum[NS] = {};
    for (int k = 0; k < nz; ++k) {
        const int z = z0 + k, buf = k & 1;
        const bool more = k + 1 < nz;
        Row qn, qh;
        Aux an;
        if (more) {
            load(qn, y, z + 2, true);
            if (lo || hi) load(qh, yh, z + 1, false);
            load_aux(an, z + 1);
        }
        lds_strow<double, VEC>(rows[buf][w + 1], lane, c);
        if (lo) lds_strow<double, VEC>(rows[buf][0], lane, h);
        if (hi) lds_strow<double, VEC>(rows[buf][kWaves + 1], lane, h);
        __syncthreads();
        double ym[VEC], yp[VEC], Mu[VEC], o[VEC];
        lds_ldrow<double, VEC>(ym, rows[buf][w], lane);
        lds_ldrow<double, VEC>(yp, rows[buf][w + 2], lane);
        flat7_row_seg<double, VEC, S>(c, ym, yp, zm, zp, ih2, Mu, hc);
        const size_t i = g.row(y, z) + off;
        if constexpr (P == DOTS) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                sum[0] += ax.r[e] * (double)ax.z[e];
                sum[1] += (double)ax.z[e] * Mu[e];
            }
        } else if constexpr (P == DIRECTION) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) sum[0] += c[e] * Mu[e];
            strow<double, VEC>(out + i, c);
        } else {
            double res[VEC];
            TI ri[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                if constexpr (P == UPDATE) {
                    o[e] = fma_rn(alpha, c[e], ax.a[e]);
                    res[e] = fma_rn(-alpha, Mu[e], ax.r[e]);
                    sum[0] += res[e] * res[e];
                } else {
                    const double bs = ax.a[e] - bmean;
                    res[e] = bs - Mu[e];
                    sum[0] += bs * bs;
                    sum[1] += res[e] * res[e];
                    sum[2] += c[e];
                }
                ri[e] = (TI)res[e];
            }
            if constexpr (P == UPDATE) strow<double, VEC>(out + i, o);
            strow<double, VEC>(r + i, res);
            if constexpr (!SAME) strow<TI, VEC>(rin + i, ri);
        }
        if (more) {
            copyrow(zm, c);
            copyrow(c, zp);
            hc = hp;
            form(zp, hp, qn, true);
            if (lo || hi) form(h, unused, qh, false);
            ax = an;
        }
    }
    store_sums<NS>(sum, partials, gridDim.x);
}

// (r, z) alone: the first iteration after a restart.
template <typename TI>
__global__ __launch_bounds__(64 * kWaves) void k_pcg_first_dot(size_t per, const double* __restrict__ r,
                                                              const TI* __restrict__ zv, double* partials) {
    double sum[1] = {0.0};
    const size_t i0 = (size_t)blockIdx.x * per;
    for (size_t i = i0 + 2 * threadIdx.x; i < i0 + per; i += 2 * 64 * kWaves) {
        double a[2];
        TI z[2];
        ldrow<double, 2>(a, r + i);
        ldrow<TI, 2>(z, zv + i);
        sum[0] += a[0] * (double)z[0] + a[1] * (double)z[1];
    }
    store_sums<1>(sum, partials, gridDim.x);
}

// Chunks of planes: 1024 blocks where the grid has them (four per CU; the
// chunk's first and last plane are read by two blocks, so not shorter than
// kMinPlanes).
inline int planes(int n) {
    const int rowblocks = n / kWaves * (n > 64 * kMaxVec ? n / (64 * kMaxVec) : 1);
    int nz = n;
    while (nz > kMinPlanes && (long)rowblocks * (n / nz) < kTargetBlocks) nz >>= 1;
    return nz;
}

template <Pass P, bool PREV, typename TI>
hipError_t go(int n, double ih2, const double* u, const TI* z, const double* b, double* out, double* r, TI* rin,
              Mean mean, const double* scal, double* partials, hipStream_t s) {
    const int nz = planes(n);
    const dim3 grid(pcg_row_blocks(n)), block(64 * kWaves);
#define MG_PCG_ROW(VEC, SPLIT)                                                                                       \
    hipLaunchKernelGGL((k_pcg_row<P, PREV, TI, VEC, SPLIT>), grid, block, 0, s, n, ih2, u, z, b, out, r, rin, mean, \
                       scal, partials, nz, n / kWaves)
    switch (n) {
        case 64: MG_PCG_ROW(1, false); break;
        case 128: MG_PCG_ROW(2, false); break;
        case 256:
        case 512:
        case 1024: MG_PCG_ROW(kMaxVec, true); break;
        default: return hipErrorInvalidValue;
    }
#undef MG_PCG_ROW
    return hipGetLastError();
}

}  // namespace

bool pcg_row_applies(int n) { return n >= 64 && n <= 1024 && (n & (n - 1)) == 0; }

int pcg_row_blocks(int n) {
    return n / kWaves * (n > 64 * kMaxVec ? n / (64 * kMaxVec) : 1) * (n / planes(n));
}

template <typename TI>
hipError_t launch_pcg_row_residual(int n, double ih2, const double* phi, const double* b, Mean mean, double* r,
                                   TI* rin, double* partials, hipStream_t s) {
    return go<RESIDUAL, false, TI>(n, ih2, phi, nullptr, b, nullptr, r, rin, mean, nullptr, partials, s);
}

template <typename TI>
hipError_t launch_pcg_row_dots(int n, double ih2, const double* r, const TI* z, const double* p_prev,
                               double* partials, hipStream_t s) {
    if (p_prev)
        return go<DOTS, true, TI>(n, ih2, p_prev, z, nullptr, nullptr, const_cast<double*>(r), nullptr, Mean{},
                                  nullptr, partials, s);
    if (!pcg_row_applies(n)) return hipErrorInvalidValue;
    const int nb = pcg_row_blocks(n);
    hipLaunchKernelGGL((k_pcg_first_dot<TI>), dim3(nb), dim3(64 * kWaves), 0, s, (size_t)n * n * n / nb, r, z,
                       partials);
    return hipGetLastError();
}

template <typename TI>
hipError_t launch_pcg_row_direction(int n, double ih2, const TI* z, const double* p_prev, double* p,
                                    const double* scal, double* partials, hipStream_t s) {
    return p_prev ? go<DIRECTION, true, TI>(n, ih2, p_prev, z, nullptr, p, nullptr, nullptr, Mean{}, scal, partials, s)
                  : go<DIRECTION, false, TI>(n, ih2, nullptr, z, nullptr, p, nullptr, nullptr, Mean{}, scal, partials, s);
}

template <typename TI>
hipError_t launch_pcg_row_update(int n, double ih2, double* phi, const double* p, double* r, TI* rin,
                                 const double* scal, double* partials, hipStream_t s) {
    return go<UPDATE, true, TI>(n, ih2, p, nullptr, nullptr, phi, r, rin, Mean{}, scal, partials, s);
}

#define MG_PCG_INST(TI)                                                                                          \
    template hipError_t launch_pcg_row_residual<TI>(int, double, const double*, const double*, Mean, double*, TI*, \
                                                    double*, hipStream_t);                                       \
    template hipError_t launch_pcg_row_dots<TI>(int, double, const double*, const TI*, const double*, double*,   \
                                                hipStream_t);                                                    \
    template hipError_t launch_pcg_row_direction<TI>(int, double, const TI*, const double*, double*,             \
                                                     const double*, double*, hipStream_t);                       \
    template hipError_t launch_pcg_row_update<TI>(int, double, double*, const double*, double*, TI*,             \
                                                  const double*, double*, hipStream_t);
MG_PCG_INST(float)
MG_PCG_INST(double)
#undef MG_PCG_INST

}  // namespace mg
