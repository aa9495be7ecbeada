// Reverse mode of the moving-mesh geometry in one pass.
//
// Per cell the cotangents of C and sqrt(g) give that of the triad,
//   Jbar = t K - d (P + P^T),  P = K G K^2,  t = d <G, K^2> + sqrtgbar d,
// with K = J^-1, d = det J and G the full symmetric cotangent of C (stored
// off-diagonals halved); psibar is the adjoint Hessian stencil applied to
// Jbar.  Jbar (six fields) never leaves the block: a tile of 32 x 8 points
// marches a chunk of planes, forms Jbar on the tile with a halo of one point
// (340 cells for 256 points) into a ring of four LDS planes and applies the
// adjoint one plane behind, one barrier per plane.  psi goes through a ring
// of four planes too, and Cbar and sqrtgbar are loaded a plane ahead.
//
// It moves nine fields (psi, Cbar, sqrtgbar, psibar; 29 us at 128^3) and is
// bound by the FP64 chain of a cell, about 250 dependent operations per plane.
// 128^3: 66 us, in place of 62 + 42 us for two passes through a temporary of
// 6 n^3 doubles, its allocation (about 110 us) and a synchronisation.  Cbar
// loaded before the cells instead of after them made no difference (68 us).
#include "geometry_bwd.h"

#include "stencil.h"

namespace mg {
namespace {

constexpr int kTX = 32, kTY = 8;              // points of a tile
constexpr int kCX = kTX + 2, kCY = kTY + 2;   // cells
constexpr int kPX = kTX + 4, kPY = kTY + 4;   // psi values
constexpr int kC = kCX * kCY, kP = kPX * kPY;
constexpr int kThr = 384;
constexpr int kPK = (kP + kThr - 1) / kThr;   // psi values per thread
static_assert(kC <= kThr, "a cell per thread");

__global__ __launch_bounds__(kThr) void k_geometry_bwd(int n, double ih2, const double* __restrict__ psi,
                                                       const double* __restrict__ Cbar,
                                                       const double* __restrict__ sbar, double* __restrict__ psibar,
                                                       int nz) {
    __shared__ double J[4][6][kC];
    __shared__ double S[4][kP];
    const Grid g{n, n - 1};
    const size_t N = (size_t)n * n * n;
    const int t = threadIdx.x;
    const int x0 = blockIdx.x * kTX, y0 = blockIdx.y * kTY, z0 = blockIdx.z * nz;
    // the thread's cell, its psi value, and the point of threads t < 256
    const bool cell = t < kC;
    const int cq = cell ? t : kC - 1;
    const int cx = cq % kCX, cy = cq / kCX;
    const size_t ci = g(x0 - 1 + cx, y0 - 1 + cy, 0);
    const int ps = (cy + 1) * kPX + cx + 1;
    int pi[kPK];
#pragma unroll
    for (int k = 0; k < kPK; ++k) {
        const int q = t + k * kThr < kP ? t + k * kThr : kP - 1;
        pi[k] = (int)g(x0 - 2 + q % kPX, y0 - 2 + q / kPX, 0);
    }
    const int ox = t % kTX, oy = t / kTX;
    const bool out = t < kTX * kTY && x0 + ox < n && y0 + oy < n;
    const int j0 = (oy + 1) * kCX + ox + 1;
    const size_t plane = (size_t)n * n;
    auto at = [&](int z) { return (size_t)(z & g.mask) * plane; };
    double pv[kPK], cb[6], sb = 0.0;
    auto load_psi = [&](int z) {
#pragma unroll
        for (int k = 0; k < kPK; ++k) pv[k] = psi[at(z) + pi[k]];
    };
    auto put_psi = [&](int z) {
#pragma unroll
        for (int k = 0; k < kPK; ++k)
            if (t + k * kThr < kP) S[z & 3][t + k * kThr] = pv[k];
    };
    auto load_bar = [&](int z) {
#pragma unroll
        for (int c = 0; c < 6; ++c) cb[c] = Cbar[c * N + at(z) + ci];
        if (sbar) sb = sbar[at(z) + ci];
    };
    for (int z = z0 - 2; z <= z0; ++z) {
        load_psi(z);
        put_psi(z);
    }
    load_bar(z0 - 1);
    __syncthreads();
    for (int k = -1; k <= nz; ++k) {  // cells of plane z, points of plane z - 1
        const int z = z0 + k;
        const bool more = k < nz;
        if (more) load_psi(z + 2);
        if (cell) {
            const double *pm = S[(z - 1) & 3] + ps, *pc = S[z & 3] + ps, *pp = S[(z + 1) & 3] + ps;
            double H[6];
            H[0] = (pc[1] - 2.0 * pc[0] + pc[-1]) * ih2 + 1.0;
            H[1] = (pc[kPX] - 2.0 * pc[0] + pc[-kPX]) * ih2 + 1.0;
            H[2] = (pp[0] - 2.0 * pc[0] + pm[0]) * ih2 + 1.0;
            H[3] = (pc[kPX + 1] - pc[-kPX + 1] - pc[kPX - 1] + pc[-kPX - 1]) * 0.25 * ih2;
            H[4] = (pp[1] - pm[1] - pp[-1] + pm[-1]) * 0.25 * ih2;
            H[5] = (pp[kPX] - pm[kPX] - pp[-kPX] + pm[-kPX]) * 0.25 * ih2;
            Sym3 A, K, K2, G, KG, P;
            sym_from6(H, A);
            const double d = inv3(A, K);
            mul3(K, K, K2);
            double gs[6];
#pragma unroll
            for (int c = 0; c < 6; ++c) gs[c] = cb[c] * (c < 3 ? 1.0 : 0.5);
            sym_from6(gs, G);
            double tr = 0.0;
#pragma unroll
            for (int a = 0; a < 3; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b) tr += G.m[a][b] * K2.m[a][b];
            tr *= d;
            if (sbar) tr += sb * d;
            mul3(K, G, KG);
            mul3(KG, K2, P);
            constexpr int pa[6] = {0, 1, 2, 0, 0, 1}, pb[6] = {0, 1, 2, 1, 2, 2};
#pragma unroll
            for (int c = 0; c < 6; ++c) {
                const int a = pa[c], b = pb[c];
                const double jab = tr * K.m[a][b] - d * (P.m[a][b] + P.m[b][a]);
                const double jba = tr * K.m[b][a] - d * (P.m[b][a] + P.m[a][b]);
                J[z & 3][c][t] = c < 3 ? jab : jab + jba;
            }
        }
        if (more) {
            load_bar(z + 1);
            put_psi(z + 2);
        }
        __syncthreads();
        if (k >= 1 && out) {
            const double(*m)[kC] = J[(z - 2) & 3], (*c)[kC] = J[(z - 1) & 3], (*p)[kC] = J[z & 3];
            double acc = (c[0][j0 + 1] - 2.0 * c[0][j0] + c[0][j0 - 1]) * ih2;
            acc += (c[1][j0 + kCX] - 2.0 * c[1][j0] + c[1][j0 - kCX]) * ih2;
            acc += (p[2][j0] - 2.0 * c[2][j0] + m[2][j0]) * ih2;
            acc += (c[3][j0 + kCX + 1] - c[3][j0 - kCX + 1] - c[3][j0 + kCX - 1] + c[3][j0 - kCX - 1]) * 0.25 * ih2;
            acc += (p[4][j0 + 1] - m[4][j0 + 1] - p[4][j0 - 1] + m[4][j0 - 1]) * 0.25 * ih2;
            acc += (p[5][j0 + kCX] - m[5][j0 + kCX] - p[5][j0 - kCX] + m[5][j0 - kCX]) * 0.25 * ih2;
            psibar[at(z - 1) + (size_t)(y0 + oy) * n + x0 + ox] = acc;
        }
    }
}

}  // namespace

hipError_t launch_geometry_bwd(int n, double ih2, const double* psi, const double* Cbar, const double* sbar,
                               double* psibar, hipStream_t s) {
    const int bx = (n + kTX - 1) / kTX, by = (n + kTY - 1) / kTY;
    // two blocks per CU; a chunk forms the cells of nz + 2 planes
    int nz = n < 16 ? n : 16;
    while (nz > 4 && bx * by * (n / nz) < 512) nz >>= 1;
    hipLaunchKernelGGL(k_geometry_bwd, dim3(bx, by, n / nz), dim3(kThr), 0, s, n, ih2, psi, Cbar, sbar, psibar, nz);
    return hipGetLastError();
}

}  // namespace mg
