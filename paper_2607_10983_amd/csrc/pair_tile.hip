// Two consecutive smoothing steps in one pass on rows of 4 KB and more.
//
//   y1 = x  + a1 (x  - xp) + cd1 (b - M x)
//   y2 = y1 + a2 (y1 - x ) + cd2 (b - M y1)
//
// Only y2 (and, with Y1OUT, y1) is written, so the two steps move 3 or 4
// fields instead of 7 or 8; the pass is bound by those bytes.  A whole row per
// block (the split rows of k_smooth2x_lds) leaves few rows per block when the
// row is long: 4 KB rows would have 2 output rows of 4.  Here a block of NW waves owns one x tile of 64 VEC points (1 KB) of
// NW consecutive rows, NW - 2 of them outputs, whatever the length of the row.
//
// The price is the x halo.  y1 is needed one point beyond the tile on either
// side, so the first and the last lane form that point as one element more,
// from two extra values of each row (a 2-element load by half-waves, left
// pair and right pair) and single values of b and x_prev.
//
// As in k_smooth2x_lds a wave marches a chunk of NZC planes with its rows in a
// register queue, publishes its x row one plane ahead and its y1 row one plane
// behind through LDS (two planes each, one barrier per plane), and the edge
// waves load the block's outer rows.  Same arithmetic as single steps
// (flat_rows.h), same bits.
#include "pair_tile.h"

#include "flat_rows.h"
#include "launch.h"

#include <type_traits>

namespace mg {
namespace {

// Values around the tile's ends: lanes 0 .. 31 hold the pair before the tile,
// lanes 32 .. 63 the pair after it (lanes 0 and 63 use them).
template <typename T>
struct Ends {
    T h[2];
    // the point next to the tile, and the one beyond it
    __device__ __forceinline__ T at(bool left) const { return left ? h[1] : h[0]; }
    __device__ __forceinline__ T beyond(bool left) const { return left ? h[0] : h[1]; }
};
template <typename T>
__device__ __forceinline__ void ld_pair(Ends<T>& e, const T* row, int hx) {
    typedef T T2 __attribute__((ext_vector_type(2)));
    const T2 v = *reinterpret_cast<const T2*>(row + hx);
    e.h[0] = v.x;
    e.h[1] = v.y;
}

// Coarse values under the two fine points of an Ends: columns A (under the
// even one) and A + 1, on the rows the prolongation of (y, z) reads.
template <typename T>
struct EndsCoarse {
    T a00, b00, a01, b01, a10, b10, a11, b11;
};
template <typename T>
__device__ __forceinline__ void ld_coarse(EndsCoarse<T>& c, const T* e, const RowGrid& gc, int y, int z, int ca,
                                          int cb) {
    const int Y = y >> 1, Z = z >> 1, oy = y & 1, oz = z & 1;
    const T* r = e + gc.row(Y, Z);
    c.a00 = r[ca];
    c.b00 = r[cb];
    if (oy) {
        r = e + gc.row(Y + 1, Z);
        c.a01 = r[ca];
        c.b01 = r[cb];
    }
    if (oz) {
        r = e + gc.row(Y, Z + 1);
        c.a10 = r[ca];
        c.b10 = r[cb];
    }
    if (oy && oz) {
        r = e + gc.row(Y + 1, Z + 1);
        c.a11 = r[ca];
        c.b11 = r[cb];
    }
}
// x += P e on the two points (rounding as prolong_add_seg)
template <typename T>
__device__ __forceinline__ void prolong_ends(Ends<T>& x, const EndsCoarse<T>& c, int y, int z) {
#pragma clang fp contract(off)
    const int oy = y & 1, oz = z & 1;
    auto col = [&](T v00, T v01, T v10, T v11) {
        T a = oy ? T(0.5) * (v00 + v01) : v00;
        if (oz) {
            const T q = oy ? T(0.5) * (v10 + v11) : v10;
            a = T(0.5) * (a + q);
        }
        return a;
    };
    const T wa = col(c.a00, c.a01, c.a10, c.a11), wb = col(c.b00, c.b01, c.b10, c.b11);
    x.h[0] = x.h[0] + wa;
    x.h[1] = x.h[1] + T(0.5) * (wa + wb);
}

// M x at one point from its six neighbours, as flat7_row
template <typename T>
__device__ __forceinline__ T flat7_one(T c, T l, T r, T ym, T yp, T zm, T zp, T ih2) {
#pragma clang fp contract(off)
    const T s = ((l + r) + (ym + yp)) + (zm + zp);
    return fma_rn(T(-6), c, s) * ih2;
}

struct NoCoarse {};

template <typename T, int VEC, int NW, PairStart START, bool PREV1, bool Y1OUT, int NZC, bool PFA>
__global__ __launch_bounds__(64 * NW) void k_pair_tile(int n, T ih2, const T* __restrict__ x,
                                                       const T* __restrict__ xp, const T* __restrict__ b,
                                                       T* __restrict__ y2, T* __restrict__ y1o, T a1, T cd1, T a2,
                                                       T cd2, int nyb, T cd0, SumsJob job,
                                                       const T* __restrict__ ec) {
    constexpr bool FROMB = START == PAIR_ZERO, PREVB = START == PAIR_PREVB, PRO = START == PAIR_PRO;
    constexpr bool LDP = PREV1 && !PREVB;  // x_prev is loaded
    static_assert(!FROMB || !PREV1, "a pass from zero has no x_prev");
    static_assert(!PREVB || PREV1, "x_prev formed by the pair");
    static_assert(!PRO || !PREV1, "the prolongation starts a pass");
    static_assert(VEC * sizeof(T) == 16, "a tile row is 1 KB");
    constexpr int NR = 64 * VEC;
    constexpr int W = NW - 2;  // output rows
    __shared__ T xs[2][NW][NR];    // x (FROMB: b) rows of a plane, one plane ahead
    __shared__ T rows[2][NW][NR];  // first-step rows of a plane
    __shared__ T xe[2][NW][2];     // x beside the tile's ends, with xs
    const RowGrid g{n, n - 1}, gc{n >> 1, (n >> 1) - 1};
    int nb = gridDim.x, bid = blockIdx.x;
    if constexpr (FROMB || PREVB) {
        if (job.count > 0) {  // block 0 finishes the sums, dispatched first
            nb -= 1;
            bid -= 1;
            if (bid < 0) {
                __shared__ double sh[kSumLanes];
                finish_sums(job, sh);
                return;
            }
        }
    }
    const int lb = xcd_logical(bid, nb);
    const int tiles = n / NR;
    const int tx = lb % tiles * NR, yb = lb / tiles % nyb, zc = lb / (tiles * nyb);
    const int w = wave_id();
    const int lane = threadIdx.x & 63;
    const bool left = lane < 32;
    const int y = yb * W - 1 + w;  // rows outside [0, n) wrap for loads
    const bool outw = w >= 1 && w <= W && y < n;
    const bool lo = w == 0, hi = w == NW - 1;
    const int yo = lo ? y - 1 : y + 1;  // outer neighbour row of an edge row
    const int z0 = zc * NZC;
    const size_t off = (size_t)tx + (size_t)lane * VEC;
    const int hx = left ? (tx - 2) & g.mask : (tx + NR) & g.mask;       // the pair beside the tile
    const int h1 = left ? (tx - 1) & g.mask : (tx + NR) & g.mask;       // its point next to the tile
    const int ca = hx >> 1, cb = (ca + 1) & gc.mask;                    // coarse columns under the pair
    const int cseg = tx / NR;
    const T* src = FROMB ? b : x;
    typedef std::conditional_t<PRO, CoarseSeg<T, VEC>, NoCoarse> CRow;
    typedef std::conditional_t<PRO, EndsCoarse<T>, NoCoarse> CEnd;
    int z1 = z0 - 1;
    // first step at z1: this row at z1-1, z1, z1+1, the outer row (edges) at z1, b and xp at z1
    T xm[VEC], xc[VEC], xq[VEC], o1[VEC] = {}, b1[VEC], p1[VEC];
    // the same beside the tile's ends: the point at z1-1, the pairs at z1 and z1+1, the outer row's point, b, xp
    T em, eo = T(0), eb = T(0), ep = T(0);
    Ends<T> el, eq;
    // second step at z2 = z1 - 1: first-step rows at z2-1, z2; b at z2; x_prev = xm
    T sm[VEC] = {}, sc[VEC] = {}, b2[VEC] = {}, se = T(0);
    auto load_x = [&](T (&v)[VEC], Ends<T>& e, CRow& c, CEnd& ce, int yy, int z) {
        const T* r = src + g.row(yy, z);
        ldrow<T, VEC>(v, r + off);
        ld_pair<T>(e, r, hx);
        if constexpr (PRO) {
            coarse_load_seg<T, VEC>(c, ec, gc, yy, z, cseg, lane);
            ld_coarse<T>(ce, ec, gc, yy, z, ca, cb);
        }
    };
    auto add_x = [&](T (&v)[VEC], Ends<T>& e, const CRow& c, const CEnd& ce, int yy, int z) {
        if constexpr (PRO) {
            prolong_add_seg<T, VEC>(v, c, yy, z);
            prolong_ends<T>(e, ce, yy, z);
        }
    };
    auto load_p = [&](T (&v)[VEC], T& e, int z) {
        if constexpr (LDP) {
            const T* r = xp + g.row(y, z);
            ldrow<T, VEC>(v, r + off);
            e = r[h1];
        }
    };
    auto load_b = [&](T (&v)[VEC], T& e, int z) {
        if constexpr (!FROMB) {
            const T* r = b + g.row(y, z);
            ldrow<T, VEC>(v, r + off);
            e = r[h1];
        }
    };
    {
        CRow c;
        CEnd ce;
        Ends<T> e;
        load_x(xm, e, c, ce, y, z1 - 1);
        add_x(xm, e, c, ce, y, z1 - 1);
        em = e.at(left);
        load_x(xc, el, c, ce, y, z1);
        add_x(xc, el, c, ce, y, z1);
        load_x(xq, eq, c, ce, y, z1 + 1);
        add_x(xq, eq, c, ce, y, z1 + 1);
        if (lo || hi) {
            load_x(o1, e, c, ce, yo, z1);
            add_x(o1, e, c, ce, yo, z1);
            eo = e.at(left);
        }
        load_b(b1, eb, z1);
        load_p(p1, ep, z1);
    }
    auto publish = [&](int buf, const T (&v)[VEC], const Ends<T>& e) {
        lds_strow<T, VEC>(xs[buf][w], lane, v);
        if (lane == 0) xe[buf][w][0] = e.at(true);
        if (lane == 63) xe[buf][w][1] = e.at(false);
    };
    publish(0, xc, el);
    constexpr int steps = NZC + 2;
    // PFA: the rows of the next plane are loaded one iteration earlier into a
    // second register set, i.e. two planes ahead of their use
    constexpr int ahead = PFA ? 1 : 0;
    T xa[VEC], oa[VEC] = {}, ba[VEC], pa[VEC], eba = T(0), epa = T(0);
    Ends<T> ea, eoa;
    CRow ca1, co1;
    CEnd cea, ceo;
    if constexpr (PFA) {
        load_x(xa, ea, ca1, cea, y, z1 + 2);
        if (lo || hi) load_x(oa, eoa, co1, ceo, yo, z1 + 1);
        load_b(ba, eba, z1 + 1);
        load_p(pa, epa, z1 + 1);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < steps; ++j, ++z1) {
        const bool more = j + 1 < steps;
        const bool load = j + 1 + ahead < steps;
        const int cbuf = j & 1;
        T xn[VEC], bn[VEC], pn[VEC], on[VEC], ebn = T(0), epn = T(0);
        Ends<T> en, eon;
        CRow cn, con;
        CEnd cen, ceon;
        if (load) {
            load_x(xn, en, cn, cen, y, z1 + 2 + ahead);
            if (lo || hi) load_x(on, eon, con, ceon, yo, z1 + 1 + ahead);
            load_b(bn, ebn, z1 + 1 + ahead);
            load_p(pn, epn, z1 + 1 + ahead);
        }
        // first step at z1
        T ym[VEC], yp[VEC], M1[VEC], sp[VEC];
        T eym = eo, eyp = eo;
        if (lo) copyrow(ym, o1);
        else {
            lds_ldrow<T, VEC>(ym, xs[cbuf][w - 1], lane);
            eym = xe[cbuf][w - 1][left ? 0 : 1];
        }
        if (hi) copyrow(yp, o1);
        else {
            lds_ldrow<T, VEC>(yp, xs[cbuf][w + 1], lane);
            eyp = xe[cbuf][w + 1][left ? 0 : 1];
        }
        const T ec0 = el.at(left), in = left ? xc[0] : xc[VEC - 1];
        T spe;  // the first step beside the tile's end
        if constexpr (FROMB) {
            T fc[VEC], fm[VEC], fq[VEC], fym[VEC], fyp[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                fc[e] = first_step<T, FROMB>(xc[e], cd0);
                fm[e] = first_step<T, FROMB>(xm[e], cd0);
                fq[e] = first_step<T, FROMB>(xq[e], cd0);
                fym[e] = first_step<T, FROMB>(ym[e], cd0);
                fyp[e] = first_step<T, FROMB>(yp[e], cd0);
            }
            auto f = [&](T v) { return first_step<T, FROMB>(v, cd0); };
            flat7_row_seg<T, VEC, 2>(fc, fym, fyp, fm, fq, ih2, M1, f(ec0));
#pragma unroll
            for (int e = 0; e < VEC; ++e) sp[e] = cheb_step<T>(fc[e], T(0), xc[e], M1[e], a1, cd1);
            const T Me = flat7_one<T>(f(ec0), f(el.beyond(left)), f(in), f(eym), f(eyp), f(em), f(eq.at(left)), ih2);
            spe = cheb_step<T>(f(ec0), T(0), ec0, Me, a1, cd1);
        } else {
            flat7_row_seg<T, VEC, 2>(xc, ym, yp, xm, xq, ih2, M1, ec0);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const T xpe = PREVB ? first_step<T, true>(b1[e], cd0) : PREV1 ? p1[e] : T(0);
                sp[e] = cheb_step<T>(xc[e], xpe, b1[e], M1[e], a1, cd1);
            }
            const T Me = flat7_one<T>(ec0, el.beyond(left), in, eym, eyp, em, eq.at(left), ih2);
            const T xpe = PREVB ? first_step<T, true>(eb, cd0) : PREV1 ? ep : T(0);
            spe = cheb_step<T>(ec0, xpe, eb, Me, a1, cd1);
        }
        if constexpr (Y1OUT) {
            if (outw && j >= 1 && j <= NZC) strow<T, VEC>(y1o + g.row(y, z1) + off, sp);
        }
        // publish x at z1+1 (used by the next plane's first step) and the first step at z1-1
        if (more) publish(cbuf ^ 1, xq, eq);
        if (j >= 2) lds_strow<T, VEC>(rows[cbuf][w], lane, sc);
        __syncthreads();
        if (j >= 2 && outw) {  // second step at z1-1
            T nm[VEC], np[VEC], M2[VEC], o[VEC];
            lds_ldrow<T, VEC>(nm, rows[cbuf][w - 1], lane);
            lds_ldrow<T, VEC>(np, rows[cbuf][w + 1], lane);
            flat7_row_seg<T, VEC, 2>(sc, nm, np, sm, sp, ih2, M2, se);
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                if constexpr (FROMB)  // x_prev = first step at z2, b at z2 = the raw queue row
                    o[e] = cheb_step<T>(sc[e], first_step<T, FROMB>(xm[e], cd0), xm[e], M2[e], a2, cd2);
                else
                    o[e] = cheb_step<T>(sc[e], xm[e], b2[e], M2[e], a2, cd2);
            }
            strow<T, VEC>(y2 + g.row(y, z1 - 1) + off, o);
        }
        copyrow(sm, sc);
        copyrow(sc, sp);
        se = spe;
        if constexpr (!FROMB) copyrow(b2, b1);
        if (more) {
            em = ec0;
            el = eq;
            copyrow(xm, xc);
            copyrow(xc, xq);
            if constexpr (PFA) {  // two iterations after their loads were issued
                add_x(xa, ea, ca1, cea, y, z1 + 2);
                if (lo || hi) add_x(oa, eoa, co1, ceo, yo, z1 + 1);
                copyrow(xq, xa);
                eq = ea;
                if (lo || hi) {
                    copyrow(o1, oa);
                    eo = eoa.at(left);
                }
                if constexpr (!FROMB) copyrow(b1, ba);
                eb = eba;
                if constexpr (LDP) copyrow(p1, pa);
                ep = epa;
                if (load) {
                    copyrow(xa, xn);
                    ea = en;
                    ca1 = cn;
                    cea = cen;
                    if (lo || hi) {
                        copyrow(oa, on);
                        eoa = eon;
                        co1 = con;
                        ceo = ceon;
                    }
                    if constexpr (!FROMB) copyrow(ba, bn);
                    eba = ebn;
                    if constexpr (LDP) copyrow(pa, pn);
                    epa = epn;
                }
            } else {  // a whole iteration after their loads were issued
                add_x(xn, en, cn, cen, y, z1 + 2);
                if (lo || hi) add_x(on, eon, con, ceon, yo, z1 + 1);
                copyrow(xq, xn);
                eq = en;
                if (lo || hi) {
                    copyrow(o1, on);
                    eo = eon.at(left);
                }
                if constexpr (!FROMB) copyrow(b1, bn);
                eb = ebn;
                if constexpr (LDP) copyrow(p1, pn);
                ep = epn;
            }
        }
    }
}

constexpr size_t kTileMinRowBytes = 4096;
constexpr int kTileNz = 16;  // output planes of a block: x is read on 20, b and x_prev on 18
// Waves of a block and whether rows are loaded two planes ahead of their use.
// 12 waves give 10 output rows of 12 and leave a wave 170 registers: float
// then holds the second register set (1024^3 mixed, degree 4: 23.9 ms per
// cycle; 16 waves without it 24.0 to 24.2), double does not (512^3, degree 4:
// 6.04 ms; 8 waves with it 6.14, without 6.21, 10 waves 6.28, 16 waves, which
// spill, 8.76).  With the prolongation double takes 8 waves (256 registers).
template <typename T, PairStart START>
struct TileShape {
    static constexpr bool pro = START == PAIR_PRO, dbl = sizeof(T) == 8;
    static constexpr int NW = pro && dbl ? 8 : 12;
    static constexpr bool PFA = !pro && !dbl;
};

template <typename T, PairStart START, bool PREV1, bool Y1OUT>
hipError_t go(int n, double ih2, const T* x, const T* xp, const T* b, T* y2, T* y1, const T* ec, double a1, double cd1,
              double a2, double cd2, double cd0, const SumsJob& sums, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    typedef TileShape<T, START> Sh;
    constexpr int VEC = 16 / (int)sizeof(T), NW = Sh::NW, W = NW - 2;
    const int nyb = (n + W - 1) / W;
    const int blocks = n / (64 * VEC) * nyb * (n / kTileNz);
    const int extra = (START == PAIR_ZERO || START == PAIR_PREVB) && sums.count > 0 ? 1 : 0;
    MG_LAUNCH((k_pair_tile<T, VEC, NW, START, PREV1, Y1OUT, kTileNz, Sh::PFA>), dim3(blocks + extra), dim3(64 * NW), s,
              ev0, ev1, n, (T)ih2, x, xp, b, y2, y1, (T)a1, (T)cd1, (T)a2, (T)cd2, nyb, (T)cd0, sums, ec);
    return hipGetLastError();
}

}  // namespace

// Rows of 4 KB and more.  Rows of 2 KB keep the split rows of k_smooth2x_lds,
// whose 6 output rows of 8 cost less than the x halo here (512^3 mixed, degree
// 4: 2.86 ms per cycle there, 3.05 in tiles; 256^3 double, degree 3: 0.60 and
// 0.74).  Longer rows had single steps only: one cycle of degree 4 at 512^3
// double 7.06 -> 6.04 ms, 1024^3 double 62.2 -> 49.9, 1024^3 mixed 30.3 -> 23.9.
bool pair_tile_applies(int n, size_t elem) { return n <= 1024 && (size_t)n * elem >= kTileMinRowBytes; }

template <typename T>
hipError_t launch_pair_tile(int n, double ih2, PairStart start, const T* x, const T* xp, const T* b, T* y2, T* y1,
                            const T* ec, double a1, double cd1, double a2, double cd2, double cd0,
                            const SumsJob& sums, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    if (!pair_tile_applies(n, sizeof(T)) || b == nullptr || y2 == nullptr || (start != PAIR_ZERO && x == nullptr))
        return hipErrorInvalidValue;
#define MG_TILE(START, PREV1, Y1OUT)                                                                                \
    return go<T, START, PREV1, Y1OUT>(n, ih2, x, xp, b, y2, y1, ec, a1, cd1, a2, cd2, cd0, sums, s, ev0, ev1)
    switch (start) {
        case PAIR_PLAIN:
            if (xp && y1) MG_TILE(PAIR_PLAIN, true, true);
            if (xp) MG_TILE(PAIR_PLAIN, true, false);
            if (y1) MG_TILE(PAIR_PLAIN, false, true);
            MG_TILE(PAIR_PLAIN, false, false);
        case PAIR_ZERO:
            if (xp) return hipErrorInvalidValue;
            if (y1) MG_TILE(PAIR_ZERO, false, true);
            MG_TILE(PAIR_ZERO, false, false);
        case PAIR_PREVB:
            if (xp || y1) return hipErrorInvalidValue;
            MG_TILE(PAIR_PREVB, true, false);
        case PAIR_PRO:
            if (xp || !ec) return hipErrorInvalidValue;
            if (y1) MG_TILE(PAIR_PRO, false, true);
            MG_TILE(PAIR_PRO, false, false);
    }
#undef MG_TILE
    return hipErrorInvalidValue;
}

template hipError_t launch_pair_tile<float>(int, double, PairStart, const float*, const float*, const float*, float*,
                                            float*, const float*, double, double, double, double, double,
                                            const SumsJob&, hipStream_t, hipEvent_t, hipEvent_t);
template hipError_t launch_pair_tile<double>(int, double, PairStart, const double*, const double*, const double*,
                                             double*, double*, const double*, double, double, double, double, double,
                                             const SumsJob&, hipStream_t, hipEvent_t, hipEvent_t);

}  // namespace mg
