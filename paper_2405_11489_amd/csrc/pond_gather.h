// pond_gather.h -- the gather of a node's populations at their departure
// points, in the frame of the current predictor-corrector iterate.
//
// Population (a, b) of f is the order-N Hermite reconstruction, at the
// velocity c_ab = (c_a, c_b) of the frame (u, T), of the moments interpolated
// at x - C_ab:
//   f_ab = w_a w_b sum_{k + l <= N} He_k(c_a) He_l(c_b) / (k! l!) A_kl,
//   A_kl = sum over the moments of He_k(xi_x) He_l(xi_y), xi = (V - d) / sqrt(T)
// (V about u_ref, d = u - u_ref).  Both the reconstruction and the
// interpolation are products of an x- and a y-factor, and all of it is linear,
// so the work is split by axis and shared:
//   - the departure abscissa depends on a alone and the ordinate on b alone, so
//     a stencil row is interpolated along x once for the Q1 velocities of an
//     x-component (X, 2 NM moments);
//   - the row is reduced at once to the N + 1 numbers per distribution that the
//     velocities of the x-component still need,
//       D_l = sum_p al_pl Y_pl,   Y_pl = sum_{q <= l} gy_lq X_pq   (p + l <= N),
//     gy the coefficients of He_l(xi_y) T^(l/2) (a monic polynomial in V_y) and
//     al the x-factor sum_{k <= N - l} He_k(c_a) / k! He_k(xi_x), scaled by
//     T^(-l/2);
//   - velocity b adds its row weight times sum_l He_l(c_b) / l! D_l; the even and
//     the odd orders of +-c_b are formed once for both.
// The weights w_a w_b are left to the sums over the populations, which take them
// in double (gather_weight).  Rounded to float, their sums would differ from 1
// by 2e-8, the same way at every node and step: a drift of the mass wherever the
// moments interpolated are not small (a shock tube's right state, seen from its
// left).  For the same reason al_00 is held without its leading 1, which
// enters D_0 exactly.
// By orders of T^(1/2) the coefficients follow from the Hermite addition
// theorem, He_k(x + y) = sum_p C(k, p) x^p He_(k-p)(y).
#pragma once

namespace pond {

// kap[a][(p, m)] = He_{p + m}(c_a) / (p! m!): the x-factors' constants.
template <typename P, class L>
struct GatherTables {
    P kap[L::Q1][L::NM];
};
template <typename P, class L>
constexpr GatherTables<P, L> make_gather_tables() {
    GatherTables<P, L> t{};
    for (int a = 0; a < L::Q1; ++a)
        for (int k = 0; k < L::NM; ++k) {
            const int p = mom_px(k), m = mom_py(k);
            t.kap[a][k] = P(he_value(p + m, L::c(a)) / (factorial_c(p) * factorial_c(m)));
        }
    return t;
}
static __constant__ GatherTables<float, D2Q16> kGather16F = make_gather_tables<float, D2Q16>();
static __constant__ GatherTables<double, D2Q16> kGather16D = make_gather_tables<double, D2Q16>();
static __constant__ GatherTables<float, D2Q25> kGather25F = make_gather_tables<float, D2Q25>();
static __constant__ GatherTables<double, D2Q25> kGather25D = make_gather_tables<double, D2Q25>();

template <typename P, class L>
__device__ __forceinline__ const GatherTables<P, L> &gather_tab() {
    if constexpr (L::Q == 16) {
        if constexpr (sizeof(P) == 4)
            return kGather16F;
        else
            return kGather16D;
    } else if constexpr (sizeof(P) == 4) {
        return kGather25F;
    } else {
        return kGather25D;
    }
}

// Weights of the one-dimensional lattice for the sums over gathered populations.
// In FP32 the constants He_2 / 2 (and He_4 / 24) of the reconstruction are
// rounded, so that sum_b w_b He_2(c_b) / 2 is 7e-9 and not 0, and the second
// moments would leak into the mass; these weights (1e-8 off the lattice's) make
// the rounded constants' sums vanish and sum to 1.
template <typename P, class L>
constexpr double gather_weight(int a) {
    if (sizeof(P) == 8) return L::w(a);
    const int m = a < L::Q1 - 1 - a ? a : L::Q1 - 1 - a;  // 0 outer, 1 inner (2 zero)
    const double h0 = float(he_value(2, L::c(0)) / 2.0), h1 = float(he_value(2, L::c(1)) / 2.0);
    if (L::Q1 == 4) {
        // 2 (w0 + w1) = 1, w0 h0 + w1 h1 = 0
        const double w1 = 0.5 * h0 / (h0 - h1);
        return m == 0 ? 0.5 - w1 : w1;
    }
    // 2 (w0 + w1) + w2 = 1 and the sums of He_2 / 2 (-1/2 at zero) and of He_4 / 24
    // (1/8) zero: 2 w0 (h0 + 1/2) + 2 w1 (h1 + 1/2) = 1/2, the same with k and -1/8
    const double k0 = float(he_value(4, L::c(0)) / 24.0), k1 = float(he_value(4, L::c(1)) / 24.0);
    const double a0 = h0 + 0.5, a1 = h1 + 0.5, b0 = k0 - 0.125, b1 = k1 - 0.125;
    const double det = a0 * b1 - a1 * b0;
    const double w0 = 0.5 * (0.5 * b1 + 0.125 * a1) / det;
    const double w1 = 0.5 * (-0.125 * a0 - 0.5 * b0) / det;
    return m == 0 ? w0 : (m == 1 ? w1 : 1.0 - 2.0 * (w0 + w1));
}
static_assert(gather_weight<float, D2Q16>(0) - D2Q16::w(0) < 1e-7 &&
                  D2Q16::w(0) - gather_weight<float, D2Q16>(0) < 1e-7 &&
                  gather_weight<float, D2Q25>(0) - D2Q25::w(0) < 1e-7 &&
                  D2Q25::w(0) - gather_weight<float, D2Q25>(0) < 1e-7 &&
                  gather_weight<float, D2Q25>(1) - D2Q25::w(1) < 1e-7 &&
                  D2Q25::w(1) - gather_weight<float, D2Q25>(1) < 1e-7,
              "the gather's weights are the lattice's to rounding");

// y-factors of an iterate frame: coefficient of V^q, q < l, of the monic
// polynomial T^(l/2) He_l((V - d) / sqrt T); g[m] = its value at V = 0.
template <typename P, class L>
struct YFactors {
    P c[L::N + 1][L::N + 1];
    __device__ __forceinline__ YFactors(P d, P T) {
        P g[L::N + 1];
        g[0] = P(1);
        g[1] = -d;
#pragma unroll
        for (int m = 1; m < L::N; ++m) g[m + 1] = g[1] * g[m] - P(m) * T * g[m - 1];
#pragma unroll
        for (int l = 1; l <= L::N; ++l)
#pragma unroll
            for (int q = 0; q < l; ++q) c[l][q] = P(binom_c(l, q)) * g[l - q];
    }
};

// x-factors of x-component a: al[(p, l)] = T^(-(p + l)/2) sum_{m <= N - l - p}
// kap[a][(p, m)] He_m(delta), delta = -d / sqrt T; al[(0, 0)] less its first term, 1.
template <typename P, class L>
struct XFrame {
    P he[L::N + 1], sc[L::N + 1];
    __device__ __forceinline__ XFrame(P d, P is) {
        he[0] = sc[0] = P(1);
        he[1] = -d * is;
        sc[1] = is;
#pragma unroll
        for (int m = 1; m < L::N; ++m) {
            he[m + 1] = he[1] * he[m] - P(m) * he[m - 1];
            sc[m + 1] = sc[m] * is;
        }
    }
    __device__ __forceinline__ void factors(const P kap[L::NM], P al[L::NM]) const {
#pragma unroll
        for (int p = 0; p <= L::N; ++p) {
            P sum = p == 0 ? P(0) : kap[mom_index(p, 0)];
#pragma unroll
            for (int l = L::N - p; l >= 0; --l) {
                const int m = L::N - l - p;
                if (m > 0) sum += kap[mom_index(p, m)] * he[m];
                const P full = p == 0 ? P(1) + sum : sum;
                al[mom_index(p, l)] = p + l > 0 ? full * sc[p + l] : sum;
            }
        }
    }
};

// One distribution's row: the x-interpolated moments X to the D_l.
template <typename P, class L>
__device__ __forceinline__ void row_factors(const P *X, const P al[L::NM], const YFactors<P, L> &y,
                                            P D[L::N + 1]) {
#pragma unroll
    for (int l = 0; l <= L::N; ++l) {
#pragma unroll
        for (int p = 0; p <= L::N - l; ++p) {
            P Y = X[mom_index(p, l)];
#pragma unroll
            for (int q = l - 1; q >= 0; --q) Y += y.c[l][q] * X[mom_index(p, q)];
            if (p > 0)
                D[l] += al[mom_index(p, l)] * Y;
            else
                D[l] = l == 0 ? Y + al[0] * Y : al[mom_index(0, l)] * Y;
        }
    }
}

// Adds the row's share of the x-component's Q1 populations (over w_a w_b): the
// row weight w[b] times sum_l He_l(c_b) / l! D_l.
template <typename P, class L>
__device__ __forceinline__ void add_row(const P D[L::N + 1], const P w[L::Q1], P acc[L::Q1]) {
#pragma unroll
    for (int h = 0; h < L::Q1 / 2; ++h) {
        const double c = L::c(L::Q1 - 1 - h);
        P e = D[0] + P(he_value(2, c) / 2.0) * D[2];
        if constexpr (L::N >= 4) e += P(he_value(4, c) / 24.0) * D[4];
        const P o = D[1] + P(he_value(3, c) / (6.0 * c)) * D[3];
        const P lo = e - P(c) * o, hi = e + P(c) * o;
        acc[h] += w[h] * lo;
        acc[L::Q1 - 1 - h] += w[L::Q1 - 1 - h] * hi;
    }
    if constexpr (L::Q1 % 2 == 1) {  // the zero abscissa
        const P e = D[0] + P(he_value(2, 0.0) / 2.0) * D[2] + P(he_value(4, 0.0) / 24.0) * D[4];
        acc[L::Q1 / 2] += w[L::Q1 / 2] * e;
    }
}

// The rows of an x-component, read ahead: a row's moments come in chunks (some
// columns of f's groups, then of g's), and while a chunk is interpolated the
// loads of the next one -- of the next row after a row's last -- are in flight,
// so that the wave waits for LDS once per pass and not once per chunk.
// CT: columns per chunk.
template <typename P, int NP, class L, int CT>
struct RowReader {
    using MV = MomVec<P, nmom<L>()>;
    using V = typename MV::V;
    static constexpr int GF = (L::NM + MV::W - 1) / MV::W;  // groups that hold f's moments
    static constexpr int CH = (NP + CT - 1) / CT;           // chunks per distribution
    V buf[2][CT][GF];

    // loads chunk c of the row: row(k, p) is moment group k in column p
    template <class Row>
    __device__ __forceinline__ void load(const Row &row, int c) {
        const int k0 = c < CH ? 0 : GF, k1 = c < CH ? GF : MV::G, p0 = (c % CH) * CT;
#pragma unroll
        for (int p = p0; p < p0 + CT && p < NP; ++p)
#pragma unroll
            for (int k = k0; k < k1; ++k) buf[c % 2][p - p0][k - k0] = row(k, p);
    }

    // x-interpolation of the row's loaded chunk c into X
    template <class Row>
    __device__ __forceinline__ void interpolate(const Row &row, int c, const P wx[NP],
                                                P X[MV::G * MV::W]) const {
        const int k0 = c < CH ? 0 : GF, k1 = c < CH ? GF : MV::G, p0 = (c % CH) * CT;
#pragma unroll
        for (int p = p0; p < p0 + CT && p < NP; ++p)
#pragma unroll
            for (int k = k0; k < k1; ++k) {
                const V v = row.deviation(k, buf[c % 2][p - p0][k - k0]);
                const P w = wx[p];
                P *x = X + MV::W * k;
                x[0] = p == 0 ? w * v.x : x[0] + w * v.x;
                x[1] = p == 0 ? w * v.y : x[1] + w * v.y;
                if constexpr (MV::W == 4) {
                    x[2] = p == 0 ? w * v.z : x[2] + w * v.z;
                    x[3] = p == 0 ? w * v.w : x[3] + w * v.w;
                }
            }
    }

    // One row, whose first chunk is loaded: f's moments are interpolated along x
    // and reduced, then g's, w[b] times the result added to af and ag.  ahead()
    // loads the first chunk of the row to visit next, if it is to be read ahead.
    template <class Row, class Ahead>
    __device__ __forceinline__ void row(const Row &row, Ahead &&ahead, const P wx[NP],
                                        const P al[L::NM], const YFactors<P, L> &y,
                                        const P w[L::Q1], P af[L::Q1], P ag[L::Q1]) {
        P X[MV::G * MV::W], D[L::N + 1];
#pragma unroll
        for (int c = 0; c < 2 * CH; ++c) {
            if (c + 1 < 2 * CH)
                load(row, c + 1);
            else
                ahead();
            __builtin_amdgcn_sched_barrier(0);
            interpolate(row, c, wx, X);
            if (c == CH - 1 || c == 2 * CH - 1) {
                row_factors<P, L>(X + (c < CH ? 0 : L::NM), al, y, D);
                add_row<P, L>(D, w, c < CH ? af : ag);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// Columns per chunk.  Two chunks of two columns (FP32 D2Q16: six loads of 16 bytes
// in flight) cover the LDS latency: whole rows took 80 more registers and the same
// time (512^2 Mach 2: 0.1108 against 0.1106 ms per step).
template <int NP>
constexpr int chunk_columns() { return NP < 2 ? NP : 2; }

// Rows of the unrolled gather: the union of an x-component's row stencils when
// its velocities' first rows lie within NP + 2 rows of each other: for certain where
// 2 c_out sqrt T <= NP + 2 (D2Q16: T <= 1.65 with the cubic stencil, 1.14 with the
// quadratic one; D2Q25: T <= 1.10), by position below NP + 3 (T < 2.25, 1.65; 1.50).
template <int NP>
constexpr int table_rows() { return 2 * NP + 2; }

// The weights w shifted up by o < 8 places, bit by bit of o.
template <int M, typename P>
__device__ __forceinline__ void shift_weights(P (&w)[M], int o) {
#pragma unroll
    for (int bit = 1; bit < 8; bit *= 2)
#pragma unroll
        for (int r = M - 1; r >= 0; --r) {
            const P lower = r >= bit ? w[r >= bit ? r - bit : 0] : P(0);
            w[r] = (o & bit) ? lower : w[r];
        }
}

// Rows R .. of the union over the weight table, the first chunk of row R loaded.
// The row read ahead is this one again after a lane's last; a lane whose union
// is shorter than the wave's stays on its last row, at weight 0.  (Written as a
// recursion: the compiler does not unroll a loop with these exits reliably.)
template <int R, int RS, typename P, int NP, class L, int CT, class Row>
__device__ __forceinline__ void unrolled_rows(RowReader<P, NP, L, CT> &rd, Row &at, int span,
                                              bool flat, const P wx[NP], const P al[L::NM],
                                              const YFactors<P, L> &y, const P (&wt)[RS][L::Q1],
                                              P af[L::Q1], P ag[L::Q1]) {
    rd.row(
        at,
        [&] {
            if (R + 1 < NP ? !flat : span > R + 1) at.next();
            rd.load(at, 0);
        },
        wx, al, y, wt[R], af, ag);
    if constexpr (R + 1 < RS) {
        if (R == 0 && flat) return;
        if (R + 1 >= NP && __ballot(span > R + 1) == 0) return;
        unrolled_rows<R + 1, RS>(rd, at, span, flat, wx, al, y, wt, af, ag);
    }
}

// The gather of x-component ia by per-velocity queues of row weights, one row at a
// time: staged rows with read-ahead where the x-component's rows are all staged in
// every lane of the wave, else rows in HBM.  One column per chunk: two take registers
// that the unrolled rows need (D2Q25 FP64 spilled, 0.43 against 0.35 ms per step of
// 384^2 at T = 1).  Reading rows that are half staged from either place took longer
// than from HBM alone (D2Q25 at T = 3, Mach 2: FP32 0.58 against 0.50 ms, FP64 1.84
// against 1.45), and so did rows column by column without read-ahead (D2Q16 512^2 at
// T = 2, FP32: 0.226 against 0.144 ms; FP64 0.91 against 0.43).
template <typename P, int NP, class L, class Taps>
__device__ __forceinline__ void gather_general(const Taps &taps, int ia, double xu, double yu,
                                               double sc, const XFrame<P, L> &xf,
                                               const YFactors<P, L> &y, P (&af)[L::Q1],
                                               P (&ag)[L::Q1]) {
    constexpr int Q1 = L::Q1;
    const bool flat = taps.flat();
    P wx[NP], al[L::NM];
    const int bx = lagrange<NP>(fma(-sc, L::c(ia), xu), wx);
    xf.factors(gather_tab<P, L>().kap[ia], al);
    int by[Q1];
    P q[Q1][NP];  // row weights, shifted out first to last
#pragma unroll
    for (int b = 0; b < Q1; ++b) {
        by[b] = lagrange<NP>(fma(-sc, L::c(b), yu), q[b]);
        af[b] = ag[b] = P(0);
#pragma unroll
        for (int k = 0; k < NP; ++k) q[b][k] = flat ? P(k == 0 ? 1.0 : 0.0) : q[b][k];
    }
    const int span = flat ? 1 : by[0] - by[Q1 - 1] + NP;
    // the union's rows in turn, every velocity whose stencil holds the row; a union
    // longer than the separate stencils velocity by velocity
    const bool whole = span <= Q1 * NP;
    auto take = [&](int b, bool on, P (&w)[Q1]) {  // velocity b's weight of this row
        w[b] = on ? q[b][0] : P(0);
#pragma unroll
        for (int k = 0; k + 1 < NP; ++k) q[b][k] = on ? q[b][k + 1] : q[b][k];
        q[b][NP - 1] = on ? P(0) : q[b][NP - 1];
    };
    if (Taps::kStaged && __ballot(!(whole && taps.inside(bx, NP, flat ? 0 : by[Q1 - 1], span))) == 0) {
        RowReader<P, NP, L, 1> rd;
        auto at = taps.staged(bx, flat ? 0 : by[Q1 - 1]);
        rd.load(at, 0);
#pragma unroll 1
        for (int t = 0; __ballot(t < span) != 0; ++t) {
            P w[Q1];
#pragma unroll
            for (int b = 0; b < Q1; ++b) take(b, flat || t >= by[b] - by[Q1 - 1], w);
            rd.row(
                at,
                [&] {  // a lane's last row again after its last
                    if (t + 1 < span) at.next();
                    rd.load(at, 0);
                },
                wx, al, y, w, af, ag);
        }
        return;
    }
    int v = Q1 - 1, r = flat ? 0 : by[Q1 - 1], left = whole ? span : NP;
#pragma unroll 1
    for (;;) {
        RowReader<P, NP, L, 1> rd;
        P w[Q1];
        auto weights = [&] {
#pragma unroll
            for (int b = 0; b < Q1; ++b) take(b, whole ? flat || r >= by[b] : v == b, w);
        };
        weights();
        const auto at = taps.outside(bx, r);
        rd.load(at, 0);
        rd.row(at, [] {}, wx, al, y, w, af, ag);
        ++r;
        if (--left == 0) {
            if (whole || v == 0) break;
            --v;
            left = NP;
            r = by[0];
#pragma unroll
            for (int u = 1; u < Q1; ++u) r = v == u ? by[u] : r;
        }
    }
}

// The gather of every population of a node in the iterate frame: departure
// offsets xu = x - u, yu = y - u relative to the grid, scale sc = sqrt T, frame
// shift (dux, duy) from u_ref, is = 1 / sqrt T, T.  column(ia, f, g) receives the
// Q1 populations of each x-component over their weights w_a w_b, in turn.
//
// In FP32 the populations handed over are those of the interpolated deviations
// from the reference moments only: the reference's own share is the same
// reconstruction of one moment vector for every velocity, and the
// reconstruction keeps the moments up to order N (the quadrature is exact to
// degree 2 N + 1), so its share of every sum that column forms -- mass,
// momentum, energy, the lab moments -- follows from M_ref itself; the caller
// adds it once after the gather.
//
// The rows of an x-component are those of the union of its velocities'
// stencils, each visited once.  Where that union has at most table_rows and the
// node's stencils lie in the staged region, the row loop is unrolled over a
// table of row weights (zero where a velocity's stencil does not hold the row)
// that serves all x-components; a wave with a node where that is not so shifts the
// weights out of per-velocity queues row by row (gather_general), for all its
// nodes: both paths one after the other would take the sum of their times.  A union
// longer than the separate stencils (very hot flows) is visited stencil by stencil.
// The sums are the same numbers either way: each velocity's rows are added in
// ascending order, the others add zero.  On a single-row grid every stencil row is
// that row, and the weights sum to one.
//
// Quad: this lane gathers x-component threadIdx.x % 4 alone.
template <typename P, int NP, class L, bool Quad, class Taps, class Column>
__device__ __forceinline__ void gather_rows(const Taps &taps, double xu, double yu, double sc,
                                            P dux, P duy, P is, P T, Column &column) {
    constexpr int NM = L::NM, Q1 = L::Q1, RS = table_rows<NP>();
    const bool flat = taps.flat();
    const YFactors<P, L> y(duy, T);
    const XFrame<P, L> xf(dux, is);
    const auto &tab = gather_tab<P, L>();
    int by[Q1];
    P wy[Q1][NP];
#pragma unroll
    for (int b = 0; b < Q1; ++b) by[b] = lagrange<NP>(fma(-sc, L::c(b), yu), wy[b]);
    // the ordinates descend with b, and so do the first stencil rows (and with ia
    // the first columns)
    const int r0 = flat ? 0 : by[Q1 - 1], span = flat ? 1 : by[0] - by[Q1 - 1] + NP;
    const int x0 = stencil_base<NP>(fma(-sc, L::c(Q1 - 1), xu));
    const int x1 = stencil_base<NP>(fma(-sc, L::c(0), xu));
    const bool fits = span <= RS && taps.inside(x0, x1 + NP - x0, r0, span);
    // How likely the unrolled rows are, for the register allocator: it takes the loops
    // of the other path for the hot ones and spills here for them unless told, in FP32
    // strongly (2048^2 quadrants 0.77 ms per step untold, 0.73 here, 24 % more bytes
    // written at the usual 0.9995; hot flows of T = 4 0.164 and 0.174 of 512^2).  In
    // FP64 the surer it is the more it spills here (D2Q16 512^2 0.30 when sure, 0.28 so,
    // T = 4 0.52 and 0.48), and on D2Q25 in any case (400^2 0.43 untold, 0.48 so).
    const bool unroll = __ballot(!fits) == 0;
    if (Taps::kStaged &&
        (sizeof(P) == 4 ? __builtin_expect_with_probability(unroll, 1, 0.999999)
                        : L::Q == 25 ? unroll
                                     : __builtin_expect_with_probability(unroll, 1, 0.99))) {
        P wt[RS][Q1];
#pragma unroll
        for (int b = 0; b < Q1; ++b) {
            P t[RS];
#pragma unroll
            for (int r = 0; r < RS; ++r) t[r] = r < NP ? wy[b][r < NP ? r : 0] : P(0);
            if (b + 1 < Q1) shift_weights<RS>(t, by[b] - by[Q1 - 1]);
#pragma unroll
            for (int r = 0; r < RS; ++r) wt[r][b] = t[r];
            if (flat) wt[0][b] = P(1);
        }
        auto component = [&](int ia) {
            P wx[NP], al[NM], af[Q1], ag[Q1];
            const int bx = lagrange<NP>(fma(-sc, L::c(ia), xu), wx);
            xf.factors(tab.kap[ia], al);
#pragma unroll
            for (int b = 0; b < Q1; ++b) af[b] = ag[b] = P(0);
            auto at = taps.staged(bx, r0);
            RowReader<P, NP, L, chunk_columns<NP>()> rd;
            rd.load(at, 0);
            unrolled_rows<0, RS>(rd, at, span, flat, wx, al, y, wt, af, ag);
            column(ia, af, ag);
        };
        if constexpr (Quad) {
            component(int(threadIdx.x) & 3);
        } else {
#pragma unroll 1
            for (int ia = 0; ia < Q1; ++ia) component(ia);
        }
    } else {
        auto component = [&](int ia) {
            P f[Q1], g[Q1];
            gather_general<P, NP, L>(taps, ia, xu, yu, sc, xf, y, f, g);
            column(ia, f, g);
        };
        if constexpr (Quad) {
            component(int(threadIdx.x) & 3);
        } else {
#pragma unroll 1
            for (int ia = 0; ia < Q1; ++ia) component(ia);
        }
    }
}

}  // namespace pond
