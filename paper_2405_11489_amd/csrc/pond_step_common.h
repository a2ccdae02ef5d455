// pond_step_common.h -- per-node body of the PonD step shared by the step
// kernels: departure stencils, the predictor-corrector loop over a tap source,
// re-projection, collision in Grad-coefficient space and the store.
//
// Moment storage ("grouped planes"): the 2 NM moments of a node (f moments
// 0..NM-1, g moments NM..2NM-1, ordering of pond_device.h; NM = 10 on D2Q16,
// 15 on D2Q25) are held as G vector groups (float: float4, the last padded;
// double: double2); in the HBM moment planes group k of node idx sits at
// base[k * stride + idx] (stride = nodes per plane: lanes of a wave read
// consecutive vectors); the LDS tiles hold a node's groups contiguously
// (lds_stride below).
#pragma once

#include <utility>

#include "pond_device.h"
#include "pond_internal.h"

namespace pond {

template <typename P, int NMOM>
struct MomVec;
template <int NMOM>
struct MomVec<float, NMOM> {
    using V = float4;
    static constexpr int W = 4;
    static constexpr int G = (NMOM + 3) / 4;
};
template <int NMOM>
struct MomVec<double, NMOM> {
    using V = double2;
    static constexpr int W = 2;
    static constexpr int G = (NMOM + 1) / 2;
};

constexpr int kNMom = 2 * kNM;  // 20 moments per node on D2Q16

// Moments per node of a lattice, and the values a node's groups hold (padded).
template <class L>
constexpr int nmom() { return 2 * L::NM; }
template <typename P, class L>
constexpr int nmom_padded() {
    return MomVec<P, nmom<L>()>::G * MomVec<P, nmom<L>()>::W;
}

template <typename P, int NMOM = kNMom>
__device__ __forceinline__ void load_moments(const P *__restrict__ base, long long stride,
                                             long long idx, P *M) {
    using MV = MomVec<P, NMOM>;
    using V = typename MV::V;
    const V *b = reinterpret_cast<const V *>(base);
    if constexpr (MV::W == 4) {
#pragma unroll
        for (int k = 0; k < MV::G; ++k) {
            const V v = b[k * stride + idx];
            M[4 * k] = v.x;
            M[4 * k + 1] = v.y;
            M[4 * k + 2] = v.z;
            M[4 * k + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < MV::G; ++k) {
            const V v = b[k * stride + idx];
            M[2 * k] = v.x;
            M[2 * k + 1] = v.y;
        }
    }
}

// Stores of the step's outputs in HBM.  This step never reads what it writes,
// so they may stream past the caches (non-temporal stores), leaving L2 to the
// halo moments that neighbouring tiles re-read.  POND_STREAM_STORE is a mask
// of the streams stored that way: 1 the populations, 2 the frame, 4 the
// moment planes.  Off by default: on the 2048^2 quadrants streaming the moment
// planes (and the frame) cut the read bytes by 3 % (7.5 %) at the same step
// time, and streamed population stores (one dword per lane) raised the written
// bytes by half and slowed the step.
#ifndef POND_STREAM_STORE
#define POND_STREAM_STORE 0
#endif
typedef float pond_f4v __attribute__((ext_vector_type(4)));
typedef double pond_d2v __attribute__((ext_vector_type(2)));

template <int Stream, typename T>
__device__ __forceinline__ void out_store(T *p, T v) {
    if constexpr ((POND_STREAM_STORE & Stream) != 0)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}
template <int Stream>
__device__ __forceinline__ void out_store(float4 *p, float4 v) {
    if constexpr ((POND_STREAM_STORE & Stream) != 0)
        __builtin_nontemporal_store(pond_f4v{v.x, v.y, v.z, v.w}, reinterpret_cast<pond_f4v *>(p));
    else
        *p = v;
}
template <int Stream>
__device__ __forceinline__ void out_store(double2 *p, double2 v) {
    if constexpr ((POND_STREAM_STORE & Stream) != 0)
        __builtin_nontemporal_store(pond_d2v{v.x, v.y}, reinterpret_cast<pond_d2v *>(p));
    else
        *p = v;
}
constexpr int kStreamPops = 1, kStreamFrame = 2, kStreamMoments = 4;

template <typename P, int NMOM = kNMom>
__device__ __forceinline__ void store_moments_out(P *__restrict__ base, long long stride,
                                                  long long idx, const P *M) {
    using MV = MomVec<P, NMOM>;
    using V = typename MV::V;
    V *b = reinterpret_cast<V *>(base);
    if constexpr (MV::W == 4) {
#pragma unroll
        for (int k = 0; k < MV::G; ++k)
            out_store<kStreamMoments>(&b[k * stride + idx],
                                      V{M[4 * k], M[4 * k + 1], M[4 * k + 2], M[4 * k + 3]});
    } else {
#pragma unroll
        for (int k = 0; k < MV::G; ++k) out_store<kStreamMoments>(&b[k * stride + idx], V{M[2 * k], M[2 * k + 1]});
    }
}

template <typename P, int NMOM = kNMom>
__device__ __forceinline__ void store_moments(P *__restrict__ base, long long stride,
                                              long long idx, const P *M) {
    using MV = MomVec<P, NMOM>;
    using V = typename MV::V;
    V *b = reinterpret_cast<V *>(base);
    if constexpr (MV::W == 4) {
#pragma unroll
        for (int k = 0; k < MV::G; ++k)
            b[k * stride + idx] = V{M[4 * k], M[4 * k + 1], M[4 * k + 2], M[4 * k + 3]};
    } else {
#pragma unroll
        for (int k = 0; k < MV::G; ++k) b[k * stride + idx] = V{M[2 * k], M[2 * k + 1]};
    }
}

// LDS tiles of the FP32 D2Q16 kernels hold the moment groups of a node
// contiguously (node-major, 5 float4 = 80 B per node), so every tap and group of
// a stencil row is reached from one address with immediate offsets; lanes
// reading neighbouring nodes then touch disjoint banks (a stride of 20 banks).
// FP64 and D2Q25 stage the region as grouped planes
// instead: group k of staged node idx at vector k * cap + idx, so the lanes of
// a wave, which read neighbouring nodes, read neighbouring vectors.  Node-major
// tiles of those variants either share banks between lanes (D2Q25 FP32, 128 B
// per node: 161 against 495 MLUPS on the 512^2 Mach-2 modes) or, padded by a
// group against that, hold fewer nodes (365 MLUPS; FP64 D2Q16 at 512^2: 528
// against 657).  The staged values are the same in either layout, only their
// addresses differ.
template <typename P, class L>
constexpr bool lds_planar() {
    return !(sizeof(P) == 4 && L::Q == 16);
}

// Vectors (float4 / double2) per node of the LDS array: the node's groups.
template <typename P, class L>
constexpr int lds_stride() {
    return MomVec<P, nmom<L>()>::G;
}

// Bytes of one node in the LDS array.
template <typename P, class L>
constexpr unsigned lds_node_bytes() {
    return unsigned(lds_stride<P, L>() * sizeof(typename MomVec<P, nmom<L>()>::V));
}

template <typename P, class L>
__device__ __forceinline__ void store_node_lds(P *lds, int idx, int cap, const P *M) {
    if constexpr (lds_planar<P, L>()) {
        store_moments<P, nmom<L>()>(lds, cap, idx, M);
        return;
    }
    using MV = MomVec<P, nmom<L>()>;
    using V = typename MV::V;
    V *b = reinterpret_cast<V *>(lds) + idx * lds_stride<P, L>();
#pragma unroll
    for (int k = 0; k < MV::G; ++k) {
        if constexpr (MV::W == 4)
            b[k] = V{M[4 * k], M[4 * k + 1], M[4 * k + 2], M[4 * k + 3]};
        else
            b[k] = V{M[2 * k], M[2 * k + 1]};
    }
}

template <typename P>
__device__ __forceinline__ P *pop_plane(void *base, int i, long long N) {
    return static_cast<P *>(base) + (long long)i * N;
}
template <typename P>
__device__ __forceinline__ const P *pop_plane(const void *base, int i, long long N) {
    return static_cast<const P *>(base) + (long long)i * N;
}

static __constant__ VelocityTablesP<float> kTabF = make_velocity_tables_p<float>();
static __constant__ VelocityTablesP<double> kTabD = make_velocity_tables_p<double>();
static __constant__ LatticeTablesP<float, D2Q25> kTab25F = make_lattice_tables_p<float, D2Q25>();
static __constant__ LatticeTablesP<double, D2Q25> kTab25D = make_lattice_tables_p<double, D2Q25>();

template <typename P>
__device__ __forceinline__ const VelocityTablesP<P> &vtab();
template <>
__device__ __forceinline__ const VelocityTablesP<float> &vtab<float>() {
    return kTabF;
}
template <>
__device__ __forceinline__ const VelocityTablesP<double> &vtab<double>() {
    return kTabD;
}

// Reconstruction table of lattice L (herm; see pond_device.h).
template <typename P, class L>
__device__ __forceinline__ const auto &ltab() {
    if constexpr (L::Q == 16)
        return vtab<P>();
    else if constexpr (sizeof(P) == 4)
        return kTab25F;
    else
        return kTab25D;
}

// Moment-plane row of the (unwrapped) grid row y: periodic wrap, clamp, or with
// walls (bc 2) the ghost rows -wall_h .. -1 and ny .. ny + wall_h - 1 around
// the grid (rows further out read the last ghost row).
__device__ __forceinline__ int mom_row(int y, int ny, int bc, int wall_h) {
    if (bc == 2) return min(max(y, -wall_h), ny + wall_h - 1);
    return wrap_index(y, ny, bc);
}

// Tap source reading the HBM moment planes with periodic / clamp wrapping.
//
// Reference blocks.  The gather interpolates the deviations M - M_ref of the
// taps' moments from those of a reference node and adds M_ref's share once:
// equal to interpolating M itself (the weights sum to 1), but the rounding of
// the weights -- whose sum differs from 1 by ~1e-8 in FP32, the same way at
// every node of a uniform flow -- then scales only the deviation.  (Otherwise a
// uniform flow at rest gains or loses ~2e-8 of its mass every step, 7e-8 at
// T = 0.04.)  The reference node of a destination node is the first node of
// the aligned kRefBlockX x kRefBlockY block holding it: every tile shape
// divides the block, so a tile has one reference, and every kernel and tile
// shape interpolate the same deviations.
//
// FP64 interpolates the moments themselves (the weights' sum is 1 to 1e-16
// there): where the taps' state lies far from the reference node's, the
// populations of deviations would cancel against the reference's share, and
// lose that factor in every step (the 400 x 1 shock tube, density 1 against
// 0.125: 7e-12 off the oracle after 400 steps instead of 1e-13).
constexpr int kRefBlockX = 256, kRefBlockY = 16;
template <typename P>
constexpr bool deviations() { return sizeof(P) == 4; }
__device__ __forceinline__ long long ref_node(int x, int y, int nx) {
    return (long long)(y / kRefBlockY * kRefBlockY) * nx + (x / kRefBlockX * kRefBlockX);
}

template <typename P, int NP, class L = D2Q16>
struct GlobalTaps {
    using MV = MomVec<P, nmom<L>()>;
    using V = typename MV::V;
    static constexpr bool kStaged = false;  // no rows in LDS
    const P *mom;
    long long N;  // nodes per moment plane
    int nx, ny, bc_x, bc_y;
    long long moff;  // node offset of grid row 0
    int wall_h;
    P ref[deviations<P>() ? nmom_padded<P, L>() : 1];  // moments of the reference node

    // reads the reference of destination node (x, y)
    __device__ __forceinline__ void set_reference(int x, int y) {
        if constexpr (deviations<P>())
            load_moments<P, nmom<L>()>(mom, N, moff + ref_node(x, y, nx), ref);
    }
    __device__ __forceinline__ P ref_at(int k) const { return deviations<P>() ? ref[k] : P(0); }
    // a single grid row without walls: every stencil row is row 0
    __device__ __forceinline__ bool flat() const { return ny == 1 && bc_y != 2; }
    __device__ __forceinline__ bool inside(int, int, int, int) const { return false; }

    // A row in HBM, columns bx .. bx + NP - 1 of the (unwrapped) grid row y: (k, p) is
    // moment group k in column p, deviation(k, v) the group's value v as deviations
    // from the reference node's.
    struct Row {
        const V *base;
        long long N;
        int col[NP];
        const P *ref;
        __device__ __forceinline__ V operator()(int k, int p) const {
            return base[k * N + col[p]];
        }
        __device__ __forceinline__ V deviation(int k, V v) const {
            if constexpr (deviations<P>()) {
                v.x -= ref[4 * k];
                v.y -= ref[4 * k + 1];
                v.z -= ref[4 * k + 2];
                v.w -= ref[4 * k + 3];
            }
            return v;
        }
        __device__ __forceinline__ void next() {}  // unused: rows in HBM are visited one by one
    };
    __device__ __forceinline__ Row outside(int bx, int y) const {
        Row r;
        r.base = reinterpret_cast<const V *>(mom) + moff + (long long)mom_row(y, ny, bc_y, wall_h) * nx;
        r.N = N;
#pragma unroll
        for (int p = 0; p < NP; ++p) r.col[p] = wrap_index(bx + p, nx, bc_x);
        r.ref = ref;
        return r;
    }
    // nothing is staged
    __device__ __forceinline__ Row staged(int bx, int y) const { return outside(bx, y); }
};

// How many lanes gather a node (node_step).
enum class NodeLanes { kOne, kRegroup, kFour };

// Four lanes per node: lane j of a group of four holds x-component
// j's share.  quad_lane(v, j): the value of the group's lane j.
template <int J>
__device__ __forceinline__ int quad_lane(int v) {
    return __builtin_amdgcn_mov_dpp(v, J * 0x55, 0xf, 0xf, true);  // quad_perm [J, J, J, J]
}
template <int J>
__device__ __forceinline__ float quad_lane(float v) {
    return __int_as_float(quad_lane<J>(__float_as_int(v)));
}
template <int J>
__device__ __forceinline__ double quad_lane(double v) {
    return __hiloint2double(quad_lane<J>(__double2hiint(v)), quad_lane<J>(__double2loint(v)));
}

// Position of the k-th set bit of mask (k = 0 the lowest), which has more than k.
__device__ __forceinline__ int nth_set_bit(unsigned long long mask, int k) {
    int pos = 0;
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
        const int c = __popcll((mask >> pos) & ((1ull << w) - 1));
        const bool up = k >= c;
        k -= up ? c : 0;
        pos += up ? w : 0;
    }
    return pos;
}

// Lanes of the wave for which c holds (a ballot and a scalar bit count).
__device__ __forceinline__ unsigned long long wave_count(bool c) {
    return (unsigned long long)__popcll(__ballot(c));
}

// Moments sum_i f_i V_ix^p V_iy^q of Q populations at the velocities V_i =
// s c_i + d (c_i = (c(a), c(b)) for i = Q1 a + b; one scale s and offset d for
// all i) through the lattice sums C_pq = sum_i f_i c(a)^p c(b)^q, which the
// x-components build in turn: column_sums takes the populations f[0..Q1) of an
// x-component into S_q = sum_b f_b c(b)^q (the even and odd parts of +-c(b) first),
// column_flush adds c(a)^p S_q to C_pq; moments_from_lattice_sums expands
// (s c + d)^p by the binomial theorem at the end.  (Three operations per
// population and NM per x-component, where the monomials of each V_i and their
// products with f_i cost about 3 NM.)  Weighted: the populations come over
// their weights w(a) w(b).
template <class L, bool Weighted = false, typename P>
__device__ __forceinline__ void column_sums(const P f[L::Q1], P S[L::N + 1]) {
#pragma unroll
    for (int h = 0; h < L::Q1 / 2; ++h) {
        const double cb = L::c(L::Q1 - 1 - h);
        const P even = f[L::Q1 - 1 - h] + f[h], odd = f[L::Q1 - 1 - h] - f[h];
        double cq = Weighted ? L::w(h) : 1.0;
#pragma unroll
        for (int q = 0; q <= L::N; ++q) {
            const P k = P(cq), v = q % 2 ? odd : even;
            if (q == 0 && !Weighted)
                S[0] = h == 0 ? v : S[0] + v;
            else
                S[q] = h == 0 ? k * v : S[q] + k * v;
            cq *= cb;
        }
    }
    if constexpr (L::Q1 % 2 == 1)  // the zero abscissa
        S[0] += Weighted ? P(L::w(L::Q1 / 2)) * f[L::Q1 / 2] : f[L::Q1 / 2];
}
template <class L, bool Weighted = false, typename P>
__device__ __forceinline__ void column_flush(P C[L::NM], const P S[L::N + 1], int a) {
    const P ca = P(L::c(a));
    P cp = Weighted ? P(L::w(a)) : P(1);
#pragma unroll
    for (int p = 0; p <= L::N; ++p) {
#pragma unroll
        for (int q = 0; p + q <= L::N; ++q)
            C[mom_index(p, q)] += p == 0 && !Weighted ? S[q] : cp * S[q];
        cp *= ca;
    }
}
template <class L, typename P>
__device__ __forceinline__ void column_add(P C[L::NM], const P f[L::Q1], int a) {
    P S[L::N + 1];
    column_sums<L>(f, S);
    column_flush<L>(C, S, a);
}

template <class L, typename P>
__device__ __forceinline__ void moments_from_lattice_sums(const P C[L::NM], P s, P dx, P dy,
                                                          P M[L::NM]) {
    constexpr int N = L::N, NM = L::NM;
    P ex[N + 1], ey[N + 1], sc[N + 1];
    ex[0] = ey[0] = sc[0] = P(1);
#pragma unroll
    for (int j = 1; j <= N; ++j) {
        ex[j] = ex[j - 1] * dx;
        ey[j] = ey[j - 1] * dy;
        sc[j] = sc[j - 1] * s;
    }
    // U_rt = s^(r+t) C_rt; then T[p][t] = sum_r C(p,r) dx^(p-r) U[r][t] and
    // M[p][q] = sum_t C(q,t) dy^(q-t) T[p][t], each sum starting at its unit term
    P U[NM], T[NM];
#pragma unroll
    for (int k = 0; k < NM; ++k) {
        const int o = mom_px(k) + mom_py(k);
        U[k] = o == 0 ? C[k] : C[k] * sc[o];
    }
#pragma unroll
    for (int k = 0; k < NM; ++k) {
        const int p = mom_px(k), t = mom_py(k);
        P acc = U[k];
#pragma unroll
        for (int r = p - 1; r >= 0; --r) acc += (P(binom_c(p, r)) * ex[p - r]) * U[mom_index(r, t)];
        T[k] = acc;
    }
#pragma unroll
    for (int k = 0; k < NM; ++k) {
        const int p = mom_px(k), q = mom_py(k);
        P acc = T[k];
#pragma unroll
        for (int t = q - 1; t >= 0; --t) acc += (P(binom_c(q, t)) * ey[q - t]) * T[mom_index(p, t)];
        M[k] = acc;
    }
}

// The second moment along x (the same along y) of the float weights that an
// equilibrium of density 1 is stored with, sum_i herm[i][0] c_ix^2: the weights sum
// to 1 exactly, but this to 1 + 7.3e-8 on D2Q16 and 1 - 5.4e-8 on D2Q25.
template <class L>
constexpr double stored_second_moment() {
    const LatticeTablesP<float, L> t = make_lattice_tables_p<float, L>();
    double sum = 0.0;
    for (int i = 0; i < L::Q; ++i) sum += double(t.herm[i][0]) * L::c(i / L::Q1) * L::c(i / L::Q1);
    return sum;
}
static_assert(stored_second_moment<D2Q16>() - 1.0 < 1e-7 && 1.0 - stored_second_moment<D2Q16>() < 1e-7 &&
                  stored_second_moment<D2Q25>() - 1.0 < 1e-7 &&
                  1.0 - stored_second_moment<D2Q25>() < 1e-7,
              "the stored weights' second moment is the lattice's to rounding");

// The moments about u_ref of a node's stored populations, which the next step
// gathers, built from its x-components in turn (add) in the frame the populations
// are stored in (moments).  The zeroth moments are summed in FP64.
//
// In FP32 so are f's sums of odd order along x and its second moments along the
// axes, these in units of stored_second_moment: a uniform flow repeats the rounding
// of a float sum in every step, and the momentum and, in the non-translational
// split, the temperature are read from them.  (A symmetric f had odd float sums of
// 1e-8, which pushed the rounding of its populations one way; along y they cancel
// pair by pair.  On D2Q25 at T = 1 the float second moments summed to 1 - 6e-8, and
// T fell by 1.9e-5 in 2000 steps.)  100 random uniform flows of each split and
// lattice over 2000 steps, rms errors with float sums and populations rounded term
// by term, and with these: u / max(|u|, sqrt T) 1.5e-6 .. 2.0e-5 and 2e-14, T
// 1.2e-7 .. 1.1e-6 and 5e-8 .. 7e-8.  They cost 1 % of the time of a step.
template <typename P, class L>
struct StoredMoments {
    static constexpr int NM = L::NM, Q1 = L::Q1;
    P Cf[NM], Cg[NM];  // lattice sums
    double mass = 0.0, gzero = 0.0;
    // FP32: lattice sums of f (fodd: those of odd order in x but the first)
    double fx = 0.0, fy = 0.0, fxx = 0.0, fyy = 0.0, fodd[NM];
    __host__ __device__ static constexpr bool odd_sum(int k) {
        return mom_px(k) % 2 == 1 && mom_px(k) + mom_py(k) > 1;
    }

    __device__ __forceinline__ StoredMoments() {
#pragma unroll
        for (int k = 0; k < NM; ++k) {
            Cf[k] = Cg[k] = P(0);
            fodd[k] = 0.0;
        }
    }

    __device__ __forceinline__ void add(int ia, const P (&f)[Q1], const P (&g)[Q1]) {
        P S[L::N + 1];
        column_sums<L>(f, S);
        if constexpr (sizeof(P) == 4) {
            double m = 0.0;
#pragma unroll
            for (int b = 0; b < Q1 / 2; ++b) {
                const double cb = L::c(Q1 - 1 - b);
                const double lo = double(f[b]), hi = double(f[Q1 - 1 - b]);
                m += hi + lo;
                fy += cb * (hi - lo);
                fyy += (cb * cb) * (hi + lo);
            }
            if constexpr (Q1 % 2 == 1) m += double(f[Q1 / 2]);
            const double ca = L::c(ia);
            mass += m;
            fx += ca * m;
            fxx += (ca * ca) * m;
            double cp = ca;
#pragma unroll
            for (int p = 1; p <= L::N; p += 2) {
#pragma unroll
                for (int q = p == 1 ? 1 : 0; p + q <= L::N; ++q)
                    fodd[mom_index(p, q)] += cp * (q == 0 ? m : double(S[q]));
                cp *= ca * ca;
            }
#pragma unroll
            for (int b = 0; b < Q1; ++b) gzero += double(g[b]);
        } else {
#pragma unroll
            for (int b = 0; b < Q1; ++b) {
                mass += double(f[b]);
                gzero += double(g[b]);
            }
        }
        column_flush<L>(Cf, S, ia);
        column_add<L>(Cg, g, ia);
    }

    // M[0 .. 2 NM): f's and g's moments; frame (ux, uy, T), s = sqrt T, offset
    // (dx, dy) of its velocity from u_ref
    __device__ __forceinline__ void moments(double s, double T, double dx, double dy, P *M) {
        constexpr int k10 = mom_index(1, 0), k01 = mom_index(0, 1);
        constexpr int k20 = mom_index(2, 0), k02 = mom_index(0, 2);
        constexpr bool kSums = sizeof(P) == 4;
        if constexpr (kSums) {
            constexpr double unit = 1.0 / stored_second_moment<L>();
            fxx *= unit;
            fyy *= unit;
            Cf[0] = P(mass);
            Cf[k10] = P(fx);
            Cf[k01] = P(fy);
            Cf[k20] = P(fxx);
            Cf[k02] = P(fyy);
#pragma unroll
            for (int k = 0; k < NM; ++k)
                if (odd_sum(k)) Cf[k] = P(fodd[k]);
        }
        moments_from_lattice_sums<L>(Cf, P(s), P(dx), P(dy), M);
        moments_from_lattice_sums<L>(Cg, P(s), P(dx), P(dy), M + NM);
        M[0] = P(mass);
        M[NM] = P(gzero);
        if constexpr (kSums) {
            M[k10] = P(s * fx + dx * mass);
            M[k01] = P(s * fy + dy * mass);
            M[k20] = P(T * fxx + dx * (2.0 * s * fx + dx * mass));
            M[k02] = P(T * fyy + dy * (2.0 * s * fy + dy * mass));
        }
    }
};

// Unwrapped index range [lo, hi] of the stencils of every velocity of a node at
// coordinate x with frame velocity u and sqrt(T) = s along one axis.
template <int NP, class L = D2Q16>
__device__ __forceinline__ void stencil_extent(int x, double u, double s, int &lo, int &hi) {
    // departure coordinates x - (s c + u) for c = +-c_out bound all stencils
    const double dlo = double(x) - (s * L::c(L::Q1 - 1) + u), dhi = double(x) - (s * L::c(0) + u);
    const double clo = fmin(fmax(dlo, double(x) - 4096.0), double(x) + 4096.0);
    const double chi = fmin(fmax(dhi, double(x) - 4096.0), double(x) + 4096.0);
    if (NP == 4) {
        lo = int(floor(clo)) - 1;
        hi = int(floor(chi)) + 2;
    } else {
        lo = int(floor(clo + 0.5)) - 1;
        hi = int(floor(chi + 0.5)) + 1;
    }
}

// Velocity gradient of frame velocities (ux, uy) at grid node (x, y), for the
// internal-energy split: central differences of the four neighbours' velocities
// (wrapped or clamped like the stencil; with walls a neighbour row beyond a wall
// takes the ghost frame velocity of the wall closure, the mirror node -- here
// the node itself -- reflected about the wall velocity).
// g = (d_x u_x, d_x u_y, d_y u_x, d_y u_y).
__device__ __forceinline__ void node_gradient(const StepArgs &a, const double *__restrict__ ux,
                                              const double *__restrict__ uy, int x, int y,
                                              double g[4]) {
    const long long row = (long long)y * a.nx;
    const long long xm = row + wrap_index(x - 1, a.nx, a.bc_x);
    const long long xp = row + wrap_index(x + 1, a.nx, a.bc_x);
    const long long ym = (long long)wrap_index(y - 1, a.ny, a.bc_y) * a.nx + x;
    const long long yp = (long long)wrap_index(y + 1, a.ny, a.bc_y) * a.nx + x;
    double uxm = ux[ym], uym = uy[ym], uxp = ux[yp], uyp = uy[yp];
    if (a.bc_y == 2 && y == 0) {
        uxm = 2.0 * a.wall_ux[0] - ux[row + x];
        uym = -uy[row + x];
    }
    if (a.bc_y == 2 && y == a.ny - 1) {
        uxp = 2.0 * a.wall_ux[1] - ux[row + x];
        uyp = -uy[row + x];
    }
    g[0] = 0.5 * (ux[xp] - ux[xm]);
    g[1] = 0.5 * (uy[xp] - uy[xm]);
    g[2] = 0.5 * (uxp - uxm);
    g[3] = 0.5 * (uyp - uym);
}

// Velocity gradient of frame velocities (ux, uy) at the point (px, py): the
// bilinear interpolation of node_gradient over the four nodes around it
// (columns and rows wrapped or clamped like the stencil; with walls a row
// beyond them is the last row).  The point is clamped to a finite range first,
// so a non-physical frame still indexes inside the grid.
__device__ __forceinline__ void point_gradient(const StepArgs &a, const double *__restrict__ ux,
                                               const double *__restrict__ uy, double px, double py,
                                               double g[4]) {
    px = fmin(fmax(px, -1.0e8), 1.0e8);
    py = fmin(fmax(py, -1.0e8), 1.0e8);
    const double fx = floor(px), fy = floor(py);
    const double ax = px - fx, ay = py - fy;
    const int x0 = int(fx), y0 = int(fy);
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k] = 0.0;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int yj = wrap_index(y0 + j, a.ny, a.bc_y);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int xi = wrap_index(x0 + i, a.nx, a.bc_x);
            const double w = (i ? ax : 1.0 - ax) * (j ? ay : 1.0 - ay);
            double gn[4];
            node_gradient(a, ux, uy, xi, yj, gn);
#pragma unroll
            for (int k = 0; k < 4; ++k) g[k] += w * gn[k];
        }
    }
}

// The internal-energy split's velocity gradient for destination node (x, y)
// with time-t frame velocity (u0, u1): taken at the end of the step, where the
// collision and the source act, by linear extrapolation along the node's
// trajectory from the last two time levels, 2 G_t(x - u) - G_{t-1}(x - 2u)
// (G_t: point_gradient of the time-t frames, G_{t-1}: of the previous level's;
// exact for a velocity field advected with the flow).
__device__ __forceinline__ void source_gradient(const StepArgs &a, const DevState &src, int x,
                                                int y, double u0, double u1, double g[4]) {
    double ga[4], gb[4];
    point_gradient(a, src.ux, src.uy, double(x) - u0, double(y) - u1, ga);
    point_gradient(a, src.uxp, src.uyp, double(x) - 2.0 * u0, double(y) - 2.0 * u1, gb);
#pragma unroll
    for (int k = 0; k < 4; ++k) g[k] = 2.0 * ga[k] - gb[k];
}

}  // namespace pond

#include "pond_gather.h"

namespace pond {

// The whole step of one destination node (x, y) = node n whose time-t frame
// is (l0, l1, l2), for the energy split S (0: total energy, 1: internal
// energy, 2: non-translational energy) on lattice L; src is the time-t state
// (its frames feed the velocity gradient of the internal-energy split).  The
// node's moments of the new state (those the next step interpolates) go to
// mom_out, computed from the stored populations and frame exactly as the
// moments pre-pass computes them.  Lanes with live == false take part in the
// wave-level predictor-corrector exit and the counter reduction only.
//
// Per predictor-corrector gather (gather_rows): the populations of f and g at
// their departure points in the iterate frame, one x-component at a time; the
// FP64 sums rho, j, E and the lattice sums of the gathered populations (their
// lab moments follow once, from the last gather's) are accumulated on the fly,
// so no population array is kept.
//
// NodeLanes::kFour: four lanes share the node (every argument alike), one per x-component:
// each gathers and reconstructs its own x-component, and the sums over the
// x-components are formed by every lane, in the order of the loop over them, so
// the bits are those of one lane per node.  Small grids, whose few waves leave
// most of the chip idle, take a quarter of the gather's time per step this way.
//
// kRegroup: one lane per node, but once at most 16 of a wave's nodes are left to
// converge, they are gathered the same way, four lanes each (the wave's nodes must
// share their reference node).  Near shocks most waves iterate for a few nodes only
// (a 308^2 shock tube: 0.6 of 1.8 gathers per wave and step), and the launch ends
// with the wave of the most iterations: 0.100 / 0.065 ms per step of that tube
// without / with, 0.237 / 0.191 of the 613 x 377 quadrants in FP64.
template <typename P, int NP, int S, class L, NodeLanes Lanes, class Taps>
__device__ __forceinline__ void node_step(const StepArgs &a, const Taps &taps, int x, int y,
                                          long long n, bool live, double l0, double l1, double l2,
                                          const DevState &src, DevState dst,
                                          P *__restrict__ mom_out, DevCounters *cnt) {
    constexpr int NM = L::NM;
    const auto &tab = ltab<P, L>();
    double lg0 = l0, lg1 = l1, lg2 = l2;     // frame of the current gather
    double ln0 = lg0, ln1 = lg1, ln2 = lg2;  // frame of the gathered moments
    double rho = 1.0, gsum = 0.0;  // FP64 sums of the last gather's f and g
    P Cf[NM], Cg[NM];  // lattice sums of the last gather's populations, in its frame
#pragma unroll
    for (int k = 0; k < NM; ++k) Cf[k] = Cg[k] = P(0);
    bool done = !live, conv = false, bad = false, overrun = false;
    constexpr bool Quad = Lanes == NodeLanes::kFour;
    const int quad = Quad ? int(threadIdx.x) & 3 : 0;
    const bool owner = quad == 0;  // the lane that counts its node
    constexpr bool kRegroup = Lanes == NodeLanes::kRegroup;
    unsigned long long itc = 0;  // gathers of the wave's lanes
    // internal split: the source's velocity gradient (the same for every
    // iterate), in the arithmetic's precision
    P gxx = P(0), gxy = P(0), gyx = P(0), gyy = P(0);
    if constexpr (S == 1) {
        if (live) {
            double gr[4];
            source_gradient(a, src, x, y, l0, l1, gr);
            gxx = P(gr[0]);
            gxy = P(gr[1]);
            gyx = P(gr[2]);
            gyy = P(gr[3]);
        }
    }

    // lab moments of a gather's populations from their lattice sums C (frame scale sP,
    // offset (dux, duy) from u_ref); where the gather sums the deviations from the
    // reference moments, their share is added here (first: its place among them)
    auto lab_moments = [&](const P (&C)[NM], int first, P sP, P dux, P duy, P (&M)[NM]) {
        moments_from_lattice_sums<L>(C, sP, dux, duy, M);
        if constexpr (deviations<P>()) {
#pragma unroll
            for (int k = 0; k < NM; ++k) M[k] += taps.ref_at(first + k);
        }
    };

    struct Sums {
        double sr, r, mx, my, m2, Eg;
    };
    // The gather of node (gx, gy) in the frame (g0, g1, g2): the FP64 sums and the
    // lattice sums of its populations.  four: by a group of four lanes (see above).
    auto gather = [&](auto four, int gx, int gy, double g0, double g1, double g2, Sums &o,
                      P (&Of)[NM], P (&Og)[NM]) {
        constexpr bool kFour = decltype(four)::value;
        double s, isd;
        frame_scale(g2, s, isd);
        const P dux = P(g0 - a.uref_x), duy = P(g1 - a.uref_y), is = P(isd);
        const double sr = rounded_scale(s, is);
        // departure coordinates x - (s c + u) = (x - u) - s c, from the iterate
        // frame clamped to a finite range (a non-physical iterate, which the
        // test below flags, must still index inside the grid)
        const double sc = fmin(fmax(s, 0.0), 1.0e6);
        const double xu = double(gx) - fmin(fmax(g0, -1.0e8), 1.0e8);
        const double yu = double(gy) - fmin(fmax(g1, -1.0e8), 1.0e8);
        o = Sums{sr, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < NM; ++k) Of[k] = Og[k] = P(0);
        // x-component ia's populations gathered in the iterate frame, over their
        // weights: the FP64 sums of f, f c and g (and f |c|^2), and the lattice sums
        auto add = [&](int ia, double s0, double s1, double s2, double sg,
                       const P (&Sf)[L::N + 1], const P (&Sg)[L::N + 1]) {
            const double ca = L::c(ia), wa = gather_weight<P, L>(ia);
            s0 *= wa;
            o.r += s0;
            o.mx += ca * s0;
            o.my += wa * s1;
            if constexpr (S == 2) o.m2 += ca * ca * s0 + wa * s2;
            o.Eg += wa * sg;
            column_flush<L, true>(Of, Sf, ia);
            column_flush<L, true>(Og, Sg, ia);
        };
        auto column = [&](int ia, const P (&f)[L::Q1], const P (&g)[L::Q1]) {
            double s0 = 0.0, s1 = 0.0, s2 = 0.0, sg = 0.0;
#pragma unroll
            for (int b = 0; b < L::Q1; ++b) {
                const double fd = double(f[b]), cb = L::c(b);
                const double wb = gather_weight<P, L>(b);
                s0 += wb * fd;
                if (cb != 0.0) s1 += (wb * cb) * fd;
                if constexpr (S == 2) s2 += (wb * cb * cb) * fd;
                sg += wb * double(g[b]);
            }
            P Sf[L::N + 1], Sg[L::N + 1];
            column_sums<L, true>(f, Sf);
            column_sums<L, true>(g, Sg);
            if constexpr (kFour) {
                auto from = [&](auto lane) {
                    constexpr int J = decltype(lane)::value;
                    P Tf[L::N + 1], Tg[L::N + 1];
#pragma unroll
                    for (int q = 0; q <= L::N; ++q) {
                        Tf[q] = quad_lane<J>(Sf[q]);
                        Tg[q] = quad_lane<J>(Sg[q]);
                    }
                    add(J, quad_lane<J>(s0), quad_lane<J>(s1),
                        S == 2 ? quad_lane<J>(s2) : 0.0, quad_lane<J>(sg), Tf, Tg);
                };
                from(std::integral_constant<int, 0>{});
                from(std::integral_constant<int, 1>{});
                from(std::integral_constant<int, 2>{});
                from(std::integral_constant<int, 3>{});
            } else {
                add(ia, s0, s1, s2, sg, Sf, Sg);
            }
        };
        gather_rows<P, NP, L, kFour>(taps, xu, yu, sc, dux, duy, is, P(sr * sr), column);
    };

    for (int it = 0; it < a.pc_max_iter; ++it) {
        const unsigned long long open = __ballot(!done);
        itc += (unsigned long long)__popcll(open) / (Quad ? 4 : 1);
        Sums o{};
        if (!kRegroup || __popcll(open) > 16) {
            if (!done)
                gather(std::integral_constant<bool, Quad>{}, x, y, lg0, lg1, lg2, o, Cf, Cg);
        } else if constexpr (kRegroup) {
            // a few nodes are left: four lanes for each, whether their own nodes are
            // done or not; group k takes the k-th node left
            const int k = (int(threadIdx.x) & 63) >> 2;
            const bool mine = k < __popcll(open);
            const int from = nth_set_bit(open, mine ? k : 0);
            Sums q{};
            P Kf[NM], Kg[NM];
            const int gx = __shfl(x, from), gy = __shfl(y, from);
            const double g0 = __shfl(lg0, from), g1 = __shfl(lg1, from), g2 = __shfl(lg2, from);
            if (mine) gather(std::true_type{}, gx, gy, g0, g1, g2, q, Kf, Kg);
            const int group = 4 * __popcll(open & ((1ull << (threadIdx.x & 63)) - 1));
            const int at = done ? 0 : group;
            o.sr = __shfl(q.sr, at);
            o.r = __shfl(q.r, at);
            o.mx = __shfl(q.mx, at);
            o.my = __shfl(q.my, at);
            if constexpr (S == 2) o.m2 = __shfl(q.m2, at);
            o.Eg = __shfl(q.Eg, at);
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                const P f = __shfl(Kf[i], at), g = __shfl(Kg[i], at);
                if (!done) {
                    Cf[i] = f;
                    Cg[i] = g;
                }
            }
        }
        if (!done) {
            if (a.bc_y == 2) {
                // walls: every stencil row must lie within the ghost rows
                double s, isd;
                frame_scale(lg2, s, isd);
                int lo, hi;
                stencil_extent<NP, L>(y, lg1, s, lo, hi);
                if (lo < -a.wall_h || hi > a.ny - 1 + a.wall_h) overrun = true;
            }
            const double sr = o.sr, mx = o.mx, my = o.my, m2 = o.m2;
            double r = o.r, Eg = o.Eg;
            // momentum, and in the non-translational split the energy f carries, at
            // the velocities C = s c + u of the iterate frame
            double jx = sr * mx + lg0 * r, jy = sr * my + lg1 * r, E = Eg;
            if constexpr (S == 2)
                E += 0.5 * (sr * sr * m2 + 2.0 * sr * (lg0 * mx + lg1 * my) +
                            (lg0 * lg0 + lg1 * lg1) * r);
            if constexpr (deviations<P>()) {
                // the reference moments' share of the sums (moments about u_ref; the lab
                // velocity is V + u_ref), added once after the deviations'
                const double m00 = double(taps.ref_at(0));
                const double m10 = double(taps.ref_at(mom_index(1, 0)));
                const double m01 = double(taps.ref_at(mom_index(0, 1)));
                r += m00;
                jx += m10 + a.uref_x * m00;
                jy += m01 + a.uref_y * m00;
                E += double(taps.ref_at(NM));
                if constexpr (S == 2) {
                    Eg += double(taps.ref_at(NM));
                    const double m20 = double(taps.ref_at(mom_index(2, 0)));
                    const double m02 = double(taps.ref_at(mom_index(0, 2)));
                    E += 0.5 * (m20 + m02) + a.uref_x * m10 + a.uref_y * m01 +
                         0.5 * (a.uref_x * a.uref_x + a.uref_y * a.uref_y) * m00;
                }
            }
            rho = r;
            gsum = S == 2 ? Eg : E;
            const double rinv = 1.0 / r;
            ln0 = jx * rinv;
            ln1 = jy * rinv;

            // total split: sum g = E = rho c_v T + |j|^2 / (2 rho); internal: sum g = rho c_v T;
            // non-translational: E = sum g + sum f |C|^2 / 2 = rho c_v T + |j|^2 / (2 rho)
            if constexpr (S == 1) {
                // the energy of the step's middle, U = sum g + (sum G) / 2, with the
                // source's sum G = -(omega / 2) rho T div u - (1 - omega / 2) P : grad u
                // (P the pressure tensor of the gathered f about u, from its moments
                // about u_ref): rho c_v T = U solved for T
                P Mf[NM];
                lab_moments(Cf, 0, P(sr), P(lg0 - a.uref_x), P(lg1 - a.uref_y), Mf);
                const double dx = ln0 - a.uref_x, dy = ln1 - a.uref_y;
                const double m00 = double(Mf[mom_index(0, 0)]), m10 = double(Mf[mom_index(1, 0)]);
                const double m01 = double(Mf[mom_index(0, 1)]), m20 = double(Mf[mom_index(2, 0)]);
                const double m11 = double(Mf[mom_index(1, 1)]), m02 = double(Mf[mom_index(0, 2)]);
                const double Pxx = m20 - 2.0 * dx * m10 + dx * dx * m00;
                const double Pxy = m11 - dx * m01 - dy * m10 + dx * dy * m00;
                const double Pyy = m02 - 2.0 * dy * m01 + dy * dy * m00;
                const double PdU = Pxx * double(gxx) + Pxy * (double(gxy) + double(gyx)) +
                                   Pyy * double(gyy);
                ln2 = (E - 0.5 * (1.0 - 0.5 * a.omega) * PdU) /
                      (r * (a.cv + 0.25 * a.omega * (double(gxx) + double(gyy))));
            } else
                ln2 = (E - 0.5 * (jx * ln0 + jy * ln1)) * (rinv * a.rcv);
            if (!(r > 0.0) || !(ln2 > 0.0) || !isfinite(ln0) || !isfinite(ln1) || !isfinite(ln2) ||
                !isfinite(E)) {
                bad = true;
                done = true;
            } else {
                // du / sqrt(T) <= tol and dT / Tscale <= tol, without the divisions
                const double du = fmax(fabs(ln0 - lg0), fabs(ln1 - lg1));
                // FP64: the change of T relative to T.  FP32: relative to the scale of
                // the energy T is recovered from, E / (rho c_v) (T itself in the internal
                // split, T + |u|^2 / (2 c_v) in the total split): single-precision
                // populations resolve E, and so T, only to a fraction of that scale
                double Tscale = ln2;
                if constexpr (sizeof(P) == 4) Tscale = E * (rinv * a.rcv);
                const double dT = fabs(ln2 - lg2);
                if (du * du <= a.pc_tol * a.pc_tol * ln2 && dT <= a.pc_tol * Tscale) {
                    conv = true;
                    done = true;
                } else if (it + 1 < a.pc_max_iter) {
                    lg0 = ln0;
                    lg1 = ln1;
                    lg2 = ln2;
                }
            }
        }
        if (__all(done)) break;  // wave-uniform exit once every lane has converged
    }

    if (live) {
        P Mf[NM], Mg[NM];  // about u_ref
        {
            // the last gather's frame (lam is only advanced when another gather follows)
            double s, isd;
            frame_scale(lg2, s, isd);
            const P sP = P(rounded_scale(s, P(isd)));
            const P dux = P(lg0 - a.uref_x), duy = P(lg1 - a.uref_y);
            lab_moments(Cf, 0, sP, dux, duy, Mf);
            lab_moments(Cg, NM, sP, dux, duy, Mg);
        }
        // re-projection onto lam* = (ln0, ln1, ln2): Grad coefficients there
        double sT, isT;
        frame_scale(ln2, sT, isT);
        const P is = P(isT);
        const P tx = P(ln0 - a.uref_x), ty = P(ln1 - a.uref_y);
        P m[NM], af[NM], ag[NM];
        // the zeroth moments are the exact FP64 sums of the gathered populations,
        // rounded once: a float sum of the Q populations loses ~1e-7 of the mass
        // in a way that repeats from step to step in a near-uniform flow (a
        // drift); in FP64 the two are the same sums
        Mf[0] = P(rho);
        Mg[0] = P(gsum);
        if constexpr (L::Q == 16) {
            central_normalised(Mf, tx, ty, is, m);
            hermite_from_central(m, af);
            central_normalised(Mg, tx, ty, is, m);
            hermite_from_central(m, ag);
        } else {
            central_normalised_n<L>(Mf, tx, ty, is, m);
            hermite_from_central_n<L>(m, af);
            central_normalised_n<L>(Mg, tx, ty, is, m);
            hermite_from_central_n<L>(m, ag);
        }

        // BGK collision in lam*, on the Grad coefficients.
        // f: f^eq = rho w_i has only a0; every higher coefficient decays by (1 - omega).
        // g, total split: g^eq = w_i [rho (c_v - 1) T + rho |C_i|^2 / 2] has
        //    a0 = rho c_v T + rho |u|^2 / 2, a1 = rho sqrt(T) u, a2 = rho T I, a3 = 0;
        // g, internal split: C_i - u in place of C_i, so a0 = rho c_v T, a1 = 0;
        // g, non-translational split: g^eq = w_i rho (c_v - 1) T, a0 only.
        const double om = a.omega;
        double geq[NM];
#pragma unroll
        for (int k = 0; k < NM; ++k) geq[k] = 0.0;
        if constexpr (S == 1) {
            geq[0] = rho * a.cv * ln2;
            geq[1] = geq[2] = 0.0;
        } else if constexpr (S == 2) {
            geq[0] = rho * (a.cv - 1.0) * ln2;
        } else {
            geq[0] = rho * (a.cv - 1.0) * ln2 + 0.5 * rho * (2.0 * ln2 + ln0 * ln0 + ln1 * ln1);
            geq[1] = rho * sT * ln0;
            geq[2] = rho * sT * ln1;
        }
        if constexpr (S != 2) {
            geq[3] = rho * ln2;
            geq[4] = 0.0;
            geq[5] = rho * ln2;
            geq[6] = geq[7] = geq[8] = geq[9] = 0.0;
        }
        if (S == 1 || S == 2 || a.unit_prandtl) {
            // internal split: the flux of g is the heat flux alone, relaxed at omega_1
            // (omega at Pr = 1); the non-translational split runs at Pr = 1 only
            const double og = a.unit_prandtl ? om : a.omega1;
#pragma unroll
            for (int k = 0; k < NM; ++k) ag[k] = ag[k] + P(og) * (P(geq[k]) - ag[k]);
        } else {
            // quasi-equilibrium: energy flux of g^eq plus the viscous heating u . P^neq,
            // P^neq = T a2(f) + sqrt(T) (u a1(f) + a1(f) u) in lam*.
            const double a1x = double(af[1]), a1y = double(af[2]);
            const double Pxx = ln2 * double(af[3]) + sT * 2.0 * ln0 * a1x;
            const double Pxy = ln2 * double(af[4]) + sT * (ln0 * a1y + a1x * ln1);
            const double Pyy = ln2 * double(af[5]) + sT * 2.0 * ln1 * a1y;
            const double dqx = ln0 * Pxx + ln1 * Pxy;
            const double dqy = ln0 * Pxy + ln1 * Pyy;
            double gqe[NM];
#pragma unroll
            for (int k = 0; k < NM; ++k) gqe[k] = geq[k];
            gqe[1] += dqx * isT;
            gqe[2] += dqy * isT;
            const double om1 = a.omega1;
#pragma unroll
            for (int k = 0; k < NM; ++k)
                ag[k] = ag[k] + P(om1) * (P(gqe[k]) - ag[k]) + P(om) * (P(geq[k]) - P(gqe[k]));
        }
        // internal split: source of the g-equation, S_i = -f_i (C_i - u) . (a + C_i . grad u)
        // with f the step's time-centred population (the mean of the re-projected
        // pre-collision and the collided f: a0 and (1 - omega / 2) times the higher
        // coefficients, whose stress is the physical one), a = d_t u = u* - u(t),
        // grad u from source_gradient; g receives (1 - omega_g / 2) S, omega_g its
        // relaxation rate (its equilibrium already holds the other half of sum S)
        P afp[NM];
        P ax = P(0), ay = P(0), src_w = P(0);
        if constexpr (S == 1) {
            const P half_decay = P(1.0 - 0.5 * om);
            afp[0] = af[0];
#pragma unroll
            for (int k = 1; k < NM; ++k) afp[k] = af[k] * half_decay;
            // the time-t velocity is read again rather than kept live across the loop
            ax = P(ln0 - src.ux[n]);
            ay = P(ln1 - src.uy[n]);
            src_w = P(1.0 - 0.5 * (a.unit_prandtl ? om : a.omega1));
        }
        const P decay = P(1.0 - om);
#pragma unroll
        for (int k = 1; k < NM; ++k) af[k] *= decay;
        // a non-physical node's populations are all NaN
        if (bad) af[0] = ag[0] = P(NAN);

        // reconstruct and store the post-collision populations, and accumulate the
        // moments of the stored values about u_ref (the next step's taps)
        const P sTP = P(sT), u0 = P(ln0), u1 = P(ln1);
        const double Tst = bad ? NAN : ln2, uxst = bad ? NAN : ln0, uyst = bad ? NAN : ln1;
        P MM[nmom_padded<P, L>()];
#pragma unroll
        for (int k = 0; k < nmom_padded<P, L>(); ++k) MM[k] = P(0);
        StoredMoments<P, L> sums;
        // x-component ia's post-collision populations, stored
        auto rebuild = [&](int ia, P (&fc)[L::Q1], P (&gc)[L::Q1]) {
#pragma unroll
            for (int b = 0; b < L::Q1; ++b) {
                const int i = L::Q1 * ia + b;
                // the small terms first, the weight's last: one rounding at the
                // population's own size, where adding them to it one by one rounds each
                P fv = P(0), gv = P(0);
#pragma unroll
                for (int k = NM - 1; k >= 0; --k) {
                    fv += tab.herm[i][k] * af[k];
                    gv += tab.herm[i][k] * ag[k];
                }
                if constexpr (S == 1) {
                    P ft = P(0);
#pragma unroll
                    for (int k = 0; k < NM; ++k) ft += tab.herm[i][k] * afp[k];
                    const P ex = sTP * P(L::c(ia)), ey = sTP * P(L::c(b));
                    const P Cx = ex + u0, Cy = ey + u1;
                    gv -= src_w * ft * (ex * (ax + Cx * gxx + Cy * gyx) + ey * (ay + Cx * gxy + Cy * gyy));
                }
                out_store<kStreamPops>(&pop_plane<P>(dst.f, i, a.N)[n], fv);
                out_store<kStreamPops>(&pop_plane<P>(dst.g, i, a.N)[n], gv);
                fc[b] = fv;
                gc[b] = gv;
            }
        };
        if constexpr (Quad) {
            P fc[L::Q1], gc[L::Q1];
            rebuild(quad, fc, gc);
            auto from = [&](auto lane) {
                constexpr int J = decltype(lane)::value;
                P fj[L::Q1], gj[L::Q1];
#pragma unroll
                for (int b = 0; b < L::Q1; ++b) {
                    fj[b] = quad_lane<J>(fc[b]);
                    gj[b] = quad_lane<J>(gc[b]);
                }
                sums.add(J, fj, gj);
            };
            from(std::integral_constant<int, 0>{});
            from(std::integral_constant<int, 1>{});
            from(std::integral_constant<int, 2>{});
            from(std::integral_constant<int, 3>{});
        } else {
#pragma unroll 1
            for (int ia = 0; ia < L::Q1; ++ia) {
                P fc[L::Q1], gc[L::Q1];
                rebuild(ia, fc, gc);
                sums.add(ia, fc, gc);
            }
        }
        sums.moments(bad ? NAN : sT, Tst, uxst - a.uref_x, uyst - a.uref_y, MM);
        if (owner) {
            out_store<kStreamFrame>(&dst.ux[n], uxst);
            out_store<kStreamFrame>(&dst.uy[n], uyst);
            out_store<kStreamFrame>(&dst.T[n], Tst);
            if constexpr (S == 1) {
                // the time-t frame becomes the new state's previous level (read again
                // rather than kept live across the loop)
                out_store<kStreamFrame>(&dst.uxp[n], src.ux[n]);
                out_store<kStreamFrame>(&dst.uyp[n], src.uy[n]);
            }
            store_moments_out<P, nmom<L>()>(mom_out, a.mstride, a.moff + n, MM);
        }
    }

    // counters: one atomic per wave
    const unsigned long long nc = wave_count(live && owner && !conv && !bad);
    const unsigned long long nb = wave_count(live && owner && bad);
    const unsigned long long no = wave_count(live && owner && overrun);
    if ((threadIdx.x & 63) == 0) {
        DevCounters::Slot *slot = &cnt->slot[blockIdx.x % kCounterSlots];
        if (itc) atomicAdd(&slot->pc_iterations, itc);
        if (nc) atomicAdd(&slot->nonconverged, nc);
        if (nb) atomicAdd(&slot->nonphysical, nb);
        if (no) atomicAdd(&slot->ghost_overrun, no);
    }
}

}  // namespace pond
