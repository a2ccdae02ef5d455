// pond_tile.h -- one block's share of the PonD step: a rectangular tile of
// destination nodes whose source moments are staged in LDS.  Shared by the
// single-instance tiled kernel (tile shape fixed at compile time) and the
// batched kernel (shape chosen per instance at run time).
#pragma once

#include "pond_step_common.h"

namespace pond {

// Tap source of a tile: the moments of the block's source region (unwrapped
// rectangle [X0, X1] x [Y0, Y1], W wide, row-major) staged in LDS (in FP32 as
// deviations from the tile's reference node, rounded as GlobalTaps rounds them:
// both give the same bits), cap nodes at most; rows whose stencil leaves the region read
// HBM.  With a single grid row the region is that row.
template <typename P, int NP, class L = D2Q16>
struct TileTaps {
    using MV = MomVec<P, nmom<L>()>;
    using V = typename MV::V;
    static constexpr bool kStaged = true;
    const P *lds;
    int cap, X0, Y0, X1, Y1, W;
    GlobalTaps<P, NP, L> glob;

    __device__ __forceinline__ P ref_at(int k) const { return glob.ref[k]; }
    __device__ __forceinline__ bool flat() const { return glob.flat(); }
    // columns bx .. bx + m - 1 of rows r .. r + n - 1 are staged
    __device__ __forceinline__ bool inside(int bx, int m, int r, int n) const {
        return bx >= X0 && bx + m - 1 <= X1 && (flat() || (r >= Y0 && r + n - 1 <= Y1));
    }

    // A staged row from column bx: (k, p) is moment group k of the node in column
    // bx + p; next() moves to the row above.  Byte offsets: the region is under 2^24
    // bytes, so the products are 24-bit multiplies (full rate, where 32-bit ones take
    // four cycles).
    struct Row {
        const char *base;
        unsigned off, pitch;
        int cap;
        __device__ __forceinline__ V operator()(int k, int p) const {
            if constexpr (lds_planar<P, L>())
                return *reinterpret_cast<const V *>(base + off + unsigned(k * cap) * sizeof(V) +
                                                    unsigned(p * sizeof(V)));
            else
                return *reinterpret_cast<const V *>(base + off +
                                                    unsigned(p) * lds_node_bytes<P, L>() +
                                                    unsigned(k * sizeof(V)));
        }
        __device__ __forceinline__ V deviation(int, V v) const { return v; }  // staged as such
        __device__ __forceinline__ void next() { off += pitch; }
    };
    __device__ __forceinline__ Row staged(int bx, int r) const {
        constexpr unsigned NB = lds_planar<P, L>() ? sizeof(V) : lds_node_bytes<P, L>();
        const unsigned pitch = flat() ? 0u : unsigned(W) * NB;
        return Row{reinterpret_cast<const char *>(lds),
                   unsigned(__umul24(unsigned(flat() ? 0 : r - Y0), pitch)) +
                       unsigned(__umul24(unsigned(bx - X0), NB)),
                   pitch, cap};
    }
    __device__ __forceinline__ auto outside(int bx, int r) const { return glob.outside(bx, r); }
};

// Ints of shared memory of block_bounds for a block of NT lanes: four per wave.
template <int NT>
constexpr int bound_slots() {
    return 4 * ((NT + 63) / 64);
}

// Minimum over the wave, in every lane: data-parallel shifts within rows of 16
// lanes, then across them (the last lane holds the result).
__device__ __forceinline__ int wave_min(int v) {
    constexpr int kMax = 0x7fffffff;
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x111, 0xf, 0xf, false));  // row_shr:1
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x112, 0xf, 0xf, false));  // row_shr:2
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x114, 0xf, 0xf, false));  // row_shr:4
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x118, 0xf, 0xf, false));  // row_shr:8
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x142, 0xa, 0xf, false));  // row_bcast:15
    v = min(v, __builtin_amdgcn_update_dpp(kMax, v, 0x143, 0xc, 0xf, false));  // row_bcast:31
    return __builtin_amdgcn_readlane(v, 63);
}

// Minima of four values over the block (NT lanes, every one calling); one
// barrier, none for a single wave.  red: bound_slots<NT>() ints.
template <int NT>
__device__ __forceinline__ void block_bounds(int (&v)[4], int *red) {
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = wave_min(v[k]);
    if constexpr (NT > 64) {
        const int w = int(threadIdx.x) / 64;
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) red[4 * w + k] = v[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            int r = red[k];
#pragma unroll
            for (int u = 1; u < NT / 64; ++u) r = min(r, red[4 * u + k]);
            v[k] = __builtin_amdgcn_readfirstlane(r);
        }
    }
}

// Minimum waves per SIMD asked of the register allocator for the step kernels.  FP32 needs nearly 256 VGPRs: two waves (three, at 168 VGPRs,
// spill 36 of them: 2048^2 quadrants 0.82 against 0.71 ms per step, 512^2 Mach 2
// 0.117 against 0.113).  FP64 holds the weight table and a row in twice the
// registers: one wave of 512 (two spill 130: 512^2 Mach 2 0.51 against 0.34 ms).
template <typename P>
constexpr int step_min_waves() {
    return sizeof(P) == 4 ? 2 : 1;
}

// Blocks are dispatched round-robin over the 8 XCDs (block b on XCD b % 8);
// give each XCD a contiguous range of tiles so that neighbouring tiles, which
// share halo moments, share that XCD's L2.
__device__ __forceinline__ int xcd_tile(int b, int nb) {
    const int q = nb / 8, r = nb % 8, x = b % 8;
    return x * q + (x < r ? x : r) + b / 8;
}

// Order of the tiles within the range: column bands about POND_BAND_NODES
// nodes wide (0: plain row-major order), each walked row by row.  The blocks an
// XCD holds at once take consecutive tiles, so in row-major order they form a
// strip one tile high across the grid (8 x 2048 nodes for 8 x 8 tiles on
// 2048^2), whose source region carries halo rows above and below every tile;
// in a band they form a square of about POND_BAND_NODES^2 nodes, whose halo is
// only its perimeter.  (The halo rows shared with the previous set of tiles are
// gone from L2 by then either way: each set writes more than L2 holds.)  Off by
// default: on the 2048^2 quadrants bands of 128 (256) nodes cut the step's HBM
// reads by 21 % (25 %) but lengthened it by 6 % (a band's set of tiles spans
// 128 rows of every plane where a strip spans 8); on 512^2 the order made no
// difference.
#ifndef POND_BAND_NODES
#define POND_BAND_NODES 0
#endif
template <int TX>
__device__ __forceinline__ void band_tile(int t, int tiles_x, int tiles_y, int &tx, int &ty) {
    constexpr int bw = POND_BAND_NODES / TX > 1 ? POND_BAND_NODES / TX : 1;  // tiles per band
    if constexpr (POND_BAND_NODES == 0 || bw == 1) {
        tx = t % tiles_x;
        ty = t / tiles_x;
    } else {
        const int full = tiles_x / bw, per = bw * tiles_y;  // full bands, tiles per band
        if (t < full * per) {
            const int band = t / per, r = t - band * per;
            ty = r / bw;
            tx = band * bw + (r - ty * bw);
        } else {
            // the last band, narrower (tiles_x is no multiple of bw)
            const int w = tiles_x - full * bw, r = t - full * per;
            ty = r / w;
            tx = full * bw + (r - ty * w);
        }
    }
}

// Tile shapes: TX x TY destination nodes, one lane each: lane t at (t % TX, t / TX),
// in 16-wide tiles within pairs of rows so that the lanes which a 16-byte LDS
// read serves together -- 0-3, 12-15, 20-23 and 24-27 of each 32, and the other
// sixteen -- are those of one row: neighbouring staged nodes, which lie on
// different banks, where two rows' would share some (2048^2 quadrants, 16 x 8
// tiles in row order: 47 % of the LDS cycles were conflicts).
__device__ __forceinline__ int pair_row(int t) {  // of lane t, 0 or 1
    return (0x96 >> ((t >> 2) & 7)) & 1;          // odd parity of its group of four
}
__device__ __forceinline__ int pair_column(int t) { return ((t >> 1) & 12) | (t & 3); }

template <int TX, int TY>
struct FixedShape {
    static constexpr int kThreads = TX * TY;
    __device__ __forceinline__ int tx() const { return TX; }
    __device__ __forceinline__ int ty() const { return TY; }
    __device__ __forceinline__ int lx(int t) const { return TX == 16 ? pair_column(t) : t % TX; }
    __device__ __forceinline__ int ly(int t) const {
        return TX == 16 ? 2 * (t / 32) + pair_row(t) : t / TX;
    }
};
// 256 lanes, TX = 2^lg, TY = 256 / TX.
struct Shape256 {
    static constexpr int kThreads = 256;
    int lg;
    __device__ __forceinline__ int tx() const { return 1 << lg; }
    __device__ __forceinline__ int ty() const { return 256 >> lg; }
    __device__ __forceinline__ int lx(int t) const {
        return lg == 4 ? pair_column(t) : t & ((1 << lg) - 1);
    }
    __device__ __forceinline__ int ly(int t) const {
        return lg == 4 ? 2 * (t >> 5) + pair_row(t) : t >> lg;
    }
};

// Source region of a tile: the union [X0, X1] x [Y0, Y1] of its lanes'
// predictor stencils.  When that exceeds cap nodes, the parts sticking out of
// the tile are cut to at most h nodes per side, with the largest h whose
// region fits (h = 0, the tile itself, always fits); an asymmetric halo (the
// upwind side of an advected flow) is kept whole when it fits.  A single-row
// grid stages one row.
__device__ __forceinline__ void clip_region(int tx0, int ty0, int tx, int ty, int cap, bool flat_y,
                                            int &X0, int &X1, int &Y0, int &Y1) {
    if (flat_y) Y0 = Y1 = 0;
    if (X1 < X0 || Y1 < Y0) return;  // no live lane
    const int tx1 = tx0 + tx - 1, ty1 = ty0 + ty - 1;
    auto area = [&](int h) {
        const long long w = (long long)min(X1, tx1 + h) - max(X0, tx0 - h) + 1;
        const long long v = flat_y ? 1 : (long long)min(Y1, ty1 + h) - max(Y0, ty0 - h) + 1;
        return w * v;
    };
    int hi = max(max(tx0 - X0, X1 - tx1), flat_y ? 0 : max(ty0 - Y0, Y1 - ty1));
    if (hi <= 0 || area(hi) <= cap) return;
    int lo = 0;  // area(lo) <= cap < area(hi)
    while (hi - lo > 1) {
        const int mid = lo + (hi - lo) / 2;
        if (area(mid) <= cap)
            lo = mid;
        else
            hi = mid;
    }
    X0 = max(X0, tx0 - lo);
    X1 = min(X1, tx1 + lo);
    if (!flat_y) {
        Y0 = max(Y0, ty0 - lo);
        Y1 = min(Y1, ty1 + lo);
    }
}

// The tile with first node (tx0, ty0): load the time-t frames, bound the
// source region (clip_region), stage the region's moments, then run every
// lane's node step (energy split S, lattice L; Quad: four lanes per node, so a
// block of four times the tile's lanes).  Every thread of the block must
// call it (it synchronises the block).  red: bound_slots ints
// of shared memory for the block's lanes.
template <typename P, int NP, int S, class L, bool Quad = false, class Shape>
__device__ __forceinline__ void tile_step(const StepArgs &a, DevState src, const P *__restrict__ mom,
                                          DevState dst, P *__restrict__ mom_out, DevCounters *cnt,
                                          P *lds, int cap, int tx0, int ty0, Shape sh, int *red) {
    constexpr int kLanes = Quad ? 4 : 1;  // per node
    const int nthreads = kLanes * sh.tx() * sh.ty(), t = int(threadIdx.x) / kLanes;
    const int x = tx0 + sh.lx(t), y = ty0 + sh.ly(t);
    const bool live = x < a.nx && y < a.ny;
    const long long n = live ? (long long)y * a.nx + x : 0;
    double l0 = 0.0, l1 = 0.0, l2 = 1.0;
    if (live) {
        l0 = src.ux[n];
        l1 = src.uy[n];
        l2 = src.T[n];
    }

    constexpr int kFar = 1 << 30;
    int lx = kFar, hx = -kFar, ly = kFar, hy = -kFar;
    if (live && isfinite(l0) && isfinite(l1) && l2 > 0.0 && isfinite(l2)) {
        const double s = sqrt(l2);
        stencil_extent<NP, L>(x, l0, s, lx, hx);
        stencil_extent<NP, L>(y, l1, s, ly, hy);
    }
    const bool flat_y = a.ny == 1 && a.bc_y != 2;  // walls: the ghost rows differ
    int bound[4] = {lx, -hx, ly, -hy};
    block_bounds<kLanes * Shape::kThreads>(bound, red);
    int X0 = bound[0], X1 = -bound[1], Y0 = bound[2], Y1 = -bound[3];
    clip_region(tx0, ty0, sh.tx(), sh.ty(), cap, flat_y, X0, X1, Y0, Y1);
    const int W = X1 >= X0 ? X1 - X0 + 1 : 0;
    const int H = Y1 >= Y0 ? Y1 - Y0 + 1 : 0;

    // the tile's reference moments (every node of the tile shares its block)
    GlobalTaps<P, NP, L> glob{mom, a.mstride, a.nx, a.ny, a.bc_x, a.bc_y, a.moff, a.wall_h, {}};
    glob.set_reference(tx0, ty0);

    // kStage nodes per lane at a time, their loads in flight together; rows and
    // columns by a multiplication with 2^32 / W (exact: the region holds few nodes)
    constexpr int kStage = sizeof(P) == 4 ? 3 : 2;
    const int count = W * H;
    const unsigned inv = W > 1 ? 0xffffffffu / unsigned(W) + 1u : 0u;
    for (int base = int(threadIdx.x); base < count; base += kStage * nthreads) {
        P M[kStage][nmom_padded<P, L>()];
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            const int idx = min(base + u * nthreads, count - 1);
            const int row = W > 1 ? int(__umulhi(unsigned(idx), inv)) : idx;
            const int gx = wrap_index(X0 + idx - row * W, a.nx, a.bc_x);
            const int gy = mom_row(Y0 + row, a.ny, a.bc_y, a.wall_h);
            load_moments<P, nmom<L>()>(mom, a.mstride, a.moff + (long long)gy * a.nx + gx, M[u]);
        }
#pragma unroll
        for (int u = 0; u < kStage; ++u) {
            const int idx = base + u * nthreads;
            if (idx >= count) break;
            if constexpr (deviations<P>()) {
#pragma unroll
                for (int k = 0; k < nmom<L>(); ++k) M[u][k] -= glob.ref[k];
            }
            store_node_lds<P, L>(lds, idx, cap, M[u]);
        }
    }
    __syncthreads();

    const TileTaps<P, NP, L> taps{lds, cap, X0, Y0, X1, Y1, W, glob};
    // regrouping costs registers, which FP64 blocks of 512 lanes lack (256 per lane:
    // 0.36 against 0.29 ms per step of 512^2, Mach 2)
    constexpr NodeLanes kNodeLanes =
        Quad ? NodeLanes::kFour
        : L::Q1 == 4 && (sizeof(P) == 4 || Shape::kThreads <= 256) ? NodeLanes::kRegroup
                                                                   : NodeLanes::kOne;
    node_step<P, NP, S, L, kNodeLanes>(a, taps, x, y, n, live, l0, l1, l2, src, dst, mom_out, cnt);
}

// Moments up to the lattice's Grad order (three on D2Q16, four on D2Q25) of
// f and g of node n (Eq. genericMomentUptoO3), about u_ref, stored as grouped
// planes.
template <typename P, class L = D2Q16>
__device__ __forceinline__ void node_moments(const StepArgs &a, DevState st, P *__restrict__ mom,
                                             long long n) {
    const double T = st.T[n];
    double s, is;
    frame_scale(T, s, is);
    P M[nmom_padded<P, L>()];
#pragma unroll
    for (int k = 0; k < nmom_padded<P, L>(); ++k) M[k] = P(0);
    StoredMoments<P, L> sums;  // as the step forms them (the same bits)
#pragma unroll
    for (int ia = 0; ia < L::Q1; ++ia) {
        P fc[L::Q1], gc[L::Q1];
#pragma unroll
        for (int b = 0; b < L::Q1; ++b) {
            const int i = L::Q1 * ia + b;
            fc[b] = pop_plane<P>(st.f, i, a.N)[n];
            gc[b] = pop_plane<P>(st.g, i, a.N)[n];
        }
        sums.add(ia, fc, gc);
    }
    sums.moments(s, T, st.ux[n] - a.uref_x, st.uy[n] - a.uref_y, M);
    store_moments<P, nmom<L>()>(mom, a.mstride, a.moff + n, M);
}

}  // namespace pond
