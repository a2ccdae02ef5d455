// pond_internal.h -- host-side interface between the C ABI (pond_api.hip) and
// the kernel launchers (pond_kernels.hip).  Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace pond {

// Device state of one instance.  Population planes: pop[i * N + n] for
// velocity i and node n = y * nx + x.  Frame planes: double ux, uy, T.  The
// internal-energy split also keeps the frame velocities of the previous time
// level (uxp, uyp: its source extrapolates the velocity gradient along
// trajectories from the last two levels); NULL for the other splits.
struct DevState {
    void *f, *g;          // Q planes each (float or double), Q = 16 or 25
    double *ux, *uy, *T;  // frame
    double *uxp, *uyp;    // frame velocities of the previous time level (internal split)
};

// Counters accumulated on the device (64-bit integer atomics only, so the sums
// do not depend on scheduling).  The step kernels count into slots, block b into
// slot b % kCounterSlots, and the host adds them up (fold): atomics on one
// address from every XCD are served one after the other, about 13 ns each, so
// one counter for the 65536 waves of a 2048^2 step alone takes 0.88 ms (the
// step without it 0.86; with two counters 1.77).  A slot is a cache line and is
// shared by blocks of one XCD only.
constexpr int kCounterSlots = 64;
struct DevCounters {
    unsigned long long pc_iterations;
    unsigned long long nonconverged;
    unsigned long long nonphysical;
    unsigned long long init_rejected;
    // node-steps (or, at initialisation, nodes) whose departure stencil reached
    // beyond the ghost rows of a wall
    unsigned long long ghost_overrun;
    double partial[5];  // scratch for deterministic reductions
    struct alignas(64) Slot {
        unsigned long long pc_iterations, nonconverged, nonphysical, ghost_overrun;
    } slot[kCounterSlots];

    // host: the slots' counts into the totals
    void fold() {
        for (Slot &x : slot) {
            pc_iterations += x.pc_iterations;
            nonconverged += x.nonconverged;
            nonphysical += x.nonphysical;
            ghost_overrun += x.ghost_overrun;
            x = Slot{};
        }
    }
};

struct StepArgs {
    int nx, ny, bc_x, bc_y;
    long long N;
    int interp_points;   // 3 or 4
    int pc_max_iter;
    double pc_tol;
    double omega;        // 1 / tau
    double omega1;       // 1 / tau_1 (Fourier part of the energy flux)
    int unit_prandtl;    // 1: plain BGK for g
    int split;           // 0: total energy in g; 1: internal energy in g (plus its source);
                         // 2: non-translational energy in g
    int lattice;         // 16 (D2Q16) or 25 (D2Q25)
    long long mstride;   // nodes per moment plane: N, or (ny + 2 wall_h) nx with walls
    long long moff;      // node offset of grid row 0 in a moment plane (wall_h nx)
    int wall_h;          // ghost rows beyond each wall (bc_y == 2), else 0
    double wall_ux[2], wall_T[2];
    double cv;           // 1 / (gamma - 1)
    double rcv;          // 1 / cv
    double uref_x, uref_y;
};

// Tiled step launch configuration: block shape, LDS capacity (nodes of the
// staged source region).
enum class TileShape : int { T16x16 = 0, T32x8 = 1, T16x8 = 2, T8x8 = 3, T256x1 = 4, T64x1 = 5,
                             T32x16 = 6 };

struct TileConfig {
    TileShape shape;
    int cap;  // nodes of LDS per block
};

inline void tile_dims(TileShape s, int &tx, int &ty) {
    switch (s) {
    case TileShape::T16x16: tx = 16; ty = 16; return;
    case TileShape::T32x8: tx = 32; ty = 8; return;
    case TileShape::T16x8: tx = 16; ty = 8; return;
    case TileShape::T8x8: tx = 8; ty = 8; return;
    case TileShape::T256x1: tx = 256; ty = 1; return;
    case TileShape::T64x1: tx = 64; ty = 1; return;
    case TileShape::T32x16: tx = 32; ty = 16; return;
    }
    tx = ty = 0;
}

// Whether the 64-node tiles (8 x 8, 64 x 1) of a D2Q16 grid of N nodes run four
// lanes per node.  One lane per node leaves such a grid a few waves on part of the
// CUs, each working through its node's x-components in turn; four lanes take a
// step to half the time or less until the blocks of 256 lanes need more than one
// or two rounds of the chip (two per CU in FP32, one in FP64).  Milliseconds per
// step with them / with the best other tile, Mach 2 and quadrants: FP32 64^2
// 0.019 / 0.042 and 0.021 / 0.043, 160^2 0.025 / 0.043 and 0.025 / 0.047, 192^2
// 0.038 / 0.045 and 0.033 / 0.048, 256^2 0.046 / 0.048 and 0.045 / 0.050; FP64
// 64^2 0.035 / 0.094 and 0.034 / 0.086, 160^2 0.067 / 0.094 and 0.060 / 0.088,
// 192^2 0.086 / 0.101 and 0.072 / 0.089, 256^2 0.113 / 0.084 and 0.102 / 0.089.
inline bool quad_lanes(long long N, bool dbl) { return N <= (dbl ? 36864 : 49152); }
// Blocks per CU of the four-lane kernels by registers (the LDS share of a block); the
// FP64 quadratic one would fit twice, but keeps the whole LDS as the cubic one does.
inline int quad_blocks_per_cu(bool dbl) { return dbl ? 1 : 2; }

// Blocks of a kernel per CU by registers and static LDS.  A property of the built
// kernel, asked of the runtime once per kernel (a query takes some 10 us, and
// contexts and batches are made per request).
hipError_t blocks_per_cu(const void *kernel, int threads, int *out);
// Blocks of the tiled step kernel (lattice, precision, stencil, energy split,
// shape) that fit one CU by registers and waves alone (no dynamic LDS).
int tiled_blocks_per_cu(int lattice, bool dbl, int np, int split, TileShape shape);

// Calls f(np, split) with both as std::integral_constant (np: 3 or 4 stencil
// points per axis, split: 0 total, 1 internal, 2 non-translational energy), so
// kernels can be picked by compile-time variant: the D2Q16 variants, of the
// single-instance and the batched paths alike.
template <class F>
inline auto with_variant(int np, int split, F &&f) {
    using std::integral_constant;
    if (np == 3) {
        if (split == 2) return f(integral_constant<int, 3>{}, integral_constant<int, 2>{});
        return split == 1 ? f(integral_constant<int, 3>{}, integral_constant<int, 1>{})
                          : f(integral_constant<int, 3>{}, integral_constant<int, 0>{});
    }
    if (split == 2) return f(integral_constant<int, 4>{}, integral_constant<int, 2>{});
    return split == 1 ? f(integral_constant<int, 4>{}, integral_constant<int, 1>{})
                      : f(integral_constant<int, 4>{}, integral_constant<int, 0>{});
}

// The single-instance variants of a lattice: D2Q16 takes both stencils and the
// three energy splits (0 total, 1 internal, 2 non-translational); D2Q25 the
// cubic stencil with the three splits (the API rejects other combinations
// before a launch).
template <class L, class F>
inline auto with_lattice_variant(int np, int split, F &&f) {
    using std::integral_constant;
    if constexpr (L::Q == 16) {
        return with_variant(np, split, static_cast<F &&>(f));
    } else {
        if (split == 2) return f(integral_constant<int, 4>{}, integral_constant<int, 2>{});
        return split == 1 ? f(integral_constant<int, 4>{}, integral_constant<int, 1>{})
                          : f(integral_constant<int, 4>{}, integral_constant<int, 0>{});
    }
}

template <typename P>
hipError_t launch_init(const StepArgs &a, const double *rho, const double *ux, const double *uy,
                       const double *T, DevState st, DevCounters *cnt, hipStream_t s);
template <typename P>
hipError_t launch_moments_prepass(const StepArgs &a, DevState st, P *mom, hipStream_t s);
// Ghost rows of the moment planes beyond walls (bc_y == 2), from the moments
// the pre-pass wrote; launched after it.
template <typename P>
hipError_t launch_wall_ghosts(const StepArgs &a, DevState st, P *mom, hipStream_t s);
// A step reads the moments of src (mom) and writes those of dst (mom_out).
template <typename P>
hipError_t launch_step(const StepArgs &a, DevState src, const P *mom, DevState dst, P *mom_out,
                       DevCounters *cnt, hipStream_t s);
template <typename P>
hipError_t launch_step_tiled(const StepArgs &a, const TileConfig &tc, DevState src, const P *mom,
                             DevState dst, P *mom_out, DevCounters *cnt, hipStream_t s);
// Walls (bc_y == 2): adds to cnt->ghost_overrun the nodes of st's frame whose
// departure stencil reaches beyond the ghost rows.
template <typename P>
hipError_t launch_ghost_check(const StepArgs &a, DevState st, DevCounters *cnt, hipStream_t s);
template <typename P>
hipError_t launch_macro(const StepArgs &a, DevState st, double *rho, double *ux, double *uy,
                        double *T, double *p, hipStream_t s);
template <typename P>
hipError_t launch_export(const StepArgs &a, DevState st, double *f, double *g, double *frame,
                         hipStream_t s);
template <typename P>
hipError_t launch_import(const StepArgs &a, const double *f, const double *g, const double *frame,
                         DevState st, hipStream_t s);
// Of fields: the sums of rho, rho ux, rho uy (fixed summation order) into
// cnt->partial[0..2], the largest stencil reach max(|u_x|, |u_y|) + c_out sqrt(T)
// into cnt->partial[3] and the largest c_out sqrt(T) into cnt->partial[4].
hipError_t launch_field_sums(long long N, const double *rho, const double *ux, const double *uy,
                             const double *T, double *scratch, int scratch_len, DevCounters *cnt,
                             hipStream_t s);
// The same of a stored state (populations + frame); without `mean` the reach alone.
template <typename P>
hipError_t launch_state_sums(const StepArgs &a, DevState st, bool mean, double *scratch,
                             int scratch_len, DevCounters *cnt, hipStream_t s);

}  // namespace pond
