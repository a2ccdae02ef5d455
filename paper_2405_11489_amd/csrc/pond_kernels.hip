// pond_kernels.hip -- HIP kernels of the PonD f+g step for gfx950 (MI355X):
// the D2Q16 instantiation of the lattice-dependent kernels
// (pond_lattice_kernels.h; D2Q25 in pond_kernels25.hip), the launchers that
// pick the lattice, and the lattice-independent reductions.
//
// One kernel source, instantiated for P = double (FP64 mode) and P = float
// (FP32 mode: populations, moments, interpolation and frame transformation in
// float; conserved sums, temperature recovery and the predictor-corrector test
// in double).
#include <map>
#include <mutex>

#include "pond_lattice_kernels.h"

namespace pond {

template struct Launch<float, D2Q16>;
template struct Launch<double, D2Q16>;
extern template struct Launch<float, D2Q25>;
extern template struct Launch<double, D2Q25>;

namespace {

using lk::kBlock;
using lk::grid_for;
using lk::partial_sums_kernel;

// ------------------------------------------- deterministic reductions ----
constexpr int kRedBlocks = 256;

// per-block maxima of the reach of a node's departure stencils in nodes, max(|u_x|,
// |u_y|) + c_out sqrt(T), and of its thermal part; non-finite values are skipped
__global__ __launch_bounds__(kBlock) void reach_partial_kernel(long long N, const double *ux,
                                                               const double *uy, const double *T,
                                                               double *scratch) {
    __shared__ double sh[2][kBlock];
    const long long chunk = (N + gridDim.x - 1) / gridDim.x;
    const long long lo = (long long)blockIdx.x * chunk;
    const long long hi = lo + chunk < N ? lo + chunk : N;
    double m = 0.0, mt = 0.0;
    for (long long n = lo + threadIdx.x; n < hi; n += blockDim.x) {
        const double rt = c1(3) * sqrt(fmax(T[n], 0.0)), r = fmax(fabs(ux[n]), fabs(uy[n])) + rt;
        if (isfinite(r)) {
            m = fmax(m, r);
            mt = fmax(mt, rt);
        }
    }
    const int t = threadIdx.x;
    sh[0][t] = m;
    sh[1][t] = mt;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (t < w)
            for (int c = 0; c < 2; ++c) sh[c][t] = fmax(sh[c][t], sh[c][t + w]);
        __syncthreads();
    }
    if (t < 2) scratch[t * gridDim.x + blockIdx.x] = sh[t][0];
}

// The blocks' partial results to cnt->partial: the sums of (rho, rho u) if `sums`
// is given, in block order, and the largest reaches.  One block stages the partial
// results in LDS, where the in-order sums cost an add each instead of a memory
// round trip (one thread over global memory: 28 us for the sums, 16 us for the
// reach; this: 4.7 us for both, most of it the launch).
__global__ __launch_bounds__(kRedBlocks) void reduce_final_kernel(const double *sums,
                                                                  const double *reach,
                                                                  DevCounters *cnt) {
    __shared__ double sh[5][kRedBlocks + 1];
    const int t = threadIdx.x;
    if (sums)
        for (int c = 0; c < 3; ++c) {
            const int i = c * kRedBlocks + t;
            sh[i % 3][i / 3] = sums[i];
        }
    sh[3][t] = reach[t];
    sh[4][t] = reach[kRedBlocks + t];
    __syncthreads();
    if (sums && t < 3) {
        double s = 0.0;
#pragma unroll 16
        for (int b = 0; b < kRedBlocks; ++b) s += sh[t][b];
        cnt->partial[t] = s;
    }
    if (t == 64 || t == 65) {
        const int c = t - 64 + 3;
        double m = 0.0;
#pragma unroll 16
        for (int b = 0; b < kRedBlocks; ++b) m = fmax(m, sh[c][b]);
        cnt->partial[c] = m;
    }
}

struct FieldLoader {
    const double *rho, *ux, *uy;
    __device__ void operator()(long long n, double &r, double &jx, double &jy) const {
        r = rho[n];
        jx = rho[n] * ux[n];
        jy = rho[n] * uy[n];
    }
};

}  // namespace

template <typename P>
hipError_t launch_init(const StepArgs &a, const double *rho, const double *ux, const double *uy,
                       const double *T, DevState st, DevCounters *cnt, hipStream_t s) {
    return a.lattice == 25 ? Launch<P, D2Q25>::init(a, rho, ux, uy, T, st, cnt, s)
                           : Launch<P, D2Q16>::init(a, rho, ux, uy, T, st, cnt, s);
}

template <typename P>
hipError_t launch_moments_prepass(const StepArgs &a, DevState st, P *mom, hipStream_t s) {
    return a.lattice == 25 ? Launch<P, D2Q25>::moments(a, st, mom, s)
                           : Launch<P, D2Q16>::moments(a, st, mom, s);
}

template <typename P>
hipError_t launch_wall_ghosts(const StepArgs &a, DevState st, P *mom, hipStream_t s) {
    return a.lattice == 25 ? Launch<P, D2Q25>::wall_ghosts(a, st, mom, s)
                           : Launch<P, D2Q16>::wall_ghosts(a, st, mom, s);
}

template <typename P>
hipError_t launch_step(const StepArgs &a, DevState src, const P *mom, DevState dst, P *mom_out,
                       DevCounters *cnt, hipStream_t s) {
    return a.lattice == 25 ? Launch<P, D2Q25>::step(a, src, mom, dst, mom_out, cnt, s)
                           : Launch<P, D2Q16>::step(a, src, mom, dst, mom_out, cnt, s);
}

template <typename P>
hipError_t launch_step_tiled(const StepArgs &a, const TileConfig &tc, DevState src, const P *mom,
                             DevState dst, P *mom_out, DevCounters *cnt, hipStream_t s) {
    return a.lattice == 25 ? Launch<P, D2Q25>::step_tiled(a, tc, src, mom, dst, mom_out, cnt, s)
                           : Launch<P, D2Q16>::step_tiled(a, tc, src, mom, dst, mom_out, cnt, s);
}

hipError_t blocks_per_cu(const void *kernel, int threads, int *out) {
    static std::mutex mu;
    static std::map<const void *, int> known;  // one entry per kernel of this library
    std::lock_guard<std::mutex> lk(mu);
    auto it = known.find(kernel);
    if (it != known.end()) {
        *out = it->second;
        return hipSuccess;
    }
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(out, kernel, threads, 0);
    if (e != hipSuccess) return e;
    try {
        known.emplace(kernel, *out);
    } catch (...) {  // no memory to note it
    }
    return hipSuccess;
}

int tiled_blocks_per_cu(int lattice, bool dbl, int np, int split, TileShape shape) {
    if (lattice == 25)
        return dbl ? Launch<double, D2Q25>::tiled_blocks_per_cu(np, split, shape)
                   : Launch<float, D2Q25>::tiled_blocks_per_cu(np, split, shape);
    return dbl ? Launch<double, D2Q16>::tiled_blocks_per_cu(np, split, shape)
               : Launch<float, D2Q16>::tiled_blocks_per_cu(np, split, shape);
}

template <typename P>
hipError_t launch_ghost_check(const StepArgs &a, DevState st, DevCounters *cnt, hipStream_t s) {
    return a.lattice == 25 ? Launch<P, D2Q25>::ghost_check(a, st, cnt, s)
                           : Launch<P, D2Q16>::ghost_check(a, st, cnt, s);
}

template <typename P>
hipError_t launch_macro(const StepArgs &a, DevState st, double *rho, double *ux, double *uy,
                        double *T, double *p, hipStream_t s) {
    return a.lattice == 25 ? Launch<P, D2Q25>::macro(a, st, rho, ux, uy, T, p, s)
                           : Launch<P, D2Q16>::macro(a, st, rho, ux, uy, T, p, s);
}

template <typename P>
hipError_t launch_export(const StepArgs &a, DevState st, double *f, double *g, double *frame,
                         hipStream_t s) {
    return a.lattice == 25 ? Launch<P, D2Q25>::exp(a, st, f, g, frame, s)
                           : Launch<P, D2Q16>::exp(a, st, f, g, frame, s);
}

template <typename P>
hipError_t launch_import(const StepArgs &a, const double *f, const double *g, const double *frame,
                         DevState st, hipStream_t s) {
    return a.lattice == 25 ? Launch<P, D2Q25>::imp(a, f, g, frame, st, s)
                           : Launch<P, D2Q16>::imp(a, f, g, frame, st, s);
}

hipError_t launch_field_sums(long long N, const double *rho, const double *ux, const double *uy,
                             const double *T, double *scratch, int scratch_len, DevCounters *cnt,
                             hipStream_t s) {
    if (scratch_len < 5 * kRedBlocks) return hipErrorInvalidValue;
    double *reach = scratch + 3 * kRedBlocks;
    hipLaunchKernelGGL(partial_sums_kernel<FieldLoader>, dim3(kRedBlocks), dim3(kBlock), 0, s, N,
                       FieldLoader{rho, ux, uy}, scratch);
    hipLaunchKernelGGL(reach_partial_kernel, dim3(kRedBlocks), dim3(kBlock), 0, s, N, ux, uy, T,
                       reach);
    hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(kRedBlocks), 0, s, scratch, reach, cnt);
    return hipGetLastError();
}

template <typename P>
hipError_t launch_state_sums(const StepArgs &a, DevState st, bool mean, double *scratch,
                             int scratch_len, DevCounters *cnt, hipStream_t s) {
    if (scratch_len < 5 * kRedBlocks) return hipErrorInvalidValue;
    double *reach = scratch + 3 * kRedBlocks;
    if (mean) {
        hipError_t e = a.lattice == 25
                           ? Launch<P, D2Q25>::state_partial_sums(a, st, scratch, kRedBlocks, s)
                           : Launch<P, D2Q16>::state_partial_sums(a, st, scratch, kRedBlocks, s);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(reach_partial_kernel, dim3(kRedBlocks), dim3(kBlock), 0, s, a.N, st.ux,
                       st.uy, st.T, reach);
    hipLaunchKernelGGL(reduce_final_kernel, dim3(1), dim3(kRedBlocks), 0, s,
                       mean ? scratch : nullptr, reach, cnt);
    return hipGetLastError();
}

#define POND_INSTANTIATE(P)                                                                        \
    template hipError_t launch_init<P>(const StepArgs &, const double *, const double *,           \
                                       const double *, const double *, DevState, DevCounters *,    \
                                       hipStream_t);                                               \
    template hipError_t launch_moments_prepass<P>(const StepArgs &, DevState, P *, hipStream_t);   \
    template hipError_t launch_wall_ghosts<P>(const StepArgs &, DevState, P *, hipStream_t);       \
    template hipError_t launch_step<P>(const StepArgs &, DevState, const P *, DevState, P *,       \
                                       DevCounters *, hipStream_t);                                \
    template hipError_t launch_step_tiled<P>(const StepArgs &, const TileConfig &, DevState,       \
                                             const P *, DevState, P *, DevCounters *,              \
                                             hipStream_t);                                         \
    template hipError_t launch_ghost_check<P>(const StepArgs &, DevState, DevCounters *,       \
                                              hipStream_t);                                        \
    template hipError_t launch_macro<P>(const StepArgs &, DevState, double *, double *, double *,  \
                                        double *, double *, hipStream_t);                          \
    template hipError_t launch_export<P>(const StepArgs &, DevState, double *, double *, double *, \
                                         hipStream_t);                                             \
    template hipError_t launch_import<P>(const StepArgs &, const double *, const double *,         \
                                         const double *, DevState, hipStream_t);                   \
    template hipError_t launch_state_sums<P>(const StepArgs &, DevState, bool, double *, int,      \
                                             DevCounters *, hipStream_t);

POND_INSTANTIATE(float)
POND_INSTANTIATE(double)

}  // namespace pond
