// lbm_batch_kernels.h -- many independent lattices of uneven sizes advanced
// together: one launch per time step (large FP32 and FP64 batches: per two
// steps) covers the update tiles of every active case (per-case parameters come
// from a device table), and every check interval a monitor evaluates per-case
// residual and force on the device and retires the converged cases (their state
// freezes).
//
// Residual of case c over its fluid nodes (u the Guo velocity):
//   r = ||u_t - u_{t-k}||_2 / (k ||u_t||_2),
// against the snapshot of the previous check, k steps earlier.
#pragma once

#include "lbm_kernels.h"

namespace lbm {

// A case's parameters, those of the step first and from a cache line's start: a
// workgroup reads its case's anew, and the lines it touches are part of its latency
// (in the order of their subjects: 2% more per step of 20 to 72 MiB of cases).
struct alignas(64) CaseDev {
    int wpr;                // waves per row (rowlen / 64)
    int nwaves;             // ny * wpr
    int solid_base;         // first solid record / vtab entry of the case
    int nsol;               // bodies + 1
    int64_t f_off[2];       // element offsets of the two population buffers
    int64_t own_off;        // byte offset of the owner map
    StepArgs sa;            // lattice shape and strides
    CollideParams<double> cp64;
    PairArgs pair;          // split of the two-step update
    CollideParams<float> cp32;
    ForceArgs fa;           // force arguments (hist unused)
    int64_t snap_off;       // element offset of the velocity snapshot [2][ny][nx]
    int links_base;         // first link of the case in the global link array
    int chunk_first, chunk_count;  // force chunks of the case
};

// Update tile: `waves` consecutive waves of one case, starting at wave0.
struct Tile {
    int c;
    int wave0;
};

template <typename T>
__device__ inline const CollideParams<typename Sto<T>::C>& case_cp(const CaseDev& cd);
template <>
__device__ inline const CollideParams<double>& case_cp<double>(const CaseDev& cd) { return cd.cp64; }
template <>
__device__ inline const CollideParams<double>& case_cp<float>(const CaseDev& cd) { return cd.cp64; }
template <>
__device__ inline const CollideParams<float>& case_cp<_Float16>(const CaseDev& cd) { return cd.cp32; }
template <>
__device__ inline const CollideParams<float>& case_cp<bf16_t>(const CaseDev& cd) { return cd.cp32; }

// One time step of every listed tile; a case marked converged is skipped
// (its state stays as it was at retirement).  WAVES waves per workgroup.
template <typename T, bool NT, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_batch_step(const CaseDev* __restrict__ cases,
                                                           const Tile* __restrict__ tiles,
                                                           const int* __restrict__ converged, T* __restrict__ fbase,
                                                           const uint8_t* __restrict__ obase,
                                                           const double* __restrict__ vtab_all, int parity,
                                                           int64_t* __restrict__ tdev) {
    const Tile tl = tiles[xcd_remap(blockIdx.x, gridDim.x)];
    if (blockIdx.x == 0 && threadIdx.x == 0 && tdev) tdev[parity ^ 1] = tdev[parity] + 1;
    if (converged[tl.c]) return;
    const CaseDev& cd = cases[tl.c];
    // (copies: read together, beside the populations' loads, and not again after
    // every store; read where they are used they cost three round trips in a row,
    // 26.4 us per step of 72 MiB of FP32 cases against 25.6, FP16 75 against 38.  The
    // 16-bit collision keeps its reference: a copy changes which of its products the
    // compiler fuses, and so the last bits of every result)
    using CP = CollideParams<typename Sto<T>::C>;
    std::conditional_t<Sto<T>::kSplit, const CP&, const CP> cp = case_cp<T>(cd);
    const StepArgs sa = cd.sa;
    const int w = tl.wave0 + (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w >= cd.nwaves) return;
    const int y = w / cd.wpr;
    const int x = (w - y * cd.wpr) * 64 + (int)(threadIdx.x & 63);
    if constexpr (!Sto<T>::kSplit) {
        if (x >= sa.nx) return;
    }
    step_node<T, NT>(x, y, fbase + cd.f_off[parity], fbase + cd.f_off[parity ^ 1], obase + cd.own_off,
                     vtab_all + 2 * cd.solid_base, nullptr, nullptr, 0, sa, cp, nullptr, x < sa.nx);
}

// Node flags of every case, in one launch (a launch per case added 8 us each to a
// batch's creation).
__global__ __launch_bounds__(kBlock) void k_batch_node_flags(const CaseDev* __restrict__ cases, int n_cases,
                                                             const uint8_t* __restrict__ obase,
                                                             uint8_t* __restrict__ flags) {
    for (int c = (int)blockIdx.y; c < n_cases; c += (int)gridDim.y) {
        const CaseDev& cd = cases[c];
        const int64_t words = (int64_t)cd.sa.ny * cd.sa.rowlen / 8;
        for (int64_t w = (int64_t)blockIdx.x * kBlock + threadIdx.x; w < words; w += (int64_t)gridDim.x * kBlock)
            node_flags_word(obase + cd.own_off, flags + cd.own_off, cd.sa, w);
    }
}

// Two time steps of every listed workgroup of the two-step update (strip and run
// of a case; c < 0: none); a case marked converged is skipped.  slot: the buffer
// read, toggled by every launch, as is the slot of the step counter.
struct PairTile {
    int c, strip, run, pad;
};

template <typename T>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 4, 8))) void k_batch_pair(
    const CaseDev* __restrict__ cases, const PairTile* __restrict__ tiles, const int* __restrict__ converged,
    T* __restrict__ fbase, const uint8_t* __restrict__ obase, const uint8_t* __restrict__ flags,
    const double* __restrict__ vtab_all, int slot, int64_t* __restrict__ tdev) {
    __shared__ PairShared<T> sh;
    const PairTile tl = tiles[blockIdx.x];
    if (blockIdx.x == 0 && threadIdx.x == 0) tdev[slot ^ 1] = tdev[slot] + 2;
    if (tl.c < 0 || converged[tl.c]) return;
    const CaseDev& cd = cases[tl.c];
    // (copies: scalars held through the loop over rows)
    const StepArgs sa = cd.sa;
    const CollideParams<double> cp = cd.cp64;
    const PairArgs pa = cd.pair;
    const int x0 = tl.strip * pa.width, nout = x0 + pa.width <= sa.nx ? pa.width : sa.nx - x0;
    const int Ya = (int)((int64_t)sa.ny * tl.run / pa.runs), Yb = (int)((int64_t)sa.ny * (tl.run + 1) / pa.runs);
    pair_strip<T>(sh, fbase + cd.f_off[slot], fbase + cd.f_off[slot ^ 1], obase + cd.own_off, flags + cd.own_off,
                  vtab_all + 2 * cd.solid_base, x0, nout, Ya, Yb, sa, cp);
}

// Force chunks of every active case at the current state (parity).
struct BatchChunk {
    int c, s, start;
};

template <typename T>
__global__ __launch_bounds__(kBlock) void k_batch_force(const CaseDev* __restrict__ cases,
                                                        const BatchChunk* __restrict__ chunks,
                                                        const int* __restrict__ converged,
                                                        const T* __restrict__ fbase,
                                                        const uint32_t* __restrict__ links,
                                                        const int* __restrict__ seg_cnt,
                                                        const int* __restrict__ seg_off,
                                                        const SolidDev* __restrict__ sol_all,
                                                        const double* __restrict__ vtab_all,
                                                        double* __restrict__ partial, int parity,
                                                        int64_t t) {
    __shared__ ForceShared fs;
    const BatchChunk ch = chunks[blockIdx.x];
    if (converged[ch.c]) return;
    const CaseDev& cd = cases[ch.c];
    // force_role addresses the case's solids from its own base; chunk tables
    // are per case here, so pass one-element views
    const int cs = ch.s, cstart = ch.start;
    // (half-way bounce-back: the owner map is not consulted)
    force_role<T, false>(0, fs, fbase + cd.f_off[parity], nullptr, links + cd.links_base, seg_cnt + cd.solid_base,
                  seg_off + cd.solid_base, &cs, &cstart, sol_all + cd.solid_base,
                  vtab_all + 2 * cd.solid_base, nullptr, partial + (size_t)blockIdx.x * 6, t, cd.fa);
}

// Per-tile sums of |u - u_snap|^2 and |u|^2 over fluid nodes; the snapshot is
// replaced by u.
template <typename T, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void k_batch_monitor(const CaseDev* __restrict__ cases,
                                                              const Tile* __restrict__ tiles,
                                                              const int* __restrict__ converged,
                                                              const T* __restrict__ fbase,
                                                              const uint8_t* __restrict__ obase,
                                                              double* __restrict__ snap_base,
                                                              double* __restrict__ mon_partial,
                                                              int parity) {
    __shared__ double red[WAVES][2];
    const Tile tl = tiles[blockIdx.x];
    double dd = 0.0, uu = 0.0;
    if (!converged[tl.c]) {
        const CaseDev& cd = cases[tl.c];
        const int w = tl.wave0 + (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if (w < cd.nwaves) {
            const int y = w / cd.wpr;
            const int x = (w - y * cd.wpr) * 64 + (int)(threadIdx.x & 63);
            if (x < cd.sa.nx && obase[cd.own_off + (int64_t)y * cd.sa.opitch + x] == 0) {
                const T* f = fbase + cd.f_off[parity];
                double d[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) d[i] = (double)pop_at(f, cd.sa, i, x, y);
                const double drho = ((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7])) + d[8];
                const double r = cd.sa.rho0 + drho;
                const double jx = (d[1] - d[3]) + (d[5] - d[6]) + (d[8] - d[7]);
                const double jy = (d[2] - d[4]) + (d[5] + d[6]) - (d[7] + d[8]);
                // Guo velocity of the pre-collision state: rho u = sum e f~ - rho g / 2
                const double ux = jx / r - 0.5 * cd.cp64.gx;
                const double uy = jy / r - 0.5 * cd.cp64.gy;
                double* sn = snap_base + cd.snap_off + (int64_t)y * cd.sa.nx + x;
                const int64_t plane = (int64_t)cd.sa.nx * cd.sa.ny;
                const double px = sn[0], py = sn[plane];
                dd = (ux - px) * (ux - px) + (uy - py) * (uy - py);
                uu = ux * ux + uy * uy;
                sn[0] = ux;
                sn[plane] = uy;
            }
        }
    }
    dd = wave_sum(dd);
    uu = wave_sum(uu);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        red[wv][0] = dd;
        red[wv][1] = uu;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        double v = 0.0;
        for (int k = 0; k < WAVES; ++k) v += red[k][threadIdx.x];
        mon_partial[(size_t)blockIdx.x * 2 + threadIdx.x] = v;
    }
}

// One workgroup per case: residual from the tile partials (thread j takes tiles
// j, j + 256, ... in order, then a fixed tree), force totals per solid from the
// chunk partials (in chunk order, one component per thread); retire the case
// when a previous snapshot exists and r < tol.  (Bound by latency: one thread per
// case walking its up to 2048 tile partials in turn took 747 us per check of 64
// cases of up to 1024 x 512, four steps' worth.)
struct CaseResult {
    int converged;
    int have_snap;
    int64_t steps;
    double residual;
};

__global__ __launch_bounds__(kBlock) void k_batch_finalize(
    const CaseDev* __restrict__ cases, const int* __restrict__ tile_first, const int* __restrict__ tile_count,
    const double* __restrict__ mon_partial, const BatchChunk* __restrict__ chunks,
    const double* __restrict__ force_partial, CaseResult* __restrict__ res, int* __restrict__ converged,
    double* __restrict__ forces, int max_nsol, const int64_t* __restrict__ tdev, int parity, int k_steps, double tol) {
    __shared__ double red[kBlock / 64][2];
    const int c = (int)blockIdx.x;
    if (converged[c]) return;
    const CaseDev& cd = cases[c];
    double dd = 0.0, uu = 0.0;
    const int b1 = tile_first[c] + tile_count[c];
    for (int b = tile_first[c] + (int)threadIdx.x; b < b1; b += kBlock) {
        dd += mon_partial[2 * (size_t)b];
        uu += mon_partial[2 * (size_t)b + 1];
    }
    dd = wave_sum(dd);
    uu = wave_sum(uu);
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6][0] = dd;
        red[threadIdx.x >> 6][1] = uu;
    }
    // chunks of a case are listed solid by solid: chunk order is summation order
    double* fc = forces + (size_t)c * max_nsol * 6;
    const int c1 = cd.chunk_first + cd.chunk_count;
    for (int r = (int)threadIdx.x; r < cd.nsol * 6; r += kBlock) {
        const int s = r / 6, q = r - 6 * s;
        double v = 0.0;
        for (int cc = cd.chunk_first; cc < c1; ++cc)
            if (chunks[cc].s == s) v += force_partial[(size_t)cc * 6 + q];
        fc[r] = v;
    }
    __syncthreads();  // (every thread has read the case's flag)
    if (threadIdx.x != 0) return;
    dd = (red[0][0] + red[1][0]) + (red[2][0] + red[3][0]);
    uu = (red[0][1] + red[1][1]) + (red[2][1] + red[3][1]);
    // a state that is not finite (a diverged start) reports NaN and never retires
    const double r = !(isfinite(dd) && isfinite(uu))
                         ? __builtin_nan("")
                         : (uu > 0.0 ? sqrt(dd) / ((double)k_steps * sqrt(uu)) : (dd > 0.0 ? 1.0 : 0.0));
    CaseResult rr = res[c];
    rr.residual = rr.have_snap ? r : -1.0;
    rr.steps = tdev[parity];
    if (rr.have_snap && r < tol) {
        rr.converged = 1;
        converged[c] = 1;
    }
    rr.have_snap = 1;
    res[c] = rr;
}

}  // namespace lbm
