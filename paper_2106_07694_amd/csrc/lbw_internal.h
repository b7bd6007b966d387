// lbw_internal.h -- definitions shared by the HIP translation units of
// liblbw.so (not part of the public ABI; see include/lbw.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/lbw.h"

namespace lbw {

// ---------------------------------------------------------------------------
// Lattices (velocity sets, weights, opposite directions) in the order fixed by
// the public header.  D3Q19 is the lattice of the paper's Fig. 3; D2Q9 is its
// two-dimensional counterpart.  Weights are the standard second-order ones
// (cs^2 = 1/3, eq. 21).
// ---------------------------------------------------------------------------
template <int Q> struct Lattice;

template <> struct Lattice<9> {
    static constexpr int D = 2;
    static constexpr int cx[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
    static constexpr int cy[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
    static constexpr int cz[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    static constexpr int opp[9] = {0, 3, 4, 1, 2, 7, 8, 5, 6};
    static constexpr double w[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9,
                                    1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};
};

template <> struct Lattice<19> {
    static constexpr int D = 3;
    static constexpr int cx[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
    static constexpr int cy[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
    static constexpr int cz[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
    static constexpr int opp[19] = {0, 2, 1, 4, 3, 6, 5, 8, 7, 10, 9, 12, 11, 14, 13, 16, 15, 18, 17};
    static constexpr double w[19] = {1.0 / 3,  1.0 / 18, 1.0 / 18, 1.0 / 18, 1.0 / 18,
                                     1.0 / 18, 1.0 / 18, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                                     1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36,
                                     1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};
};

// ---------------------------------------------------------------------------
// One run as the kernels see it (passed by value).
// ---------------------------------------------------------------------------
struct RunDev {
    void *f;
    void *c, *c1, *c2;   // C and the two RK stage buffers
    void *s, *s2;        // S and its work buffer (current S is `s`)
    void *u;             // dim*N node velocity
    void *rho;           // N node density, written only when non-NULL
    double *dep;         // per-column deposit
    int32_t nx, ny, nz;  // grid
    int32_t vper;        // vertical axis periodic
    int64_t N;           // nodes
    int64_t ncol;        // bottom columns
    int32_t has_s;
    int32_t scheme;
    int32_t ncls;        // particle size classes: c holds ncls fields of N,
    int32_t pad_;        // dep ncls * ncol counters, class after class
    double tau, omega, guo;          // 1/tau and 1 - 1/(2 tau)
    double body[3], utop[3];
    double vs, kappa_c, gp_c, kappa_s, gp_s, eps;
    double vs_s;         // settling speed Vs (1 - vs_s S) (eq. 13), 0: constant
    double phi_c;        // volume fraction per unit C in the (1 - phi) of eq. 10
};

// The size classes a transport launch advances together: classes first ..
// first + n - 1 of a run with `of` of them (of = 1: the run as it stands).
// Each has its own C, stage buffers and deposit counters (class after class in
// the run's arrays), settling speed and diffusivity; the S update rides with
// class 0.
struct ClassSet {
    int32_t first = 0, n = 1, of = 1;
    double vs[LBW_MAX_CLASSES], kappa[LBW_MAX_CLASSES];
};

// Make r the run as class i sees it; true if the class carries the S update.
template <typename T>
__device__ __forceinline__ bool select_class(RunDev &r, const ClassSet &cs, int i) {
    if (cs.of <= 1) return true;
    const int64_t off = i * r.N;
    r.c = (T *)r.c + off;
    r.c1 = (T *)r.c1 + off;
    r.c2 = (T *)r.c2 + off;
    r.dep += i * r.ncol;
    r.vs = cs.vs[i];
    r.kappa_c = cs.kappa[i];
    return i == 0;
}

// Tile shape of the tiled transport kernels: tx x ty columns marching `chunk`
// vertical planes.
struct TileShape {
    int tx, ty, chunk;
};

// Arguments of the batched (persistent, work-list) transport launch.  Its
// entries are runs, or size classes of runs (one entry per class, the S
// update carried by the first).
struct BatchArgs {
    const RunDev *runs;        // device copy of the entry table
    const int *tile_start;     // device prefix sum of tiles per entry (nbatch + 1)
    const RunDev *host_runs;   // host copy of the same table
    int nbatch;                // entries
    TileShape shape;
    int sflip;                 // 1: S and its work buffer are swapped
    int grid;                  // persistent grid size
    int stage = 0;             // 0: the three RK stages and the S update; 1-3: that stage only
    int form = -1;             // -1: every entry; 0 / 1: only the entries with a constant /
                               // S-dependent settling speed (each form in its own kernels)
};

// Blocks are dealt round-robin to the 8 XCDs, so n of them are an eighth to each,
// the first n % 8 XCDs one more.  First of the n work items that XCD `xcd` takes
// (the end of its range for xcd + 1), as many as it has blocks in a launch of n.
__host__ __device__ __forceinline__ int xcd_first(int xcd, int n) {
    const int extra = n & 7;
    return xcd * (n >> 3) + (xcd < extra ? xcd : extra);
}

// Work item of block b of a launch of nb blocks: a contiguous range for each XCD,
// whose neighbours then meet in its L2.  2D march, us per step, item b for block b
// where nb is no multiple of 8, and this: 3000x2000 by 64-wide tiles and 4 planes
// 133, 100; 700x2000 44.1, 37.0; 1153x1100 44.7, 35.5.
__host__ __device__ __forceinline__ int xcd_order(int b, int nb) { return xcd_first(b & 7, nb) + (b >> 3); }

// Entry of a work list that holds item w, at or after entry b: start[i] is the
// first item of entry i (n entries, start[n] the total, which exceeds w).
// Called by whole waves; each lane looks at one entry, so 64 of them cost one
// load.  Entry by entry it was a chain of dependent scalar loads before a block
// could start on its tile, five times over in a step.
__device__ __forceinline__ int entry_of(const int *__restrict__ start, int n, int b, int w) {
    const int lane = (int)(threadIdx.x & 63);
    for (;;) {
        const int at_or_before = __popcll(__ballot(start[min(b + lane + 1, n)] <= w));
        b += at_or_before;
        if (at_or_before < 64) return b;
    }
}

// Launchers (return the launch error, if any).  `odd` selects the second
// kernel of the in-place streaming pair.
hipError_t launch_collide_stream(int q, int precision, const RunDev &r, bool odd,
                                 int block, hipStream_t st);
hipError_t launch_equilibrium(int q, int precision, const RunDev &r, bool odd, const void *rho,
                              const void *u, hipStream_t st);
hipError_t launch_import_f(int q, int precision, const RunDev &r, bool odd, const void *src,
                           hipStream_t st);
hipError_t launch_export_f(int q, int precision, const RunDev &r, bool odd, void *dst,
                           hipStream_t st);
hipError_t launch_transport_plain(int dim, int precision, const RunDev &r, hipStream_t st);
hipError_t launch_transport_tiled(int dim, int precision, const RunDev &r, const ClassSet &cs,
                                  const lbw_launch &l, hipStream_t st);
hipError_t launch_s_update(int dim, int precision, const RunDev &r, hipStream_t st);
// One RK stage (1, 2 or 3) of the tiled transport over the whole grid (runs
// with a constant settling speed).
hipError_t launch_one_stage(int dim, int precision, const RunDev &r, const lbw_launch &l,
                            int stage, hipStream_t st);
// Whether a run takes the fused transport: 2D, no launch shape set, and a grid
// small enough.
bool rk3_fused2d_applies(int dim, int precision, const RunDev &r, const lbw_launch &l);
// The same per element type (one unit each).
template <typename T>
hipError_t fused_unit(const RunDev &r, const ClassSet &cs, void *cout, void *a1, void *a2, hipStream_t st);
// The whole transport of a 2D step in one launch: reads C (of every class) from
// r.c, writes the result to cout (another buffer) and, where given, the stages
// to a1 and a2.
hipError_t launch_rk3_fused2d(int precision, const RunDev &r, const ClassSet &cs, void *cout, void *a1,
                              void *a2, hipStream_t st);
// The launch's tile shape for n runs advanced together, or for `classes` size
// classes of one; fields the caller left at 0 are chosen for their sizes.
TileShape resolve_tile_shape(int dim, int precision, const lbw_launch &l, const RunDev *runs, int n,
                             int classes = 1);
// Tiles (blocks) of one run in that shape, over all vertical chunks.
int64_t transport_tiles(int dim, const RunDev &r, const TileShape &s);
hipError_t launch_transport_batched(int dim, int precision, const BatchArgs &b, hipStream_t st);
// The tiled stages in one unit per dimension, element type and settling form
// (VSS: a settling speed that depends on S), of the classes cs of the single run
// r or, when b is not NULL, of the batched entries.  stage 0: all three; 1-3:
// that one only (single runs).
template <typename T, int D, bool VSS>
hipError_t tiled_unit(const RunDev &r, const ClassSet &cs, const TileShape &sh, int stage, hipStream_t st,
                      const BatchArgs *b);
// nodes: total nodes of the batch (chooses the cache policy of the
// population accesses)
hipError_t launch_collide_stream_batched(int q, int precision, const RunDev *runs, const int *blk_start,
                                         int nbatch, int sflip, bool odd, int block, int grid,
                                         int64_t nodes, hipStream_t st);
size_t adjoint_work_bytes(int dim, int precision, int64_t N);
hipError_t launch_adjoint(int q, int precision, const RunDev &r, bool frozen, const void *f_n,
                          const void *c_n, const void *u_n, const void *rho_n, const void *a1_n,
                          const void *a2_n,
                          const void *fbar_next, const void *cbar_next,
                          double dep_bar, void *fbar, void *cbar, double *vs_bar, void *work,
                          const lbw_launch &l, hipStream_t st);
// Per-block partials of each run into part (kReduceBlocks per run) and, when
// out is not NULL, each run's sum into out[run]; both writable by the device.
// plane >= 0: MASS_C / MASS_S sum only the cells below that horizontal plane
// (the first plane * ncol nodes of each run); -1: all nodes.  cls >= 0:
// MASS_C and DEPOSIT of that particle size class only; -1: every class.
hipError_t launch_reduce(int q, int precision, const RunDev *runs, int nbatch, int what,
                         bool odd, double *part, double *out, hipStream_t st, int plane = -1,
                         int cls = -1);
// The sum of one run's kReduceBlocks partials, bit for bit as the reduction's
// last pass forms it.
double final_sum(const double *part);
// Power spectral density of a front height (device, ncol values) along
// lateral axis `axis` for slice `index` (-1: mean over slices); out[len/2+1].
hipError_t launch_front_psd(const RunDev &r, int dim, const double *h, int axis, int index,
                            double *out, hipStream_t st);
// Front of the particle field (total over the classes) per bottom column
// into out (device, ncol).
hipError_t launch_front_height(int precision, const RunDev &r, int dim, double thr, double *out,
                               hipStream_t st);

constexpr int kReduceBlocks = 256;  // partial sums per run

}  // namespace lbw
