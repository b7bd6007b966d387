// transport_tiled.hip -- launch shapes and launchers of the tiled RK3 stage
// kernels (transport_tiled.h, built in transport_tiled_unit.hip) and of the
// fused 2D transport (transport_fused.hip).
#include <algorithm>

#include "lbw_internal.h"

namespace lbw {

namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Columns of a run covered by whole tx x ty tiles.
int64_t padded_columns(int dim, const RunDev &r, int tx, int ty) {
    const int64_t ny = dim == 3 ? r.ny : 1;
    return ceil_div(r.nx, tx) * tx * ceil_div(ny, ty) * ty;
}

int64_t padded_columns(int dim, const RunDev *runs, int n, int tx, int ty) {
    int64_t c = 0;
    for (int i = 0; i < n; ++i) c += padded_columns(dim, runs[i], tx, ty);
    return c;
}

int planes(int dim, const RunDev &r) { return dim == 3 ? r.nz : r.ny; }

// Tile for runs whose caller chose none.  2D: the widest row (512 columns, 256
// in double precision, whose 512-thread blocks measured 10-27% slower on grids of
// few planes) that pads the runs' columns by at most a tenth more than 64-column
// rows do: a wider row stages fewer halo cells, which a tenth of idle lanes
// outweighs.  us per step of transport, single precision, each at its best
// chunk: 3000x2000 64 columns 92.8, 512 (2% more columns) 81.6; 1345x2000 55.0,
// 512 (9%) 51.3; 700x2000 37.0, 256 (9%) 36.1; 515x3000 40.9, 128 (11%) 41.0;
// 300x6000 42.7, 128 (20%) 45.7; double: 3000x2000 64 columns 170.7, 256 158.3,
// 260x5000 58.1, 128 (20%) 60.7.  3D: 64x8
// (one block of eight waves stages fewer halo columns per cell than 32x8: 59.7
// against 65.2 us per step's transport on 128x96x160), unless its padding
// exceeds that of 32x8 by a tenth (200 columns: 42.1 against 40.2 us).
TileShape default_tile(int dim, int precision, const RunDev *runs, int n) {
    if (dim == 3) {
        const int64_t wide = padded_columns(3, runs, n, 64, 8), narrow = padded_columns(3, runs, n, 32, 8);
        return wide * 10 <= narrow * 11 ? TileShape{64, 8, 0} : TileShape{32, 8, 0};
    }
    TileShape s{64, 1, 0};
    const int64_t least = padded_columns(2, runs, n, 64, 1);
    for (int tx : {128, 256, 512}) {
        if (tx == 512 && precision != LBW_FP32_SHIFTED) break;
        if (padded_columns(2, runs, n, tx, 1) * 10 <= least * 11) s.tx = tx;
    }
    return s;
}

// Estimated us of a step's three stages of a 2D run in single precision:
// 512 threads to a block (of several narrower tiles, counted by threads),
// k = ceil(blocks / 256) of them on the busiest CU (up to four run beside each
// other), `chunk` planes each: the issue slots of two blocks are filled better by
// four shorter ones, and one block beyond a multiple of 256 costs a block's time.
// Fitted to 512-column rows on 1024x1024 .. 4096x2048.  On 33 grids of 1.2 to 17
// million cells it is 7% low to 3% high with those, up to 11% low with narrower
// rows (129x12000 42.6, measured 47.9), and the shape it chooses takes at most 5%
// longer than the best of 4 widths by 15 chunks.
float march2d_us(int64_t k, int chunk) {
    constexpr float plane[4] = {2.12f, 2.92f, 3.74f, 4.98f}, start[4] = {15.5f, 18.1f, 20.2f, 22.4f};
    return start[k - 1] + plane[k - 1] * (float)chunk;
}

// Vertical chunk for runs whose caller chose none: the shortest with which the
// blocks still start together.  A plane of a march takes 0.7-1.4 us however
// few blocks there are, so a chip that is not full wants more blocks, down to
// one plane each; once it is full, shorter chunks only repeat the prologue
// (seven planes of the vertical stencil).  us per step of transport, measured:
// 2D 64x128 in double precision 102 at 32 planes, 15 at one; 1024x1024 84 at
// 32, 28 at four; 1024x2048 85 at 32, 41 at eight, 42 at four; 3D 64x48x96 89
// at 24, 26 at three; 128x128x192 93 at 24, 73 at eight; 256x256x400 (an earlier
// form) 620 at 64, 528 at 24, 572 at eight.  A last chunk cut short counts as a
// block: 100x100x400 in double precision 242 at 21 planes (520 blocks), 183 at 22
// (494); 300x100x150 125 at 13, 100 at 14.  Full means 16 waves a CU in 2D and the
// blocks of stages 2 and 3 that fit beside each other in 3D (registers: three of
// 64x8 in single precision, two in double).  Where S rides with stage 1 that stage
// holds two and one (LDS: 66 and 87 KB a block), but the chunk serves all three:
// sized for stage 1 the transport of 15 grids with S took 2% longer in the mean.
int default_chunk(int dim, int precision, const TileShape &s, const RunDev *runs, int n, int classes) {
    auto blocks = [&](int chunk) {
        int64_t b = 0;
        for (int i = 0; i < n; ++i) b += transport_tiles(dim, runs[i], TileShape{s.tx, s.ty, chunk});
        return b * classes;
    };
    constexpr int64_t cus = 256;
    if (dim == 2 && precision == LBW_FP32_SHIFTED && n == 1) {
        // 16 waves a CU (below) against the estimate's choice, us per step:
        // 4096x2048 32 planes 110, 16 planes 100; 129x12000 51.4 and 47.9; 40x50000
        // 62.4 and 58.7; 200x9000 49.6 and 45.1; 1000x3000 54.6 and 52.4;
        // 1024x1280 .. 1024x2048 and 4096x4096 the same chunk
        int best = 32;
        float least = 0.f;
        for (int c = 32; c >= 1; --c) {
            const int64_t k = ceil_div(blocks(c) * s.tx, 512 * cus);
            if (k > 4) break;
            const float us = march2d_us(k, c);
            if (c == 32 || us < least) {
                best = c;
                least = us;
            }
        }
        return best;
    }
    int64_t full;
    int lo, hi;
    if (dim == 2) {
        full = cus * 16 * 64 / s.tx;
        lo = 1;
        hi = 32;
    } else {
        const bool eight_waves = s.tx * s.ty == 512;
        if (precision == LBW_FP32_SHIFTED) full = cus * (eight_waves ? 3 : 5);
        else full = cus * (eight_waves ? 2 : 4);
        lo = eight_waves ? 3 : 2;
        hi = eight_waves ? 24 : 16;
    }
    int c = lo;
    while (c < hi && blocks(c) > full) ++c;
    return c;
}

}  // namespace

// A field the caller set is used as given.  The shape never needs 2^32
// work-items for a run that could launch with 32x8 columns and 64 planes (256
// and 32 in 2D) in place of the fields left at 0: those are what creation and
// lbw_set_launch check.
TileShape resolve_tile_shape(int dim, int precision, const lbw_launch &l, const RunDev *runs, int n,
                             int classes) {
    TileShape s;
    if (l.tile_x || l.tile_rows) {
        s.tx = l.tile_x ? l.tile_x : (dim == 3 ? 32 : 256);
        s.ty = dim == 2 ? 1 : (l.tile_rows ? l.tile_rows : 256 / s.tx);
    } else {
        s = default_tile(dim, precision, runs, n);
    }
    s.chunk = l.tile_y > 0 ? l.tile_y : default_chunk(dim, precision, s, runs, n, classes);
    if (n == 1) {
        auto too_many = [&] { return transport_tiles(dim, runs[0], s) * s.tx * s.ty >= ((int64_t)1 << 32); };
        if (!l.tile_x && !l.tile_rows && l.tile_y > 0 && dim == 3 && too_many()) s.tx = 32;
        while (l.tile_y == 0 && s.chunk < planes(dim, runs[0]) && too_many()) s.chunk *= 2;
    }
    return s;
}

int64_t transport_tiles(int dim, const RunDev &r, const TileShape &s) {
    const int nv = planes(dim, r), chunk = std::min(s.chunk, nv);
    return padded_columns(dim, r, s.tx, s.ty) / (s.tx * s.ty) * ceil_div(nv, chunk);
}

namespace {

hipError_t tiled_any(int dim, int precision, bool vss, const RunDev &r, const ClassSet &cs,
                     const TileShape &sh, int stage, hipStream_t st, const BatchArgs *b) {
    if (precision == LBW_FP32_SHIFTED) {
        if (dim == 2) return vss ? tiled_unit<float, 2, true>(r, cs, sh, stage, st, b) : tiled_unit<float, 2, false>(r, cs, sh, stage, st, b);
        return vss ? tiled_unit<float, 3, true>(r, cs, sh, stage, st, b) : tiled_unit<float, 3, false>(r, cs, sh, stage, st, b);
    }
    if (dim == 2) return vss ? tiled_unit<double, 2, true>(r, cs, sh, stage, st, b) : tiled_unit<double, 2, false>(r, cs, sh, stage, st, b);
    return vss ? tiled_unit<double, 3, true>(r, cs, sh, stage, st, b) : tiled_unit<double, 3, false>(r, cs, sh, stage, st, b);
}

}  // namespace

hipError_t launch_transport_tiled(int dim, int precision, const RunDev &r, const ClassSet &cs,
                                  const lbw_launch &l, hipStream_t st) {
    const TileShape sh = resolve_tile_shape(dim, precision, l, &r, 1, cs.n);
    return tiled_any(dim, precision, r.vs_s != 0.0, r, cs, sh, 0, st, nullptr);
}

hipError_t launch_one_stage(int dim, int precision, const RunDev &r, const lbw_launch &l,
                            int stage, hipStream_t st) {
    if (r.vs_s != 0.0) return hipErrorInvalidValue;   // constant settling speed only
    const TileShape sh = resolve_tile_shape(dim, precision, l, &r, 1);
    // one block per tile and chunk, fewer than 2^32 work-items a launch
    if (transport_tiles(dim, r, sh) * sh.tx * sh.ty >= ((int64_t)1 << 32)) return hipErrorInvalidConfiguration;
    return tiled_any(dim, precision, false, r, ClassSet(), sh, stage, st, nullptr);
}

hipError_t launch_transport_batched(int dim, int precision, const BatchArgs &b, hipStream_t st) {
    const RunDev &r = b.host_runs[0];
    bool any_var = false, any_const = false;
    for (int i = 0; i < b.nbatch; ++i) (b.host_runs[i].vs_s != 0.0 ? any_var : any_const) = true;
    if (!any_var || !any_const) return tiled_any(dim, precision, any_var, r, ClassSet(), b.shape, 0, st, &b);
    // both settling forms: each stage runs once per form, each kernel over
    // its own entries, so every run takes the kernels it takes alone
    BatchArgs x = b;
    for (int k = 1; k <= 3; ++k) {
        x.stage = k;
        for (int form = 0; form < 2; ++form) {
            x.form = form;
            const hipError_t e = tiled_any(dim, precision, form == 1, r, ClassSet(), b.shape, 0, st, &x);
            if (e != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

// Grids up to 9 * 2^17 cells (in double precision 4 * 2^17, with the first-order
// flux, whose recomputed halo costs least, 6 * 2^17): beyond, three launches of
// the march fill the chip and the recomputed halo decides.  us per step of
// transport, fused against march, single precision: 515x1030 20.7, 25.9;
// 1024x1024 27.4, 28.1; 900x1300 33.2, 34.2; 1024x1152 29.5, 30.7; 1024x1280
// 32.4, 31.2; 1024x1536 35.9, 34.2; double: 256x512 13.5, 19.0; 500x800 29.5,
// 29.1; 512x1024 30.2, 30.7; 600x1000 36.0, 35.4; 600x1200 41.3, 36.1; 700x1100
// 41.6, 39.9 (third order 512x1024 27.1, 28.0; 600x1200 38.5, 34.6; first order
// 512x1024 17.4, 23.4; 768x1024 21.7, 24.2; 900x1000 27.7, 29.0).  Rows count in
// sixteens, the lowest of the tiles, since a flat grid's tiles are mostly outside
// it (single precision 100000x8 50.1, 28.6; 20000x8 16.4, 18.3; 60000x16 34.8,
// 29.4; double 50000x8 44.6, 30.7; 20000x33 51.9, 38.5); columns count as they
// are, the march's rows being 64 wide (3x300000 196, 223).  A launch shape set by
// the caller asks for the march.  One block row per 16 or more grid rows, 65535 at
// most.
bool rk3_fused2d_applies(int dim, int precision, const RunDev &r, const lbw_launch &l) {
    const int64_t most = (int64_t)(precision == LBW_FP32_SHIFTED ? 9 : (r.scheme == LBW_UPWIND1 ? 6 : 4)) << 17;
    return dim == 2 && l.variant == 0 && !l.tile_x && !l.tile_y && !l.tile_rows &&
           ceil_div(r.ny, 16) * 16 * r.nx * r.ncls <= most && r.ny <= 65535 * 16;
}

hipError_t launch_rk3_fused2d(int precision, const RunDev &r, const ClassSet &cs, void *cout, void *a1,
                              void *a2, hipStream_t st) {
    return precision == LBW_FP32_SHIFTED ? fused_unit<float>(r, cs, cout, a1, a2, st)
                                         : fused_unit<double>(r, cs, cout, a1, a2, st);
}

}  // namespace lbw
