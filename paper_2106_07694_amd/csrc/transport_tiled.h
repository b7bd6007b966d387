// transport_tiled.h -- the tiled RK3 stage kernels of the particle
// transport, as templates shared by the units that build them (one per
// dimension, element type and settling form: transport_tiled_unit.hip).
//
// RK3 stage kernels of the particle transport, tiled for CDNA: a block owns a
// TX x TY tile of vertical columns and marches up a chunk of the vertical axis.
// Per plane:
//   * the plane of the stage input a, with a three-cell lateral halo, and the
//     lateral velocities sit in LDS; each lateral face flux is computed once
//     into LDS and differenced by the two cells that share it;
//   * each thread keeps its own column's six-node vertical stencil of a and
//     of the vertical transport velocity in registers, computes the face
//     above its cell and carries it down as the face below the next cell
//     (3D, single precision, WENO5: the stencil's node data instead, each
//     node's flux and indicators computed once, as the node enters);
//   * the plane after next is loaded while a plane is finished and the next
//     one is published after its faces (software pipelining, one barrier).
// What bounds it: instruction issue, vector and scalar alike.  A SIMD issues
// one of each every four cycles, and the march's scalar work (plane addresses,
// the vertical rule, masks) once outnumbered its vector work, 200 against 142
// instructions a plane in 2D; kept free of branches, masks and 64-bit products
// it is about 100 (3D 236 -> 130 against 206).  Measured, us per step: 3D
// 256x256x512 transport 640 -> 610, 97x63x130 45 -> 38, 2D + S 1024x2048 49.6
// -> 46.4, the 30-run sweep 250 -> 236 in all; double precision unchanged (its
// vector work is twice as long).
//
// Arithmetic and wall rules are those of the plain kernels (transport.hip):
// WENO face fluxes from the upwind side, central diffusion, mirror ghosts
// with a sign flip of the vertical fluid velocity, closed top, absorbing
// bottom feeding the deposit counter.  In single precision the weights use
// the hardware reciprocal.
#pragma once

#include "transport_face.h"

namespace lbw {
namespace {

struct TileGeom {
    int nx, ny, nv;     // lateral sizes (ny = 1 in 2D) and vertical extent
    int64_t sv;         // stride of the vertical axis
    int64_t N;
    int vper;
    int chunk;          // vertical planes per block
    int gx, gy, gz;     // tiles along x, y and vertical chunks launched
    int bz0;            // first vertical chunk launched
};

// Position of the block, in the order in which tiles meet in one XCD's L2, the
// size classes of one tile next to each other (they read the same velocity).
__device__ __forceinline__ void block_tile(const TileGeom &g, int ncls, int &bx, int &by, int &bz, int &cls) {
    int logical = xcd_order(blockIdx.x, g.gx * g.gy * g.gz * ncls);
    cls = 0;
    if (ncls > 1) {
        cls = logical % ncls;
        logical /= ncls;
    }
    bx = logical % g.gx;
    const int t = logical / g.gx;
    by = t % g.gy;
    bz = g.bz0 + t / g.gy;
}

// Addressing: a vertical plane's base pointer is the same for the whole
// block (uniform, held in scalar registers) and each lane adds a 32-bit byte
// offset within the plane, so the loads and stores need no 64-bit vector
// arithmetic.  This needs nx * ny * sizeof(T) < 2^32 (checked at creation).
template <typename T>
__device__ __forceinline__ const T &at(const void *plane, uint32_t off) {
    return *(const T *)((const char *)plane + off);
}

// FULL: the grid is a whole number of tiles, so every lane owns a cell and
// the store needs no lane mask (a masked store on a path that may be skipped
// would make every later wait on the load counter drain it completely).
// VSS: the settling speed is set by the local fluid density (eq. 13 with rho
// linear in S), Vs (1 - vs_s S) with S at the node (the mirrored node beyond
// a wall); the conservative face fluxes then carry the -phi d(Vs)/dz term of
// eq. 7.  S is read at time level n, which the S update of this step does not
// overwrite (it writes the other S buffer).
// FS (stage 1 only): the S update (S5-S6 in conservative form, the
// arithmetic and sum order of k_s_update) rides with the march.  It needs the
// velocity this stage already stages (lateral components in LDS, the
// vertical one read per plane) plus S on the plane with a one-cell lateral
// halo and at the next plane of the column; s_entry is false for a batch
// entry that carries no S (a size class after the first), which then loads
// C in its place and stores nothing.
template <typename T, int D, int SCHEME, int STAGE, int TX, int TY, bool FULL, bool VSS,
          bool FS = false>
__device__ __forceinline__ void stage_tile(const RunDev &r, const TileGeom &g, int bx, int by, int bz,
                                           bool s_entry = true) {
    static_assert(!FS || STAGE == 1, "the S update rides with stage 1");
    constexpr int NT = TX * TY;
    constexpr int AX = TX + 6;                  // a plane row length (x halo 3 + 3)
    constexpr int AY = (D == 3) ? TY + 6 : 1;   // a plane rows
    // NV (3D, single precision, WENO5): the vertical faces share each node's
    // work (its flux w a and the three indicators it centres, weno5_node),
    // done once as the node enters the column's window; the fluxes and
    // differences stay in registers, the indicators in a per-thread LDS ring
    // (in registers they would cost a block of occupancy).  The lateral faces
    // keep the whole stencil (face6_lds): shared node data there needs an extra
    // LDS round trip and barrier per plane, which cost more than the arithmetic
    // saves.
    constexpr bool NV = (SCHEME == LBW_WENO5 && D == 3 && sizeof(T) == 4);
    constexpr int SXL = TX + 2;                         // S row with a one-cell x halo
    constexpr int SYL = (D == 3) ? TY + 2 : 1;          // S rows (one-cell y halo in 3D)
    // The LDS arrays are pieces of one allocation at fixed offsets, so that
    // accesses which share a lane-dependent index can share one address
    // register and differ only in the instruction's constant offset.
    constexpr int O_A = 0, O_UX = AY * AX, O_UY = O_UX + TY * AX,
                  O_FX = O_UY + ((D == 3) ? (TY + 6) * AX : 1), O_FY = O_FX + TY * (TX + 1),
                  O_S = O_FY + ((D == 3) ? (TY + 1) * TX : 1), O_GX = O_S + (FS ? SXL * SYL : 1),
                  O_GY = O_GX + (FS ? TY * (TX + 1) : 1),
                  O_END = O_GY + ((FS && D == 3) ? (TY + 1) * TX : 1);
    // Two sets of them, taken in turn, so that a plane costs one barrier: the
    // next plane is published into the other set after a plane's faces, and the
    // barrier between the faces and their use is also the one between that
    // publication and the next plane's faces.  Transport, us per step: 2D
    // 1024x2048 with S 46.4 -> 43.9, 2048x2048 68.3 -> 63.6, 1024x1024 in double
    // precision 44.9 -> 42.2, the 30-run sweep 136 -> 121; 3D 256x256x512 615 ->
    // 598, four classes of 128x128x192 216 -> 212, the smaller grids even.  With S
    // in 3D they leave stage 1 a block less a CU (64x8: two in single precision, one
    // in double) and are still no loss: single precision even, double 128x96x160
    // 103 -> 98, 256^3 803 -> 746, 97x63x130 71.5 -> 69.8.
    constexpr int SET = O_END + 64;
    __shared__ T smem[2 * SET];

    const int tid = threadIdx.x;
    const int tx = tid % TX, ty = tid / TX;
    const int x0 = bx * TX, y0 = by * TY;
    const int gxl = x0 + tx, gyl = y0 + ty;         // own column (may be outside)
    const bool active = FULL || (gxl < g.nx && (D == 2 || gyl < g.ny));
    const int xw = FULL ? gxl : min(gxl, g.nx - 1); // column for loads
    const int yw = (D == 3) ? (FULL ? gyl : min(gyl, g.ny - 1)) : 0;
    const int col = xw + g.nx * yw;                 // < nx * ny
    uint32_t colb = (uint32_t)col * (uint32_t)sizeof(T);
    const int v0 = bz * g.chunk;
    const int v1 = min(v0 + g.chunk, g.nv);

    const T *__restrict__ ain = (const T *)(STAGE == 1 ? r.c : (STAGE == 2 ? r.c1 : r.c2));
    const T *__restrict__ ux = (const T *)r.u;
    const T *__restrict__ uy = ux + g.N;
    const T *__restrict__ uv = ux + (int64_t)(D - 1) * g.N;
    const T vs = (T)r.vs, kap = (T)r.kappa_c, eps = (T)r.eps;
    const bool walls = !g.vper;
    // (a 32 x 32-bit product: planes and plane bytes both fit)
    const uint32_t plane_bytes = (uint32_t)(g.sv * (int64_t)sizeof(T));
    auto plane = [&](const void *base, int v) -> const void * {
        return (const char *)base + (uint64_t)(uint32_t)v * plane_bytes;
    };
    // settling speed at plane vv of this column
    auto vs_at = [&](int vv) -> T {
        if constexpr (VSS) return vs * ((T)1 - (T)r.vs_s * at<T>(plane(r.s, vv), colb));
        else return vs;
    };
    auto wplane = [&](void *base, int v) -> void * {
        return (char *)base + (uint64_t)(uint32_t)v * plane_bytes;
    };

    // vertical index with the wall/periodic rule, and the sign the vertical
    // fluid velocity takes there (-1 at a mirrored node).  The march reaches
    // at most three planes below and four above the axis (v in [-3, nv + 3])
    // and nv >= 6, so one reflection or wrap suffices.  Selects on scalars, not
    // branches: a wave issues one scalar instruction where it issues one
    // vector instruction, and the march has few vector ones to hide them
    auto vidx_up = [&](int v, T &sgn) -> int {      // v >= 0
        const bool over = v >= g.nv;
        sgn = over && walls ? (T)-1 : (T)1;
        const int past = walls ? 2 * g.nv - 1 - v : v - g.nv;
        return over ? past : v;
    };
    auto vidx = [&](int v, T &sgn) -> int {
        const bool under = v < 0;
        const int up = vidx_up(v, sgn);
        sgn = under && walls ? (T)-1 : sgn;
        const int past = walls ? -1 - v : v + g.nv;
        return under ? past : up;
    };
    auto load_at = [&](int vv, T sgn, T &a, T &w) {
        a = at<T>(plane(ain, vv), colb);
        const T u = at<T>(plane(uv, vv), colb);
        w = sgn * u - vs_at(vv);
    };
    auto load_av = [&](int v, T &a, T &w) {
        T sgn;
        const int vv = vidx(v, sgn);
        load_at(vv, sgn, a, w);
    };

    // lateral halo slots of this thread (fixed over the march), as byte
    // offsets within a plane and LDS indices; a spare slot (its array filled)
    // reads column 0 and writes to a place of its lane's past the arrays, so
    // publication needs no lane masks
    // a-plane cross: rows ty in [0,TY) x cols [0,AX), plus (3D) y-halo rows
    constexpr int NA = (D == 3) ? AX * TY + TX * 6 : AX;
    constexpr int NUX = AX * TY;
    constexpr int NUY = (D == 3) ? TX * (TY + 6) : 0;
    constexpr int SA = (NA + NT - 1) / NT, SUX = (NUX + NT - 1) / NT, SUY = (NUY + NT - 1) / NT;
    uint32_t offA[SA];
    int ldsA[SA];
    uint32_t offX[SUX];
    int ldsX[SUX];
    uint32_t offY[(SUY > 0) ? SUY : 1];
    int ldsY[(SUY > 0) ? SUY : 1];
    // lateral wrap of a position from three cells below the axis on.  Positions
    // past its third cell beyond are read by no cell of the grid and are
    // clamped there, so one wrap does unless the axis has fewer than three
    // cells (the general remainder, twelve of which cost as much as two planes
    // of the march)
    auto wrap = [](int j, int n) {
        j = min(j, n + 2);
        if (n < 3) j %= n;
        j += j < 0 ? n : 0;
        return j - (j >= n ? n : 0);
    };
    auto wrapx = [&](int x) { return wrap(x, g.nx); };
    auto wrapy = [&](int y) { return wrap(y, g.ny); };
    auto lat = [&](int x, int y) { return (uint32_t)(x + g.nx * y) * (uint32_t)sizeof(T); };
#pragma unroll
    for (int s = 0; s < SA; ++s) {
        const int i = tid + s * NT;
        ldsA[s] = O_END + (tid & 63);
        offA[s] = 0;
        if (i < NA) {
            int lx, ly;  // plane-local coords, halo origin at (-3, -3)
            if (i < AX * TY) { lx = i % AX; ly = (D == 3) ? (i / AX) + 3 : 0; }
            else { const int j = i - AX * TY; lx = (j % TX) + 3; ly = (j / TX) < 3 ? (j / TX) : (j / TX) + TY; }
            offA[s] = lat(wrapx(x0 + lx - 3), (D == 3) ? wrapy(y0 + ly - 3) : 0);
            ldsA[s] = O_A + ly * AX + lx;
        }
    }
#pragma unroll
    for (int s = 0; s < SUX; ++s) {
        const int i = tid + s * NT;
        ldsX[s] = O_END + (tid & 63);
        offX[s] = 0;
        if (i < NUX) {
            const int lx = i % AX, ly = i / AX;
            offX[s] = lat(wrapx(x0 + lx - 3), (D == 3) ? wrapy(y0 + ly) : 0);
            ldsX[s] = O_UX + ly * AX + lx;
        }
    }
#pragma unroll
    for (int s = 0; s < SUY; ++s) {
        const int i = tid + s * NT;
        ldsY[s] = O_END + (tid & 63);
        offY[s] = 0;
        if (i < NUY) {
            const int lx = i % TX, ly = i / TX;
            offY[s] = lat(wrapx(x0 + lx), wrapy(y0 + ly - 3));
            ldsY[s] = O_UY + ly * AX + lx + 3;
        }
    }

    // S slots (FS): the plane's S on the tile with a one-cell halo (the 3D
    // corners are loaded and not read)
    constexpr int NSS = FS ? SXL * SYL : 0;
    constexpr int SSS = (NSS + NT - 1) / NT;
    uint32_t offS[(SSS > 0) ? SSS : 1];
    int ldsS[(SSS > 0) ? SSS : 1];
#pragma unroll
    for (int s = 0; s < SSS; ++s) {
        const int i = tid + s * NT;
        ldsS[s] = O_END + (tid & 63);
        offS[s] = 0;
        if (i < NSS) {
            const int lx = i % SXL, ly = i / SXL;
            offS[s] = lat(wrapx(x0 + lx - 1), (D == 3) ? wrapy(y0 + ly - 1) : 0);
            ldsS[s] = O_S + i;
        }
    }
    const T *__restrict__ sin = (const T *)(FS && s_entry ? r.s : r.c);
    const T kaps = (T)r.kappa_s;
    auto sface = [&](T a2, T a3, T w2, T w3) -> T { return s_face<T>(a2, a3, w2, w3, kaps); };

    constexpr int NEX = (D == 3) ? TX + TY : 1;   // faces on the tile's far edges

    // vertical windows for the face above v: a and w at v-2 .. v+3 (face6),
    // or (NV) the node data of the same nodes: fluxes vH at v-2 .. v+3, the
    // indicators e_l, e_c, e_r of nodes v-1 .. v+2 (EL, EC, ER), and for the
    // faces j+1/2, j = v .. v+2, the upwind side vP (w_j + w_{j+1} >= 0) and
    // the difference vD = a_{j+1} - a_j (a face's slot is its lower node's);
    // a_last, w_last hold node v+3
    const T eps12 = (T)(12.0 / 13.0) * eps;
    T aw[6], ww[6];
    T vH[6], vD[6];
    // the indicators of the window's nodes, per thread in LDS (each thread reads
    // only what it wrote), in rings as long as their nodes wait: a node enters
    // at position 5, its e_l is last read at position 1, e_c at 2, e_r at 3
    __shared__ T sE[NV ? 11 * NT : 1];
    auto EL = [&](int slot) -> T & { return sE[slot * NT + tid]; };
    auto EC = [&](int slot) -> T & { return sE[(6 + slot % 3) * NT + tid]; };
    auto ER = [&](int slot) -> T & { return sE[(9 + slot % 2) * NT + tid]; };
    bool vP[6];
    T a_last = (T)0, w_last = (T)0, a_first;
    T fbelow;                                       // face below the first plane
    if constexpr (NV) {
        T an[7], wn[7], hn[7], dn[6], sn[6], ln[7], cn[7], rn[7];   // nodes v0-3 .. v0+3
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            load_av(v0 - 3 + k, an[k], wn[k]);
            hn[k] = wn[k] * an[k];
        }
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            dn[k] = an[k + 1] - an[k];
            sn[k] = wn[k] + wn[k + 1];
        }
#pragma unroll
        for (int k = 1; k < 6; ++k) weno5_node<T>(dn[k - 1], dn[k], eps12, ln[k], cn[k], rn[k]);
        // window position m is node v0-2+m, index k = m+1 here
#pragma unroll
        for (int m = 0; m < 6; ++m) vH[m] = hn[m + 1];
#pragma unroll
        for (int m = 1; m < 5; ++m) {
            EL(m) = ln[m + 1];
            if (m >= 2) EC(m) = cn[m + 1];
            if (m >= 3) ER(m) = rn[m + 1];
        }
#pragma unroll
        for (int m = 2; m < 5; ++m) {
            vP[m] = sn[m + 1] >= (T)0;
            vD[m] = dn[m + 1];
        }
        a_last = an[6];
        w_last = wn[6];
        a_first = an[3];
        if (!(walls && v0 == 0))
            fbelow = weno5_flux_nodes<T>(sn[2] >= (T)0, hn[0], hn[1], hn[2], hn[3], hn[4], hn[5], ln[1],
                                         ln[2], cn[2], cn[3], rn[3], rn[4], dn[2], kap);
    } else {
#pragma unroll
        for (int m = 0; m < 6; ++m) load_av(v0 - 2 + m, aw[m], ww[m]);
        a_first = aw[2];
        if (!(walls && v0 == 0)) {
            T ab, wb;
            load_av(v0 - 3, ab, wb);
            fbelow = face6<T, SCHEME>(ab, aw[0], aw[1], aw[2], aw[3], aw[4], wb, ww[0], ww[1], ww[2],
                                      ww[3], ww[4], kap, eps);
        }
    }
    if (walls && v0 == 0) fbelow = -vs_at(0) * a_first;   // absorbing bottom

    // S and the raw vertical velocity at this plane of the column, and the S
    // face below the first plane (closed walls; periodic: wrapped)
    T s_c = (T)0, us_c = (T)0, gbelow = (T)0;
    if constexpr (FS) {
        s_c = at<T>(plane(sin, v0), colb);
        us_c = at<T>(plane(uv, v0), colb);
        if (!(walls && v0 == 0)) {
            T sgn;
            const int vb = vidx(v0 - 1, sgn);
            gbelow = sface(at<T>(plane(sin, vb), colb), s_c, at<T>(plane(uv, vb), colb), us_c);
        }
    }

    // deposit of stage 3 (D += Vs (C/6 + a1/6 + 2 a2/3) at the bottom cell),
    // done before the march so that no load or store sits on a path of its own
    if constexpr (STAGE == 3) {
        if (walls && v0 == 0 && active) {
            r.dep[col] += deposit_of<T, VSS>(r, (const T *)r.s, col, at<T>(plane(r.c, 0), colb),
                                             at<T>(plane(r.c1, 0), colb), a_first);
        }
    }

    // prefetch registers for the lateral planes
    T pA[SA], pX[SUX], pY[(SUY > 0) ? SUY : 1], pS[(SSS > 0) ? SSS : 1];
    auto prefetch = [&](int v) {
        T sgn;
        const int vv = vidx_up(v, sgn);
        const void *pa = plane(ain, vv), *px = plane(ux, vv), *py = plane(uy, vv);
#pragma unroll
        for (int s = 0; s < SSS; ++s) pS[s] = at<T>(plane(sin, vv), offS[s]);
        // unconditional, so no load sits behind a branch
#pragma unroll
        for (int s = 0; s < SA; ++s) pA[s] = at<T>(pa, offA[s]);
#pragma unroll
        for (int s = 0; s < SUX; ++s) pX[s] = at<T>(px, offX[s]);
#pragma unroll
        for (int s = 0; s < SUY; ++s) pY[s] = at<T>(py, offY[s]);
    };
    auto publish = [&](int set) {
#pragma unroll
        for (int s = 0; s < SA; ++s) smem[set * SET + ldsA[s]] = pA[s];
#pragma unroll
        for (int s = 0; s < SUX; ++s) smem[set * SET + ldsX[s]] = pX[s];
#pragma unroll
        for (int s = 0; s < SUY; ++s) smem[set * SET + ldsY[s]] = pY[s];
#pragma unroll
        for (int s = 0; s < SSS; ++s) smem[set * SET + ldsS[s]] = pS[s];
    };
    prefetch(v0);
    publish(0);
    prefetch(v0 + 1);
    __syncthreads();

    // The march is unrolled six planes at a time with the window slots
    // rotating: at phase ph, window position m lives in slot (ph + m) % 6,
    // and the node entering at v + 4 takes the slot position 0 leaves, so no
    // register moves shift the window from plane to plane.
    for (int vb = v0; vb < v1; vb += 6) {
#pragma unroll
        for (int ph = 0; ph < 6; ++ph) {
            const int v = vb + ph;
            if (v >= v1) break;
            // window position m (node v - 2 + m) of this phase
            auto A = [&](int m) -> T & { return aw[(ph + m) % 6]; };
            auto W = [&](int m) -> T & { return ww[(ph + m) % 6]; };
            // the lane offsets pass through an empty asm every plane: the
            // compiler can then no longer fold them into per-lane 64-bit
            // pointers hoisted out of the march (each plane's offset would be
            // added to those in vector instructions), and the loads keep the
            // scalar-base plus 32-bit-offset form
            asm volatile("" : "+v"(colb));
#pragma unroll
            for (int s = 0; s < SA; ++s) asm volatile("" : "+v"(offA[s]));
#pragma unroll
            for (int s = 0; s < SUX; ++s) asm volatile("" : "+v"(offX[s]));
#pragma unroll
            for (int s = 0; s < SUY; ++s) asm volatile("" : "+v"(offY[s]));
#pragma unroll
            for (int s = 0; s < SSS; ++s) asm volatile("" : "+v"(offS[s]));
            const int cur = ph & 1;
            T *const set = smem + cur * SET;
            T *const sA = set + O_A;                   // stage input a, plane with halos
            T *const sUx = set + O_UX;                 // x velocity, rows with x halo
            T *const sUy = set + O_UY;                 // y velocity, columns with y halo
            T *const sFx = set + O_FX;                 // x face fluxes
            T *const sFy = set + O_FY;                 // y face fluxes
            T *const sS = set + O_S;                   // S plane with a one-cell halo
            T *const sGx = set + O_GX;                 // S face fluxes
            T *const sGy = set + O_GY;
            // loads, in the order they are consumed (the load counter drains in
            // issue order, so waiting for one waits for all issued before it):
            // this cell's C and the vertical pair at v+4, both used at the end of
            // this plane, which the lateral plane v+2, loaded after its faces, is
            // in flight past (beyond the chunk it is still a valid plane: the
            // vertical rule maps it inside)
            T cown = (T)0;
            if (STAGE != 1) cown = at<T>(plane(r.c, v), colb);
            T anext, wnext, snext;
            const int vnext = vidx_up(v + 4, snext);
            load_at(vnext, snext, anext, wnext);
            T s_n = (T)0, us_n = (T)0;
            if constexpr (FS) {
                T sgn;
                const int vn = vidx_up(v + 1, sgn);
                s_n = at<T>(plane(sin, vn), colb);
                us_n = at<T>(plane(uv, vn), colb);
            }

            // each thread the x face on the left of its cell and (3D) the y
            // face below it; the stage input at the cell is the x stencil's
            // fourth node
            // byte offsets of the faces' first nodes from cell (tx, ty)'s place in a
            // row of AX: x nodes tx-3 .. tx+2 of the row, y rows ty-3 .. ty+2 of the
            // column
            constexpr int XA = (O_A + ((D == 3) ? 3 * AX : 0)) * (int)sizeof(T), XW = O_UX * (int)sizeof(T);
            constexpr int YA = (O_A + 3) * (int)sizeof(T), YW = (O_UY + 3) * (int)sizeof(T);
            const uint32_t cell = (uint32_t)((cur * SET + ty * AX + tx) * (int)sizeof(T));
            T a_own;
            {
                const T *ar = sA + ((D == 3) ? (ty + 3) : 0) * AX + tx;   // nodes tx-3 .. tx+2
                sFx[ty * (TX + 1) + tx] = face6_lds<T, SCHEME, 1, XA, XW>(smem, cell, kap, eps);
                a_own = ar[3];
            }
            if constexpr (D == 3) {
                sFy[ty * TX + tx] = face6_lds<T, SCHEME, AX, YA, YW>(smem, cell, kap, eps);
            }
            if constexpr (FS) {
                // S faces on the left of the cell and (3D) below it
                const T *sr = sS + ((D == 3) ? ty + 1 : 0) * SXL + tx;     // x - 1, x
                const T *ur = sUx + ty * AX + tx + 2;
                sGx[ty * (TX + 1) + tx] = sface(sr[0], sr[1], ur[0], ur[1]);
                if constexpr (D == 3) {
                    const T *sc = sS + ty * SXL + tx + 1;                  // y - 1, y
                    const T *uc = sUy + (ty + 2) * AX + tx + 3;
                    sGy[ty * TX + tx] = sface(sc[0], sc[SXL], uc[0], uc[AX]);
                }
            }
            // faces on the far edges of the tile, taken by the first lanes in
            // one extra pass, so that the main passes are exactly one face
            // per thread: (3D) the y faces of row TY first, so that they
            // fill whole waves (a lane with tid < TX has ty = 0 and tx = tid,
            // so their addresses are the main pass's plus a constant), then
            // the x faces of column TX
            static_assert(NEX <= NT, "one pass of edge faces");
            if (D == 3 && tid < TX) {
                if constexpr (D == 3) {
                    sFy[(ty + TY) * TX + tx] = face6_lds<T, SCHEME, AX, YA, YW>(smem, cell + TY * AX * (int)sizeof(T), kap, eps);
                    if constexpr (FS) {
                        const T *sc = sS + (ty + TY) * SXL + tx + 1;
                        const T *uc2 = sUy + (ty + TY + 2) * AX + tx + 3;
                        sGy[(ty + TY) * TX + tx] = sface(sc[0], sc[SXL], uc2[0], uc2[AX]);
                    }
                }
            } else if (tid < NEX) {
                const int fy = tid - ((D == 3) ? TX : 0);
                sFx[fy * (TX + 1) + TX] =
                    face6_lds<T, SCHEME, 1, XA, XW>(smem, (uint32_t)((cur * SET + fy * AX + TX) * (int)sizeof(T)), kap, eps);
                if constexpr (FS) {
                    const T *sr = sS + ((D == 3) ? fy + 1 : 0) * SXL + TX;
                    const T *ur2 = sUx + fy * AX + TX + 2;
                    sGx[fy * (TX + 1) + TX] = sface(sr[0], sr[1], ur2[0], ur2[1]);
                }
            }
            // vertical face above this cell
            T fabove;
            if constexpr (NV) {
                auto S6 = [&](int m) { return (ph + m) % 6; };
                fabove = weno5_flux_nodes<T>(vP[S6(2)], vH[S6(0)], vH[S6(1)], vH[S6(2)],
                                             vH[S6(3)], vH[S6(4)], vH[S6(5)], EL(S6(1)), EL(S6(2)),
                                             EC(S6(2)), EC(S6(3)), ER(S6(3)), ER(S6(4)), vD[S6(2)], kap);
            } else {
                fabove = face6<T, SCHEME>(A(0), A(1), A(2), A(3), A(4), A(5), W(0), W(1), W(2), W(3),
                                          W(4), W(5), kap, eps);
            }
            fabove = walls && v == g.nv - 1 ? (T)0 : fabove;
            T gabove = (T)0;
            if constexpr (FS) gabove = (walls && v == g.nv - 1) ? (T)0 : sface(s_c, s_n, us_c, us_n);
            publish(1 - cur);           // plane v + 1, its loads in flight since the last plane
            prefetch(v + 2);
            __syncthreads();
            T L = -(fabove - fbelow);
            L -= sFx[ty * (TX + 1) + tx + 1] - sFx[ty * (TX + 1) + tx];
            if constexpr (D == 3) L -= sFy[(ty + 1) * TX + tx] - sFy[ty * TX + tx];
            const T a = a_own;
            if (active) {
                if constexpr (STAGE == 1) {
                    *(T *)((char *)wplane(r.c1, v) + colb) = a + L;
                } else if constexpr (STAGE == 2) {
                    *(T *)((char *)wplane(r.c2, v) + colb) = rk3_stage2<T>(cown, a, L);
                } else {
                    *(T *)((char *)wplane(r.c, v) + colb) = rk3_stage3<T>(cown, a, L);
                }
            }
            if constexpr (FS) {
                T Ls = -(sGx[ty * (TX + 1) + tx + 1] - sGx[ty * (TX + 1) + tx]);
                if constexpr (D == 3) Ls -= sGy[(ty + 1) * TX + tx] - sGy[ty * TX + tx];
                Ls -= gabove - gbelow;
                if (active && s_entry) *(T *)((char *)wplane(r.s2, v) + colb) = s_c + Ls;
                gbelow = gabove;
                s_c = s_n;
                us_c = us_n;
            }
            fbelow = fabove;
            // node v + 4 enters, position 0 leaves
            if constexpr (NV) {
                const T dnew = anext - a_last;
                T el, ec, er;
                weno5_node<T>(vD[(ph + 4) % 6], dnew, eps12, el, ec, er);
                EL((ph + 5) % 6) = el;
                EC((ph + 5) % 6) = ec;
                ER((ph + 5) % 6) = er;
                vD[(ph + 5) % 6] = dnew;
                vP[(ph + 5) % 6] = (w_last + wnext) >= (T)0;
                vH[ph % 6] = wnext * anext;
                a_last = anext;
                w_last = wnext;
            } else {
                A(0) = anext;
                W(0) = wnext;
            }
            // no barrier here: the next publication writes the set whose last
            // readers passed the barrier above, and the face arrays read since
            // are next written two planes on
        }
    }
}

template <typename T, int D, int SCHEME, int STAGE, int TX, int TY, bool FULL, bool VSS, bool FS = false>
__global__ void __launch_bounds__(TX *TY) k_stage_tiled(RunDev r, ClassSet cs, TileGeom g) {
    int bx, by, bz, cls;
    block_tile(g, cs.n, bx, by, bz, cls);
    const bool s_entry = select_class<T>(r, cs, cs.first + cls);
    stage_tile<T, D, SCHEME, STAGE, TX, TY, FULL, VSS, FS>(r, g, bx, by, bz, s_entry);
}

template <int D>
__host__ __device__ inline TileGeom make_geom(const RunDev &r, int chunk, int TX, int TY) {
    TileGeom g;
    g.nx = r.nx;
    g.ny = (D == 3) ? r.ny : 1;
    g.nv = (D == 3) ? r.nz : r.ny;
    g.sv = (D == 3) ? (int64_t)r.nx * r.ny : (int64_t)r.nx;
    g.N = r.N;
    g.vper = r.vper;
    g.chunk = chunk < g.nv ? chunk : g.nv;
    g.gx = (r.nx + TX - 1) / TX;
    g.gy = (D == 3) ? (r.ny + TY - 1) / TY : 1;
    g.gz = (g.nv + g.chunk - 1) / g.chunk;
    g.bz0 = 0;
    return g;
}

// Batched form: one persistent grid walks the tiles of every run.  Each XCD
// takes a contiguous range of the global tile list (runs in order, tiles of
// a run x-fastest), so neighbouring tiles share an L2.  tile_start[b] is the
// first global tile of run b (prefix sum, nbatch + 1 entries).
template <typename T, int D, int SCHEME, int STAGE, int TX, int TY, bool VSS, bool FS = false>
__global__ void __launch_bounds__(TX *TY) k_stage_batched(const RunDev *__restrict__ runs,
                                                          const int *__restrict__ tile_start,
                                                          int nbatch, int chunk, int sflip,
                                                          int form) {
    const int total = tile_start[nbatch];
    const int G = gridDim.x;
    // with 8 blocks or more, block i runs on XCD i % 8 and that XCD walks its
    // own contiguous range; a smaller grid would leave some ranges with no
    // block, so it walks the whole list instead
    int first = blockIdx.x, stride = G, hi = total;
    if (G >= 8) {
        const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
        first = xcd_first(xcd, total) + slot;
        hi = xcd_first(xcd + 1, total);
        stride = xcd_first(xcd + 1, G) - xcd_first(xcd, G);   // blocks on this XCD (>= 1)
    }
    int b = 0;
    for (int w = first; w < hi; w += stride) {
        b = entry_of(tile_start, nbatch, b, w);            // w only grows, so b only grows
        RunDev r = runs[b];
        if (form >= 0 && (r.vs_s != 0.0) != (form == 1)) continue;   // the other form's entry
        if (sflip) { void *t = r.s; r.s = r.s2; r.s2 = t; }
        const TileGeom g = make_geom<D>(r, chunk, TX, TY);
        const int t = w - tile_start[b];
        const int bx = t % g.gx, rest = t / g.gx;
        stage_tile<T, D, SCHEME, STAGE, TX, TY, false, VSS, FS>(r, g, bx, rest % g.gy, rest / g.gy,
                                                               r.has_s != 0);
    }
}

// The whole-tile form when the grid divides into tiles, else the masked one
// (runs with a variable settling speed always take the masked form, which
// halves the kernels built for them).
template <typename T, int D, int SCHEME, int STAGE, int TX, int TY, bool VSS, bool FS = false>
void launch_stage(const RunDev &r, const ClassSet &cs, const TileGeom &g, unsigned nb, hipStream_t st) {
    if constexpr (!VSS) {
        if (g.nx % TX == 0 && (D == 2 || g.ny % TY == 0)) {
            k_stage_tiled<T, D, SCHEME, STAGE, TX, TY, true, false, FS><<<nb, TX * TY, 0, st>>>(r, cs, g);
            return;
        }
    }
    k_stage_tiled<T, D, SCHEME, STAGE, TX, TY, false, VSS, FS><<<nb, TX * TY, 0, st>>>(r, cs, g);
}

// Stage 1, carrying the S update when the run has S.
template <typename T, int D, int SCHEME, int TX, int TY, bool VSS>
void launch_stage1(const RunDev &r, const ClassSet &cs, const TileGeom &g, unsigned nb, hipStream_t st) {
    if (r.has_s) launch_stage<T, D, SCHEME, 1, TX, TY, VSS, true>(r, cs, g, nb, st);
    else launch_stage<T, D, SCHEME, 1, TX, TY, VSS, false>(r, cs, g, nb, st);
}

// The three stages (stage 0) or one of them of a single run's classes: one
// launch per stage for all of them, so that they fill the chip together, class
// by class only where one launch would need 2^32 work-items.
template <typename T, int D, int SCHEME, int TX, int TY, bool VSS>
hipError_t stages(const RunDev &r, const ClassSet &cs, int chunk, int stage, hipStream_t st) {
    const TileGeom g = make_geom<D>(r, chunk, TX, TY);
    const int64_t tiles = (int64_t)g.gx * g.gy * g.gz, nb = tiles * cs.n;
    if (cs.n > 1 && (nb > 0x7fffffff || nb * TX * TY >= ((int64_t)1 << 32))) {
        hipError_t e = hipSuccess;
        ClassSet one = cs;
        one.n = 1;
        for (int i = 0; i < cs.n && e == hipSuccess; ++i) {
            one.first = cs.first + i;
            e = stages<T, D, SCHEME, TX, TY, VSS>(r, one, chunk, stage, st);
        }
        return e;
    }
    if (nb > 0x7fffffff) return hipErrorInvalidValue;
    if (stage == 0 || stage == 1) launch_stage1<T, D, SCHEME, TX, TY, VSS>(r, cs, g, (unsigned)nb, st);
    if (stage == 0 || stage == 2) launch_stage<T, D, SCHEME, 2, TX, TY, VSS>(r, cs, g, (unsigned)nb, st);
    if (stage == 0 || stage == 3) launch_stage<T, D, SCHEME, 3, TX, TY, VSS>(r, cs, g, (unsigned)nb, st);
    return hipGetLastError();
}

// Calls fn(integral_constant TX, integral_constant TY) for the tile shape:
// 3D 32x8, 64x4, 128x2 (256 threads), 32x16, 64x8 (512 threads); 2D one row
// of 64, 128, 256 or 512 columns.
template <int D, typename F>
hipError_t with_tile(const TileShape &sh, F &&fn) {
    using std::integral_constant;
    if constexpr (D == 3) {
        if (sh.tx == 64 && sh.ty == 8) return fn(integral_constant<int, 64>{}, integral_constant<int, 8>{});
        if (sh.tx == 32 && sh.ty == 16) return fn(integral_constant<int, 32>{}, integral_constant<int, 16>{});
        if (sh.tx == 64) return fn(integral_constant<int, 64>{}, integral_constant<int, 4>{});
        if (sh.tx == 128) return fn(integral_constant<int, 128>{}, integral_constant<int, 2>{});
        return fn(integral_constant<int, 32>{}, integral_constant<int, 8>{});
    } else {
        if (sh.tx == 64) return fn(integral_constant<int, 64>{}, integral_constant<int, 1>{});
        if (sh.tx == 128) return fn(integral_constant<int, 128>{}, integral_constant<int, 1>{});
        if (sh.tx == 512) return fn(integral_constant<int, 512>{}, integral_constant<int, 1>{});
        return fn(integral_constant<int, 256>{}, integral_constant<int, 1>{});
    }
}

template <typename T, int D, int SCHEME, int TX, int TY, bool VSS>
hipError_t stages_batched(const BatchArgs &a, hipStream_t st) {
    bool any_s = false;
    for (int i = 0; i < a.nbatch; ++i) any_s = any_s || a.host_runs[i].has_s;
    auto stage = [&](int k) {
        if (k == 1 && any_s)
            k_stage_batched<T, D, SCHEME, 1, TX, TY, VSS, true><<<a.grid, TX * TY, 0, st>>>(
                a.runs, a.tile_start, a.nbatch, a.shape.chunk, a.sflip, a.form);
        else if (k == 1)
            k_stage_batched<T, D, SCHEME, 1, TX, TY, VSS><<<a.grid, TX * TY, 0, st>>>(
                a.runs, a.tile_start, a.nbatch, a.shape.chunk, a.sflip, a.form);
        else if (k == 2)
            k_stage_batched<T, D, SCHEME, 2, TX, TY, VSS><<<a.grid, TX * TY, 0, st>>>(
                a.runs, a.tile_start, a.nbatch, a.shape.chunk, a.sflip, a.form);
        else
            k_stage_batched<T, D, SCHEME, 3, TX, TY, VSS><<<a.grid, TX * TY, 0, st>>>(
                a.runs, a.tile_start, a.nbatch, a.shape.chunk, a.sflip, a.form);
        return hipGetLastError();
    };
    if (a.stage != 0) return stage(a.stage);
    hipError_t e = stage(1);
    if (e == hipSuccess) e = stage(2);
    if (e == hipSuccess) e = stage(3);
    return e;
}

template <typename T, int D, int SCHEME, bool VSS>
hipError_t stages_shape(const RunDev &r, const ClassSet &cs, const TileShape &sh, int stage, hipStream_t st,
                        const BatchArgs *batch) {
    return with_tile<D>(sh, [&](auto tx, auto ty) {
        constexpr int TX = decltype(tx)::value, TY = decltype(ty)::value;
        return batch ? stages_batched<T, D, SCHEME, TX, TY, VSS>(*batch, st)
                     : stages<T, D, SCHEME, TX, TY, VSS>(r, cs, sh.chunk, stage, st);
    });
}

}  // namespace

template <typename T, int D, bool VSS>
hipError_t tiled_unit(const RunDev &r, const ClassSet &cs, const TileShape &sh, int stage, hipStream_t st,
                      const BatchArgs *b) {
    switch (r.scheme) {
        case LBW_WENO5: return stages_shape<T, D, LBW_WENO5, VSS>(r, cs, sh, stage, st, b);
        case LBW_WENO3: return stages_shape<T, D, LBW_WENO3, VSS>(r, cs, sh, stage, st, b);
        case LBW_UPWIND1: return stages_shape<T, D, LBW_UPWIND1, VSS>(r, cs, sh, stage, st, b);
    }
    return hipErrorInvalidValue;
}

}  // namespace lbw
