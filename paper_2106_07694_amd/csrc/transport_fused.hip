// transport_fused.hip -- the whole transport of one 2D step (three RK stages,
// the S update and the deposit) in one launch, for grids too small to fill
// the chip with three.
//
// What bounds it: on such grids a stage launch costs its fixed latency (start,
// first loads, two barriers, about 4.4 us) whatever the cells in it, and the
// next stage cannot start before it ends.  Here a block keeps C, the velocity
// and both intermediate stages of its TX x TY cells in LDS, with the halo the
// stages reach (nine cells of C, six of stage 1, three of stage 2), and
// recomputes the halo instead of exchanging it.  The recomputed cells
// (TX + 12)(TY + 12) + (TX + 6)(TY + 6) cost more arithmetic than three
// launches spend, so larger grids keep the tiled stages.
//
// The step reads C from r.c and writes the result to another buffer (a
// neighbouring block still reads the old values for its halo), so the caller
// alternates two buffers over consecutive steps.  On the smallest grids the
// block's chain of loads and six barriers bounds it (8 us at 64x128 in double
// precision); near the upper limit vector issue does (512x1024 in single
// precision: the kernel takes 15.5 us, of which 13 are its 896 vector
// instructions per cell).  Faces and combinations are those of the tiled stages,
// in the same order: the same bits.
#include "transport_face.h"

namespace lbw {
namespace {

// Position outside [0, n) reached by a halo or an overhanging tile, on a
// periodic axis.
__device__ __forceinline__ int wrap_index(int j, int n) {
    j += j < 0 ? n : 0;
    j -= j >= n ? n : 0;
    if ((unsigned)j < (unsigned)n) return j;
    j %= n;                                          // an axis shorter than the reach
    return j < 0 ? j + n : j;
}

template <typename T, int SCHEME, bool VSS, bool FS, int TX, int TY, int NT>
__global__ void __launch_bounds__(NT) k_rk3_2d(RunDev r, ClassSet cs, T *__restrict__ cout,
                                               T *__restrict__ a1out, T *__restrict__ a2out) {
    // C on the tile with nine halo cells, stage 1 with six, stage 2 with three;
    // the x velocity on stage 1's rows, the vertical transport velocity on
    // stage 1's columns
    constexpr int RX = TX + 18, RY = TY + 18, PX = TX + 12, PY = TY + 12, QX = TX + 6, QY = TY + 6;
    __shared__ T sC[RY * RX], sU[PY * RX], sW[RY * PX], sA1[PY * PX], sA2[QY * QX];
    __shared__ T sFx[PY * (PX + 1)], sFy[(PY + 1) * PX];

    const int64_t off = (int64_t)blockIdx.z * r.N;      // block z: size class z
    cout += off;
    if (a1out) a1out += off;
    if (a2out) a2out += off;
    const bool s_entry = select_class<T>(r, cs, (int)blockIdx.z);

    const int tid = threadIdx.x;
    const int nx = r.nx, ny = r.ny;
    const int x0 = (int)blockIdx.x * TX, y0 = (int)blockIdx.y * TY;
    const bool walls = !r.vper;
    const T *__restrict__ c = (const T *)r.c;
    const T *__restrict__ ux = (const T *)r.u;
    const T *__restrict__ uy = ux + r.N;
    const T *__restrict__ s = (const T *)r.s;
    const T vs = (T)r.vs, kap = (T)r.kappa_c, eps = (T)r.eps;
    auto settle = [&](int k) -> T {
        if constexpr (VSS) return vs * ((T)1 - (T)r.vs_s * s[k]);
        else return vs;
    };
    // stored row of position p (mirrored beyond a wall; rows further out than
    // the three that any cell of the grid reads are clamped into range)
    auto row = [&](int p, bool &ghost) -> int {
        ghost = walls && (p < 0 || p >= ny);
        if (!walls) return wrap_index(p, ny);
        p = p < 0 ? -1 - p : (p >= ny ? 2 * ny - 1 - p : p);
        return min(max(p, 0), ny - 1);
    };

    // stage the inputs, every load issued before the first store to LDS; one
    // position serves C and both velocities (whose regions lie inside C's).
    // Wide tiles give a wave whole rows and a lane one of their columns, so the
    // row's address is scalar and the column's is found once: element by
    // element, the index arithmetic was a quarter of their vector
    // instructions.  The narrow tile's rows would leave half of the lanes idle
    // (64x128 in double precision 13.3 against 12.7 us per step)
    constexpr bool ROWS = RX >= 48;
    static_assert(!ROWS || RX <= 64, "one lane per staged column");
    constexpr int WAVES = NT / 64, LOADS = ROWS ? (RY + WAVES - 1) / WAVES : (RY * RX + NT - 1) / NT;
    auto place = [&](int q, int &ry, int &cx) -> bool {
        if constexpr (ROWS) {
            ry = __builtin_amdgcn_readfirstlane(tid >> 6) + q * WAVES;
            cx = tid & 63;
            return ry < RY && cx < RX;
        } else {
            const int i = tid + q * NT;
            ry = i / RX;
            cx = i % RX;
            return i < RY * RX;
        }
    };
    T pc[LOADS], pu[LOADS], pw[LOADS], ps[VSS ? LOADS : 1], sg[LOADS];
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
        int ry, cx;
        bool g;
        place(q, ry, cx);
        const int64_t at = (int64_t)row(y0 - 9 + min(ry, RY - 1), g) * nx;
        const uint32_t xoff = (uint32_t)wrap_index(x0 - 9 + min(cx, RX - 1), nx) * (uint32_t)sizeof(T);
        auto load = [&](const T *p) { return *(const T *)((const char *)(p + at) + xoff); };
        sg[q] = g ? (T)-1 : (T)1;
        pc[q] = load(c);
        pu[q] = load(ux);
        pw[q] = load(uy);
        if constexpr (VSS) ps[q] = load(s);
    }
#pragma unroll
    for (int q = 0; q < LOADS; ++q) {
        int ry, cx;
        if (!place(q, ry, cx)) continue;
        sC[ry * RX + cx] = pc[q];
        if (ry >= 3 && ry < RY - 3) sU[(ry - 3) * RX + cx] = pu[q];
        if (cx >= 3 && cx < RX - 3) {
            const T fall = VSS ? vs * ((T)1 - (T)r.vs_s * ps[q]) : vs;
            sW[ry * PX + cx - 3] = sg[q] * pw[q] - fall;
        }
    }

    // S: forward Euler on the tile's own cells, straight from memory
    if constexpr (FS) {
        const T kaps = (T)r.kappa_s;
        for (int i = tid; i < (s_entry ? TX * TY : 0); i += NT) {
            const int x = x0 + i % TX, y = y0 + i / TX;
            if (x >= nx || y >= ny) continue;
            const int k = x + nx * y;
            const int kl = x == 0 ? k + nx - 1 : k - 1, kr = x == nx - 1 ? k - (nx - 1) : k + 1;
            const int kd = y == 0 ? k + nx * (ny - 1) : k - nx, ku = y == ny - 1 ? k - nx * (ny - 1) : k + nx;
            const T s0 = s[k], u0 = ux[k], v0 = uy[k];
            const T gl = s_face<T>(s[kl], s0, ux[kl], u0, kaps), gr = s_face<T>(s0, s[kr], u0, ux[kr], kaps);
            const T gd = (walls && y == 0) ? (T)0 : s_face<T>(s[kd], s0, uy[kd], v0, kaps);
            const T gu = (walls && y == ny - 1) ? (T)0 : s_face<T>(s0, s[ku], v0, uy[ku], kaps);
            T L = -(gr - gl);
            L -= gu - gd;
            ((T *)r.s2)[k] = s0 + L;
        }
    }
    __syncthreads();

    // one RK stage on the tile with a halo of H cells; `in` holds its input
    // with three more
    auto stage = [&](auto stage_id, auto halo, const T *in) {
        constexpr int STAGE = decltype(stage_id)::value, H = decltype(halo)::value;
        constexpr int OX = TX + 2 * H, OY = TY + 2 * H, IX = OX + 6;
        constexpr int FX = OY * (OX + 1), FY = (OY + 1) * OX;
        // a thread takes an x face and a y face at once, without branches, so
        // that the two chains of dependent arithmetic overlap
        for (int i = tid; i < (FX > FY ? FX : FY); i += NT) {
            const int fx = min(i, FX - 1), fy = min(i, FY - 1);
            T fl, fb;
            {                                            // face on the left of cell (cx, ry)
                const int ry = fx / (OX + 1), cx = fx % (OX + 1);
                const T *a = in + (ry + 3) * IX + cx, *w = sU + (ry + 6 - H) * RX + cx + 6 - H;
                fl = face6<T, SCHEME>(a[0], a[1], a[2], a[3], a[4], a[5], w[0], w[1], w[2], w[3], w[4],
                                      w[5], kap, eps);
            }
            {                                            // face below cell (cx, ry)
                const int ry = fy / OX, cx = fy % OX, y = y0 - H + ry;
                const T *a = in + ry * IX + cx + 3, *w = sW + (ry + 6 - H) * PX + cx + 6 - H;
                fb = face6<T, SCHEME>(a[0], a[IX], a[2 * IX], a[3 * IX], a[4 * IX], a[5 * IX], w[0], w[PX],
                                      w[2 * PX], w[3 * PX], w[4 * PX], w[5 * PX], kap, eps);
                if (walls && y == ny) fb = (T)0;         // closed top; rows further out are not read
                if (walls && y == 0) fb = -settle(wrap_index(x0 - H + cx, nx)) * a[3 * IX];   // absorbing bottom
            }
            sFx[fx] = fl;
            sFy[fy] = fb;
        }
        __syncthreads();
        for (int i = tid; i < OX * OY; i += NT) {
            const int ry = i / OX, cx = i % OX, x = x0 - H + cx, y = y0 - H + ry;
            if (walls && (y < 0 || y >= ny)) continue;   // rows beyond a wall are mirrored below
            T L = -(sFy[i + OX] - sFy[i]);
            L -= sFx[ry * (OX + 1) + cx + 1] - sFx[ry * (OX + 1) + cx];
            const T a = in[(ry + 3) * IX + cx + 3];
            const bool own = cx >= H && cx < H + TX && ry >= H && ry < H + TY && x < nx && y < ny;
            const int k = x + nx * y;
            if constexpr (STAGE == 3) {
                const T c0 = sC[(ry + 9) * RX + cx + 9];
                if (own) {
                    cout[k] = rk3_stage3<T>(c0, a, L);
                    if (walls && y == 0) r.dep[x] += deposit_of<T, VSS>(r, s, k, c0, sA1[6 * PX + cx + 6], a);
                }
            } else {
                T *out = STAGE == 1 ? sA1 : sA2, *global = STAGE == 1 ? a1out : a2out;
                const T v = STAGE == 1 ? a + L : rk3_stage2<T>(sC[(ry + 9 - H) * RX + cx + 9 - H], a, L);
                out[i] = v;
                if (walls) {                             // images beyond the walls
                    const int lo = -1 - y - (y0 - H), hi = 2 * ny - 1 - y - (y0 - H);
                    if (lo >= 0) out[lo * OX + cx] = v;
                    if (hi < OY) out[hi * OX + cx] = v;
                }
                if (global && own) global[k] = v;
            }
        }
        if constexpr (STAGE != 3) __syncthreads();
    };
    using std::integral_constant;
    stage(integral_constant<int, 1>{}, integral_constant<int, 6>{}, sC);
    stage(integral_constant<int, 2>{}, integral_constant<int, 3>{}, sA1);
    stage(integral_constant<int, 3>{}, integral_constant<int, 0>{}, sA2);
}

template <typename T, int SCHEME, int TX, int TY, int NT>
hipError_t fused_tile(const RunDev &r, const ClassSet &cs, void *cout, void *a1, void *a2, hipStream_t st) {
    const dim3 grid((unsigned)((r.nx + TX - 1) / TX), (unsigned)((r.ny + TY - 1) / TY), (unsigned)cs.n);
    T *o = (T *)cout, *p = (T *)a1, *q = (T *)a2;
    if (r.vs_s != 0.0 && r.has_s) k_rk3_2d<T, SCHEME, true, true, TX, TY, NT><<<grid, NT, 0, st>>>(r, cs, o, p, q);
    else if (r.vs_s != 0.0) k_rk3_2d<T, SCHEME, true, false, TX, TY, NT><<<grid, NT, 0, st>>>(r, cs, o, p, q);
    else if (r.has_s) k_rk3_2d<T, SCHEME, false, true, TX, TY, NT><<<grid, NT, 0, st>>>(r, cs, o, p, q);
    else k_rk3_2d<T, SCHEME, false, false, TX, TY, NT><<<grid, NT, 0, st>>>(r, cs, o, p, q);
    return hipGetLastError();
}

// The tile whose launch is estimated to end first.  A CU holds two blocks (32
// waves) at a time, one of the two largest tiles in double precision (92 and 111
// KB of LDS), and with k = ceil(blocks / 256) of them to work off it takes about
// start + k * block us (measured as the transport of a step, launch included, on
// grids from 128x256 to 1024x1536, each tile on all of them; within 1 us up to
// k = 4): a small tile recomputes more halo per cell, a large one leaves CUs idle,
// and one block beyond a multiple of 256 costs a whole block's time (515x1030 in
// single precision: 561 blocks of 32x32 take 23.2 us, 442 of 32x40 20.1;
// 512x1024: 512 of 32x32 16.8, 416 of 32x40 19.6).
struct FusedTile {
    int tx, ty;
    float start, block;
};
constexpr FusedTile kTilesF32[] = {{16, 16, 6.9f, 2.45f}, {32, 16, 6.2f, 3.55f}, {32, 24, 7.0f, 4.4f},
                                   {32, 32, 6.5f, 5.25f}, {32, 40, 7.6f, 6.35f}, {32, 48, 8.0f, 7.05f}};
constexpr FusedTile kTilesF64[] = {{16, 16, 7.5f, 3.85f}, {32, 16, 7.6f, 5.5f}, {32, 24, 5.0f, 10.5f},
                                   {32, 32, 4.0f, 12.7f}};

// LDS of a block of k_rk3_2d, bytes
constexpr int fused_lds(const FusedTile &t, int element) {
    const int rx = t.tx + 18, ry = t.ty + 18, px = t.tx + 12, py = t.ty + 12;
    return element * (ry * rx + py * rx + ry * px + py * px + (t.tx + 6) * (t.ty + 6) + py * (px + 1) + (py + 1) * px);
}
constexpr int kLds = 160 << 10;
static_assert(2 * fused_lds(kTilesF32[5], 4) <= kLds && 2 * fused_lds(kTilesF64[1], 8) <= kLds &&
                  2 * fused_lds(kTilesF64[2], 8) > kLds && fused_lds(kTilesF64[3], 8) <= kLds,
              "blocks a CU holds, as said above");

template <typename T, int SCHEME>
hipError_t fused_scheme(const RunDev &r, const ClassSet &cs, void *cout, void *a1, void *a2, hipStream_t st) {
    const FusedTile *best = nullptr;
    float least = 0.f;
    auto consider = [&](const FusedTile &t) {
        const int64_t blocks = (int64_t)((r.nx + t.tx - 1) / t.tx) * ((r.ny + t.ty - 1) / t.ty) * cs.n;
        const float us = t.start + t.block * (float)((blocks + 255) / 256);
        if (!best || us < least) {
            best = &t;
            least = us;
        }
    };
    if constexpr (sizeof(T) == 4) {
        for (const FusedTile &t : kTilesF32) consider(t);
    } else {
        for (const FusedTile &t : kTilesF64) consider(t);
    }
    if (best->tx == 16) return fused_tile<T, SCHEME, 16, 16, 1024>(r, cs, cout, a1, a2, st);
    switch (best->ty) {
        case 16: return fused_tile<T, SCHEME, 32, 16, 1024>(r, cs, cout, a1, a2, st);
        case 24: return fused_tile<T, SCHEME, 32, 24, 1024>(r, cs, cout, a1, a2, st);
        case 32: return fused_tile<T, SCHEME, 32, 32, 1024>(r, cs, cout, a1, a2, st);
    }
    if constexpr (sizeof(T) == 4) {
        if (best->ty == 40) return fused_tile<T, SCHEME, 32, 40, 1024>(r, cs, cout, a1, a2, st);
        if (best->ty == 48) return fused_tile<T, SCHEME, 32, 48, 1024>(r, cs, cout, a1, a2, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace

template <typename T>
hipError_t fused_unit(const RunDev &r, const ClassSet &cs, void *cout, void *a1, void *a2, hipStream_t st) {
    switch (r.scheme) {
        case LBW_WENO5: return fused_scheme<T, LBW_WENO5>(r, cs, cout, a1, a2, st);
        case LBW_WENO3: return fused_scheme<T, LBW_WENO3>(r, cs, cout, a1, a2, st);
        case LBW_UPWIND1: return fused_scheme<T, LBW_UPWIND1>(r, cs, cout, a1, a2, st);
    }
    return hipErrorInvalidValue;
}

// built once per element type (LBW_T)
template hipError_t fused_unit<LBW_T>(const RunDev &, const ClassSet &, void *, void *, void *, hipStream_t);

}  // namespace lbw
