// adjoint.hip -- reverse mode of one coupled step (WENO5 transport, no S).
//
// Objective sensitivities flow backwards through the step of lbm.hip and
// transport.hip:  J depends on the state at n+1 through (fbar_next of the
// populations, cbar_next of C, dep_bar of every deposit counter); this step
// returns the adjoints of the state at n (fbar, cbar) and adds dJ/dVs.
//
//  1. recompute, from the saved forward state at n: the node velocity u^n
//     (moments, eq. 19-20 with the Guo shift) and the RK stages a1, a2;
//  2. RK3 in reverse (S21-S23 transposed) with the deposit update: each stage
//     needs lam^T dL/da and lam^T dL/du at its input.  The transpose of L is
//     taken face by face: one kernel evaluates every interior face once,
//     multiplies its local Jacobian (six stencil values of a and of the
//     transport velocity, the WENO5 weights differentiated through the
//     smoothness indicators, the upwind side held at its forward choice) by
//     the face's adjoint lam_{j+1} - lam_j and stores the twelve products;
//     a second kernel gathers, for every node, the products of every face
//     stencil that reads it, including stencils that read it as a mirror
//     image beyond a wall (where the vertical velocity enters with a sign
//     flip and the settling speed unchanged);
//  3. streaming in reverse (each population pulls the adjoint from where the
//     forward step sent it), then BGK + Guo collision and the moments in
//     reverse, adding the transport's velocity sensitivity; the force's C
//     dependence closes the loop into cbar.  This runs in the gather kernel
//     of the last reversed stage, once the node's velocity adjoint is whole.
// Every node's adjoint is written by exactly one thread; dJ/dVs is gathered
// per node and summed in a fixed order (FP64).
#include "lbm_device.h"
#include "transport_device.h"

// The one-kernel and the two-kernel form of a reversed stage give the same
// bits, so multiply-adds are fused only within one source expression: the
// default fast contraction also fuses across statements, differently in each
// kernel.  What is better fused is written as one expression.
#pragma clang fp contract(on)

namespace lbw {
namespace {

struct AdjDev {
    RunDev r;
    const void *f_n, *c_n, *rho_n, *fbar_next, *cbar_next;
    void *fbar, *cbar;
    void *u, *a1, *a2, *abar1, *abar2, *ubar, *faceA, *faceW;
    double *vs_part, *partials, *vs_bar;
    double dep_bar;
    int frozen;
    int have_u, have_rho, have_stages;   // forward intermediates supplied by the caller
};

// Periodic index of a position at most three cells outside [0, n): one
// conditional add when n >= 4, the general remainder for tiny axes.
__device__ __forceinline__ int wrap_near(int j, int n) {
    if (n >= 4) return j < 0 ? j + n : (j >= n ? j - n : j);
    j %= n;
    return j < 0 ? j + n : j;
}

template <int D>
__device__ __forceinline__ void xyz(const RunDev &r, int64_t k, int &x, int &y, int &z) {
    coords<D>(r, k, x, y, z);
}

// ---------------------------------------------------------------------------
// 1. moments of the saved populations: u^n (force-shifted)
// ---------------------------------------------------------------------------
template <int Q, typename T, bool SH>
__global__ void __launch_bounds__(256) k_adj_moments(AdjDev a) {
    using L = Lattice<Q>;
    constexpr int D = L::D;
    const RunDev &r = a.r;
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= r.N) return;
    const T *f = (const T *)a.f_n;
    T fi[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) fi[i] = f[(int64_t)i * r.N + k];
    T F[3], u[3], rho, drho;
    lbm_force<D, T>(r, (const T *)a.c_n, nullptr, k, F);
    lbm_rho_u<Q, T, SH>(fi, F, rho, drho, u);
    T *uo = (T *)a.u;
#pragma unroll
    for (int d = 0; d < D; ++d) uo[(int64_t)d * r.N + k] = u[d];
}

// ---------------------------------------------------------------------------
// 2. transpose of the spatial operator
// ---------------------------------------------------------------------------

// Reciprocal: exact in double; the hardware reciprocal (about 1 ulp) in
// single precision.
template <typename T> __device__ __forceinline__ T rcp(T x) { return (T)1 / x; }
template <> __device__ __forceinline__ float rcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }

// Reciprocals of three indicators, none of them below `least` (the same for
// every face): one division for all of them in double precision (a division is
// some ten instructions there) as long as their products stay in range, which
// indicators from 1e-100 on and with a product up to 1e200 do; a smaller
// weno_eps takes a division each.  In single precision the hardware reciprocal
// of each.
__device__ __forceinline__ void rcp3(float e0, float e1, float e2, float, float &i0, float &i1, float &i2) {
    i0 = rcp<float>(e0);
    i1 = rcp<float>(e1);
    i2 = rcp<float>(e2);
}
__device__ __forceinline__ void rcp3(double e0, double e1, double e2, double least, double &i0, double &i1,
                                     double &i2) {
    const double e12 = e1 * e2, e = e0 * e12;
    if (least >= 1e-100 && e <= 1e200) {
        const double i = 1.0 / e;
        i0 = i * e12;
        i1 = i * (e0 * e2);
        i2 = i * (e0 * e1);
    } else {
        i0 = 1.0 / e0;
        i1 = 1.0 / e1;
        i2 = 1.0 / e2;
    }
}

// Products of one face's local Jacobian with its adjoint pb, for the five
// nodes its WENO5-JS reconstruction reads, ordered upwind -> downwind (values
// a, transport velocities w; the sixth node of the stencil enters nothing):
//   A[s] = pb * dPhi/da_s (through the fluxes h = w a, the indicators and the
//          central diffusion -kd (a_3 - a_2)),  W[s] = pb * dPhi/dw_s.
// Indicators are scaled by 12/13 as in the forward faces (weights are ratios):
// e_k = t_k^2 + (3/13) s_k^2 + eps12 with t_k, s_k built from the four first
// differences g, and the reverse runs through g as well: 130 vector
// instructions a face in single precision, 200 with the differences of a
// written out and the upwind side selected among the results.
template <typename T>
__device__ __forceinline__ void face_vjp(const T a[5], const T w[5], T pb, T kd, T eps12, T A[5], T W[5]) {
    const T g0 = a[1] - a[0], g1 = a[2] - a[1], g2 = a[3] - a[2], g3 = a[4] - a[3];
    const T t0 = g1 - g0, t1 = g2 - g1, t2 = g3 - g2;
    const T s0 = t0 + (T)2 * g1;          // a0 - 4 a1 + 3 a2
    const T s1 = g1 + g2;                 // a3 - a1
    const T s2 = t2 - (T)2 * g2;          // 3 a2 - 4 a3 + a4
    constexpr T k = (T)(3.0 / 13.0);
    const T r0 = k * s0, r1 = k * s1, r2 = k * s2;
    T i0, i1, i2;
    rcp3(t0 * t0 + (r0 * s0 + eps12), t1 * t1 + (r1 * s1 + eps12), t2 * t2 + (r2 * s2 + eps12), eps12, i0, i1,
         i2);
    // weights in the ratio 1 : 6 : 3, their sum below 1 / weno_eps^2
    const T al0 = (T)0.0625 * i0 * i0, al1 = (T)0.375 * i1 * i1, al2 = (T)0.1875 * i2 * i2;
    const T iS = rcp<T>(al0 + al1 + al2);
    // candidates less h_2, from the first differences of h: only q_k - f enters,
    // which 1 / e_k multiplies, so its rounding is the face's leading error
    const T y0 = w[1] * a[1] - w[0] * a[0], y1 = w[2] * a[2] - w[1] * a[1];
    const T y2 = w[3] * a[3] - w[2] * a[2], y3 = w[4] * a[4] - w[3] * a[3];
    const T q0 = (T)(5.0 / 6.0) * y1 - (T)(1.0 / 3.0) * y0;
    const T q1 = (T)(1.0 / 6.0) * y1 + (T)(1.0 / 3.0) * y2;
    const T q2 = (T)(2.0 / 3.0) * y2 - (T)(1.0 / 6.0) * y3;
    const T fS = al0 * q0 + al1 * q1 + al2 * q2;
    // f = fS / S: df/dq_k = al_k / S, df/dal_k = (q_k - f) / S,
    // dal_k/de_k = -2 al_k / e_k, de_k/dt_k = 2 t_k, de_k/ds_k = 2 (3/13) s_k
    const T p = pb * iS;
    const T b0 = al0 * p, b1 = al1 * p, b2 = al2 * p;
    const T m0 = (q0 - fS * iS) * b0 * ((T)-4 * i0);
    const T m1 = (q1 - fS * iS) * b1 * ((T)-4 * i1);
    const T m2 = (q2 - fS * iS) * b2 * ((T)-4 * i2);
    const T v0 = r0 * m0, v1 = r1 * m1, v2 = r2 * m2;        // of s_k
    const T d0 = t0 * m0 + v0, d2 = t2 * m2 + v2;            // of t_0, t_2 (s_0, s_2 hold them); of t_1 t_1 m_1
    const T c1 = (d0 + (T)2 * v0) + (v1 - t1 * m1);          // of g_1; of g_0 -d0, of g_3 d2
    const T c2 = ((v1 + t1 * m1) - (d2 + (T)2 * v2)) - kd * pb;   // of g_2
    W[0] = (T)(1.0 / 3.0) * b0;
    W[1] = (T)(-7.0 / 6.0) * b0 - (T)(1.0 / 6.0) * b1;
    W[2] = (T)(11.0 / 6.0) * b0 + ((T)(5.0 / 6.0) * b1 + (T)(1.0 / 3.0) * b2);
    W[3] = (T)(1.0 / 3.0) * b1 + (T)(5.0 / 6.0) * b2;
    W[4] = (T)(-1.0 / 6.0) * b2;
    A[0] = d0 + W[0] * w[0];
    A[1] = (-d0 - c1) + W[1] * w[1];
    A[2] = (c1 - c2) + W[2] * w[2];
    A[3] = (c2 - d2) + W[3] * w[3];
    A[4] = d2 + W[4] * w[4];
#pragma unroll
    for (int s = 0; s < 5; ++s) W[s] = W[s] * a[s];
}

// For every interior face j+1/2 (stored at its lower node j) and axis d:
//   faceA[d][s] = phibar * dPhi/da_{j-2+s},  faceW[d][s] = phibar * dPhi/dw_{j-2+s}
// with phibar = scale * (lam_{j+1} - lam_j).  Wall faces store zeros.
template <typename T, int D>
__global__ void __launch_bounds__(256) k_adj_face(AdjDev A, const T *__restrict__ a,
                                                  const T *__restrict__ lam, T scale) {
    const RunDev &r = A.r;
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= r.N) return;
    int x, y, z;
    xyz<D>(r, k, x, y, z);
    const T *u = (const T *)(A.frozen ? r.u : A.u);
    T *fa = (T *)A.faceA, *fw = (T *)A.faceW;
    const T vs = (T)r.vs, kap = (T)r.kappa_c, eps12 = (T)(12.0 / 13.0) * (T)r.eps;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const bool vert = (d == D - 1);
        const bool walls = vert && !r.vper;
        const int j = d == 0 ? x : (d == 1 ? y : z);
        const int n = d == 0 ? r.nx : (d == 1 ? r.ny : r.nz);
        const int64_t stride = d == 0 ? 1 : (d == 1 ? (int64_t)r.nx : (int64_t)r.nx * r.ny);
        const int64_t base = ((int64_t)d * 6) * r.N + k;
        if (walls && j == n - 1) {
#pragma unroll
            for (int s = 0; s < 6; ++s) { fa[base + s * r.N] = (T)0; fw[base + s * r.N] = (T)0; }
            continue;
        }
        T av[6], wv[6];
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            int jj = j + s - 2;
            bool ghost = false;
            if (!walls) jj = wrap_near(jj, n);
            else if (jj < 0) { jj = -1 - jj; ghost = true; }
            else if (jj >= n) { jj = 2 * n - 1 - jj; ghost = true; }
            const int64_t kk = k + (int64_t)(jj - j) * stride;
            av[s] = a[kk];
            T uu = u[(int64_t)d * r.N + kk];
            if (ghost) uu = -uu;
            wv[s] = vert ? uu - vs : uu;
        }
        int jn = j + 1;
        if (jn >= n) jn -= n;   // periodic neighbour (walls never reach here at the top)
        const T pb = scale * (lam[k + (int64_t)(jn - j) * stride] - lam[k]);
        // the stencil read from its upwind end (selects, so that lanes of a
        // wave do not diverge); the node beyond the downwind end gets zeros
        const bool pos = (wv[2] + wv[3]) >= (T)0;
        T a5[5], w5[5], fa5[5], fw5[5];
#pragma unroll
        for (int s = 0; s < 5; ++s) {
            a5[s] = pos ? av[s] : av[5 - s];
            w5[s] = pos ? wv[s] : wv[5 - s];
        }
        face_vjp<T>(a5, w5, pb, pos ? kap : -kap, eps12, fa5, fw5);
#pragma unroll
        for (int s = 0; s < 6; ++s) {
            const T ap = s < 5 ? fa5[s] : (T)0, an = s > 0 ? fa5[5 - s] : (T)0;
            const T wp = s < 5 ? fw5[s] : (T)0, wn = s > 0 ? fw5[5 - s] : (T)0;
            fa[base + s * r.N] = pos ? ap : an;
            fw[base + s * r.N] = pos ? wp : wn;
        }
    }
}

// ---------------------------------------------------------------------------
// 3. streaming, collision and moments in reverse
// ---------------------------------------------------------------------------
// Reverse of streaming, collision and moments at node k given the node's
// total velocity adjoint ub (transport part included); writes fbar and
// returns the adjoint of the force's vertical component.
//
// With f* = f - omega (f - feq(rho, u)) + G(u, F), g_i = w_i fsb_i (fsb the
// adjoint of f*) and its moments M0 = sum g, M1 = sum g c, M2 = sum g c c,
//   sum_i dfeq_i/drho fsb_i = M0 + 3 M1.u + 9/2 u.M2 u - 3/2 u.u M0,
//   sum_i dfeq_i/du   fsb_i = rho V,  V = 3 M1 + 9 M2 u - 3 u M0,
//   sum_i dG_i/dF     fsb_i = guo V,  sum_i dG_i/du fsb_i = guo (9 M2 F - 3 F M0),
// the sums taken over pairs of opposite directions: vector issue bounded the
// stage this ends (2D 536 of its 1072 instructions a node with the terms
// written out per direction).
template <int Q, typename T, bool SH>
__device__ __forceinline__ T collide_reverse_node(const AdjDev &A, int64_t k, int x, int y, int z,
                                                  const T ubt[3]) {
    using L = Lattice<Q>;
    constexpr int D = L::D;
    const RunDev &r = A.r;
    const T *fbn = (const T *)A.fbar_next;
    // the node's neighbours one step down (0) and up (1) each axis, and the
    // walls they lie beyond
    const int64_t nx = r.nx, plane = nx * r.ny;
    const int64_t sx[2] = {x == 0 ? nx - 1 : -1, x == r.nx - 1 ? 1 - nx : 1};
    const int64_t sy[2] = {y == 0 ? plane - nx : -nx, y == r.ny - 1 ? nx - plane : nx};
    const int64_t sz[2] = {z == 0 ? r.N - plane : -plane, z == r.nz - 1 ? plane - r.N : plane};
    const int v = D == 2 ? y : z, nv = D == 2 ? r.ny : r.nz;
    const bool low = !r.vper && v == 0, high = !r.vper && v == nv - 1;
    T fi[Q], fsb[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        // forward streaming sent f*_i(x) to slot i of x + c_i, or to slot
        // opp(i) of x across a wall: pull the adjoint from there (a load of
        // the wrapped node stands in until the wall's own below)
        int64_t n = k;
        if (L::cx[i]) n += sx[L::cx[i] > 0];
        if (L::cy[i]) n += sy[L::cy[i] > 0];
        if (D == 3 && L::cz[i]) n += sz[L::cz[i] > 0];
        fsb[i] = (fbn + (int64_t)i * r.N)[n];
    }
    if (low || high) {
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int cv = D == 2 ? L::cy[i] : L::cz[i];
            if (cv && (cv < 0 ? low : high)) fsb[i] = (fbn + (int64_t)L::opp[i] * r.N)[k];
        }
    }
    T F[3], u[3] = {0, 0, 0}, rho;
    lbm_force<D, T>(r, (const T *)A.c_n, nullptr, k, F);
    if (A.have_rho) {
        // the forward step's own moments (what lbm_rho_u gives from f^n, bit
        // for bit): the populations themselves are not needed
        const T *uu = (const T *)A.u;
#pragma unroll
        for (int d = 0; d < D; ++d) u[d] = uu[(int64_t)d * r.N + k];
        rho = ((const T *)A.rho_n)[k];
    } else {
        const T *f = (const T *)A.f_n;
#pragma unroll
        for (int i = 0; i < Q; ++i) fi[i] = f[(int64_t)i * r.N + k];
        T drho;
        lbm_rho_u<Q, T, SH>(fi, F, rho, drho, u);
    }
    const T omega = (T)r.omega, guo = (T)r.guo;
    T m0 = (T)L::w[0] * fsb[0], m1[3] = {0, 0, 0}, m2[3][3] = {};
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        const int o = L::opp[i];
        if (o < i) continue;
        const int c[3] = {L::cx[i], L::cy[i], L::cz[i]};
        const T w = (T)L::w[i], sum = fsb[i] + fsb[o], dif = fsb[i] - fsb[o];
        m0 += w * sum;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            if (c[d]) m1[d] += (c[d] > 0 ? w : -w) * dif;
#pragma unroll
            for (int e = d; e < D; ++e)
                if (c[d] && c[e]) m2[d][e] += (c[d] * c[e] > 0 ? w : -w) * sum;
        }
    }
    T V[3] = {0, 0, 0}, ub[3] = {0, 0, 0}, Vu = 0, Mu = 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        T Au = 0, AF = 0;
#pragma unroll
        for (int e = 0; e < D; ++e) {
            const T m = d < e ? m2[d][e] : m2[e][d];
            Au += m * u[e];
            AF += m * F[e];
        }
        V[d] = (T)3 * (m1[d] - u[d] * m0) + (T)9 * Au;
        ub[d] = ubt[d] + (omega * rho * V[d] + guo * ((T)9 * AF - (T)3 * F[d] * m0));
        Vu += V[d] * u[d];
        Mu += m1[d] * u[d];
    }
    // u = (m + F/2) / rho, m = sum f c, rho = sum f (+1 when shifted)
    T rb = omega * (m0 + ((T)0.5 * Vu + (T)1.5 * Mu)), mb[3] = {0, 0, 0};
    const T irho = rcp<T>(rho);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        mb[d] = ub[d] * irho;
        rb -= mb[d] * u[d];
    }
    T *fb = (T *)A.fbar;
#pragma unroll
    for (int i = 0; i < Q; ++i)
        (fb + (int64_t)i * r.N)[k] = ((T)1 - omega) * fsb[i] + (rb + cdot<Q>(i, mb[0], mb[1], mb[2]));
    return guo * V[D - 1] + (T)0.5 * mb[D - 1];
}

// ---------------------------------------------------------------------------
// gather of the transport transpose (the last reversed stage also reverses
// the collision at the node)
// ---------------------------------------------------------------------------
// Node-wise gather of the face products.  STAGE selects the RK stage being
// reversed (3, 2, 1 in that order) and how the result combines.
// The per-node end of a reversed RK stage, given the node's gathered face
// products (abar, the velocity parts ubs and the settling part vsp): the
// absorbing bottom face, the deposit update, the RK combination and, after the
// last stage, the collision and moments in reverse.  With A_s the transpose of L
// in stage s, the stage adjoints are a2b = 2/3 cbn + A_3 and a1b = 1/4 a2b + A_2,
// and cbar = 1/3 cbn + 3/4 a2b + a1b + A_1 = cbn + (A_3 + A_2 + A_1): summed in
// the last form, the small terms first (cbar holds them between the stages), so
// that a step rounds a value of cbar's size once, and thirds and quarters of it
// need not add up again (single precision, error of the gradient against 64
// bits, mean of four seeds: 512x1024 over 100 steps 8.3e-7 -> 5.3e-7, 64x48x96
// over 20 steps 5.0e-7 -> 3.0e-7).
template <int Q, typename T, bool SH, int STAGE>
__device__ __forceinline__ void gather_finish(const AdjDev &A, int64_t k, int x, int y, int z, T abar,
                                              const T ubs[3], double vsp) {
    constexpr int D = Lattice<Q>::D;
    const RunDev &r = A.r;
    T *ub = (T *)A.ubar;
    // bottom wall face: L_0 contains -vs a_0
    const int v = (D == 2) ? y : z;
    const bool bottom = !r.vper && v == 0;
    const T *lam_in;
    T lam_scale;
    const T *a_fwd;
    if constexpr (STAGE == 3) { lam_in = (const T *)A.cbar_next; lam_scale = (T)(2.0 / 3.0); a_fwd = (const T *)A.a2; }
    else if constexpr (STAGE == 2) { lam_in = (const T *)A.abar2; lam_scale = (T)0.25; a_fwd = (const T *)A.a1; }
    else { lam_in = (const T *)A.abar1; lam_scale = (T)1; a_fwd = (const T *)A.c_n; }
    const T lam = lam_scale * lam_in[k];
    if (bottom) {
        abar += -(T)r.vs * lam;
        vsp += -(double)a_fwd[k] * (double)lam;
    }
    const double db = A.dep_bar;
    const T *cbn = (const T *)A.cbar_next;
    T *cb = (T *)A.cbar;
    if constexpr (STAGE == 3) {
        T da = abar, dc = abar;
        if (bottom) {
            // D+ = D + vs (C/6 + a1/6 + 2 a2/3)
            da += (T)(2.0 / 3.0 * r.vs * db);
            dc += (T)(5.0 / 6.0 * r.vs * db);
            vsp += db * ((double)((const T *)A.c_n)[k] / 6.0 + (double)((const T *)A.a1)[k] / 6.0 +
                         2.0 / 3.0 * (double)((const T *)A.a2)[k]);
        }
        ((T *)A.abar2)[k] = (T)(2.0 / 3.0) * cbn[k] + da;
        cb[k] = dc;               // cbar - cbn so far
#pragma unroll
        for (int d = 0; d < D; ++d) ub[(int64_t)d * r.N + k] = ubs[d];
        A.vs_part[k] += vsp;      // accumulates across steps until summed
    } else if constexpr (STAGE == 2) {
        if (bottom) abar += (T)(r.vs / 6.0 * db);
        ((T *)A.abar1)[k] = (T)0.25 * ((const T *)A.abar2)[k] + abar;
        cb[k] += abar;
#pragma unroll
        for (int d = 0; d < D; ++d) ub[(int64_t)d * r.N + k] += ubs[d];
        A.vs_part[k] += vsp;
    } else {
        // every load of the node before the collision's stores, past which the
        // compiler may not move them (double precision, us: 64x60x90 42.8 -> 41.2,
        // 512x1024 30.7 -> 30.0)
        T dc = cb[k] + abar;
        const T c0 = cbn[k];
        A.vs_part[k] += vsp;
        if (!A.frozen) {
            // last stage reversed: the node's velocity adjoint is complete, so
            // the collision and moments are reversed here as well
            T ut[3] = {0, 0, 0};
#pragma unroll
            for (int d = 0; d < D; ++d) ut[d] = ub[(int64_t)d * r.N + k] + ubs[d];
            dc -= (T)r.gp_c * collide_reverse_node<Q, T, SH>(A, k, x, y, z, ut);
        }
        cb[k] = c0 + dc;
    }
}

template <int Q, typename T, bool SH, int STAGE>
__global__ void __launch_bounds__(256) k_adj_gather(AdjDev A) {
    constexpr int D = Lattice<Q>::D;
    const RunDev &r = A.r;
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= r.N) return;
    int x, y, z;
    xyz<D>(r, k, x, y, z);
    const T *fa = (const T *)A.faceA, *fw = (const T *)A.faceW;
    double vsp = 0.0;
    T abar = 0;
    T ubs[3] = {0, 0, 0};
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const bool vert = (d == D - 1);
        const bool walls = vert && !r.vper;
        const int m = d == 0 ? x : (d == 1 ? y : z);
        const int n = d == 0 ? r.nx : (d == 1 ? r.ny : r.nz);
        const int64_t stride = d == 0 ? 1 : (d == 1 ? (int64_t)r.nx : (int64_t)r.nx * r.ny);
        // images of node m as seen by stencils: itself, and beyond each wall
        // (only rows m <= 1 and m >= n - 2 have images that a face reads)
        const int nimg = (walls && (m <= 1 || m >= n - 2)) ? 3 : 1;
        for (int im = 0; im < nimg; ++im) {
            const int p = im == 0 ? m : (im == 1 ? -1 - m : 2 * n - 1 - m);
            const bool ghost = im != 0;
#pragma unroll
            for (int s = 0; s < 6; ++s) {
                int jf = p - s + 2;              // face whose slot s reads position p
                if (walls) {
                    if (jf < 0 || jf > n - 2) continue;
                } else {
                    jf = wrap_near(jf, n);
                }
                const int64_t kf = k + (int64_t)(jf - m) * stride;
                const int64_t idx = ((int64_t)d * 6 + s) * r.N + kf;
                abar += fa[idx];
                const T wb = fw[idx];
                if (vert) {
                    ubs[d] += ghost ? -wb : wb;
                    vsp -= (double)wb;
                } else {
                    ubs[d] += wb;
                }
            }
        }
    }
    gather_finish<Q, T, SH, STAGE>(A, k, x, y, z, abar, ubs, vsp);
}

// ---------------------------------------------------------------------------
// One reversed RK stage in one kernel.  A block owns a TX x TY x TZ tile of
// nodes (2D: TZ = 1) and takes the axes one after the other: it stages the
// stage input, the axis' transport velocity and the face adjoints lam of the
// tile's lines with the halo the line's face stencils reach (wall images
// already mirrored, with the sign of the vertical velocity flipped), evaluates
// every face the tile's nodes read (five beyond the tile on each line) and
// gathers the products per node.  Faces are evaluated with the same face_vjp
// on the same values as the two-kernel form and gathered in the same order, so
// the results are identical bit for bit; the workspace round trip of the face
// products (6 D values of A and of W per node, written and read) disappears,
// at the price of the faces neighbouring tiles also evaluate.
//
// Vector issue takes more than half of it (2D 512x1024 in single precision: 513
// vector instructions per node, 7 of a stage's 12 us; 790 and 15.5 with the
// upwind side chosen by selects and per-lane positions; 3D 64x48x96 1045, 8.5 of
// 15), the rest is the loads before the first of its barriers (eight, in 3D
// twelve) and the end of a launch of one round of blocks, so tiles are as large as
// occupancy allows (2D 64x8 evaluates 2.7 faces per node, 3D 16x4x4 5.8), a
// stencil's upwind side is an address, a wave stages one position of 64 lines
// (its place on the axis, wrap and mirror are scalar work), and faces beyond a
// wall hold zeros so that a node adds its six products unchecked.  All the
// tile's loads are in flight before the first is stored to LDS; LDS holds one
// axis at a time, and of its products first A, then W (kept in registers
// meanwhile), so that a CU holds 32 waves (2D) and 20 to 24 (3D) in single
// precision, 16 and 12 in double (both at once: 2D 0.4% faster, 3D 4% slower).
// us per reverse step: 2D 512x1024 61.5 -> 41 (against 32x8 tiles with the whole
// set of products in LDS); 3D 64x48x96 81 -> 48 (against the two-kernel form).
// ---------------------------------------------------------------------------

// Stored position of j on a periodic axis, for the at most five cells a line's
// halo reaches below it and any number above; positions past its fifth cell
// beyond, which no node of the grid reads, are clamped there.
__device__ __forceinline__ int wrap_halo(int j, int n) {
    j = min(j, n + 4);
    if (n < 5) j %= n;
    j += j < 0 ? n : 0;
    return j - (j >= n ? n : 0);
}

template <int TX, int TY, int TZ, int D> struct AdjTile {
    static constexpr int NODES = TX * TY * TZ;
    static constexpr int extent(int ax) { return ax == 0 ? TX : (ax == 1 ? TY : TZ); }
    static constexpr int lines(int ax) { return NODES / extent(ax); }
    static constexpr int most(int a, int b) { return a > b ? a : b; }
    // faces of an axis, and values staged for it: a, w and lam on extent + 10
    // positions of every line
    static constexpr int faces(int ax) { return (extent(ax) + 5) * lines(ax); }
    static constexpr int staged(int ax) { return 3 * (extent(ax) + 10) * lines(ax); }
    static constexpr int max_faces = most(faces(0), most(faces(1), D == 3 ? faces(2) : 0));
    static constexpr int max_staged = most(staged(0), most(staged(1), D == 3 ? staged(2) : 0));
};

template <int Q, typename T, bool SH, int STAGE, int TX, int TY, int TZ, int NT, int WAVES_PER_SIMD>
__global__ void __launch_bounds__(NT, WAVES_PER_SIMD) k_adj_stage(AdjDev A, const T *__restrict__ a,
                                                          const T *__restrict__ lam, T scale) {
    constexpr int D = Lattice<Q>::D;
    using G = AdjTile<TX, TY, TZ, D>;
    constexpr int PER = G::NODES / NT, NP = G::max_faces;
    static_assert(G::NODES % NT == 0, "tile must be a multiple of the block");
    __shared__ T sS[G::max_staged], sP[6 * NP];

    const RunDev &r = A.r;
    const int nx = r.nx, ny = r.ny, nz = D == 3 ? r.nz : 1;
    const int gx = (nx + TX - 1) / TX, gy = (ny + TY - 1) / TY;
    const int tile = xcd_order((int)blockIdx.x, (int)gridDim.x);
    const int x0 = tile % gx * TX, y0 = tile / gx % gy * TY, z0 = D == 3 ? tile / gx / gy * TZ : 0;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int WAVES = NT / 64, E = (int)sizeof(T);
    const bool walls = !r.vper;
    const T *u = (const T *)(A.frozen ? r.u : A.u);
    const T vs = (T)r.vs, kap = (T)r.kappa_c, eps12 = (T)(12.0 / 13.0) * (T)r.eps;
    const int64_t plane = (int64_t)nx * ny;

    auto vertical = [](auto ax) { return decltype(ax)::value == D - 1; };
    auto origin = [&](auto ax) { return decltype(ax)::value == 0 ? x0 : (decltype(ax)::value == 1 ? y0 : z0); };
    auto length = [&](auto ax) { return decltype(ax)::value == 0 ? nx : (decltype(ax)::value == 1 ? ny : nz); };

    // Position c of line `line` that this thread stages in round q.  Lines of y
    // and z are 64, one per lane, so a wave stages one position of each and
    // its place on the axis is uniform; a line of x is a row, taken by a wave
    // where it is as wide as one, else the rows are dealt flat.
    static_assert(G::lines(1) == 64 && (D == 2 || G::lines(2) == 64), "a lane per line of y and z");
    constexpr bool ROWS = TX == 64 && TY * TZ == WAVES;
    auto place = [&](auto ax, int q, int &line, int &c) {
        constexpr int AX = decltype(ax)::value, HL = G::extent(AX) + 10;
        if constexpr (AX > 0) { line = lane; c = wave + q * WAVES; }
        else if constexpr (ROWS) { line = wave; c = lane + q * 64; }
        else { line = (tid + q * NT) / HL; c = (tid + q * NT) % HL; }
    };
    constexpr int XR = ROWS ? (TX + 10 + 63) / 64 : ((TX + 10) * G::lines(0) + NT - 1) / NT;
    constexpr int YR = (TY + 10 + WAVES - 1) / WAVES, ZR = D == 3 ? (TZ + 10 + WAVES - 1) / WAVES : 1;
    // load an axis' values into registers, unconditionally (a spare slot
    // repeats the last position).  One address serves a, w and lam; positions
    // beyond a wall are mirrored (rows no face of the tile reads are clamped
    // into range), those of a periodic axis wrap
    const int lx = min(x0 + (D == 2 ? lane : lane % TX), nx - 1);
    auto load = [&](auto ax, T *pa, T *pw, T *pl) {
        constexpr int AX = decltype(ax)::value, HL = G::extent(AX) + 10;
        constexpr int R = AX == 0 ? XR : (AX == 1 ? YR : ZR);
        const int o = origin(ax), n = length(ax);
        const T *ud = u + (int64_t)AX * r.N;
        // lane's part of the node index, for lines of y and z
        const int64_t across = D == 2 || AX == 0 ? lx
                               : AX == 1 ? lx + plane * min(lane / TX, nz - 1 - z0)
                                         : lx + (int64_t)nx * min(y0 + lane / TX, ny - 1);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            int line, c;
            place(ax, q, line, c);
            int p = o - 5 + min(c, HL - 1);
            bool ghost = false;
            if (vertical(ax) && walls) {
                if (p < 0) { p = -1 - p; ghost = true; }
                else if (p >= n) { p = 2 * n - 1 - p; ghost = true; }
                p = min(max(p, 0), n - 1);
            } else {
                p = wrap_halo(p, n);
            }
            int64_t row, in;                               // uniform part, lane's part
            if constexpr (AX == 0 && ROWS) {
                row = (int64_t)nx * min(y0 + line, ny - 1);
                in = p;
            } else if constexpr (AX == 0) {
                row = 0;
                in = p + (int64_t)nx * min(y0 + line % TY, ny - 1) + plane * min(z0 + line / TY, nz - 1);
            } else if constexpr (AX == 1) {
                row = (int64_t)nx * p + (D == 3 ? plane * z0 : 0);
                in = across;
            } else {
                row = plane * p;
                in = across;
            }
            T w;
            if constexpr (D == 2 || AX == 2) {             // within a row or plane: 32-bit byte offsets
                const uint32_t off = (uint32_t)in * E;
                pa[q] = *(const T *)((const char *)(a + row) + off);
                w = *(const T *)((const char *)(ud + row) + off);
                pl[q] = *(const T *)((const char *)(lam + row) + off);
            } else {
                pa[q] = a[row + in];
                w = ud[row + in];
                pl[q] = lam[row + in];
            }
            pw[q] = vertical(ax) ? (ghost ? -w : w) - vs : w;
        }
    };
    auto publish = [&](auto ax, const T *pa, const T *pw, const T *pl) {
        constexpr int AX = decltype(ax)::value, NL = G::lines(AX), HL = G::extent(AX) + 10, NH = HL * NL;
        constexpr int R = AX == 0 ? XR : (AX == 1 ? YR : ZR);
#pragma unroll
        for (int q = 0; q < R; ++q) {
            int line, c;
            place(ax, q, line, c);
            if (AX == 0 ? (c < HL && line < NL) : c < HL) {
                const int i = AX == 0 ? line * HL + c : c * NL + line;
                sS[i] = pa[q];
                sS[NH + i] = pw[q];
                sS[2 * NH + i] = pl[q];
            }
        }
    };

    T abar[PER], ubs[PER][3];
    double vsp[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        abar[e] = 0;
        ubs[e][0] = ubs[e][1] = ubs[e][2] = 0;
        vsp[e] = 0.0;
    }
    auto coords_of = [&](int e, int &lx, int &ly, int &lz) {
        const int node = tid + e * NT;
        lx = node % TX;
        ly = node / TX % TY;
        lz = node / (TX * TY);
    };
    // nodes of the grid only: for a row beyond the top of a ragged tile the
    // image above the wall could name a face outside the tile's range.  For a
    // grid node every face it reads lies in [o - 3, o + extent + 1]: its own
    // faces m - 3 .. m + 2, the bottom images (faces 0, 1, read only when
    // m <= 1, so o = 0) and the top images (faces >= n - 3 >= m - 2, read only
    // when m >= n - 3)
    auto in_grid = [&](int lx, int ly, int lz) { return x0 + lx < nx && y0 + ly < ny && z0 + lz < nz; };

    // the faces of one axis and their gather; `then` runs once the staged
    // values are used up (the next axis' values take their place)
    auto sweep = [&](auto ax, auto &&then) {
        constexpr int AX = decltype(ax)::value, TD = G::extent(AX), NL = G::lines(AX), HL = TD + 10,
                      NF = TD + 5, NH = HL * NL, ROUNDS = (NF * NL + NT - 1) / NT;
        constexpr int SI = AX == 0 ? 1 : NL;                  // stride between positions of a line
        const int o = origin(ax), n = length(ax);
        const bool wall_ax = vertical(ax) && walls;
        // each face reads its stencil from the upwind end and stores its
        // products in that order by address: slot s of face f at byte
        // at0 + s at1 (slot 5, the node beyond the downwind end, is zero)
        T fw[ROUNDS][5];
        uint32_t at0[ROUNDS], at1[ROUNDS];
        bool live[ROUNDS];
        auto S = [&](uint32_t off, int c) { return *(const T *)((const char *)sS + off + c * E); };
        auto P = [&](uint32_t off) -> T & { return *(T *)((char *)sP + off); };
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            const int f = tid + q * NT;
            const int line = AX == 0 ? f / NF : lane, i = AX == 0 ? f % NF : wave + q * WAVES;
            const int j = o - 3 + i;
            live[q] = false;
            if (AX == 0 ? f >= NF * NL : i >= NF) continue;
            if (wall_ax && (j < 0 || j > n - 2)) {            // no such face: adds nothing to a node
#pragma unroll
                for (int s = 0; s < 6; ++s) sP[s * NP + f] = (T)0;
                continue;
            }
            live[q] = true;
            const uint32_t base = (uint32_t)(AX == 0 ? line * HL + i : i * NL + line) * E;
            const bool pos = (S(base, NH + 2 * SI) + S(base, NH + 3 * SI)) >= (T)0;
            const T pb = scale * (S(base, 2 * NH + 3 * SI) - S(base, 2 * NH + 2 * SI));
            const uint32_t step = pos ? (uint32_t)(SI * E) : (uint32_t)(-SI * E);
            uint32_t nd = pos ? base : base + 5 * SI * E;
            T a5[5], w5[5], fa[5];
#pragma unroll
            for (int s = 0; s < 5; ++s, nd += step) {
                a5[s] = S(nd, 0);
                w5[s] = S(nd, NH);
            }
            face_vjp<T>(a5, w5, pb, pos ? kap : -kap, eps12, fa, fw[q]);
            at0[q] = (uint32_t)f * E + (pos ? 0u : (uint32_t)(5 * NP * E));
            at1[q] = pos ? (uint32_t)(NP * E) : (uint32_t)(-NP * E);
            uint32_t to = at0[q];
#pragma unroll
            for (int s = 0; s < 5; ++s, to += at1[q]) P(to) = fa[s];
            P(to) = (T)0;
        }
        __syncthreads();
        // wall images reach only rows m <= 1 (the image -1 - m feeds faces 0
        // and 1) and m >= n - 2 (the image 2 n - 1 - m feeds faces n - 3 and
        // n - 2); tiles clear of both take the node itself only (the same sum:
        // the skipped images add nothing)
        const bool images = wall_ax && (o < 2 || o + TD > n - 2);
        auto gather = [&](auto &&add) {
#pragma unroll
            for (int e = 0; e < PER; ++e) {
                int lx, ly, lz;
                coords_of(e, lx, ly, lz);
                if (!in_grid(lx, ly, lz)) continue;
                const int l = AX == 0 ? lx : (AX == 1 ? ly : lz), m = o + l;
                const int line = AX == 0 ? ly + TY * lz : (AX == 1 ? lx + TX * lz : lx + TX * ly);
#pragma unroll
                for (int s = 0; s < 6; ++s) {                 // face m - s + 2 reads the node in slot s
                    const int i = l - s + 5;
                    add(e, false, sP[s * NP + (AX == 0 ? line * NF + i : i * NL + line)]);
                }
                if (!images) continue;
                for (int im = 1; im < 3; ++im) {
                    const int p = im == 1 ? -1 - m : 2 * n - 1 - m;
#pragma unroll
                    for (int s = 0; s < 6; ++s) {
                        const int jf = p - s + 2;             // face whose slot s reads position p
                        if (jf < 0 || jf > n - 2) continue;
                        const int i = jf - (o - 3);
                        add(e, true, sP[s * NP + (AX == 0 ? line * NF + i : i * NL + line)]);
                    }
                }
            }
        };
        gather([&](int e, bool, T p) { abar[e] += p; });
        then();
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ROUNDS; ++q) {
            if (!live[q]) continue;
            uint32_t to = at0[q];
#pragma unroll
            for (int s = 0; s < 5; ++s, to += at1[q]) P(to) = fw[q][s];
        }
        __syncthreads();
        gather([&](int e, bool ghost, T p) {
            if constexpr (AX == D - 1) {
                ubs[e][AX] += ghost ? -p : p;
                vsp[e] -= (double)p;
            } else {
                ubs[e][AX] += p;
            }
        });
    };

    using std::integral_constant;
    constexpr integral_constant<int, 0> X{};
    constexpr integral_constant<int, 1> Y{};
    constexpr integral_constant<int, 2> Z{};
    T ax_a[XR], ax_w[XR], ax_l[XR], ay_a[YR], ay_w[YR], ay_l[YR], az_a[ZR], az_w[ZR], az_l[ZR];
    load(X, ax_a, ax_w, ax_l);
    load(Y, ay_a, ay_w, ay_l);
    if constexpr (D == 3) load(Z, az_a, az_w, az_l);
    publish(X, ax_a, ax_w, ax_l);
    __syncthreads();
    sweep(X, [&] { publish(Y, ay_a, ay_w, ay_l); });
    __syncthreads();
    if constexpr (D == 3) {
        sweep(Y, [&] { publish(Z, az_a, az_w, az_l); });
        __syncthreads();
        sweep(Z, [] {});
    } else {
        sweep(Y, [] {});
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        int lx, ly, lz;
        coords_of(e, lx, ly, lz);
        if (!in_grid(lx, ly, lz)) continue;
        const int x = x0 + lx, y = y0 + ly, z = z0 + lz;
        const int64_t k = D == 2 ? (int64_t)x + (int64_t)nx * y : (int64_t)(x + nx * y) + plane * z;
        gather_finish<Q, T, SH, STAGE>(A, k, x, y, z, abar[e], ubs[e], vsp[e]);
    }
}

// ---------------------------------------------------------------------------
// dJ/dVs: fixed-order FP64 sum of the per-node parts, added to *vs_bar
// ---------------------------------------------------------------------------
__device__ __forceinline__ double block_sum_adj(double acc) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    __shared__ double waves[16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) waves[wid] = acc;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)((blockDim.x + 63) >> 6); ++i) t += waves[i];
    return t;
}

__global__ void __launch_bounds__(256) k_adj_vs_partial(double *__restrict__ part, int64_t n,
                                                        double *__restrict__ out) {
    double acc = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
        acc += part[k];
        part[k] = 0.0;            // the accumulator starts over
    }
    const double t = block_sum_adj(acc);
    if (threadIdx.x == 0) out[blockIdx.x] = t;
}

__global__ void __launch_bounds__(256) k_adj_vs_final(const double *__restrict__ part, int n,
                                                      double *__restrict__ vs_bar) {
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) acc += part[i];
    const double t = block_sum_adj(acc);
    if (threadIdx.x == 0) *vs_bar += t;
}

template <int Q, typename T, bool SH>
hipError_t adjoint_t(const AdjDev &A, const lbw_launch &l, hipStream_t st) {
    constexpr int D = Lattice<Q>::D;
    const int block = 256;
    const dim3 grid((unsigned)((A.r.N + block - 1) / block));
    if (!A.frozen && !A.have_u) k_adj_moments<Q, T, SH><<<grid, block, 0, st>>>(A);
    hipError_t e = hipSuccess;
    if (!A.have_stages) {
        // forward stages 1 and 2 from the saved C^n and u^n, with the same
        // tiled kernels as the forward step (a1, a2 are its own values)
        RunDev fr = A.r;
        fr.c = const_cast<void *>(A.c_n);
        fr.c1 = A.a1;
        fr.c2 = A.a2;
        fr.u = A.frozen ? A.r.u : A.u;
        const int prec = sizeof(T) == 4 ? LBW_FP32_SHIFTED : LBW_FP64;
        lbw_launch lt = l;
        lt.variant = 0;
        e = launch_one_stage(D, prec, fr, lt, 1, st);
        if (e == hipSuccess) e = launch_one_stage(D, prec, fr, lt, 2, st);
        if (e != hipSuccess) return e;
    }
    // one kernel per reversed stage, unless its launch would need 2^32
    // work-items (then, and with variant 1, the two-kernel form: the same sums
    // in the same order, the same bits)
    constexpr bool f32 = sizeof(T) == 4;
    constexpr int TX = D == 2 ? 64 : 16, TY = D == 2 ? 8 : 4, TZ = D == 2 ? 1 : 4;
    constexpr int NT = D == 2 ? 512 : 256, WPS = D == 2 ? 4 : (f32 ? 5 : 3);
    const int64_t tiles = (int64_t)((A.r.nx + TX - 1) / TX) * ((A.r.ny + TY - 1) / TY) *
                          (D == 3 ? (A.r.nz + TZ - 1) / TZ : 1);
    if (l.variant != 1 && tiles * NT < ((int64_t)1 << 32)) {
        const dim3 tg((unsigned)tiles);
        k_adj_stage<Q, T, SH, 3, TX, TY, TZ, NT, WPS><<<tg, NT, 0, st>>>(A, (const T *)A.a2, (const T *)A.cbar_next, (T)(2.0 / 3.0));
        k_adj_stage<Q, T, SH, 2, TX, TY, TZ, NT, WPS><<<tg, NT, 0, st>>>(A, (const T *)A.a1, (const T *)A.abar2, (T)0.25);
        k_adj_stage<Q, T, SH, 1, TX, TY, TZ, NT, WPS><<<tg, NT, 0, st>>>(A, (const T *)A.c_n, (const T *)A.abar1, (T)1);
    } else {
        k_adj_face<T, D><<<grid, block, 0, st>>>(A, (const T *)A.a2, (const T *)A.cbar_next, (T)(2.0 / 3.0));
        k_adj_gather<Q, T, SH, 3><<<grid, block, 0, st>>>(A);
        k_adj_face<T, D><<<grid, block, 0, st>>>(A, (const T *)A.a1, (const T *)A.abar2, (T)0.25);
        k_adj_gather<Q, T, SH, 2><<<grid, block, 0, st>>>(A);
        k_adj_face<T, D><<<grid, block, 0, st>>>(A, (const T *)A.c_n, (const T *)A.abar1, (T)1);
        k_adj_gather<Q, T, SH, 1><<<grid, block, 0, st>>>(A);
    }
    if (A.vs_bar) {
        k_adj_vs_partial<<<kReduceBlocks, 256, 0, st>>>(A.vs_part, A.r.N, A.partials);
        k_adj_vs_final<<<1, 256, 0, st>>>(A.partials, kReduceBlocks, A.vs_bar);
    }
    return hipGetLastError();
}

}  // namespace

size_t adjoint_work_bytes(int dim, int precision, int64_t N) {
    const size_t es = precision == LBW_FP32_SHIFTED ? 4 : 8;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    size_t b = 0;
    b += al(es * dim * N);          // u
    b += 4 * al(es * N);            // a1, a2, abar1, abar2
    b += al(es * dim * N);          // ubar
    b += 2 * al(es * 6 * dim * N);  // face products
    b += al(sizeof(double) * N);    // vs parts
    b += al(sizeof(double) * kReduceBlocks);
    return b;
}

hipError_t launch_adjoint(int q, int precision, const RunDev &r, bool frozen, const void *f_n,
                          const void *c_n, const void *u_n, const void *rho_n, const void *a1_n,
                          const void *a2_n,
                          const void *fbar_next, const void *cbar_next,
                          double dep_bar, void *fbar, void *cbar, double *vs_bar, void *work,
                          const lbw_launch &l, hipStream_t st) {
    const int dim = q == 9 ? 2 : 3;
    const size_t es = precision == LBW_FP32_SHIFTED ? 4 : 8;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    char *w = (char *)work;
    AdjDev A;
    A.r = r;
    A.f_n = f_n;
    A.c_n = c_n;
    A.rho_n = rho_n;
    A.fbar_next = fbar_next;
    A.cbar_next = cbar_next;
    A.fbar = fbar;
    A.cbar = cbar;
    A.u = w; w += al(es * dim * r.N);
    A.a1 = w; w += al(es * r.N);
    A.a2 = w; w += al(es * r.N);
    A.abar1 = w; w += al(es * r.N);
    A.abar2 = w; w += al(es * r.N);
    A.ubar = w; w += al(es * dim * r.N);
    A.faceA = w; w += al(es * 6 * dim * r.N);
    A.faceW = w; w += al(es * 6 * dim * r.N);
    A.vs_part = (double *)w; w += al(sizeof(double) * r.N);
    A.partials = (double *)w;
    A.vs_bar = vs_bar;
    A.dep_bar = dep_bar;
    A.frozen = frozen ? 1 : 0;
    A.have_u = (u_n != nullptr && !frozen) ? 1 : 0;
    A.have_rho = (A.have_u && rho_n != nullptr) ? 1 : 0;
    A.have_stages = (a1_n != nullptr && a2_n != nullptr) ? 1 : 0;
    if (A.have_u) A.u = const_cast<void *>(u_n);
    if (A.have_stages) {
        A.a1 = const_cast<void *>(a1_n);
        A.a2 = const_cast<void *>(a2_n);
    }
    switch (precision) {
        case LBW_FP64: return q == 9 ? adjoint_t<9, double, false>(A, l, st) : adjoint_t<19, double, false>(A, l, st);
        case LBW_FP64_SHIFTED: return q == 9 ? adjoint_t<9, double, true>(A, l, st) : adjoint_t<19, double, true>(A, l, st);
        case LBW_FP32_SHIFTED: return q == 9 ? adjoint_t<9, float, true>(A, l, st) : adjoint_t<19, float, true>(A, l, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace lbw
