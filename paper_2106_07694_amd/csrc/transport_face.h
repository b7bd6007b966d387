// transport_face.h -- face fluxes of the fast transport kernels (the tiled
// RK3 stages and the fused 2D step): WENO reconstruction with one reciprocal,
// first-order S faces, and the node-shared form of the vertical faces.
//
// Every kernel that inlines these must give the same bits for the same
// values (a batch equals its runs alone, a fused step equals three stage
// launches), so multiply-adds are fused only within one source expression
// from here to the end of the including unit: the default fast contraction
// may also fuse across statements, differently in each kernel.
#pragma once

#include "transport_device.h"

#pragma clang fp contract(on)

namespace lbw {
namespace {

template <typename T> __device__ __forceinline__ T fast_rcp(T x) { return (T)1 / x; }
template <> __device__ __forceinline__ float fast_rcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }

// WENO5-JS face value (the formula of weno5_face) rearranged for issue
// count, with one reciprocal.  The normalised weights are ratios, so every
// indicator may be scaled by one constant and every ideal weight by another:
// with e_k = (12/13)(eps + beta_k) = t_k^2 + (3/13) s_k^2 + (12/13) eps
// (t_k the second difference, s_k the one-sided first difference of
// sub-stencil k, both built from the four first differences) and the
// weights multiplied through by 10 e_0^2 e_1^2 e_2^2, the face value is
//   (P q_0 + Q q_1' + R q_2') / (P + 6 Q + 3 R),
//   P = e_1^2 e_2^2, Q = e_0^2 e_2^2, R = e_0^2 e_1^2,
// where q_0 is the first candidate and q_1' = 6 q_1, q_2' = 3 q_2.
// eps12 is (12/13) eps.  With e_k >= eps12 and concentrations of order one
// every product stays far inside the single-precision range.
template <typename T>
__device__ __forceinline__ T weno5_rcp(T h0, T h1, T h2, T h3, T h4, T a0, T a1, T a2, T a3, T a4,
                                       T eps12) {
    const T g0 = a1 - a0, g1 = a2 - a1, g2 = a3 - a2, g3 = a4 - a3;
    const T t0 = g1 - g0, t1 = g2 - g1, t2 = g3 - g2;
    const T s0 = t0 + (T)2 * g1;          // a0 - 4 a1 + 3 a2
    const T s1 = g1 + g2;                 // a3 - a1
    const T s2 = t2 - (T)2 * g2;          // 3 a2 - 4 a3 + a4
    constexpr T k = (T)(3.0 / 13.0);
    const T e0 = t0 * t0 + (k * s0 * s0 + eps12);
    const T e1 = t1 * t1 + (k * s1 * s1 + eps12);
    const T e2 = t2 * t2 + (k * s2 * s2 + eps12);
    const T S0 = e0 * e0, S1 = e1 * e1, S2 = e2 * e2;
    const T P = S1 * S2, Q = S0 * S2, R = S0 * S1;
    const T q0 = (T)(1.0 / 3.0) * h0 - (T)(7.0 / 6.0) * h1 + (T)(11.0 / 6.0) * h2;
    const T q1 = (T)5 * h2 - h1 + (T)2 * h3;
    const T q2 = h2 + (T)2.5 * h3 - (T)0.5 * h4;
    return (P * q0 + Q * q1 + R * q2) * fast_rcp<T>(P + (T)6 * Q + (T)3 * R);
}

template <typename T>
__device__ __forceinline__ T weno3_rcp(T h0, T h1, T h2, T a0, T a1, T a2, T eps) {
    const T qu = (T)0.5 * ((T)3 * h1 - h0);
    const T qc = (T)0.5 * (h1 + h2);
    const T eu = eps + (a1 - a0) * (a1 - a0);
    const T ec = eps + (a2 - a1) * (a2 - a1);
    const T au = (T)(1.0 / 3.0) * fast_rcp<T>(eu * eu);
    const T ac = (T)(2.0 / 3.0) * fast_rcp<T>(ec * ec);
    return (au * qu + ac * qc) * fast_rcp<T>(au + ac);
}

// Face flux from six nodes j-2..j+3 (a and w given as separate scalars):
// the upwind side is chosen by selects, not branches, so lanes of a wave
// with different face-velocity signs do not diverge.
template <typename T, int SCHEME>
__device__ __forceinline__ T face6(T a0, T a1, T a2, T a3, T a4, T a5, T w0, T w1, T w2, T w3,
                                   T w4, T w5, T kappa, T eps) {
    const bool pos = (w2 + w3) >= (T)0;
    T hh;
    if constexpr (SCHEME == LBW_WENO5) {
        const T A0 = pos ? a0 : a5, A1 = pos ? a1 : a4, A2 = pos ? a2 : a3, A3 = pos ? a3 : a2,
                A4 = pos ? a4 : a1;
        const T W0 = pos ? w0 : w5, W1 = pos ? w1 : w4, W2 = pos ? w2 : w3, W3 = pos ? w3 : w2,
                W4 = pos ? w4 : w1;
        hh = weno5_rcp<T>(W0 * A0, W1 * A1, W2 * A2, W3 * A3, W4 * A4, A0, A1, A2, A3, A4,
                          (T)(12.0 / 13.0) * eps);
    } else if constexpr (SCHEME == LBW_WENO3) {
        const T A0 = pos ? a1 : a4, A1 = pos ? a2 : a3, A2 = pos ? a3 : a2;
        const T W0 = pos ? w1 : w4, W1 = pos ? w2 : w3, W2 = pos ? w3 : w2;
        hh = weno3_rcp<T>(W0 * A0, W1 * A1, W2 * A2, A0, A1, A2, eps);
    } else {
        hh = pos ? w2 * a2 : w3 * a3;
    }
    return hh - kappa * (a3 - a2);
}

// face6 of six nodes in LDS, S elements apart, a at byte offset base + CA and w
// at base + CW: the upwind side is chosen by the address the stencil is read
// from (node j-2 upwards or j+3 downwards), which costs one select and an add
// per node where selecting among loaded values costs two selects (four in
// double precision); a and w of a node share the address.
template <typename T, int SCHEME, int S, int CA, int CW>
__device__ __forceinline__ T face6_lds(const T *smem, uint32_t base, T kappa, T eps) {
    constexpr int E = (int)sizeof(T);
    auto at = [&](uint32_t off, int c) { return *(const T *)((const char *)smem + off + c); };
    const bool pos = (at(base, CW + 2 * S * E) + at(base, CW + 3 * S * E)) >= (T)0;
    const uint32_t n0 = base + (pos ? 0u : (uint32_t)(5 * S * E)), step = pos ? (uint32_t)(S * E) : (uint32_t)(-S * E);
    const uint32_t n1 = n0 + step, n2 = n1 + step, n3 = n2 + step, n4 = n3 + step;
    const T a2 = at(n2, CA), a3 = at(n3, CA), kd = pos ? kappa : -kappa;
    T hh;
    if constexpr (SCHEME == LBW_WENO5) {
        const T a0 = at(n0, CA), a1 = at(n1, CA), a4 = at(n4, CA);
        hh = weno5_rcp<T>(at(n0, CW) * a0, at(n1, CW) * a1, at(n2, CW) * a2, at(n3, CW) * a3, at(n4, CW) * a4,
                          a0, a1, a2, a3, a4, (T)(12.0 / 13.0) * eps);
    } else if constexpr (SCHEME == LBW_WENO3) {
        const T a1 = at(n1, CA);
        hh = weno3_rcp<T>(at(n1, CW) * a1, at(n2, CW) * a2, at(n3, CW) * a3, a1, a2, a3, eps);
    } else {
        hh = at(n2, CW) * a2;
    }
    return hh - kd * (a3 - a2);
}

// WENO5 with the work of each node done once (the arithmetic of weno5_rcp
// regrouped by node).  Node m is the centre of three sub-stencils that faces
// read: with t = a_{m+1} - 2 a_m + a_{m-1} and c = a_{m+1} - a_{m-1}, their
// scaled indicators are
//   e_c = t^2 + (3/13) c^2 + eps12        (the face's centre sub-stencil),
//   e_l = e_c + (12/13) t (t + c)          (one-sided difference 2t + c, at m+1),
//   e_r = e_c + (12/13) t (t - c)          (one-sided difference 2t - c, at m-1),
// the last two being t^2 + (3/13)(2t +- c)^2 + eps12 expanded (each stays
// within a few units in the last place of its value: e_l, e_r >= t^2 + eps12
// and the cancelling part is at most 2 t^2).  A face takes three of them and
// five node fluxes h = w a, chosen by its upwind side.
template <typename T>
__device__ __forceinline__ void weno5_node(T dl, T dr, T eps12, T &el, T &ec, T &er) {
    const T t = dr - dl, c = dr + dl;            // dl = a_m - a_{m-1}, dr = a_{m+1} - a_m
    ec = t * t + ((T)(3.0 / 13.0) * c * c + eps12);
    const T kt = (T)(12.0 / 13.0) * t;
    el = kt * (t + c) + ec;
    er = kt * (t - c) + ec;
}

// Total flux through face j+1/2 from node data: fluxes h at j-2 .. j+3, e_l
// at j-1 and j, e_c at j and j+1, e_r at j+1 and j+2, the upwind side (pos:
// the face velocity w_j + w_{j+1} >= 0) and d = a_{j+1} - a_j for diffusion.
// Upwind from j the sub-stencils are centred at j-1 (as the upwind-most), j,
// j+1 (as the downwind-most); upwind from j+1 at j+2, j+1, j, mirrored.
template <typename T>
__device__ __forceinline__ T weno5_flux_nodes(bool pos, T h0, T h1, T h2, T h3, T h4, T h5,
                                              T el_jm1, T el_j, T ec_j, T ec_jp1, T er_jp1,
                                              T er_jp2, T d, T kappa) {
    const T H0 = pos ? h0 : h5, H1 = pos ? h1 : h4, H2 = pos ? h2 : h3, H3 = pos ? h3 : h2,
            H4 = pos ? h4 : h1;
    const T e0 = pos ? el_jm1 : er_jp2, e1 = pos ? ec_j : ec_jp1, e2 = pos ? er_jp1 : el_j;
    const T S0 = e0 * e0, S1 = e1 * e1, S2 = e2 * e2;
    const T P = S1 * S2, Q = S0 * S2, R = S0 * S1;
    const T q0 = (T)(1.0 / 3.0) * H0 - (T)(7.0 / 6.0) * H1 + (T)(11.0 / 6.0) * H2;
    const T q1 = (T)5 * H2 - H1 + (T)2 * H3;
    const T q2 = H2 + (T)2.5 * H3 - (T)0.5 * H4;
    const T hh = (P * q0 + Q * q1 + R * q2) * fast_rcp<T>(P + (T)6 * Q + (T)3 * R);
    return hh - kappa * d;
}

// S face between nodes j (a2, w2) and j + 1 (a3, w3): first-order upwind
// (S5-S6 in conservative form) and central diffusion.
template <typename T>
__device__ __forceinline__ T s_face(T a2, T a3, T w2, T w3, T kappa) {
    const T hh = ((T)0.5 * (w2 + w3) >= (T)0) ? w2 * a2 : w3 * a3;
    return hh - kappa * (a3 - a2);
}

}  // namespace
}  // namespace lbw
