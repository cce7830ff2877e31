// Arithmetic of the float32 magnetic sweep, shared by every kernel that runs it (the plane-marching
// sweeps, their batched forms and the resident iteration): one cell's new value is the same bits
// whichever kernel, tile or lane computes it. Contraction is off in here and every fused
// multiply-add is written out, so that no instantiation rounds differently from another.
#pragma once

#include "mhd_device.h"

namespace mhd {

// Weights of the plane decomposition: a0f, a0c = in-plane face and corner neighbours of the
// cell's own plane; a1c, a1f, a1k = centre, face and corner of a neighbouring plane.
// D3Q19: 1/18, 1/36 | 1/18, 1/36, 0.  D3Q27 (the product of the 1D weights 2/3, 1/6, 1/6):
// 2/27, 1/54 | 2/27, 1/54, 1/216. Both give a neighbouring plane the total weight 1/6.
template <bool Q27>
struct Lat {
    static constexpr float A0F = 1.0f / 18.0f, A0C = 1.0f / 36.0f, A1C = 1.0f / 18.0f, A1F = 1.0f / 36.0f,
                           A1K = 0.0f;
};
template <>
struct Lat<true> {
    static constexpr float A0F = 2.0f / 27.0f, A0C = 1.0f / 54.0f, A1C = 2.0f / 27.0f, A1F = 1.0f / 54.0f,
                           A1K = 1.0f / 216.0f;
};

// The same weights with omega (b terms) and kappa * omega (flux terms) folded in: the staged flux
// is u_c B_a - u_a B_c and the increment comes out already relaxed.
struct SweepWeights {
    float b0f, b0c, b1f, b1k, l0f, l0c, l1c, l1f, l1k, w6;
};
template <bool Q27>
__device__ __forceinline__ SweepWeights sweep_weights(float kappa, float omega) {
#pragma clang fp contract(off)
    using LW = Lat<Q27>;
    const float ko = kappa * omega;
    return {LW::A0F * omega, LW::A0C * omega, LW::A1F * omega, LW::A1K * omega, LW::A0F * ko,
            LW::A0C * ko,    LW::A1C * ko,    LW::A1F * ko,    LW::A1K * ko,    (1.0f / 6.0f) * omega};
}

// Flux u_c B_a - u_a B_c of one cell: xy, xz, yz.
__device__ __forceinline__ void sweep_flux(float Bx, float By, float Bz, float ux, float uy, float uz, float &lxy,
                                           float &lxz, float &lyz) {
#pragma clang fp contract(off)
    lxy = fmaf(uy, Bx, -(ux * By));
    lxz = fmaf(uz, Bx, -(ux * Bz));
    lyz = fmaf(uz, By, -(uy * Bz));
}

// Contributions of one plane to the outputs at z + 1 (S + P), z (B) and z - 1 (S - P) of E cells
// neighbouring in x (P is zero for the z component), and the cells' own b. rows(k, v) gives rows
// y - 1, y, y + 1 of field k (b_x, b_y, b_z, flux xy, xz, yz) at columns x - 1 .. x + E.
//
// The b sums are differences to the centre, built from second differences along y of each
// column and along x at the cell,
//   faces - 4 c = d2x + d2y(x),   corners - 4 c = d2y(x - 1) + d2y(x + 1) + 2 d2x,
// so that neighbouring cells share their columns: every rounding stays relative to a neighbour
// difference. The flux terms are of order b / R, so plain weighted sums keep their rounding
// below that of b; their column sums s and differences q over rows y -+ 1 are shared as well.
template <int E, bool Q27, typename ROWS>
__device__ __forceinline__ void plane_terms(ROWS rows, const SweepWeights &W, float (&S)[E][3], float (&B)[E][3],
                                            float (&P)[E][2], float (&cen)[E][3]) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        float v[3][E + 2], d2y[E + 2], g[E + 1];
        rows(k, v);
#pragma unroll
        for (int j = 0; j < E + 2; ++j) d2y[j] = (v[2][j] - v[1][j]) - (v[1][j] - v[0][j]);
#pragma unroll
        for (int j = 0; j <= E; ++j) g[j] = v[1][j + 1] - v[1][j];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float d2x = g[e + 1] - g[e];
            const float f = d2x + d2y[1 + e];
            const float q = fmaf(2.0f, d2x, d2y[e] + d2y[e + 2]);
            cen[e][k] = v[1][1 + e];
            B[e][k] = fmaf(W.b0c, q, W.b0f * f);
            S[e][k] = W.b1f * f;
            if constexpr (Q27) S[e][k] = fmaf(W.b1k, q, S[e][k]);
        }
    }
    {  // flux xy: along y (component x) and along x (component y)
        float v[3][E + 2], q[E + 2], s[E + 2];
        rows(3, v);
#pragma unroll
        for (int j = 0; j < E + 2; ++j) {
            q[j] = v[0][j] - v[2][j];
            s[j] = v[0][j] + v[2][j];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float dy = q[1 + e], cdy = q[e] + q[e + 2];
            const float dx = v[1][e] - v[1][e + 2], cdx = s[e] - s[e + 2];
            B[e][0] = fmaf(W.l0c, cdy, fmaf(W.l0f, dy, B[e][0]));
            S[e][0] = fmaf(W.l1f, dy, S[e][0]);
            B[e][1] = fmaf(-W.l0c, cdx, fmaf(-W.l0f, dx, B[e][1]));
            S[e][1] = fmaf(-W.l1f, dx, S[e][1]);
            if constexpr (Q27) {
                S[e][0] = fmaf(W.l1k, cdy, S[e][0]);
                S[e][1] = fmaf(-W.l1k, cdx, S[e][1]);
            }
        }
    }
    float t[E], ct[E];  // component z: flux xz along x and flux yz along y, faces and corners
    {                   // flux xz: through the planes (component x)
        float v[3][E + 2], s[E + 2];
        rows(4, v);
#pragma unroll
        for (int j = 0; j < E + 2; ++j) s[j] = v[0][j] + v[2][j];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            t[e] = v[1][e] - v[1][e + 2];
            ct[e] = s[e] - s[e + 2];
            P[e][0] = fmaf(W.l1c, v[1][1 + e], W.l1f * ((v[1][e] + v[1][e + 2]) + s[1 + e]));
            if constexpr (Q27) P[e][0] = fmaf(W.l1k, s[e] + s[e + 2], P[e][0]);
        }
    }
    {  // flux yz: through the planes (component y)
        float v[3][E + 2], q[E + 2], s[E + 2];
        rows(5, v);
#pragma unroll
        for (int j = 0; j < E + 2; ++j) {
            q[j] = v[0][j] - v[2][j];
            s[j] = v[0][j] + v[2][j];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            P[e][1] = fmaf(W.l1c, v[1][1 + e], W.l1f * ((v[1][e] + v[1][e + 2]) + s[1 + e]));
            if constexpr (Q27) P[e][1] = fmaf(W.l1k, s[e] + s[e + 2], P[e][1]);
            t[e] += q[1 + e];
            ct[e] += q[e] + q[e + 2];
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        B[e][2] = fmaf(-W.l0c, ct[e], fmaf(-W.l0f, t[e], B[e][2]));
        S[e][2] = fmaf(-W.l1f, t[e], S[e][2]);
        if constexpr (Q27) S[e][2] = fmaf(-W.l1k, ct[e], S[e][2]);
    }
}

// Rolling state of a march along z, per cell and component: acc = A(p-2) + B(p-1) (the output at
// p-1 without its C(p) part), ap = A(p-1), cc = b(p-1) at the centre, dz = b(p-1) - b(p-2), with
// A = S + P and C = S - P of plane_terms. Taking plane p gives the output at p-1.
template <int E>
struct March {
    float acc[E][3] = {}, ap[E][3] = {}, cc[E][3] = {}, dz[E][3] = {};
    __device__ __forceinline__ void take(const SweepWeights &W, const float (&S)[E][3], const float (&B)[E][3],
                                         const float (&P)[E][2], const float (&cen)[E][3], float (&out)[E][3]) {
#pragma clang fp contract(off)
#pragma unroll
        for (int e = 0; e < E; ++e)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float A = k < 2 ? S[e][k] + P[e][k < 2 ? k : 0] : S[e][k];
                const float C = k < 2 ? S[e][k] - P[e][k < 2 ? k : 0] : S[e][k];
                const float dzc = cen[e][k] - cc[e][k];
                out[e][k] = fmaf(W.w6, dzc - dz[e][k], acc[e][k] + C) + cc[e][k];
                acc[e][k] = ap[e][k] + B[e][k];
                ap[e][k] = A;
                cc[e][k] = cen[e][k];
                dz[e][k] = dzc;
            }
    }
};

}  // namespace mhd
