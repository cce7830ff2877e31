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
// neighbouring in x (P is zero for the z component), and the cells' own b.
//
// The b sums are differences to the centre, built from second differences along y of each
// column and along x at the cell,
//   faces - 4 c = d2x + d2y(x),   corners - 4 c = d2y(x - 1) + d2y(x + 1) + 2 d2x,
// so that neighbouring cells share their columns: every rounding stays relative to a neighbour
// difference. The flux terms are of order b / R, so plain weighted sums keep their rounding
// below that of b; their column sums s and differences q over rows y -+ 1 are shared as well.
//
// Of the columns beside it a cell needs only their combinations and their centre row: cols.second(k,
// c, d2y) and cols.first(k, c, q, s) give them for field k (b_x, b_y, b_z; flux xy, xz, yz) and columns
// x - 1 .. x + E. A kernel that reads every column from LDS forms them all (ColumnsRows); one whose
// neighbouring lanes hold the neighbouring columns forms its own E and takes the others' combinations
// from there (ColumnsWave): the same operations on the same values, so the same bits.
__device__ __forceinline__ float column_d2(float m, float c, float p) {
#pragma clang fp contract(off)
    return (p - c) - (c - m);
}
template <int E, bool Q27, typename COLS>
__device__ __forceinline__ void plane_terms(COLS cols, const SweepWeights &W, float (&S)[E][3], float (&B)[E][3],
                                            float (&P)[E][2], float (&cen)[E][3]) {
#pragma clang fp contract(off)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        float c[E + 2], d2y[E + 2], g[E + 1];
        cols.second(k, c, d2y);
#pragma unroll
        for (int j = 0; j <= E; ++j) g[j] = c[j + 1] - c[j];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float d2x = g[e + 1] - g[e];
            const float f = d2x + d2y[1 + e];
            const float q = fmaf(2.0f, d2x, d2y[e] + d2y[e + 2]);
            cen[e][k] = c[1 + e];
            B[e][k] = fmaf(W.b0c, q, W.b0f * f);
            S[e][k] = W.b1f * f;
            if constexpr (Q27) S[e][k] = fmaf(W.b1k, q, S[e][k]);
        }
    }
    {  // flux xy: along y (component x) and along x (component y)
        float c[E + 2], q[E + 2], s[E + 2];
        cols.template first<true, true>(3, c, q, s);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const float dy = q[1 + e], cdy = q[e] + q[e + 2];
            const float dx = c[e] - c[e + 2], cdx = s[e] - s[e + 2];
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
        float c[E + 2], q[E + 2], s[E + 2];
        cols.template first<false, true>(4, c, q, s);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            t[e] = c[e] - c[e + 2];
            ct[e] = s[e] - s[e + 2];
            P[e][0] = fmaf(W.l1c, c[1 + e], W.l1f * ((c[e] + c[e + 2]) + s[1 + e]));
            if constexpr (Q27) P[e][0] = fmaf(W.l1k, s[e] + s[e + 2], P[e][0]);
        }
    }
    {  // flux yz: through the planes (component y); beside the cell, s only on D3Q27
        float c[E + 2], q[E + 2], s[E + 2];
        cols.template first<true, Q27>(5, c, q, s);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            P[e][1] = fmaf(W.l1c, c[1 + e], W.l1f * ((c[e] + c[e + 2]) + s[1 + e]));
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

// Columns from rows: rows(k, v) gives rows y - 1, y, y + 1 of field k at columns x - 1 .. x + E.
template <int E, typename ROWS>
struct ColumnsRows {
    ROWS rows;
    __device__ __forceinline__ void second(int k, float (&c)[E + 2], float (&d2y)[E + 2]) {
        float v[3][E + 2];
        rows(k, v);
#pragma unroll
        for (int j = 0; j < E + 2; ++j) {
            c[j] = v[1][j];
            d2y[j] = column_d2(v[0][j], v[1][j], v[2][j]);
        }
    }
    // NQ, NS: whether q and s of the columns beside the cells are used
    template <bool NQ, bool NS>
    __device__ __forceinline__ void first(int k, float (&c)[E + 2], float (&q)[E + 2], float (&s)[E + 2]) {
#pragma clang fp contract(off)
        float v[3][E + 2];
        rows(k, v);
#pragma unroll
        for (int j = 0; j < E + 2; ++j) {
            c[j] = v[1][j];
            q[j] = v[0][j] - v[2][j];
            s[j] = v[0][j] + v[2][j];
        }
    }
};
template <int E, typename ROWS>
__device__ __forceinline__ ColumnsRows<E, ROWS> columns_rows(ROWS rows) {
    return {rows};
}

// Columns of a wave whose lanes hold consecutive groups of E columns: own(k, v) gives rows y - 1, y,
// y + 1 at the lane's columns. Two instructions a combination replace six reads or moves of raw rows
// and the arithmetic of two columns: 256 x 132^2 (4-row tiles, 36 aligned reads a plane -> 18 and 18 of
// one word) 43.8 -> 36.8 us a sweep, 512 x 256^2 240.2 -> 234.9, 128^3 16.5 -> 16.3, 200 x 132^2 (one
// cell a lane) 40.5 -> 37.1. Launches of few workgroups are the slower for it, and form all columns (few_workgroups in
// mhd_sweep.hip). HALO: end(k, h) gives the rows of the column beyond the wave,
// left of lane 0 and right of lane 63 (the lanes below 32 hold the left one, the others the right);
// without it the wave is a whole periodic row and the ends wrap.
__device__ __forceinline__ float wave_ror1(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x13C, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_rol1(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x134, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_shr1(float end, float v) {  // lane 0 keeps end
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(end), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float wave_shl1(float end, float v) {  // lane 63 keeps end
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(end), __float_as_int(v), 0x130, 0xf, 0xf, false));
}
template <int E, bool HALO, typename OWN, typename END>
struct ColumnsWave {
    OWN own;
    END end;
    // the columns beside the lane's: x holds its own at 1 .. E, h is the value at the wave's end
    static __device__ __forceinline__ void beside(float (&x)[E + 2], float h) {
        x[0] = HALO ? wave_shr1(h, x[E]) : wave_ror1(x[E]);
        x[E + 1] = HALO ? wave_shl1(h, x[1]) : wave_rol1(x[1]);
    }
    __device__ __forceinline__ void second(int k, float (&c)[E + 2], float (&d2y)[E + 2]) {
        float v[3][E], h[3] = {0.0f, 0.0f, 0.0f};
        own(k, v);
        if constexpr (HALO) end(k, h);
#pragma unroll
        for (int j = 0; j < E; ++j) {
            c[1 + j] = v[1][j];
            d2y[1 + j] = column_d2(v[0][j], v[1][j], v[2][j]);
        }
        beside(c, h[1]);
        beside(d2y, column_d2(h[0], h[1], h[2]));
    }
    template <bool NQ, bool NS>
    __device__ __forceinline__ void first(int k, float (&c)[E + 2], float (&q)[E + 2], float (&s)[E + 2]) {
#pragma clang fp contract(off)
        float v[3][E], h[3] = {0.0f, 0.0f, 0.0f};
        own(k, v);
        if constexpr (HALO) end(k, h);
#pragma unroll
        for (int j = 0; j < E; ++j) {
            c[1 + j] = v[1][j];
            q[1 + j] = v[0][j] - v[2][j];
            s[1 + j] = v[0][j] + v[2][j];
        }
        beside(c, h[1]);
        if constexpr (NQ) beside(q, h[0] - h[2]);
        if constexpr (NS) beside(s, h[0] + h[2]);
    }
};
template <int E, bool HALO, typename OWN, typename END>
__device__ __forceinline__ ColumnsWave<E, HALO, OWN, END> columns_wave(OWN own, END end) {
    return {own, end};
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
