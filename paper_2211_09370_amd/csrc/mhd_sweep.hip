// gfx950 magnetic sweep of the quasi-static induction iteration (arXiv:2211.09370, Sec. 5.7):
// the single-cell-per-lane and paired (two x cells per lane) plane-marching kernels, each in a
// single-box and a batched instantiation, and their host-side launchers.
#include <hip/hip_ext.h>

#include <type_traits>

#include "mhd_device.h"
#include "mhd_sweep_math.h"

namespace mhd {

// -------------------------------------------------------------------------------------------
// Magnetic sweep (Sec. 5.7): tau_m = 1, particle speed c = 6 eta, so c_i / c_s^2 = e_i / (2 eta).
//
//   b*_a(x) = sum_i w_i [ b_a(x - e_i) + kappa sum_c e_ic Lam_ac(x - e_i) ],
//   Lam_ac = u_c B_a - u_a B_c,  B = B_ext + b,  kappa = 1 / (2 eta).
//
// Written per plane: a workgroup owns a TX x TY column of cells and marches along z over a
// chunk of planes. Each new plane (with a one-cell x/y halo) is staged in LDS as
// (b_x, b_y, b_z, kappa Lam_xy, kappa Lam_xz, kappa Lam_yz); every thread forms from its 3x3
// in-plane neighbourhood the plane's contributions to the outputs at z-1, z and z+1
// (A, B, C below) and keeps the running sums in registers, so each field value is read from
// memory once per plane and every neighbour access is an LDS read.
//
// With D_c[f](x) = sum_i w_i e_ic f(x - e_i) and the in-plane sums
//   P0 = c/3 + (faces)/18 + (corners)/36,  P1 = c/18 + (faces)/36,
//   Q0x = (xm - xp)/18 + (mm + mp - pm - pp)/36,  Q1x = (xm - xp)/36   (Q*y likewise in y),
// one has avg[f](z) = P0(z) + P1(z-1) + P1(z+1), D_x[f](z) = Q0x(z) + Q1x(z-1) + Q1x(z+1),
// D_y likewise and D_z[f](z) = P1(z-1) - P1(z+1); then
//   b*_x = avg b_x + D_y Lxy + D_z Lxz,  b*_y = avg b_y - D_x Lxy + D_z Lyz,
//   b*_z = avg b_z - D_x Lxz - D_y Lyz.
//
// Units: the sweep works on stored values (b / b_scale, u / u_scale), with B_ext divided by
// b_scale once per workgroup and kappa multiplied by u_scale, which keeps the same map (it is
// linear in (b, B_ext)) and leaves no per-value scaling: staging and output are plain
// conversions and additions (float32 storage has both scales 1).
//
// Accelerated iteration (Sec. 5.8): with rest weight w_0 - 1 + alpha and the sum divided by
// alpha, the update is b + (b* - b) / alpha, i.e. the increment above times omega = 1 / alpha.
//
// BYZ: B_ext also has a (y, z) part (six magnets): a 3 x (ny nz) table, requested with each
// plane's loads and added while staging.
//
// SPLIT: b is held as two float16 arrays, b = (hi + lo) b_scale. hi is fixed within a fluid
// step; the sweep stages hi + lo and writes lo* = lo + increment, so the 16-bit rounding is
// relative to lo, not to b. The first sweep of a step (a.bho set) re-splits v = hi + lo +
// increment into a new hi = fp16(v) and lo = fp16(v - hi).
// -------------------------------------------------------------------------------------------

// The tile of this workgroup (its index within its box; -1: none) and, in a batch, its box's arguments.
// XCD-aware order: the hardware hands consecutive workgroups to the 8 XCDs in turn; give each XCD a
// contiguous run of tiles so neighbouring tiles share halo rows in one L2.
template <bool BATCH>
__device__ __forceinline__ int sweep_tile(SweepArgs &a, const PipeStep *tab, const BlockMap *map, int which, int nbatch) {
    const int per = gridDim.x >> 3;
    const int lb = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if constexpr (BATCH) {
        if (lb >= nbatch) return -1;
        const BlockMap m = map[lb];
        a = tab[m.pipe].sw[which];
        return m.local;
    }
    return lb < a.nblocks ? lb : -1;
}

template <int TX, int TY>
constexpr int kSweepLds = 2 * 6 * (TX + 2) * (TY + 2);  // two LDS planes (floats)

template <int TX, int TY, typename TU, typename TB, bool SPLIT, bool BYZ, bool Q27, bool FEW = false>
__device__ __forceinline__ void sweep_cells(const SweepArgs &a, const int lb, float *lds) {
    using LW = Lat<Q27>;
    constexpr int NT = TX * TY, HX = TX + 2, HY = TY + 2, HN = HX * HY;
    constexpr int NSLOT = (HN + NT - 1) / NT;
    // two LDS planes: the next plane is staged while the current one is reduced
    float (*s_pl)[6][HN] = reinterpret_cast<float (*)[6][HN]>(lds);
    const int tix = lb % a.tiles_x;
    const int rest = lb / a.tiles_x;
    const int tiy = rest % a.tiles_y;
    const int tiz = rest / a.tiles_y;
    const int x0 = tix * TX, y0 = tiy * TY;
    const int z0 = tiz * a.zchunk;
    const int z1 = min(z0 + a.zchunk, a.nz);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const unsigned N = (unsigned)nx * ny * nz;  // 3 N < 2^31: 32-bit offsets from uniform bases
    const unsigned plane = (unsigned)nx * ny;

    const TU *u0 = (const TU *)a.u, *u1 = u0 + N, *u2 = u0 + 2 * (size_t)N;
    const TB *b0 = (const TB *)a.b, *b1 = b0 + N, *b2 = b0 + 2 * (size_t)N;
    TB *o0 = (TB *)a.bo, *o1 = o0 + N, *o2 = o0 + 2 * (size_t)N;
    const TB *bh0 = (const TB *)a.bh, *bh1 = bh0 + N, *bh2 = bh0 + 2 * (size_t)N;  // SPLIT: hi part
    const bool resplit = SPLIT && a.bho != nullptr;

    const int tid = threadIdx.x;
    const int lx = tid % TX, ly = tid / TX;
    const int gx = x0 + lx, gy = y0 + ly;
    const bool own = gx < nx && gy < ny;

    // halo slots handled by this thread: fixed (x, y) for the whole march
    unsigned sxy[NSLOT];
    int sy[NSLOT];
    float sbe[NSLOT][3];
    bool sval[NSLOT];
#pragma unroll
    for (int s = 0; s < NSLOT; ++s) {
        const int i = tid + s * NT;
        sval[s] = i < HN;
        const int hx = i % HX, hy = i / HX;
        const int hxg = wrapi(x0 - 1 + hx, nx), hyg = wrapi(y0 - 1 + hy, ny);
        sxy[s] = (unsigned)(hxg + nx * hyg);
        sy[s] = hyg;
        sbe[s][0] = sval[s] ? a.bext[hxg] * a.inv_b_scale : 0.f;
        sbe[s][1] = sval[s] ? a.bext[nx + hxg] * a.inv_b_scale : 0.f;
        sbe[s][2] = sval[s] ? a.bext[2 * nx + hxg] * a.inv_b_scale : 0.f;
    }

    // raw stored values of the next plane: converted only when they are written to LDS, so the
    // loads stay in flight while the current plane is reduced
    TU ru[NSLOT][3];
    TB rb[NSLOT][3];
    TB rh[NSLOT][3];
    float rt[NSLOT][3];  // BYZ: B_ext (y, z) part of the next plane
    const unsigned pyz = (unsigned)ny * nz;
    auto load_plane = [&](int p) {
        const unsigned off = (unsigned)wrapi(p, nz) * plane;
        if constexpr (BYZ) {
#pragma unroll
            for (int s = 0; s < NSLOT; ++s) {
                const unsigned o = (unsigned)(sy[s] + ny * wrapi(p, nz));
                rt[s][0] = sval[s] ? a.bext_yz[o] : 0.f;
                rt[s][1] = sval[s] ? a.bext_yz[pyz + o] : 0.f;
                rt[s][2] = sval[s] ? a.bext_yz[2 * pyz + o] : 0.f;
            }
        }
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) {
            if (sval[s]) {
                const unsigned ku = (off + sxy[s]) * (unsigned)sizeof(TU);
                const unsigned kb = (off + sxy[s]) * (unsigned)sizeof(TB);
                ru[s][0] = ld_off(u0, ku);
                ru[s][1] = ld_off(u1, ku);
                ru[s][2] = ld_off(u2, ku);
                rb[s][0] = ld_off(b0, kb);
                rb[s][1] = ld_off(b1, kb);
                rb[s][2] = ld_off(b2, kb);
                if constexpr (SPLIT) {
                    rh[s][0] = ld_off(bh0, kb);
                    rh[s][1] = ld_off(bh1, kb);
                    rh[s][2] = ld_off(bh2, kb);
                }
            }
        }
    };

    const int c0 = (ly + 1) * HX + (lx + 1);
    constexpr bool F32 = std::is_same<TB, float>::value;  // shared float32 arithmetic (mhd_sweep_math.h)
    const SweepWeights W = sweep_weights<Q27>(a.kappa, a.omega);
    March<1> march;
    const float kap = a.kappa * a.u_scale;
    constexpr float W6 = 1.0f / 6.0f;  // total weight of a neighbouring plane (both lattices)
    // running sums of the plane contributions (difference form), and the column's own values
    float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f;
    float ap0 = 0.f, ap1 = 0.f, ap2 = 0.f;
    float cm0 = 0.f, cm1 = 0.f, cm2 = 0.f;  // b at (x, y, z-1)
    float cc0 = 0.f, cc1 = 0.f, cc2 = 0.f;  // b at (x, y, z)

    // stage the raw values in the registers into LDS buffer S as (b, kappa Lam)
    auto stage = [&](auto buf) {
        constexpr int S = decltype(buf)::value;
#pragma unroll
        for (int s = 0; s < NSLOT; ++s) {
            if (sval[s]) {
                const int i = tid + s * NT;
                float bx = St<TB>::cvt(rb[s][0]);
                float by = St<TB>::cvt(rb[s][1]);
                float bz = St<TB>::cvt(rb[s][2]);
                if constexpr (SPLIT) {
                    bx += St<TB>::cvt(rh[s][0]);
                    by += St<TB>::cvt(rh[s][1]);
                    bz += St<TB>::cvt(rh[s][2]);
                }
                float be0 = sbe[s][0], be1 = sbe[s][1], be2 = sbe[s][2];
                if constexpr (BYZ) {
                    be0 += rt[s][0] * a.inv_b_scale;
                    be1 += rt[s][1] * a.inv_b_scale;
                    be2 += rt[s][2] * a.inv_b_scale;
                }
                const float Bx = bx + be0;
                const float By = by + be1;
                const float Bz = bz + be2;
                const float ux = St<TU>::cvt(ru[s][0]);
                const float uy = St<TU>::cvt(ru[s][1]);
                const float uz = St<TU>::cvt(ru[s][2]);
                s_pl[S][0][i] = bx;
                s_pl[S][1][i] = by;
                s_pl[S][2][i] = bz;
                if constexpr (F32) {
                    sweep_flux(Bx, By, Bz, ux, uy, uz, s_pl[S][3][i], s_pl[S][4][i], s_pl[S][5][i]);
                } else {
                    s_pl[S][3][i] = kap * (uy * Bx - ux * By);
                    s_pl[S][4][i] = kap * (uz * Bx - ux * Bz);
                    s_pl[S][5][i] = kap * (uz * By - uy * Bz);
                }
            }
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    // plane r = p - (z0 - 1) is reduced from LDS buffer r % 2; while it is, the next plane is
    // staged into the other buffer and the one after that is requested into the registers
    load_plane(z0 - 1);
    stage(I0{});
    load_plane(z0);
    __syncthreads();
    auto body = [&](auto par, int p) {
        constexpr int P = decltype(par)::value;  // parity of plane p
        using Q = std::integral_constant<int, 1 - P>;
        // plane p+1 goes from the registers to the other LDS buffer (its last readers passed
        // the previous barrier); the registers then request plane p+2
        if (p < z1) {
            stage(Q{});
            if (p + 2 <= z1) load_plane(p + 2);
        }
        // SPLIT: the stored lo (and, re-splitting, hi) of this column's output cell, requested
        // now and used after the reduction
        const unsigned ko = ((unsigned)(p - 1) * plane + (unsigned)(gx + nx * gy)) * (unsigned)sizeof(TB);
        TB lc[3], hc[3];
        if constexpr (SPLIT) {
            if (own && p >= z0 + 1) {
                lc[0] = ld_off(b0, ko);
                lc[1] = ld_off(b1, ko);
                lc[2] = ld_off(b2, ko);
                if (resplit) {
                    hc[0] = ld_off(bh0, ko);
                    hc[1] = ld_off(bh1, ko);
                    hc[2] = ld_off(bh2, ko);
                }
            }
        }
        const int cur = P;
        const float *s_bx = s_pl[cur][0], *s_by = s_pl[cur][1], *s_bz = s_pl[cur][2];
        const float *s_lxy = s_pl[cur][3], *s_lxz = s_pl[cur][4], *s_lyz = s_pl[cur][5];
        if constexpr (F32) {
            float S[1][3], B[1][3], Pz[1][2], cen[1][3], out[1][3];
            auto take = [&](auto cols) {
                plane_terms<1, Q27>(cols, W, S, B, Pz, cen);
                march.take(W, S, B, Pz, cen, out);
                if (own && p >= z0 + 1) {
                    st_off(o0, ko, out[0][0]);
                    st_off(o1, ko, out[0][1]);
                    st_off(o2, ko, out[0][2]);
                }
            };
            if constexpr (TX == 64 && !FEW) {
                // A wave is a row: 18 reads of the own column and 18 of the halo column instead of 54 (which FEW
                // takes), and the columns beside it from the lanes beside it. Lanes beyond n_x hold staged
                // (wrapped) cells, so the last cell's neighbour is there too.
                if (gy < ny) {
                    auto cells = [&](int k, float (&v)[3][1]) {
#pragma unroll
                        for (int r = 0; r < 3; ++r) v[r][0] = s_pl[cur][k][c0 + (r - 1) * HX];
                    };
                    auto end = [&](int k, float (&h)[3]) {
#pragma unroll
                        for (int r = 0; r < 3; ++r) h[r] = s_pl[cur][k][(ly + r) * HX + (lx < 32 ? 0 : HX - 1)];
                    };
                    take(columns_wave<1, true>(cells, end));
                }
            } else if (own) {
                take(columns_rows<1>([&](int k, float (&v)[3][3]) {
#pragma unroll
                    for (int r = 0; r < 3; ++r)
#pragma unroll
                        for (int j = 0; j < 3; ++j) v[r][j] = s_pl[cur][k][c0 + (r - 1) * HX + (j - 1)];
                }));
            }
        } else if (own) {
            // b components: centre value and in-plane sums of differences to it
            //   dP0 = sum_faces a0f (f - c) + sum_corners a0c (f - c),
            //   dP1 = sum_faces a1f (f - c) [+ sum_corners a1k (f - c) on D3Q27]
            float c_x, c_y, c_z, dP0x, dP1x, dP0y, dP1y, dP0z, dP1z;
#define MHD_PLANE_DIFFS(F, C, DP0, DP1)                                                              \
    {                                                                                                \
        const float *f = F;                                                                          \
        C = f[c0];                                                                                   \
        const float fs = ((f[c0 - 1] - C) + (f[c0 + 1] - C)) + ((f[c0 - HX] - C) + (f[c0 + HX] - C)); \
        const float cs = ((f[c0 - HX - 1] - C) + (f[c0 - HX + 1] - C)) +                              \
                         ((f[c0 + HX - 1] - C) + (f[c0 + HX + 1] - C));                               \
        DP0 = LW::A0F * fs + LW::A0C * cs;                                                           \
        DP1 = LW::A1F * fs;                                                                          \
        if constexpr (Q27) DP1 += LW::A1K * cs;                                                      \
    }
            MHD_PLANE_DIFFS(s_bx, c_x, dP0x, dP1x)
            MHD_PLANE_DIFFS(s_by, c_y, dP0y, dP1y)
            MHD_PLANE_DIFFS(s_bz, c_z, dP0z, dP1z)
            // kappa Lam_xy: Q0x, Q1x, Q0y, Q1y (differences across the cell)
            float Q0xA, Q1xA, Q0yA, Q1yA;
            {
                const float *f = s_lxy;
                const float dx = f[c0 - 1] - f[c0 + 1], dy = f[c0 - HX] - f[c0 + HX];
                const float mm = f[c0 - HX - 1], pm = f[c0 - HX + 1], mp = f[c0 + HX - 1], pp = f[c0 + HX + 1];
                Q0xA = LW::A0F * dx + LW::A0C * ((mm - pm) + (mp - pp));
                Q1xA = LW::A1F * dx;
                Q0yA = LW::A0F * dy + LW::A0C * ((mm - mp) + (pm - pp));
                Q1yA = LW::A1F * dy;
                if constexpr (Q27) {
                    Q1xA += LW::A1K * ((mm - pm) + (mp - pp));
                    Q1yA += LW::A1K * ((mm - mp) + (pm - pp));
                }
            }
            // kappa Lam_xz: P1, Q0x, Q1x and kappa Lam_yz: P1, Q0y, Q1y. These flux terms are
            // of order b / R, so plain weighted sums keep their rounding below that of b.
            float P1B, Q0xB, Q1xB;
            {
                const float *f = s_lxz;
                const float xm = f[c0 - 1], xp = f[c0 + 1];
                const float mm = f[c0 - HX - 1], pm = f[c0 - HX + 1], mp = f[c0 + HX - 1], pp = f[c0 + HX + 1];
                P1B = LW::A1C * f[c0] + LW::A1F * ((xm + xp) + (f[c0 - HX] + f[c0 + HX]));
                Q0xB = LW::A0F * (xm - xp) + LW::A0C * ((mm - pm) + (mp - pp));
                Q1xB = LW::A1F * (xm - xp);
                if constexpr (Q27) {
                    P1B += LW::A1K * ((mm + pm) + (mp + pp));
                    Q1xB += LW::A1K * ((mm - pm) + (mp - pp));
                }
            }
            float P1C, Q0yC, Q1yC;
            {
                const float *f = s_lyz;
                const float ym = f[c0 - HX], yp = f[c0 + HX];
                const float mm = f[c0 - HX - 1], pm = f[c0 - HX + 1], mp = f[c0 + HX - 1], pp = f[c0 + HX + 1];
                P1C = LW::A1C * f[c0] + LW::A1F * ((f[c0 - 1] + f[c0 + 1]) + (ym + yp));
                Q0yC = LW::A0F * (ym - yp) + LW::A0C * ((mm - mp) + (pm - pp));
                Q1yC = LW::A1F * (ym - yp);
                if constexpr (Q27) {
                    P1C += LW::A1K * ((mm + pm) + (mp + pp));
                    Q1yC += LW::A1K * ((mm - mp) + (pm - pp));
                }
            }
            // contributions of this plane to the outputs at z+1 (A), z (B), z-1 (C)
            const float A0 = dP1x + Q1yA + P1B, B0 = dP0x + Q0yA, C0 = dP1x + Q1yA - P1B;
            const float A1 = dP1y - Q1xA + P1C, B1 = dP0y - Q0xA, C1 = dP1y - Q1xA - P1C;
            const float A2 = dP1z - Q1xB - Q1yC, B2 = dP0z - Q0xB - Q0yC;
            if (p >= z0 + 1) {
                // output plane p-1: b* = b_c + increment, the increment built from differences
                const float d0 = a.omega * ((acc0 + C0) + W6 * ((cm0 - cc0) + (c_x - cc0)));
                const float d1 = a.omega * ((acc1 + C1) + W6 * ((cm1 - cc1) + (c_y - cc1)));
                const float d2 = a.omega * ((acc2 + A2) + W6 * ((cm2 - cc2) + (c_z - cc2)));
                if constexpr (SPLIT) {
                    const float d[3] = {d0, d1, d2};
                    TB *oo[3] = {o0, o1, o2};
                    TB *ho = (TB *)a.bho;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const float lo = St<TB>::cvt(lc[q]);
                        if (resplit) {
                            const float v = (St<TB>::cvt(hc[q]) + lo) + d[q];
                            const TB hi = St<TB>::from(v, 1.0f);
                            st_off(ho + q * (size_t)N, ko, hi);
                            st_off(oo[q], ko, St<TB>::from(v - St<TB>::cvt(hi), 1.0f));
                        } else {
                            st_off(oo[q], ko, St<TB>::from(lo + d[q], 1.0f));
                        }
                    }
                } else {
                    st_off(o0, ko, St<TB>::from(cc0 + d0, 1.0f));
                    st_off(o1, ko, St<TB>::from(cc1 + d1, 1.0f));
                    st_off(o2, ko, St<TB>::from(cc2 + d2, 1.0f));
                }
            }
            acc0 = ap0 + B0;
            acc1 = ap1 + B1;
            acc2 = ap2 + B2;
            ap0 = A0;
            ap1 = A1;
            ap2 = A2;
            cm0 = cc0;
            cm1 = cc1;
            cm2 = cc2;
            cc0 = c_x;
            cc1 = c_y;
            cc2 = c_z;
        }
        __syncthreads();  // plane p+1 is staged; buffer `cur` may be overwritten next
    };
    for (int p = z0 - 1; p <= z1; p += 2) {
        body(I0{}, p);
        if (p + 1 <= z1) body(I1{}, p + 1);
    }
#undef MHD_PLANE_DIFFS
}

template <int TX, int TY, typename TU, typename TB, bool BATCH, bool SPLIT, bool BYZ, bool Q27, bool FEW>
__global__ void __launch_bounds__(TX *TY) __attribute__((amdgpu_waves_per_eu(std::is_same<TB, float>::value && !BYZ && !FEW ? 4 : 1)))
k_mag_sweep(SweepArgs a, const PipeStep *tab, const BlockMap *map, int which, int nbatch) {
    __shared__ float lds[kSweepLds<TX, TY>];
    const int lb = sweep_tile<BATCH>(a, tab, map, which, nbatch);
    if (lb >= 0) sweep_cells<TX, TY, TU, TB, SPLIT, BYZ, Q27, FEW>(a, lb, lds);
}

// -------------------------------------------------------------------------------------------
// Paired magnetic sweep for boxes with n_x a multiple of 128: the same plane march and the same
// update as k_mag_sweep, but every lane owns two neighbouring x cells, so a wave covers a
// 128-cell row. Rows are loaded and stored as 8-byte (float32) or 4-byte (16-bit) pairs: half
// the memory instructions per cell. The 16-bit kinds read the four values x-1 .. x+2 of a staged
// row from LDS with two aligned 8-byte reads and share work between the two cells (differences
// against one reference, shared column sums, weights with kappa and the relaxation folded in).
// float32 (4-row tiles; mhd_sweep_rows.hip has those of 8 rows) reads only the lane's own pair of
// each row: of the columns beside it just d2y, the row difference sums and the centre enter, and the
// neighbouring lanes have formed those (DPP), the wave's ends taking them from the halo columns. It
// is bound by the plane's chain in a CU, vector instructions and LDS reads, so the fewer reads show:
// 256 x 132^2 43.8 -> 36.8 us, 128^3 16.5 -> 16.3 us. FEW (launches of few workgroups, few_workgroups below)
// reads the columns beside as the 16-bit kinds do. Its arithmetic is mhd_sweep_math.h, in every form
// the same bits. Single boxes with n_x = 128 (XWRAP: one tile spans the periodic row) stage no
// halo columns, x neighbours come by wave rotation, the ends wrapping as the row does; the batch
// keeps the halo form, since one of its launches can mix pipes of different n_x. In float32 XWRAP
// also stages by 16-byte loads, four cells per lane and two rows per wave, which halves the load
// instructions of a plane.
// -------------------------------------------------------------------------------------------
template <typename T>
struct Pair;
template <>
struct Pair<float> {
    using raw = float2;
    static __device__ __forceinline__ float lo(raw v, float) { return v.x; }
    static __device__ __forceinline__ float hi(raw v, float) { return v.y; }
    static __device__ __forceinline__ raw make(float a, float b, float) { return make_float2(a, b); }
};
template <>
struct Pair<__half> {
    using raw = __half2;
    static __device__ __forceinline__ float lo(raw v, float s) { return __low2float(v) * s; }
    static __device__ __forceinline__ float hi(raw v, float s) { return __high2float(v) * s; }
    static __device__ __forceinline__ raw make(float a, float b, float inv) {
        return __halves2half2(__float2half_rn(a * inv), __float2half_rn(b * inv));
    }
};
template <>
struct Pair<__hip_bfloat16> {
    using raw = unsigned;  // low half = element x, high half = element x + 1
    static __device__ __forceinline__ float lo(raw v, float s) { return __uint_as_float(v << 16) * s; }
    static __device__ __forceinline__ float hi(raw v, float s) { return __uint_as_float(v & 0xffff0000u) * s; }
    static __device__ __forceinline__ raw make(float a, float b, float inv) {
        const __hip_bfloat16 x = __float2bfloat16(a * inv), y = __float2bfloat16(b * inv);
        return (unsigned)__bfloat16_as_ushort(x) | ((unsigned)__bfloat16_as_ushort(y) << 16);
    }
};

template <int TY>
constexpr int kPairLds = 2 * 6 * (TY + 2) * 132;

template <int TY, typename TU, typename TB, bool SPLIT, bool BYZ, bool Q27, bool XWRAP, bool FEW = false>
__device__ __forceinline__ void sweep_pairs(const SweepArgs &a, const int lb, float *lds) {
    using LW = Lat<Q27>;
    constexpr int HY = TY + 2;        // staged rows
    // LDS row stride: x0-1 at 0, x0 .. x0+127 at 1 .. 128, x0+128 at 129. XWRAP (n_x = 128, one tile
    // per row, periodic in x): x0 .. x0+127 at 0 .. 127 and no halo columns; the x neighbours of a
    // lane's two cells come from the neighbouring lanes, across the wave ends for the wrap.
    constexpr int RS = 132;
    // WAVE (float32, x neighbours from the lanes beside): x0 .. x0+127 at 0 .. 127, the halo columns at
    // 128 and 129.
    constexpr bool F32 = std::is_same<TB, float>::value;  // shared float32 arithmetic (mhd_sweep_math.h)
    constexpr bool WAVE = F32 && (XWRAP || !FEW);
    constexpr int X0 = XWRAP || WAVE ? 0 : 1;
    float (*s_pl)[6][HY * RS] = reinterpret_cast<float (*)[6][HY * RS]>(lds);
    const int tix = lb % a.tiles_x;
    const int rest = lb / a.tiles_x;
    const int tiy = rest % a.tiles_y;
    const int tiz = rest / a.tiles_y;
    const int x0 = tix * 128, y0 = tiy * TY;
    const int z0 = tiz * a.zchunk;
    const int z1 = min(z0 + a.zchunk, a.nz);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const unsigned N = (unsigned)nx * ny * nz;
    const unsigned plane = (unsigned)nx * ny;
    const TU *u0 = (const TU *)a.u, *u1 = u0 + N, *u2 = u0 + 2 * (size_t)N;
    const TB *b0 = (const TB *)a.b, *b1 = b0 + N, *b2 = b0 + 2 * (size_t)N;
    TB *o0 = (TB *)a.bo, *o1 = o0 + N, *o2 = o0 + 2 * (size_t)N;
    const TB *bh0 = (const TB *)a.bh, *bh1 = bh0 + N, *bh2 = bh0 + 2 * (size_t)N;  // SPLIT: hi part
    const bool resplit = SPLIT && a.bho != nullptr;
    using PU = Pair<TU>;
    using PB = Pair<TB>;
    using RU = typename PU::raw;
    using RB = typename PB::raw;

    const int tid = threadIdx.x;
    const int w = tid >> 6, l = tid & 63;
    const int xa = x0 + 2 * l;            // this lane's cells: xa, xa + 1 (always inside: nx % 128 == 0)
    const int gy = y0 + w;
    const bool own = gy < ny;
    const float ib = a.inv_b_scale;
    // Weights with omega (b terms) and kappa * u_scale * omega (flux terms) folded in: the staged
    // flux is u_c B_a - u_a B_c in stored units, and the increment comes out already relaxed.
    const float om = a.omega, ko = a.kappa * a.u_scale * a.omega;
    const float b0f = LW::A0F * om, b0c = LW::A0C * om, b1f = LW::A1F * om, b1k = LW::A1K * om;
    const float l0f = LW::A0F * ko, l0c = LW::A0C * ko, l1c = LW::A1C * ko, l1f = LW::A1F * ko, l1k = LW::A1K * ko;
    const float w6 = (1.0f / 6.0f) * om;  // total weight of a neighbouring plane (both lattices)
    const SweepWeights W = sweep_weights<Q27>(a.kappa, a.omega);
    March<2> march;

    // Staging (float32 with XWRAP: QUAD below, 16-byte loads staging two rows per wave): wave w
    // stages row hy = w (its own pair of cells per lane). With 4-row tiles the
    // two remaining rows hy = TY, TY + 1 are staged as pairs by waves 0 and 1 (fewer memory
    // instructions); with 8-row tiles one cell per lane by waves 0 .. 3 (lane -> x = 64 (w & 1)
    // + l), which measured faster there. Lanes 0 .. 2*HY-1 of the last wave stage the halo
    // columns x0 - 1 and x0 + 128 (not with XWRAP).
    const int pyr = wrapi(y0 - 1 + w, ny);
    const unsigned poff = (unsigned)(xa + nx * pyr);
    constexpr bool SPAIR = TY == 4;
    const bool sval = SPAIR ? w < 2 : w < 4;
    const int shy = SPAIR ? TY + min(w, 1) : TY + (w >> 1), sxl = ((w & 1) << 6) + l;
    const int syr = wrapi(y0 - 1 + shy, ny);
    const unsigned soff = SPAIR ? (unsigned)(xa + nx * syr) : (unsigned)(x0 + sxl + nx * syr);
    const int sidx = SPAIR ? shy * RS + X0 + 2 * l : shy * RS + X0 + sxl;
    const bool hval = !XWRAP && (w == TY - 1) && (l < 2 * HY);
    const int hhy = l >> 1, hside = l & 1;
    const int hx = hside ? wrapi(x0 + 128, nx) : wrapi(x0 - 1, nx);
    const int hyg = wrapi(y0 - 1 + min(hhy, HY - 1), ny);
    const unsigned hoff = (unsigned)(hx + nx * hyg);
    const int hidx = min(hhy, HY - 1) * RS + (hside ? 129 : WAVE ? 128 : 0);
    // B_ext / b_scale of the staged columns
    const float bea[3] = {a.bext[xa] * ib, a.bext[nx + xa] * ib, a.bext[2 * nx + xa] * ib};
    const float beb[3] = {a.bext[xa + 1] * ib, a.bext[nx + xa + 1] * ib, a.bext[2 * nx + xa + 1] * ib};
    const int xs = x0 + sxl;
    const float bes[3] = {a.bext[xs] * ib, a.bext[nx + xs] * ib, a.bext[2 * nx + xs] * ib};
    const float hbe[3] = {a.bext[hx] * ib, a.bext[nx + hx] * ib, a.bext[2 * nx + hx] * ib};
    // QUAD (float32 with XWRAP): staging by 16-byte loads, wave w < HY/2 staging rows 2w (lanes
    // 0 .. 31) and 2w + 1 (lanes 32 .. 63), four cells per lane
    constexpr bool QUAD = XWRAP && std::is_same<TU, float>::value && std::is_same<TB, float>::value;
    const int qhy = min(2 * w + (l >> 5), HY - 1), qxl = 4 * (l & 31);
    const bool qval = QUAD && w < HY / 2;
    const int qyr = wrapi(y0 - 1 + qhy, ny);
    const unsigned qoff = (unsigned)(x0 + qxl + nx * qyr);
    const int qidx = qhy * RS + X0 + qxl;
    float qbe[3][4];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i) qbe[c][i] = QUAD ? a.bext[c * nx + x0 + qxl + i] * ib : 0.0f;
    float4 qu[3], qb[3];
    float tq[3];

    RU ru[3];
    RB rb[3], rq[3];        // pair row (rq: SPLIT hi part)
    std::conditional_t<SPAIR, RU, TU> su[3];
    std::conditional_t<SPAIR, RB, TB> sb[3], sq[3];  // pair of rows TY, TY + 1, or single cell
    TU hu[3];
    TB hb[3], hq[3];        // halo column
    float tp[3], ts[3], th[3];  // BYZ: B_ext (y, z) part at the pair row, single cell, halo column
    const unsigned pyz = (unsigned)ny * nz;
    auto load_plane = [&](int p) {
        const int zz = wrapi(p, nz);
        const unsigned off = (unsigned)zz * plane;
        if constexpr (BYZ) {
            const unsigned op = (unsigned)(pyr + ny * zz), os = (unsigned)(syr + ny * zz), oh = (unsigned)(hyg + ny * zz);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                tp[q] = a.bext_yz[q * pyz + op];
                ts[q] = a.bext_yz[q * pyz + os];
                th[q] = a.bext_yz[q * pyz + oh];
                if constexpr (QUAD) tq[q] = a.bext_yz[q * pyz + (unsigned)(qyr + ny * zz)];
            }
        }
        if constexpr (QUAD) {
            if (qval) {
                const unsigned kq = (off + qoff) * (unsigned)sizeof(float);
                qu[0] = ld_off(reinterpret_cast<const float4 *>(u0), kq);
                qu[1] = ld_off(reinterpret_cast<const float4 *>(u1), kq);
                qu[2] = ld_off(reinterpret_cast<const float4 *>(u2), kq);
                qb[0] = ld_off(reinterpret_cast<const float4 *>(b0), kq);
                qb[1] = ld_off(reinterpret_cast<const float4 *>(b1), kq);
                qb[2] = ld_off(reinterpret_cast<const float4 *>(b2), kq);
            }
        } else {
        {
            const unsigned ku = (off + poff) * (unsigned)sizeof(TU), kb = (off + poff) * (unsigned)sizeof(TB);
            ru[0] = ld_off(reinterpret_cast<const RU *>(u0), ku);
            ru[1] = ld_off(reinterpret_cast<const RU *>(u1), ku);
            ru[2] = ld_off(reinterpret_cast<const RU *>(u2), ku);
            rb[0] = ld_off(reinterpret_cast<const RB *>(b0), kb);
            rb[1] = ld_off(reinterpret_cast<const RB *>(b1), kb);
            rb[2] = ld_off(reinterpret_cast<const RB *>(b2), kb);
            if constexpr (SPLIT) {
                rq[0] = ld_off(reinterpret_cast<const RB *>(bh0), kb);
                rq[1] = ld_off(reinterpret_cast<const RB *>(bh1), kb);
                rq[2] = ld_off(reinterpret_cast<const RB *>(bh2), kb);
            }
        }
        if (sval) {
            using SU = std::conditional_t<SPAIR, RU, TU>;
            using SB = std::conditional_t<SPAIR, RB, TB>;
            const unsigned ku = (off + soff) * (unsigned)sizeof(TU), kb = (off + soff) * (unsigned)sizeof(TB);
            su[0] = ld_off(reinterpret_cast<const SU *>(u0), ku);
            su[1] = ld_off(reinterpret_cast<const SU *>(u1), ku);
            su[2] = ld_off(reinterpret_cast<const SU *>(u2), ku);
            sb[0] = ld_off(reinterpret_cast<const SB *>(b0), kb);
            sb[1] = ld_off(reinterpret_cast<const SB *>(b1), kb);
            sb[2] = ld_off(reinterpret_cast<const SB *>(b2), kb);
            if constexpr (SPLIT) {
                sq[0] = ld_off(reinterpret_cast<const SB *>(bh0), kb);
                sq[1] = ld_off(reinterpret_cast<const SB *>(bh1), kb);
                sq[2] = ld_off(reinterpret_cast<const SB *>(bh2), kb);
            }
        }
        }
        if (hval) {
            const unsigned ku = (off + hoff) * (unsigned)sizeof(TU), kb = (off + hoff) * (unsigned)sizeof(TB);
            hu[0] = ld_off(u0, ku);
            hu[1] = ld_off(u1, ku);
            hu[2] = ld_off(u2, ku);
            hb[0] = ld_off(b0, kb);
            hb[1] = ld_off(b1, kb);
            hb[2] = ld_off(b2, kb);
            if constexpr (SPLIT) {
                hq[0] = ld_off(bh0, kb);
                hq[1] = ld_off(bh1, kb);
                hq[2] = ld_off(bh2, kb);
            }
        }
    };
    // staged: b (stored units) and the flux u_c B_a - u_a B_c with B = b + B_ext
    auto put = [&](int buf, int idx, float bx, float by, float bz, float ux, float uy, float uz, const float *be) {
        const float Bx = bx + be[0], By = by + be[1], Bz = bz + be[2];
        s_pl[buf][0][idx] = bx;
        s_pl[buf][1][idx] = by;
        s_pl[buf][2][idx] = bz;
        if constexpr (F32) {
            sweep_flux(Bx, By, Bz, ux, uy, uz, s_pl[buf][3][idx], s_pl[buf][4][idx], s_pl[buf][5][idx]);
        } else {
            s_pl[buf][3][idx] = uy * Bx - ux * By;
            s_pl[buf][4][idx] = uz * Bx - ux * Bz;
            s_pl[buf][5][idx] = uz * By - uy * Bz;
        }
    };
    auto stage = [&](auto bufc) {
        constexpr int S = decltype(bufc)::value;
        constexpr float us = 1.0f, bs = 1.0f;  // stored units
        if constexpr (QUAD) {
            if (qval) {
                const float ub[3][4] = {{qu[0].x, qu[0].y, qu[0].z, qu[0].w}, {qu[1].x, qu[1].y, qu[1].z, qu[1].w},
                                        {qu[2].x, qu[2].y, qu[2].z, qu[2].w}};
                const float bb[3][4] = {{qb[0].x, qb[0].y, qb[0].z, qb[0].w}, {qb[1].x, qb[1].y, qb[1].z, qb[1].w},
                                        {qb[2].x, qb[2].y, qb[2].z, qb[2].w}};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    float e[3] = {qbe[0][i], qbe[1][i], qbe[2][i]};
                    if constexpr (BYZ) {
#pragma unroll
                        for (int q = 0; q < 3; ++q) e[q] += tq[q] * ib;
                    }
                    put(S, qidx + i, bb[0][i], bb[1][i], bb[2][i], ub[0][i], ub[1][i], ub[2][i], e);
                }
            }
        } else {
        {
            float b[2][3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                b[0][q] = PB::lo(rb[q], bs);
                b[1][q] = PB::hi(rb[q], bs);
                if constexpr (SPLIT) {
                    b[0][q] += PB::lo(rq[q], bs);
                    b[1][q] += PB::hi(rq[q], bs);
                }
            }
            float ea[3] = {bea[0], bea[1], bea[2]}, eb[3] = {beb[0], beb[1], beb[2]};
            if constexpr (BYZ) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    ea[q] += tp[q] * ib;
                    eb[q] += tp[q] * ib;
                }
            }
            const int idx = w * RS + X0 + 2 * l;
            put(S, idx, b[0][0], b[0][1], b[0][2], PU::lo(ru[0], us), PU::lo(ru[1], us), PU::lo(ru[2], us), ea);
            put(S, idx + 1, b[1][0], b[1][1], b[1][2], PU::hi(ru[0], us), PU::hi(ru[1], us), PU::hi(ru[2], us), eb);
        }
        if constexpr (SPAIR) {
            if (sval) {
                float b[2][3];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    b[0][q] = PB::lo(sb[q], bs);
                    b[1][q] = PB::hi(sb[q], bs);
                    if constexpr (SPLIT) {
                        b[0][q] += PB::lo(sq[q], bs);
                        b[1][q] += PB::hi(sq[q], bs);
                    }
                }
                float ea[3] = {bea[0], bea[1], bea[2]}, eb[3] = {beb[0], beb[1], beb[2]};
                if constexpr (BYZ) {
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        ea[q] += ts[q] * ib;
                        eb[q] += ts[q] * ib;
                    }
                }
                put(S, sidx, b[0][0], b[0][1], b[0][2], PU::lo(su[0], us), PU::lo(su[1], us), PU::lo(su[2], us), ea);
                put(S, sidx + 1, b[1][0], b[1][1], b[1][2], PU::hi(su[0], us), PU::hi(su[1], us), PU::hi(su[2], us),
                    eb);
            }
        } else {
            if (sval) {
                float b[3], e[3] = {bes[0], bes[1], bes[2]};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    b[q] = St<TB>::cvt(sb[q]);
                    if constexpr (SPLIT) b[q] += St<TB>::cvt(sq[q]);
                    if constexpr (BYZ) e[q] += ts[q] * ib;
                }
                put(S, sidx, b[0], b[1], b[2], St<TU>::cvt(su[0]), St<TU>::cvt(su[1]), St<TU>::cvt(su[2]), e);
            }
        }
        }
        if (hval) {
            float b[3], e[3] = {hbe[0], hbe[1], hbe[2]};
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                b[q] = St<TB>::cvt(hb[q]);
                if constexpr (SPLIT) b[q] += St<TB>::cvt(hq[q]);
                if constexpr (BYZ) e[q] += th[q] * ib;
            }
            put(S, hidx, b[0], b[1], b[2], St<TU>::cvt(hu[0]), St<TU>::cvt(hu[1]), St<TU>::cvt(hu[2]), e);
        }
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;

    // rolling state of the march, per cell and component: acc = A(p-2) + B(p-1) (the output at
    // p-1 without its C(p) part), ap = A(p-1), cc = b(p-1) at the centre, dz = b(p-1) - b(p-2)
    float acc[2][3] = {}, ap[2][3] = {}, cc[2][3] = {}, dz[2][3] = {};

    load_plane(z0 - 1);
    stage(I0{});
    load_plane(z0);
    __syncthreads();
    auto body = [&](auto par, int p) {
        constexpr int P = decltype(par)::value;
        using Q = std::integral_constant<int, 1 - P>;
        if (p < z1) {
            stage(Q{});
            if (p + 2 <= z1) load_plane(p + 2);
        }
        // SPLIT: stored lo (and, re-splitting, hi) of the output pair, requested now
        const unsigned ko_ = ((unsigned)(p - 1) * plane + (unsigned)(xa + nx * gy)) * (unsigned)sizeof(TB);
        RB lc[3], hc[3];
        if constexpr (SPLIT) {
            if (own && p >= z0 + 1) {
                lc[0] = ld_off(reinterpret_cast<const RB *>(b0), ko_);
                lc[1] = ld_off(reinterpret_cast<const RB *>(b1), ko_);
                lc[2] = ld_off(reinterpret_cast<const RB *>(b2), ko_);
                if (resplit) {
                    hc[0] = ld_off(reinterpret_cast<const RB *>(bh0), ko_);
                    hc[1] = ld_off(reinterpret_cast<const RB *>(bh1), ko_);
                    hc[2] = ld_off(reinterpret_cast<const RB *>(bh2), ko_);
                }
            }
        }
        if (own) {
            // Plane p's contributions to the outputs at p+1 (A = S + P), p (B) and p-1
            // (C = S - P) of both cells: S and B collect the in-plane sums, P the flux through
            // the planes (components x, y; zero for z, so A = C there).
            float S[2][3], B[2][3], Pz[2][2], cen[2][3];
            // without WAVE: rows y-1, y, y+1 of a field at columns xa-1 .. xa+2 (two aligned 8-byte reads per row)
            auto rows = [&](int k, float (&v)[3][4]) {
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const float *row = &s_pl[P][k][(w + r) * RS + 2 * l];
                    if constexpr (XWRAP) {
                        const float2 c = *reinterpret_cast<const float2 *>(row);
                        v[r][0] = wave_ror1(c.y);
                        v[r][1] = c.x;
                        v[r][2] = c.y;
                        v[r][3] = wave_rol1(c.x);
                    } else {
                        const float2 lo = *reinterpret_cast<const float2 *>(row);
                        const float2 hi = *reinterpret_cast<const float2 *>(row + 2);
                        v[r][0] = lo.x;
                        v[r][1] = lo.y;
                        v[r][2] = hi.x;
                        v[r][3] = hi.y;
                    }
                }
            };
            float out[2][3];
            if constexpr (F32 && !WAVE) {
                plane_terms<2, Q27>(columns_rows<2>(rows), W, S, B, Pz, cen);
                march.take(W, S, B, Pz, cen, out);
            } else if constexpr (F32) {
                auto cells = [&](int k, float (&v)[3][2]) {
#pragma unroll
                    for (int r = 0; r < 3; ++r) {
                        const float2 c = *reinterpret_cast<const float2 *>(&s_pl[P][k][(w + r) * RS + 2 * l]);
                        v[r][0] = c.x;
                        v[r][1] = c.y;
                    }
                };
                auto end = [&](int k, float (&h)[3]) {
#pragma unroll
                    for (int r = 0; r < 3; ++r) h[r] = s_pl[P][k][(w + r) * RS + 128 + (l >> 5)];
                };
                plane_terms<2, Q27>(columns_wave<2, !XWRAP>(cells, end), W, S, B, Pz, cen);
                march.take(W, S, B, Pz, cen, out);
            } else {
            // b components: face and corner sums of differences to each centre, taken against
            // the first centre r0 and shifted by 4 (c1 - r0) for the second cell; the column
            // sums t_j of rows y-1 and y+1 serve both cells
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                float v[3][4];
                rows(k, v);
                const float r0 = v[1][1];
                float d[3][4];
#pragma unroll
                for (int r = 0; r < 3; ++r)
#pragma unroll
                    for (int j = 0; j < 4; ++j) d[r][j] = v[r][j] - r0;
                const float dl = d[1][2];  // c1 - c0
                const float t0 = d[0][0] + d[2][0], t1 = d[0][1] + d[2][1], t2 = d[0][2] + d[2][2],
                            t3 = d[0][3] + d[2][3];
                const float fs0 = (d[1][0] + dl) + t1, cs0 = t0 + t2;
                const float fs1 = fmaf(-4.0f, dl, d[1][3] + t2), cs1 = fmaf(-4.0f, dl, t1 + t3);
                cen[0][k] = r0;
                cen[1][k] = v[1][2];
                B[0][k] = fmaf(b0c, cs0, b0f * fs0);
                B[1][k] = fmaf(b0c, cs1, b0f * fs1);
                S[0][k] = b1f * fs0;
                S[1][k] = b1f * fs1;
                if constexpr (Q27) {
                    S[0][k] = fmaf(b1k, cs0, S[0][k]);
                    S[1][k] = fmaf(b1k, cs1, S[1][k]);
                }
            }
            {  // flux xy: in-plane differences along x (component y) and along y (component x)
                float v[3][4];
                rows(3, v);
                float q[4], s[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    q[j] = v[0][j] - v[2][j];
                    s[j] = v[0][j] + v[2][j];
                }
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float dx = v[1][e] - v[1][e + 2], cdx = s[e] - s[e + 2];
                    const float dy = q[1 + e], cdy = q[e] + q[e + 2];
                    B[e][0] = fmaf(l0c, cdy, fmaf(l0f, dy, B[e][0]));
                    S[e][0] = fmaf(l1f, dy, S[e][0]);
                    B[e][1] = fmaf(-l0c, cdx, fmaf(-l0f, dx, B[e][1]));
                    S[e][1] = fmaf(-l1f, dx, S[e][1]);
                    if constexpr (Q27) {
                        S[e][0] = fmaf(l1k, cdy, S[e][0]);
                        S[e][1] = fmaf(-l1k, cdx, S[e][1]);
                    }
                }
            }
            {  // flux xz: through-plane sum (component x) and differences along x (component z)
                float v[3][4];
                rows(4, v);
                float s[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) s[j] = v[0][j] + v[2][j];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float dx = v[1][e] - v[1][e + 2], cdx = s[e] - s[e + 2];
                    float pz = fmaf(l1c, v[1][1 + e], l1f * ((v[1][e] + v[1][e + 2]) + s[1 + e]));
                    if constexpr (Q27) pz = fmaf(l1k, s[e] + s[e + 2], pz);
                    Pz[e][0] = pz;
                    B[e][2] = fmaf(-l0c, cdx, fmaf(-l0f, dx, B[e][2]));
                    S[e][2] = fmaf(-l1f, dx, S[e][2]);
                    if constexpr (Q27) S[e][2] = fmaf(-l1k, cdx, S[e][2]);
                }
            }
            {  // flux yz: through-plane sum (component y) and differences along y (component z)
                float v[3][4];
                rows(5, v);
                float q[4], s[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    q[j] = v[0][j] - v[2][j];
                    s[j] = v[0][j] + v[2][j];
                }
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float dy = q[1 + e], cdy = q[e] + q[e + 2];
                    float pz = fmaf(l1c, v[1][1 + e], l1f * ((v[1][e] + v[1][e + 2]) + s[1 + e]));
                    if constexpr (Q27) pz = fmaf(l1k, s[e] + s[e + 2], pz);
                    Pz[e][1] = pz;
                    B[e][2] = fmaf(-l0c, cdy, fmaf(-l0f, dy, B[e][2]));
                    S[e][2] = fmaf(-l1f, dy, S[e][2]);
                    if constexpr (Q27) S[e][2] = fmaf(-l1k, cdy, S[e][2]);
                }
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    // output plane p-1: b* = b_c + increment, the increment built from
                    // differences only; C = S - P (P = 0 for z)
                    const float Ck = k < 2 ? S[e][k] - Pz[e][k] : S[e][k];
                    const float dzc = cen[e][k] - cc[e][k];  // b(p) - b(p-1)
                    out[e][k] = fmaf(w6, dzc - dz[e][k], acc[e][k] + Ck);
                    if constexpr (!SPLIT) out[e][k] += cc[e][k];
                    const float Ak = k < 2 ? S[e][k] + Pz[e][k] : S[e][k];
                    acc[e][k] = ap[e][k] + B[e][k];
                    ap[e][k] = Ak;
                    cc[e][k] = cen[e][k];
                    dz[e][k] = dzc;
                }
            }
            }
            if (p >= z0 + 1) {
                RB *oo[3] = {reinterpret_cast<RB *>(o0), reinterpret_cast<RB *>(o1), reinterpret_cast<RB *>(o2)};
                if constexpr (SPLIT) {
                    // out holds the increments: lo* = lo + increment, or a re-split of hi + lo + increment
                    RB *ho = reinterpret_cast<RB *>(a.bho);
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        constexpr float bs = 1.0f, inv = 1.0f;  // stored units
                        const float l0 = PB::lo(lc[q], bs), l1 = PB::hi(lc[q], bs);
                        if (resplit) {
                            const float v0 = (PB::lo(hc[q], bs) + l0) + out[0][q];
                            const float v1 = (PB::hi(hc[q], bs) + l1) + out[1][q];
                            const RB hn = PB::make(v0, v1, inv);
                            st_off(ho + q * (size_t)(N / 2), ko_, hn);
                            st_off(oo[q], ko_, PB::make(v0 - PB::lo(hn, bs), v1 - PB::hi(hn, bs), inv));
                        } else {
                            st_off(oo[q], ko_, PB::make(l0 + out[0][q], l1 + out[1][q], inv));
                        }
                    }
                } else if constexpr (std::is_same<TB, float>::value) {
                    // float32 pairs go out as agent-scope relaxed atomic stores, which write through
                    // the L2 (the same values; measured in the step: 128^3 sweep 17.6 -> 16.6-17.1
                    // us, 512 x 256^2 270.2 -> 268.4 us, the 64-pipe batch unchanged)
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const RB v = PB::make(out[0][q], out[1][q], 1.0f);
                        unsigned long long bits;
                        __builtin_memcpy(&bits, &v, 8);
                        __hip_atomic_store(reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(oo[q]) + ko_),
                                           bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
                } else {
                    st_off(oo[0], ko_, PB::make(out[0][0], out[1][0], 1.0f));
                    st_off(oo[1], ko_, PB::make(out[0][1], out[1][1], 1.0f));
                    st_off(oo[2], ko_, PB::make(out[0][2], out[1][2], 1.0f));
                }
            }
        }
        __syncthreads();
    };
    for (int p = z0 - 1; p <= z1; p += 2) {
        body(I0{}, p);
        if (p + 1 <= z1) body(I1{}, p + 1);
    }
}

// The halo form (without the six-magnet table) is held to three waves per SIMD (at most 168
// VGPRs, no spills), so that three 4-row workgroups share a CU on large boxes instead of two: the
// 16-bit forms' steps on 512 x 256 x 256 then run 5-6% faster and the float32 64-pipe batch 5%.
// The single-box float32 form is left unbounded (the bound made its step 0.4% slower).
template <int TY, typename TU, typename TB, bool BATCH, bool SPLIT, bool BYZ, bool Q27, bool XWRAP, bool FEW>
__global__ void __launch_bounds__(64 * TY)
__attribute__((amdgpu_waves_per_eu(XWRAP || BYZ || FEW || (std::is_same<TB, float>::value && !BATCH) ? 1 : 3)))
k_mag_sweep_pair(SweepArgs a, const PipeStep *tab, const BlockMap *map, int which, int nbatch) {
    __shared__ __align__(16) float lds[kPairLds<TY>];
    const int lb = sweep_tile<BATCH>(a, tab, map, which, nbatch);
    if (lb >= 0) sweep_pairs<TY, TU, TB, SPLIT, BYZ, Q27, XWRAP, FEW>(a, lb, lds);
}

// float32 boxes of a batch with different tile forms in one launch (256 work-items in each form):
// launched form by form, every launch has its own first loads and its own last wave, and the groups
// of few boxes leave CUs idle. The form is the box's, so a workgroup takes one branch. 16 pipes of
// 32 to 256 planes, radii 16 to 64, three forms: a step and its read back 355 -> 346 ms (six steps).
template <bool BYZ, bool Q27>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(BYZ ? 1 : 3)))
k_mag_sweep_mixed(const PipeStep *tab, const BlockMap *map, int which, int nbatch) {
    __shared__ __align__(16) float lds[kPairLds<4>];
    static_assert(kPairLds<4> >= kSweepLds<64, 4> && kPairLds<4> >= kSweepLds<32, 8> &&
                      kPairLds<4> >= kSweepLds<16, 16> && kPairLds<4> >= kSweepLds<8, 32>,
                  "one buffer for every form");
    SweepArgs a;
    const int lb = sweep_tile<true>(a, tab, map, which, nbatch);
    if (lb < 0) return;
    switch (a.tile_x) {
        case 128: sweep_pairs<4, float, float, false, BYZ, Q27, false>(a, lb, lds); break;
        case 64: sweep_cells<64, 4, float, float, false, BYZ, Q27>(a, lb, lds); break;
        case 32: sweep_cells<32, 8, float, float, false, BYZ, Q27>(a, lb, lds); break;
        case 16: sweep_cells<16, 16, float, float, false, BYZ, Q27>(a, lb, lds); break;
        default: sweep_cells<8, 32, float, float, false, BYZ, Q27>(a, lb, lds); break;
    }
}


// ===========================================================================================
// Host-side launchers of the sweep
// ===========================================================================================
SweepArgs make_sweep_args(const void *u, const void *b, void *bo, const float *bext, StepConst c, SweepLaunch L) {
    SweepArgs a;
    a.u = u;
    a.b = b;
    a.bo = bo;
    a.bh = nullptr;
    a.bho = nullptr;
    a.bext = bext;
    a.bext_yz = nullptr;
    a.q27 = c.lattice == 27;
    a.nx = c.nx;
    a.ny = c.ny;
    a.nz = c.nz;
    const bool pair = L.pair && c.nx % 128 == 0;
    const int tx = pair ? 128 : L.tx;
    const int ty = pair ? (L.ty >= 8 ? 8 : 4) : 256 / L.tx;
    a.tile_x = tx;
    a.tiles_x = (c.nx + tx - 1) / tx;
    a.tiles_y = (c.ny + ty - 1) / ty;
    a.zchunk = L.zchunk;
    a.nzc = (c.nz + L.zchunk - 1) / L.zchunk;
    a.nblocks = a.tiles_x * a.tiles_y * a.nzc;
    a.kappa = c.kappa;
    a.u_scale = c.u_scale;
    a.b_scale = c.b_scale;
    a.inv_b_scale = c.inv_b_scale;
    a.omega = c.omega;
    return a;
}

// grid of a sweep launch: a multiple of 8 so the XCD-aware remap is a permutation
static inline unsigned sweep_grid(int nblocks) { return (unsigned)(((nblocks + 7) / 8) * 8); }

// Sweeps are launched through hipExtLaunchKernelGGL: when profiling, its start / stop events
// are stamped when the kernel itself starts and ends (no event packets around the launch).
template <typename TU, typename TB, bool BATCH, bool SPLIT, bool BYZ, bool Q27, bool FEW>
static hipError_t sweep_form(hipStream_t s, const SweepArgs &a, SweepLaunch L, const PipeStep *tab,
                             const BlockMap *map, int which, int nblocks, hipEvent_t e0, hipEvent_t e1) {
    const dim3 grid(sweep_grid(nblocks));
    if (L.pair) {
        if constexpr (!BATCH) {
            if (a.nx == 128) {  // one tile per row: x neighbours by wave rotation
                if constexpr (!std::is_same<TB, float>::value)
                    if (L.ty >= 8) {
                        hipExtLaunchKernelGGL(k_mag_sweep_pair<8, TU, TB, false, SPLIT, BYZ, Q27, true, false>, grid, dim3(512), 0, s, e0,
                                              e1, 0, a, tab, map, which, nblocks);
                        return hipGetLastError();
                    }
                hipExtLaunchKernelGGL(k_mag_sweep_pair<4, TU, TB, false, SPLIT, BYZ, Q27, true, false>, grid, dim3(256), 0, s, e0, e1, 0, a,
                                      tab, map, which, nblocks);
                return hipGetLastError();
            }
        }
        if constexpr (!std::is_same<TB, float>::value)
            if (L.ty >= 8) {
                hipExtLaunchKernelGGL(k_mag_sweep_pair<8, TU, TB, BATCH, SPLIT, BYZ, Q27, false, false>, grid, dim3(512), 0, s, e0, e1, 0, a,
                                      tab, map, which, nblocks);
                return hipGetLastError();
            }
        hipExtLaunchKernelGGL(k_mag_sweep_pair<4, TU, TB, BATCH, SPLIT, BYZ, Q27, false, FEW>, grid, dim3(256), 0, s, e0, e1, 0, a, tab, map,
                              which, nblocks);
        return hipGetLastError();
    }
    switch (L.tx) {
        case 64:
            hipExtLaunchKernelGGL(k_mag_sweep<64, 4, TU, TB, BATCH, SPLIT, BYZ, Q27, FEW>, grid, dim3(256), 0, s, e0, e1, 0, a, tab, map,
                                  which, nblocks);
            break;
        case 32:
            hipExtLaunchKernelGGL(k_mag_sweep<32, 8, TU, TB, BATCH, SPLIT, BYZ, Q27, FEW>, grid, dim3(256), 0, s, e0, e1, 0, a, tab, map,
                                  which, nblocks);
            break;
        case 16:
            hipExtLaunchKernelGGL(k_mag_sweep<16, 16, TU, TB, BATCH, SPLIT, BYZ, Q27, FEW>, grid, dim3(256), 0, s, e0, e1, 0, a, tab,
                                  map, which, nblocks);
            break;
        default:
            hipExtLaunchKernelGGL(k_mag_sweep<8, 32, TU, TB, BATCH, SPLIT, BYZ, Q27, FEW>, grid, dim3(256), 0, s, e0, e1, 0, a, tab, map,
                                  which, nblocks);
            break;
    }
    return hipGetLastError();
}

// FEW: float32 launches whose workgroups all find a place at once. There the latency of a plane's chain
// counts, and it is shorter where every lane reads its neighbours' columns and nothing bounds the
// registers; beyond that, fewer reads and another workgroup on a CU count more. The unbounded forms hold
// three workgroups of single cells on a CU (against four) and two of pairs (against three), so the line is
// at 768 and 512 workgroups; pairs of 769 to 1024 take two rounds either way. Per sweep, many-form
// against this: 64 x 90 x 90 (276) 12.8 -> 11.7 us, 64 x 128 x 128 (512) 13.4 -> 12.2, 64 x 150 x 150 (722)
// 15.7 -> 15.1, but 100 x 112 x 112 (784) 18.1 -> 21.2; pairs 256 x 80 x 80 (400) 16.7 -> 15.9, 512 x 80 x
// 80 (800) 30.4 -> 29.9, but 256 x 100 x 100 (650) 21.2 -> 27.9.
static bool few_workgroups(bool pair, int n) { return pair ? n <= 512 || (n > 768 && n <= 1024) : n <= 768; }

template <typename TU, typename TB, bool BATCH, bool SPLIT, bool BYZ, bool Q27>
static hipError_t sweep_typed(hipStream_t s, const SweepArgs &a, SweepLaunch L, const PipeStep *tab,
                              const BlockMap *map, int which, int nblocks, hipEvent_t e0, hipEvent_t e1) {
    if constexpr (std::is_same<TB, float>::value)
        if (few_workgroups(L.pair, nblocks))
            return sweep_form<TU, TB, BATCH, SPLIT, BYZ, Q27, true>(s, a, L, tab, map, which, nblocks, e0, e1);
    return sweep_form<TU, TB, BATCH, SPLIT, BYZ, Q27, false>(s, a, L, tab, map, which, nblocks, e0, e1);
}

template <bool BATCH, bool BYZ>
static hipError_t sweep_kinds_yz(hipStream_t s, int kinds, const SweepArgs &a, SweepLaunch L, const PipeStep *tab,
                                 const BlockMap *map, int which, int nblocks, hipEvent_t e0, hipEvent_t e1) {
    const int ku = (kinds >> 4) & 15, kb = (kinds >> 8) & 15;
    // float32 tiles of 8 rows have a kernel of their own; those of 4 rows are faster here (both measured
    // there)
    if (!L.mixed && L.pair && L.ty >= 8 && ku == MHD_KIND_F32 && kb == MHD_KIND_F32)
        return launch_sweep_rows(s, BATCH, a, L, tab, map, which, nblocks, e0, e1);
    if constexpr (BATCH) {
        if (L.mixed) {
            const dim3 grid(sweep_grid(nblocks));
            if (L.q27)
                hipExtLaunchKernelGGL(k_mag_sweep_mixed<BYZ, true>, grid, dim3(256), 0, s, e0, e1, 0, tab, map, which, nblocks);
            else
                hipExtLaunchKernelGGL(k_mag_sweep_mixed<BYZ, false>, grid, dim3(256), 0, s, e0, e1, 0, tab, map, which, nblocks);
            return hipGetLastError();
        }
    }
    if (L.q27) {  // D3Q27: float32 and the split form
        if (ku == MHD_KIND_F32 && kb == MHD_KIND_F32)
            return sweep_typed<float, float, BATCH, false, BYZ, true>(s, a, L, tab, map, which, nblocks, e0, e1);
        if (ku == MHD_KIND_F32 && kb == MHD_KIND_F16_SPLIT)
            return sweep_typed<__half, __half, BATCH, true, BYZ, true>(s, a, L, tab, map, which, nblocks, e0, e1);
        return hipErrorInvalidValue;
    }
    if (ku == MHD_KIND_F32 && kb == MHD_KIND_F32)
        return sweep_typed<float, float, BATCH, false, BYZ, false>(s, a, L, tab, map, which, nblocks, e0, e1);
    if (ku == MHD_KIND_F16 && kb == MHD_KIND_F16)
        return sweep_typed<__half, __half, BATCH, false, BYZ, false>(s, a, L, tab, map, which, nblocks, e0, e1);
    if (ku == MHD_KIND_BF16 && kb == MHD_KIND_F16)
        return sweep_typed<__hip_bfloat16, __half, BATCH, false, BYZ, false>(s, a, L, tab, map, which, nblocks, e0,
                                                                             e1);
    if (ku == MHD_KIND_BF16 && kb == MHD_KIND_BF16)
        return sweep_typed<__hip_bfloat16, __hip_bfloat16, BATCH, false, BYZ, false>(s, a, L, tab, map, which, nblocks,
                                                                                     e0, e1);
    if (ku == MHD_KIND_F32 && kb == MHD_KIND_F16_SPLIT)  // reads the float16 copy of u
        return sweep_typed<__half, __half, BATCH, true, BYZ, false>(s, a, L, tab, map, which, nblocks, e0, e1);
    return hipErrorInvalidValue;
}
template <bool BATCH>
static hipError_t sweep_kinds(hipStream_t s, int kinds, const SweepArgs &a, SweepLaunch L, const PipeStep *tab,
                              const BlockMap *map, int which, int nblocks, hipEvent_t e0, hipEvent_t e1) {
    if (L.byz) return sweep_kinds_yz<BATCH, true>(s, kinds, a, L, tab, map, which, nblocks, e0, e1);
    return sweep_kinds_yz<BATCH, false>(s, kinds, a, L, tab, map, which, nblocks, e0, e1);
}

hipError_t launch_mag_sweep(hipStream_t s, int kinds, const SweepArgs &a0, SweepLaunch L, hipEvent_t e0,
                            hipEvent_t e1) {
    L.pair = L.pair && a0.nx % 128 == 0;
    L.byz = a0.bext_yz != nullptr;
    L.q27 = a0.q27;
    return sweep_kinds<false>(s, kinds, a0, L, nullptr, nullptr, 0, a0.nblocks, e0, e1);
}

hipError_t launch_mag_sweep_batch(hipStream_t s, int kinds, SweepLaunch L, const PipeStep *tab, const BlockMap *map,
                                  int which, int nblocks, hipEvent_t e0, hipEvent_t e1) {
    if (nblocks <= 0) return hipSuccess;
    return sweep_kinds<true>(s, kinds, SweepArgs{}, L, tab, map, which, nblocks, e0, e1);
}

}  // namespace mhd
