// The whole magnetic iteration of a fluid step (n_mag sweeps, each followed by the b wall
// correction) in one launch, for float32 boxes whose fields fit the chip's LDS and whose wall, if
// any, is made of lines along x.
//
// What bounds small boxes is the chain of launches: a sweep, an interpolation and a spreading are
// 16 us per iteration on 8 x 32 x 32 as on 32^3, whatever the cells. Here a workgroup owns the rows
// (x lines, or TX cells of them with a halo column at each end) of a TY x TZ tile of the
// cross-section and keeps their b in LDS and u in registers for all n_mag sweeps. Per iteration it
// sweeps its rows, writes those that other tiles read as b* (uncorrected) to the buffer of b that the
// iteration's parity names, raises its flag, waits for the flags of the tiles it exchanges with,
// reads the halo rows and the rows its markers' taps need, and corrects tile and halo rows from LDS.
// Only that exchange goes through memory: 1.9 us a round for up to 4 KB a workgroup and any number of
// workgroups (against 3.8 us and more for a barrier over the whole grid).
//
// Per iteration, launch sequence against this: 8 x 32 x 32 15.3 -> 3.8 us, 32^3 14.8 -> 4.4, 5 x 83 x 83
// 17.2 -> 4.1, 100 x 75 x 75 (D3Q27) 20.0 -> 11.3, 160 x 39 x 39 16.8 -> 8.3, 192 x 70 x 70 (941 k cells,
// all the LDS) 21.1 -> 14.9; a step's start and end add 7 to 25 us, so few sweeps are launched one by
// one (resident_min_sweeps). Cut along x, a box that is long and narrow fills the CUs: 32^3 in 64
// workgroups of whole rows took 6.0 us, in 256 5.0 (with the columns formed anew in every lane).
//
// The exchange needs no cache maintenance: exported rows and flags are written with agent-scope
// (write-through) stores and read with agent-scope loads, and a workgroup waits for its stores
// (s_waitcnt and a workgroup barrier) before it raises its flag. A buffer is overwritten two
// iterations later, by when every reader has raised a later flag (the exchange lists are symmetric).
//
// Waiting workgroups must all be on the chip, which an ordinary launch does not promise when other
// work holds CUs. The launch therefore begins with a roll call: each workgroup counts itself in;
// the last one to arrive turns the state from "counting" to "go", and one that has waited
// roll_ticks turns it to "given up" instead, by compare-and-swap, so all agree. After "go" every
// workgroup is resident and each wait ends; after "given up" all leave with b untouched, and the
// launch that follows on the stream, the stand-in, does the iteration; it leaves at once after "go".
//
// The stand-in needs no more of its workgroups on the chip than one. They take the tiles' turns (an
// iteration of a tile) from a counter, iteration by iteration, wait for the tile's neighbours to have
// had their turns of the iteration before, and take the tile from memory to memory. A turn waits for
// turns of lower numbers only, which running workgroups have taken, so every wait ends however few
// there are. A roll call given up is remembered for kResHoldSteps steps, which go to the stand-in at
// once, and counted in host memory, where the next step calls see it and launch their sweeps one by
// one for a while (ResidentCall, mhd_runtime.cpp): so a GPU that other work keeps busy costs one
// roll call, not one a step. A step of 12 sweeps in the stand-in (in it as one workgroup that took
// every tile before; resident): 8 x 32 x 32 100 us (2.7 ms; 81 us), 32^3 122 us (11.8 ms; 91 us),
// 192 x 70 x 70 335 us (43 ms; 273 us).
//
// The arithmetic per cell is that of the other float32 kernels (mhd_sweep_math.h, and the wall
// correction's sums in the same order), so the fields are the same bit for bit.
#include <hip/hip_runtime.h>

#include "mhd_device.h"
#include "mhd_resident.h"
#include "mhd_sweep_math.h"

namespace mhd {

namespace {

__device__ __forceinline__ float ld_agent(const float *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(float *p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_agent(const int *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A value the compiler may not derive addresses from ahead of time: the addresses of all rows and
// planes of an iteration, hoisted out of it, would take more registers than there are.
__device__ __forceinline__ int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// Roll call; true if every workgroup of the grid is resident. Thread 0's answer, for all.
__device__ __forceinline__ bool roll_call(int *sync, int nwg, long long ticks, int *answer) {
    if (threadIdx.x == 0) {
        int *state = sync + kResState;  // kResHeld from the start: no roll call
        const int before = __hip_atomic_fetch_add(sync + kResCount, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int expect = kResCounting;
        if (ticks < 0)  // never resident (tests of the fallback)
            __hip_atomic_compare_exchange_strong(state, &expect, kResGivenUp, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        else if (before == nwg - 1)
            __hip_atomic_compare_exchange_strong(state, &expect, kResGo, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
        const long long t0 = wall_clock64();
        int s;
        while ((s = ld_agent(state)) == kResCounting) {
            if (wall_clock64() - t0 > ticks) {
                expect = kResCounting;
                __hip_atomic_compare_exchange_strong(state, &expect, kResGivenUp, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
            }
            __builtin_amdgcn_s_sleep(1);
        }
        *answer = s;
    }
    __syncthreads();
    return *answer == kResGo;
}

}  // namespace

// NS: staged rows (tile and halo) per work-item, CZ: cells of a z column per work-item. A work-item
// keeps one x for the whole iteration and takes rows tr, tr + RS, ... of every list.
template <int NS, int CZ, bool Q27, bool STAND_IN>
__global__ void __launch_bounds__(kResMaxThreads) k_mag_resident(ResArgs a) {
    extern __shared__ __align__(16) float lds[];
    __shared__ int s_state;
    const int t = threadIdx.x, NT = blockDim.x;
    if constexpr (STAND_IN) {
        if (ld_agent(a.sync + kResState) == kResGo) return;  // the launch before this one has done the iteration
    } else {
        if (!roll_call(a.sync, a.nwg, a.roll_ticks, &s_state)) return;
    }

    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int64_t N = (int64_t)nx * ny * nz;
    // local columns: the tile's, between its two halo columns where the box is cut along x (xh = 1); a
    // whole row wraps onto itself (xh = 0)
    const int LW = a.lw, xh = a.gx > 1 ? 1 : 0;
    const int RS = NT / LW, tr0 = t / LW < RS ? t / LW : kResNoRow, xt = t % LW;
    const int PY = a.ty + 2;                 // local row slot = hy + PY hz, then the extra rows
    const int GR = PY * (a.tz + 2);          // rows of tile and halo
    // LDS, three components of a cell side by side (few addresses, and lanes on consecutive words)
    float *sb = lds;                         // [slots][LW][3] b
    float *sl = sb + 3 * a.slots * LW;       // [GR][LW][3] flux; reused for the corrections [mk][LW][3]
    float *syz = sl + 3 * max(GR, a.mk_max) * LW;  // [GR][3] (y, z) part of B_ext
    // this tile's table, 16-byte aligned as its entries are
    int *stab = (int *)lds + ((3 * (a.slots * LW + max(GR, a.mk_max) * LW + GR) + 3) & ~3);
    const SweepWeights W = sweep_weights<Q27>(a.kappa, a.omega);
    float be0, be1, be2;

    // the tile: first row and column, rows in y and z, columns, and this work-item's column of the box
    int y0 = 0, z0 = 0, th = 0, tw = 0, wx = 0, cx = 0;
    float u[NS][3];

    // the tile's table to LDS, u of its staged cells to registers (0 where there is no cell)
    auto setup = [&](int tile) {
        const int x = opaque(xt), tr = opaque(tr0);
        __syncthreads();
        const int tix = tile % a.gx, tyz = tile / a.gx;
        const int *src = a.tab + a.tab_off[tyz];
        const int len = a.tab_off[tyz + 1] - a.tab_off[tyz];
        for (int k = t; k < len; k += NT) stab[k] = src[k];
        y0 = (tyz % a.gy) * a.ty;
        z0 = (tyz / a.gy) * a.tz;
        th = min(a.ty, ny - y0);
        tw = min(a.tz, nz - z0);
        wx = min(a.tx, nx - tix * a.tx);
        cx = wrapi(tix * a.tx - xh + x, nx);
        be0 = a.bext[cx];
        be1 = a.bext[nx + cx];
        be2 = a.bext[2 * nx + cx];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int slot = tr + s * RS, hz = slot / PY, hy = slot - hz * PY;
            u[s][0] = u[s][1] = u[s][2] = 0.0f;
            if (slot < GR && hy < th + 2 && hz < tw + 2) {
                const int64_t row = wrapi(y0 - 1 + hy, ny) + (int64_t)ny * wrapi(z0 - 1 + hz, nz);
#pragma unroll
                for (int c = 0; c < 3; ++c) u[s][c] = a.u[c * N + cx + nx * row];
                if (a.bext_yz && x == 0)
                    for (int c = 0; c < 3; ++c) syz[3 * slot + c] = a.bext_yz[c * (int64_t)ny * nz + row];
            }
        }
        __syncthreads();
    };
    auto tab_hdr = [&](int k) { return stab[k]; };

    // rows of the list (halo and extra rows) from buffer src; own: the tile's rows as well
    // kBatch rows a work-item are in flight at once: the reads are a microsecond from the memory side
    constexpr int kBatch = 6;
    auto load_rows = [&](const float *src, bool own) {
        const int x = opaque(xt), tr = opaque(tr0);
        // the tile's own rows: all, or only the halo columns of them; nothing beyond the columns of a
        // shorter last tile, whose work-items still come to the barrier below as all do
        const bool edge = xh && (x == 0 || x == wx + 1);
        const int nl = tab_hdr(kResNLoad), n = x < wx + 2 * xh ? nl + (own || edge ? th * tw : 0) : 0;
        const int *list = stab + tab_hdr(kResOLoad);
        for (int r0 = tr; r0 < n; r0 += kBatch * RS) {
            float v[kBatch][3];
            int to[kBatch];
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const int r = r0 + q * RS;
                to[q] = -1;
                if (r < n) {
                    int at;
                    if (r < nl) {
                        const int2 e = *reinterpret_cast<const int2 *>(list + 2 * r);
                        to[q] = e.x;
                        at = e.y;
                    } else {
                        const int lz = (r - nl) / th, ly = (r - nl) - lz * th;
                        to[q] = 3 * LW * (ly + 1 + PY * (lz + 1));
                        at = nx * (y0 + ly + ny * (z0 + lz));
                    }
                    const float *p = src + (cx + at);
                    v[q][0] = ld_agent(p);
                    v[q][1] = ld_agent(p + N);
                    v[q][2] = ld_agent(p + 2 * N);
                }
            }
#pragma unroll
            for (int q = 0; q < kBatch; ++q)
                if (to[q] >= 0) {
                    float *d = sb + to[q] + 3 * x;
                    d[0] = v[q][0];
                    d[1] = v[q][1];
                    d[2] = v[q][2];
                }
        }
        __syncthreads();
    };

    // wall correction of tile and halo rows in LDS (k_ib_interp and k_ib_spread's sums)
    // (s, wall values) of the work-item's first marker, requested ahead of the wait for the neighbours
    float pre[4];
    auto marker_data = [&](int line, float (&d)[4]) {
        const int64_t j = (int64_t)line * nx + cx;
        d[0] = a.sj[j];
        d[1] = a.wall[j];
        d[2] = a.wall[a.M + j];
        d[3] = a.wall[2 * a.M + j];
    };
    auto request = [&]() {
        if (tr0 < tab_hdr(kResNMk)) marker_data(stab[tab_hdr(kResOMk) + tr0 * kResMkInts + kResTaps], pre);
    };
    // Table entries are fixed in length and 16-byte aligned, so that an entry's reads, and then the
    // field reads they address, are each issued together: two LDS latencies a marker or row.
    auto correct = [&]() {
        const int nm = tab_hdr(kResNMk), nc = tab_hdr(kResNCor);
        if (nm == 0) return;
        const int x = opaque(xt), tr = opaque(tr0);
        const int *mk = stab + tab_hdr(kResOMk), *cor = stab + tab_hdr(kResOCor);
        for (int m = tr; m < nm; m += RS) {
            int e[kResMkInts];
#pragma unroll
            for (int i = 0; i < kResMkInts; i += 4)
                *reinterpret_cast<int4 *>(e + i) = *reinterpret_cast<const int4 *>(mk + m * kResMkInts + i);
            float sw[4] = {pre[0], pre[1], pre[2], pre[3]};
            if (m != tr0) marker_data(e[kResTaps], sw);
            float I0 = 0.f, I1 = 0.f, I2 = 0.f;
#pragma unroll
            for (int i = 0; i < kResTaps; ++i) {
                const float *q = sb + e[i] + 3 * x;
                const float w = __int_as_float(e[kResTaps + 1 + i]);
                I0 = fmaf(w, q[0], I0);
                I1 = fmaf(w, q[1], I1);
                I2 = fmaf(w, q[2], I2);
            }
            float *d = sl + 3 * (m * LW + x);
            d[0] = sw[0] * (sw[1] - I0);
            d[1] = sw[0] * (sw[2] - I1);
            d[2] = sw[0] * (sw[3] - I2);
        }
        __syncthreads();
        const int km4 = a.km4, len = 2 * km4 + 4;  // entries in groups of four
        for (int r = tr; r < nc; r += RS) {
            const int *e = cor + r * len;
            float *q = sb + e[2 * km4] + 3 * x;
            const float v0 = q[0], v1 = q[1], v2 = q[2];
            float c0 = 0.f, c1 = 0.f, c2 = 0.f;
            for (int i = 0; i < km4; i += 4) {
                const int4 j = *reinterpret_cast<const int4 *>(e + i);
                const float4 w = *reinterpret_cast<const float4 *>(e + km4 + i);
                const int jj[4] = {j.x, j.y, j.z, j.w};
                const float ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float *d = sl + jj[k] + 3 * x;
                    c0 = fmaf(ww[k], d[0], c0);
                    c1 = fmaf(ww[k], d[1], c1);
                    c2 = fmaf(ww[k], d[2], c2);
                }
            }
            q[0] = v0 + c0;
            q[1] = v1 + c1;
            q[2] = v2 + c2;
        }
        __syncthreads();
    };

    // One sweep of the tile's rows: flux of tile and halo rows to LDS, the column's new values to
    // LDS and, where a row is read by another tile (or all = true), to buffer dst.
    auto sweep = [&](float *dst, bool all) {
        const int x = opaque(xt), tr = opaque(tr0);
        const int xm = x == 0 ? LW - 1 : x - 1, xp = x == LW - 1 ? 0 : x + 1;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int slot = tr + s * RS;
            if (slot < GR) {
                const int i = 3 * (slot * LW + x);
                float e0 = be0, e1 = be1, e2 = be2;
                if (a.bext_yz) {
                    e0 += syz[3 * slot];
                    e1 += syz[3 * slot + 1];
                    e2 += syz[3 * slot + 2];
                }
                sweep_flux(sb[i] + e0, sb[i + 1] + e1, sb[i + 2] + e2, u[s][0], u[s][1], u[s][2], sl[i], sl[i + 1], sl[i + 2]);
            }
        }
        __syncthreads();
        const int chunk = tr / a.ty, ly = tr - chunk * a.ty, zb = chunk * CZ;
        const bool own = ly < th && zb < tw && x >= xh && x < xh + wx;
        float res[CZ][3];
        if (own) {
            March<1> march;
            // cells x - 1, x, x + 1 of row ly and plane zb; opaque, so that the addresses of every plane
            // are not kept in registers across the iterations (and, for tall
            // columns, one plane's reads at a time)
            int cm = 3 * ((ly + PY * zb) * LW + xm), cc = 3 * ((ly + PY * zb) * LW + x), cp = 3 * ((ly + PY * zb) * LW + xp);
#pragma unroll
            for (int p = 0; p < CZ + 2; ++p) {
                if constexpr (CZ > 1) asm volatile("" : "+v"(cm), "+v"(cc), "+v"(cp) : : "memory");
                float c[3][3][6];
#pragma unroll
                for (int r = 0; r < 3; ++r)
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        const int o = (j == 0 ? cm : j == 1 ? cc : cp) + 3 * LW * r;
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            c[r][j][k] = sb[o + k];
                            c[r][j][3 + k] = sl[o + k];
                        }
                    }
                auto rows = [&](int k, float (&v)[3][3]) {
#pragma unroll
                    for (int r = 0; r < 3; ++r)
#pragma unroll
                        for (int j = 0; j < 3; ++j) v[r][j] = c[r][j][k];
                };
                float S[1][3], B[1][3], P[1][2], cen[1][3], out[1][3];
                plane_terms<1, Q27>(columns_rows<1>(rows), W, S, B, P, cen);
                march.take(W, S, B, P, cen, out);
                if (p >= 2)
#pragma unroll
                    for (int c = 0; c < 3; ++c) res[p - 2][c] = out[0][c];
                const int up = zb + p <= tw ? 3 * LW * PY : 0;  // past the tile's last plane: taken again, unused
                cm += up;
                cc += up;
                cp += up;
            }
        }
        __syncthreads();
        if (own) {
            const int x = opaque(xt);
            const int *exported = stab + tab_hdr(kResOExp);
#pragma unroll
            for (int p = 0; p < CZ; ++p) {
                const int lz = zb + p;
                if (lz >= tw) break;
                float *o = sb + 3 * ((ly + 1 + PY * (lz + 1)) * LW + x);
                o[0] = res[p][0];
                o[1] = res[p][1];
                o[2] = res[p][2];
                if (all || exported[ly + a.ty * lz] || (xh && (x == 1 || x == wx))) {
                    float *g = dst + (cx + (int64_t)nx * (y0 + ly + (int64_t)ny * (z0 + lz)));
                    st_agent(g, res[p][0]);
                    st_agent(g + N, res[p][1]);
                    st_agent(g + 2 * N, res[p][2]);
                }
            }
        }
        __builtin_amdgcn_s_waitcnt(0);  // this wave's exports are written
        __syncthreads();
    };
    auto store_tile = [&](float *dst) {
        const int x = opaque(xt), tr = opaque(tr0);
        if (x < xh || x >= xh + wx) return;
        for (int r = tr; r < th * tw; r += RS) {
            const int lz = r / th, ly = r - lz * th;
            float *p = dst + (cx + (int64_t)nx * (y0 + ly + (int64_t)ny * (z0 + lz)));
            const float *q = sb + 3 * ((ly + 1 + PY * (lz + 1)) * LW + x);
            st_agent(p, q[0]);
            st_agent(p + N, q[1]);
            st_agent(p + 2 * N, q[2]);
        }
    };

    // Flags count a tile's iterations. A wait guards against a stall of the machine with the clock, and
    // reports it as an error of the step.
    int *flag = a.sync + kResFlags;
    // the tiles exchanged with: those of the list, and where the box is cut along x also those before and
    // after each in x (itself listed; a tile waits for itself at once)
    const int wide = xh ? 3 : 1;
    auto neighbour = [&](int tile) {
        return t < wide * tab_hdr(kResNNb) ? wrapi(tile % a.gx + (xh ? t % 3 - 1 : 0), a.gx) + a.gx * stab[tab_hdr(kResONb) + t / wide]
                                           : -1;
    };
    auto wait_for = [&](int nb, int done) {
        if (nb >= 0) {
            const long long t0 = wall_clock64();
            int polls = 0;
            while (ld_agent(flag + kResFlagStride * nb) < done) {
                if ((++polls & 1023) == 0 &&
                    (wall_clock64() - t0 > kResStallTicks || ld_agent(a.sync + kResStalled))) {
                    __hip_atomic_store(a.sync + kResStalled, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    *a.stalled = 1;
                    break;
                }
            }
        }
        __syncthreads();
    };
    auto raise = [&](int tile, int done) {
        if (t == 0) __hip_atomic_store(flag + kResFlagStride * tile, done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };

    if constexpr (STAND_IN) {
        // turn k: iteration k / nwg of tile k % nwg; after the last iteration a turn a tile corrects it
        for (;;) {
            __syncthreads();
            if (t == 0) s_state = __hip_atomic_fetch_add(a.sync + kResTicket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const int turn = s_state, i = turn / a.nwg, tile = turn - i * a.nwg;
            if (i > a.n_mag) return;
            if (turn == 0 && t == 0) {  // for the next steps and calls (one workgroup of a step comes here)
                if (a.record && ld_agent(a.sync + kResState) == kResGivenUp) {
                    a.sync[kResHold] = kResHoldSteps;
                    const int n = ++a.sync[kResGiveUps];
                    __hip_atomic_store(a.host, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                }
                const int n = ++a.sync[kResStandIns];
                __hip_atomic_store(a.host + 1, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
            setup(tile);
            wait_for(neighbour(tile), i);
            load_rows(a.b[i & 1], true);
            request();
            if (i) correct();
            if (i < a.n_mag) {
                sweep(a.b[1 - (i & 1)], true);
                raise(tile, i + 1);
            } else {
                store_tile(a.b[1 - (i & 1)]);
            }
        }
    } else {
        const int me = blockIdx.x;
        setup(me);
        load_rows(a.b[0], true);
        const int nb = neighbour(me);
        for (int i = 0; i < a.n_mag; ++i) {
            float *next = a.b[1 - (i & 1)];
            sweep(next, false);
            raise(me, i + 1);
            request();
            wait_for(nb, i + 1);
            load_rows(next, false);
            correct();
        }
        store_tile(a.b[1 - (a.n_mag & 1)]);
    }
}

// The kernels of a launch shape: [D3Q27][stand-in]
struct ResForms {
    const void *k[2][2];
};
template <int NS, int CZ>
static ResForms forms_t() {
    return {{{(const void *)k_mag_resident<NS, CZ, false, false>, (const void *)k_mag_resident<NS, CZ, false, true>},
             {(const void *)k_mag_resident<NS, CZ, true, false>, (const void *)k_mag_resident<NS, CZ, true, true>}}};
}
static ResForms resident_forms(const ResPlan &p) {
    if (p.ns == 1) return forms_t<1, 1>();
    if (p.ns == 2) return forms_t<2, 1>();
    if (p.cz == 2) return forms_t<6, 2>();
    if (p.cz == 4) return forms_t<6, 4>();
    return forms_t<6, 6>();
}

hipError_t prepare_mag_resident(const ResPlan &p) {
    const ResForms f = resident_forms(p);
    for (const auto &lattice : f.k)
        for (const void *k : lattice) {  // the same limit for every plan: boxes share the kernels
            const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResMaxLds);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

hipError_t launch_mag_resident(hipStream_t s, const ResArgs &a, const ResPlan &p, bool q27) {
    const ResForms f = resident_forms(p);
    void *args[] = {const_cast<ResArgs *>(&a)};
    for (const void *k : f.k[q27]) {  // the iteration, its stand-in
        const hipError_t e = hipLaunchKernel(k, dim3(p.nwg), dim3(p.threads), args, p.lds_bytes, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace mhd
