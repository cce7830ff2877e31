// float32 magnetic sweep for boxes with n_x a multiple of 128, 8-row tiles: every lane owns two
// neighbouring x cells, a wave a 128-cell row, a workgroup 8 rows, and it marches along z over a chunk
// of planes (mhd_sweep.hip describes the update; the arithmetic is mhd_sweep_math.h).
//
// What bounds a march of this kind is the chain of each plane in a CU: the vector instructions and
// around them the LDS latencies and the issue of the loads. The planes go straight to LDS
// (global_load_lds, 16 bytes a lane, two rows an instruction, no registers held), a ring of four raw
// planes of u and b, requested three planes ahead; the flux of a plane takes the place of its u,
// which nothing else reads. What is left is arranged by who has time: two waves share a SIMD, the
// older one is served first and ends its plane before the other, so the requests, the two extra rows
// and the halo columns are work of the first four waves, at the end of the plane, and the raw values
// of the next plane are read ahead of the reduction and become flux after it.
// Against the form that stages through registers (k_mag_sweep_pair, which the 16-bit kinds keep): 512 x
// 256^2, 128-plane chunks 263.5 -> 240.2 us, and 234.9 us (5.14 TB/s algorithmic) since the columns beside
// a lane's come from its neighbours; 128 x 256^2, 32 planes 57.4 -> 55.2 -> 54.0 us. With 4-row tiles
// it is the slower one (128^3, 8 planes 17.3 against 16.7 us; 256 x 132^2 46.0 against 44.0): two
// workgroups a CU already fill each other's gaps there, so the 4-row tiles keep the register form.
//
// Step p of the march: wait for this wave's part of plane p + 1, workgroup barrier, reduce plane p
// (b and flux from its ring slot), write the outputs of plane p - 1, form the flux of plane p + 1,
// request plane p + 3 (into the slot of plane p - 1, whose readers have passed the barrier). One
// barrier a plane.
//
// The waits are counted: vector-memory operations complete in order, so s_waitcnt vmcnt(n) with n
// the operations this wave issued after the plane's last request leaves later planes and stores
// in flight. n is never larger than what was issued (waits()); operations that the compiler adds
// only make the wait longer.
#include <hip/hip_ext.h>

#include "mhd_device.h"
#include "mhd_sweep_math.h"

namespace mhd {

namespace {

constexpr int kRows = 8;  // rows of a tile

__device__ __forceinline__ unsigned lds_offset(const void *p) {
    return (unsigned)(size_t)(__attribute__((address_space(3))) const void *)p;
}
// m0 is named as written, so that no value of the compiler's own is kept there across a load; it warns
// that the register is one it reserves for such uses.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
// 16 bytes a lane from base + voff (bytes, per lane) to LDS at lds + 16 lane
__device__ __forceinline__ void load_lds16(unsigned lds, unsigned voff, const void *base) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(voff), "s"(base) : "m0", "memory");
}
// 4 bytes a lane from an address of its own, lanes of the execution mask only
__device__ __forceinline__ void load_lds4(unsigned lds, const char *src) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(lds), "v"(src) : "m0", "memory");
}
#pragma clang diagnostic pop
template <int N>
__device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

}  // namespace

// XWRAP: n_x = 128, one tile spans the periodic row and x neighbours come by wave rotation; otherwise
// the two halo columns of every row are staged beside the rows. BYZ: B_ext has a (y, z) table.
template <bool BATCH, bool BYZ, bool Q27, bool XWRAP>
__global__ void __launch_bounds__(64 * kRows) k_sweep_rows(SweepArgs a, const PipeStep *tab, const BlockMap *map, int which,
                                                           int nbatch) {
    constexpr int TY = kRows, HY = TY + 2, RING = 4;  // staged rows, raw planes in LDS
    constexpr int ROWB = 512, FIELDB = HY * ROWB, SLOTB = 6 * FIELDB;
    // fields 0 .. 2: b, 3 .. 5: u, then the flux
    __shared__ __align__(16) float s_pl[RING][6][HY][128];
    __shared__ __align__(16) float s_col[XWRAP ? 1 : RING][6][HY][2];  // halo columns x0 - 1, x0 + 128

    const int per = gridDim.x >> 3;  // XCD-aware order (as for the other sweeps)
    int lb = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if constexpr (BATCH) {
        if (lb >= nbatch) return;
        const BlockMap m = map[lb];
        a = tab[m.pipe].sw[which];
        lb = m.local;
    } else {
        if (lb >= a.nblocks) return;
    }
    const int tix = lb % a.tiles_x, rest = lb / a.tiles_x;
    const int tiy = rest % a.tiles_y, tiz = rest / a.tiles_y;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int x0 = tix * 128, y0 = tiy * TY, z0 = tiz * a.zchunk, z1 = min(z0 + a.zchunk, nz);
    const unsigned N = (unsigned)nx * ny * nz;  // 3 N < 2^31: 32-bit byte offsets from uniform bases
    const unsigned plane = (unsigned)nx * ny * 4u;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    const int xa = x0 + 2 * l, gy = y0 + w;
    const bool own = gy < ny;
    const SweepWeights W = sweep_weights<Q27>(a.kappa, a.omega);

    // Requests of a plane, one for two rows of a field (lanes 0 .. 31 and 32 .. 63): wave w < 4 asks for
    // rows 2 w and 2 w + 1 of all six fields; of rows 8 and 9, waves 0 and 1 for two fields, waves 2 and 3
    // for one and for half of the halo columns (60 values each).
    const char *fp[6];
#pragma unroll
    for (int f = 0; f < 6; ++f) fp[f] = (const char *)(f < 3 ? a.b : a.u) + (size_t)(f % 3) * N * 4;
    auto row_off = [&](int pair) { return (unsigned)(x0 + 4 * (l & 31) + nx * wrapi(y0 - 1 + 2 * pair + (l >> 5), ny)) * 4u; };
    const unsigned vmain = row_off(min(w, 3)), vex = row_off(4);
    const int nex = w < 2 ? 2 : w < 4 ? 1 : 0;
    unsigned lex[2];
    const char *pex[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int f = w < 2 ? 2 * w + e : min(w + 2, 5);
        lex[e] = (unsigned)(f * FIELDB + 8 * ROWB);
        pex[e] = (const char *)(f < 3 ? a.b : a.u) + (size_t)(f % 3) * N * 4;
    }
    const int hi = 60 * (w - 2) + l;  // halo value: (field, row, side)
    const bool hload = !XWRAP && (w == 2 || w == 3) && l < 60;
    const char *hsrc = nullptr;
    if (hload) {
        const int f = hi / (2 * HY), hy = (hi >> 1) % HY, x = hi & 1 ? wrapi(x0 + 128, nx) : wrapi(x0 - 1, nx);
        hsrc = (const char *)(f < 3 ? a.b : a.u) + (size_t)(f % 3) * N * 4 + (unsigned)(x + nx * wrapi(y0 - 1 + hy, ny)) * 4u;
    }
    const unsigned lds0 = lds_offset(&s_pl[0][0][0][0]), ldsc = lds_offset(&s_col[0][0][0][0]);
    auto request = [&](int p, int slot) {
        if (w >= 4) return;
        const unsigned off = (unsigned)wrapi(p, nz) * plane, at = lds0 + (unsigned)slot * SLOTB;
#pragma unroll
        for (int f = 0; f < 6; ++f) load_lds16(at + f * FIELDB + (unsigned)w * (2 * ROWB), vmain + off, fp[f]);
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (e < nex) load_lds16(at + lex[e], vex + off, pex[e]);
        if constexpr (!XWRAP)
            if (hload) load_lds4(ldsc + (unsigned)slot * (12 * HY * 4) + (unsigned)(w - 2) * 240u, hsrc + off);
    };
    const int nreq = w >= 4 ? 0 : 6 + nex + (XWRAP || w < 2 ? 0 : 1);  // 8, or 7 without halo columns

    // B_ext of this lane's cells and of the halo column it stages (lane 2 row + side of wave 2)
    const float bea[3] = {a.bext[xa], a.bext[nx + xa], a.bext[2 * nx + xa]};
    const float beb[3] = {a.bext[xa + 1], a.bext[nx + xa + 1], a.bext[2 * nx + xa + 1]};
    const bool hstage = !XWRAP && w == 2 && l < 2 * HY;
    const int hrow = min(l >> 1, HY - 1), hx = l & 1 ? wrapi(x0 + 128, nx) : wrapi(x0 - 1, nx);
    const float beh[3] = {a.bext[hx], a.bext[nx + hx], a.bext[2 * nx + hx]};
    const unsigned pyz = (unsigned)ny * nz;

    // flux of plane p in row hy from its raw values v, in place of u
    auto read_raw = [&](int slot, int hy, float2 (&v)[6]) {
#pragma unroll
        for (int q = 0; q < 6; ++q) v[q] = *reinterpret_cast<const float2 *>(&s_pl[slot][q][hy][2 * l]);
    };
    auto write_flux = [&](int p, int slot, int hy, const float2 (&v)[6]) {
        float ea[3] = {bea[0], bea[1], bea[2]}, eb[3] = {beb[0], beb[1], beb[2]};
        if constexpr (BYZ) {
            const unsigned o = (unsigned)(wrapi(y0 - 1 + hy, ny) + ny * wrapi(p, nz));
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                ea[q] += a.bext_yz[q * pyz + o];
                eb[q] += a.bext_yz[q * pyz + o];
            }
        }
        float2 f[3];
        sweep_flux(v[0].x + ea[0], v[1].x + ea[1], v[2].x + ea[2], v[3].x, v[4].x, v[5].x, f[0].x, f[1].x, f[2].x);
        sweep_flux(v[0].y + eb[0], v[1].y + eb[1], v[2].y + eb[2], v[3].y, v[4].y, v[5].y, f[0].y, f[1].y, f[2].y);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<float2 *>(&s_pl[slot][3 + q][hy][2 * l]) = f[q];
    };
    auto stage_rest = [&](int p, int slot) {  // the two extra rows, the halo columns
        if (w < 2) {
            float2 v[6];
            read_raw(slot, TY + w, v);
            write_flux(p, slot, TY + w, v);
        }
        if constexpr (!XWRAP) {
            if (hstage) {
                float e[3] = {beh[0], beh[1], beh[2]}, v[6], f[3];
                if constexpr (BYZ) {
                    const unsigned o = (unsigned)(wrapi(y0 - 1 + hrow, ny) + ny * wrapi(p, nz));
#pragma unroll
                    for (int q = 0; q < 3; ++q) e[q] += a.bext_yz[q * pyz + o];
                }
#pragma unroll
                for (int q = 0; q < 6; ++q) v[q] = s_col[slot][q][hrow][l & 1];
                sweep_flux(v[0] + e[0], v[1] + e[1], v[2] + e[2], v[3], v[4], v[5], f[0], f[1], f[2]);
#pragma unroll
                for (int q = 0; q < 3; ++q) s_col[slot][3 + q][hrow][l & 1] = f[q];
            }
        }
    };
    // This wave's part of plane p + 1 has arrived. Issued after its requests: the stores of step p - 1
    // (three, once the march writes) and the requests of plane p + 2.
    auto waits = [&](int p) {
        const int st = own && p >= z0 + 2 ? 3 : 0, n = p + 2 <= z1 ? nreq : 0;
        switch (n + st) {
            case 3: wait_vm<3>(); break;
            case 7: wait_vm<7>(); break;
            case 8: wait_vm<8>(); break;
            case 10: wait_vm<10>(); break;
            case 11: wait_vm<11>(); break;
            default: wait_vm<0>(); break;
        }
    };

    March<2> march;
    float *o0 = (float *)a.bo, *o1 = o0 + N, *o2 = o0 + 2 * (size_t)N;

    request(z0 - 1, 0);
    request(z0, 1);
    request(z0 + 1, 2);
    wait_vm<14>();  // the first plane: at least 7 requests for each of the two after it, or none at all
    __syncthreads();
    {
        float2 v[6];
        read_raw(0, w, v);
        write_flux(z0 - 1, 0, w, v);
        stage_rest(z0 - 1, 0);
    }

    int slot = 0;  // of plane p
    for (int p = z0 - 1; p <= z1; ++p) {
        const int next = (slot + 1) & 3;
        if (p < z1 && nreq > 0) waits(p);
        __syncthreads();
        float2 raw[6];
        if (p < z1) read_raw(next, w, raw);
        if (own) {
            auto cells = [&](int k, float (&v)[3][2]) {
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const float2 c = *reinterpret_cast<const float2 *>(&s_pl[slot][k][w + r][2 * l]);
                    v[r][0] = c.x;
                    v[r][1] = c.y;
                }
            };
            auto end = [&](int k, float (&h)[3]) {
#pragma unroll
                for (int r = 0; r < 3; ++r) h[r] = s_col[slot][k][w + r][l >> 5];
            };
            float S[2][3], B[2][3], P[2][2], cen[2][3], out[2][3];
            plane_terms<2, Q27>(columns_wave<2, !XWRAP>(cells, end), W, S, B, P, cen);
            march.take(W, S, B, P, cen, out);
            if (p >= z0 + 1) {
                // written through the L2 (agent-scope relaxed atomic stores of the same values): the next
                // launch reads them, and no dirty lines wait for the kernel's end
                const unsigned ko = ((unsigned)(p - 1) * (unsigned)(nx * ny) + (unsigned)(xa + nx * gy)) * 4u;
                float *oo[3] = {o0, o1, o2};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const float2 v = make_float2(out[0][q], out[1][q]);
                    unsigned long long bits;
                    __builtin_memcpy(&bits, &v, 8);
                    __hip_atomic_store(reinterpret_cast<unsigned long long *>(reinterpret_cast<char *>(oo[q]) + ko), bits,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        if (p < z1) {
            write_flux(p + 1, next, w, raw);
            stage_rest(p + 1, next);
            if (p + 3 <= z1) request(p + 3, (slot + 3) & 3);
        }
        slot = next;
    }
}

template <bool BATCH, bool BYZ, bool Q27>
static hipError_t rows_t(hipStream_t s, const SweepArgs &a, const PipeStep *tab, const BlockMap *map, int which, int nblocks,
                         hipEvent_t e0, hipEvent_t e1) {
    const dim3 grid((unsigned)(((nblocks + 7) / 8) * 8)), block(64 * kRows);
    if constexpr (!BATCH) {
        if (a.nx == 128) {  // a batched launch can mix boxes of different n_x, so it stages halo columns
            hipExtLaunchKernelGGL((k_sweep_rows<false, BYZ, Q27, true>), grid, block, 0, s, e0, e1, 0, a, tab, map, which, nblocks);
            return hipGetLastError();
        }
    }
    hipExtLaunchKernelGGL((k_sweep_rows<BATCH, BYZ, Q27, false>), grid, block, 0, s, e0, e1, 0, a, tab, map, which, nblocks);
    return hipGetLastError();
}
template <bool BATCH>
static hipError_t rows_q(hipStream_t s, const SweepArgs &a, SweepLaunch L, const PipeStep *tab, const BlockMap *map, int which,
                         int nblocks, hipEvent_t e0, hipEvent_t e1) {
    if (L.byz)
        return L.q27 ? rows_t<BATCH, true, true>(s, a, tab, map, which, nblocks, e0, e1)
                     : rows_t<BATCH, true, false>(s, a, tab, map, which, nblocks, e0, e1);
    return L.q27 ? rows_t<BATCH, false, true>(s, a, tab, map, which, nblocks, e0, e1)
                 : rows_t<BATCH, false, false>(s, a, tab, map, which, nblocks, e0, e1);
}
hipError_t launch_sweep_rows(hipStream_t s, bool batch, const SweepArgs &a, SweepLaunch L, const PipeStep *tab,
                             const BlockMap *map, int which, int nblocks, hipEvent_t e0, hipEvent_t e1) {
    return batch ? rows_q<true>(s, a, L, tab, map, which, nblocks, e0, e1) : rows_q<false>(s, a, L, tab, map, which, nblocks, e0, e1);
}

}  // namespace mhd
