// Stand-in for the HIP headers that compiles a kernel source for the CPU (tests/emu/resident_emu.cpp): a
// workgroup is one thread of the host whose work-items are fibers that run from barrier to barrier.
// Only what the resident iteration and the headers it includes use is here.
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>

using std::max;
using std::min;

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct alignas(8) float2 { float x, y; };
struct alignas(16) float4 { float x, y, z, w; };
struct alignas(8) int2 { int x, y; };
struct alignas(16) int4 { int x, y, z, w; };
typedef void *hipStream_t;
typedef void *hipEvent_t;
enum hipError_t { hipSuccess = 0, hipErrorUnknown = 999 };
enum hipFuncAttribute { hipFuncAttributeMaxDynamicSharedMemorySize = 8 };

namespace emu {
struct Lane {
    unsigned tid, block, threads, blocks;
};
extern thread_local Lane lane;  // of the work-item that runs
void barrier(int line);         // ends when every work-item of the workgroup has come to this line
void pause();                   // a wait for another workgroup
long long clock();
struct Coord {
    unsigned Lane::*m;
    operator unsigned() const { return lane.*m; }
};
}  // namespace emu
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute a, int v);
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t s);

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define __shared__ thread_local
#define threadIdx (emu::LaneIndex{})
#define blockIdx (emu::BlockIndex{})
#define blockDim (emu::BlockDim{})
#define gridDim (emu::GridDim{})
namespace emu {
struct LaneIndex { Coord x{&Lane::tid}; };
struct BlockIndex { Coord x{&Lane::block}; };
struct BlockDim { Coord x{&Lane::threads}; };
struct GridDim { Coord x{&Lane::blocks}; };
}  // namespace emu
#define __syncthreads() emu::barrier(__LINE__)

#define __HIP_MEMORY_SCOPE_WORKGROUP 2
#define __HIP_MEMORY_SCOPE_AGENT 3
#define __HIP_MEMORY_SCOPE_SYSTEM 4
template <typename T>
inline T emu_load(T *p) {
    emu::pause();
    return __atomic_load_n(p, __ATOMIC_SEQ_CST);
}
inline float emu_load(const float *p) {
    int v = __atomic_load_n(reinterpret_cast<const int *>(p), __ATOMIC_SEQ_CST);
    float f;
    memcpy(&f, &v, 4);
    return f;
}
template <typename T>
inline void emu_store(T *p, T v) {
    __atomic_store(p, &v, __ATOMIC_SEQ_CST);
}
#define __hip_atomic_load(p, order, scope) emu_load(p)
#define __hip_atomic_store(p, v, order, scope) emu_store(p, v)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_fetch_or(p, v, order, scope) __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_compare_exchange_strong(p, e, v, o1, o2, scope) \
    __atomic_compare_exchange_n(p, e, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)

inline long long wall_clock64() { return emu::clock(); }
inline void __builtin_amdgcn_s_sleep(int) { emu::pause(); }
inline void __builtin_amdgcn_s_waitcnt(int) {}
inline int __builtin_amdgcn_mov_dpp(int v, int, int, int, bool) { return v; }         // not reached: the lane
inline int __builtin_amdgcn_update_dpp(int, int v, int, int, int, bool) { return v; }  // shifts of the marches
inline float __int_as_float(int v) {
    float f;
    memcpy(&f, &v, 4);
    return f;
}
inline int __float_as_int(float v) {
    int i;
    memcpy(&i, &v, 4);
    return i;
}

// empty asm statements that hide a value from the optimiser
#define asm
#define volatile(...)
