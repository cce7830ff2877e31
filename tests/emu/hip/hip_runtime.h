// Stand-in for the HIP headers, to compile sources of the library for the CPU. resident_emu.cpp takes a
// kernel: a workgroup is one thread of the host whose work-items are fibers that run from barrier to
// barrier. runtime_emu.cpp takes the host runtime: it implements the calls below on host memory. Only
// what those sources use is here.
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
typedef struct emuStream *hipStream_t;
typedef struct emuEvent *hipEvent_t;
typedef struct emuGraph *hipGraph_t;
typedef struct emuGraph *hipGraphExec_t;
typedef struct emuNode *hipGraphNode_t;
enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorInvalidHandle = 400, hipErrorNotReady = 600, hipErrorUnknown = 999 };
enum hipFuncAttribute { hipFuncAttributeMaxDynamicSharedMemorySize = 8 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2, hipMemcpyDeviceToDevice = 3 };
enum hipStreamCaptureMode { hipStreamCaptureModeRelaxed = 2 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0, hipStreamCaptureStatusActive = 1 };
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount = 63 };
constexpr unsigned hipEventDisableTiming = 2, hipHostMallocDefault = 0, hipHostMallocMapped = 2;

hipError_t hipGetLastError();
const char *hipGetErrorString(hipError_t e);
hipError_t hipGetDevice(int *d);
hipError_t hipSetDevice(int d);
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d);
hipError_t hipHostMalloc(void **p, size_t n, unsigned flags);
hipError_t hipHostFree(void *p);
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned flags);
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st);
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st);
hipError_t hipStreamSynchronize(hipStream_t s);
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned flags);
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c);
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode m);
hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t *g);
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *n, char *log, size_t len);
hipError_t hipGraphDestroy(hipGraph_t g);
hipError_t hipGraphExecDestroy(hipGraphExec_t e);
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s);
hipError_t hipEventCreate(hipEvent_t *e);
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned flags);
hipError_t hipEventDestroy(hipEvent_t e);
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s);
hipError_t hipEventQuery(hipEvent_t e);
hipError_t hipEventSynchronize(hipEvent_t e);
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b);

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
