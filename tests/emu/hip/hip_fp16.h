#pragma once
struct __half {
    unsigned short v;
};
inline float __half2float(__half) { return 0.0f; }  // not reached by the float32 kernels
inline __half __float2half_rn(float) { return {0}; }
