// Device helpers shared by the detection kernel (detect.hip) and the other kernels
// of libcrb (kernels.hip).
#pragma once

#include "kernels.h"

namespace crb {

__device__ __forceinline__ float vmin(float a, float b) { return fminf(a, b); }
__device__ __forceinline__ float vmax(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double vmin(double a, double b) { return fmin(a, b); }
__device__ __forceinline__ double vmax(double a, double b) { return fmax(a, b); }

__device__ __forceinline__ int clampi(int i, int n) { return min(max(i, 0), n - 1); }
__device__ __forceinline__ float med3f(float a, float b, float c) {
    return __builtin_amdgcn_fmed3f(a, b, c);
}
__device__ __forceinline__ float min3f(float a, float b, float c) { return fminf(fminf(a, b), c); }
__device__ __forceinline__ float max3f(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// Clears the counters of the list of iteration k (by one block).
__device__ __forceinline__ void lists_clear(const StepLists &l, int k, int tid) {
    if (tid < l.nseg)
        l.count[((k % 3) * l.nseg + tid) * kTicketStride] = 0u;
}
// Before iteration 1, which fills the list of iteration 2 and clears that of iteration 3.
__device__ __forceinline__ void lists_start(const StepLists &l, int tid) {
    if (l.list[0])
        lists_clear(l, 2, tid);
}

}  // namespace crb
