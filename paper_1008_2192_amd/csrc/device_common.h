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

// The bit rows of a frame with f.narrow != 0 (DevFrame), planes of a tile at `base` by number.
typedef uint16_t __attribute__((may_alias)) bit_unit;

__device__ __forceinline__ unsigned long long narrow_row(const DevFrame &f,
                                                         const unsigned long long *base,
                                                         size_t plane, int row) {
    if (f.narrow < 0)
        return base[plane * (size_t)-f.narrow + row];
    const int p = f.narrow, b = row * p;
    const bit_unit *u = reinterpret_cast<const bit_unit *>(base) + plane * (size_t)(2 * p);
    return (unsigned long long)((uint32_t)u[b >> 4] >> (b & 15) & ((1u << p) - 1u));
}
// Stores n rows of a plane from row r0 on (16 rows or a multiple) by a block's threads, row(i)
// being row r0 + i; rows past the frame are left out or empty.
template <class F>
__device__ __forceinline__ void narrow_store(const DevFrame &f, unsigned long long *base,
                                             size_t plane, int r0, int n, int tid, int nthreads,
                                             F row) {
    if (f.narrow < 0) {
#pragma unroll 1
        for (int i = tid; i < n && r0 + i < -f.narrow; i += nthreads)
            base[plane * (size_t)-f.narrow + r0 + i] = row(i);
        return;
    }
    const int p = f.narrow, per = 16 / p;              // rows of a unit
    bit_unit *u = reinterpret_cast<bit_unit *>(base) + plane * (size_t)(2 * p) + r0 / per;
#pragma unroll 1
    for (int i = tid; i < n / per; i += nthreads) {
        uint32_t v = 0u;
#pragma unroll 1
        for (int q = 0; q < per; ++q)
            v |= ((uint32_t)row(i * per + q) & ((1u << p) - 1u)) << (q * p);
        u[i] = (bit_unit)v;
    }
}

}  // namespace crb
