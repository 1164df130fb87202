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

// Rows `row` of the three code planes from number `plane` on.
__device__ __forceinline__ void narrow_codes(const DevFrame &f, size_t plane, int row,
                                             unsigned long long (&v)[3]) {
    if (f.narrow < 0) {
        const unsigned long long *b = f.bits + plane * (size_t)-f.narrow + row;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            v[i] = b[i * -f.narrow];
    } else {
        const int p = f.narrow, at = row * p;
        const bit_unit *u =
            reinterpret_cast<const bit_unit *>(f.bits) + plane * (size_t)(2 * p) + (at >> 4);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            v[i] = (uint32_t)u[i * 2 * p] >> (at & 15) & ((1u << p) - 1u);
    }
}
__device__ __forceinline__ unsigned long long narrow_mask(const DevFrame &f, size_t tile, int row) {
    if (f.narrow < 0)
        return f.mbits[tile * (size_t)-f.narrow + row];
    const int p = f.narrow, at = row * p;
    const bit_unit *u = reinterpret_cast<const bit_unit *>(f.mbits) + tile * (size_t)(2 * p);
    return (uint32_t)u[at >> 4] >> (at & 15) & ((1u << p) - 1u);
}
// Stores a plane by a whole wave, lane l < 32 holding row l in v (empty past the frame).
__device__ __forceinline__ void narrow_store(const DevFrame &f, unsigned long long *base,
                                             size_t plane, int lane, unsigned long long v) {
    if (f.narrow < 0) {
        if (lane < -f.narrow)
            base[plane * (size_t)-f.narrow + lane] = v;
        return;
    }
    const int p = f.narrow, per = 16 / p;              // rows of a unit, gathered by their lanes
    uint32_t b = ((uint32_t)v & ((1u << p) - 1u)) << ((lane & (per - 1)) * p);
    for (int s = 1; s < per; s *= 2)
        b |= (uint32_t)__shfl_xor((int)b, s);
    if (lane < kSumTY && (lane & (per - 1)) == 0)
        reinterpret_cast<bit_unit *>(base)[plane * (size_t)(2 * p) + (lane * p >> 4)] =
            (bit_unit)b;
}

}  // namespace crb
