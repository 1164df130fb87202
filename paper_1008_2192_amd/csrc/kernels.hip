// Helper kernels of libcrb for gfx950 (MI355X): niter = 0 copies, per-frame results,
// subimage copies and parity-test helpers.  The method's kernels are detect.hip (the first
// iteration's detection) and step.hip (everything after it).
#include "kernels.h"
#include "device_common.h"

#include <math.h>

namespace crb {

// ---------------------------------------------------------------------------
// init and stats
// ---------------------------------------------------------------------------

// Grid rows (blockIdx.y) take the frames in turn.
__global__ __launch_bounds__(kThreads) void k_init(const DevFrame *__restrict__ frames,
                                                   int nframes, DevFrame single) {
    const size_t gid = (size_t)blockIdx.x * kThreads + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * kThreads;
    const int nf = frames ? nframes : 1;
    for (int fi = blockIdx.y; fi < nf; fi += gridDim.y) {
        const DevFrame f = frames ? frames[fi] : single;
        if (f.niter == 0) {
            const size_t n = (size_t)f.H * (size_t)f.W;
            for (size_t i = gid; i < n; i += stride) {
                if (f.img != f.J)
                    f.J[i] = f.img[i];
                f.mask[i] = 0;
            }
        }
    }
}

__device__ __forceinline__ long long flagged(const DevFrame &f) {
    unsigned long long n = 0ull;
    for (int i = 0; i < kCountSlots; ++i)
        n += f.count[i * kCountStride];
    return (long long)n;
}

__global__ void k_stats(const DevFrame *__restrict__ frames, int nframes,
                        long long *__restrict__ stats) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nframes)
        return;
    const DevFrame &f = frames[i];
    int iters = 0;
    while (iters < f.niter) {
        ++iters;
        if (!f.any_new[iters - 1] && !(f.flags & kNoEarlyStop))
            break;
    }
    stats[2 * i] = iters;
    stats[2 * i + 1] = f.niter ? flagged(f) : 0;
}

__global__ void k_round_stats(const DevFrame *__restrict__ frames, int nframes,
                              long long *__restrict__ stats) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nframes)
        return;
    const DevFrame &f = frames[i];
    stats[2 * i] = (long long)f.any_new[f.k - 1];
    stats[2 * i + 1] = flagged(f);
}

__global__ void k_count(DevFrame f, long long *__restrict__ out) {
    if (threadIdx.x == 0)
        *out = flagged(f);
}

// ---------------------------------------------------------------------------
// subimage partition (the paper's 2-D split with a border, Section 6.2)
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(kThreads) void k_extract(const float *__restrict__ img, int W,
                                                      const SubRect *__restrict__ subs) {
    const SubRect r = subs[blockIdx.y];
    const size_t n = (size_t)r.h * r.w;
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (size_t)gridDim.x * kThreads) {
        const int y = (int)(i / r.w), x = (int)(i - (size_t)y * r.w);
        r.sub_img[i] = img[(size_t)(r.a0 + y) * W + r.b0 + x];
    }
}

__global__ __launch_bounds__(kThreads) void k_stitch(float *__restrict__ out_clean,
                                                     uint8_t *__restrict__ out_mask, int W,
                                                     const SubRect *__restrict__ subs) {
    const SubRect r = subs[blockIdx.y];
    const int ih = r.y1 - r.y0, iw = r.x1 - r.x0;
    const size_t n = (size_t)ih * iw;
    for (size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x; i < n;
         i += (size_t)gridDim.x * kThreads) {
        const int y = r.y0 + (int)(i / iw), x = r.x0 + (int)(i % iw);
        const size_t q = (size_t)(y - r.a0) * r.w + (x - r.b0);
        out_clean[(size_t)y * W + x] = r.sub_clean[q];
        out_mask[(size_t)y * W + x] = r.sub_mask[q];
    }
}

// ---------------------------------------------------------------------------
// parity-test kernels: the median networks alone, binary64 sqrt and division
// ---------------------------------------------------------------------------

// A copy by 4-byte buffer loads and stores, one element per lane in consecutive order
// (the detection stages J with the same 4-byte buffer loads): its HBM counter readings
// against its known byte count calibrate the counters for that access width.  Blocks
// take 2^20-element chunks (each within one buffer resource, below 2^32 bytes).
__global__ __launch_bounds__(kThreads) void k_debug_copy_b32(const float *__restrict__ src,
                                                             float *__restrict__ dst,
                                                             long long n) {
    constexpr long long kChunk = 1ll << 20;
    const long long nchunks = (n + kChunk - 1) / kChunk;
    for (long long c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const long long base = c * kChunk;
        const long long len = n - base < kChunk ? n - base : kChunk;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(src + base), (short)0, (int)(len * 4), 0x00020000);
        const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
            (void *)(dst + base), (short)0, (int)(len * 4), 0x00020000);
        for (int i = threadIdx.x; i < (int)len; i += kThreads) {
            const unsigned int v = __builtin_amdgcn_raw_buffer_load_b32(rs, i * 4, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(v, rd, i * 4, 0, 0);
        }
    }
}

__global__ void k_debug_fp64(const double *__restrict__ x, const double *__restrict__ y, int n,
                             double *__restrict__ os, double *__restrict__ od) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        os[i] = sqrt(x[i]);
        od[i] = x[i] / y[i];
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

static unsigned int grid_for(size_t items, unsigned int cap) {
    size_t g = (items + kThreads - 1) / kThreads;
    if (g < 1)
        g = 1;
    return (unsigned int)(g < cap ? g : cap);
}

hipError_t launch_init(const DevFrame *d_frames, int nframes, const DevFrame &single,
                       size_t max_pixels, hipStream_t s) {
    const int rows = d_frames ? (nframes < 65535 ? nframes : 65535) : 1;
    const unsigned int cap = 4096u / (unsigned int)rows > 16u ? 4096u / (unsigned int)rows : 16u;
    const unsigned int gx = grid_for(max_pixels, cap);
    k_init<<<dim3(gx, rows), kThreads, 0, s>>>(d_frames, nframes, single);
    return hipGetLastError();
}

hipError_t launch_stats(const DevFrame *d_frames, int nframes, long long *d_stats,
                        hipStream_t s) {
    k_stats<<<(nframes + 63) / 64, 64, 0, s>>>(d_frames, nframes, d_stats);
    return hipGetLastError();
}

hipError_t launch_count(const DevFrame &f, long long *out, hipStream_t s) {
    k_count<<<1, 64, 0, s>>>(f, out);
    return hipGetLastError();
}

hipError_t launch_round_stats(const DevFrame *d_frames, int nframes, long long *d_stats,
                              hipStream_t s) {
    k_round_stats<<<(nframes + 63) / 64, 64, 0, s>>>(d_frames, nframes, d_stats);
    return hipGetLastError();
}

hipError_t launch_extract(const float *img, int W, const SubRect *d_subs, int nsub,
                          size_t max_pixels, hipStream_t s) {
    dim3 grid(grid_for(max_pixels, 1024), nsub);
    k_extract<<<grid, kThreads, 0, s>>>(img, W, d_subs);
    return hipGetLastError();
}

hipError_t launch_stitch(float *out_clean, uint8_t *out_mask, int W, const SubRect *d_subs,
                         int nsub, size_t max_pixels, hipStream_t s) {
    dim3 grid(grid_for(max_pixels, 1024), nsub);
    k_stitch<<<grid, kThreads, 0, s>>>(out_clean, out_mask, W, d_subs);
    return hipGetLastError();
}

hipError_t launch_debug_copy_b32(const float *src, float *dst, long long n, hipStream_t s) {
    if (n <= 0)
        return hipSuccess;
    const long long nchunks = (n + (1ll << 20) - 1) >> 20;
    k_debug_copy_b32<<<(unsigned int)(nchunks < 4096 ? nchunks : 4096), kThreads, 0, s>>>(src,
                                                                                        dst, n);
    return hipGetLastError();
}

hipError_t launch_debug_fp64(const double *x, const double *y, int n, double *out_sqrt,
                             double *out_div, hipStream_t s) {
    k_debug_fp64<<<(n + kThreads - 1) / kThreads, kThreads, 0, s>>>(x, y, n, out_sqrt, out_div);
    return hipGetLastError();
}

}  // namespace crb
