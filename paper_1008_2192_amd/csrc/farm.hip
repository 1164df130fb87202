// Tile farm of libcrb (gfx950) and its work functions: POISSON and WAITER, the
// paper's framework probes (Section 6.3), and SOURCES, its example of a work
// function whose actors return structures (peak positions and aperture sums) rather
// than subimages (Section 7).  The contract between the farm and a work function is
// stated in farm.h.
#include "farm.h"

#include <math.h>

#include <type_traits>

// Exclusive prefix sum over the lanes of a wave (all lanes active), from the device library.
extern "C" __device__ unsigned int __ockl_wfscan_add_u32(unsigned int, bool);

namespace crb {

// ---------------------------------------------------------------------------
// POISSON: Knuth's multiplication method on a counter-based generator
// ---------------------------------------------------------------------------

// Philox4x32-10 counter-based generator (Salmon et al., SC 2011): ten rounds of
// two 32x32->64-bit products with the multipliers 0xD2511F53 and 0xCD9E8D57; the
// key advances by 0x9E3779B9 and 0xBB67AE85 after each round.
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        // (one 64-bit product each: half the multiply instructions of a low and a high one)
        const unsigned long long p0 = (unsigned long long)0xD2511F53u * c.x;
        const unsigned long long p1 = (unsigned long long)0xCD9E8D57u * c.z;
        c = make_uint4((uint32_t)(p1 >> 32) ^ c.y ^ k0, (uint32_t)p1,
                       (uint32_t)(p0 >> 32) ^ c.w ^ k1, (uint32_t)p0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// e^-x for 0 <= x <= 500: split x by ln 2 (Cody-Waite: a short high part of ln 2
// makes k * ln2_hi exact), degree-13 Taylor series of e^r by Horner's rule, then an
// exact power-of-two scale.  Only correctly rounded operations in a fixed order.
__device__ __forceinline__ double exp_neg(double x) {
    const double ln2_hi = 6.93147180369123816490e-01;
    const double ln2_lo = 1.90821492927058770002e-10;
    const double inv_ln2 = 1.44269504088896338700e+00;
    const double y = -x;
    const double kf = floor(y * inv_ln2 + 0.5);
    const double r = (y - kf * ln2_hi) - kf * ln2_lo;
    const double inv_fact[14] = {1.0, 1.0, 0.5, 1.0 / 6.0, 1.0 / 24.0, 1.0 / 120.0,
                                 1.0 / 720.0, 1.0 / 5040.0, 1.0 / 40320.0, 1.0 / 362880.0,
                                 1.0 / 3628800.0, 1.0 / 39916800.0, 1.0 / 479001600.0,
                                 1.0 / 6227020800.0};
    double p = inv_fact[13];
#pragma unroll
    for (int n = 12; n >= 0; --n)
        p = p * r + inv_fact[n];
    return ldexp(p, (int)kf);
}

// The limit e^-mean of Knuth's method for a pixel's mean (clamped to [0, 500]; non-finite: 0).
__device__ __forceinline__ double poisson_limit(float mean_f) {
    double mean = (double)mean_f;
    if (!(mean > 0.0))
        mean = 0.0;
    if (mean > 500.0)
        mean = 500.0;
    return exp_neg(mean);
}

// The deviate of pixel i with that limit (uniform j from word j % 4 of the generator at counter
// (i_lo, i_hi, j / 4, 0)).
__device__ __forceinline__ float poisson_draw(size_t i, double limit, uint32_t k0, uint32_t k1) {
    double prod = 1.0;
    unsigned int k = 0;
    for (uint32_t blk = 0;; ++blk) {
        const uint4 w = philox4x32_10(make_uint4((uint32_t)i, (uint32_t)(i >> 32), blk, 0u), k0,
                                      k1);
        const uint32_t words[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            prod = prod * (((double)words[q] + 0.5) * (1.0 / 4294967296.0));
            if (!(prod > limit))
                return (float)k;
            ++k;
        }
    }
}

// A float in the global address space: loads through it are global (not flat) loads.
typedef __attribute__((address_space(1))) const float GFloat;
// Fourth word of a raw buffer resource on gfx9-family GPUs: 32-bit data format,
// range-checked against the byte count given with the base.
constexpr int kBufWord3 = 0x00020000;

// Where a work function finds its pixel: the frame (resident in HBM; neighbours are
// read through the caches, never beyond the declared radius) and the position.
struct FarmCtx {
    const float *in;      // frame, H x W
    int y, x, H, W;       // the pixel's frame coordinates, frame size
};

// POISSON: deviates by multiplying uniforms until the product drops to e^-mean (Knuth's
// method); uniform j of pixel i comes from word j % 4 of the generator at counter (i_lo, i_hi,
// j / 4, 0).  A wave takes a tile in chunks of kChunk pixels per lane: the lanes form their
// pixels' limits together, and then each goes through its own pixels without waiting for the
// others' -- with one pixel per lane at a time a wave drew for the largest of 64 deviates (10
// blocks of four uniforms at mean 24.3, where a pixel needs 6.8).  Bound by the generator's
// multiplies at one wave per SIMD: 750 x 750 pixels of mean 24.3 in rows on 1024 actors took
// 60.7 us, with 64-bit products and this order 52.8 (two pixels of a lane at once: 52.3), and
// with the farm's tickets on lines of their own 37.1.
struct WorkPoisson {
    static constexpr bool kList = false;
    static constexpr bool kNeighbours = false;
    static constexpr int kChunk = 16;
    __host__ __device__ static int radius(const WorkArgs &) { return 0; }
    // The tile of tw columns and n pixels at (y0, x0); limits: the wave's kChunk x 64 doubles.
    __device__ static void tile(const float *__restrict__ in, float *__restrict__ out, int W,
                                const WorkArgs &a, int y0, int x0, int tw, long long n,
                                double *limits) {
        const int lane = __lane_id();
        const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
        const int q = 64 / tw, rem = 64 - q * tw;     // a step of 64 pixels
        int ly = lane / tw, lx = lane - ly * tw;
        // (a pixel per lane at most: no lane has a second one to go on to, and the chunk's passes
        // over the limits, most of them empty, cost an actor 0.9 us a tile: 256 tiles of one
        // pixel on one actor took 782 us with them)
        if (n <= 64) {
            if (lane < n) {
                const size_t i = (size_t)(y0 + ly) * W + x0 + lx;
                out[i] = poisson_draw(i, poisson_limit(in[i]), k0, k1);
            }
            return;
        }
        for (long long j0 = 0; j0 < n; j0 += 64 * kChunk) {
            int my = 0;                               // the lane's pixels of the chunk
            int y = ly, x = lx;                       // (the first of them)
            float mean[kChunk];
#pragma unroll
            for (int p = 0; p < kChunk; ++p) {
                if (j0 + 64 * p >= n)                 // (uniform)
                    break;
                const bool on = j0 + 64 * p + lane < n;
                my += on ? 1 : 0;
                mean[p] = on ? in[(size_t)(y0 + ly) * W + x0 + lx] : 0.0f;
                ly += q;
                lx += rem;
                if (lx >= tw) {
                    lx -= tw;
                    ++ly;
                }
            }
#pragma unroll
            for (int p = 0; p < kChunk; ++p) {
                if (j0 + 64 * p >= n)
                    break;
                limits[p * 64 + lane] = poisson_limit(mean[p]);
            }
            // (each lane reads only what it wrote)
            size_t i = (size_t)(y0 + y) * W + x0 + x;
            double limit = limits[lane], prod = 1.0;
            unsigned int k = 0;
            uint32_t blk = 0;
            for (int p = 0; p < my;) {
                const uint4 w = philox4x32_10(make_uint4((uint32_t)i, (uint32_t)(i >> 32), blk, 0u),
                                              k0, k1);
                ++blk;
                const uint32_t words[4] = {w.x, w.y, w.z, w.w};
                bool done = false;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double next = prod * (((double)words[u] + 0.5) * (1.0 / 4294967296.0));
                    prod = done ? prod : next;
                    done = done || !(prod > limit);
                    k += done ? 0u : 1u;
                }
                if (done) {
                    out[i] = (float)k;
                    ++p;
                    y += q;
                    x += rem;
                    if (x >= tw) {
                        x -= tw;
                        ++y;
                    }
                    i = (size_t)(y0 + y) * W + x0 + x;
                    limit = limits[(p < kChunk ? p : 0) * 64 + lane];
                    prod = 1.0;
                    k = 0;
                    blk = 0;
                }
            }
        }
    }
};

// WAITER: wait in[i] microseconds (clamped to [0, 1e6]), then copy the pixel.
struct WorkWaiter {
    static constexpr bool kList = false;
    static constexpr bool kNeighbours = false;
    __host__ __device__ static int radius(const WorkArgs &) { return 0; }
    __device__ static float pixel(const FarmCtx &c, const WorkArgs &a) {
        const float v = c.in[(size_t)c.y * c.W + c.x];
        float us = v;
        if (!(us > 0.0f))
            us = 0.0f;
        if (us > 1.0e6f)
            us = 1.0e6f;
        const long long ticks = (long long)((double)us * (double)a.wall_khz / 1000.0);
        const long long t0 = (long long)wall_clock64();
        while ((long long)wall_clock64() - t0 < ticks)
            __builtin_amdgcn_s_sleep(1);
        return v;
    }
};

// SOURCES: a pixel is a source when it exceeds the threshold and every other pixel
// of the frame within Chebyshev distance r is smaller, or equal and later in raster
// order (a plateau reports its first pixel).  The record's sums run over the
// in-frame pixels of the (2a+1)^2 box, row by row, in binary64 (no contraction),
// which fixes their rounding.  candidate() is the cheap test every pixel takes;
// find() runs on the candidates only.  The window is read row by row with 2R+1
// loads per row at clamped columns (R = max(r, a) <= 4, a compile-time bound chosen
// by a uniform switch), all rows unrolled, so the loads of a candidate overlap instead
// of each waiting for the one before.
template <int R>
__device__ __forceinline__ bool sources_find(const FarmCtx &c, const WorkArgs &a,
                                             SourceRec &rec) {
    constexpr int K = 2 * R + 1;
    const GFloat *in = (const GFloat *)c.in;
    const float v = in[(size_t)c.y * c.W + c.x];
    // away from the side edges a row's window is 2R+1 consecutive pixels: one address
    const bool inner = c.x >= R && c.x + R < c.W;
    bool peak = true;
#pragma unroll
    for (int dy = -R; dy <= R; ++dy) {
        const int yy = c.y + dy;
        if (dy < -a.r || dy > a.r || yy < 0 || yy >= c.H)
            continue;
        const GFloat *row = in + (size_t)yy * c.W;
        float q[K];
        if (inner) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                q[k] = row[c.x - R + k];
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k)
                q[k] = row[min(max(c.x - R + k, 0), c.W - 1)];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int dx = k - R, xx = c.x + dx;
            if (dx < -a.r || dx > a.r || xx < 0 || xx >= c.W || (dy == 0 && dx == 0))
                continue;
            const bool later = dy > 0 || (dy == 0 && dx > 0);
            if (!(q[k] < v) && !(later && q[k] == v))
                peak = false;
        }
    }
    if (!peak)
        return false;
    rec.y = c.y;
    rec.x = c.x;
    rec.peak = v;
    int npix = 0;
    double flux = 0.0, sy = 0.0, sx = 0.0;
    const double sky = (double)a.sky;
#pragma unroll
    for (int dy = -R; dy <= R; ++dy) {
        const int yy = c.y + dy;
        if (dy < -a.a || dy > a.a || yy < 0 || yy >= c.H)
            continue;
        const GFloat *row = in + (size_t)yy * c.W;
        float q[K];
        if (inner) {
#pragma unroll
            for (int k = 0; k < K; ++k)
                q[k] = row[c.x - R + k];
        } else {
#pragma unroll
            for (int k = 0; k < K; ++k)
                q[k] = row[min(max(c.x - R + k, 0), c.W - 1)];
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int dx = k - R, xx = c.x + dx;
            if (dx < -a.a || dx > a.a || xx < 0 || xx >= c.W)
                continue;
            const double d = (double)q[k] - sky;
            flux = flux + d;
            sy = sy + (double)dy * d;
            sx = sx + (double)dx * d;
            ++npix;
        }
    }
    rec.npix = npix;
    rec.flux = flux;
    rec.sy = sy;
    rec.sx = sx;
    return true;
}

// The same test and sums with run-time loops, for radii above 4 (larger unrolled
// windows would not fit in registers).
__device__ __forceinline__ bool sources_find_loops(const FarmCtx &c, const WorkArgs &a,
                                                   SourceRec &rec) {
    const float *p = c.in + (size_t)c.y * c.W + c.x;
    const float v = p[0];
    const int ya = max(c.y - a.r, 0), yb = min(c.y + a.r, c.H - 1);
    const int xa = max(c.x - a.r, 0), xb = min(c.x + a.r, c.W - 1);
    for (int yy = ya; yy <= yb; ++yy) {
        const float *row = c.in + (size_t)yy * c.W;
        for (int xx = xa; xx <= xb; ++xx) {
            const float q = row[xx];
            const bool later = yy > c.y || (yy == c.y && xx > c.x);
            if (!(q < v) && !(later && q == v) && (yy != c.y || xx != c.x))
                return false;
        }
    }
    rec.y = c.y;
    rec.x = c.x;
    rec.peak = v;
    int npix = 0;
    double flux = 0.0, sy = 0.0, sx = 0.0;
    const double sky = (double)a.sky;
    for (int dy = -a.a; dy <= a.a; ++dy) {
        if (c.y + dy < 0 || c.y + dy >= c.H)
            continue;
        const float *row = p + (ptrdiff_t)dy * c.W;
        for (int dx = -a.a; dx <= a.a; ++dx) {
            if (c.x + dx < 0 || c.x + dx >= c.W)
                continue;
            const double d = (double)row[dx] - sky;
            flux = flux + d;
            sy = sy + (double)dy * d;
            sx = sx + (double)dx * d;
            ++npix;
        }
    }
    rec.npix = npix;
    rec.flux = flux;
    rec.sy = sy;
    rec.sx = sx;
    return true;
}

struct WorkSources {
    static constexpr bool kList = true;
    static constexpr bool kNeighbours = true;
    __host__ __device__ static int radius(const WorkArgs &a) { return a.r > a.a ? a.r : a.a; }
    __device__ static bool candidate(float v, const WorkArgs &a) { return v > a.threshold; }
    // Necessary for a source when r >= 1: the direct neighbours above and to the left
    // (earlier in raster order) are smaller, those below and to the right are not
    // larger.  A neighbour the scan does not know, or that lies outside the frame,
    // comes as -inf and passes.
    __device__ static bool neighbours(float v, float up, float dn, float lf, float rt,
                                      const WorkArgs &a) {
        return a.r < 1 || (up < v && lf < v && !(dn > v) && !(rt > v));
    }
    __device__ static bool find(const FarmCtx &c, const WorkArgs &a, SourceRec &rec) {
        switch (radius(a)) {
        case 1: return sources_find<1>(c, a, rec);
        case 2: return sources_find<2>(c, a, rec);
        case 3: return sources_find<3>(c, a, rec);
        case 4: return sources_find<4>(c, a, rec);
        default: return sources_find_loops(c, a, rec);
        }
    }
};

// Queues in use, nq: no more than waves, a power of two (an actor that walks through queues nobody
// else takes from pays an atomic for each: with 32 queues for 16 actors, 64 rows of 128 pixels at
// mean 0.5 took 43 us, with 16 they take 29).
__host__ __device__ inline int queues_log2(int waves) {
    int l = 0;
    while (2 << l <= waves && 2 << l <= kFarmQueues)
        ++l;
    return l;
}

// A queue's line of tickets: [0] the tiles handed out, [1] a copy of the mask of drained
// queues.  The first run of each wave needs no ticket (wave g takes run g / nq of queue g % nq),
// so the counters start behind these runs.
__global__ void k_farm_reset(unsigned int *tickets, long long ntiles, int waves, int chunk,
                             unsigned long long *count) {
    const int q = (int)threadIdx.x;               // one wave
    const int lq = queues_log2(waves), nq = 1 << lq;
    const long long size = (ntiles * (q + 1) >> lq) - (ntiles * q >> lq);
    const long long start = (long long)((waves - q + nq - 1) >> lq) * chunk;
    const unsigned int drained = (unsigned int)__ballot(q < nq && start >= size);
    if (q < nq) {
        tickets[q * kFarmStride] = (unsigned int)start;
        tickets[q * kFarmStride + 1] = drained;
    }
    if (q == 0 && count)
        *count = 0ull;
}

// The value of the lane before and of the lane after (-inf at the wave's ends).
__device__ __forceinline__ float lane_before(float v) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(
        (int)0xff800000, (int)__float_as_uint(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_after(float v) {
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(
        (int)0xff800000, (int)__float_as_uint(v), 0x130, 0xf, 0xf, false));
}

// The next run of tiles for the calling wave, or t0 = -1 when every queue is drained.
// The wave's first run is `first` of its queue (then first is -1); after that lane 0 takes a
// ticket from the wave's current queue, and once that queue is drained the wave moves to the
// next one (in cyclic order) that it does not know to be.  The wave that draws the first ticket
// past a queue's end says so in every line's mask; the others read the mask in the line they
// draw from.  (Atomics, and reads past the L2s, of one line serialise at about 11 ns: with all
// counters in one line, and each wave reading all of them at its end, SOURCES on a 4096 x 4096
// frame took 206 us on 4096 actors and POISSON on 750 x 750 pixels in rows 49 on 1024; with a
// line for each, the first runs without tickets and the masks, 59 and 33.)
__device__ __forceinline__ void next_tiles(unsigned int *__restrict__ tickets, long long ntiles,
                                           int chunk, int lq, int &first,
                                           unsigned int &drained, int &queue, long long &t0,
                                           long long &t1) {
    const int lane = __lane_id();
    for (;;) {
        const long long q0 = ntiles * queue >> lq;
        const long long q1 = ntiles * (queue + 1) >> lq;
        unsigned int *const line = tickets + queue * kFarmStride;
        const bool ticket = first < 0;
        unsigned int got = ticket ? 0u : (unsigned int)first * (unsigned int)chunk;
        if (ticket && lane == 0)
            got = atomicAdd(&line[0], (unsigned int)chunk);
        first = -1;
        got = __builtin_amdgcn_readfirstlane(got);
        if (q0 + got < q1) {
            t0 = q0 + got;
            t1 = min(q1, t0 + chunk);
            return;
        }
        if (ticket && q0 + got - chunk < q1 && lane < 1 << lq)
            atomicOr(&tickets[lane * kFarmStride + 1], 1u << queue);
        unsigned int seen = 0u;
        if (lane == 0)
            seen = __hip_atomic_load(&line[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        drained |= __builtin_amdgcn_readfirstlane(seen) | 1u << queue;
        const unsigned int open = ~drained;
        if (!open) {
            t0 = t1 = -1;
            return;
        }
        const unsigned int after = open & ~((2u << queue) - 1u);
        queue = __ffs((int)(after ? after : open)) - 1;
    }
}

// The first of n slots of the caller's list, reserved for the wave by one atomic on the counter.
__device__ __forceinline__ unsigned long long reserve_records(int n,
                                                              unsigned long long *count) {
    unsigned long long base = 0ull;
    if (__lane_id() == 0)
        base = atomicAdd(count, (unsigned long long)n);
    const unsigned int lo = __builtin_amdgcn_readfirstlane((unsigned int)base);
    const unsigned int hi = __builtin_amdgcn_readfirstlane((unsigned int)(base >> 32));
    return ((unsigned long long)hi << 32) | lo;
}
// Moves n buffered records to the slots from base on, by the wave, as 8-byte words.
__device__ __forceinline__ void flush_records(const SourceRec *__restrict__ buf, int n,
                                              SourceRec *__restrict__ out_list,
                                              long long capacity, unsigned long long base) {
    constexpr int kWords = (int)(sizeof(SourceRec) / 8);
    const int lane = __lane_id();
    const unsigned long long *src = reinterpret_cast<const unsigned long long *>(buf);
    unsigned long long *dst = reinterpret_cast<unsigned long long *>(out_list);
    for (int i = lane; i < n * kWords; i += 64)
        if (base + (unsigned long long)(i / kWords) < (unsigned long long)capacity)
            dst[base * kWords + i] = src[i];
}

// The farm.  Every wave is an actor: it takes runs of `chunk` tiles from the tickets
// (tiles numbered row-major, split into nq contiguous ranges, up to kFarmQueues; a wave starts
// on the queue of its global wave index modulo nq -- workgroups are dealt
// round-robin to the XCDs, so a queue's tiles mostly stay in one XCD's L2) and works
// through each tile 64 pixels at a time, with no workgroup barrier.
//   Image work functions compute every pixel of the tile.
//   List work functions first scan the tile with a batch of loads in flight per lane
//   and compact the pixels that pass candidate() (and, for a function that declares
//   kNeighbours, neighbours() on the direct neighbours the batch holds) into a
//   per-wave LDS list; all lanes then run find() on the list (one candidate per lane)
//   and buffer the records they find per wave, moving them to the caller's list when
//   the buffer could not take another pass and at the end.  When tile_w is a multiple
//   of 64 (at most 256, with at most 256 rows) a batch is 16 rows of 64 pixels read by
//   buffer loads with a uniform row offset, and a tile's candidates gather in one list
//   (16-bit positions) so that find() runs on full passes.
template <class WF>
__global__ __launch_bounds__(256) void k_farm(const float *__restrict__ in, int H, int W,
                                              WorkArgs args, int tile_h, int tile_w, int chunk,
                                              int waves, float *__restrict__ out_img,
                                              SourceRec *__restrict__ out_list,
                                              long long capacity,
                                              unsigned long long *__restrict__ count,
                                              unsigned int *__restrict__ tickets) {
    constexpr int kScanBatch = 16;
    constexpr int kBufBatch = 16;   // rows of 64 pixels per batch of the buffer scan
    __shared__ int sCand[WF::kList ? 4 * kFarmCandidates : 1];
    __shared__ SourceRec sRec[WF::kList ? 4 * kFarmWaveRecords : 1];
    constexpr bool kTiles = std::is_same<WF, WorkPoisson>::value;
    __shared__ double sLimits[kTiles ? 4 * WorkPoisson::kChunk * 64 : 1];
    const int wave = threadIdx.x >> 6, lane = __lane_id();
    const int gwave = blockIdx.x * 4 + wave;
    __shared__ int sLeft[4];                // records a wave leaves at its end
    __shared__ unsigned int sEnded;         // waves that have ended
    if constexpr (WF::kList) {
        if (threadIdx.x == 0)
            sEnded = 0u;
        __syncthreads();
    }
    if (gwave >= waves)
        return;
    int *cand = sCand + (WF::kList ? wave * kFarmCandidates : 0);
    SourceRec *rbuf = sRec + (WF::kList ? wave * kFarmWaveRecords : 0);
    int nrec = 0;
    const int ntx = (W - 1) / tile_w + 1;
    const long long ntiles = (long long)ntx * ((H - 1) / tile_h + 1);
    const int lq = queues_log2(waves);
    int queue = gwave & ((1 << lq) - 1), first = gwave >> lq;
    unsigned int drained = lq == 5 ? 0u : ~0u << (1 << lq);      // the queues not in use
    static_assert(kFarmQueues == 32, "a mask of 32 queues");
    FarmCtx c;
    c.in = in;
    c.H = H;
    c.W = W;
    for (;;) {
        long long t0, t1;
        next_tiles(tickets, ntiles, chunk, lq, first, drained, queue, t0, t1);
        if (t0 < 0)
            break;
        for (long long t = t0; t < t1; ++t) {
            const int y0 = (int)(t / ntx) * tile_h, x0 = (int)(t % ntx) * tile_w;
            const int th = min(tile_h, H - y0), tw = min(tile_w, W - x0);
            const long long n = (long long)th * tw;
            const int q = 64 / tw, rem = 64 - q * tw;
            int ly = lane / tw, lx = lane - ly * tw;
            if constexpr (kTiles) {
                WF::tile(in, out_img, W, args, y0, x0, tw, n,
                         sLimits + wave * WorkPoisson::kChunk * 64);
            } else if constexpr (!WF::kList) {
                for (long long j0 = 0; j0 < n; j0 += 64) {
                    if (j0 + lane < n) {
                        c.y = y0 + ly;
                        c.x = x0 + lx;
                        out_img[(size_t)c.y * W + c.x] = WF::pixel(c, args);
                    }
                    ly += q;
                    lx += rem;
                    if (lx >= tw) {
                        lx -= tw;
                        ++ly;
                    }
                }
            } else {
                // candidates run on one lane each; the find pass over the list
                uint16_t *const cand16 = reinterpret_cast<uint16_t *>(cand);
                auto run_candidates = [&](int ncand, bool packed) {
                    for (int i0 = 0; i0 < ncand; i0 += 64) {
                        SourceRec rec;
                        bool found = false;
                        if (i0 + lane < ncand) {
                            const int p = packed ? (int)cand16[i0 + lane] : cand[i0 + lane];
                            c.y = y0 + (packed ? (p >> 8) : p / tw);
                            c.x = x0 + (packed ? (p & 0xFF) : p % tw);
                            found = WF::find(c, args, rec);
                        }
                        const unsigned long long m = __ballot(found);
                        if (found)
                            rbuf[nrec + __popcll(m & ((1ull << lane) - 1ull))] = rec;
                        nrec += __popcll(m);
                        if (nrec > kFarmWaveRecords - 64) {
                            flush_records(rbuf, nrec, out_list, capacity,
                                          reserve_records(nrec, count));
                            nrec = 0;
                        }
                    }
                };
                int ncand = 0;
                if ((tile_w & 63) == 0 && tile_w <= 256 && th <= 256 &&
                    (long long)(th - 1) * W + tw < (1ll << 29)) {
                    // rows of whole 64-pixel segments: buffer loads over the tile's rows
                    // with the lane's byte offset and a uniform segment offset, so a load
                    // costs no vector instruction; candidates packed in 16 bits as
                    // (row << 8) | col, so twice as many wait for a full pass
                    const int nseg = tile_w >> 6;
                    const long long steps = (long long)th * nseg;
                    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
                        (void *)(in + (size_t)y0 * W + x0), (short)0,
                        (int)(((long long)(th - 1) * W + tw) * 4), kBufWord3);
                    float carry = -INFINITY;        // the row above a batch (nseg == 1)
                    // batch s0: rows of 64 pixels s0 .. s0+kBufBatch-1 in segment order
                    auto load_batch = [&](float (&v)[kBufBatch], long long s0) {
                        int row = (int)(s0 / nseg), seg = (int)(s0 - (long long)row * nseg);
#pragma unroll
                        for (int b = 0; b < kBufBatch; ++b) {
                            v[b] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                                rows, lane * 4, s0 + b < steps ? (row * W + seg * 64) * 4 : 0,
                                0));
                            if (++seg == nseg) {
                                seg = 0;
                                ++row;
                            }
                        }
                    };
                    for (long long s0 = 0; s0 < steps; s0 += kBufBatch) {
                        float v[kBufBatch];
                        load_batch(v, s0);
                        int row = (int)(s0 / nseg), seg = (int)(s0 - (long long)row * nseg);
#pragma unroll
                        for (int b = 0; b < kBufBatch; ++b) {
                            const int col = seg * 64 + lane;
                            bool hit = s0 + b < steps && col < tw && WF::candidate(v[b], args);
                            if constexpr (WF::kNeighbours) {
                                // direct neighbours this batch holds (same row: adjacent
                                // lanes; rows above and below: adjacent batch entries
                                // when a row is one segment)
                                const float lf = lane_before(v[b]), rt = lane_after(v[b]);
                                float up = -INFINITY, dn = -INFINITY;
                                if (nseg == 1) {
                                    up = b > 0 ? v[b > 0 ? b - 1 : 0] : carry;
                                    if (b + 1 < kBufBatch && s0 + b + 1 < steps)
                                        dn = v[b + 1 < kBufBatch ? b + 1 : b];
                                }
                                hit = hit && WF::neighbours(v[b], up, dn,
                                                           lf, col + 1 < tw ? rt : -INFINITY,
                                                           args);
                            }
                            const unsigned long long m = __ballot(hit);
                            if (hit)
                                cand16[ncand + __popcll(m & ((1ull << lane) - 1ull))] =
                                    (uint16_t)((row << 8) | col);
                            ncand += __popcll(m);
                            if (++seg == nseg) {
                                seg = 0;
                                ++row;
                            }
                        }
                        carry = v[kBufBatch - 1];
                        if (ncand > 2 * kFarmCandidates - kBufBatch * 64 ||
                            s0 + kBufBatch >= steps) {
                            run_candidates(ncand, true);
                            ncand = 0;
                        }
                    }
                } else {
                long long j0 = 0;
                while (j0 < n) {
                    // scan up to kScanBatch passes, all loads first
                    float v[kScanBatch];
                    int pos[kScanBatch];
#pragma unroll
                    for (int b = 0; b < kScanBatch; ++b) {
                        // unconditional loads (a lane past the tile's end rereads the
                        // tile's first pixel and ignores it), so none waits for another
                        const bool in_tile = j0 + b * 64 + lane < n;
                        const int yy = in_tile ? y0 + ly : y0, xx = in_tile ? x0 + lx : x0;
                        v[b] = in[(size_t)yy * W + xx];
                        pos[b] = in_tile ? ly * tw + lx : -1;
                        ly += q;
                        lx += rem;
                        if (lx >= tw) {
                            lx -= tw;
                            ++ly;
                        }
                    }
#pragma unroll
                    for (int b = 0; b < kScanBatch; ++b) {
                        const bool hit = pos[b] >= 0 && WF::candidate(v[b], args);
                        const unsigned long long m = __ballot(hit);
                        if (hit)
                            cand[ncand + __popcll(m & ((1ull << lane) - 1ull))] = pos[b];
                        ncand += __popcll(m);
                    }
                    j0 += kScanBatch * 64;
                    // run the candidates when the list could not take another batch,
                    // and at the end of the tile
                    if (ncand > kFarmCandidates - kScanBatch * 64 || j0 >= n) {
                        run_candidates(ncand, false);
                        ncand = 0;
                    }
                }
                }
            }
        }
    }
    if constexpr (WF::kList) {
        // the records left over go out together, by the block's last wave to end: the
        // reservations of all waves are atomics on one address, which take 11 ns each
        unsigned int ended = 0u;
        if (lane == 0) {
            sLeft[wave] = nrec;
            __threadfence_block();
            ended = atomicAdd(&sEnded, 1u);
            __threadfence_block();
        }
        const int nw = min(4, waves - (int)blockIdx.x * 4);
        if (__builtin_amdgcn_readfirstlane(ended) + 1u == (unsigned int)nw) {
            int total = 0;
            for (int w = 0; w < nw; ++w)
                total += sLeft[w];
            unsigned long long base = total ? reserve_records(total, count) : 0ull;
            for (int w = 0; w < nw; ++w) {
                flush_records(sRec + w * kFarmWaveRecords, sLeft[w], out_list, capacity, base);
                base += (unsigned long long)sLeft[w];
            }
        }
    }
}

template <class WF>
hipError_t launch_kind(const WorkArgs &args, const float *in, int H, int W, int workers,
                       int tile_h, int tile_w, float *out_img, SourceRec *out_list,
                       long long capacity, unsigned long long *count, unsigned int *tickets,
                       hipStream_t s) {
    // tickets of `chunk` tiles: about 2 per wave; atomics on a ticket counter serialise
    // in its L2, so few and spread over kFarmQueues counters keep them off the path
    const long long ntiles = (long long)((W - 1) / tile_w + 1) * ((H - 1) / tile_h + 1);
    long long chunk = ntiles / ((long long)workers * 2);
    chunk = chunk < 1 ? 1 : (chunk > 64 ? 64 : chunk);
    const int blocks = (workers + 3) / 4;
    k_farm_reset<<<1, 64, 0, s>>>(tickets, ntiles, workers, (int)chunk, count);
    k_farm<WF><<<blocks, 256, 0, s>>>(in, H, W, args, tile_h, tile_w, (int)chunk, workers,
                                      out_img, out_list, capacity, count, tickets);
    return hipGetLastError();
}

int work_radius(int kind, const WorkArgs &a, int niter) {
    switch (kind) {
    case kWorkLacosmic:
        return 8 * niter;     // per iteration: detection 4, two grows 1 each, replacement 2
    case kWorkPoisson:
        return WorkPoisson::radius(a);
    case kWorkWaiter:
        return WorkWaiter::radius(a);
    case kWorkSources:
        return WorkSources::radius(a);
    default:
        return -1;
    }
}

hipError_t launch_farm(int kind, const WorkArgs &args, const float *in, int H, int W,
                       int workers, int tile_h, int tile_w, float *out_img,
                       SourceRec *out_list, long long capacity, unsigned long long *count,
                       unsigned int *tickets, hipStream_t s) {
    switch (kind) {
    case kWorkPoisson:
        return launch_kind<WorkPoisson>(args, in, H, W, workers, tile_h, tile_w, out_img,
                                        out_list, capacity, count, tickets, s);
    case kWorkWaiter:
        return launch_kind<WorkWaiter>(args, in, H, W, workers, tile_h, tile_w, out_img,
                                       out_list, capacity, count, tickets, s);
    case kWorkSources:
        return launch_kind<WorkSources>(args, in, H, W, workers, tile_h, tile_w, out_img,
                                        out_list, capacity, count, tickets, s);
    default:
        return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// raster order of a SOURCES list
// ---------------------------------------------------------------------------
//
// Every record sits on a pixel of its own, so a bitmap of the frame's pixels sorts the list:
// a record's place is the number of set bits before its own.  Five short launches: clear and
// set the bitmap, sum it per chunk of kOrderChunk words, prefix sums per word, and the copy.
// They move 12 bytes per 64 pixels twice and the records once (about 20 us for 43,000 records
// of a 4096 x 4096 frame, where sorting them on the host took 4 ms).

__global__ __launch_bounds__(256) void k_order_clear(unsigned long long *__restrict__ map,
                                                     long long words) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < words;
         i += (long long)gridDim.x * 256)
        map[i] = 0ull;
}

// The pixel index of a record, or -1 outside the frame.
__device__ __forceinline__ long long record_pixel(const SourceRec &r, int H, int W) {
    return r.y >= 0 && r.y < H && r.x >= 0 && r.x < W ? (long long)r.y * W + r.x : -1ll;
}

__global__ __launch_bounds__(256) void k_order_mark(const SourceRec *__restrict__ list,
                                                    long long n, int H, int W,
                                                    unsigned long long *__restrict__ map) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n;
         i += (long long)gridDim.x * 256) {
        const long long p = record_pixel(list[i], H, W);
        if (p >= 0)
            atomicOr(&map[p >> 6], 1ull << (p & 63));
    }
}

// One block per chunk: the set bits of its words.
__global__ __launch_bounds__(256) void k_order_sum(const unsigned long long *__restrict__ map,
                                                   long long words,
                                                   unsigned int *__restrict__ sums) {
    __shared__ unsigned int part[4];
    const long long w0 = (long long)blockIdx.x * kOrderChunk;
    unsigned int c = 0u;
    for (int i = threadIdx.x; i < kOrderChunk; i += 256)
        c += w0 + i < words ? (unsigned int)__popcll(map[w0 + i]) : 0u;
    c = __ockl_wfred_add_u32(c);
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0)
        sums[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}

// One block per chunk: the set bits before each of its words.
__global__ __launch_bounds__(256) void k_order_prefix(const unsigned long long *__restrict__ map,
                                                      long long words,
                                                      const unsigned int *__restrict__ sums,
                                                      unsigned int *__restrict__ before) {
    constexpr int kPer = kOrderChunk / 256;
    __shared__ unsigned int part[8];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned int base = 0u;              // the chunks before this one
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256)
        base += sums[i];
    base = __ockl_wfred_add_u32(base);
    const long long w0 = (long long)blockIdx.x * kOrderChunk + (long long)threadIdx.x * kPer;
    unsigned int c[kPer], tot = 0u;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        c[i] = w0 + i < words ? (unsigned int)__popcll(map[w0 + i]) : 0u;
        tot += c[i];
    }
    unsigned int at = __ockl_wfscan_add_u32(tot, false);
    if (lane == 63)
        part[wave] = at + tot;
    if (lane == 0)
        part[4 + wave] = base;
    __syncthreads();
    at += part[4] + part[5] + part[6] + part[7];
    for (int q = 0; q < wave; ++q)
        at += part[q];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (w0 + i < words)
            before[w0 + i] = at;
        at += c[i];
    }
}

// Five lanes per record, 8 bytes each.
__global__ __launch_bounds__(256) void k_order_copy(const SourceRec *__restrict__ list,
                                                    long long n, int H, int W,
                                                    const unsigned long long *__restrict__ map,
                                                    const unsigned int *__restrict__ before,
                                                    SourceRec *__restrict__ out) {
    constexpr int kWords = (int)(sizeof(SourceRec) / 8);
    const unsigned long long *src = reinterpret_cast<const unsigned long long *>(list);
    unsigned long long *dst = reinterpret_cast<unsigned long long *>(out);
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n * kWords;
         i += (long long)gridDim.x * 256) {
        const long long rec = i / kWords;
        const long long p = record_pixel(list[rec], H, W);
        if (p >= 0) {
            const long long at = (long long)before[p >> 6] +
                                 __popcll(map[p >> 6] & ((1ull << (p & 63)) - 1ull));
            dst[at * kWords + (i - rec * kWords)] = src[i];
        }
    }
}

hipError_t launch_order(const SourceRec *list, long long n, int H, int W, SourceRec *out,
                        void *work, hipStream_t s) {
    const long long words = (long long)order_words(H, W);
    const int chunks = (int)order_chunks(H, W);
    unsigned long long *map = static_cast<unsigned long long *>(work);
    unsigned int *before = reinterpret_cast<unsigned int *>(map + words);
    unsigned int *sums = before + words;
    auto grid = [](long long items) {
        const long long g = (items + 255) / 256;
        return (unsigned int)(g < 4096 ? g : 4096);
    };
    k_order_clear<<<grid(words), 256, 0, s>>>(map, words);
    k_order_mark<<<grid(n), 256, 0, s>>>(list, n, H, W, map);
    k_order_sum<<<chunks, 256, 0, s>>>(map, words, sums);
    k_order_prefix<<<chunks, 256, 0, s>>>(map, words, sums, before);
    k_order_copy<<<grid(n * 5), 256, 0, s>>>(list, n, H, W, map, before, out);
    return hipGetLastError();
}

}  // namespace crb
