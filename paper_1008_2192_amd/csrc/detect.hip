// First-iteration detection of libcrb for gfx950 (MI355X): the first stage of an L.A.Cosmic
// iteration (Mighell, Section 5) -- L+ (2x-subsampled clipped Laplacian, rebinned),
// N from med5(J), S = L+/(2N), S' = S - med5(S), F^ from med3(J) - med7(med3(J)),
// the first selection and the two threshold bits the grow reads -- on LDS tiles of 64
// columns by 16, 32 or 64 rows with the halo each quantity needs, one block per tile or
// persistent blocks taking tiles from ticket counters, plus the parity-test kernels of
// its median networks.  Later iterations re-evaluate the codes where J changed (step.hip).
//
// Numerics: medians are exact selections by min/max networks.  Every decision (a
// threshold bit, the contrast test) is the one the binary64 definition takes: S is
// estimated in FP32 with a proven error bound, a decision is taken from the estimate
// only when the bound settles it, and otherwise from binary64 statistics evaluated in
// the definition's operation order (no contraction: built with -ffp-contract=off).
// So the codes for a given J are independent of the tiling and of the launch shape.
#include "detect_tile.h"

namespace crb {

// Run length of the 3x3 median network's parity kernel (sorted columns shared by runs).
constexpr int kRun3 = 14;

// The first iteration's detection of one tile (origin y0, x0 of frame f), by the whole
// block: the codes of the input frame, and the state every later launch starts from -- J (a
// copy of the input), a cleared mask and its bitmap, the tile's code buffer and list mark, the
// frame's counters.  Every early return is taken by all threads alike.
// NARROW: the frame may store its bit rows in a narrow form (DevFrame::narrow).
template <int TY, bool NARROW>
__device__ __forceinline__ void detect_tile(const DevFrame &f, int y0, int x0, int tid) {
    using L = DetectLds<TY, 4, false>;
    constexpr int TX = L::TX, NT = L::NT;
    __shared__ L s;
    // 12 blocks of 16 rows, 6 of 32 rows, 3 of 64 rows per CU (the CU hands out LDS in
    // 1 KiB units): about 24 waves
    static_assert(sizeof(L) <= (TY == 16 ? 15360 : (TY == 32 ? 26624 : 53248)),
                  "the LDS of a detection block must let its resident blocks share a CU");
    static_assert(TY * TX == 8 * NT, "one 8-pixel row segment per thread");
    static_assert(kSumTX == TX && kSumTY == 32 && (TY == 16 || TY % kSumTY == 0),
                  "tiles on the summary grid");
    if (f.niter < 1)
        return;
    const int H = f.H, W = f.W;
    detect_clear(s, tid);
    JStage<L, 4> stage;
#pragma unroll
    for (int b0 = 0; b0 < stage.kBlocks; b0 += stage.kRound) {
        stage.load(f.img, H, W, y0, x0, tid, b0);
        stage.store(s, tid, b0);
    }
    if (f.count && y0 == 0 && x0 == 0) {
        for (int i = tid; i < f.niter; i += NT)
            f.any_new[i] = 0u;
        if (tid < kCountSlots)
            f.count[tid * kCountStride] = 0ull;
    }
    __syncthreads();
    const int ntx = (W + kSumTX - 1) / kSumTX;
    {
        const int r = tid / (TX / 8), cs = (tid - r * (TX / 8)) * 8;
        const int gy = y0 + r, gx = x0 + cs;
        const bool inside = gy < H && gx < W;
        // the tile's own pixels of the input become J, 8 per thread
        if (f.img != f.J && inside) {
            const float *src = &s.j4()[(r + 4) * L::JWP + cs + 4];
            float *dst = f.J + (size_t)gy * W + gx;
            if (gx + 8 <= W && ((uintptr_t)dst & 15u) == 0u) {
                reinterpret_cast<float4 *>(dst)[0] = make_float4(src[0], src[1], src[2], src[3]);
                reinterpret_cast<float4 *>(dst)[1] = make_float4(src[4], src[5], src[6], src[7]);
            } else {
                const int nb = min(8, W - gx);
                for (int j = 0; j < nb; ++j)
                    dst[j] = src[j];
            }
        }
        // an uninitialised mask is cleared; a given one becomes the tile's mask bitmap
        uint32_t mbyte = 0u;
        if (f.mask && inside) {
            uint8_t *dst = f.mask + (size_t)gy * W + gx;
            if (!(f.flags & kFreshMask)) {
                for (int j = 0; j < min(8, W - gx); ++j)
                    mbyte |= dst[j] ? 1u << j : 0u;
            } else if (gx + 8 <= W && ((uintptr_t)dst & 7u) == 0u) {
                *reinterpret_cast<uint2 *>(dst) = make_uint2(0u, 0u);
            } else {
                const int nb = min(8, W - gx);
                for (int j = 0; j < nb; ++j)
                    dst[j] = 0;
            }
        }
        if (f.mbits && !(NARROW && f.narrow)) {
            const int t = (y0 + r) / kSumTY * ntx + x0 / kSumTX;
            if (y0 + r < (H + kSumTY - 1) / kSumTY * kSumTY)
                reinterpret_cast<uint8_t *>(f.mbits + (size_t)t * kSumTY +
                                            ((y0 + r) & (kSumTY - 1)))[cs >> 3] = (uint8_t)mbyte;
        }
    }
    detect_staged(s, f, y0, x0, tid);

    // the code planes of the summary tiles the block covers (buffer 0), their state words
    const unsigned long long *code = reinterpret_cast<const unsigned long long *>(s.code);
    if constexpr (NARROW) {
        static_assert(!NARROW || (TY == kSumTY && NT == 256), "a summary tile, four waves");
        if (f.narrow && f.bits) {
            // a plane per wave: the codes, and the mask's bits
            const int p = __builtin_amdgcn_readfirstlane(tid >> 6), row = tid & 63;
            const size_t t = (size_t)(y0 / kSumTY * ntx + x0 / kSumTX);
            unsigned long long v = 0ull;
            if (p < 3) {
                v = row < TY ? code[p * TY + row] : 0ull;
            } else if (row < TY && y0 + row < H && !(f.flags & kFreshMask)) {
                for (int c = 0; c < TX && x0 + c < W; ++c)
                    v |= f.mask[(size_t)(y0 + row) * W + x0 + c] ? 1ull << c : 0ull;
            }
            narrow_store(f, p < 3 ? f.bits : f.mbits, p < 3 ? t * 6 + p : t, row, v);
        }
    }
    if (f.bits) {
        for (int i = tid; i < 3 * TY && !(NARROW && f.narrow); i += NT) {
            const int p = i / TY, r = i - p * TY;
            if (y0 + (r & ~(kSumTY - 1)) < H)
                f.bits[((size_t)((y0 + r) / kSumTY * ntx + x0 / kSumTX) * 2 * 3 + p) * kSumTY +
                       ((y0 + r) & (kSumTY - 1))] = code[i];
        }
        // (the halves of a summary tile, in tiles of 16 rows, write the same words)
        if (tid < (TY + kSumTY - 1) / kSumTY && y0 + kSumTY * tid < H) {
            const size_t t = (size_t)(y0 / kSumTY + tid) * ntx + x0 / kSumTX;
            f.state[t] = 1u << 1;
            f.mark[t] = 0u;
        }
    }
    if (f.codes) {        // parity tests: the codes as bytes
        const int r = tid / (TX / 8), cs = (tid - r * (TX / 8)) * 8;
        for (int j = 0; j < 8; ++j)
            if (y0 + r < H && x0 + cs + j < W)
                f.codes[(size_t)(y0 + r) * W + x0 + cs + j] =
                    (uint8_t)((code[r] >> (cs + j) & 1ull) |
                              (code[TY + r] >> (cs + j) & 1ull) << 1 |
                              (code[2 * TY + r] >> (cs + j) & 1ull) << 2);
    }
}

// (frame, tile origin) of tile t of a launch: from the work list, or for a single frame
// (tiles == null) the row-major tile t of its grid.
template <int TY>
__device__ __forceinline__ void tile_of(const DevFrame *__restrict__ frames,
                                        const TileRef *__restrict__ tiles, const DevFrame &single,
                                        int t, DevFrame &f, int &y0, int &x0) {
    if (tiles) {
        const TileRef r = tiles[t];
        f = frames[r.frame];
        y0 = r.y0;
        x0 = r.x0;
    } else {
        f = single;
        const int ntx = (single.W + kSumTX - 1) / kSumTX;
        y0 = (t / ntx) * TY;
        x0 = (t - (t / ntx) * ntx) * kSumTX;
    }
}

// One block per tile.
template <int TY, bool NARROW>
__global__ __launch_bounds__(8 * TY) __attribute__((amdgpu_waves_per_eu(TY == 16 ? 4 : 6)))
void k_detect(const DevFrame *__restrict__ frames, const TileRef *__restrict__ tiles,
              DevFrame single, StepLists lists) {
    DevFrame f;
    int y0, x0;
    tile_of<TY>(frames, tiles, single, (int)blockIdx.x, f, y0, x0);
    if (blockIdx.x == 0)
        lists_start(lists, (int)threadIdx.x);
    detect_tile<TY, NARROW>(f, y0, x0, (int)threadIdx.x);
}

// Persistent blocks over a (frame, tile) work list: the grid holds about as many
// blocks as are resident at once, and each block takes runs of kRun consecutive tiles
// from kDetectQueues ticket counters (zero at launch, each on its own cache line),
// counter q over the q-th contiguous part of the list (the first iteration kernel after
// this launch zeroes them for the next).  Blocks are dispatched
// round-robin over the XCDs, so block b starts on part b mod kDetectQueues, and the
// tiles in flight on one XCD are neighbours sharing halo rows and columns in its L2; a
// block whose part is used up moves to the next, and it returns once all parts are
// (every counter only grows, so every block gets there).
template <int TY>
__global__ __launch_bounds__(8 * TY) __attribute__((amdgpu_waves_per_eu(TY == 16 ? 4 : 6)))
void k_detect_persistent(const DevFrame *__restrict__ frames, const TileRef *__restrict__ tiles,
                         StepLists lists, int ntiles, unsigned int *__restrict__ tickets) {
    constexpr int kRun = 2;
    __shared__ int sTile, sEnd;
    int q = (int)(blockIdx.x % kDetectQueues), tried = 0;
    if (blockIdx.x == 0)
        lists_start(lists, (int)threadIdx.x);
    for (;;) {
        __syncthreads();      // the previous run is done with the LDS and with sTile
        if (threadIdx.x == 0) {
            int t = -1, end = -1;
            while (tried < kDetectQueues) {
                const unsigned int lo = (unsigned int)((long long)ntiles * q / kDetectQueues);
                const unsigned int hi =
                    (unsigned int)((long long)ntiles * (q + 1) / kDetectQueues);
                const unsigned int got =
                    lo + (unsigned int)kRun * atomicAdd(&tickets[q * kTicketStride], 1u);
                if (got < hi) {
                    t = (int)got;
                    end = (int)min(got + (unsigned int)kRun, hi);
                    break;
                }
                q = (q + 1) % kDetectQueues;
                ++tried;
            }
            sTile = t;
            sEnd = end;
        }
        __syncthreads();
        // uniform over the block: the tile and frame records then load into scalar
        // registers, as with blockIdx.x in the one-block-per-tile kernel
        const int t0 = __builtin_amdgcn_readfirstlane(sTile);
        const int t1 = __builtin_amdgcn_readfirstlane(sEnd);
        if (t0 < 0)
            return;
        for (int t = t0; t < t1; ++t) {
            if (t > t0)
                __syncthreads();   // the previous tile is done with the LDS
            const TileRef r = tiles[t];
            // the frame record is read in place, each field where the tile first needs it,
            // rather than copied whole into scalar registers at the start of every tile
            const DevFrame &f = frames[r.frame];
            // the thread index passes through an empty asm statement each round, so that
            // values derived from it are recomputed per tile rather than held in registers
            // across the loop
            int tid = (int)threadIdx.x;
            asm volatile("" : "+v"(tid));
            detect_tile<TY, false>(f, r.y0, r.x0, tid);
        }
    }
}

// ---------------------------------------------------------------------------
// parity-test kernels: the median networks alone
// ---------------------------------------------------------------------------

// Output tile of one thread of k_debug_median: the shapes the kernels use (med3 in runs,
// med5 in 2 x 2 quads, by the quad network on even tile rows and the one-row network on
// odd ones, med7 single).
__host__ __device__ constexpr int debug_median_ty(int r) { return r == 2 ? 2 : 1; }
__host__ __device__ constexpr int debug_median_tx(int r) { return r == 1 ? kRun3 : (r == 2 ? 2 : 1); }

template <int R>
__global__ __launch_bounds__(kThreads) void k_debug_median(const float *__restrict__ in, int H,
                                                           int W, float *__restrict__ out) {
    constexpr int TY = debug_median_ty(R), TX = debug_median_tx(R);
    constexpr int PH = TY + 2 * R, PW = TX + 2 * R;
    const int ntx = (W + TX - 1) / TX, nty = (H + TY - 1) / TY;
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t >= ntx * nty)
        return;
    const int y0 = (t / ntx) * TY, x0 = (t % ntx) * TX;
    float v[PH * PW], o[TY * TX];
#pragma unroll
    for (int i = 0; i < PH; ++i)
#pragma unroll
        for (int j = 0; j < PW; ++j)
            v[i * PW + j] = in[(size_t)clampi(y0 - R + i, H) * W + clampi(x0 - R + j, W)];
    if constexpr (R == 1) {
        float a[kRun3 + 2], b[kRun3 + 2], c[kRun3 + 2];
#pragma unroll
        for (int j = 0; j < kRun3 + 2; ++j) {
            a[j] = v[j];
            b[j] = v[PW + j];
            c[j] = v[2 * PW + j];
        }
        med3_run<kRun3>(a, b, c, o);
    } else if constexpr (R == 2) {
        if (((t / ntx) & 1) == 0) {
            med5_t2x2(v, o);
        } else {
            // odd tile rows: the one-row network (two outputs) on each of the two rows
            float a[5 * PW], b[5 * PW], oa[2], ob[2];
#pragma unroll
            for (int i = 0; i < 5 * PW; ++i) {
                a[i] = v[i];
                b[i] = v[PW + i];
            }
            med5_t1x2(a, oa);
            med5_t1x2(b, ob);
            o[0] = oa[0];
            o[1] = oa[1];
            o[2] = ob[0];
            o[3] = ob[1];
        }
    } else {
        med7_t1x1(v, o);
    }
#pragma unroll
    for (int i = 0; i < TY; ++i)
#pragma unroll
        for (int j = 0; j < TX; ++j)
            if (y0 + i < H && x0 + j < W)
                out[(size_t)(y0 + i) * W + x0 + j] = o[i * TX + j];
}

// 5x5 clamped median of binary64 values by the single-output network (the one the
// detection applies to the FP32 estimates of S, here on binary64 inputs).
__global__ __launch_bounds__(kThreads) void k_debug_median5_f64(const double *__restrict__ in,
                                                                int H, int W,
                                                                double *__restrict__ out) {
    const long long t = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (t >= (long long)H * W)
        return;
    const int y = (int)(t / W), x = (int)(t - (long long)y * W);
    double v[25], o[1];
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int j = 0; j < 5; ++j)
            v[i * 5 + j] = in[(size_t)clampi(y - 2 + i, H) * W + clampi(x - 2 + j, W)];
    med5_t1x1(v, o);
    out[t] = o[0];
}

// The detection kernel's FP32 estimate of S and its error bound, one pixel per thread
// (clamped neighbours and med5(J) from a single-output network).
__global__ __launch_bounds__(kThreads) void k_debug_s_estimate(DevFrame f,
                                                               float *__restrict__ out_s,
                                                               float *__restrict__ out_err) {
    const long long t = (long long)blockIdx.x * kThreads + threadIdx.x;
    const int H = f.H, W = f.W;
    if (t >= (long long)H * W)
        return;
    const int y = (int)(t / W), x = (int)(t - (long long)y * W);
    float w[25], m5[1];
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int j = 0; j < 5; ++j)
            w[i * 5 + j] = f.img[(size_t)clampi(y - 2 + i, H) * W + clampi(x - 2 + j, W)];
    med5_t1x1(w, m5);
    float err;
    out_s[t] = s_estimate(w[12], w[7], w[17], w[11], w[13], m5[0], sest_params(f), err);
    out_err[t] = err;
}

// The detection's dense upper bound of S at every pixel of one frame: 2 x 5 cell tiles
// aligned at the frame's origin, one per thread, each from its clamped 6 x 9 patch;
// INFINITY where the bound's analysis does not hold.
__global__ __launch_bounds__(kThreads) void k_debug_s_bound(DevFrame f, float *__restrict__ out_u) {
    const int H = f.H, W = f.W;
    const int ntx = (W + 4) / 5, nty = (H + 1) / 2;
    const long long t = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (t >= (long long)ntx * nty)
        return;
    const int y0 = (int)(t / ntx) * 2, x0 = (int)(t % ntx) * 5;
    float v[6 * 9], u[10];
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
        for (int j = 0; j < 9; ++j)
            v[i * 9 + j] = f.img[(size_t)clampi(y0 - 2 + i, H) * W + clampi(x0 - 2 + j, W)];
    const bool ok = dense_bounds(v, sest_params(f), u);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 5; ++j)
            if (y0 + i < H && x0 + j < W)
                out_u[(size_t)(y0 + i) * W + x0 + j] = ok ? u[i * 5 + j] : INFINITY;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

hipError_t launch_debug_s_bound(const DevFrame &f, float *out_u, hipStream_t s) {
    const size_t n = (size_t)((f.W + 4) / 5) * (size_t)((f.H + 1) / 2);
    k_debug_s_bound<<<(unsigned int)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(f, out_u);
    return hipGetLastError();
}

hipError_t launch_debug_s_estimate(const DevFrame &f, float *out_s, float *out_err,
                                   hipStream_t s) {
    const size_t n = (size_t)f.H * (size_t)f.W;
    k_debug_s_estimate<<<(unsigned int)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(
        f, out_s, out_err);
    return hipGetLastError();
}

// Resident blocks of a persistent detection launch: the occupancy the runtime reports
// for the kernel, times the compute units (looked up once per device and tile height).
template <int TY>
static int persistent_grid() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return 0;
    if (!cached[dev]) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_detect_persistent<TY>,
                                                         8 * TY, 0) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) !=
                hipSuccess)
            return 0;
        cached[dev] = (per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1);
    }
    return cached[dev];
}

template <int TY>
static hipError_t launch_detect_ty(const DevFrame *d_frames, const TileRef *d_tiles,
                                   int ntiles, const DevFrame &single, const StepLists &lists,
                                   bool persistent, unsigned int *tickets, hipStream_t s) {
    if (ntiles <= 0)
        return hipSuccess;
    if (persistent && tickets && d_tiles) {
        const int cap = persistent_grid<TY>();
        if (cap <= 0)
            return hipErrorInvalidValue;
        const int grid = ntiles < cap ? ntiles : cap;
        k_detect_persistent<TY><<<grid, 8 * TY, 0, s>>>(d_frames, d_tiles, lists, ntiles,
                                                           tickets);
    } else {
        k_detect<TY, false><<<ntiles, 8 * TY, 0, s>>>(d_frames, d_tiles, single, lists);
    }
    return hipGetLastError();
}

hipError_t launch_detect(const DevFrame *d_frames, const TileRef *d_tiles, int ntiles,
                         const DevFrame &single, const LaunchCfg &cfg, bool narrow,
                         const StepLists &lists, unsigned int *tickets, hipStream_t s) {
    if (!d_tiles)
        ntiles = detect_tiles(single.H, single.W, cfg.tile_h);
    if (narrow) {
        if (cfg.tile_h != kDetectTYDefault || cfg.persistent)
            return hipErrorInvalidValue;
        if (ntiles > 0)
            k_detect<kDetectTYDefault, true><<<ntiles, 8 * kDetectTYDefault, 0, s>>>(
                d_frames, d_tiles, single, lists);
        return hipGetLastError();
    }
    switch (cfg.tile_h) {
    case 16:
        return launch_detect_ty<16>(d_frames, d_tiles, ntiles, single, lists,
                                    cfg.persistent != 0, tickets, s);
    case 32:
        return launch_detect_ty<32>(d_frames, d_tiles, ntiles, single, lists,
                                    cfg.persistent != 0, tickets, s);
    case 64:
        return launch_detect_ty<64>(d_frames, d_tiles, ntiles, single, lists,
                                    cfg.persistent != 0, tickets, s);
    default:
        return hipErrorInvalidValue;
    }
}

hipError_t launch_debug_median5_f64(const double *in, int H, int W, double *out,
                                   hipStream_t s) {
    const size_t n = (size_t)H * (size_t)W;
    k_debug_median5_f64<<<(unsigned int)((n + kThreads - 1) / kThreads), kThreads, 0, s>>>(in, H,
                                                                                         W, out);
    return hipGetLastError();
}

hipError_t launch_debug_median(const float *in, int H, int W, int r, float *out, hipStream_t s) {
    const int ty = debug_median_ty(r), tx = debug_median_tx(r);
    const size_t n = (size_t)((H + ty - 1) / ty) * (size_t)((W + tx - 1) / tx);
    const unsigned int grid = (unsigned int)((n + kThreads - 1) / kThreads);
    if (r == 1)
        k_debug_median<1><<<grid, kThreads, 0, s>>>(in, H, W, out);
    else if (r == 2)
        k_debug_median<2><<<grid, kThreads, 0, s>>>(in, H, W, out);
    else
        k_debug_median<3><<<grid, kThreads, 0, s>>>(in, H, W, out);
    return hipGetLastError();
}

}  // namespace crb
