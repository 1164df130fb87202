// Device-side frame descriptor and kernel launchers of libcrb (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace crb {

// Upper bound on iterations per frame (sizes the per-frame counters).
constexpr int kMaxIter = 1024;
// Detection tiles are kDetectTX = 64 columns by 16, 32 (default) or 64 rows, one block of
// 8 threads per row.  The state the iterations share (code planes, mask bitmap, where A
// occurs, which tiles the next iteration visits) lives on a fixed grid of kSumTY x kSumTX
// summary tiles, whatever the detection tile.
constexpr int kDetectTX = 64;
constexpr int kDetectTYDefault = 32;
constexpr int kSumTY = 32;
constexpr int kSumTX = 64;
// ticket counters of one persistent detection launch (one per XCD), each on its own
// 128-byte line (kTicketStride words apart) so that the XCDs do not contend for one line
constexpr int kDetectQueues = 8;
constexpr int kTicketStride = 32;
constexpr int kTicketWords = kDetectQueues * kTicketStride;   // per launch
// Counters a frame's blocks add their new flags to, each on its own 128-byte line.
constexpr int kCountSlots = 32;
constexpr int kCountStride = 16;
// Segments of a list of tiles (StepLists): appends spread over that many counters.
constexpr int kListSegments = 64;
constexpr int kThreads = 256;

// Kernel classes for per-launch timing (crb_plan_kernel_times order).
// (kind 3, once the replacement, is never recorded: it is part of an iteration's launch)
constexpr int kKindInit = 0, kKindDetect = 1, kKindStep = 2;
constexpr int kNumKernelKinds = 4;

// DevFrame::flags bits.  kNoEarlyStop has the value of CRB_FLAG_NO_EARLY_STOP;
// kFreshMask: the mask is uninitialised before iteration 1, whose detection clears it.
// kCountWork: detection adds its work-set size, contrast-test count and number of
// binary64 re-evaluations to f.work[0..2].
// kExactDetect: detection evaluates S' of every work-set pixel in binary64 from J
// (parity tests of that path).
constexpr int kNoEarlyStop = 1;
constexpr int kFreshMask = 1 << 8;
constexpr int kCountWork = 1 << 9;
constexpr int kExactDetect = 1 << 10;
// kIncremental (the value of CRB_FLAG_INCREMENTAL): with kCountWork, count the detection
// work that is done (only where J changed); without it a counting run re-evaluates every
// pixel at every iteration.  Without counting, both do the former.
constexpr int kIncremental = 2;
constexpr int kWorkCounters = 4;

// Everything a kernel needs to know about one frame.  All pointers are device
// pointers; J is the image being cleaned in place (out_clean).  The per-tile arrays are
// indexed by summary tile, row-major.
struct DevFrame {
    const float *img;             // input frame (copied into J by the first detection)
    float *J;                     // working / output image, H x W
    uint8_t *mask;                // cumulative mask, H x W (0/1)
    uint8_t *codes;               // optional: detection codes as bytes (parity tests), or null
    uint8_t *g2;                  // optional: selection of this iteration (debug), or null
    // detection codes: per tile two buffers of three planes (A, [S' > sigclip], [S' >
    // sigfrac sigclip]) of 32 rows, bit c of a row for column c
    unsigned long long *bits;
    unsigned long long *mbits;    // cumulative mask, per tile 32 rows of 64 bits
    // per tile: 2 * s + b, codes in buffer b since the launch of iteration s - 1 (1: the
    // first detection).  An iteration writes new codes to the other buffer, so that its
    // neighbours still read the codes it started from
    unsigned int *state;
    // per tile: the last iteration it was listed for (each lists a tile once)
    unsigned int *mark;
    // flagged pixels: the sum of kCountSlots counters, kCountStride apart
    unsigned long long *count;
    unsigned int *any_new;        // per iteration: whether n_k > 0 [kMaxIter]
    unsigned long long *work;     // with kCountWork: kWorkCounters counters, or null
    int H, W;
    float gain, readnoise, sky, sigclip, sigfrac, objlim;
    int niter;
    int flags;
    int k;                        // current iteration when a kernel is launched with k = 0
    int tile_base;                // index of the frame's first tile in the launch's tiles
    int list_base[3];             // its first entry in the lists of k_tiles, per tile height
                                  // 16, 32, 64 (-1: not listed)
    // Detection constants, derived from the parameters above by derive_detect_consts (on
    // the host, in the operations the detection would otherwise repeat per tile): the
    // FP32 thresholds sigclip and sigfrac * sigclip widened and narrowed by 2^-20
    // relative, objlim by 2^-21, 1 / objlim; and the parameters of the FP32 estimate of S
    // (gain / 8, 1 / gain, readnoise^2, and whether gain lies in [2^-100, 2^100]).
    float sc_lo, sc_hi, ll_lo, ll_hi;
    float olim_lo, olim_hi, inv_olim;
    float g8, inv_gain, rn2f;
    int est_ok;
    // How the tiles' bit rows are stored.  0: 32 rows of 64 bits a plane.  Frames that cover
    // little of their tiles keep what they cover, so that their workspace is not larger than
    // reported (ws_layout): -H, for one row of tiles, H rows of 64 bits; p = 1, 2, 4, 8 or 16,
    // for one column of tiles, 32 rows of p bits in units of 16 bits, the first in the low bits.
    int narrow;
};

// Fills the detection constants of f from its parameters (every DevFrame passes through
// it: make_devframe calls it).  Plain IEEE single-precision operations, each rounded
// once, as the device would evaluate them.
inline void derive_detect_consts(DevFrame &f) {
    const float ll = f.sigfrac * f.sigclip;
    f.sc_lo = f.sigclip * (1.0f - 0x1p-20f);
    f.sc_hi = f.sigclip * (1.0f + 0x1p-20f);
    f.ll_lo = ll * (1.0f - 0x1p-20f);
    f.ll_hi = ll * (1.0f + 0x1p-20f);
    f.olim_lo = f.objlim * (1.0f - 0x1p-21f);
    f.olim_hi = f.objlim * (1.0f + 0x1p-21f);
    f.inv_olim = 1.0f / f.objlim;
    f.g8 = f.gain * 0.125f;
    f.inv_gain = 1.0f / f.gain;
    f.rn2f = f.readnoise * f.readnoise;
    f.est_ok = (f.gain >= 0x1p-100f && f.gain <= 0x1p100f) ? 1 : 0;
}

struct TileRef {                  // one (frame, tile origin) work item
    int frame, y0, x0, pad;
};

// Lists of the tiles (by index in the launch's tiles) that an iteration visits: iteration k
// >= 2 reads list k & 1 and appends to list (k + 1) & 1.  A list has nseg segments of cap
// entries, tile g in segment g % nseg, each with its own counter (kTicketStride words
// apart); the counters of list k are set k % 3 of three, and iteration k clears the set that
// iteration k + 1 fills.  list[0] null: no lists (the tiles' marks alone say what to visit).
struct StepLists {
    unsigned int *list[2];
    unsigned int *count;
    int nseg, cap;
};
// Segments of the lists of ntiles tiles (a power of two), and their words.
inline int list_segments(size_t ntiles) {
    int n = 1;
    while (n < kListSegments && (size_t)(2 * n) <= ntiles)
        n *= 2;
    return n;
}
inline size_t list_words(size_t ntiles, int nseg) {
    const size_t n = (size_t)nseg;
    return 2 * n * ((ntiles + n - 1) / n) + 3 * n * kTicketStride;
}
inline StepLists make_lists(void *p, size_t ntiles, int nseg) {
    StepLists l;
    l.nseg = nseg;
    l.cap = (int)((ntiles + (size_t)nseg - 1) / (size_t)nseg);
    l.list[0] = static_cast<unsigned int *>(p);
    l.list[1] = l.list[0] + (size_t)l.nseg * l.cap;
    l.count = l.list[1] + (size_t)l.nseg * l.cap;
    return l;
}

// A list of some tiles of a launch, built by launch_tiles: nseg segments of cap entries with a
// counter each (kTicketStride words apart, zero before).
struct TileList {
    unsigned int *list;
    unsigned int *count;
    int nseg, cap;
};
// (64 consecutive tiles share a segment; the frames' tile_base are multiples of 64)
inline size_t tile_list_cap(size_t ntiles) {
    return ((ntiles + 63) / 64 + kListSegments - 1) / kListSegments * 64;
}

// Builds the (frame, tile) lists of a table of frames on the device: out[h] (may be null), the
// tiles of height 16, 32, 64 of the frames with list_base[h] >= 0; step (may be null), the
// summary tiles of the frames at iteration f.k >= 2 from f.tile_base on, and in `active` those
// that the previous iteration marked.  Clears zero_words words at `zero`.
hipError_t launch_tiles(const DevFrame *d_frames, int nframes, size_t max_tiles, TileRef *out16,
                        TileRef *out32, TileRef *out64, TileRef *step, const TileList &active,
                        unsigned int *zero, int zero_words, hipStream_t s);

// For frames with niter == 0: copies img into J and clears the mask (otherwise the first
// detection does both).  max_pixels: the largest such frame, which sizes the grid.
hipError_t launch_init(const DevFrame *d_frames, int nframes, const DevFrame &single,
                       size_t max_pixels, hipStream_t s);

// How a pass is launched (the autotuner's choices; every choice gives identical
// results).  tile_h: tile rows of the first detection (16, 32 or 64); persistent: that
// detection by resident blocks taking tiles from ticket counters instead of one block per
// tile.  fused and grow_h are kept as set and have no effect.
struct LaunchCfg {
    int tile_h = kDetectTYDefault;
    int persistent = 0;
    int fused = 0;
    int grow_h = 0;
};

// The first iteration's detection for one frame (d_tiles == null: tiles over `single`) or a
// work list of (frame, tile) built for cfg.tile_h.  Persistent launches take kTicketWords
// zeroed words of ticket counters.  narrow, here and below: some frame has f.narrow != 0 (these
// launches take the default shape).
hipError_t launch_detect(const DevFrame *d_frames, const TileRef *d_tiles, int ntiles,
                         const DevFrame &single, const LaunchCfg &cfg, bool narrow,
                         const StepLists &lists, unsigned int *tickets, hipStream_t s);
// Number of detection tiles of an H x W frame at tile height tile_h.
__host__ __device__ inline int detect_tiles(int H, int W, int tile_h) {
    return ((H + tile_h - 1) / tile_h) * ((W + kDetectTX - 1) / kDetectTX);
}
// Iteration k from its codes on: grow, new-flag count, cumulative mask, replacement, and
// (before the last) the next iteration's codes.  d_tiles: the summary tiles of the launch
// (null: those of `single`); k == 0: each frame's own f.k, with no lists.  all: visit every
// tile at every iteration (frames that re-evaluate every pixel).  tickets, if not null:
// kTicketWords words that iteration 1 zeroes.
hipError_t launch_step(const DevFrame *d_frames, const TileRef *d_tiles, int ntiles,
                       const DevFrame &single, int k, bool all, bool narrow,
                       const StepLists &lists, unsigned int *tickets, hipStream_t s);
// Each frame's own iteration f.k on the tiles of a list built by launch_tiles.
hipError_t launch_step_active(const DevFrame *d_frames, const TileRef *d_tiles, size_t ntiles,
                              bool narrow, const TileList &active, hipStream_t s);
// Per-frame (iters_run, n_flagged) into d_stats[2 * i].
hipError_t launch_stats(const DevFrame *d_frames, int nframes, long long *d_stats,
                        hipStream_t s);

// Serving rounds: per frame, whether the iteration f.k just run flagged a new pixel, and the
// flagged pixels so far, into d_stats[2 * i] and d_stats[2 * i + 1].
// (launch_count: the flagged pixels of one frame into *out.)
hipError_t launch_count(const DevFrame &f, long long *out, hipStream_t s);
// Clears the counters of the round's active list for the next one.
hipError_t launch_round_stats(const DevFrame *d_frames, int nframes, long long *d_stats,
                              const TileList &active, hipStream_t s);

// Subimage of a frame: the extended rectangle [a0, a0+h) x [b0, b0+w) is copied into
// sub (pitch w); its interior [y0, y1) x [x0, x1) (image coordinates) is written back.
struct SubRect {
    float *sub_img;        // h x w copy of the extended rectangle
    float *sub_clean;      // h x w cleaned subimage
    uint8_t *sub_mask;     // h x w mask of the subimage
    int a0, b0, h, w;      // extended rectangle
    int y0, y1, x0, x1;    // interior
};
hipError_t launch_extract(const float *img, int W, const SubRect *d_subs, int nsub,
                          size_t max_pixels, hipStream_t s);
hipError_t launch_stitch(float *out_clean, uint8_t *out_mask, int W, const SubRect *d_subs,
                         int nsub, size_t max_pixels, hipStream_t s);

hipError_t launch_debug_median(const float *in, int H, int W, int r, float *out, hipStream_t s);
// FP32 estimate of S and its error bound at every pixel of one frame (the detection
// kernel's estimate, for parity tests of the bound).
hipError_t launch_debug_s_estimate(const DevFrame &f, float *out_s, float *out_err,
                                   hipStream_t s);
hipError_t launch_debug_median5_f64(const double *in, int H, int W, double *out,
                                   hipStream_t s);
// The detection's dense upper bound of S at every pixel of one frame (+inf where its
// analysis does not hold), for parity tests of the bound.
hipError_t launch_debug_s_bound(const DevFrame &f, float *out_u, hipStream_t s);
// n FP32 elements copied by 4-byte buffer loads and stores (counter calibration).
hipError_t launch_debug_copy_b32(const float *src, float *dst, long long n, hipStream_t s);
hipError_t launch_debug_fp64(const double *x, const double *y, int n, double *out_sqrt,
                             double *out_div, hipStream_t s);

}  // namespace crb
