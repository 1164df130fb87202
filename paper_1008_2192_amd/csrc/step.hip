// Iteration kernel of libcrb for gfx950 (MI355X): from the codes of iteration k (Mighell,
// Section 5) to those of iteration k + 1 in one launch -- the two gated 3x3 dilations, the
// new-flag count, the cumulative mask, the replacement of the flagged pixels by the median
// of their unflagged 5x5 neighbours, and the detection's codes wherever the replacement
// changed J.
//
// A block takes a summary tile of 32 x 64 pixels and computes everything it needs itself
// from the codes within 8 pixels of it (an iteration's reach: 2 for the grows, 2 for the
// replacement window, 4 for the codes), so no launch separates the stages: the grow on 80-bit
// rows, one row per lane of the first wave; the replacement of the flagged pixels within 4
// of the tile, from J staged within 6; the codes of the tile's pixels within 4 of those.
//
// Measured on one MI355X, four iterations: the mixed batch (64 frames, 295 Mpx) 4.48 -> 3.06
// ms, a 256 x 256 frame 84 -> 51 us, 61 x 67 68 -> 32 us, a 4096 x 4096 crowded field 0.43 ->
// 0.38 ms, against three or four launches an iteration that each passed over the frame
// (detection of every pixel, grow over code bytes, flagged list, replacement by gathers).
//
// Blocks share their halos without ordering.  Codes are double-buffered per tile.  The mask
// bitmap of a neighbour may be read before or after its owner ORs G2 into it: the reader ORs
// the G2 it computes from the same codes, so both give M_k.  J of a neighbour may be read
// before or after its owner replaces pixels: those are in M_k, where the reader either
// replaces the pixel itself (the same rule on the same codes, so the same pixels) or, with
// no unflagged neighbour, both leave it.
#include "detect_tile.h"

namespace crb {

// A row of 80 pixels, columns x0 - 8 .. x0 + 71 of a tile: bit j of lo, then of hi.
struct Row80 {
    unsigned long long lo;
    uint32_t hi;
};

__device__ __forceinline__ uint32_t lane_above(uint32_t v) {      // lane - 1 (0 at lane 0)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t lane_below(uint32_t v) {      // lane + 1 (0 at lane 63)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, false);
}
__device__ __forceinline__ unsigned long long pack64(uint32_t lo, uint32_t hi) {
    return ((unsigned long long)hi << 32) | lo;
}

// 3x3 dilation of the 80-bit rows held one per lane (rows outside the lanes are empty; bits
// past the ends of a row are lost).
__device__ __forceinline__ Row80 dilate(const Row80 &r) {
    Row80 h;
    h.lo = r.lo | (r.lo << 1) | (r.lo >> 1) | ((unsigned long long)r.hi << 63);
    h.hi = (r.hi | (r.hi << 1) | (r.hi >> 1) | (uint32_t)(r.lo >> 63)) & 0xFFFFu;
    const uint32_t a = (uint32_t)h.lo, b = (uint32_t)(h.lo >> 32);
    Row80 o;
    o.lo = h.lo | pack64(lane_above(a), lane_above(b)) | pack64(lane_below(a), lane_below(b));
    o.hi = h.hi | lane_above(h.hi) | lane_below(h.hi);
    return o;
}
__device__ __forceinline__ Row80 row_and(const Row80 &a, const Row80 &b) {
    return Row80{a.lo & b.lo, a.hi & b.hi};
}
__device__ __forceinline__ Row80 row_or(const Row80 &a, const Row80 &b) {
    return Row80{a.lo | b.lo, a.hi | b.hi};
}
// Columns 64 .. 127 of a triple of 64-bit words with 8 bits of either neighbour.
__device__ __forceinline__ Row80 row80(unsigned long long left, unsigned long long mid,
                                       unsigned long long right) {
    return Row80{(left >> 56) | (mid << 8),
                 (uint32_t)(mid >> 56) | (uint32_t)(right & 0xFFull) << 8};
}
// The tile's own 64 columns of a row.
__device__ __forceinline__ unsigned long long own64(const Row80 &r) {
    return (r.lo >> 8) | ((unsigned long long)(r.hi & 0xFFu) << 56);
}

using StepLds = DetectLds<32, 6, true>;
constexpr int kRepMax = 1024;       // listed pixels to replace; further ones from the bitmap
struct StepShared {
    StepLds d;
    // rows y0 - 8 .. y0 + 39: M_k (at clamped columns) and the pixels to replace (D4 of the
    // tile); and G2 of the tile's own rows for the parity tests
    unsigned long long m_lo[48], r_lo[48];
    uint32_t m_hi[48], r_hi[48];
    unsigned int nrep;
};
static_assert(kRepMax * 2 <= (int)sizeof(StepLds::S), "the replacement list in the S plane");
static_assert(sizeof(StepShared) <= 32768, "five blocks per CU");

// The replacement value of the pixel whose staged J cell is p (pitch jp) with bit j of fl set
// where the 5x5 window's pixel j is flagged: the median of the unflagged values (an even
// count: the mean of the two middle ones, formed in binary64 and rounded once); false with
// no unflagged value.
__device__ __forceinline__ bool window_median(const float *p, int jp, uint32_t fl, float &out) {
    float v[25];
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int j = 0; j < 5; ++j)
            v[i * 5 + j] = (fl >> (i * 5 + j)) & 1u ? INFINITY : p[(i - 2) * jp + j - 2];
    const int cnt = 25 - __popc(fl);
    if (cnt == 0)
        return false;
    sort25(v);
    const int ia = (cnt - 1) >> 1, ib = cnt >> 1;
    float a = v[0], b = v[0];
#pragma unroll
    for (int j = 1; j < 13; ++j) {        // the middle of at most 25 values
        a = (j == ia) ? v[j] : a;
        b = (j == ib) ? v[j] : b;
    }
    out = (ia == ib) ? a : (float)(((double)a + (double)b) * 0.5);
    return true;
}

// Appends tile g to the list of iteration k.
__device__ __forceinline__ void list_tile(const StepLists &l, int k, int g) {
    const int seg = g & (l.nseg - 1);
    const unsigned int at = atomicAdd(&l.count[((k % 3) * l.nseg + seg) * kTicketStride], 1u);
    if (at < (unsigned int)l.cap)         // (a tile is listed once, so always)
        l.list[k & 1][(size_t)seg * l.cap + at] = (unsigned int)g;
}

// Iteration k of frame f on its summary tile (ty, tx), by the whole block.
__device__ __forceinline__ void step_tile(const DevFrame &f, int ty, int tx, int k,
                                          const StepLists &lists, StepShared &sh, int tid) {
    using L = StepLds;
    L &s = sh.d;
    uint16_t *const rep = reinterpret_cast<uint16_t *>(s.S);    // (the S plane is filled later)
    const int H = f.H, W = f.W, y0 = ty * kSumTY, x0 = tx * kSumTX;
    const int ntx = (W + kSumTX - 1) / kSumTX, nty = (H + kSumTY - 1) / kSumTY;
    const int lane = tid & 63;
    const bool last = k >= f.niter;
    // a counting run of a frame without kIncremental re-evaluates the whole tile
    const bool full = (f.flags & kCountWork) && !(f.flags & kIncremental);
    const float *J = k == 1 ? f.img : f.J;

    detect_clear(s, tid);
    if (tid < 64) {
        // the grow: lane l holds row y0 - 8 + l
        const int y = y0 - 8 + lane, vt = ty + (lane < 8 ? -1 : (lane < 40 ? 0 : 1));
        const int rr = y & (kSumTY - 1);
        const bool row_ok = lane < 48 && y >= 0 && y < H;
        unsigned long long w[4][3];            // planes A, high, low; mask -- left, own, right
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const int vx = tx + d - 1;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                w[p][d] = 0ull;
            if (row_ok && vx >= 0 && vx < ntx) {
                const size_t t = (size_t)vt * ntx + vx;
                unsigned int buf = 0u;
                if (k > 1) {
                    // a neighbour whose state is already iteration k + 1's still has the
                    // codes of iteration k in its other buffer
                    const unsigned int st = f.state[t];
                    buf = (st & 1u) ^ ((st >> 1) == (unsigned int)(k + 1) ? 1u : 0u);
                }
                const unsigned long long *b = f.bits + (t * 2 + buf) * (3 * kSumTY) + rr;
                w[0][d] = b[0];
                w[1][d] = b[kSumTY];
                w[2][d] = b[2 * kSumTY];
                if (k > 1 || !(f.flags & kFreshMask))
                    w[3][d] = f.mbits[t * kSumTY + rr];
            }
        }
        const Row80 a = row80(w[0][0], w[0][1], w[0][2]), hi = row80(w[1][0], w[1][1], w[1][2]);
        const Row80 lo = row80(w[2][0], w[2][1], w[2][2]), mp = row80(w[3][0], w[3][1], w[3][2]);
        const Row80 g2 = row_and(dilate(row_and(dilate(a), hi)), lo);
        Row80 m = row_or(mp, g2);
        const bool own = lane >= 8 && lane < 40 && y < H;
        const unsigned long long nw = own ? own64(g2) & ~w[3][1] : 0ull;
        if (nw)
            f.mbits[((size_t)ty * ntx + tx) * kSumTY + rr] = own64(m);
        const unsigned int n = __ockl_wfred_add_u32((unsigned int)__popcll(nw));
        if (n && lane == 0) {
            // (a sum that all of a frame's blocks add to would serialise them: 8192 blocks
            // took 95 us)
            atomicAdd(&f.count[(blockIdx.x % kCountSlots) * kCountStride], (unsigned long long)n);
            f.any_new[k - 1] = 1u;
        }
        if (f.g2 && own)       // parity tests
            for (int c = 0; c < kSumTX && x0 + c < W; ++c)
                f.g2[(size_t)y * W + x0 + c] = (uint8_t)(own64(g2) >> c & 1ull);
        // The pixels to replace: at iteration 1 all of M_k; later those of M_k with a pixel
        // of G2 within 2 (the only ones whose unflagged window can have changed; a superset
        // of those near a new flag that does not depend on M_{k-1}, which neighbours update)
        Row80 rp = k == 1 ? m : row_and(m, dilate(dilate(g2)));
        // within 4 of the tile: rows 4 .. 43, columns 4 .. 75 of the region
        const bool r4 = lane >= 4 && lane < 44;
        rp.lo &= r4 ? ~0xFull : 0ull;
        rp.hi &= r4 ? 0xFFFu : 0u;
        // the codes that can change lie within 4 of those, and read S within 2 more
        const bool tile_row = lane >= 8 && lane < 40;
        Row80 act = full ? Row80{~0ull, 0xFFFFu} : dilate(dilate(dilate(dilate(rp))));
        act.lo &= tile_row ? ~0xFFull : 0ull;
        act.hi &= tile_row ? 0xFFu : 0u;
        const Row80 reach = dilate(dilate(act));
        if (tile_row) {
            const unsigned long long c = own64(act);
            s.act[2 * (lane - 8)] = (uint32_t)c;
            s.act[2 * (lane - 8) + 1] = (uint32_t)(c >> 32);
        }
        if (lane >= 6 && lane < 42) {          // the S region: rows 6 .. 41, columns 6 .. 73
            uint32_t *q = &s.reach[(lane - 6) * L::HW];
            q[0] = (uint32_t)(reach.lo >> 6);
            q[1] = (uint32_t)(reach.lo >> 38) | reach.hi << 26;
            q[2] = (reach.hi >> 6) & 0xFu;
        }
        // M_k at clamped columns: the windows read it two columns past the frame's edges
        if (x0 == 0)
            m.lo |= (m.lo >> 8 & 1ull) * 0xC0ull;
        const int e = W - 1 - x0 + 8;          // the region column of the last frame column
        if (e < 78) {
            const uint32_t b = e < 64 ? (uint32_t)(m.lo >> e) & 1u : (m.hi >> (e - 64)) & 1u;
            for (int c = e + 1; c <= e + 2; ++c) {
                m.lo |= c < 64 ? (unsigned long long)b << c : 0ull;
                m.hi |= c >= 64 ? b << (c - 64) : 0u;
            }
        }
        if (lane < 48) {
            sh.m_lo[lane] = m.lo;
            sh.m_hi[lane] = m.hi;
            sh.r_lo[lane] = rp.lo;
            sh.r_hi[lane] = rp.hi;
        }
        // list them (in any order): region position row * 80 + column
        const unsigned int cnt = (unsigned int)__popcll(rp.lo) + (unsigned int)__popc(rp.hi);
        unsigned int at = __ockl_wfscan_add_u32(cnt, false);
        if (lane == 63)
            sh.nrep = at + cnt;
        for (unsigned long long v = rp.lo; v; v &= v - 1ull, ++at)
            if (at < (unsigned int)kRepMax)
                rep[at] = (uint16_t)(lane * 80 + __ffsll((long long)v) - 1);
        for (uint32_t v = rp.hi; v; v &= v - 1u, ++at)
            if (at < (unsigned int)kRepMax)
                rep[at] = (uint16_t)(lane * 80 + 64 + __ffs((int)v) - 1);
    }
    stage_j(s, J, H, W, y0, x0, tid);
    __syncthreads();
    const int nrep = (int)sh.nrep;
    if (nrep == 0 && !full)
        return;

    // replacement (a flagged pixel's J is read by no other window, so it is updated in
    // place), and meanwhile, by the other waves, the list of the 2 x 5 cell tiles of S that a
    // re-evaluated code reads
    const bool listed = nrep <= kRepMax;
    for (int i = tid; i < (listed ? nrep : 48 * 80); i += L::NT) {
        const int pos = listed ? (int)rep[i] : i;
        const int r = pos / 80, c = pos - r * 80;
        const unsigned long long in = c < 64 ? sh.r_lo[r] >> c : sh.r_hi[r] >> (c - 64);
        if (!listed && !(in & 1ull))
            continue;
        const int y = y0 - 8 + r, x = x0 - 8 + c;
        uint32_t fl = 0u;
#pragma unroll
        for (int i5 = 0; i5 < 5; ++i5) {
            const int q = clampi(y + i5 - 2, H) - y0 + 8, sft = c - 2;
            const unsigned long long lo = sh.m_lo[q];
            const uint32_t hi = sh.m_hi[q];
            const uint32_t b = sft < 64 ? (uint32_t)((lo >> sft) |
                                                     (unsigned long long)hi << (64 - sft))
                                        : hi >> (sft - 64);
            fl |= (b & 31u) << (5 * i5);
        }
        float *p = &s.J[(r - 2) * L::JWP + c - 2];
        float nv;
        const bool mine = r >= 8 && r < 40 && c >= 8 && c < 72;
        if (window_median(p, L::JWP, fl, nv)) {
            *p = nv;
            if (mine)
                f.J[(size_t)y * W + x] = nv;
        }
        if (mine)
            f.mask[(size_t)y * W + x] = 1;
    }
    if (last)
        return;
    for (int t = L::NT - 1 - tid; t < L::NTY * L::NTX; t += L::NT) {
        const int rp = t / L::NTX, cx = t - rp * L::NTX;
        const int c5 = min(5 * cx, L::SW - 5), w = c5 >> 5, sft = c5 & 31;
        const uint32_t *q = &s.reach[2 * rp * L::HW + w];
        const uint32_t lo = q[0] | q[L::HW];
        const uint32_t hi = w + 1 < L::HW ? q[1] | q[L::HW + 1] : 0u;
        if ((uint32_t)(pack64(lo, hi) >> sft) & 31u)
            s.cells[atomicAdd(&s.ncells, 1u)] = (uint16_t)(rp * 16 + cx);
    }
    __syncthreads();
    // staged cells outside the frame follow the pixel they repeat
    if (y0 < 6 || x0 < 6 || y0 + kSumTY + 6 > H || x0 + kSumTX + 6 > W) {
        for (int i = tid; i < L::JH * L::JW; i += L::NT) {
            const int r = i / L::JW, c = i - r * L::JW;
            const int gy = y0 - 6 + r, gx = x0 - 6 + c;
            if (gy < 0 || gy >= H || gx < 0 || gx >= W)
                s.J[r * L::JWP + c] =
                    s.J[(clampi(gy, H) - y0 + 6) * L::JWP + clampi(gx, W) - x0 + 6];
        }
        __syncthreads();
    }
    detect_staged(s, f, y0, x0, tid);

    // the tile's codes of iteration k + 1 into its other buffer, and the tiles it lists
    if (tid < 64) {
        const size_t t = (size_t)ty * ntx + tx;
        const unsigned int buf = f.state[t] & 1u;
        unsigned long long a = 0ull;
        if (lane < kSumTY) {
            const unsigned long long *code = reinterpret_cast<const unsigned long long *>(s.code);
            const unsigned long long act = pack64(s.act[2 * lane], s.act[2 * lane + 1]);
            const unsigned long long *b = f.bits + (t * 2 + buf) * (3 * kSumTY) + lane;
            unsigned long long *o = f.bits + (t * 2 + (buf ^ 1u)) * (3 * kSumTY) + lane;
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const unsigned long long v =
                    y0 + lane < H ? (b[p * kSumTY] & ~act) | code[p * kSumTY + lane] : 0ull;
                o[p * kSumTY] = v;
                if (p == 0)
                    a = v;
            }
        }
        const uint32_t dirs = reach_bits((uint32_t)__ballot(a != 0ull),
                                         (uint32_t)__ballot((a & 0xFFull) != 0ull),
                                         (uint32_t)__ballot((a >> 56) != 0ull));
        // The next iteration has work only within reach of A.  Every tile that holds A now
        // was re-evaluated in this launch (a tile with A at iteration k replaces pixels, A
        // being part of G2), so each lists the tiles that its own A reaches
        const int dy = lane / 3 - 1, dx = lane - (lane / 3) * 3 - 1;
        const int vy = ty + dy, vx = tx + dx;
        const bool there = lane < 9 && vy >= 0 && vy < nty && vx >= 0 && vx < ntx;
        const size_t v = (size_t)(there ? vy : ty) * ntx + (there ? vx : tx);
        if (lane == 0)
            f.state[t] = 2u * (unsigned int)(k + 1) | (buf ^ 1u);
        if (there && (dirs >> lane & 1u) &&
            atomicMax(&f.mark[v], (unsigned int)(k + 1)) < (unsigned int)(k + 1) && lists.list[0])
            list_tile(lists, k + 1, f.tile_base + (int)v);
    }
}

// The (frame, tile) g of a launch.
__device__ __forceinline__ void step_one(const DevFrame *__restrict__ frames,
                                         const TileRef *__restrict__ tiles,
                                         const DevFrame &single, int g, int kiter, bool by_mark,
                                         const StepLists &lists, StepShared &sh, int tid) {
    DevFrame f;
    int ty, tx;
    if (tiles) {
        const TileRef r = tiles[g];
        f = frames[r.frame];
        ty = r.y0 / kSumTY;
        tx = r.x0 / kSumTX;
    } else {
        f = single;
        const int ntx = (single.W + kSumTX - 1) / kSumTX;
        ty = g / ntx;
        tx = g - ty * ntx;
    }
    const int k = kiter ? kiter : f.k;
    if (k > f.niter)
        return;
    // early stop (result-neutral: the listed tiles would find nothing new)
    if (k >= 2 && !(f.flags & kNoEarlyStop) && !f.any_new[k - 2])
        return;
    // from iteration 2 on, only the tiles that the previous one listed (a neighbour's block of
    // this launch may have raised the mark to k + 1 meanwhile: a tile visited without need
    // gives what it has)
    if (by_mark && k >= 2 && !((f.flags & kCountWork) && !(f.flags & kIncremental)) &&
        f.mark[(size_t)ty * ((f.W + kSumTX - 1) / kSumTX) + tx] < (unsigned int)k)
        return;
    step_tile(f, ty, tx, k, lists, sh, tid);
}

// Iteration k on every tile of the launch (k == 0: each frame's own).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5)))
void k_step(const DevFrame *__restrict__ frames, const TileRef *__restrict__ tiles,
            DevFrame single, int kiter, StepLists lists, unsigned int *__restrict__ tickets) {
    __shared__ StepShared sh;
    const int tid = (int)threadIdx.x;
    if (blockIdx.x == 0) {
        if (lists.list[0])
            lists_clear(lists, kiter + 2, tid);
        if (tickets && kiter == 1)
            for (int i = tid; i < kTicketWords; i += 256)
                tickets[i] = 0u;
    }
    step_one(frames, tiles, single, (int)blockIdx.x, kiter, true, lists, sh, tid);
}

// Iteration k on the tiles listed for it: block b takes entries b / nseg, b / nseg + stride,
// ... of segment b % nseg.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5)))
void k_step_listed(const DevFrame *__restrict__ frames, const TileRef *__restrict__ tiles,
                   DevFrame single, int kiter, StepLists lists) {
    __shared__ StepShared sh;
    if (blockIdx.x == 0)
        lists_clear(lists, kiter + 2, (int)threadIdx.x);
    const int seg = (int)blockIdx.x & (lists.nseg - 1), stride = (int)gridDim.x / lists.nseg;
    const unsigned int *list = lists.list[kiter & 1] + (size_t)seg * lists.cap;
    const int n = min((int)lists.count[((kiter % 3) * lists.nseg + seg) * kTicketStride],
                      lists.cap);
    for (int e = (int)blockIdx.x / lists.nseg; e < n; e += stride) {
        // as in the persistent detection, thread-derived values are not held across tiles
        int tid = (int)threadIdx.x;
        asm volatile("" : "+v"(tid));
        step_one(frames, tiles, single, (int)list[e], kiter, false, lists, sh, tid);
        __syncthreads();       // the tile is done with the LDS
    }
}

hipError_t launch_step(const DevFrame *d_frames, const TileRef *d_tiles, int ntiles,
                       const DevFrame &single, int k, bool all, const StepLists &lists,
                       unsigned int *tickets, hipStream_t s) {
    if (!d_tiles)
        ntiles = detect_tiles(single.H, single.W, kSumTY);
    if (ntiles <= 0)
        return hipSuccess;
    if (k <= 1 || all || !lists.list[0]) {
        k_step<<<ntiles, 256, 0, s>>>(d_frames, d_tiles, single, k, lists, tickets);
    } else {
        // a multiple of the segments, about as many blocks as the device holds
        int per = (ntiles + lists.nseg - 1) / lists.nseg;
        const int most = 1280 / lists.nseg;
        per = per < most ? per : most;
        k_step_listed<<<per * lists.nseg, 256, 0, s>>>(d_frames, d_tiles, single, k, lists);
    }
    return hipGetLastError();
}

}  // namespace crb
