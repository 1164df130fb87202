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
// ms when this kernel came (2.35 now), a 256 x 256 frame 84 -> 51 us (39 now), 61 x 67 68 -> 32
// us (24 now), a 4096 x 4096 crowded field 0.43 -> 0.38 ms (0.30 now), against three or four
// launches an iteration that each passed over the frame (detection of every pixel, grow over
// code bytes, flagged list, replacement by gathers).  A single tile is bound by the latency of
// its chain, many of them by that and by issue (waves wait 72% of their cycles, VALU issue is
// at 43% of its rate): with J's loads in flight during the grow, rows in 32-bit words and no
// pass over the staged cells past the frame's edges, the first iteration of the batch took
// 1.48 -> 1.11 ms, with pairs of lanes for a replacement 1.08 and with fewer registers 0.91; the
// second, on the listed tiles, takes 0.16 ms.
//
// Blocks share their halos without ordering.  Codes are double-buffered per tile.  The mask
// bitmap of a neighbour may be read before or after its owner ORs G2 into it: the reader ORs
// the G2 it computes from the same codes, so both give M_k.  J of a neighbour may be read
// before or after its owner replaces pixels: those are in M_k, where the reader either
// replaces the pixel itself (the same rule on the same codes, so the same pixels) or, with
// no unflagged neighbour, both leave it.
#include "detect_tile.h"

namespace crb {

// A row of 80 pixels, columns x0 - 8 .. x0 + 71 of a tile: bit j % 32 of word j / 32.  (A
// dilation may spread into the unused bits 80 .. 95, and back no further than it would on a
// longer row.)
struct Row80 {
    uint32_t w[3];
};

__device__ __forceinline__ uint32_t lane_above(uint32_t v) {      // lane - 1 (0 at lane 0)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, false);
}
__device__ __forceinline__ uint32_t lane_below(uint32_t v) {      // lane + 1 (0 at lane 63)
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, false);
}
// Bits s .. s + 31 of the pair (hi, lo), s < 32.
__device__ __forceinline__ uint32_t bits_at(uint32_t hi, uint32_t lo, int s) {
    return __builtin_amdgcn_alignbit(hi, lo, (uint32_t)s);
}

// 3x3 dilation of the rows held one per lane (rows outside the lanes are empty).
__device__ __forceinline__ Row80 dilate(const Row80 &r) {
    const uint32_t a = r.w[0], b = r.w[1], c = r.w[2];
    const uint32_t h[3] = {a | a << 1 | bits_at(b, a, 1), b | bits_at(b, a, 31) | bits_at(c, b, 1),
                           c | bits_at(c, b, 31) | c >> 1};
    Row80 o;
#pragma unroll
    for (int i = 0; i < 3; ++i)
        o.w[i] = h[i] | lane_above(h[i]) | lane_below(h[i]);
    return o;
}
__device__ __forceinline__ Row80 row_and(const Row80 &a, const Row80 &b) {
    return Row80{{a.w[0] & b.w[0], a.w[1] & b.w[1], a.w[2] & b.w[2]}};
}
__device__ __forceinline__ Row80 row_or(const Row80 &a, const Row80 &b) {
    return Row80{{a.w[0] | b.w[0], a.w[1] | b.w[1], a.w[2] | b.w[2]}};
}
// A tile's 64 columns with 8 columns of either neighbour.
__device__ __forceinline__ Row80 row80(unsigned long long left, unsigned long long mid,
                                       unsigned long long right) {
    const uint32_t m0 = (uint32_t)mid, m1 = (uint32_t)(mid >> 32);
    return Row80{{bits_at(m0, (uint32_t)(left >> 32), 24), bits_at(m1, m0, 24),
                  bits_at((uint32_t)right, m1, 24) & 0xFFFFu}};
}
// The tile's own 64 columns of a row.
__device__ __forceinline__ unsigned long long own64(const Row80 &r) {
    return (unsigned long long)bits_at(r.w[2], r.w[1], 8) << 32 | bits_at(r.w[1], r.w[0], 8);
}
// Bit c (0 .. 79) of a row.
__device__ __forceinline__ uint32_t row_bit(const Row80 &r, int c) {
    return (c < 32 ? r.w[0] : (c < 64 ? r.w[1] : r.w[2])) >> (c & 31) & 1u;
}

using StepLds = DetectLds<32, 6, true>;
constexpr int kRepMax = 1024;       // listed pixels to replace; further ones from the bitmap
struct StepShared {
    StepLds d;
    // rows y0 - 8 .. y0 + 39: M_k (at clamped columns; a fourth word for two-word reads) and
    // the pixels to replace (within 4 of the tile)
    uint32_t m[48][4], r[48][3];
    unsigned int nrep, buf;
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

// The same by the lanes of a pair (2 i, 2 i + 1; h: which of them), each with half of the
// window: rows 0 and 1 and the first three of row 2, or rows 3 and 4 and the last two of row 2.
// The flagged values take +inf and -inf in turn, so that the middle is that of the 25 whatever
// their number: value 12, or for an odd number the mean of values 11 and 12.  (A third of row 2
// that the second lane does not have is a 26th value +inf, behind both.)  Each lane sorts its
// 13; the n-th smallest of two sorted lists is the least over i of max(a_i, b_{n - i}), the
// larger of the ends when i are taken from one list and n - i from the other.  nan: the
// window's unflagged values hold a NaN, whose place the two networks do not agree on.
__device__ __forceinline__ bool window_median_half(const float *p, int jp, uint32_t fl, int h,
                                                   float &out, bool &nan) {
    float v[13], o[13];
    const float *rows = p + (h ? jp : -2 * jp) - 2, *mid = p + (h ? 1 : -2);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 5; ++j)
            v[i * 5 + j] = rows[i * jp + j];
#pragma unroll
    for (int j = 0; j < 3; ++j)
        v[10 + j] = mid[j];
    uint32_t odd = fl;                   // an odd number of flags up to and with the bit
#pragma unroll
    for (int s = 1; s < 32; s *= 2)
        odd ^= odd << s;
    const uint32_t neg = fl & ~odd;
    const uint32_t f = h ? fl >> 15 | (fl >> 13 & 3u) << 10 | 1u << 12 : fl;
    const uint32_t n = h ? neg >> 15 | (neg >> 13 & 3u) << 10 : neg;
    uint32_t top = 0u;
#pragma unroll
    for (int i = 0; i < 13; ++i) {
        const uint32_t inf = (n << (31 - i) & 0x80000000u) | 0x7f800000u;
        const uint32_t m = (uint32_t)((int32_t)(f << (31 - i)) >> 31);
        const uint32_t b = (m & inf) | (~m & __float_as_uint(v[i]));
        top = max(top, b & 0x7fffffffu);
        v[i] = __uint_as_float(b);
    }
    sort13(v);
    top = max(top, (uint32_t)__builtin_amdgcn_mov_dpp((int)top, 0xB1, 0xf, 0xf, false));
    nan = top > 0x7f800000u;
#pragma unroll
    for (int i = 0; i < 13; ++i)         // the other lane's
        o[i] = __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v[i]), 0xB1,
                                                                  0xf, 0xf, false));
    float a = fminf(v[11], o[11]), b = fminf(v[12], o[12]);
#pragma unroll
    for (int i = 1; i < 12; ++i)
        a = fminf(a, fmaxf(v[i - 1], o[11 - i]));
#pragma unroll
    for (int i = 1; i < 13; ++i)
        b = fminf(b, fmaxf(v[i - 1], o[12 - i]));
    out = __popc(fl) & 1 ? (float)(((double)a + (double)b) * 0.5) : b;
    return fl != 0x1FFFFFFu;
}

// Appends tile g to the list of iteration k.
__device__ __forceinline__ void list_tile(const StepLists &l, int k, int g) {
    const int seg = g & (l.nseg - 1);
    const unsigned int at = atomicAdd(&l.count[((k % 3) * l.nseg + seg) * kTicketStride], 1u);
    if (at < (unsigned int)l.cap)         // (a tile is listed once, so always)
        l.list[k & 1][(size_t)seg * l.cap + at] = (unsigned int)g;
}

// Iteration k of frame f on its summary tile (ty, tx), by the whole block.  NARROW: the frame
// may store its bit rows in a narrow form (DevFrame::narrow).
template <bool NARROW>
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

    detect_clear(s, tid);
    JStage<L, 6> stage;
    static_assert(stage.kRound == stage.kBlocks, "one round");
    stage.load(k == 1 ? f.img : f.J, H, W, y0, x0, tid, 0);
    if (tid < 64) {
        // the grow: lane l holds row y0 - 8 + l
        const int y = y0 - 8 + lane, vt = ty + (lane < 8 ? -1 : (lane < 40 ? 0 : 1));
        const int rr = y & (kSumTY - 1);
        const bool row_ok = lane < 48 && y >= 0 && y < H;
        unsigned long long w[4][3];            // planes A, high, low; mask -- left, own, right
        unsigned int own_buf = 0u;
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
                const bool mask = k > 1 || !(f.flags & kFreshMask);
                if (!(NARROW && f.narrow)) {
                    const unsigned long long *b = f.bits + (t * 2 + buf) * (3 * kSumTY) + rr;
                    w[0][d] = b[0];
                    w[1][d] = b[kSumTY];
                    w[2][d] = b[2 * kSumTY];
                    if (mask)
                        w[3][d] = f.mbits[t * kSumTY + rr];
                } else {
                    unsigned long long v[3];
                    narrow_codes(f, (t * 2 + buf) * 3, rr, v);
                    if (mask)
                        w[3][d] = narrow_mask(f, t, rr);
                    w[0][d] = v[0];
                    w[1][d] = v[1];
                    w[2][d] = v[2];
                }
                own_buf = d == 1 ? buf : own_buf;
            }
        }
        const Row80 a = row80(w[0][0], w[0][1], w[0][2]), hi = row80(w[1][0], w[1][1], w[1][2]);
        const Row80 lo = row80(w[2][0], w[2][1], w[2][2]), mp = row80(w[3][0], w[3][1], w[3][2]);
        const Row80 g2 = row_and(dilate(row_and(dilate(a), hi)), lo);
        Row80 m = row_or(mp, g2);
        const bool tile_row = lane >= 8 && lane < 40;
        const unsigned long long nw = tile_row && y < H ? own64(g2) & ~w[3][1] : 0ull;
        if (nw) {
            const size_t t = (size_t)ty * ntx + tx;
            if (!(NARROW && f.narrow))
                f.mbits[t * kSumTY + rr] = own64(m);
            else if (f.narrow < 0)
                f.mbits[t * (size_t)-f.narrow + rr] = own64(m);
            else          // (other rows of the word are other lanes')
                atomicOr(reinterpret_cast<uint32_t *>(f.mbits) + t * (size_t)f.narrow +
                             (rr * f.narrow >> 5),
                         (uint32_t)nw << (rr * f.narrow & 31));
        }
        const unsigned int n = __ockl_wfred_add_u32((unsigned int)__popcll(nw));
        if (n && lane == 0) {
            // (a sum that all of a frame's blocks add to would serialise them: 8192 blocks
            // took 95 us)
            atomicAdd(&f.count[(blockIdx.x % kCountSlots) * kCountStride], (unsigned long long)n);
            f.any_new[k - 1] = 1u;
        }
        if (f.g2 && tile_row && y < H)       // parity tests
            for (int c = 0; c < kSumTX && x0 + c < W; ++c)
                f.g2[(size_t)y * W + x0 + c] = (uint8_t)(own64(g2) >> c & 1ull);
        // The pixels to replace: at iteration 1 all of M_k; later those of M_k with a pixel
        // of G2 within 2 (the only ones whose unflagged window can have changed; a superset
        // of those near a new flag that does not depend on M_{k-1}, which neighbours update)
        Row80 rp = k == 1 ? m : row_and(m, dilate(dilate(g2)));
        // within 4 of the tile: rows 4 .. 43, columns 4 .. 75 of the region
        const bool r4 = lane >= 4 && lane < 44;
        rp.w[0] &= r4 ? ~0xFu : 0u;
        rp.w[1] &= r4 ? ~0u : 0u;
        rp.w[2] &= r4 ? 0xFFFu : 0u;
        // the tile's codes that can change lie within 4 of those, and read S within 2 more
        Row80 act = full ? Row80{{~0u, ~0u, 0xFFFFu}} : dilate(dilate(dilate(dilate(rp))));
        act.w[0] &= tile_row ? ~0xFFu : 0u;
        act.w[1] &= tile_row ? ~0u : 0u;
        act.w[2] &= tile_row ? 0xFFu : 0u;
        const Row80 reach = dilate(dilate(act));
        if (tile_row) {
            const unsigned long long c = own64(act);
            const int q = 2 * (lane - 8);
            s.act[q] = (uint32_t)c;
            s.act[q + 1] = (uint32_t)(c >> 32);
            // the codes that stay, to which the detection adds
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                const unsigned long long v = w[p][1] & ~c;
                s.code[p * L::kTileWords + q] = (uint32_t)v;
                s.code[p * L::kTileWords + q + 1] = (uint32_t)(v >> 32);
            }
        }
        if (lane == 8)
            sh.buf = own_buf;
        if (lane >= 6 && lane < 42) {          // the S region: rows 6 .. 41, columns 6 .. 73
            uint32_t *q = &s.reach[(lane - 6) * L::HW];
            q[0] = bits_at(reach.w[1], reach.w[0], 6);
            q[1] = bits_at(reach.w[2], reach.w[1], 6);
            q[2] = (reach.w[2] >> 6) & 0xFu;
        }
        // M_k at clamped columns: the windows read it two columns past the frame's edges
        if (x0 == 0)
            m.w[0] |= (m.w[0] >> 8 & 1u) * 0xC0u;
        const int e = W - 1 - x0 + 8;          // the region column of the last frame column
        if (e < 78) {
            const uint32_t b = row_bit(m, e);
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int c = 1; c <= 2; ++c)
                    m.w[i] |= (e + c) >> 5 == i ? b << ((e + c) & 31) : 0u;
        }
        if (lane < 48) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                sh.m[lane][i] = m.w[i];
                sh.r[lane][i] = rp.w[i];
            }
        }
        // list them (in any order): region position row * 80 + column
        const unsigned int cnt = (unsigned int)(__popc(rp.w[0]) + __popc(rp.w[1]) + __popc(rp.w[2]));
        unsigned int at = __ockl_wfscan_add_u32(cnt, false);
        if (lane == 63)
            sh.nrep = at + cnt;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            for (uint32_t v = rp.w[i]; v; v &= v - 1u, ++at)
                if (at < (unsigned int)kRepMax)
                    rep[at] = (uint16_t)(lane * 80 + 32 * i + __ffs((int)v) - 1);
    }
    stage.store(s, tid, 0);
    __syncthreads();
    const int nrep = (int)sh.nrep;
    if (nrep == 0 && !full)
        return;

    // replacement (a flagged pixel's J is read by no other window, so it is updated in
    // place), and meanwhile, by the other waves, the list of the 2 x 5 cell tiles of S that a
    // re-evaluated code reads
    const bool listed = nrep <= kRepMax;
    // (up to NT / 2 of them by pairs of lanes: 240 instructions where one lane takes 430, and most
    // tiles leave half of the lanes idle; the first iteration of the mixed batch 1.11 -> 1.08 ms)
    const bool pairs = nrep <= L::NT / 2;
    for (int i = tid; i < (pairs ? 2 * nrep : (listed ? nrep : 48 * 80)); i += L::NT) {
        const int pos = pairs ? (int)rep[i >> 1] : (listed ? (int)rep[i] : i);
        const int r = pos / 80, c = pos - r * 80;
        if (!listed && !(sh.r[r][c >> 5] >> (c & 31) & 1u))
            continue;
        const int y = y0 - 8 + r, x = x0 - 8 + c;
        uint32_t fl = 0u;
#pragma unroll
        for (int i5 = 0; i5 < 5; ++i5) {
            const uint32_t *q = &sh.m[clampi(y + i5 - 2, H) - y0 + 8][(c - 2) >> 5];
            fl |= (bits_at(q[1], q[0], (c - 2) & 31) & 31u) << (5 * i5);
        }
        const int jr = r - 2, jc = c - 2;
        float nv;
        const bool mine = r >= 8 && r < 40 && c >= 8 && c < 72;
        const float *const pj = &s.J[jr * L::JWP + jc];
        bool some, nan = !pairs;
        if (pairs)
            some = window_median_half(pj, L::JWP, fl, tid & 1, nv, nan);
        if (nan)
            some = window_median(pj, L::JWP, fl, nv);
        if (pairs && (tid & 1))
            continue;
        if (some) {
            s.J[jr * L::JWP + jc] = nv;
            // the staged cells past the frame's edges that repeat this pixel
            if (y == 0 || y == H - 1 || x == 0 || x == W - 1) {
                const int ra = y == 0 ? 0 : jr, rb = y == H - 1 ? L::JH - 1 : jr;
                const int ca = x == 0 ? 0 : jc, cb = x == W - 1 ? L::JW - 1 : jc;
                for (int q = ra; q <= rb; ++q)
                    for (int p = ca; p <= cb; ++p)
                        s.J[q * L::JWP + p] = nv;
            }
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
        if (bits_at(hi, lo, sft) & 31u)
            s.cells[atomicAdd(&s.ncells, 1u)] = (uint16_t)(rp * 16 + cx);
    }
    __syncthreads();
    detect_staged(s, f, y0, x0, tid);

    // the tile's codes of iteration k + 1 into its other buffer, and the tiles it lists
    if (tid < 64) {
        const size_t t = (size_t)ty * ntx + tx;
        const unsigned int buf = sh.buf ^ 1u;
        const unsigned long long *code = reinterpret_cast<const unsigned long long *>(s.code);
        if (!(NARROW && f.narrow)) {
            unsigned long long *o = f.bits + (t * 2 + buf) * (3 * kSumTY);
            o[lane] = code[lane];
            if (lane < kSumTY)
                o[64 + lane] = code[64 + lane];
        } else {
#pragma unroll
            for (int p = 0; p < 3; ++p)
                narrow_store(f, f.bits, (t * 2 + buf) * 3 + p, lane,
                             lane < kSumTY ? code[p * kSumTY + lane] : 0ull);
        }
        // where A lies: bit 3 (dy + 1) + dx + 1 when it is within 8 pixels (an iteration's
        // reach) of the neighbour in direction (dy, dx)
        const unsigned long long a = lane < kSumTY ? code[lane] : 0ull;
        const uint32_t all = (uint32_t)__ballot(a != 0ull);
        const uint32_t left = (uint32_t)__ballot((a & 0xFFull) != 0ull);
        const uint32_t right = (uint32_t)__ballot((a >> 56) != 0ull);
        uint32_t dirs = 0u;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const uint32_t rows = q == 0 ? 0xFFu : (q == 1 ? ~0u : 0xFF000000u);
            dirs |= ((left & rows) ? 1u : 0u) << (3 * q) | ((all & rows) ? 2u : 0u) << (3 * q) |
                    ((right & rows) ? 4u : 0u) << (3 * q);
        }
        // The next iteration has work only within reach of A.  Every tile that holds A now
        // was re-evaluated in this launch (a tile with A at iteration k replaces pixels, A
        // being part of G2), so each lists the tiles that its own A reaches
        const int dy = lane / 3 - 1, dx = lane - (lane / 3) * 3 - 1;
        const int vy = ty + dy, vx = tx + dx;
        const bool there = lane < 9 && vy >= 0 && vy < nty && vx >= 0 && vx < ntx;
        const size_t v = (size_t)(there ? vy : ty) * ntx + (there ? vx : tx);
        if (lane == 0)
            f.state[t] = 2u * (unsigned int)(k + 1) | buf;
        if (there && (dirs >> lane & 1u) &&
            atomicMax(&f.mark[v], (unsigned int)(k + 1)) < (unsigned int)(k + 1) && lists.list[0])
            list_tile(lists, k + 1, f.tile_base + (int)v);
    }
}

// Tile g of a launch, and its frame in the table (-1: the launch's single one).  The kernels copy
// the frame's record themselves, in scalar registers: with the copy inside a function that then
// runs the tile, the compiler held 95 vector registers where it now holds 87, 11 more dwords in
// scratch in the listed form, and issued 61 vector instructions a pixel for 47 (first iterations of the mixed batch 1083 and 206 us
// against 910 and 162, of the 4096 x 4096 field 97 and 87 against 88 and 77; read in place 957
// and 170, 91 and 81).
__device__ __forceinline__ int step_place(const TileRef *__restrict__ tiles, const DevFrame &single,
                                          int g, int &ty, int &tx) {
    if (tiles) {
        const TileRef r = tiles[g];
        ty = r.y0 / kSumTY;
        tx = r.x0 / kSumTX;
        return r.frame;
    }
    const int ntx = (single.W + kSumTX - 1) / kSumTX;
    ty = g / ntx;
    tx = g - ty * ntx;
    return -1;
}
template <bool NARROW>
__device__ __forceinline__ void step_one(const DevFrame &f, int ty, int tx, int kiter, bool by_mark,
                                         const StepLists &lists, StepShared &sh, int tid) {
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
    step_tile<NARROW>(f, ty, tx, k, lists, sh, tid);
}

// Iteration k on every tile of the launch (k == 0: each frame's own).
template <bool NARROW>
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
    int ty, tx;
    DevFrame f;
    const int fi = step_place(tiles, single, (int)blockIdx.x, ty, tx);
    if (tiles)
        f = frames[fi];
    else
        f = single;
    step_one<NARROW>(f, ty, tx, kiter, true, lists, sh, tid);
}

// The tiles of a list: block b takes entries b / nseg, b / nseg + stride, ... of segment
// b % nseg.  kiter: the iteration (0: each frame's own).
template <bool NARROW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5)))
void k_step_listed(const DevFrame *__restrict__ frames, const TileRef *__restrict__ tiles,
                   DevFrame single, int kiter, TileList in, StepLists lists) {
    __shared__ StepShared sh;
    if (blockIdx.x == 0 && lists.list[0])
        lists_clear(lists, kiter + 2, (int)threadIdx.x);
    const int seg = (int)blockIdx.x & (in.nseg - 1), stride = (int)gridDim.x / in.nseg;
    const unsigned int *list = in.list + (size_t)seg * in.cap;
    const int n = min((int)in.count[seg * kTicketStride], in.cap);
    for (int e = (int)blockIdx.x / in.nseg; e < n; e += stride) {
        // as in the persistent detection, thread-derived values are not held across tiles
        int tid = (int)threadIdx.x;
        asm volatile("" : "+v"(tid));
        // (uniform: the tile and frame records then load into scalar registers)
        const int g = __builtin_amdgcn_readfirstlane((int)list[e]);
        int ty, tx;
        DevFrame f;
        const int fi = step_place(tiles, single, g, ty, tx);
        if (tiles)
            f = frames[fi];
        else
            f = single;
        step_one<NARROW>(f, ty, tx, kiter, false, lists, sh, tid);
        __syncthreads();       // the tile is done with the LDS
    }
}

// Blocks of a listed launch: a multiple of the segments, about as many as the device holds.
static int listed_grid(size_t ntiles, int nseg) {
    const size_t per = (ntiles + nseg - 1) / nseg, most = 1280 / nseg;
    return (int)(per < most ? per : most) * nseg;
}

template <bool NARROW>
static hipError_t launch_step_as(const DevFrame *d_frames, const TileRef *d_tiles, int ntiles,
                                 const DevFrame &single, int k, bool all, const StepLists &lists,
                                 unsigned int *tickets, hipStream_t s) {
    if (k <= 1 || all || !lists.list[0]) {
        k_step<NARROW><<<ntiles, 256, 0, s>>>(d_frames, d_tiles, single, k, lists, tickets);
    } else {
        const TileList in = {lists.list[k & 1],
                             lists.count + (size_t)(k % 3) * lists.nseg * kTicketStride,
                             lists.nseg, lists.cap};
        k_step_listed<NARROW><<<listed_grid((size_t)ntiles, in.nseg), 256, 0, s>>>(
            d_frames, d_tiles, single, k, in, lists);
    }
    return hipGetLastError();
}

hipError_t launch_step(const DevFrame *d_frames, const TileRef *d_tiles, int ntiles,
                       const DevFrame &single, int k, bool all, bool narrow,
                       const StepLists &lists, unsigned int *tickets, hipStream_t s) {
    if (!d_tiles)
        ntiles = detect_tiles(single.H, single.W, kSumTY);
    if (ntiles <= 0)
        return hipSuccess;
    const auto as = narrow ? launch_step_as<true> : launch_step_as<false>;
    return as(d_frames, d_tiles, ntiles, single, k, all, lists, tickets, s);
}

hipError_t launch_step_active(const DevFrame *d_frames, const TileRef *d_tiles, size_t ntiles,
                              bool narrow, const TileList &active, hipStream_t s) {
    DevFrame none = {};
    const StepLists lists = {};
    const auto kernel = narrow ? k_step_listed<true> : k_step_listed<false>;
    kernel<<<listed_grid(ntiles, active.nseg), 256, 0, s>>>(d_frames, d_tiles, none, 0, active,
                                                            lists);
    return hipGetLastError();
}

}  // namespace crb
