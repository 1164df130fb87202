// The detection of one LDS tile, shared by the first-iteration kernel (detect.hip), which
// evaluates whole tiles, and the iteration kernel (step.hip), which re-evaluates a tile only
// near the pixels its replacement changed.
#pragma once

#include "kernels.h"
#include "device_common.h"

#include <math.h>

namespace crb {

#include "medtile.inc"

// Exclusive prefix sum over the lanes of a wave (all lanes active), from the device
// library's cross-lane (DPP) primitives.
extern "C" __device__ unsigned int __ockl_wfscan_add_u32(unsigned int, bool);

// 3x3 medians of a run of N horizontally adjacent outputs from three rows of N+2
// inputs.  Each column of three is sorted once (shared by up to three windows);
// the median of a 3x3 window with sorted columns is the median of
// (max of the column minima, median of the column medians, min of the column maxima).
template <int N>
__device__ __forceinline__ void med3_run(const float (&a)[N + 2], const float (&b)[N + 2],
                                         const float (&c)[N + 2], float (&o)[N]) {
    float lo[N + 2], mi[N + 2], hi[N + 2];
#pragma unroll
    for (int j = 0; j < N + 2; ++j) {
        lo[j] = min3f(a[j], b[j], c[j]);
        mi[j] = med3f(a[j], b[j], c[j]);
        hi[j] = max3f(a[j], b[j], c[j]);
    }
#pragma unroll
    for (int j = 0; j < N; ++j)
        o[j] = med3f(max3f(lo[j], lo[j + 1], lo[j + 2]), med3f(mi[j], mi[j + 1], mi[j + 2]),
                     min3f(hi[j], hi[j + 1], hi[j + 2]));
}

// The four sub-pixels of the 2x block of a pixel of value c each have two
// neighbours inside the block (value c) and two outside (u above or d below,
// l left or r right).  Clipped Laplacian 4c - u - d - l - r of each, in that order,
// then the 2x2 mean, matching the literal 2x-grid computation term for term.
__device__ __forceinline__ double lplus(double c, double u, double d, double l, double r) {
    double s00 = 4.0 * c - u - c - l - c;
    double s01 = 4.0 * c - u - c - c - r;
    double s10 = 4.0 * c - c - d - l - c;
    double s11 = 4.0 * c - c - d - c - r;
    s00 = s00 > 0.0 ? s00 : 0.0;
    s01 = s01 > 0.0 ? s01 : 0.0;
    s10 = s10 > 0.0 ? s10 : 0.0;
    s11 = s11 > 0.0 ? s11 : 0.0;
    return (s00 + s01 + s10 + s11) / 4.0;
}

// ---------------------------------------------------------------------------
// detection
// ---------------------------------------------------------------------------

// Fourth word of a raw buffer resource on gfx9-family GPUs: 32-bit data format, no
// swizzle, range-checked against the byte count given with the base.
constexpr int kBufferWord3 = 0x00020000;

// FP32 parameters of the S estimate; ok is false for gains outside [2^-100, 2^100]
// (where g/8 could round), which leaves every decision to the binary64 evaluation.
struct SEstParams {
    float gain, g8, inv_gain, sky, rn2;
    bool ok;
};

__device__ __forceinline__ SEstParams sest_params(const DevFrame &f) {
    SEstParams p;
    p.gain = f.gain;
    p.g8 = f.g8;
    p.inv_gain = f.inv_gain;
    p.sky = f.sky;
    p.rn2 = f.rn2f;
    p.ok = f.est_ok != 0;
    return p;
}

// The sum l4 over the four sub-pixels of max(2c - v1 - v2, 0) (v1 in {up, dn}, v2 in
// {lf, rt}), which is 4 L+ at a pixel of value c with 4-neighbours up, dn, lf, rt.  The
// terms pair up by their vertical neighbour: with a = 2c - up, max(a - lf, 0) +
// max(a - rt, 0) = max(2a - (lf + rt), a - min(lf, rt), 0) (the first argument wins when
// a is above both horizontal neighbours, the second when it lies between them, 0 below
// both), and the same with b = 2c - dn.  Evaluated as written (two FMAs for a and b,
// lf + rt, the minimum, per pair one FMA, one subtraction and a max3, one final
// addition; 11 operations where the term-by-term sum takes 13), with u = 2^-24 and round
// to nearest: each pair is within 2u M_a of its exact value, M_a = 4|c| + 2|up| + |lf| +
// |rt| (likewise M_b), and the sum within 3u (M_a + M_b) = 6u M of 4 L+, M = 4|c| + |up|
// + |dn| + |lf| + |rt|.
__device__ __forceinline__ float lplus4(float c, float up, float dn, float lf, float rt) {
    const float a = fmaf(2.0f, c, -up), b = fmaf(2.0f, c, -dn);
    const float s = lf + rt, m = fminf(lf, rt);
    return max3f(fmaf(2.0f, a, -s), a - m, 0.0f) + max3f(fmaf(2.0f, b, -s), b - m, 0.0f);
}

// FP32 estimate s of S at a pixel of value c with 4-neighbours up, dn, lf, rt and
// med5(J) = m5, and a bound err >= |s - S|, S being the binary64 value of the
// definition (S = L+ / (2N), L+ = a quarter of the sum over the four sub-pixels of
// max(2c - v1 - v2, 0), N = sqrt(g m + rn^2) / g).  Error analysis, u = 2^-24,
// round to nearest with FP32 denormals preserved, M = 4|c| + |up| + |dn| + |lf| + |rt|:
//   the sub-pixel sum l4 (lplus4) is 4 L+ within 6.01 u M;
//   t = g m + rn^2 (positive terms, m itself rounded once) carries at most 3.03 u
//     relative error, so t^-1/2 at most 1.52 u; the reciprocal square root (v_rsq_f32,
//     within 1 ulp = 2u), the scaling by g/8 (exact) and the two products add 2u + 2u;
//   the binary64 evaluation is within 2^-49 (M R + S) of the exact value;
// so |s - S| <= 6.01 u M R + 5.52 u s with R = g/(8 sqrt t), which err = 2^-19 (M R + s)
// overstates at least four-fold (the s-term tolerates a reciprocal square root 14 ulp
// off).  Outside t in [2^-100, 2^100] and M <= 2^100 (where the
// analysis has no overflow, underflow or domain edge) s = err = +inf, which sends every
// decision that reads the pixel to the binary64 evaluation.
__device__ __forceinline__ float s_estimate(float c, float up, float dn, float lf, float rt,
                                            float m5, const SEstParams &p, float &err) {
    const float l4 = lplus4(c, up, dn, lf, rt);
    float m = m5 + p.sky;
    m = (m <= 0.0f) ? 1e-4f : m;
    const float t = fmaf(p.gain, m, p.rn2);
    const float R = p.g8 * __builtin_amdgcn_rsqf(t);
    const float s = l4 * R;
    const float M = fmaf(4.0f, fabsf(c), fabsf(up)) + fabsf(dn) + (fabsf(lf) + fabsf(rt));
    const bool sane = __builtin_amdgcn_fmed3f(t, 0x1p-100f, 0x1p100f) == t && M <= 0x1p100f && p.ok;
    err = sane ? (M * R + s) * 0x1p-19f : INFINITY;
    return sane ? s : INFINITY;
}

// The factor R = (g/8) t^-1/2 of the S estimate, t = g m + rn^2, for a lower bound x of
// med5(J): m = x + sky, or 0 where that is at most 1e-4 (N of the definition never falls
// below rn/g, while above the definition's floor it grows with med5(J)), so the estimate
// from R, with its error bound, bounds S from above for every med5(J) >= x.  INFINITY
// where the error analysis of the estimate does not hold.
__device__ __forceinline__ float r_bound(float x, const SEstParams &p) {
    float m = x + p.sky;
    m = (m <= 1e-4f) ? 0.0f : m;
    const float t = fmaf(p.gain, m, p.rn2);
    const bool sane = __builtin_amdgcn_fmed3f(t, 0x1p-100f, 0x1p100f) == t && p.ok;
    return sane ? p.g8 * __builtin_amdgcn_rsqf(t) : INFINITY;
}

// An upper bound of S at a pixel of value c with 4-neighbours up, dn, lf, rt, given
// Rp = R (1 + 2^-19) rounded, R = r_bound(x) finite for a lower bound x of its med5(J),
// and E = 2^-19 * 8 v * R with v >= each |value| read and 8 v <= 2^100.  With l4 =
// lplus4 (within 6u M of 4 L+) and R's own error (at most 5u relative, as in
// s_estimate), S <= (l4 + 6u M) R (1 + 5u), while fl(l4 Rp + E) >= l4 R (1 + 2^-19 -
// 2.1u) + E (1 - u) and E >= 32u M R (1 - u): the returned value exceeds S, so where it
// is at most sigclip (less 2^-20), S <= sigclip.
__device__ __forceinline__ float s_upper(float c, float up, float dn, float lf, float rt,
                                         float Rp, float E) {
    return fmaf(lplus4(c, up, dn, lf, rt), Rp, E);
}

// The dense bound of a 2 x 5 cell tile from its 6 x 9 patch of J (patch row i, column j
// is cell row i - 2, column j - 2; clamped where the patch leaves the frame): u[5 i + j]
// >= S at cell (i, j) for every cell of the tile, unless the function returns false (R
// not finite or a value above 2^96 in magnitude: the analysis of the bound does not
// hold, and every cell must count as a candidate).
//   x: a lower bound of med5(J) shared by the tile's ten windows, the least value of
//   patch rows 1-4 (every window holds those four rows of its five columns, so 20 of its
//   25 values are >= x; 18 three-input minima).  S does not increase with med5(J), so
//   the estimate at x with its error bound bounds S from above.  (The least over the
//   columns of each column's second smallest in rows 1-4 is a tighter bound, with 15
//   values >= it, but costs 63 operations; with the least value H' grows by about 3%
//   and the region of exact med5(J) by about 7%.)
//   E: one error term for the ten cells: every value their M reads lies in patch rows
//   1-4, columns 1-7, so M <= 8 vmax.
__device__ __forceinline__ bool dense_bounds(const float (&v)[6 * 9], const SEstParams &sp,
                                             float (&u)[10]) {
    constexpr int PW = 9, NV = 4 * PW;
    float x = v[PW];
#pragma unroll
    for (int k = 1; k + 1 < NV; k += 2)
        x = min3f(x, v[PW + k], v[PW + k + 1]);
    if (NV % 2 == 0)
        x = fminf(x, v[PW + NV - 1]);
    const float R = r_bound(x, sp);
    float vmax = 0.0f;
#pragma unroll
    for (int i = 1; i <= 4; ++i)
#pragma unroll
        for (int j = 1; j <= 7; ++j)
            vmax = fmaxf(vmax, fabsf(v[i * PW + j]));
    const float E = (8.0f * vmax) * R * 0x1p-19f;
    const float Rp = fmaf(R, 0x1p-19f, R);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 5; ++j) {
            const int pc = (i + 2) * PW + (j + 2);
            u[i * 5 + j] = s_upper(v[pc], v[pc - PW], v[pc + PW], v[pc - 1], v[pc + 1], Rp, E);
        }
    return R < INFINITY && vmax <= 0x1p96f;
}

// S exactly as the definition evaluates it (binary64, in its operation order), at the
// in-frame pixel whose staged J cell is p (pitch jp; the staged plane holds J at clamped
// positions, so the cells around p are the clamped 5 x 5 window), and the N it is formed with.
__device__ __forceinline__ double s_exact(const float *p, int jp, double gain, double sky,
                                          double rn2, double &N) {
    float w[25], m5[1];
#pragma unroll
    for (int i = 0; i < 5; ++i)
#pragma unroll
        for (int j = 0; j < 5; ++j)
            w[i * 5 + j] = p[(i - 2) * jp + j - 2];
    med5_t1x1(w, m5);
    const double lp = lplus(w[12], w[7], w[17], w[11], w[13]);
    double m = (double)m5[0] + sky;
    if (m <= 0.0)
        m = 1e-4;
    N = sqrt(gain * m + rn2) / gain;
    return lp / (2.0 * N);
}

// med3(J) at the pixel whose staged J cell is p (pitch jp).  The staged plane holds
// J at clamped positions, so for an in-frame pixel this is the clamped 3 x 3 window:
// with each column sorted, the median of nine is the median of the largest column
// minimum, the median of the column medians and the smallest column maximum.
__device__ __forceinline__ float med3_at(const float *p, int jp) {
    float lo[3], mi[3], hi[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        const float a = p[-jp + j - 1], b = p[j - 1], c = p[jp + j - 1];
        lo[j] = min3f(a, b, c);
        mi[j] = med3f(a, b, c);
        hi[j] = max3f(a, b, c);
    }
    return med3f(max3f(lo[0], lo[1], lo[2]), med3f(mi[0], mi[1], mi[2]),
                 min3f(hi[0], hi[1], hi[2]));
}

// Staged J cell (pitch jp, apron 4 around the tile at (y0, x0)) of the in-frame pixel
// nearest to tile position (r + dy, c + dx): where med3(J) is read for the 7 x 7 window
// of a tile pixel (the window is clamped to the frame).
__device__ __forceinline__ const float *med3_cell(const float *sJ, int jp, int y0, int x0,
                                                  int H, int W, int r, int c, int dy, int dx) {
    return &sJ[(clampi(y0 + r + dy, H) - y0 + 4) * jp + (clampi(x0 + c + dx, W) - x0 + 4)];
}

// The contrast test S'/F^ > objlim in binary64 at tile pixel (r, c), med3 taken from the
// staged J, F^ = max((med3 - med7(med3)) / N, 0.01), by the calling wave (all lanes active,
// arguments uniform).  The test, evaluated in the definition's operations with a value x in
// place of med7, is monotone in x (every step and every rounding is), and med7 is the 25th of
// the 49 window values, with 24 on either side; so the test holds at med7 iff it holds at 25 or
// more of them.  Lane l < 49 takes window cell (l / 7 - 3, l % 7 - 3).
__device__ __forceinline__ bool contrast_exact(const float *sJ, int jp, int y0, int x0, int H,
                                               int W, int r, int c, double spr, double N,
                                               double objlim, int lane) {
    const int l49 = lane < 49 ? lane : 24;
    const float xf = med3_at(med3_cell(sJ, jp, y0, x0, H, W, r, c, l49 / 7 - 3, l49 % 7 - 3), jp);
    const double m3 = (double)__int_as_float(__builtin_amdgcn_readlane(__float_as_int(xf), 24));
    const double x = (double)xf;
    double fh = (m3 - x) / N;
    fh = fh < 0.01 ? 0.01 : fh;
    return __popcll(__ballot(lane < 49 && spr / fh > objlim)) >= 25;
}

// N at a pixel from its FP32 estimate s = l4 R of S (s_estimate; R = (g/8) rsq(t), and l4
// the pixel's L+ sum formed as the estimate formed it): N = 1 / (8 R) = l4 / (8 s).  R is
// within 4.52u of g / (8 sqrt(t)) for the definition's t (t to 3.03u, so its -1/2 power
// to 1.52u; the reciprocal square root to 1 ulp = 2u; the product by g/8 to u), s adds
// u and the division u: N is within 6.52u of the definition's (u = 2^-24), for any
// s > 0 with a finite error bound.
__device__ __forceinline__ float noise_from_estimate(float l4, float s) {
    return l4 / (8.0f * s);
}

// The switching values of the contrast test below, from med3 (m3) and N at the pixel:
// a window value x > t_sure makes the test hold for every S' >= lo, one with x >= t_maybe
// lets it hold for some S' <= hi.
__device__ __forceinline__ void contrast_thresholds(float m3, float N, float lo, float hi,
                                                    float inv_olim, float &t_sure,
                                                    float &t_maybe) {
    const float klo = N * lo * inv_olim, khi = N * hi * inv_olim;
    t_sure = (m3 - klo) + fmaf(0x1p-19f, fabsf(m3) + klo, 0x1p-126f);
    t_maybe = (m3 - khi) - fmaf(0x1p-19f, fabsf(m3) + khi, 0x1p-126f);
}

// The contrast test S'/F^ > objlim at tile pixel (r, c), for every S' in [lo, hi]
// (0 < lo), without selecting med7, by the calling wave (all lanes active, arguments
// uniform): 1 if it holds for all of them, 0 if it fails for all, -1 if undecided.
//   F^ does not increase with med7 (m3 - med7, the division by N > 0, the floor at 0.01
//   and their roundings are monotone), so at fixed S' the test, as a function of the
//   value x taken by med7, holds above a switching value and nowhere below it; med7 is
//   the 25th smallest of the 49 window values, so the test holds at med7 iff it holds
//   at 25 or more of them.
//   If fl(S'/0.01) <= objlim the test fails whatever x (F^ >= 0.01); 100 S' in FP32 is
//   within 1.01u of that binary64 quotient (u = 2^-24), so comparing it with objlim
//   widened or narrowed by 2^-21 relative decides this for the whole interval (the
//   caller does, before listing the pixel).
//   Otherwise the test holds at x iff m3 - x < K (1 + e), K = N S'/objlim, |e| <=
//   4 * 2^-53.  K from N in FP32 (within 8u: noise_from_estimate gives 6.52u) and two
//   more products is within 11u, so x above T = m3 - K up to a band of 2^-19 (|m3| + K)
//   + 2^-126 (three-fold the roundings) decides the test.  The test is larger for larger
//   S', so lo bounds its certain holding and hi its possible holding.
// N is the noise at the pixel (noise_from_estimate); lane l < 49 takes the med3 value of
// window cell (l / 7 - 3, l % 7 - 3), and ballots count them.
__device__ __forceinline__ int contrast_by_count(const float *sJ, int jp, int y0, int x0,
                                                 int H, int W, int r, int c, float N, float lo,
                                                 float hi, float inv_olim, int lane) {
    const int l49 = lane < 49 ? lane : 24;
    const float x = med3_at(med3_cell(sJ, jp, y0, x0, H, W, r, c, l49 / 7 - 3, l49 % 7 - 3), jp);
    const float m3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 24));
    float t_sure, t_maybe;
    contrast_thresholds(m3, N, lo, hi, inv_olim, t_sure, t_maybe);
    const int sure = __popcll(__ballot(lane < 49 && x > t_sure));
    const int maybe = __popcll(__ballot(lane < 49 && x >= t_maybe));
    return sure >= 25 ? 1 : (maybe < 25 ? 0 : -1);
}

// The same test by one thread (for pixels beyond the contrast list): the 49 med3 values
// one after another.
__device__ __forceinline__ int contrast_by_count_lane(const float *sJ, int jp, int y0, int x0,
                                                      int H, int W, int r, int c, float N,
                                                      float lo, float hi, float inv_olim) {
    const float m3 = med3_at(med3_cell(sJ, jp, y0, x0, H, W, r, c, 0, 0), jp);
    float t_sure, t_maybe;
    contrast_thresholds(m3, N, lo, hi, inv_olim, t_sure, t_maybe);
    int sure = 0, maybe = 0;
#pragma unroll 1
    for (int i = 0; i < 7; ++i) {
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const float x = med3_at(med3_cell(sJ, jp, y0, x0, H, W, r, c, i - 3, j - 3), jp);
            sure += x > t_sure ? 1 : 0;
            maybe += x >= t_maybe ? 1 : 0;
        }
    }
    return sure >= 25 ? 1 : (maybe < 25 ? 0 : -1);
}

// Exclusive prefix sums of the set-bit counts of the NWORDS words of a bitmap into
// pre[0 .. NWORDS-1], the total into pre[NWORDS]; by the first wave (all 64 lanes), each
// lane taking NWORDS / 64 consecutive words (or one, or none past NWORDS, when NWORDS is
// at most 64).
template <int NWORDS>
__device__ __forceinline__ void bitmap_prefix(const uint32_t *bits, uint32_t *pre) {
    static_assert(NWORDS <= 64 || NWORDS % 64 == 0, "whole words per lane");
    constexpr int WPL = NWORDS > 64 ? NWORDS / 64 : 1;
    const int lane = threadIdx.x & 63;
    unsigned int c[WPL], tot = 0u;
#pragma unroll
    for (int i = 0; i < WPL; ++i) {
        const int w = lane * WPL + i;
        c[i] = w < NWORDS ? (unsigned int)__popc(bits[w]) : 0u;
        tot += c[i];
    }
    unsigned int ex = __ockl_wfscan_add_u32(tot, false);
#pragma unroll
    for (int i = 0; i < WPL; ++i) {
        const int w = lane * WPL + i;
        if (w < NWORDS)
            pre[w] = ex;
        ex += c[i];
    }
    if (lane == 63)
        pre[NWORDS] = ex;
}

// Position (word * 32 + bit) of the q-th set bit of an NWORDS-word bitmap with prefix pre.
template <int NWORDS>
__device__ __forceinline__ int bitmap_select(const uint32_t *bits, const uint32_t *pre, int q) {
    int lo = 0, hi = NWORDS - 1;    // last word whose prefix is <= q
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((int)pre[mid] <= q)
            lo = mid;
        else
            hi = mid - 1;
    }
    uint32_t b = bits[lo];
    for (int n = q - (int)pre[lo]; n > 0; --n)
        b &= b - 1u;
    return lo * 32 + __ffs(b) - 1;
}

// Appends pos0 + b for every set bit b of m (one word per lane; called by whole waves) to
// an LDS list: places within the wave by a DPP prefix sum, the wave's base by one LDS
// atomic on *count, so that several waves append in any order.  Entries at or beyond cap
// are not stored; *count ends as the number of bits appended by all waves.
__device__ __forceinline__ void list_append(uint32_t m, int pos0, uint16_t *list,
                                            unsigned int *count, unsigned int cap, int lane) {
    const unsigned int cnt = (unsigned int)__popc(m);
    unsigned int at = __ockl_wfscan_add_u32(cnt, false);
    const unsigned int total = (unsigned int)__builtin_amdgcn_readlane((int)(at + cnt), 63);
    unsigned int base = 0u;
    if (lane == 0 && total)
        base = atomicAdd(count, total);
    at += (unsigned int)__builtin_amdgcn_readfirstlane((int)base);
    for (uint32_t mm = m; mm; mm &= mm - 1u, ++at)
        if (at < cap)
            list[at] = (uint16_t)(pos0 + __ffs(mm) - 1);
}

// Contrast tests that a block takes with one wave per pixel (94 instructions each, four at a
// time); more of them share their windows' med3 values, at three more barriers.  The first
// detection took 116 -> 98 us on a crowded 4096 x 4096 field (28 tests a tile), 30 -> 25 us on
// the 800 x 800 frame (46) and 1.28 -> 1.24 ms on the mixed batch (13); with the line at 4, 8,
// 24 tests the batch took 1.29, 1.28 and 1.27 ms, the field the same to 1%.
constexpr int kConWaves = 16;

// Work shapes inside a detection block: a lower bound of med5(J), L+ and an upper bound
// of S in 2 x 5 thread tiles over the whole tile and its 2-pixel apron; med5(J) and the S
// estimate in 2 x 2 quads near where S may exceed sigclip.  The remaining statistics,
// med3 among them, are evaluated only where a code bit can matter.

// The maps of a tile that is re-evaluated only in places: its pixels whose code is (bitmap),
// the S cells they read (bitmap rows over the S region), and the listed 2 x 5 cell tiles that
// meet those.
template <int TY, bool SPARSE>
struct DetectMaps {};
template <int TY>
struct DetectMaps<TY, true> {
    uint32_t act[2 * TY], reach[3 * (TY + 4)];
    uint16_t cells[(TY + 5) / 2 * 14];
    unsigned int ncells;
};

// The LDS of a detection tile: TY rows of 64 columns, one block of 8 * TY threads.  AP is
// the apron of the staged J (at least 4, the reach of a code into J); SPARSE adds the maps
// of a tile that is re-evaluated only in places.
template <int TY, int AP, bool SPARSE>
struct DetectLds : DetectMaps<TY, SPARSE> {
    static constexpr int TX = 64, NT = 8 * TY, NW = NT / 64;
    // logical extents of the planes and their row pitches; the pitches spread the dense
    // and exact passes' scalar accesses over the LDS banks
    static constexpr int JH = TY + 2 * AP, JW = TX + 2 * AP;
    static constexpr int JWP = JW + 1;
    static constexpr int SH = TY + 4, SW = TX + 4, SWP = TX + 6;    // S estimate, apron 2
    static constexpr int HW = (SW + 31) / 32;   // words per row of the hot bitmap
    // the hot bitmap is stored with 4 zero rows above and below and a zero word before
    // each row (which is also the word after the previous row; one more zero word ends
    // the array), so that its dilations read it without bounds tests
    static constexpr int HWP = HW + 1, HR = SH + 8;
    static constexpr int QW = TX / 32;          // words per row of the tile bitmaps
    static constexpr int kTileWords = TY * QW;
    // 2 x 5 cell tiles of the dense pass, 2 x 2 quads of the exact pass
    static constexpr int NTY = (SH + 1) / 2, NTX = (SW + 4) / 5;
    static constexpr int NP = SH / 2, kQuads = NP * SW / 2;
    // pixels per round of the binary64 re-evaluation (25 threads each)
    static constexpr int kExactBatch = NT / 25;
    // pixels whose contrast test a block lists for its contrast phase; further ones take the
    // same test in their own lanes
    static constexpr int kConMax = kQuads * 2 / 16;
    // med3 plane of the contrast phase: the tile with an apron of 3
    static constexpr int MH = TY + 6, MW = TX + 6;
    static constexpr int kSPlane = SH * SWP > MH * MW ? SH * SWP : MH * MW;
    // work-set pixels a block lists; a larger work set is taken from its bitmap instead
    static constexpr int kListMax = 8 * TY;
    static_assert(AP >= 4 && NW * 64 == NT && QW == 2, "whole waves; two bitmap words per row");
    static_assert(QW + 1 <= HW, "dilation reads two bitmap words per work word");
    static_assert(kSPlane * 4 >= kExactBatch * 27 * 8, "re-evaluation buffer in the S plane");
    static_assert((kTileWords + 1) * 4 <= kListMax * 2, "bitmap prefix in the work list");
    static_assert(SH % 2 == 0 && SW % 2 == 0, "whole quads");
    static_assert(SW == 68 && HW == 3 && NTX == 14, "the sizes of DetectMaps");

    __align__(16) float J[JH * JWP];            // J at clamped positions
    // S; after the work set, med3 near the contrast pixels; then the re-evaluation buffer
    __align__(16) float S[kSPlane];
    // (these two are also read as 64-bit rows)
    __align__(8) uint32_t code[3 * kTileWords]; // code planes A, [S' > sigclip], [S' > low]
    __align__(8) uint32_t con_map[kTileWords];  // pixels listed for the contrast phase
    uint32_t hotp[HR * HWP + 1];                // H', apron 2, in-frame
    uint32_t u[kTileWords];                     // pixels left to binary64
    // tile cells where S may exceed sigfrac*sigclip; after the work-set build, Q' itself
    uint32_t low[kTileWords];
    unsigned int err_bits, contrast, uncertain, qcount, need, exact_cells, con_count, any_hot;
    union {
        uint16_t quads[kQuads];
        // (once the quads are done) the contrast phase's pixels: position, S' interval, N
        struct {
            uint32_t con_info[kConMax];
            float con_lo[kConMax], con_hi[kConMax], con_n[kConMax];
        };
    };
    // work set Q' (up to kListMax); then runs of med3 cells; then the prefix of u
    __align__(4) uint16_t list[kListMax];

    // word w of region row r of H' (r in [-4, SH + 4), w in [-1, HW]; zero outside)
    __device__ __forceinline__ uint32_t *hot() { return &hotp[4 * HWP + 1]; }
    // the staged J as if its apron were 4: cell (r + 4, c + 4) is tile pixel (r, c)
    __device__ __forceinline__ float *j4() { return &J[(AP - 4) * (JWP + 1)]; }
};

// Clears the bitmaps and the counters of a tile, and its code planes (SPARSE: the caller
// fills them with the codes that stay), before the first barrier.
template <int TY, int AP, bool SPARSE>
__device__ __forceinline__ void detect_clear(DetectLds<TY, AP, SPARSE> &s, int tid) {
    using L = DetectLds<TY, AP, SPARSE>;
    for (int i = tid; i < L::HR * L::HWP + 1; i += L::NT)
        s.hotp[i] = 0u;
    if constexpr (!SPARSE)
        for (int i = tid; i < 3 * L::kTileWords; i += L::NT)
            s.code[i] = 0u;
    for (int i = tid; i < L::kTileWords; i += L::NT) {
        s.u[i] = 0u;
        s.low[i] = 0u;
        s.con_map[i] = 0u;
    }
    if (tid == 0) {
        s.err_bits = 0u;
        s.contrast = 0u;
        s.uncertain = 0u;
        s.qcount = 0u;
        s.need = 0u;
        s.exact_cells = 0u;
        s.con_count = 0u;
        s.any_hot = 0u;
        if constexpr (SPARSE)
            s.ncells = 0u;
    }
}

// Staging of J over [y0 - AP, y0 + TY + AP) x [x0 - AP, x0 + TX + AP), clamped reads.
// Thread t takes column t % JW of rows t / JW + kStep * b, so its clamped column is computed
// once and, on tiles whose rows are all inside the frame, each further row costs one address
// step.  A thread's loads (or a round of them, from row block b0) are all issued before its
// first LDS store, so their latencies overlap.
template <class L, int AP>
struct JStage {
    static constexpr int kStep = L::NT / L::JW;
    static constexpr int kBlocks = (L::JH + kStep - 1) / kStep;
    static constexpr int kRound = kBlocks > 16 ? (kBlocks + 1) / 2 : kBlocks;
    float v[kRound];

    __device__ __forceinline__ void load(const float *__restrict__ J, int H, int W, int y0, int x0,
                                         int tid, int b0) {
        const int c = tid % L::JW, r0 = tid / L::JW;
        if (r0 >= kStep)
            return;
        const int cc = clampi(x0 - AP + c, W);
        if (y0 >= AP && y0 - AP + L::JH <= H && (long long)L::JH * W * 4 <= 0x7fffffffll) {
            // buffer loads over the JH staged rows (below 2^31 bytes, so the byte count, the
            // lane offsets and the row steps below are exact in int): a per-lane byte offset
            // and a uniform row step, so a further row costs no vector instruction
            const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
                (void *)(J + (size_t)(y0 - AP) * W), (short)0, L::JH * W * 4, kBufferWord3);
            const int boff = (r0 * W + cc) * 4;
#pragma unroll
            for (int b = 0; b < kRound; ++b)
                if (b0 + b < kBlocks && r0 + kStep * (b0 + b) < L::JH)
                    v[b] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                        rows, boff, kStep * (b0 + b) * W * 4, 0));
        } else {
#pragma unroll
            for (int b = 0; b < kRound; ++b)
                if (b0 + b < kBlocks && r0 + kStep * (b0 + b) < L::JH)
                    v[b] = J[(size_t)clampi(y0 - AP + r0 + kStep * (b0 + b), H) * W + cc];
        }
    }
    __device__ __forceinline__ void store(L &s, int tid, int b0) const {
        const int c = tid % L::JW, r0 = tid / L::JW;
        if (r0 >= kStep)
            return;
#pragma unroll
        for (int b = 0; b < kRound; ++b)
            if (b0 + b < kBlocks && r0 + kStep * (b0 + b) < L::JH)
                s.J[(r0 + kStep * (b0 + b)) * L::JWP + c] = v[b];
    }
};

// Sets the code bits of tile position pos (r * 64 + c).
template <class L>
__device__ __forceinline__ void set_code(L &s, int pos, bool first, bool high, bool low) {
    const uint32_t b = 1u << (pos & 31);
    const int w = pos >> 5;
    if (first)
        atomicOr(&s.code[w], b);
    if (high)
        atomicOr(&s.code[L::kTileWords + w], b);
    if (low)
        atomicOr(&s.code[2 * L::kTileWords + w], b);
}

// The detection of one staged tile (origin y0, x0 of frame f), by the whole block: the code
// bits of the tile's in-frame pixels ORed into s.code (cleared; s.J staged, and both visible
// to the block), visible to the whole block on return.
// With SPARSE only the pixels of s.act are evaluated (s.code cleared there), from the S cells of s.reach (at
// least the cells within 2 of s.act) and the cell tiles listed in s.cells.
//
// Which pixels need S', F^ and the threshold bits.  With H = {S > sigclip} (S' > t
// implies S > t for t >= 0: med5(S) >= 0 because S >= 0, and rounding is monotone):
//   first(p) can be 1 only on H;
//   G1(p) needs an A pixel within distance 1, so hi(p) matters only on D1(H);
//   G2(p) needs a G1 pixel within distance 1, so lo(p) matters only on D2(H);
// and lo(p) = hi(p) = 0 wherever S(p) <= sigfrac * sigclip (sigfrac <= 1).  The block
// bounds S from above on the tile and its apron (from a lower bound of med5(J)), then
// computes the FP32 estimate s of S with its error bound err within 4 of where that
// bound exceeds sigclip, takes H' = {s + err > sigclip (less a margin)} (a superset of
// H), and evaluates the codes on Q' = D2(H') & {s + err > sigfrac * sigclip (less a
// margin)}, a superset of Q = D2(H) & {S > sigfrac*sigclip}: med5 of the estimates
// gives S' within twice the block's largest error (the median moves no more than its
// inputs), which decides the two bits, and F^ with the interval of S' decides the
// contrast test; a pixel where an interval straddles a threshold is re-evaluated in
// binary64 from J.  So every code written is the full definition's, codes outside Q'
// are 0, and the grow, which reads codes only through its two dilations, sees the full
// definition.
template <int TY, int AP, bool SPARSE>
__device__ __forceinline__ void detect_staged(DetectLds<TY, AP, SPARSE> &s, const DevFrame &f,
                                              int y0, int x0, int tid) {
    using L = DetectLds<TY, AP, SPARSE>;
    constexpr int TX = L::TX, NT = L::NT;
    constexpr int kConMax = L::kConMax, kListMax = L::kListMax, kExactBatch = L::kExactBatch;
    const int H = f.H, W = f.W;
    const int lane = tid & 63;
    const float *const sJ = s.j4();
    uint32_t *const sHot = s.hot();
    double *const sX = reinterpret_cast<double *>(s.S);
    // thresholds widened by 2^-20 relative: fl(x) beyond them decides the real x
    // against the binary64 thresholds sigclip and sigfrac * sigclip (exact products)
    const float sc_lo = f.sc_lo, sc_hi = f.sc_hi, ll_lo = f.ll_lo, ll_hi = f.ll_hi;

    // Over [y0-2, y0+TY+2) x [x0-2, x0+TX+2), in 2 x 5 cell tiles (one per thread and
    // pass).  Dense pass: the upper bound of S from a lower bound of med5(J) shared by the
    // tile's ten windows (dense_bounds); H' = the in-frame cells where that bound exceeds
    // sigclip (less a margin) holds H.
    constexpr int TTY = 2, TTX = 5, PW = TTX + 4;
    constexpr int NTY = L::NTY, NTX = L::NTX;
    const SEstParams sp = sest_params(f);
    int ncells = NTY * NTX;
    if constexpr (SPARSE)
        ncells = (int)s.ncells;
#pragma unroll 1
    for (int ti = tid; ti < ncells; ti += NT) {
        // column-major over the 2 x 5 tiles in groups of 16 row pairs, then the remaining
        // row pairs: a row pair's loads sit 2 * 73 = 18 banks (mod 32) after the previous
        // one's, so the 16 row pairs of a column tile take 16 distinct banks of one parity
        // and a half-wave's two column tiles (5 columns apart) the two parities; the
        // patch loads of a whole group are free of bank conflicts
        static_assert(SPARSE || 2 * L::JWP % 32 == 18,
                      "the bank spread assumes a J pitch of 9 mod 32");
        constexpr int NFULL = (NTY / 16) * 16;
        constexpr int NREM = NTY > NFULL ? NTY - NFULL : 1;     // (unused when 0)
        int tx, k;
        if constexpr (SPARSE) {
            k = s.cells[ti] >> 4;
            tx = s.cells[ti] & 15;
        } else if (ti < NFULL * NTX) {
            const int g = ti / (16 * NTX), e = ti - g * (16 * NTX);
            tx = e >> 4;
            k = 16 * g + (e & 15);
        } else {
            const int e = ti - NFULL * NTX;
            tx = e / NREM;
            k = NFULL + (e - tx * NREM);
        }
        const int r5 = min(k * TTY, L::SH - TTY);
        const int c5 = min(tx * TTX, L::SW - TTX);
        float v[(TTY + 4) * PW], u[TTY * TTX];
#pragma unroll
        for (int i = 0; i < TTY + 4; ++i)
#pragma unroll
            for (int j = 0; j < PW; ++j)
                v[i * PW + j] = sJ[(r5 + i) * L::JWP + c5 + j];
        const bool bound_ok = dense_bounds(v, sp, u);
        const int gx0 = x0 - 2 + c5;
        // in-frame columns of the tile's five, as a bit mask
        const uint32_t colmask = (gx0 >= 0 && gx0 + TTX <= W)
                                     ? (1u << TTX) - 1u
                                     : (((1u << TTX) - 1u) << max(-gx0, 0)) &
                                           ((1u << max(min(W - gx0, TTX), 0)) - 1u);
#pragma unroll
        for (int i = 0; i < TTY; ++i) {
            uint32_t bits = 0u;
#pragma unroll
            for (int j = 0; j < TTX; ++j)
                bits |= u[i * TTX + j] > sc_lo ? 1u << j : 0u;
            // where the analysis of the estimate does not hold at the bound, every cell
            bits = bound_ok ? bits : (1u << TTX) - 1u;
            const int gy = y0 - 2 + r5 + i;
            bits = (gy >= 0 && gy < H) ? bits & colmask : 0u;
            if (bits) {
                if (SPARSE)
                    s.any_hot = 1u;
                const int w = c5 >> 5, sh = c5 & 31;
                atomicOr(&sHot[(r5 + i) * L::HWP + w], bits << sh);
                if (sh > 32 - TTX && (bits >> (32 - sh)))
                    atomicOr(&sHot[(r5 + i) * L::HWP + w + 1], bits >> (32 - sh));
            }
        }
    }
    __syncthreads();
    if (SPARSE && !s.any_hot)
        return;           // S <= sigclip at every pixel that matters: no code bit is set
    // The later stages read S (to within the block's largest error bound) and med5(J)
    // only within 4 cells of H': the work set lies within 2 of H', and med5(S) at a work
    // pixel reads 2 further (a clamped neighbour's cell is no farther).  That region, in
    // 2 x 2 cell quads (row pair p, even column c: one 32-column word per lane), is
    // listed by the first waves and the quads take the exact med5 network in list order.
    constexpr int NP = L::NP;
    constexpr int kQuadWords = NP * L::HW;
    constexpr int kQuadWaves = (kQuadWords + 63) / 64;
    static_assert(kQuadWaves <= L::NW, "the quad bitmap words fit the block's waves");
    if (tid < 64 * kQuadWaves) {
        uint32_t m = 0u;
        const int pr = tid / L::HW, w = tid - pr * L::HW;
        if (tid < kQuadWords) {
            uint32_t a = 0u, b = 0u, c = 0u;        // words w - 1, w, w + 1 of the rows
            const uint32_t *row = &sHot[(2 * pr - 4) * L::HWP + w];
#pragma unroll
            for (int kk = 0; kk < 10; ++kk) {
                a |= row[kk * L::HWP - 1];
                b |= row[kk * L::HWP];
                c |= row[kk * L::HWP + 1];
            }
            // column 32w + k is needed when a bit lies in columns 32w + k - 4 .. + 4
            const unsigned long long hi = ((unsigned long long)c << 32) | b;
            const unsigned long long lo = ((unsigned long long)b << 32) | a;
#pragma unroll
            for (int d = 0; d <= 4; ++d)
                m |= (uint32_t)(hi >> d);
#pragma unroll
            for (int d = 1; d <= 4; ++d)
                m |= (uint32_t)(lo >> (32 - d));
            const int valid = L::SW - 32 * w;
            if (valid < 32)
                m &= (1u << valid) - 1u;
            // SPARSE: only cells that a re-evaluated pixel reads
            if constexpr (SPARSE)
                m &= s.reach[2 * pr * L::HW + w] | s.reach[(2 * pr + 1) * L::HW + w];
            // quads by their even column
            m = (m | (m >> 1)) & 0x55555555u;
        }
        list_append(m, pr * L::SW + 32 * w, s.quads, &s.need, (unsigned int)L::kQuads, lane);
    }
    __syncthreads();
    // Exact pass: med5(J), L+ and the S estimate with its error bound; the block's largest
    // bound is taken over these cells, the only ones read, and H' drops the cells where
    // the estimate at med5(J) settles S <= sigclip (so H' is {s + err > sigclip less the
    // margin} on the in-frame cells, as with the estimate everywhere).
    const int nquads = (int)s.need;
    if (!nquads)
        return;           // S <= sigclip at every pixel that matters: no code bit is set
    {
        float emax = 0.0f;
        unsigned int ncells = 0u;
        const bool counting = (f.flags & kCountWork) != 0;
        // The cells (rr, cc) and (rr, cc + 1) of a quad row (cc even), given their
        // med5(J) and their 4-neighbours (u above, d below, l left of the first cell, r
        // right of the second): the S estimates, the block's error bound, and one H' word
        // and one low word updated per row.  A quad's two columns share their word of
        // each bitmap and lie both inside the tile's columns or both outside.
        auto exact_row = [&](int rr, int cc, float u0, float u1, float l, float c0, float c1,
                             float r, float d0, float d1, float m0, float m1) {
            const int cx = cc - 2, cy = rr - 2;
            const bool tile_row = cx >= 0 && cx < TX && cy >= 0 && cy < TY;
            float e0, e1;
            const float s0 = s_estimate(c0, u0, d0, l, c1, m0, sp, e0);
            const float s1 = s_estimate(c1, u1, d1, c0, r, m1, sp, e1);
            s.S[rr * L::SWP + cc] = s0;
            s.S[rr * L::SWP + cc + 1] = s1;
            emax = fmaxf(emax, fmaxf(e0, e1));
            // H' keeps the cells whose estimate at med5(J) may exceed sigclip
            const uint32_t drop = (!(s0 + e0 > sc_lo) ? 1u << (cc & 31) : 0u) |
                                  (!(s1 + e1 > sc_lo) ? 1u << ((cc + 1) & 31) : 0u);
            // S may exceed sigfrac * sigclip here (the cell's own bound)
            const uint32_t low = (s0 + e0 > ll_lo ? 1u << (cx & 31) : 0u) |
                                 (s1 + e1 > ll_lo ? 1u << ((cx + 1) & 31) : 0u);
            uint32_t *hw = &sHot[rr * L::HWP + (cc >> 5)];
            if (drop & *hw)
                atomicAnd(hw, ~drop);
            if (tile_row && low)
                atomicOr(&s.low[cy * L::QW + (cx >> 5)], low);
            if (counting)
                ncells += tile_row ? 2u : 0u;
        };
        // One cell alone, as above.
        auto exact_cell = [&](int rr, int cc, float u0, float l, float c0, float r, float d0,
                              float m0) {
            const int cx = cc - 2, cy = rr - 2;
            const bool tile_row = cx >= 0 && cx < TX && cy >= 0 && cy < TY;
            float e0;
            const float s0 = s_estimate(c0, u0, d0, l, r, m0, sp, e0);
            s.S[rr * L::SWP + cc] = s0;
            emax = fmaxf(emax, e0);
            uint32_t *hw = &sHot[rr * L::HWP + (cc >> 5)];
            const uint32_t bit = 1u << (cc & 31);
            if (!(s0 + e0 > sc_lo) && (bit & *hw))
                atomicAnd(hw, ~bit);
            if (tile_row && s0 + e0 > ll_lo)
                atomicOr(&s.low[cy * L::QW + (cx >> 5)], 1u << (cx & 31));
            if (counting)
                ncells += tile_row ? 1u : 0u;
        };
        // As few quads per lane as the block's lanes allow, since a wave with work in few lanes
        // takes as long as a full one.  Up to NT / 4 quads: four lanes per quad, a cell each (the
        // 1 x 1 network).  Up to NT / 2: two lanes per quad, a row each (the 1 x 2 network and
        // two estimates, about 60% of a quad's instructions).  Else one quad per lane (the 2 x 2
        // network).  (With one quad per lane down to 32 of them the listed iterations of a
        // crowded 4096 x 4096 field took 95 and 50 us against 89 and 46, the first of the mixed
        // batch 236 us against 215, and the first detection the same to 1%.)
        if (nquads <= NT / 4) {
            if (tid < 4 * nquads) {
                const int q = (int)s.quads[tid >> 2];
                const int pr = q / L::SW, cc = q - pr * L::SW + (tid & 1);
                const int rr = 2 * pr + (tid >> 1 & 1);
                float v[5 * 5], m5[1];
#pragma unroll
                for (int i = 0; i < 5; ++i)
#pragma unroll
                    for (int j = 0; j < 5; ++j)
                        v[i * 5 + j] = sJ[(rr + i) * L::JWP + cc + j];
                med5_t1x1(v, m5);
                exact_cell(rr, cc, v[7], v[11], v[12], v[13], v[17], m5[0]);
            }
        } else if (nquads <= NT / 2) {
            if (tid < 2 * nquads) {
                const int q = (int)s.quads[tid >> 1];
                const int pr = q / L::SW, cc = q - pr * L::SW, rr = 2 * pr + (tid & 1);
                float v[5 * 6];
#pragma unroll
                for (int i = 0; i < 5; ++i)
#pragma unroll
                    for (int j = 0; j < 6; ++j)
                        v[i * 6 + j] = sJ[(rr + i) * L::JWP + cc + j];
                float m5[2];
                med5_t1x2(v, m5);
                constexpr int P = 6, pc = 2 * P + 2;
                exact_row(rr, cc, v[pc - P], v[pc + 1 - P], v[pc - 1], v[pc], v[pc + 1],
                          v[pc + 2], v[pc + P], v[pc + 1 + P], m5[0], m5[1]);
            }
        } else {
#pragma unroll 1
            for (int qi = tid; qi < nquads; qi += NT) {
                const int q = (int)s.quads[qi];
                const int pr = q / L::SW, cc = q - pr * L::SW, r0 = 2 * pr;
                float v[6 * 6];
#pragma unroll
                for (int i = 0; i < 6; ++i)
#pragma unroll
                    for (int j = 0; j < 6; ++j)
                        v[i * 6 + j] = sJ[(r0 + i) * L::JWP + cc + j];
                float m5[4];
                med5_t2x2(v, m5);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    constexpr int P = 6;
                    const int pc = (i + 2) * P + 2;
                    exact_row(r0 + i, cc, v[pc - P], v[pc + 1 - P], v[pc - 1], v[pc],
                              v[pc + 1], v[pc + 2], v[pc + P], v[pc + 1 + P], m5[2 * i],
                              m5[2 * i + 1]);
                }
            }
        }
        // non-negative floats order as their bit patterns: the device library's
        // cross-lane (DPP) maximum, then one LDS atomic per wave
        emax = __uint_as_float(__ockl_wfred_max_u32(__float_as_uint(emax)));
        if (lane == 0)
            atomicMax(&s.err_bits, __float_as_uint(emax));
        if (counting) {
            ncells = __ockl_wfred_add_u32(ncells);
            if (lane == 0 && ncells)
                atomicAdd(&s.exact_cells, ncells);
        }
    }
    __syncthreads();

    // Region cells outside the image must hold the value of their clamped cell: the
    // windows of the work set read S at clamped neighbour positions, at most two rows and
    // columns past the frame's edges.
    if (y0 < 2 || x0 < 2 || y0 + TY + 2 > H || x0 + TX + 2 > W) {
        for (int i = tid; i < 4 * (L::SW + L::SH); i += NT) {
            // rows -2, -1, H, H + 1 of the frame, then its columns -2, -1, W, W + 1
            const bool row = i < 4 * L::SW;
            const int q = row ? i / L::SW : (i - 4 * L::SW) / L::SH;
            const int o = row ? i - q * L::SW : i - 4 * L::SW - q * L::SH;
            const int e = q < 2 ? q - 2 : (row ? H : W) + q - 2;
            const int r = row ? e - (y0 - 2) : o, c = row ? o : e - (x0 - 2);
            if (r >= 0 && r < L::SH && c >= 0 && c < L::SW)
                s.S[r * L::SWP + c] = s.S[(clampi(y0 - 2 + r, H) - (y0 - 2)) * L::SWP +
                                          (clampi(x0 - 2 + c, W) - (x0 - 2))];
        }
    }
    const float emax = __uint_as_float(s.err_bits);
    // no estimate of the block is usable: every work pixel is re-evaluated
    const bool all_exact = !(emax < INFINITY) || (f.flags & kExactDetect);
    // work set Q' on the tile's in-frame pixels, one 32-pixel word per lane of the first
    // waves, appended to a compact list of tile positions (in any order)
    constexpr int kWorkWaves = (L::kTileWords + 63) / 64;
    if (tid < 64 * kWorkWaves) {
        uint32_t q = 0u;
        if (tid < L::kTileWords) {
            const int r = tid / L::QW, w = tid - r * L::QW;
            unsigned long long x = 0ull;
#pragma unroll
            for (int dr = 0; dr < 5; ++dr) {
                const uint32_t *row = &sHot[(r + dr) * L::HWP + w];
                x |= (unsigned long long)row[0] | ((unsigned long long)row[1] << 32);
            }
            // bit b of the dilation covers region columns 32w+b .. 32w+b+4, centred on
            // the tile column 32w+b
            q = (uint32_t)(x | (x >> 1) | (x >> 2) | (x >> 3) | (x >> 4));
            const int vc = W - x0 - 32 * w;
            if (y0 + r >= H || vc <= 0)
                q = 0u;
            else if (vc < 32)
                q &= (1u << vc) - 1u;
            q &= s.low[tid];
            if constexpr (SPARSE)
                q &= s.act[tid];
            s.low[tid] = q;
            if (all_exact)
                s.u[tid] = q;
        }
        // word tid covers tile positions tid * 32 .. (r * TX + 32 w with two words a row)
        list_append(q, tid * 32, s.list, &s.qcount, (unsigned int)kListMax, lane);
    }
    __syncthreads();

    const int total = (int)s.qcount;
    // the work set, compacted: thread t takes the t-th, (t+NT)-th, ... pixel of Q' (of
    // the tile, tested against the Q' bitmap, when the list could not hold Q').
    // S' from the estimates lies within B of the binary64 S' (B covers twice the
    // block's largest error and, with 4u, the roundings of the differences)
    const bool listed_q = total <= kListMax;
    if (!all_exact) {
        const float b2 = 2.02f * emax;
        const float olim_lo = f.olim_lo, olim_hi = f.olim_hi;
        unsigned int ncontrast = 0u, nunc = 0u;
        for (int qi = tid; qi < (listed_q ? total : TY * TX); qi += NT) {
            const int pos = listed_q ? (int)s.list[qi] : qi;
            if (!listed_q && !((s.low[pos >> 5] >> (pos & 31)) & 1u))
                continue;
            const int r = pos / TX, c = pos - r * TX;
            float w[25], ms[1];
#pragma unroll
            for (int i = 0; i < 5; ++i)
#pragma unroll
                for (int j = 0; j < 5; ++j)
                    w[i * 5 + j] = s.S[(r + i) * L::SWP + c + j];
            med5_t1x1(w, ms);
            const float spr = w[12] - ms[0];
            const float B = fmaf(fabsf(spr), 0x1p-22f, b2);
            const float lo = spr - B, hi = spr + B;
            const bool h1 = lo > sc_hi, h0 = hi <= sc_lo, l1 = lo > ll_hi, l0 = hi <= ll_lo;
            bool unc = !((h1 || h0) && (l1 || l0));
            bool listed = false, first = false;
            if (!unc && h1) {
                // S'/F^ <= S'/0.01 <= objlim for the whole interval: the test fails
                if (hi * 100.0f <= olim_lo) {
                    ++ncontrast;
                } else if (!(lo * 100.0f > olim_hi)) {
                    unc = true;
                } else {
                    const unsigned int slot = atomicAdd(&s.con_count, 1u);
                    // N from the pixel's estimate (w[12], positive here) and its L+ sum
                    const float *pj = &sJ[(r + 4) * L::JWP + c + 4];
                    const float nz = noise_from_estimate(
                        lplus4(pj[0], pj[-L::JWP], pj[L::JWP], pj[-1], pj[1]), w[12]);
                    if (slot < (unsigned int)kConMax) {
                        s.con_info[slot] = (uint32_t)pos | (l1 ? 1u << 16 : 0u);
                        s.con_lo[slot] = lo;
                        s.con_hi[slot] = hi;
                        s.con_n[slot] = nz;
                        atomicOr(&s.con_map[pos >> 5], 1u << (pos & 31));
                        listed = true;
                    } else {
                        const int t = contrast_by_count_lane(sJ, L::JWP, y0, x0, H, W, r, c,
                                                             nz, lo, hi, f.inv_olim);
                        first = t > 0;
                        unc = t < 0;
                        ncontrast += unc ? 0u : 1u;
                    }
                }
            }
            if (unc) {
                atomicOr(&s.u[pos >> 5], 1u << (pos & 31));
                ++nunc;
            } else if (!listed) {
                set_code(s, pos, first, h1, l1);
            }
        }
        if (ncontrast && (f.flags & kCountWork))
            atomicAdd(&s.contrast, ncontrast);
        if (nunc)
            atomicAdd(&s.uncertain, nunc);
    } else if (tid == 0) {
        s.uncertain = (unsigned int)total;     // s.u holds Q'
    }
    __syncthreads();

    // contrast tests of the listed pixels (S' > sigclip certain)
    const int ncon = min((int)s.con_count, kConMax);
    if (ncon) {
        const float inv_olim = f.inv_olim;
        unsigned int ncontrast = 0u, nunc = 0u;
        auto result = [&](uint32_t info, int t) {
            const int pos = (int)(info & 0xFFFFu);
            if (t < 0)
                atomicOr(&s.u[pos >> 5], 1u << (pos & 31));
            else
                set_code(s, pos, t > 0, true, (info >> 16) != 0u);
            // (sums, not a branch: that became one counter chosen in scratch memory)
            nunc += t < 0 ? 1u : 0u;
            ncontrast += t < 0 ? 0u : 1u;
        };
        if (ncon <= kConWaves) {
            // a few: one wave per pixel, its lanes the 49 window cells
            for (int it = tid >> 6; it < ncon; it += L::NW) {
                const uint32_t info = s.con_info[it];
                const int pos = (int)(info & 0xFFFFu);
                const int r = pos / TX, c = pos - r * TX;
                const int t = contrast_by_count(sJ, L::JWP, y0, x0, H, W, r, c, s.con_n[it],
                                                s.con_lo[it], s.con_hi[it], inv_olim, lane);
                if (lane == 0)
                    result(info, t);
            }
        } else {
            // more: med3 once on the union of the windows (hits are runs of neighbours, whose
            // windows share most cells), then the counts by 8 lanes per pixel.  The plane
            // holds, at (r, c), med3 at tile position (r - 3, c - 3) clamped to the frame.
            // First the 4-cell runs of plane rows that some window meets, one row per lane.
            constexpr int MH = L::MH, MW = L::MW, kRuns = (MW + 3) / 4;
            unsigned int &nruns = s.qcount;
            if (tid == 0)
                nruns = 0u;          // (read by all before the barrier that precedes)
            __syncthreads();
            if (tid < (MH + 63) / 64 * 64) {
                const unsigned long long *map =
                    reinterpret_cast<const unsigned long long *>(s.con_map);
                unsigned long long x = 0ull;
#pragma unroll
                for (int d = 0; d < 7; ++d) {
                    const int q = tid - 6 + d;
                    x |= q >= 0 && q < TY && tid < MH ? map[q] : 0ull;
                }
                // a window of tile column c covers plane columns c .. c + 6
                uint32_t w[3] = {(uint32_t)x, (uint32_t)(x >> 32), 0u};
#pragma unroll
                for (int sh = 1; sh <= 3; ++sh) {
                    w[2] |= w[2] << sh | w[1] >> (32 - sh);
                    w[1] |= w[1] << sh | w[0] >> (32 - sh);
                    w[0] |= w[0] << sh;
                }
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    list_append((w[i] | w[i] >> 1 | w[i] >> 2 | w[i] >> 3) & 0x11111111u,
                                tid * 4 * kRuns + 32 * i, s.list, &nruns, (unsigned int)kListMax,
                                lane);
            }
            __syncthreads();
            const int nr = (int)nruns;
            const bool interior = y0 >= 3 && x0 >= 3 && y0 + TY + 3 <= H && x0 + TX + 3 <= W;
            for (int i = tid; i < (nr <= kListMax ? nr : MH * kRuns); i += NT) {
                const int pos = nr <= kListMax ? (int)s.list[i] : 4 * i;
                const int pr = pos / (4 * kRuns), pc = min(pos - pr * (4 * kRuns), MW - 4);
                float o[4];
                if (interior) {
                    float v[3][6];
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int j = 0; j < 6; ++j)
                            v[q][j] = sJ[(pr + q) * L::JWP + pc + j];
                    med3_run<4>(v[0], v[1], v[2], o);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        o[j] = med3_at(med3_cell(sJ, L::JWP, y0, x0, H, W, pr - 3, pc - 3 + j, 0,
                                                 0), L::JWP);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    s.S[pr * MW + pc + j] = o[j];
            }
            __syncthreads();
            const int sub = tid & 7;
            int off[7];
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                const int j = min(sub + 8 * i, 48);
                off[i] = j / 7 * MW + j % 7;
            }
            for (int b = (tid >> 6) * 8; b < ncon; b += NT / 8) {
                const int it = min(b + (lane >> 3), ncon - 1);
                const uint32_t info = s.con_info[it];
                const int pos = (int)(info & 0xFFFFu);
                const int r = pos / TX, c = pos - r * TX;
                const float *m = &s.S[r * MW + c];
                float t_sure, t_maybe;
                contrast_thresholds(m[3 * MW + 3], s.con_n[it], s.con_lo[it], s.con_hi[it],
                                    inv_olim, t_sure, t_maybe);
                int n = 0;               // certain values, and possible ones << 8
#pragma unroll
                for (int i = 0; i < 7; ++i) {
                    const float x = m[off[i]];
                    const bool in = i < 6 || sub == 0;
                    n += (in && x > t_sure ? 1 : 0) + (in && x >= t_maybe ? 256 : 0);
                }
                n += __shfl_xor(n, 1);
                n += __shfl_xor(n, 2);
                n += __shfl_xor(n, 4);
                if (sub == 0 && b + (lane >> 3) < ncon)
                    result(info, (n & 255) >= 25 ? 1 : ((n >> 8) < 25 ? 0 : -1));
            }
        }
        if (ncontrast && (f.flags & kCountWork))
            atomicAdd(&s.contrast, ncontrast);
        if (nunc)
            atomicAdd(&s.uncertain, nunc);
        __syncthreads();
    }

    // binary64 re-evaluation of the undecided pixels from J, kExactBatch per round: 25 threads
    // compute the S window of a pixel, then one wave per pixel its codes, a window cell of the
    // contrast test per lane.  (With that test in one lane, 49 windows and 98 divisions one
    // after another, a launch over few tiles waited for a tile with such a pixel: the first
    // iteration of an 800 x 800 frame took 27 us where it takes 22, of a 1033 x 2047 one 28
    // where it takes 19, the first detection of the mixed batch 1.25 ms where it takes 1.22.)
    const int nunc = (int)s.uncertain;
    if (nunc) {
        // the binary64 parameters (read here, on this rare path only)
        const double gain = f.gain, sky = f.sky, rn = f.readnoise;
        const double rn2 = rn * rn, sigclip = f.sigclip, objlim = f.objlim;
        const double lowlim = (double)f.sigfrac * (double)f.sigclip;
        uint32_t *const upre = reinterpret_cast<uint32_t *>(s.list);
        // medians and N of a round's pixels
        double *const sMed = sX + kExactBatch * 25, *const sN = sMed + kExactBatch;
        if (tid < 64)
            bitmap_prefix<L::kTileWords>(s.u, upre);
        __syncthreads();
        unsigned int ncontrast = 0u;
        for (int base = 0; base < nunc; base += kExactBatch) {
            const int slot = tid / 25, cell = tid - slot * 25;
            if (slot < kExactBatch && base + slot < nunc) {
                const int pos = bitmap_select<L::kTileWords>(s.u, upre, base + slot);
                const int r = pos / TX, c = pos - r * TX;
                const int i = cell / 5, j = cell - i * 5;
                // window cell in frame coordinates, clamped
                const int gy = clampi(y0 + r + i - 2, H), gx = clampi(x0 + c + j - 2, W);
                double N;
                sX[slot * 25 + cell] = s_exact(&sJ[(gy - y0 + 4) * L::JWP + gx - x0 + 4],
                                               L::JWP, gain, sky, rn2, N);
                if (cell == 12)
                    sN[slot] = N;
            }
            __syncthreads();
            // med5 of the window by ranks: the value with at most 12 smaller and at
            // least 13 not larger (equal values write the same median)
            if (slot < kExactBatch && base + slot < nunc) {
                const double v = sX[slot * 25 + cell];
                int lt = 0, le = 0;
#pragma unroll 5
                for (int q = 0; q < 25; ++q) {
                    const double u = sX[slot * 25 + q];
                    lt += u < v ? 1 : 0;
                    le += u <= v ? 1 : 0;
                }
                if (lt <= 12 && le >= 13)
                    sMed[slot] = v;
            }
            __syncthreads();
            const int n = min(kExactBatch, nunc - base);
            for (int it = __builtin_amdgcn_readfirstlane(tid >> 6); it < n; it += L::NW) {
                const int pos = bitmap_select<L::kTileWords>(s.u, upre, base + it);
                const int r = pos / TX, c = pos - r * TX;
                const double spr = sX[it * 25 + 12] - sMed[it];
                const bool hbit = spr > sigclip, lbit = spr > lowlim;
                bool first = false;
                if (hbit) {
                    first = contrast_exact(sJ, L::JWP, y0, x0, H, W, r, c, spr, sN[it], objlim,
                                           lane);
                    ncontrast += lane == 0 ? 1u : 0u;
                }
                if (lane == 0)
                    set_code(s, pos, first, hbit, lbit);
            }
            __syncthreads();
        }
        if (ncontrast && (f.flags & kCountWork))
            atomicAdd(&s.contrast, ncontrast);
        __syncthreads();
    }
    if ((f.flags & kCountWork) && tid == 0 && f.work) {
        if (total)
            atomicAdd(&f.work[0], (unsigned long long)total);
        if (s.contrast)
            atomicAdd(&f.work[1], (unsigned long long)s.contrast);
        if (nunc)
            atomicAdd(&f.work[2], (unsigned long long)nunc);
        if (s.exact_cells)
            atomicAdd(&f.work[3], (unsigned long long)s.exact_cells);
    }
}

}  // namespace crb
