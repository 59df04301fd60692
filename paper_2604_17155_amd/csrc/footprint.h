// The footprint of a splat record on the pixel grid, as binning, emission and
// the tile kernels' gathers see it.
#pragma once

#include "gsc_internal.h"

namespace gsc {

// Largest q at which a pixel can still pass both the footprint test
// (q <= cut2) and the alpha floor (o exp(-q/2) >= alpha_min), with a margin
// covering the FP32 evaluation in the blend; negative when nothing passes.
__device__ inline float reach_q(float o, const BlendParams& bp) {
    if (!(o >= bp.alpha_min)) return -1.0f;
    const float qa = 2.0f * __logf(o / bp.alpha_min);
    const float q = fminf(bp.cut2, qa);
    return q * (1.0f + 1e-4f) + 1e-3f;
}

// The ellipse {q <= qmax} of a record, q = a (dx + b dy / a)^2 + cq dy^2 with
// (dx, dy) the offset from the projected centre.
struct Ellipse {
    float ia, bia, cq, qmax;
    float ry;   // row reach: |dy| <= ry
    float dyl;  // row offset of the leftmost point (the rightmost lies at -dyl)
};
__device__ inline bool make_ellipse(float4 r1, float qmax, Ellipse& e) {
    constexpr float kInvK = (float)(1.0 / kExp2Scale);
    const float a = r1.x * kInvK, b = 0.5f * r1.y * kInvK, c = r1.z * kInvK;
    const float det = a * c - b * b;
    if (!(a > 0.0f && det > 0.0f && qmax > 0.0f)) return false;
    e.ia = 1.0f / a;
    e.bia = b * e.ia;
    e.cq = det * e.ia;
    e.qmax = qmax;
    e.ry = __builtin_amdgcn_sqrtf(qmax / e.cq) * 1.0001f + 0.01f;
    // dy = -sqrt(qmax / Sxx) Sxy with Sxx = c / det, Sxy = -b / det
    const float idet = 1.0f / det, sxx = c * idet;
    e.dyl = __builtin_amdgcn_sqrtf(qmax / sxx) * b * idet;
    return true;
}
// Offsets of the left and right edge over the rows [sa, sb] (row offsets from
// the centre): the left edge is convex and the right edge concave in dy, so
// each extreme lies at the row of the ellipse's leftmost / rightmost point,
// clamped to the span.  Widened by 0.01 pixel and 1e-4 relative, so that a
// walk over these extents is conservative with respect to the blend's FP32
// test (and covers the ~1 ulp of the hardware square root).
__device__ inline void ellipse_span(const Ellipse& e, float sa, float sb, float& l, float& r) {
    const float dl = __builtin_amdgcn_fmed3f(e.dyl, sa, sb), dr = __builtin_amdgcn_fmed3f(-e.dyl, sa, sb);
    const float hl = __builtin_amdgcn_sqrtf(fmaxf(e.qmax - e.cq * dl * dl, 0.0f) * e.ia) * 1.0001f + 0.01f;
    const float hr = __builtin_amdgcn_sqrtf(fmaxf(e.qmax - e.cq * dr * dr, 0.0f) * e.ia) * 1.0001f + 0.01f;
    l = -e.bia * dl - hl;
    r = -e.bia * dr + hr;
}

// Walks a record's footprint in rows of SUB x SUB pixel blocks and calls
// visit(block_row, lo, hi) for every block row with a block whose pixel
// centres come within the footprint: blocks lo..hi of that row.  Used
// identically for counting and emitting.
template <int SUB, typename Visit>
__device__ inline void footprint_rows(float4 r0, float4 r1, float qmax, int W, int H, Visit&& visit) {
    constexpr int kShift = SUB == 8 ? 3 : 4;
    static_assert(SUB == 8 || SUB == 16, "blocks of 8 or 16 pixels");
    Ellipse e;
    if (!make_ellipse(r1, qmax, e)) return;
    const float vc = r0.y - 0.5f + r0.w;  // row index whose centre is the mean
    const float fy0 = fmaxf(ceilf(vc - e.ry), 0.0f);
    const float fy1 = fminf(floorf(vc + e.ry), (float)(H - 1));
    if (!(fy0 <= fy1)) return;
    const int y0 = (int)fy0, y1 = (int)fy1;
    const float cx = r0.x - 0.5f + r0.z;  // column index whose centre is the mean
    for (int ya = y0; ya <= y1; ya = (ya | (SUB - 1)) + 1) {
        const int yb = min(ya | (SUB - 1), y1);
        float l, r;
        ellipse_span(e, ((float)ya + 0.5f - r0.y) - r0.w, ((float)yb + 0.5f - r0.y) - r0.w, l, r);
        const float xf = fmaxf(ceilf(cx + l), 0.0f);
        const float xl = fminf(floorf(cx + r), (float)(W - 1));
        if (xf <= xl) visit(ya >> kShift, (int)xf >> kShift, (int)xl >> kShift);
    }
}

// Footprint per bin row; a bin is 2 x 2 blocks of BIN / 2 pixels and the
// 4-bit mask's bit 2h + c marks the block in row half h and column half c.
// visit(bin_row, t0, t1, mask_of, n, h) is called per bin row with the bin
// columns [t0, t1], a function giving a bin column's mask (0: not reached),
// n, the number of columns in [t0, t1] whose mask is not 0, and h = the first
// and last block column reached in each row half (lo0, hi0, lo1, hi1; lo > hi:
// none).
template <int BIN, typename Visit>
__device__ inline void footprint_bins(float4 r0, float4 r1, float qmax, int W, int H, Visit&& visit) {
    static_assert(BIN == 16 || BIN == 32, "bins are 16 or 32 pixels");
    int cur = -1, lo[2] = {1 << 30, 1 << 30}, hi[2] = {-1, -1};
    auto flush = [&]() {
        if (cur < 0) return;
        // a bin column t has a block of row half h reached exactly when
        // lo[h] >> 1 <= t <= hi[h] >> 1 (block columns are >= 0; an unreached
        // half has lo > hi and gives an empty range), so the reached columns
        // are the union of two ranges
        const int a0 = lo[0] >> 1, a1 = hi[0] >> 1, c0 = lo[1] >> 1, c1 = hi[1] >> 1;
        const int na = max(a1 - a0 + 1, 0), nc = max(c1 - c0 + 1, 0);
        const int nboth = max(min(a1, c1) - max(a0, c0) + 1, 0);
        visit(cur, min(lo[0], lo[1]) >> 1, max(hi[0], hi[1]) >> 1, [&](int t) {
            uint32_t m = 0;
            for (int h = 0; h < 2; ++h)
                for (int c = 0; c < 2; ++c)
                    m |= (lo[h] <= 2 * t + c && 2 * t + c <= hi[h]) ? (1u << (2 * h + c)) : 0u;
            return m;
        }, na + nc - nboth, make_int4(lo[0], hi[0], lo[1], hi[1]));
    };
    footprint_rows<BIN / 2>(r0, r1, qmax, W, H, [&](int br, int l, int h) {
        if ((br >> 1) != cur) {
            flush();
            cur = br >> 1;
            lo[0] = lo[1] = 1 << 30;
            hi[0] = hi[1] = -1;
        }
        // (selects, so that the ranges stay in registers)
        lo[0] = (br & 1) ? lo[0] : l;
        hi[0] = (br & 1) ? hi[0] : h;
        lo[1] = (br & 1) ? l : lo[1];
        hi[1] = (br & 1) ? h : hi[1];
    });
    flush();
}

// The 8x8 pixel blocks (bit 2 * row half + column half) of a 16x16 tile that
// a record's footprint can reach; off = the tile centre's offset from the
// projected centre (the pixel centres of a half span [-7.5, -0.5] or
// [0.5, 7.5] about the tile centre).
__device__ inline uint32_t footprint_blocks(float2 off, float4 r1, float qmax) {
    Ellipse e;
    if (!make_ellipse(r1, qmax, e)) return 0u;
    uint32_t m = 0u;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const float sa = off.y + (h ? 0.5f : -7.5f), sb = sa + 7.0f;
        const float ca = fmaxf(sa, -e.ry), cb = fminf(sb, e.ry);
        float l, r;
        ellipse_span(e, ca, cb, l, r);
        const bool in = ca <= cb;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const float xa = off.x + (c ? 0.5f : -7.5f);
            m |= (in && l <= xa + 7.0f && r >= xa) ? (1u << (2 * h + c)) : 0u;
        }
    }
    return m;
}

}  // namespace gsc
