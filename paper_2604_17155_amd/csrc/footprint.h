// The footprint of a splat record on the pixel grid, as binning, emission and
// the tile kernels' gathers see it.
#pragma once

#include "gsc_internal.h"

namespace gsc {

// Largest q at which a pixel can still pass both the footprint test
// (q <= cut2) and the alpha floor (o exp(-q/2) >= alpha_min), with a margin
// covering the FP32 evaluation in the blend; negative when nothing passes.
// (No contraction here and below: binning counts, lists and masks footprints in
// several kernels, which have to agree to the bit.)
__device__ inline float reach_q(float o, const BlendParams& bp) {
#pragma clang fp contract(off)
    if (!(o >= bp.alpha_min)) return -1.0f;
    const float qa = 2.0f * __logf(o * __builtin_amdgcn_rcpf(bp.alpha_min));
    const float q = fminf(bp.cut2, qa);
    return q * (1.0f + 1e-4f) + 1e-3f;
}

// The ellipse {q <= qmax} of a record, q = a (dx + b dy / a)^2 + cq dy^2 with
// (dx, dy) the offset from the projected centre; all of it in the record's own
// scale (-K times the conic and qmax), as the blend evaluates it.
//
// The determinant of a needle is a small difference of products (1e-5 of them at
// 200 pixels sigma): each product's rounding error is added back by an fma, and the
// coefficients are not rescaled first, so that the ellipse is the record's to a few
// ulp.  Rescaled, with plain products, the row reach of 15% of needles of 100 to 200
// pixels sigma, and 31% up to 400, fell short of the record's by up to 10 pixels.
struct Ellipse {
    float bia;  // b / a
    float qa;   // qmax / a, widened by 1e-4 in the half width it gives
    float ca;   // cq / a, likewise
    float ry;   // row reach: |dy| <= ry
    float dyl;  // row offset of the leftmost point (the rightmost lies at -dyl)
};
__device__ inline bool make_ellipse(float4 r1, float qmax, Ellipse& e) {
#pragma clang fp contract(off)
    const float a = -r1.x, b = -0.5f * r1.y, c = -r1.z, qm = qmax * (float)-kExp2Scale;
    const float bb = b * b;
    const float det = fmaf(a, c, -bb) - fmaf(b, b, -bb);
    if (!(a > 0.0f && det > 0.0f && qm > 0.0f)) return false;
    const float ia = __builtin_amdgcn_rcpf(a), cq = det * ia;
    e.bia = b * ia;
    e.qa = qm * ia * 1.0002f;
    e.ca = cq * ia * 1.0002f;
    e.ry = __builtin_amdgcn_sqrtf(qm * __builtin_amdgcn_rcpf(cq)) * 1.0001f + 0.01f;
    // dy = -sqrt(qmax / Sxx) Sxy with Sxx = c / det, Sxy = -b / det
    // (= sqrt(qmax / (c det)) b)
    e.dyl = __builtin_amdgcn_sqrtf(qm * __builtin_amdgcn_rcpf(c * det)) * b;
    return true;
}
// Left and right edge over the rows [sa, sb] (row offsets from the centre) of
// an ellipse centred at column c: the left edge is convex and the right edge
// concave in dy, so each extreme lies at the row of the ellipse's leftmost /
// rightmost point, clamped to the span.  Widened by 0.01 pixel and 1e-4
// relative, so that a walk over these extents is conservative with respect to
// the blend's FP32 test (and covers the ~1 ulp of the hardware square root,
// reciprocal and logarithm used here).
__device__ inline void ellipse_span(const Ellipse& e, float c, float sa, float sb, float& l, float& r) {
#pragma clang fp contract(off)
    const float dl = __builtin_amdgcn_fmed3f(e.dyl, sa, sb), dr = __builtin_amdgcn_fmed3f(-e.dyl, sa, sb);
    const float hl = __builtin_amdgcn_sqrtf(fmaxf(fmaf(-e.ca * dl, dl, e.qa), 0.0f));
    const float hr = __builtin_amdgcn_sqrtf(fmaxf(fmaf(-e.ca * dr, dr, e.qa), 0.0f));
    l = fmaf(-e.bia, dl, c - 0.01f) - hl;
    r = fmaf(-e.bia, dr, c + 0.01f) + hr;
}

// Pixel rows [y0, y1] and the ellipse of a record's footprint in an image of
// height H; false when no row is reached.
struct Footprint {
    Ellipse e;
    float u, ulo, v, vlo;  // the projected centre as hi / lo pairs
    int y0, y1;
};
__device__ inline bool make_footprint(float4 r0, float4 r1, float qmax, int H, Footprint& f) {
#pragma clang fp contract(off)
    if (!make_ellipse(r1, qmax, f.e)) return false;
    const float vc = r0.y - 0.5f + r0.w;  // row index whose centre is the mean
    const float fy0 = fmaxf(ceilf(vc - f.e.ry), 0.0f);
    const float fy1 = fminf(floorf(vc + f.e.ry), (float)(H - 1));
    if (!(fy0 <= fy1)) return false;
    f.u = r0.x;
    f.ulo = r0.z;
    f.v = r0.y;
    f.vlo = r0.w;
    f.y0 = (int)fy0;
    f.y1 = (int)fy1;
    return true;
}
// Pixel columns [xa, xb] of an image of width W whose centres the footprint
// reaches over the rows ya..yb; false when there are none.
__device__ inline bool footprint_cols(const Footprint& f, int ya, int yb, int W, int& xa, int& xb) {
#pragma clang fp contract(off)
    float l, r;
    const float cx = f.u - 0.5f + f.ulo;  // column index whose centre is the mean
    ellipse_span(f.e, cx, ((float)ya + 0.5f - f.v) - f.vlo, ((float)yb + 0.5f - f.v) - f.vlo, l, r);
    const float xf = fmaxf(ceilf(l), 0.0f), xl = fminf(floorf(r), (float)(W - 1));
    if (!(xf <= xl)) return false;
    xa = (int)xf;
    xb = (int)xl;
    return true;
}

// A group is 4 x 4 bins, 8 x 8 blocks of BIN / 2 pixels.
template <int BIN>
constexpr int group_shift() { return BIN == 16 ? 6 : 7; }

// Calls visit(group_row, gx0, gx1) for every group row with a group that the
// footprint reaches.
template <int BIN, typename Visit>
__device__ inline void footprint_groups(const Footprint& f, int W, Visit&& visit) {
    constexpr int kS = group_shift<BIN>();
    for (int gy = f.y0 >> kS; gy <= f.y1 >> kS; ++gy) {
        const int ya = max(f.y0, gy << kS), yb = min(f.y1, (gy << kS) + (1 << kS) - 1);
        int xa, xb;
        if (footprint_cols(f, ya, yb, W, xa, xb)) visit(gy, xa >> kS, xb >> kS);
    }
}

// The groups an item is listed in: their number, and in `rect` how to list
// them.  Footprints whose bounding box meets few groups or a single row or
// column of them (nearly all) are listed by the box, column | row << 9 |
// width << 18; others by the walk above, rect = kRectWalk.
constexpr uint32_t kRectWalk = 1u << 31;
template <int BIN>
__device__ inline uint32_t count_groups(const Footprint& f, int W, uint32_t& rect) {
    constexpr int kS = group_shift<BIN>();
    rect = 0u;
    int xa, xb;
    if (!footprint_cols(f, f.y0, f.y1, W, xa, xb)) return 0u;
    const uint32_t gx = (uint32_t)(xa >> kS), gy = (uint32_t)(f.y0 >> kS);
    const uint32_t w = (uint32_t)(xb >> kS) - gx + 1u, h = (uint32_t)(f.y1 >> kS) - gy + 1u;
    if (w * h <= 4u || w == 1u || h == 1u) {
        rect = gx | (gy << 9) | (w << 18);
        return w * h;
    }
    rect = kRectWalk;
    uint32_t n = 0;
    footprint_groups<BIN>(f, W, [&](int, int a, int b) { n += (uint32_t)(b - a + 1); });
    return n;
}

// The blocks of the group at pixel (X0, Y0) that the footprint reaches, as
// 4-bit masks of its bins: bin f = 4 * bin_row + bin_col has bits 4 (f & 7) ..
// + 3 of x (f < 8) or y.  `on`: this lane has a record.  The active lanes step
// through block rows together, each through its own footprint's, so a wave
// takes as many steps as its tallest footprint.
template <int BIN>
__device__ inline uint2 group_masks(bool on, const Footprint& f, int X0, int Y0, int W) {
#pragma clang fp contract(off)
    constexpr int kSub = BIN / 2, kS = BIN == 16 ? 3 : 4;
    const int ya0 = max(f.y0 - Y0, 0), yb0 = min(f.y1 - Y0, 8 * kSub - 1);  // rows within the group
    int s = ya0 >> kS;
    const int s1 = on ? yb0 >> kS : -1;
    // offsets of the first and last row, and of row 0 of the current block row
    const float dy0 = ((float)Y0 + 0.5f - f.v) - f.vlo;
    const float da = dy0 + (float)ya0, db = dy0 + (float)yb0;
    float d = dy0 + (float)(s << kS);
    const float cx = (f.u - (float)X0) - 0.5f + f.ulo;  // columns within the group
    const float xmax = (float)min(8 * kSub - 1, W - 1 - X0);
    uint32_t sh = 8u * (uint32_t)s;
    uint64_t m = 0;  // bit 8 * block_row + block_col
    while (__builtin_amdgcn_ballot_w64(s <= s1) != 0) {  // uniform
        float l, r;
        ellipse_span(f.e, cx, fmaxf(d, da), fminf(d + (float)(kSub - 1), db), l, r);
        const int lo = (int)fmaxf(ceilf(l), 0.0f) >> kS, hi = (int)fminf(floorf(r), xmax) >> kS;
        // block columns lo..hi (hi < lo: none)
        const uint32_t n = s <= s1 ? (uint32_t)max(hi - lo + 1, 0) : 0u;
        const uint32_t byte = ((1u << (n & 31u)) - 1u) << (lo & 31);
        m |= (uint64_t)byte << (sh & 63u);
        ++s;
        sh += 8u;
        d += (float)kSub;
    }
    // two bits per bin to the low (even rows) or high half of its nibble
    uint32_t o[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t x = h ? (uint32_t)(m >> 32) : (uint32_t)m;
        uint32_t even = x & 0x00FF00FFu, odd = (x >> 8) & 0x00FF00FFu;
        even = (even | (even << 4)) & 0x0F0F0F0Fu;
        odd = (odd | (odd << 4)) & 0x0F0F0F0Fu;
        even = (even | (even << 2)) & 0x33333333u;
        odd = (odd | (odd << 2)) & 0x33333333u;
        o[h] = even | (odd << 2);
    }
    return make_uint2(o[0], o[1]);
}
// Bit 4 (f & 7) of x or y: bin f is reached.
__device__ __forceinline__ uint2 reached_bins(uint2 m) {
    uint32_t x = m.x | (m.x >> 1), y = m.y | (m.y >> 1);
    x = (x | (x >> 2)) & 0x11111111u;
    y = (y | (y >> 2)) & 0x11111111u;
    return make_uint2(x, y);
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
        float l, r;  // about the tile centre
        ellipse_span(e, -off.x, ca, cb, l, r);
        const bool in = ca <= cb;
        m |= (in && l <= -0.5f && r >= -7.5f) ? (1u << (2 * h)) : 0u;
        m |= (in && l <= 7.5f && r >= 0.5f) ? (2u << (2 * h)) : 0u;
    }
    return m;
}

}  // namespace gsc
