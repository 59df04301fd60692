// Projection, binning and tile ranges (per view x Gaussian).
//
// Gaussian geometry follows the 3DGS renderer the paper builds on (Sec. 3,
// "Differentiable renderer"): Sigma = R(q) diag(s^2) R(q)^T, EWA projection
// Sigma_2D = J W Sigma W^T J^T + dilation*I, a 3-sigma footprint, and the
// front-to-back order of eq. 2 keyed on the camera-space depth of the mean.
#include <algorithm>

#include "footprint.h"
#include "gsc_internal.h"

namespace gsc {

// a1: 3D covariance Sigma = R(q) diag(s^2) R(q)^T, evaluated in FP64 (a few
// dozen operations per Gaussian): the projection that consumes it is FP64,
// and a binary32 covariance would be the largest error in the blend's
// footprint and alpha decisions (a thin Gaussian's rounded rotation moves q by
// up to ~1e-5 relative at its 3-sigma edge).  Record layout: float4 (mean,
// opacity), then the six terms xx xy xz yy yz zz as doubles (64 bytes).
__global__ void k_cov3d(const float* __restrict__ means, const float* __restrict__ opac,
                        const float* __restrict__ scales, const float* __restrict__ quats,
                        float* __restrict__ geo, int64_t N) {
    int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= N) return;
    double w = quats[4 * g], x = quats[4 * g + 1], y = quats[4 * g + 2], z = quats[4 * g + 3];
    const double inv = 1.0 / sqrt(w * w + x * x + y * y + z * z);
    w *= inv; x *= inv; y *= inv; z *= inv;
    const double R[3][3] = {{1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y - w * z), 2.0 * (x * z + w * y)},
                            {2.0 * (x * y + w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z - w * x)},
                            {2.0 * (x * z - w * y), 2.0 * (y * z + w * x), 1.0 - 2.0 * (x * x + y * y)}};
    const double s0 = scales[3 * g], s1 = scales[3 * g + 1], s2 = scales[3 * g + 2];
    const double d[3] = {s0 * s0, s1 * s1, s2 * s2};
    double S[6];
    int k = 0;
    for (int i = 0; i < 3; ++i)
        for (int j = i; j < 3; ++j)
            S[k++] = R[i][0] * d[0] * R[j][0] + R[i][1] * d[1] * R[j][1] + R[i][2] * d[2] * R[j][2];
    float4* o = reinterpret_cast<float4*>(geo + kGeoStride * g);
    o[0] = make_float4(means[3 * g], means[3 * g + 1], means[3 * g + 2], opac[g]);
    double2* od = reinterpret_cast<double2*>(o + 1);
    od[0] = make_double2(S[0], S[1]);
    od[1] = make_double2(S[2], S[3]);
    od[2] = make_double2(S[4], S[5]);
}

void launch_cov3d(const float* means, const float* opac, const float* scales, const float* quats,
                  float* geo, int64_t N, hipStream_t s) {
    if (N <= 0) return;
    hipLaunchKernelGGL(k_cov3d, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, means, opac,
                       scales, quats, geo, N);
}

// Sums over the Gaussians of the mean axis scale and of the mean position
// (out: 4 doubles, zeroed by the caller), for the automatic bin size.
__global__ __launch_bounds__(256) void k_geometry_stats(const float* __restrict__ means,
                                                        const float* __restrict__ scales, int64_t N,
                                                        double* __restrict__ out) {
    __shared__ double part[4][4];
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < N;
         g += (int64_t)gridDim.x * blockDim.x) {
        acc[0] += (double)(scales[3 * g] + scales[3 * g + 1] + scales[3 * g + 2]) * (1.0 / 3.0);
        for (int k = 0; k < 3; ++k) acc[1 + k] += (double)means[3 * g + k];
    }
    for (int k = 0; k < 4; ++k)
        for (int d = 32; d >= 1; d >>= 1) acc[k] += __shfl_xor(acc[k], d, 64);
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < 4; ++k) part[threadIdx.x >> 6][k] = acc[k];
    __syncthreads();
    if (threadIdx.x < 4) {
        const int k = threadIdx.x;
        unsafeAtomicAdd(out + k, part[0][k] + part[1][k] + part[2][k] + part[3][k]);
    }
}

void launch_geometry_stats(const float* means, const float* scales, int64_t N, double* out,
                           hipStream_t s) {
    launch_fill_u32(reinterpret_cast<uint32_t*>(out), 0u, 8, s);
    if (N <= 0) return;
    const int64_t blocks = std::min<int64_t>((N + 255) / 256, 1024);
    hipLaunchKernelGGL(k_geometry_stats, dim3((unsigned)blocks), dim3(256), 0, s, means, scales, N, out);
}

// a2: projection of the items in depth order: thread k handles item
// order[k] (k itself when order is null) and writes its record and tile-pair
// count at position k, so that binning reads them contiguously; the random
// reads go to the per-Gaussian geometry, which caches across views.
// The projection is evaluated in FP64 (a few dozen operations per item) and
// the pixel position is stored as an FP32 hi/lo pair, so that the blend can
// form pixel offsets d = (p - u_hi) - u_lo exactly to one FP32 ulp of d; a
// single FP32 coordinate of a 512-pixel image is only good to ~3e-5 pixel,
// enough to move alpha by ~1e-4 relative at the footprint edge.
template <int BIN>
__global__ __launch_bounds__(256) void k_project(const ViewInfo* __restrict__ views, int n_views,
                                                 uint32_t n_items, const uint32_t* __restrict__ order,
                                                 const float* __restrict__ geo,
                                                 BlendParams bp, uint32_t* __restrict__ counts,
                                                 uint32_t* __restrict__ rects, float4* __restrict__ rec) {
    __shared__ uint32_t sbase[kViewLds];
    const bool vlds = stage_view_bases(views, n_views, sbase);
    const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n_items) return;
    // (the order is view by view: place k belongs to the view of item k)
    const uint32_t i = order ? order[k] : k;
    const ViewInfo& V = views[view_of(views, n_views, sbase, vlds, k)];
    const int64_t g = V.g_offset + (int64_t)(i - V.item_base);
    // one 64-byte record per Gaussian: a single cache line per random gather
    const float4* gr = reinterpret_cast<const float4*>(geo + kGeoStride * g);
    const double2* gd = reinterpret_cast<const double2*>(gr + 1);
    const float4 ga = gr[0];
    const double2 s01 = gd[0], s23 = gd[1], s45 = gd[2];  // xx xy | xz yy | yz zz
    float mx = ga.x, my = ga.y, mz = ga.z;
    float key = __fmaf_rn(V.R[6], mx, __fmaf_rn(V.R[7], my, __fmaf_rn(V.R[8], mz, V.t[2])));
    uint32_t cnt = 0, rect = 0;
    float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0;
    const float og = ga.w;
    const float qmax = reach_q(og, bp);
    if (key > bp.znear && qmax > 0.0f) {
        double R[9];
        for (int k = 0; k < 9; ++k) R[k] = V.R[k];
        const double dmx = mx, dmy = my, dmz = mz;
        const double tx = R[0] * dmx + R[1] * dmy + R[2] * dmz + (double)V.t[0];
        const double ty = R[3] * dmx + R[4] * dmy + R[5] * dmz + (double)V.t[1];
        const double tz = R[6] * dmx + R[7] * dmy + R[8] * dmz + (double)V.t[2];
        const double iz = 1.0 / tz;
        const double fx = V.fx, fy = V.fy;
        const double j00 = fx * iz, j02 = -fx * tx * iz * iz;
        const double j11 = fy * iz, j12 = -fy * ty * iz * iz;
        const double S[3][3] = {{s01.x, s01.y, s23.x}, {s01.y, s23.y, s45.x}, {s23.x, s45.x, s45.y}};
        // Sc = W S W^T
        double M[3][3];
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b)
                M[a][b] = R[3 * a] * S[0][b] + R[3 * a + 1] * S[1][b] + R[3 * a + 2] * S[2][b];
        double Sc[3][3];
        for (int a = 0; a < 3; ++a)
            for (int b = a; b < 3; ++b)
                Sc[a][b] = M[a][0] * R[3 * b] + M[a][1] * R[3 * b + 1] + M[a][2] * R[3 * b + 2];
        const double dil = bp.dilation;
        const double sxx = j00 * j00 * Sc[0][0] + 2.0 * j00 * j02 * Sc[0][2] + j02 * j02 * Sc[2][2] + dil;
        const double sxy = j00 * j11 * Sc[0][1] + j00 * j12 * Sc[0][2] + j02 * j11 * Sc[1][2] + j02 * j12 * Sc[2][2];
        const double syy = j11 * j11 * Sc[1][1] + 2.0 * j11 * j12 * Sc[1][2] + j12 * j12 * Sc[2][2] + dil;
        const double det = sxx * syy - sxy * sxy;
        const double u = fx * tx * iz + (double)V.cx;
        const double vv = fy * ty * iz + (double)V.cy;
        if (det > 0.0 && isfinite(u) && isfinite(vv)) {
            const double inv = 1.0 / det;
            const float uh = (float)u, vh = (float)vv;
            r0 = make_float4(uh, vh, (float)(u - (double)uh), (float)(vv - (double)vh));
            r1 = make_float4((float)(kExp2Scale * syy * inv), (float)(-2.0 * kExp2Scale * sxy * inv),
                             (float)(kExp2Scale * sxx * inv), og);
            Footprint f;
            if (make_footprint(r0, r1, qmax, V.height, f)) cnt = count_groups<BIN>(f, V.width, rect);
        }
    }
    counts[k] = cnt;
    // records are read only through tile pairs: an item with none keeps its
    // slot unwritten
    if (cnt != 0) {
        rects[k] = rect;
        rec[2 * (size_t)k] = r0;
        rec[2 * (size_t)k + 1] = r1;
    }
}

void launch_project(const ViewInfo* views, int n_views, uint32_t n_items, const uint32_t* order,
                    const float* geo, BlendParams bp, uint32_t* counts, uint32_t* rects, float4* rec,
                    int bin, hipStream_t s) {
    if (n_items == 0 || n_views <= 0) return;
    if (bin == 32)
        hipLaunchKernelGGL(k_project<32>, dim3((n_items + 255) / 256), dim3(256), 0, s, views, n_views,
                           n_items, order, geo, bp, counts, rects, rec);
    else
        hipLaunchKernelGGL(k_project<16>, dim3((n_items + 255) / 256), dim3(256), 0, s, views, n_views,
                           n_items, order, geo, bp, counts, rects, rec);
}

// a3: lists.  Items are first listed by group (4x4 bins; one to four groups
// for nearly every item), in depth order; a stable sort by group id keeps that
// order, and each group's list is then spread over its 16 bins.  Against one
// (bin, rank) pair per bin reached, sorted: 21.6 M pairs become 7.6 M on the
// relighting workload (100k Gaussians, 50 views of 512x512), a bin's entries
// are written once (4 bytes) instead of emitted (8) and moved (16) per radix
// pass, and the footprint's blocks are found by waves whose lanes all have an
// entry of the same group instead of lanes that walk footprints of different
// sizes.  us a call, before -> after: that workload 1886 -> 1813, three scenes
// of 16 label channels in a plan 5247 -> 4766, 500k Gaussians x 100 views of
// 64 feature channels 24717 -> 23371.
constexpr uint32_t kEmitStage = 2048;  // pairs a block stages in LDS (16 KB: eight resident blocks per CU)

// (group, k) pairs in depth order, k being the depth rank.  The block's items
// are consecutive ranks, so their pairs form one contiguous range [base,
// end_all): when it fits, it is assembled in LDS and stored with full-width
// coalesced writes.
template <int BIN>
__global__ __launch_bounds__(256) void k_emit(const ViewInfo* __restrict__ views, int n_views,
                                              const uint32_t* __restrict__ offsets,
                                              const uint32_t* __restrict__ counts,
                                              const uint32_t* __restrict__ rects,
                                              const float4* __restrict__ rec, BlendParams bp,
                                              uint32_t n_items, uint32_t cap,
                                              uint32_t* __restrict__ overflow,
                                              uint32_t* __restrict__ pair_keys,
                                              uint32_t* __restrict__ pair_vals) {
    __shared__ uint32_t skey[kEmitStage];
    __shared__ uint32_t sval[kEmitStage];
    __shared__ uint32_t sbase[kViewLds];
    const bool vlds = stage_view_bases(views, n_views, sbase);
    const uint32_t k0 = blockIdx.x * blockDim.x;
    const uint32_t klast = min(k0 + blockDim.x, n_items) - 1;
    const uint32_t base = offsets[k0];
    const uint32_t end_all = offsets[klast] + counts[klast];
    // (offsets stay at 2^32 - 1 from there on, and an end past them wraps)
    const bool staged = end_all >= base && end_all - base <= kEmitStage;
    const uint32_t k = k0 + threadIdx.x;
    const uint32_t cnt = k < n_items ? counts[k] : 0u;
    if (cnt != 0) {
        const ViewInfo& V = views[view_of(views, n_views, sbase, vlds, k)];
        const uint32_t gbase = V.group_base, gx = (uint32_t)V.groups_x;
        const uint32_t rect = rects[k];
        uint32_t off = offsets[k];
        uint32_t end = off + cnt;
        if (end > cap || end < off) {  // capacity exceeded: keep what fits, report the rest
            if (overflow) atomicAdd(overflow, 1u);
            end = off < cap ? cap : off;
        }
        auto put = [&](uint32_t key, uint32_t val) {
            if (off >= end) return;
            if (staged) {
                skey[off - base] = key;
                sval[off - base] = val;
            } else {
                pair_keys[off] = key;
                pair_vals[off] = val;
            }
            ++off;
        };
        if (!(rect & kRectWalk)) {
            const uint32_t w = (rect >> 18) & 0x3FFu;
            uint32_t key = gbase + ((rect >> 9) & 0x1FFu) * gx + (rect & 0x1FFu);
            uint32_t c = 0;
            for (uint32_t i = 0; i < cnt; ++i) {
                put(key + c, k);
                if (++c == w) {
                    c = 0;
                    key += gx;
                }
            }
        } else {
            const float4 r0 = rec[2 * (size_t)k], r1 = rec[2 * (size_t)k + 1];
            Footprint f;
            if (make_footprint(r0, r1, reach_q(r1.w, bp), V.height, f))
                footprint_groups<BIN>(f, V.width, [&](int gy, int a, int b) {
                    for (int g = a; g <= b; ++g) put(gbase + (uint32_t)gy * gx + (uint32_t)g, k);
                });
            // The walk above and the one that counted are the same code on the
            // same record; should they ever disagree, unused slots hold void pairs
            // of the view's first group: every key names a group, and a void pair
            // reaches none of its bins.
            while (off < end) put(gbase, k | kVoidPair);
        }
    }
    if (!staged) return;  // uniform over the block
    __syncthreads();
    const uint32_t n = min(end_all, max(cap, base)) - base;
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
        pair_keys[base + i] = skey[i];
        pair_vals[base + i] = sval[i];
    }
}

void launch_emit(const ViewInfo* views, int n_views, const uint32_t* offsets, const uint32_t* counts,
                 const uint32_t* rects, const float4* rec, BlendParams bp,
                 uint32_t n_items, uint32_t* pair_keys, uint32_t* pair_vals, int bin,
                 hipStream_t s, uint32_t cap, uint32_t* overflow) {
    if (n_items == 0) return;
    if (bin == 32)
        hipLaunchKernelGGL(k_emit<32>, dim3((n_items + 255) / 256), dim3(256), 0, s, views, n_views,
                           offsets, counts, rects, rec, bp, n_items, cap, overflow, pair_keys,
                           pair_vals);
    else
        hipLaunchKernelGGL(k_emit<16>, dim3((n_items + 255) / 256), dim3(256), 0, s, views, n_views,
                           offsets, counts, rects, rec, bp, n_items, cap, overflow, pair_keys,
                           pair_vals);
}

namespace {

// The view of a group.
__device__ inline int group_view(uint32_t g, const ViewInfo* __restrict__ views, int n_views) {
    int lo = 0, hi = n_views - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].group_base <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__device__ inline uint32_t live_pairs(const GroupLists& G) { return G.n_dev ? min(G.n_pairs, *G.n_dev) : G.n_pairs; }

}  // namespace

// Bound by instruction issue and by the random 32-byte record reads: 64 pairs
// take about 500 vector instructions, most of them in the block rows (45 each,
// as many as the wave's tallest footprint has).  7.6 M pairs of the relighting
// workload: 177 us (250 us with a division per ellipse term, separate edges
// per row and one part of a group's list per wave).
template <int BIN>
__global__ __launch_bounds__(256) void k_group_masks(GroupLists G, BlendParams bp) {
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t u = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    const uint32_t n = live_pairs(G), begin = u * G.window;
    if (begin >= n) return;  // whole wave
    const uint32_t end = min(begin + G.window, n);
    // (every pair's key names a group; a lane past the window's end has 0xFFFFFFFF)
    // the next 64 pairs' records are in flight while 64 are masked
    auto pair = [&](uint32_t b, uint32_t& key, uint32_t& k) {
        const bool in = b + lane < end;
        const uint32_t at = in ? b + lane : begin;
        key = G.keys[at];
        k = G.vals[at];
        key = in ? key : 0xFFFFFFFFu;
    };
    auto load = [&](uint32_t key, uint32_t k, float4& r0, float4& r1) {
        const size_t at = 2 * (size_t)(key < G.n_groups ? k & kItemMask : 0u);
        r0 = G.rec[at];
        r1 = G.rec[at + 1];
    };
    uint32_t key, k, keyn, kn;
    pair(begin, key, k);
    pair(begin + 64, keyn, kn);
    float4 r0, r1, q0, q1;
    load(key, k, r0, r1);
    uint32_t g = (uint32_t)__builtin_amdgcn_readfirstlane((int)key);  // the current group
    if (lane == 0) G.first_group[u] = g;
    uint32_t c[16];  // its entries per bin (uniform)
#pragma unroll
    for (int q = 0; q < 16; ++q) c[q] = 0u;
    int W = 1, H = 1, X0 = 0, Y0 = 0;
    uint32_t base = 0, gx = 1, next = 0;  // the current view's first group, columns; the next view's first group
    auto enter = [&]() {
        if (g >= G.n_groups) return;
        if (g >= next) {
            const int v = group_view(g, G.views, G.n_views);
            const ViewInfo& V = G.views[v];
            W = V.width;
            H = V.height;
            base = V.group_base;
            gx = (uint32_t)V.groups_x;
            next = v + 1 < G.n_views ? G.views[v + 1].group_base : G.n_groups;
        }
        const uint32_t local = g - base, row = local / gx;
        X0 = (int)((local - row * gx) << group_shift<BIN>());
        Y0 = (int)(row << group_shift<BIN>());
    };
    auto leave = [&]() {  // writes the group's row
        if (g >= G.n_groups) return;
        uint32_t cnt = c[0];
#pragma unroll
        for (int q = 1; q < 16; ++q) cnt = (lane & 15u) == (uint32_t)q ? c[q] : cnt;
        if (lane < 16) G.counts[((size_t)u + g) * 16 + lane] = cnt;
        uint32_t t = 0;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            t += c[q];
            c[q] = 0u;
        }
        if (lane == 0 && t != 0u) atomicAdd(G.totals + g, t);
    };
    enter();
    for (uint32_t b = begin; b < end; b += 64) {
        load(keyn, kn, q0, q1);
        uint32_t keynn, knn;
        pair(b + 128, keynn, knn);
        for (;;) {
            const bool mine = key == g;
            Footprint f{};
            const bool on = mine && g < G.n_groups && !(k & kVoidPair) && make_footprint(r0, r1, reach_q(r1.w, bp), H, f);
            const uint2 m = group_masks<BIN>(on, f, X0, Y0, W);
            if (mine) {
                G.mask_lo[b + lane] = m.x;
                G.mask_hi[b + lane] = m.y;
            }
            const uint2 t = reached_bins(m);
#pragma unroll
            for (int q = 0; q < 16; ++q)
                c[q] += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64((((q < 8 ? t.x : t.y) >> (4 * (q & 7))) & 1u) != 0u));
            // the next group among these 64 pairs, if any
            const uint64_t later = __builtin_amdgcn_ballot_w64(key > g && key < G.n_groups);
            if (later == 0) break;  // uniform
            leave();
            g = (uint32_t)__builtin_amdgcn_readlane((int)key, __builtin_ctzll(later));
            enter();
        }
        key = keyn;
        k = kn;
        keyn = keynn;
        kn = knn;
        r0 = q0;
        r1 = q1;
    }
    leave();
}

void launch_group_masks(const GroupLists& g, BlendParams bp, hipStream_t s) {
    if (g.n_groups == 0 || g.n_pairs == 0) return;
    const dim3 grid((unsigned)((group_windows(g.n_pairs, g.window) + 3) / 4)), block(256);
    if (g.bin == 32) hipLaunchKernelGGL(k_group_masks<32>, grid, block, 0, s, g, bp);
    else hipLaunchKernelGGL(k_group_masks<16>, grid, block, 0, s, g, bp);
}

// One block per group; thread 16 j + f takes bin f of the j-th sixteenth of its rows.
template <int BIN>
__global__ __launch_bounds__(256) void k_bin_ranges(GroupLists G, const uint32_t* __restrict__ first,
                                                    uint2* __restrict__ ranges, uint32_t cap,
                                                    const uint32_t* __restrict__ total,
                                                    unsigned long long* __restrict__ sum) {
    __shared__ uint32_t part[16][17];
    const uint32_t g = blockIdx.x, f = threadIdx.x & 15u, j = threadIdx.x >> 4;
    if (g == 0 && threadIdx.x == 0 && sum) atomicAdd(sum, (unsigned long long)*total);
    const uint2 rg = G.ranges[g];
    const uint32_t u0 = rg.x / G.window, rows = rg.x < rg.y ? (rg.y - 1) / G.window - u0 + 1 : 0u;
    uint32_t* cnt = G.counts + ((size_t)u0 + g) * 16 + f;
    // thread j takes `per` consecutive rows
    const uint32_t per = (rows + 15u) / 16u, p0 = min(j * per, rows), p1 = min(p0 + per, rows);
    uint32_t mine = 0;
#pragma unroll 8
    for (uint32_t p = p0; p < p1; ++p) mine += cnt[(size_t)p * 16];
    part[j][f] = mine;
    __syncthreads();
    uint32_t tot = 0, before = 0;
#pragma unroll
    for (uint32_t q = 0; q < 16; ++q) {
        const uint32_t c = part[q][f];
        before += q < j ? c : 0u;
        tot += c;
    }
    uint32_t inc = tot;  // inclusive scan over the sixteen bins
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) {
        const uint32_t o = (uint32_t)__shfl_up((int)inc, d, 16);
        if ((int)f >= d) inc += o;
    }
    const uint32_t start = first[g] + inc - tot;
    uint32_t run = start + before;
#pragma unroll 8
    for (uint32_t p = p0; p < p1; ++p) {
        const uint32_t c = cnt[(size_t)p * 16];
        cnt[(size_t)p * 16] = run;
        run += c;
    }
    if (j != 0) return;
    if (f == 0 && rows != 0u) G.ranges[g].x = rg.y < live_pairs(G) ? G.keys[rg.y] : G.n_groups;
    const ViewInfo& V = G.views[group_view(g, G.views, G.n_views)];
    const uint32_t local = g - V.group_base, row = local / (uint32_t)V.groups_x;
    const uint32_t bx = 4 * (local - row * (uint32_t)V.groups_x) + (f & 3u), by = 4 * row + (f >> 2);
    if (bx < (uint32_t)V.tiles_x && by < (uint32_t)V.tiles_y)
        ranges[V.tile_base + by * (uint32_t)V.tiles_x + bx] = make_uint2(min(start, cap), min(start + tot, cap));
}

void launch_bin_ranges(const GroupLists& g, const uint32_t* first, uint2* ranges, uint32_t cap,
                       const uint32_t* total, unsigned long long* sum, hipStream_t s) {
    if (g.n_groups == 0) return;
    const dim3 grid(g.n_groups), block(256);
    if (g.bin == 32) hipLaunchKernelGGL(k_bin_ranges<32>, grid, block, 0, s, g, first, ranges, cap, total, sum);
    else hipLaunchKernelGGL(k_bin_ranges<16>, grid, block, 0, s, g, first, ranges, cap, total, sum);
}

// One wave per window: each bin's entries of 64 pairs at once, by ballot, so
// the bin lists keep the group list's (depth) order.  The 64 pairs' entries
// (180 of 1024 on the relighting workload) are packed in LDS with their places
// and stored 64 at a time; stored bin by bin, with 16 partly filled store
// instructions per 64 pairs, the kernel was bound by store issue (124 -> 87 us
// there).
template <bool CAP>
__global__ __launch_bounds__(256) void k_bin_lists(GroupLists G, uint32_t* __restrict__ lists, uint32_t cap,
                                                   uint32_t* __restrict__ overflow) {
    __shared__ uint2 stage[4][1024];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t u = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + w));
    const uint32_t n = live_pairs(G), begin = u * G.window;
    if (begin >= n) return;  // whole wave (no block barrier below)
    const uint32_t end = min(begin + G.window, n);
    uint32_t g = (uint32_t)__builtin_amdgcn_readfirstlane((int)G.first_group[u]);
    uint32_t at = begin;
    // the group lists the window meets, one after the other.  (Each names the next:
    // stepping over the groups without pairs took a load apiece, one after the
    // other: two splats in opposite corners of 16384x16384 pixels, 6.2 -> 0.49 ms.)
    while (at < end && g < G.n_groups) {
        const uint2 rg = G.ranges[g];  // the next group with pairs, the end of this one's
        const uint32_t stop = min(end, (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y));
        uint32_t pos[16];
#pragma unroll
        for (int f = 0; f < 16; ++f) pos[f] = G.counts[((size_t)u + g) * 16 + f];
        for (uint32_t b = at; b < stop; b += 64) {
            const bool in = b + lane < stop;
            const uint32_t idx = in ? b + lane : at;
            const uint32_t k = G.vals[idx];
            uint2 m = make_uint2(G.mask_lo[idx], G.mask_hi[idx]);
            m = in ? m : make_uint2(0u, 0u);
            uint32_t fill = 0;  // entries staged (uniform)
#pragma unroll
            for (int f = 0; f < 16; ++f) {
                const uint32_t bm = ((f < 8 ? m.x : m.y) >> (4 * (f & 7))) & 15u;
                const uint64_t bal = __builtin_amdgcn_ballot_w64(bm != 0u);
                const uint32_t pre = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                               __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                if (bm != 0u) stage[w][fill + pre] = make_uint2(k | (bm << kItemBits), pos[f] + pre);
                const uint32_t c = (uint32_t)__popcll(bal);
                fill += c;
                pos[f] += c;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            uint32_t lost = 0;
            for (uint32_t i = lane; i < fill; i += 64) {
                const uint2 e = stage[w][i];
                if (!CAP || e.y < cap) lists[e.y] = e.x;
                else ++lost;
            }
            if constexpr (CAP) {
                if (lost != 0u && overflow) atomicAdd(overflow, lost);
            }
            __builtin_amdgcn_wave_barrier();  // the next 64 pairs overwrite the stage
        }
        at = max(at, stop);
        g = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
    }
}

void launch_bin_lists(const GroupLists& g, uint32_t* lists, uint32_t cap, uint32_t* overflow, hipStream_t s) {
    if (g.n_groups == 0 || g.n_pairs == 0) return;
    const dim3 grid((unsigned)((group_windows(g.n_pairs, g.window) + 3) / 4)), block(256);
    if (cap != 0xFFFFFFFFu) hipLaunchKernelGGL(k_bin_lists<true>, grid, block, 0, s, g, lists, cap, overflow);
    else hipLaunchKernelGGL(k_bin_lists<false>, grid, block, 0, s, g, lists, cap, overflow);
}

// Bins listed for every item (the sizes a plan fixes): the same groups and the
// same masks as above.
template <int BIN>
__global__ __launch_bounds__(256) void k_count_bins(const ViewInfo* __restrict__ views, int n_views,
                                                    uint32_t n_items, const uint32_t* __restrict__ counts,
                                                    const uint32_t* __restrict__ rects,
                                                    const float4* __restrict__ rec, BlendParams bp,
                                                    unsigned long long* __restrict__ out) {
    __shared__ unsigned long long part[4];
    unsigned long long acc = 0;
    constexpr int kS = group_shift<BIN>();
    for (uint32_t k0 = blockIdx.x * blockDim.x; k0 < n_items; k0 += gridDim.x * blockDim.x) {
        const uint32_t k = k0 + threadIdx.x;
        const uint32_t n = k < n_items ? counts[k] : 0u;
        if (n == 0u) continue;
        const ViewInfo& V = views[find_view_item(views, n_views, k)];
        const float4 r0 = rec[2 * (size_t)k], r1 = rec[2 * (size_t)k + 1];
        Footprint f{};
        const bool on = make_footprint(r0, r1, reach_q(r1.w, bp), V.height, f);
        auto add = [&](int gx, int gy) {
            const uint2 t = reached_bins(group_masks<BIN>(on, f, gx << kS, gy << kS, V.width));
            acc += (uint32_t)(__popc(t.x) + __popc(t.y));
        };
        const uint32_t rect = rects[k];
        if (!(rect & kRectWalk)) {
            const int w = (int)((rect >> 18) & 0x3FFu), gx = (int)(rect & 0x1FFu), gy = (int)((rect >> 9) & 0x1FFu);
            int c = 0, row = 0;
            for (uint32_t i = 0; i < n; ++i) {
                add(gx + c, gy + row);
                if (++c == w) {
                    c = 0;
                    ++row;
                }
            }
        } else {
            footprint_groups<BIN>(f, V.width, [&](int gy, int ga, int gb) {
                for (int gx = ga; gx <= gb; ++gx) add(gx, gy);
            });
        }
    }
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(out, part[0] + part[1] + part[2] + part[3]);
}

void launch_count_bins(const ViewInfo* views, int n_views, uint32_t n_items, const uint32_t* counts,
                       const uint32_t* rects, const float4* rec, BlendParams bp, int bin,
                       unsigned long long* out, hipStream_t s) {
    if (n_items == 0) return;
    const dim3 grid(std::min<uint32_t>((n_items + 255) / 256, 4096u)), block(256);
    if (bin == 32) hipLaunchKernelGGL(k_count_bins<32>, grid, block, 0, s, views, n_views, n_items, counts, rects, rec, bp, out);
    else hipLaunchKernelGGL(k_count_bins<16>, grid, block, 0, s, views, n_views, n_items, counts, rects, rec, bp, out);
}

// A modest grid (one 64-bit atomic per block on the same word) reading 16
// bytes per thread and step; counts is 16-byte aligned.
__global__ __launch_bounds__(256) void k_sum_u64(const uint32_t* __restrict__ counts, uint32_t n,
                                                unsigned long long* __restrict__ out) {
    __shared__ unsigned long long part[4];
    unsigned long long acc = 0;
    const uint4* c4 = reinterpret_cast<const uint4*>(counts);
    const uint32_t n4 = n / 4;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += gridDim.x * blockDim.x) {
        const uint4 v = c4[i];
        acc += (unsigned long long)v.x + v.y + v.z + v.w;
    }
    if (blockIdx.x == 0 && threadIdx.x < n - 4 * n4) acc += counts[4 * n4 + threadIdx.x];
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(out, part[0] + part[1] + part[2] + part[3]);
}

void launch_sum_u64(const uint32_t* counts, uint32_t n, unsigned long long* out, hipStream_t s) {
    if (n == 0) return;
    // about eight 16-byte loads per thread, at most 1024 atomics
    uint32_t blocks = (n / 4 + 2047) / 2048;
    blocks = blocks < 1 ? 1 : (blocks > 1024 ? 1024 : blocks);
    hipLaunchKernelGGL(k_sum_u64, dim3(blocks), dim3(256), 0, s, counts, n, out);
}

// Thread q owns keys 4q .. 4q + 3 (one 16-byte load where all four are
// live); neighbours across threads come from the adjacent lanes, with loads
// only at the wave's edges.
__global__ __launch_bounds__(256) void k_tile_ranges(const uint32_t* __restrict__ keys, uint32_t n,
                                                     const uint32_t* __restrict__ n_dev, uint32_t n_tiles,
                                                     uint2* __restrict__ ranges) {
    if (n_dev) n = min(n, *n_dev);
    const uint32_t q = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t lane = threadIdx.x & 63;
    const uint64_t k0 = 4ull * q;
    uint32_t t[4];
    if (k0 + 3 < n) {
        const uint4 v = reinterpret_cast<const uint4*>(keys)[q];
        t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = k0 + e < n ? keys[k0 + e] : 0xFFFFFFFFu;
    }
    uint32_t prev = (uint32_t)__shfl_up((int)t[3], 1, 64);
    uint32_t next = (uint32_t)__shfl_down((int)t[0], 1, 64);
    if (lane == 0) prev = (k0 > 0 && k0 - 1 < n) ? keys[k0 - 1] : 0xFFFFFFFFu;
    if (lane == 63) next = k0 + 4 < n ? keys[k0 + 4] : 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint64_t k = k0 + e;
        if (k >= n || t[e] >= n_tiles) continue;
        const uint32_t p = e == 0 ? prev : t[e > 0 ? e - 1 : 0];
        const uint32_t x = e == 3 ? next : t[e < 3 ? e + 1 : 3];
        if (k == 0 || p != t[e]) ranges[t[e]].x = (uint32_t)k;
        if (k + 1 == n || x != t[e]) ranges[t[e]].y = (uint32_t)(k + 1);
    }
}

void launch_tile_ranges(const uint32_t* sorted_keys, uint32_t n_pairs, uint32_t n_tiles,
                        uint2* ranges, hipStream_t s, const uint32_t* n_dev) {
    if (n_pairs == 0) return;
    const uint32_t quads = (uint32_t)(((uint64_t)n_pairs + 3) / 4);
    hipLaunchKernelGGL(k_tile_ranges, dim3((quads + 255) / 256), dim3(256), 0, s, sorted_keys,
                       n_pairs, n_dev, n_tiles, ranges);
}

}  // namespace gsc
