// Backward pass: hand-written adjoints of colorize and render with respect to
// the target pixels and the opacities.
//
// Colorize.  The coefficients solve (A_g + w_g Lambda) c_g = B_g (eq. 14), so
// for an upstream gradient dL/dc_g and Bbar_g = (A_g + w_g Lambda)^{-1} dL/dc_g
//   dL = sum_g <Bbar_g, dB_g - dA_g c_g - dw_g Lambda c_g>.
// B_g, A_g and w_g are sums over contributions of w*phi*y^T, w*phi*phi^T and w
// (eqs. 10-13), hence
//   dL/dy_p  = sum_g w_gp beta_gj            beta_gj  = Bbar_g^T phi_gj
//   dL/dw_gp = beta^T y_p - delta_gj        delta_gj = beta^T gamma + rho_g
// with gamma_gj = c_g^T phi_gj and rho_g = sum_{m,c} lambda_m Bbar[m][c] c[m][c].
// Render (eqs. 1-3).  images_p = sum_g w_gp gamma_gj, so for dL/dimages_p
//   dL/dc_g  = sum_{j,p} phi_gj w_gp (dL/dimages_p)^T
//   dL/dw_gp = gamma^T (dL/dimages_p)        (beta = gamma, delta = 0).
// Both then go through the adjoint of the front-to-back blend (eq. 2):
// w_k = alpha_k T_k with T_k = prod_{i<k} (1 - alpha_i) over accepted entries, so
//   dL/dalpha_k = u_k T_k - (1 - alpha_k)^{-1} sum_{i>k} u_i w_i,  u = dL/dw,
// and alpha = min(alpha_max, o G) gives dalpha/do = G unless clamped.  The
// skip, footprint and stop decisions are piecewise constant and carry no
// derivative.
//
// The weights are recomputed, never stored: one tile pass forms per pixel the
// total S = sum_k u_k w_k (and dL/dy), a second identical pass forms the
// running prefix P_k, so that the suffix sum is S - P_k.  S and P are kept in
// FP64, which keeps the suffix accurate deep into the pixel where it is many
// orders below S.
#include "gsc_internal.h"
#include "sh.h"
#include "wave_ops.h"

namespace gsc {

namespace {

// a / d for d in (0, 1]: the hardware reciprocal (1 ulp) and one correction by
// the residual.  The residual is exact or nearly so and the reciprocal's error
// enters squared, so the result is the rounded quotient but for ties within 2^-22
// ulp (of 24 M values with the reciprocal off by -1, 0 and 1 ulp, 3 differ; largest
// error 0.5000002 ulp).  The compiler's division takes twice the instructions and
// switches the denormal mode around them.
__device__ __forceinline__ float quotient(float a, float d) {
    const float r = __builtin_amdgcn_rcpf(d);
    const float q = a * r;
    return fmaf(fmaf(-d, q, a), r, q);
}

}  // namespace

// CC: channels of this launch (chunk [c_off, c_off + CC) of C).  dL/dw is
// linear in the channels, so chunk launches add their shares of dL/do, each with
// its channels' part of delta.
// The forms of up to three channels are held to seven waves per SIMD (72
// registers), as the forward accumulate (both adjoints 4.53 ms; six 4.58).  Of
// four channels six (five with dL/dy), of eight four (20 views of 800x800, 100k
// splats, eight channels and dL/dy, bins of 32: 1912 us at three, 1691 at four).
//
// A tile without entries reads no pixel values: of a few splats they were most of
// the traffic (10 splats, 20 views of 1024x1024, 16 channels, dL/do alone: 617 ->
// 70 us; 466 splats, 38 of 570x962, 3 channels with dL/dy: 306 -> 197).
//
// Bound by vector issue, as the forward walks: 300k Gaussians, 40 views of
// 800x800, degree 3, 3 channels: colorize 3.78 -> 2.32 ms, render 3.73 -> 2.20
// (before: a live flag per pixel carried through every step, the compiler's
// division, one wave reduction and one atomic per entry).
template <int CC, bool GY>
constexpr int adj_waves_per_simd() { return CC <= 3 ? 7 : (CC == 4 ? (GY ? 5 : 6) : (CC == 8 ? 4 : 1)); }

template <int CC, bool BF16, bool GY, int BIN>
__global__ __launch_bounds__(64 * kTileWaves) __attribute__((amdgpu_waves_per_eu(adj_waves_per_simd<CC, GY>()))) void k_blend_adjoint(
    const ViewInfo* __restrict__ views, int n_views, uint32_t n_wt, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ pair_vals,
    const float4* __restrict__ rec, const uint32_t* __restrict__ items, const void* __restrict__ ypix, int C, int c_off,
    const float* __restrict__ beta, BlendParams bp, float* __restrict__ grad_y,
    float* __restrict__ grad_o, const uint32_t* __restrict__ order) {
    // the chunk's records and, for up to three channels, the entry's adjoint
    // colours and offset, read back by every lane as broadcasts
    constexpr bool kLdsB = CC <= 3;
    constexpr int kGroup = 4;
    __shared__ float4 srec1[kTileWaves][64];
    __shared__ float4 sbet[kTileWaves][kLdsB ? 64 : 1];
    __shared__ float2 srec0[kTileWaves][64];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t wi = xcd_block<128 / kTileWaves>(blockIdx.x, gridDim.x) * kTileWaves + w;
    if (wi >= n_wt) return;  // whole wave
    const uint32_t wt = queued_tile<BIN>(wi, order);  // blocks start in index order
    const TileGeom tg = tile_geom<BIN>(wt, views, n_views);
    uint2 rg = ranges[tg.bin];
    rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
    rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
    // (the pixels of a tile without entries are not read)
    const bool grads = grad_o != nullptr && rg.x < rg.y;
    if (!GY && !grads) return;
    const ViewInfo& V = views[tg.vloc];
    const int stride = beta_stride(C, CC), part = C + c_off / CC;
    // dL/do of an entry goes to Gaussian g_offset + (item - item_base), the
    // item being named by the entry's record
    const int64_t g_shift = V.g_offset - (int64_t)V.item_base;
    // loop constants in vector registers (see uniform_in_vgpr)
    const float qlim = uniform_in_vgpr((float)(kExp2Scale * (double)bp.cut2));
    const float amax = uniform_in_vgpr(bp.alpha_max), amin = uniform_in_vgpr(bp.alpha_min),
                tmin = uniform_in_vgpr(bp.t_min);

    bool inside[4];
    float yv[4][CC];  // pixel values (read only when dL/do is wanted)
    // the lane's pixel offsets from the tile's centre point; R0 below keeps,
    // per entry, the offset of that point from the projected centre
    const float lx[2] = {tile_offset_col(lane, 0), tile_offset_col(lane, 1)};
    const float ly[2] = {tile_offset_row(lane, 0), tile_offset_row(lane, 1)};
    const float ox = tile_centre(tg.x0), oy = tile_centre(tg.y0);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int ix = tg.x0 + block_px(lane, k), iy = tg.y0 + block_py(lane, k);
        inside[k] = ix < V.width && iy < V.height;
        const int64_t row = V.pixel_offset + (int64_t)iy * V.width + ix;
#pragma unroll
        for (int c = 0; c < CC; ++c)
            yv[k][c] = (inside[k] && grads && c_off + c < C) ? load_target<BF16>(ypix, row * C + c_off + c) : 0.0f;
    }

    // Both passes walk the list the same way, so that they take the same
    // decisions.  A chunk of 64 entries is gathered at once, one entry per
    // lane (records and the entry's adjoint colours), and staged in LDS, from
    // which an entry reads them back with broadcast loads (adjoint colours of
    // wider chunks by readlane); each lane forms its entry's block mask, and
    // only entries reaching a block with a live pixel are visited, four at a
    // time: `body` gets each with its place in the group, `group` ends it.
    // Liveness is refreshed once a group: a pixel that stopped (T < t_min) adds
    // nothing in either pass, so the skipped entries and blocks change no sum.
    uint32_t alive0 = 0;  // blocks holding a pixel of the image
#pragma unroll
    for (int k = 0; k < 4; ++k) alive0 |= (__builtin_amdgcn_ballot_w64(inside[k]) != 0 ? 1u : 0u) << k;
    alive0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive0);
    float T[4];
    auto walk = [&](auto&& body, auto&& group) {
#pragma unroll
        for (int k = 0; k < 4; ++k) T[k] = inside[k] ? 1.0f : kOutsideT;
        uint32_t alive = alive0;
        for (uint32_t b = rg.x; b < rg.y && alive != 0u; b += 64) {
            const uint32_t nb = min(64u, rg.y - b);
            const uint32_t pv = lane < nb ? pair_vals[b + lane] : 0u;
            const bool own = lane < nb && pair_reaches<BIN>(pv, tg.quad, alive);
            const uint32_t it = pv & kItemMask;
            const float4 r = own ? rec[2 * (size_t)it] : make_float4(0.f, 0.f, 0.f, 0.f);
            const float2 R0 = make_float2((ox - r.x) - r.z, (oy - r.y) - r.w);
            const float4 R1 = own ? rec[2 * (size_t)it + 1] : make_float4(0.f, 0.f, 0.f, 0.f);
            const uint32_t gid = own ? items[it] : 0u;
            const float* bl = beta + (int64_t)gid * stride;
            float RB[CC];
#pragma unroll
            for (int c = 0; c < CC; ++c) RB[c] = (own && c_off + c < C) ? bl[c_off + c] : 0.0f;
            const float RD = own ? -bl[part] : 0.0f;
            const uint32_t BL = own ? (entry_blocks<BIN>(pv, R0, R1, bp) & alive) : 0u;
            uint64_t todo = __builtin_amdgcn_ballot_w64(BL != 0u);
            srec1[w][lane] = R1;
            srec0[w][lane] = R0;
            if constexpr (kLdsB)
                sbet[w][lane] = make_float4(RB[0], CC > 1 ? RB[CC > 1 ? 1 : 0] : 0.0f,
                                            CC > 2 ? RB[CC > 2 ? 2 : 0] : 0.0f, RD);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            while (todo != 0u && alive != 0u) {
#pragma unroll
                for (int e = 0; e < kGroup; ++e) {
                    const bool any = todo != 0u;
                    const uint32_t j = any ? (uint32_t)__builtin_ctzll(todo) : 0u;
                    todo &= todo - 1u;
                    const uint32_t item = bcast_u(gid, j);
                    const uint32_t blocks = any ? bcast_u(BL, j) & alive : 0u;
                    float bet[CC];
                    float del;  // - delta
                    if constexpr (!kLdsB) {
#pragma unroll
                        for (int c = 0; c < CC; ++c) bet[c] = bcast(RB[c], j);
                        del = bcast(RD, j);
                    }
                    auto visit = [&](auto&& step) {
                        if (blocks == 0u) return;  // uniform
                        const float2 c0 = srec0[w][j];
                        const float4 c1 = srec1[w][j];
                        if constexpr (kLdsB) {
                            const float4 b4 = sbet[w][kLdsB ? j : 0];
                            const float bb[3] = {b4.x, b4.y, b4.z};
#pragma unroll
                            for (int c = 0; c < CC; ++c) bet[c] = bb[c < 3 ? c : 0];
                            del = b4.w;
                        }
                        const float dx[2] = {c0.x + lx[0], c0.x + lx[1]}, dy[2] = {c0.y + ly[0], c0.y + ly[1]};
                        const float a0[2] = {c1.x * dx[0] * dx[0], c1.x * dx[1] * dx[1]};
                        const float b0[2] = {c1.y * dx[0], c1.y * dx[1]};
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            if (!((blocks >> k) & 1u)) continue;  // uniform
                            const float q2 = fmaf(dy[k >> 1], fmaf(c1.z, dy[k >> 1], b0[k & 1]), a0[k & 1]);
                            float u = del;
#pragma unroll
                            for (int c = 0; c < CC; ++c) u = fmaf(bet[c], yv[k][c], u);
                            step(k, q2, c1.w, u, bet);
                        }
                    };
                    body(e, item, visit);
                }
                group();
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (((alive >> k) & 1u) && __builtin_amdgcn_ballot_w64(T[k] >= tmin) == 0) alive &= ~(1u << k);
                alive = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive);
            }
            __builtin_amdgcn_wave_barrier();  // the next chunk overwrites the records
        }
    };

    // ---- pass 1: S = sum_k u_k w_k per pixel, and dL/dy -------------------
    double S[4];
    float gy[4][GY ? CC : 1];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        S[k] = 0.0;
#pragma unroll
        for (int c = 0; c < (GY ? CC : 1); ++c) gy[k][c] = 0.0f;
    }
    walk([&](int e, uint32_t item, auto&& visit) {
        visit([&](int k, float q2, float opac, float u, const float (&bet)[CC]) {
            uint64_t taken, kept;
            const float wt = pixel_step(q2, opac, T[k], qlim, amin, amax, tmin, taken, kept);
            S[k] += (double)(wt * u);
            if constexpr (GY) {
#pragma unroll
                for (int c = 0; c < CC; ++c) gy[k][c] = fmaf(wt, bet[c], gy[k][c]);
            }
        });
    }, [] {});
    if constexpr (GY) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (!inside[k]) continue;
            const int64_t row = V.pixel_offset + (int64_t)(tg.y0 + block_py(lane, k)) * V.width + tg.x0 + block_px(lane, k);
#pragma unroll
            for (int c = 0; c < CC; ++c)
                if (c_off + c < C) grad_y[row * C + c_off + c] = gy[k][c];
        }
    }
    if (!grads) return;

    // ---- pass 2: dL/dalpha per entry, reduced to dL/do per Gaussian -------
    // The step is pixel_step's, with the transmittance before the entry kept; a
    // group's four sums share one reduction and one atomic.
    double P[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) P[k] = 0.0;
    float go[kGroup];
    uint32_t who[kGroup], hit[kGroup];
    walk([&](int e, uint32_t item, auto&& visit) {
        float sum = 0.0f;
        uint64_t hits = 0;
        visit([&](int k, float q2, float opac, float u, const float (&bet)[CC]) {
            const float G = __builtin_amdgcn_exp2f(q2);
            const float al = __builtin_amdgcn_fmed3f(opac * G, 0.0f, amax);
            const bool inq = q2 >= qlim, ina = al >= amin;
            const float ae = (inq & ina) ? al : 0.0f;
            const float Tb = T[k], wt = Tb * ae;
            T[k] = fmaf(-Tb, ae, Tb);
            const bool keep = T[k] >= tmin;
            P[k] += (double)((keep ? wt : 0.0f) * u);
            const float suffix = (float)(S[k] - P[k]);
            const float dal = fmaf(u, Tb, -quotient(suffix, 1.0f - ae));
            const bool take = inq & ina & keep;
            hits |= __builtin_amdgcn_ballot_w64(inq) & __builtin_amdgcn_ballot_w64(ina) & __builtin_amdgcn_ballot_w64(keep);
            // (al is amax where the alpha is clamped: no derivative)
            sum += (take & !(al >= amax)) ? dal * G : 0.0f;
        });
        go[e] = sum;
        who[e] = item;
        hit[e] = hits != 0 ? 1u : 0u;
    }, [&] {
        if ((hit[0] | hit[1] | hit[2] | hit[3]) != 0u) {  // uniform
            const float t = wave_sum_transposed<kGroup>(go, lane);
            const int e = transposed_index<kGroup>(lane);
            uint32_t item = who[0], h = hit[0];
#pragma unroll
            for (int q = 1; q < kGroup; ++q) {
                item = e == q ? who[q] : item;
                h = e == q ? hit[q] : h;
            }
            if (lane < (uint32_t)kGroup && h != 0u) unsafeAtomicAdd(grad_o + ((int64_t)item + g_shift), t);
        }
    });
}

// Few tiles: one wave per 8x8 block (walk_block) for both passes; CC = 4 EX - 1
// channels per launch and delta as an entry's extra values.  Two passes of the
// same arithmetic as above.
template <int EX, bool BF16, bool GY, int BIN>
__global__ __launch_bounds__(256) void k_blend_adjoint_blocks(
    const ViewInfo* __restrict__ views, int n_views, uint32_t n_tiles, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ pair_vals, const float4* __restrict__ rec,
    const uint32_t* __restrict__ items, const void* __restrict__ ypix, int C, int c_off,
    const float* __restrict__ beta, BlendParams bp, float* __restrict__ grad_y, float* __restrict__ grad_o,
    const uint32_t* __restrict__ order) {
    constexpr int CC = 4 * EX - 1;
    __shared__ WalkLds<EX> lds[4];
    const uint32_t lane = threadIdx.x & 63, kq = threadIdx.x >> 6;
    const uint32_t wi = xcd_block(blockIdx.x, gridDim.x);
    if (wi >= n_tiles) return;
    const TileGeom tg = tile_geom<BIN>(queued_tile<BIN>(wi, order), views, n_views);
    uint2 rg = ranges[tg.bin];
    rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
    rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
    const bool grads = grad_o != nullptr && rg.x < rg.y;  // (as above)
    if (!GY && !grads) return;
    const ViewInfo& V = views[tg.vloc];
    const int ix = tg.x0 + block_px(lane, (int)kq), iy = tg.y0 + block_py(lane, (int)kq);
    const bool inside = (ix < V.width) & (iy < V.height);
    if (__builtin_amdgcn_ballot_w64(inside) == 0) return;  // whole wave
    const int64_t row = V.pixel_offset + (int64_t)iy * V.width + ix;
    const int stride = beta_stride(C, CC), part = C + c_off / CC;
    const int64_t g_shift = V.g_offset - (int64_t)V.item_base;
    float yv[CC];
#pragma unroll
    for (int c = 0; c < CC; ++c)
        yv[c] = (inside && grads && c_off + c < C) ? load_target<BF16>(ypix, row * C + c_off + c) : 0.0f;
    const float tmin = uniform_in_vgpr(bp.t_min), amax = uniform_in_vgpr(bp.alpha_max);
    // an entry's adjoint colours, then the launch's part of delta
    auto load_ex = [&](bool own, uint32_t item, float4 (&ex)[EX]) {
        const float* bl = beta + (int64_t)item * stride;
        float v[4 * EX];
#pragma unroll
        for (int c = 0; c < CC; ++c) v[c] = (own && c_off + c < C) ? bl[c_off + c] : 0.0f;
        v[CC] = own ? bl[part] : 0.0f;
#pragma unroll
        for (int x = 0; x < EX; ++x) ex[x] = make_float4(v[4 * x], v[4 * x + 1], v[4 * x + 2], v[4 * x + 3]);
    };
    auto values = [](const float4 (&ex)[EX], float (&v)[4 * EX]) {
#pragma unroll
        for (int x = 0; x < EX; ++x) {
            v[4 * x] = ex[x].x;
            v[4 * x + 1] = ex[x].y;
            v[4 * x + 2] = ex[x].z;
            v[4 * x + 3] = ex[x].w;
        }
    };
    // pass 1: S = sum_k u_k w_k per pixel, and dL/dy
    double S = 0.0;
    float gy[GY ? CC : 1];
#pragma unroll
    for (int c = 0; c < (GY ? CC : 1); ++c) gy[c] = 0.0f;
    float T = inside ? 1.0f : kOutsideT;
    walk_block<BIN, EX>(tg, kq, lane, rg, pair_vals, rec, items, bp, lds[kq], load_ex,
                        [&](const WalkGroup<EX>& g) -> bool {
        uint64_t kept = 0;
#pragma unroll
        for (int e = 0; e < kWalkEntries; ++e) {
            float v[4 * EX];
            values(g.ex[e], v);
            const float w = pixel_blend(g.ae[e], T, tmin, kept);
            float u = -v[CC];
#pragma unroll
            for (int c = 0; c < CC; ++c) u = fmaf(v[c], yv[c], u);
            S += (double)(w * u);
            if constexpr (GY) {
#pragma unroll
                for (int c = 0; c < CC; ++c) gy[c] = fmaf(w, v[c], gy[c]);
            }
        }
        return kept != 0;
    });
    if constexpr (GY) {
        if (inside) {
#pragma unroll
            for (int c = 0; c < CC; ++c)
                if (c_off + c < C) grad_y[row * C + c_off + c] = gy[c];
        }
    }
    if (!grads) return;
    // pass 2: dL/dalpha per entry, reduced to dL/do per Gaussian
    double P = 0.0;
    T = inside ? 1.0f : kOutsideT;
    walk_block<BIN, EX>(tg, kq, lane, rg, pair_vals, rec, items, bp, lds[kq], load_ex,
                        [&](const WalkGroup<EX>& g) -> bool {
        uint64_t kept = 0;
        float go[kWalkEntries];
        uint32_t any[kWalkEntries], hit = 0;
#pragma unroll
        for (int e = 0; e < kWalkEntries; ++e) {
            float v[4 * EX];
            values(g.ex[e], v);
            const float Tb = T;
            const float w = pixel_blend(g.ae[e], T, tmin, kept);
            float u = -v[CC];
#pragma unroll
            for (int c = 0; c < CC; ++c) u = fmaf(v[c], yv[c], u);
            P += (double)(w * u);
            const uint64_t taken = g.cand[e] & kept;
            const float G = __builtin_amdgcn_exp2f(g.q2[e]);
            const float suffix = (float)(S - P);
            const float dal = fmaf(u, Tb, -quotient(suffix, 1.0f - g.ae[e]));
            const bool use = ((taken >> lane) & 1u) != 0u && !(g.opac[e] * G >= amax);
            go[e] = use ? dal * G : 0.0f;
            any[e] = taken != 0 ? 1u : 0u;
            hit |= any[e];
        }
        if (hit != 0u) {  // uniform
            const float t = wave_sum_transposed<kWalkEntries>(go, lane);
            const int e = transposed_index<kWalkEntries>(lane);
            uint32_t item = g.item[0], h = any[0];
#pragma unroll
            for (int q = 1; q < kWalkEntries; ++q) {
                item = e == q ? g.item[q] : item;
                h = e == q ? any[q] : h;
            }
            if (lane < (uint32_t)kWalkEntries && h != 0u) unsafeAtomicAdd(grad_o + ((int64_t)item + g_shift), t);
        }
        return kept != 0;
    });
}

template <int EX, bool GY>
static void launch_badj_blocks(const TileLists& tl, const void* ypix, int ydtype, int C, const float* beta,
                               BlendParams bp, float* grad_y, float* grad_o, hipStream_t s) {
    const uint32_t n_wt = wave_tiles(tl.n_bins, tl.bin);
    const bool bf = ydtype == GSC_BF16;
#define GSC_BADJB(BFV, BINV)                                                                               \
    hipLaunchKernelGGL((k_blend_adjoint_blocks<EX, BFV, GY, BINV>), dim3(n_wt), dim3(256), 0, s, tl.views, \
                       tl.n_views, n_wt, tl.ranges, tl.pair_vals, tl.rec, tl.items, ypix, C, c_off, beta,  \
                       bp, grad_y, grad_o, tl.order)
    for (int c_off = 0; c_off < C; c_off += 4 * EX - 1) {
        if (tl.bin == 32) {
            if (bf) GSC_BADJB(true, 32); else GSC_BADJB(false, 32);
        } else {
            if (bf) GSC_BADJB(true, 16); else GSC_BADJB(false, 16);
        }
    }
#undef GSC_BADJB
}

template <int CC, bool GY>
static void launch_badj_cc(const TileLists& tl, const void* ypix, int ydtype, int C, const float* beta,
                           BlendParams bp, float* grad_y, float* grad_o, hipStream_t s) {
    const uint32_t n_wt = wave_tiles(tl.n_bins, tl.bin);
    dim3 grid((n_wt + kTileWaves - 1) / kTileWaves), block(64 * kTileWaves);
#define GSC_BADJ(BFV, BINV)                                                                          \
    hipLaunchKernelGGL((k_blend_adjoint<CC, BFV, GY, BINV>), grid, block, 0, s, tl.views, tl.n_views, \
                       n_wt, tl.ranges, tl.pair_vals, tl.rec, tl.items, ypix, C, c_off, beta, bp,     \
                       grad_y, grad_o, tl.order)
    for (int c_off = 0; c_off < C; c_off += CC) {
        const bool bf = ydtype == GSC_BF16;
        if (tl.bin == 32) {
            if (bf) GSC_BADJ(true, 32); else GSC_BADJ(false, 32);
        } else {
            if (bf) GSC_BADJ(true, 16); else GSC_BADJ(false, 16);
        }
    }
#undef GSC_BADJ
}

int adjoint_channels(const TileLists& tl, int C) {
    if (few_tiles(tl)) return C <= 3 ? 3 : (C <= 7 ? 7 : 15);
    return accumulate_chunk(C, GSC_F32);  // vector-lane channel chunks
}

template <bool GY>
static void launch_badj(const TileLists& tl, const void* ypix, int ydtype, int C, const float* beta,
                        BlendParams bp, float* grad_y, float* grad_o, hipStream_t s) {
    const int width = adjoint_channels(tl, C);
    if (few_tiles(tl)) {
        if (width == 3) launch_badj_blocks<1, GY>(tl, ypix, ydtype, C, beta, bp, grad_y, grad_o, s);
        else if (width == 7) launch_badj_blocks<2, GY>(tl, ypix, ydtype, C, beta, bp, grad_y, grad_o, s);
        else launch_badj_blocks<4, GY>(tl, ypix, ydtype, C, beta, bp, grad_y, grad_o, s);
        return;
    }
#define GSC_BA(CCV) launch_badj_cc<CCV, GY>(tl, ypix, ydtype, C, beta, bp, grad_y, grad_o, s)
    switch (width) {
        case 1: GSC_BA(1); break;
        case 2: GSC_BA(2); break;
        case 3: GSC_BA(3); break;
        case 4: GSC_BA(4); break;
        case 8: GSC_BA(8); break;
        default: GSC_BA(16); break;
    }
#undef GSC_BA
}

void launch_blend_adjoint(const TileLists& tl, const void* ypix, int ydtype, int C, const float* beta,
                          BlendParams bp, float* grad_y, float* grad_o, hipStream_t s) {
    if (tl.n_bins == 0 || (!grad_y && !grad_o)) return;
    if (grad_y)
        launch_badj<true>(tl, ypix, ydtype, C, beta, bp, grad_y, grad_o, s);
    else
        launch_badj<false>(tl, ypix, ydtype, C, beta, bp, grad_y, grad_o, s);
}

// grad_coeffs[g][m][c] = sum_j phi_gj[m] S_gj[c] from the per-view sums
// VS[j][g] = (V_gj, S_gj[0..C)) (per_view), or phi = Y0 and one summed slot
// per Gaussian (L = 0).  One thread per (Gaussian, CH channels); FP64 sums.
template <int L>
constexpr int fold_rhs_channels() { return L >= 3 ? 3 : 4; }

// Views are taken four at a time, their visibilities loaded together (one after
// the other, each view's loads waited for the last view's), and degree 3 takes
// three channels a thread (two read every slot twice at C = 3).  300k Gaussians,
// 40 views, degree 3: 197 -> 146 us.
template <int L>
__global__ __launch_bounds__(128) void k_fold_rhs(const ViewInfo* __restrict__ views, int n_views,
                           const float* __restrict__ means, const float* __restrict__ VS,
                           int per_view, int64_t N, int C, float* __restrict__ out) {
    constexpr int NB = (L + 1) * (L + 1);
    constexpr int CH = fold_rhs_channels<L>();
    constexpr int VB = 4;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int c0 = blockIdx.y * CH;
    if (g >= N) return;
    const int stride = C + 1;
    double acc[NB][CH];
#pragma unroll
    for (int m = 0; m < NB; ++m)
#pragma unroll
        for (int c = 0; c < CH; ++c) acc[m][c] = 0.0;
    const int nv = per_view ? n_views : 1;
    const float mx = means[3 * g], my = means[3 * g + 1], mz = means[3 * g + 2];
    for (int v0 = 0; v0 < nv; v0 += VB) {
        float x[VB][CH], w[VB];
#pragma unroll
        for (int u = 0; u < VB; ++u) {
            const int v = min(v0 + u, nv - 1);
            const float* slot = VS + ((per_view ? views[v].vs_base : 0) + g) * stride;
            w[u] = v0 + u < nv ? slot[0] : 0.0f;
#pragma unroll
            for (int c = 0; c < CH; ++c) x[u][c] = slot[1 + min(c0 + c, C - 1)];
        }
#pragma unroll
        for (int u = 0; u < VB; ++u) {
            if (w[u] == 0.0f) continue;  // no contribution in this view
            float phi[NB];
            if (per_view) {
                const ViewInfo& Vw = views[v0 + u];
                const float dx = mx - (float)Vw.centre[0], dy = my - (float)Vw.centre[1],
                            dz = mz - (float)Vw.centre[2];
                const float inv = rsqrtf(dx * dx + dy * dy + dz * dz);
                sh_eval<float, L>(dx * inv, dy * inv, dz * inv, phi);
            } else {
                sh_eval<float, L>(0.0f, 0.0f, 1.0f, phi);
            }
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const double sc = (double)x[u][c];
#pragma unroll
                for (int m = 0; m < NB; ++m) acc[m][c] = fma((double)phi[m], sc, acc[m][c]);
            }
        }
    }
#pragma unroll
    for (int m = 0; m < NB; ++m)
#pragma unroll
        for (int c = 0; c < CH; ++c)
            if (c0 + c < C) out[(g * NB + m) * C + c0 + c] = (float)acc[m][c];
}

template <int L>
static void launch_fold_rhs_l(const ViewInfo* views, int n_views, const float* means, const float* VS,
                              bool per_view, int64_t N, int C, float* out, hipStream_t s) {
    constexpr int CH = fold_rhs_channels<L>();
    dim3 grid((unsigned)((N + 127) / 128), (unsigned)((C + CH - 1) / CH)), block(128);
    hipLaunchKernelGGL(k_fold_rhs<L>, grid, block, 0, s, views, n_views, means, VS, (int)per_view, N, C, out);
}

void launch_fold_rhs(const ViewInfo* views, int n_views, const float* means, const float* VS,
                     bool per_view, int64_t N, int C, int sh_deg, float* out, hipStream_t s) {
    if (N <= 0) return;
    switch (sh_deg) {
        case 0: launch_fold_rhs_l<0>(views, n_views, means, VS, per_view, N, C, out, s); break;
        case 1: launch_fold_rhs_l<1>(views, n_views, means, VS, per_view, N, C, out, s); break;
        case 2: launch_fold_rhs_l<2>(views, n_views, means, VS, per_view, N, C, out, s); break;
        default: launch_fold_rhs_l<3>(views, n_views, means, VS, per_view, N, C, out, s); break;
    }
}

}  // namespace gsc
