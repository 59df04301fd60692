// Render: per-item view colours from SH coefficients, then the same
// front-to-back tile blend as the accumulate pass, writing each pixel's
// blended colour (eq. 2 with the colours of eq. 3).
#include <algorithm>

#include "gsc_internal.h"
#include "sh.h"
#include "wave_ops.h"

namespace gsc {

// Per-item terms of the blends, from the SH coefficients (batch item i is view
// v's Gaussian g, items in their own order, phi = phi(dir_gv)):
//   kColours        out[i*C + c]       = sum_m c_g[m][c] phi_m
//   kRenderAdjoint  out[i*B + c]       the same, and 0 from C on (delta of a render)
//   kAdjoint        out[i*B + c]       = beta_c = sum_m Bbar_g[m][c] phi_m, and
//                   out[i*B + C + p]   = sum_c beta_c (c_g^T phi)_c over the p-th `width`
//                   channels, plus rho_g for p = 0 (B = beta_stride(C, width))
//
// Bound by the writes (12-16 bytes an item at C = 3) and the FP64 direction;
// the coefficients (108 bytes a Gaussian at L = 2, C = 3, twice that for
// kAdjoint) are an order more than the result if every item reads its own.  So
// a thread owns a Gaussian and takes its views kTermViews at a time: the
// block's coefficients go to LDS once, by coalesced loads of the caller's own
// layout, and one LDS read serves kTermViews items.  Where the coefficients of a
// block's threads' Gaussians do not fit, it takes fewer of them (down to four, 64
// channels at L = 3) and several threads each, which share the views: the staging
// stays one coalesced pass (a few channels at a time for each set of views, in
// 12-byte pieces of 124-byte rows: 94k Gaussians, 34 views, L = 3, kAdjoint, 31
// channels 8143 -> 810 us, 64 channels 17881 -> 1500; a thread an item 3222 and
// 7454).
// 300k Gaussians, 40 views, L = 3, C = 3: kColours 373 -> 117 us, kRenderAdjoint
// 384 -> 111, kAdjoint 749 -> 211, and two or four transposes of the
// coefficients (27-157 us) gone (before, a thread an item reading transposed
// coefficients).
enum TermMode { kColours, kRenderAdjoint, kAdjoint };
constexpr int kTermBlock = 128, kTermViews = 4;
constexpr int kTermLoads = 8;  // loads in flight a thread while staging
constexpr size_t kTermStage = 96 * (kTermBlock + 1);  // floats of LDS: three blocks a CU

// The coefficients of n Gaussians from g0 (`per` each, contiguous):
// dst[k * ld + t], the k-th of Gaussian g0 + t.
__device__ __forceinline__ void stage_terms(const float* __restrict__ src, int64_t g0, int n, int per, int ld,
                                            float* dst) {
    const int dq = kTermBlock / per, dr = kTermBlock - dq * per;
    int t = (int)threadIdx.x / per, k = (int)threadIdx.x - t * per;
    const float* from = src + g0 * per;
    const int total = n * per;
    for (int i0 = (int)threadIdx.x; i0 < total; i0 += kTermBlock * kTermLoads) {
        float x[kTermLoads];
#pragma unroll
        for (int u = 0; u < kTermLoads; ++u) x[u] = from[min(i0 + u * kTermBlock, total - 1)];
#pragma unroll
        for (int u = 0; u < kTermLoads; ++u) {
            if (i0 + u * kTermBlock < total) dst[k * ld + t] = x[u];
            t += dq;
            k += dr;
            if (k >= per) k -= per, ++t;
        }
    }
}

// GB Gaussians a block (a power of two; 0: `gaussians`), kTermBlock / GB threads each.
template <int L, int MODE, int GB>
__global__ __launch_bounds__(kTermBlock) void k_view_terms(
    const ViewInfo* __restrict__ views, int n_views, int views_per_row, int64_t N, int gaussians,
    const float* __restrict__ means, const float* __restrict__ coeffs, const float* __restrict__ bbar,
    const float* __restrict__ rho, int C, int width, float* __restrict__ out) {
    constexpr int NB = (L + 1) * (L + 1);
    extern __shared__ float stage[];
    const int gb = GB != 0 ? GB : gaussians, ld = gb + 1;
    float* sc = stage;               // c_g
    float* sb = stage + NB * C * ld; // Bbar_g
    const int64_t g0 = (int64_t)blockIdx.x * gb;
    const int n = (int)min((int64_t)gb, N - g0);
    const int slots = kTermBlock / gb, slot = GB == kTermBlock ? 0 : (int)threadIdx.x / gb;  // (uniform: scalar loads)
    const int t = GB == kTermBlock ? (int)threadIdx.x : (int)threadIdx.x & (gb - 1);
    const int64_t g = g0 + t;
    const bool own = t < n;
    const double px = own ? (double)means[3 * g] : 0.0, py = own ? (double)means[3 * g + 1] : 0.0,
                 pz = own ? (double)means[3 * g + 2] : 0.0;
    const double rg = (MODE == kAdjoint && own) ? (double)rho[g] : 0.0;
    const int v_first = (int)blockIdx.y * views_per_row, v_end = min(n_views, v_first + views_per_row);
    const int stride = MODE == kColours ? C : beta_stride(C, width);
    stage_terms(coeffs, g0, n, NB * C, ld, sc);
    if constexpr (MODE == kAdjoint) stage_terms(bbar, g0, n, NB * C, ld, sb);
    __syncthreads();
    // VT views of the thread, from v on, `slots` apart
    auto terms = [&](int v, auto vt) {
        constexpr int VT = decltype(vt)::value;
        float phi[VT][NB];
        float* dst[VT];
        double delta[VT];
#pragma unroll
        for (int j = 0; j < VT; ++j) {
            const ViewInfo& V = views[min(v + j * slots, v_end - 1)];
            const int64_t k = g - V.g_offset;
            const bool in = own && v + j * slots < v_end && k >= 0 && k < (int64_t)V.n_gauss;
            dst[j] = in ? out + ((int64_t)V.item_base + k) * stride : nullptr;
            const double dx = px - V.centre[0], dy = py - V.centre[1], dz = pz - V.centre[2];
            const double inv = 1.0 / sqrt(dx * dx + dy * dy + dz * dz);
            sh_eval<float, L>((float)(dx * inv), (float)(dy * inv), (float)(dz * inv), phi[j]);
            delta[j] = rg;
        }
        int end = min(width, C), part = C;  // of the channels that share a delta
        for (int c = 0; c < C; ++c) {
            float a[VT] = {}, b[VT] = {};
#pragma unroll
            for (int m = 0; m < NB; ++m) {
                const float x = sc[(m * C + c) * ld + t];
#pragma unroll
                for (int j = 0; j < VT; ++j) a[j] = fmaf(x, phi[j][m], a[j]);
                if constexpr (MODE == kAdjoint) {
                    const float y = sb[(m * C + c) * ld + t];
#pragma unroll
                    for (int j = 0; j < VT; ++j) b[j] = fmaf(y, phi[j][m], b[j]);
                }
            }
#pragma unroll
            for (int j = 0; j < VT; ++j) {
                if constexpr (MODE == kAdjoint) delta[j] += (double)a[j] * (double)b[j];
                if (dst[j]) dst[j][c] = MODE == kAdjoint ? b[j] : a[j];
            }
            if constexpr (MODE != kColours) {
                if (c + 1 != end) continue;  // uniform
#pragma unroll
                for (int j = 0; j < VT; ++j) {
                    if (dst[j]) dst[j][part] = MODE == kAdjoint ? (float)delta[j] : 0.0f;
                    delta[j] = 0.0;
                }
                end = min(end + width, C);
                ++part;
            }
        }
    };
    for (int vb = v_first; vb < v_end; vb += kTermViews * slots) {
        if (v_end - vb > slots) terms(vb + slot, std::integral_constant<int, kTermViews>{});
        else terms(vb + slot, std::integral_constant<int, 1>{});
    }
}

namespace {

template <int L, int MODE>
void launch_terms(const ViewInfo* views, int n_views, int64_t N, const float* means, const float* coeffs,
                  const float* bbar, const float* rho, int C, int width, float* out, hipStream_t s) {
    const size_t per = (size_t)((L + 1) * (L + 1)) * (size_t)C * (MODE == kAdjoint ? 2 : 1);
    int gb = kTermBlock;  // (64 channels of degree 3, two sets: four)
    while (gb > 1 && per * (size_t)(gb + 1) > kTermStage) gb /= 2;
    const int64_t gx = (N + gb - 1) / gb;
    // views split over grid rows where the Gaussians alone give under 4096
    // blocks (two waves each: eight a SIMD).  Each row stages the coefficients
    // again: 2344 blocks by 40 views take 117 us in one row, 127 in five
    const int set = kTermViews * (kTermBlock / gb), sets_of_views = (n_views + set - 1) / set;
    const int64_t rows = std::min<int64_t>(std::max<int64_t>(4096 / gx, 1), sets_of_views);
    const int per_row = (int)((sets_of_views + rows - 1) / rows) * set;
    dim3 grid((unsigned)gx, (unsigned)((n_views + per_row - 1) / per_row)), block(kTermBlock);
#define GSC_TERMS(GBV)                                                                                    \
    hipLaunchKernelGGL((k_view_terms<L, MODE, GBV>), grid, block, sizeof(float) * per * (size_t)(gb + 1), s, \
                       views, n_views, per_row, N, gb, means, coeffs, bbar, rho, C, width, out)
    if (gb == kTermBlock) GSC_TERMS(kTermBlock);
    else GSC_TERMS(0);
#undef GSC_TERMS
}

template <int MODE>
void launch_terms_deg(int sh_deg, const ViewInfo* views, int n_views, int64_t N, const float* means,
                      const float* coeffs, const float* bbar, const float* rho, int C, int width, float* out,
                      hipStream_t s) {
    if (N <= 0 || n_views <= 0) return;
    switch (sh_deg) {
        case 0: launch_terms<0, MODE>(views, n_views, N, means, coeffs, bbar, rho, C, width, out, s); break;
        case 1: launch_terms<1, MODE>(views, n_views, N, means, coeffs, bbar, rho, C, width, out, s); break;
        case 2: launch_terms<2, MODE>(views, n_views, N, means, coeffs, bbar, rho, C, width, out, s); break;
        default: launch_terms<3, MODE>(views, n_views, N, means, coeffs, bbar, rho, C, width, out, s); break;
    }
}

}  // namespace

void launch_view_colors(const ViewInfo* views, int n_views, int64_t N, const float* means,
                        const float* coeffs, int C, int sh_deg, float* gamma, hipStream_t s) {
    launch_terms_deg<kColours>(sh_deg, views, n_views, N, means, coeffs, nullptr, nullptr, C, C, gamma, s);
}

void launch_view_adjoint(const ViewInfo* views, int n_views, int64_t N, const float* means,
                         const float* coeffs, const float* bbar, const float* rho, int C, int width,
                         int sh_deg, float* beta, hipStream_t s) {
    if (bbar == nullptr)
        launch_terms_deg<kRenderAdjoint>(sh_deg, views, n_views, N, means, coeffs, nullptr, nullptr, C, width, beta, s);
    else
        launch_terms_deg<kAdjoint>(sh_deg, views, n_views, N, means, coeffs, bbar, rho, C, width, beta, s);
}

// images[row][c] = sum_g w_gp * gamma_gv[c]; every pixel of every tile is
// written.  Same tile walk and blend decisions as accumulate_tile.
// res.y non-null: images[row][c] = y[row][c] - the blend (the residual of a
// refinement pass, without a pass of its own over targets and images: 34 us of
// 5.2 M pixels; see residual_in_render).
__device__ __forceinline__ float pixel_out(const RenderResidual& res, int64_t at, float img) {
    if (res.y == nullptr) return img;  // uniform
    return (res.bf16 ? load_target<true>(res.y, at) : load_target<false>(res.y, at)) - img;
}

template <int CC, int BIN>
__global__ __launch_bounds__(64 * kTileWaves) void k_render(
    const ViewInfo* __restrict__ views, int n_views, uint32_t n_wt, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ pair_vals, const float4* __restrict__ rec,
    const uint32_t* __restrict__ items, const float* __restrict__ gamma, int C, int c_off, BlendParams bp, float* __restrict__ images,
    unsigned long long* __restrict__ counter, const uint32_t* __restrict__ order, const RenderResidual res) {
    static_assert(CC <= 4, "one float4 of colours per entry");
    // the chunk's records and colours, read back by every lane as broadcasts
    __shared__ float4 srec1[kTileWaves][64];
    __shared__ float4 scol[kTileWaves][64];
    __shared__ float2 srec0[kTileWaves][64];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const uint32_t wi = xcd_block<128 / kTileWaves>(blockIdx.x, gridDim.x) * kTileWaves + w;
    if (wi >= n_wt) return;
    const uint32_t wt = queued_tile<BIN>(wi, order);  // blocks start in index order
    const TileGeom tg = tile_geom<BIN>(wt, views, n_views);
    const ViewInfo& V = views[tg.vloc];
    float T[4];
    bool inside[4];
    float img[4][CC];
    uint32_t alive = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        inside[k] = tg.x0 + block_px(lane, k) < V.width && tg.y0 + block_py(lane, k) < V.height;
        T[k] = inside[k] ? 1.0f : kOutsideT;
        alive |= (__builtin_amdgcn_ballot_w64(inside[k]) != 0 ? 1u : 0u) << k;
#pragma unroll
        for (int c = 0; c < CC; ++c) img[k][c] = 0.0f;
    }
    alive = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive);
    uint2 rg = ranges[tg.bin];
    rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
    rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
    uint32_t cnt = 0;
    // loop constants in vector registers (see uniform_in_vgpr)
    const float qlim = uniform_in_vgpr((float)(kExp2Scale * (double)bp.cut2));
    const float amax = uniform_in_vgpr(bp.alpha_max), amin = uniform_in_vgpr(bp.alpha_min),
                tmin = uniform_in_vgpr(bp.t_min);
    // the lane's pixel offsets from the tile's centre point; R0 below keeps,
    // per entry, the offset of that point from the projected centre
    const float lx[2] = {tile_offset_col(lane, 0), tile_offset_col(lane, 1)};
    const float ly[2] = {tile_offset_row(lane, 0), tile_offset_row(lane, 1)};
    const float ox = tile_centre(tg.x0), oy = tile_centre(tg.y0);
    // A chunk of 64 entries is gathered at once, one entry per lane (records
    // and the item's colours), and staged in LDS, from which an entry reads
    // them back with broadcast loads; each lane forms its entry's block mask,
    // and only entries reaching a block with a live pixel are visited.
    for (uint32_t b = rg.x; b < rg.y && alive != 0u; b += 64) {
        const uint32_t nb = min(64u, rg.y - b);
        const uint32_t pv = lane < nb ? pair_vals[b + lane] : 0u;
        const bool own = lane < nb && pair_reaches<BIN>(pv, tg.quad, alive);
        const uint32_t it = pv & kItemMask;
        const float4 r = own ? rec[2 * (size_t)it] : make_float4(0.f, 0.f, 0.f, 0.f);
        const float2 R0 = make_float2((ox - r.x) - r.z, (oy - r.y) - r.w);
        const float4 R1 = own ? rec[2 * (size_t)it + 1] : make_float4(0.f, 0.f, 0.f, 0.f);
        const uint32_t gid = own ? items[it] : 0u;
        const float* gl = gamma + (int64_t)gid * C + c_off;
        float RC[CC];
#pragma unroll
        for (int c = 0; c < CC; ++c) RC[c] = (own && c_off + c < C) ? gl[c] : 0.0f;
        const uint32_t BL = own ? (entry_blocks<BIN>(pv, R0, R1, bp) & alive) : 0u;
        uint64_t todo = __builtin_amdgcn_ballot_w64(BL != 0u);
        srec1[w][lane] = R1;
        srec0[w][lane] = R0;
        scol[w][lane] = make_float4(RC[0], CC > 1 ? RC[CC > 1 ? 1 : 0] : 0.0f, CC > 2 ? RC[CC > 2 ? 2 : 0] : 0.0f,
                                    CC > 3 ? RC[CC > 3 ? 3 : 0] : 0.0f);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // (liveness is refreshed every four entries: an entry after the last live
        // pixel stopped meets T < t_min everywhere and adds nothing)
        while (todo != 0u && alive != 0u) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t j = todo != 0u ? (uint32_t)__builtin_ctzll(todo) : 0u;
                const uint32_t blocks = todo != 0u ? bcast_u(BL, j) & alive : 0u;
                todo &= todo - 1u;
                if (blocks == 0u) continue;
                const float2 c0 = srec0[w][j];
                const float4 c1 = srec1[w][j];
                const float4 c4 = scol[w][j];
                const float col[4] = {c4.x, c4.y, c4.z, c4.w};
                const float dx[2] = {c0.x + lx[0], c0.x + lx[1]}, dy[2] = {c0.y + ly[0], c0.y + ly[1]};
                const float a0[2] = {c1.x * dx[0] * dx[0], c1.x * dx[1] * dx[1]};
                const float b0[2] = {c1.y * dx[0], c1.y * dx[1]};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (!((blocks >> k) & 1u)) continue;
                    const float q2 = fmaf(dy[k >> 1], fmaf(c1.z, dy[k >> 1], b0[k & 1]), a0[k & 1]);
                    const float w = lane_step(q2, c1.w, T[k], qlim, amin, amax, tmin, cnt);
#pragma unroll
                    for (int c = 0; c < CC; ++c) img[k][c] = fmaf(w, col[c], img[k][c]);
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) alive &= __builtin_amdgcn_ballot_w64(T[k] >= tmin) != 0 ? 15u : ~(1u << k);
            alive = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive);
        }
        __builtin_amdgcn_wave_barrier();  // the next chunk overwrites the records
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (!inside[k]) continue;
        int64_t row = V.pixel_offset + (int64_t)(tg.y0 + block_py(lane, k)) * V.width + tg.x0 + block_px(lane, k);
#pragma unroll
        for (int c = 0; c < CC; ++c)
            if (c_off + c < C) images[row * C + c_off + c] = pixel_out(res, row * C + c_off + c, img[k][c]);
    }
    if (c_off == 0) {
        cnt = wave_sum_u32(cnt);
        if (lane == 0 && cnt) atomicAdd(counter, (unsigned long long)cnt);
    }
}

// Few tiles: one wave per 8x8 block (walk_block), CC = 4 * EX channels per launch.
template <int EX, int BIN>
__global__ __launch_bounds__(256) void k_render_blocks(
    const ViewInfo* __restrict__ views, int n_views, uint32_t n_tiles, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ pair_vals, const float4* __restrict__ rec,
    const uint32_t* __restrict__ items, const float* __restrict__ gamma, int C, int c_off, BlendParams bp,
    float* __restrict__ images, unsigned long long* __restrict__ counter, const uint32_t* __restrict__ order,
    const RenderResidual res) {
    constexpr int CC = 4 * EX;
    __shared__ WalkLds<EX> lds[4];
    const uint32_t lane = threadIdx.x & 63, kq = threadIdx.x >> 6;
    const uint32_t wi = xcd_block(blockIdx.x, gridDim.x);
    if (wi >= n_tiles) return;
    const TileGeom tg = tile_geom<BIN>(queued_tile<BIN>(wi, order), views, n_views);
    const ViewInfo& V = views[tg.vloc];
    const int ix = tg.x0 + block_px(lane, (int)kq), iy = tg.y0 + block_py(lane, (int)kq);
    const bool inside = (ix < V.width) & (iy < V.height);
    if (__builtin_amdgcn_ballot_w64(inside) == 0) return;  // whole wave
    uint2 rg = ranges[tg.bin];
    rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
    rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
    const float tmin = uniform_in_vgpr(bp.t_min);
    float T = inside ? 1.0f : kOutsideT;
    float img[CC];
#pragma unroll
    for (int c = 0; c < CC; ++c) img[c] = 0.0f;
    uint32_t cnt = 0;
    walk_block<BIN, EX>(tg, kq, lane, rg, pair_vals, rec, items, bp, lds[kq],
                        [&](bool own, uint32_t item, float4 (&ex)[EX]) {
        const float* gl = gamma + (int64_t)item * C + c_off;
        float v[CC];
#pragma unroll
        for (int c = 0; c < CC; ++c) v[c] = (own && c_off + c < C) ? gl[c] : 0.0f;
#pragma unroll
        for (int x = 0; x < EX; ++x) ex[x] = make_float4(v[4 * x], v[4 * x + 1], v[4 * x + 2], v[4 * x + 3]);
    }, [&](const WalkGroup<EX>& g) -> bool {
        uint64_t kept = 0;
#pragma unroll
        for (int u = 0; u < kWalkEntries; ++u) {
            const float w = pixel_blend(g.ae[u], T, tmin, kept);
            cnt += (uint32_t)__popcll(g.cand[u] & kept);
#pragma unroll
            for (int x = 0; x < EX; ++x) {
                const float4 c4 = g.ex[u][x];
                img[4 * x] = fmaf(w, c4.x, img[4 * x]);
                img[4 * x + 1] = fmaf(w, c4.y, img[4 * x + 1]);
                img[4 * x + 2] = fmaf(w, c4.z, img[4 * x + 2]);
                img[4 * x + 3] = fmaf(w, c4.w, img[4 * x + 3]);
            }
        }
        return kept != 0;
    });
    if (inside) {
        const int64_t at = (V.pixel_offset + (int64_t)iy * V.width + ix) * C + c_off;
#pragma unroll
        for (int c = 0; c < CC; ++c)
            if (c_off + c < C) images[at + c] = pixel_out(res, at + c, img[c]);
    }
    if (c_off == 0 && lane == 0 && cnt) atomicAdd(counter, (unsigned long long)cnt);
}

// Channels a launch takes.
static int render_channels(const TileLists& tl, int C) { return few_tiles(tl) && C > 4 ? 8 : 4; }
int render_launches(const TileLists& tl, int C) {
    const int ch = render_channels(tl, C);
    return (C + ch - 1) / ch;
}

// Each launch of a render would read its own channels of the targets, so every line
// of them: the stores form the residual where one launch writes all channels.  us a
// call with two passes, in the stores / by a pass: 20 views of 512x512, 100k splats, 4
// channels 2442 / 2459, 8 (two launches) 3286 / 3346, 16 7491 / 6560, 64 bf16 34286 /
// 25079; 18 views of 531x382, 700 splats, 4 767 / 777, 8 1126 / 977, 64 15310 / 6187.
bool residual_in_render(const TileLists& tl, int C) { return render_launches(tl, C) == 1; }

// images = y - images over n values from `first`.
__global__ __launch_bounds__(256) void k_residual(const void* __restrict__ y, int bf16, int64_t first, int64_t n,
                                                  float* __restrict__ images) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = first + i;
        images[e] = (bf16 ? load_target<true>(y, e) : load_target<false>(y, e)) - images[e];
    }
}

void launch_residual(const RenderResidual& res, int64_t first, int64_t n, float* images, hipStream_t s) {
    if (n <= 0) return;
    const unsigned blocks = (unsigned)std::min<int64_t>((n + 255) / 256, 16384);
    hipLaunchKernelGGL(k_residual, dim3(blocks), dim3(256), 0, s, res.y, res.bf16, first, n, images);
}

void launch_render(const TileLists& tl, const float* gamma, int C, BlendParams bp, float* images,
                   unsigned long long* counter, hipStream_t s, const RenderResidual& res) {
    if (tl.n_bins == 0) return;
    const uint32_t n_wt = wave_tiles(tl.n_bins, tl.bin);
    const int step = render_channels(tl, C);
    if (few_tiles(tl)) {
#define GSC_RENDERB(EXV, BINV)                                                                            \
    hipLaunchKernelGGL((k_render_blocks<EXV, BINV>), dim3(n_wt), dim3(256), 0, s, tl.views, tl.n_views,   \
                       n_wt, tl.ranges, tl.pair_vals, tl.rec, tl.items, gamma, C, c_off, bp, images,      \
                       counter, tl.order, res)
        for (int c_off = 0; c_off < C; c_off += step) {
            if (tl.bin == 32) {
                if (C <= 4) GSC_RENDERB(1, 32); else GSC_RENDERB(2, 32);
            } else {
                if (C <= 4) GSC_RENDERB(1, 16); else GSC_RENDERB(2, 16);
            }
        }
#undef GSC_RENDERB
        return;
    }
    dim3 grid((n_wt + kTileWaves - 1) / kTileWaves), block(64 * kTileWaves);
#define GSC_RENDER(CCV, BINV)                                                                            \
    hipLaunchKernelGGL((k_render<CCV, BINV>), grid, block, 0, s, tl.views, tl.n_views, n_wt, tl.ranges, \
                       tl.pair_vals, tl.rec, tl.items, gamma, C, c_off, bp, images, counter, tl.order, res)
    for (int c_off = 0; c_off < C; c_off += step) {
        const bool three = C <= 3 && c_off == 0;
        if (tl.bin == 32) {
            if (three) GSC_RENDER(3, 32); else GSC_RENDER(4, 32);
        } else {
            if (three) GSC_RENDER(3, 16); else GSC_RENDER(4, 16);
        }
    }
#undef GSC_RENDER
}

}  // namespace gsc
