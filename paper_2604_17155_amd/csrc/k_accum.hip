// Fused per-tile blend + accumulate (the hot loop).
//
// One wave64 owns one 16x16 tile; lane l handles pixel (l%8, l/8) of each of
// its four 8x8 blocks.  The tile's Gaussians arrive in front-to-back
// order (eq. 2).  Each lane blends its pixels in FP32; per Gaussian the wave
// reduces sum_p w and sum_p w*y_p over the tile (the per-view visibility V_gj
// of eq. 5 and the numerator of eq. 6) with DPP row reductions, and one
// atomic per value adds the tile's share to the (view, Gaussian) slot.
// Splat records for the next 64 list entries are loaded one per lane and read
// back from the wave's own LDS slots, so the loop needs no block barrier.
#include <type_traits>

#include "gsc_internal.h"
#include "wave_ops.h"

#include <algorithm>

namespace gsc {


// Adds a tile's share v to the per-view sum at p (an element of VS).  The
// default adds binary32 with a float atomic, so the order of the tiles'
// additions shows in the last bits.  DET: VS holds 64-bit fixed-point words
// instead (element k of VS is word k); v is scaled by the power of two
// `scale`, rounded to an integer and added with an integer atomic, which is
// exact and therefore independent of the order.
template <bool DET>
__device__ __forceinline__ void vs_add(float* VS, float* p, float v, float scale) {
    if constexpr (DET) {
        unsigned long long* q = reinterpret_cast<unsigned long long*>(VS) + (p - VS);
        atomicAdd(q, (unsigned long long)__float2ll_rn(v * scale));
    } else {
        unsafeAtomicAdd(p, v);
    }
}

// One tile, by one wave: blend its pixels front to back and add each
// Gaussian's tile share of V and S (channels [c_off, c_off + CC) of C) to its
// slot.  Returns the accepted contributions of the lane's pixels.
//
// A pixel that stopped has T < t_min (outside the image it starts at
// kOutsideT).  Blocks are skipped when the Gaussian's footprint misses them or
// when none of their pixels is live; the wave ends when no block is live.
template <int CC, bool BF16, int BIN, bool DET>
__device__ __forceinline__ uint32_t accumulate_tile(
    uint32_t tile, uint32_t lane, const ViewInfo* __restrict__ views, int n_views,
    const uint2* __restrict__ ranges, const uint32_t* __restrict__ pair_vals,
    const float4* __restrict__ rec, const uint32_t* __restrict__ items,
    const void* __restrict__ targets, int C, int c_off, int per_view, const BlendParams& bp,
    float* __restrict__ VS, float2 dsc, uint32_t* __restrict__ gcount, float4* __restrict__ lrec1,
    float2* __restrict__ lrec0) {
    constexpr int CCA = CC > 0 ? CC : 1;
    const TileGeom tg = tile_geom<BIN>(tile, views, n_views);
    uint2 rg = ranges[tg.bin];
    rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
    rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
    if (rg.x >= rg.y) return 0;  // no entries: the tile's targets are not read
    const ViewInfo& V = views[tg.vloc];
    // view fields read once (plain values: the conditions below need no branch)
    const int vw = V.width, vh = V.height;
    const int64_t poff = V.pixel_offset;
    const int stride = C + 1;

    float T[4];
    float y[4][CCA];
    uint32_t alive = 0;  // bit k: block k has a live pixel (wave-uniform)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int ix = tg.x0 + block_px(lane, k), iy = tg.y0 + block_py(lane, k);
        const bool inside = (ix < vw) & (iy < vh);
        T[k] = inside ? 1.0f : kOutsideT;
        alive |= (__builtin_amdgcn_ballot_w64(inside) != 0 ? 1u : 0u) << k;
        const int64_t row = poff + (int64_t)iy * vw + ix;
        // unconditional loads (element 0 stands in for pixels outside the
        // image): no branch per load
#pragma unroll
        for (int c = 0; c < CC; ++c) {
            const bool use = inside && c_off + c < C;
            const float v = load_target<BF16>(targets, use ? row * C + c_off + c : 0);
            y[k][c] = use ? v : 0.0f;
        }
    }
    alive = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive);
    uint32_t cnt = 0;  // contributions of the lane's pixels
    // item = V.item_base + g (g local to the view's scene)
    const int64_t item_base = V.item_base;
    const int64_t slot_base = per_view ? V.vs_base : V.g_offset;
    const bool first_chunk = c_off == 0;

    // loop constants in vector registers (see uniform_in_vgpr)
    const float qlim = uniform_in_vgpr((float)(kExp2Scale * (double)bp.cut2));  // q <= cut2  <=>  q2 >= qlim
    const float amax = uniform_in_vgpr(bp.alpha_max), amin = uniform_in_vgpr(bp.alpha_min),
                tmin = uniform_in_vgpr(bp.t_min);
    // the lane's pixel offsets from the tile's centre point
    const float lx[2] = {tile_offset_col(lane, 0), tile_offset_col(lane, 1)};
    const float ly[2] = {tile_offset_row(lane, 0), tile_offset_row(lane, 1)};

    // The list is walked in chunks of 64 entries.  A chunk's records are
    // gathered at once, one entry per lane, and put in LDS, from which every
    // lane reads an entry's; the next chunk's gather (and the pair values of the
    // one after) are in flight while a chunk is blended.
    auto load_pv = [&](uint32_t b) -> uint32_t {
        return b + lane < rg.y ? pair_vals[b + lane] : 0u;
    };
    // R0 keeps, per entry, the offset of the tile's centre point from the
    // projected centre, (x0 + 8 - u_hi) - u_lo and the same in y: a lane's
    // offset is then that plus its pixel's offset from the point
    // (tile_offset_col / tile_offset_row).
    const float ox = tile_centre(tg.x0), oy = tile_centre(tg.y0);
    auto gather = [&](uint32_t pv, uint32_t b, float2& R0, float4& R1, uint32_t& gi) {
        const uint32_t it = pv & kItemMask;
        const bool own = b + lane < rg.y && pair_reaches<BIN>(pv, tg.quad, 15u);
        const float4 r = own ? rec[2 * (size_t)it] : make_float4(0.f, 0.f, 0.f, 0.f);
        R0 = make_float2((ox - r.x) - r.z, (oy - r.y) - r.w);
        R1 = own ? rec[2 * (size_t)it + 1] : make_float4(0.f, 0.f, 0.f, 0.f);
        gi = own ? items[it] : 0u;
    };
    // (wide channel chunks have no registers to spare for the second buffer:
    // there the next chunk is gathered when the current one is done)
    constexpr bool kDouble = CC <= 4;
    uint32_t pv = load_pv(rg.x), pvn = load_pv(rg.x + 64);
    float2 R0;
    float4 R1;
    uint32_t gi;  // the entry's item
    gather(pv, rg.x, R0, R1, gi);
    for (uint32_t b = rg.x; b < rg.y && alive != 0u; b += 64) {
        const uint32_t nb = min(64u, rg.y - b);
        float2 Q0;
        float4 Q1;
        uint32_t qi;
        if constexpr (kDouble) gather(pvn, b + 64, Q0, Q1, qi);
        const uint32_t pvnn = load_pv(b + 128);
        // the chunk's entries that can reach a live block, one bit per lane in
        // list order: the walk visits only these
        // each lane forms its entry's block mask: taking an entry then costs
        // one broadcast of it
        const uint32_t BL = lane < nb && pair_reaches<BIN>(pv, tg.quad, alive) ? entry_blocks<BIN>(pv, R0, R1, bp) : 0u;
        uint64_t todo = __builtin_amdgcn_ballot_w64((BL & alive) != 0u);
        // the chunk's records go through LDS (this wave's 64 slots): an entry
        // reads them back with two broadcast loads instead of six readlanes
        lrec1[lane] = R1;
        lrec0[lane] = R0;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if constexpr (CC <= 3) {
            // Weights alone, 300k Gaussians, 40 views of 800x800: 1.36 -> 1.24 ms
            // (before, a reduction and an atomic per entry; contributions counted
            // by scalar instructions); one channel, 120k, 20 views: 601 -> 587 us.
            // Entries in groups: each entry's tile sums (V, S) stay in a fixed
            // register slot, and one wave reduction of the group's kGroup x
            // kVals values (lane e*kVals+v, bit-reversed) feeds one atomic per value.
            // Tile liveness is refreshed once per group: entries after the
            // last live pixel stopped meet T < t_min everywhere and add nothing.
            constexpr int kVals = CC == 0 ? 1 : (CC == 1 ? 2 : 4), kGroup = CC <= 1 ? 8 : 4;
            constexpr int kPend = kVals * kGroup;
            while (todo != 0u && alive != 0u) {
                float pend[kPend];
                uint32_t who[kGroup];
#pragma unroll
                for (int u = 0; u < kGroup; ++u) {
                    const bool any = todo != 0u;
                    const uint32_t j = any ? (uint32_t)__builtin_ctzll(todo) : 0u;
                    todo &= todo - 1u;
                    who[u] = bcast_u(gi, j);  // the entry's item
                    const uint32_t blocks = any ? bcast_u(BL, j) & alive : 0u;
                    float sv = 0.0f;
                    float ss[CCA];
#pragma unroll
                    for (int c = 0; c < CCA; ++c) ss[c] = 0.0f;
                    const uint32_t before = cnt;
                    if (blocks != 0u) {
                        const float2 c0 = lrec0[j];
                        const float4 c1 = lrec1[j];
                        const float dx[2] = {c0.x + lx[0], c0.x + lx[1]}, dy[2] = {c0.y + ly[0], c0.y + ly[1]};
                        const float a0[2] = {c1.x * dx[0] * dx[0], c1.x * dx[1] * dx[1]};
                        const float b0[2] = {c1.y * dx[0], c1.y * dx[1]};
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            if (!((blocks >> k) & 1u)) continue;  // uniform
                            const float q2 = fmaf(dy[k >> 1], fmaf(c1.z, dy[k >> 1], b0[k & 1]), a0[k & 1]);
                            const float w = lane_step(q2, c1.w, T[k], qlim, amin, amax, tmin, cnt);
                            sv += w;
#pragma unroll
                            for (int c = 0; c < CC; ++c) ss[c] = fmaf(w, y[k][c], ss[c]);
                        }
                    }
                    if (gcount != nullptr && first_chunk) {  // uniform
                        const uint32_t nh = wave_sum_u32(cnt - before);
                        if (nh != 0u && lane == 0)
                            atomicAdd(gcount + V.g_offset + ((int64_t)who[u] - item_base), nh);
                    }
                    pend[kVals * u] = sv;
#pragma unroll
                    for (int v = 1; v < kVals; ++v) pend[kVals * u + v] = v <= CC ? ss[v <= CC && CC > 0 ? v - 1 : 0] : 0.0f;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) alive &= __builtin_amdgcn_ballot_w64(T[k] >= tmin) != 0 ? 15u : ~(1u << k);
                alive = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive);
                {
                    const float t = wave_sum_transposed<kPend>(pend, lane);
                    const int idx = transposed_index<kPend>(lane);
                    const int e = idx / kVals, v = idx % kVals;
                    // lane L & (kGroup - 1) holds the V of L's entry: entries
                    // without weight in the tile add nothing
                    const uint32_t hits = (uint32_t)__builtin_amdgcn_ballot_w64(t > 0.0f);
                    const uint32_t he = (hits >> (lane & (uint32_t)(kGroup - 1))) & 1u;
                    uint32_t item = who[0];
#pragma unroll
                    for (int q = 1; q < kGroup; ++q) item = e == q ? who[q] : item;
                    const int64_t sl = slot_base + ((int64_t)item - item_base);
                    const bool use = lane < (uint32_t)kPend && he != 0u &&
                                     (v == 0 ? first_chunk : (v <= CC && c_off + v - 1 < C));
                    if (use) vs_add<DET>(VS, VS + sl * (int64_t)stride + (v == 0 ? 0 : c_off + v), t,
                                         v == 0 ? dsc.x : dsc.y);
                }
            }
        } else {
            while (todo != 0u) {
                const uint32_t j = (uint32_t)__builtin_ctzll(todo);
                todo &= todo - 1u;
                const uint32_t blocks = bcast_u(BL, j) & alive;
                if (blocks == 0u) continue;
                const uint32_t gid = bcast_u(gi, j);  // the entry's item
                const float2 c0 = lrec0[j];
                const float4 c1 = lrec1[j];
                const float dx[2] = {c0.x + lx[0], c0.x + lx[1]}, dy[2] = {c0.y + ly[0], c0.y + ly[1]};
                const float a0[2] = {c1.x * dx[0] * dx[0], c1.x * dx[1] * dx[1]};
                const float b0[2] = {c1.y * dx[0], c1.y * dx[1]};
                float sv = 0.0f;
                float ss[CCA];
#pragma unroll
                for (int c = 0; c < CCA; ++c) ss[c] = 0.0f;
                const uint32_t before = cnt;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (!((blocks >> k) & 1u)) continue;  // uniform
                    const float q2 = fmaf(dy[k >> 1], fmaf(c1.z, dy[k >> 1], b0[k & 1]), a0[k & 1]);
                    const float w = lane_step(q2, c1.w, T[k], qlim, amin, amax, tmin, cnt);
                    sv += w;
#pragma unroll
                    for (int c = 0; c < CC; ++c) ss[c] = fmaf(w, y[k][c], ss[c]);
                    if (__builtin_amdgcn_ballot_w64(T[k] >= tmin) == 0) alive &= ~(1u << k);
                }
                alive = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive);  // keep it in a scalar register
                if (__builtin_amdgcn_ballot_w64(cnt != before) != 0) {
                    // the pair carries the depth rank; the record names the item
                    const int64_t g = (int64_t)gid - item_base;
                    if (gcount != nullptr && first_chunk) {
                        const uint32_t nh = wave_sum_u32(cnt - before);
                        if (lane == 0) atomicAdd(gcount + V.g_offset + g, nh);
                    }
                    float* slot = VS + (slot_base + g) * (int64_t)stride;
                    const float tv = wave_sum(sv);
                    const float t = wave_sum_transposed<CC>(ss, lane);
                    if (lane == 0 && first_chunk) vs_add<DET>(VS, slot, tv, dsc.x);
                    if (lane < (uint32_t)CC) {
                        const int c = c_off + transposed_index<CC>(lane);
                        if (c < C) vs_add<DET>(VS, slot + 1 + c, t, dsc.y);
                    }
                }
                if (alive == 0u) break;
            }
        }
        __builtin_amdgcn_wave_barrier();  // the next chunk's records overwrite these
        if constexpr (kDouble) {
            R0 = Q0;
            R1 = Q1;
            gi = qi;
        } else {
            gather(pvn, b + 64, R0, R1, gi);
        }
        pv = pvn;
        pvn = pvnn;
    }
    return cnt;
}

// CC: channels handled by this launch (chunk [c_off, c_off + CC) of C).
// queue == nullptr: one tile per wave (kTileWaves a block) over a grid covering all
// tiles.  Otherwise persistent: a fixed grid whose waves take tiles from the
// counter *queue (zero before the launch) until none are left.  Either way
// tiles come in the order `order` gives (nullptr: tile index order).
// Waves per SIMD the register allocation is held to: the weights alone and one
// channel fit seven (72 registers), two and three channels six (80; held to
// seven they spill 18 values, 1.43 -> 1.54 ms on 300k Gaussians, 40 views), sixteen
// four (127; left alone it takes 170 and runs at two waves: a call of 16 FP32
// channels, 100k splats, 20 views of 512x512 1411 -> 1148 us); four and eight are
// left alone.
template <int CC>
constexpr int acc_waves_per_simd() { return CC <= 1 ? 7 : (CC <= 3 ? 6 : (CC == 16 ? 4 : 1)); }

template <int CC, bool BF16, int BIN, bool DET>
__global__ __launch_bounds__(64 * kTileWaves) __attribute__((amdgpu_waves_per_eu(acc_waves_per_simd<CC>()))) void k_accumulate(
    const ViewInfo* __restrict__ views, int n_views, uint32_t n_tiles, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ pair_vals,
    const float4* __restrict__ rec, const uint32_t* __restrict__ items,
    const void* __restrict__ targets, int C, int c_off,
    int per_view, BlendParams bp, float* __restrict__ VS, float2 dsc,
    unsigned long long* __restrict__ counter, uint32_t* __restrict__ gcount,
    uint32_t* __restrict__ queue, const uint32_t* __restrict__ order) {
    __shared__ float4 srec1[kTileWaves][64];
    __shared__ float2 srec0[kTileWaves][64];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t cnt = 0;
    if (queue == nullptr) {
        const uint32_t wi = xcd_block<128 / kTileWaves>(blockIdx.x, gridDim.x) * kTileWaves + w;
        if (wi >= n_tiles) return;  // whole wave
        const uint32_t tile = queued_tile<BIN>(wi, order);  // blocks start in index order
        cnt = accumulate_tile<CC, BF16, BIN, DET>(tile, lane, views, n_views, ranges, pair_vals,
                                                  rec, items, targets, C, c_off, per_view, bp,
                                                  VS, dsc, gcount, srec1[w], srec0[w]);
    } else {
        for (;;) {
            uint32_t t = 0;
            if (lane == 0) t = atomicAdd(queue, 1u);
            const uint32_t tq = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
            if (tq >= n_tiles) break;  // uniform: every wave ends here
            const uint32_t tile = queued_tile<BIN>(tq, order);
            cnt += accumulate_tile<CC, BF16, BIN, DET>(tile, lane, views, n_views, ranges, pair_vals,
                                                       rec, items, targets, C, c_off,
                                                       per_view, bp, VS, dsc, gcount, srec1[w], srec0[w]);
        }
    }
    if (c_off == 0) {
        cnt = wave_sum_u32(cnt);
        if (lane == 0 && cnt) atomicAdd(counter, (unsigned long long)cnt);
    }
}

// ---- few tiles: one wave per 8x8 block ------------------------------------
//
// See walk_block.  Four entries' values, VPE = 1, 4, 8 or 16 per entry (the
// weight and CC = VPE - 1 channels), are reduced over the wave 16 at a time
// (four entries, two or one; weights only: four values at once), one atomic
// instruction per reduction.
template <int CC, bool BF16, int BIN>
__global__ __launch_bounds__(256) void k_accumulate_blocks(
    const ViewInfo* __restrict__ views, int n_views, uint32_t n_tiles, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ pair_vals, const float4* __restrict__ rec,
    const uint32_t* __restrict__ items, const void* __restrict__ targets, int C, int c_off, int per_view,
    BlendParams bp, float* __restrict__ VS, unsigned long long* __restrict__ counter,
    uint32_t* __restrict__ gcount, const uint32_t* __restrict__ order) {
    constexpr int CCA = CC > 0 ? CC : 1;
    constexpr int VPE = CC + 1;
    static_assert(VPE == 1 || VPE == 4 || VPE == 8 || VPE == 16, "values per entry");
    __shared__ WalkLds<0> lds[4];
    const uint32_t lane = threadIdx.x & 63, kq = threadIdx.x >> 6;
    const uint32_t wi = xcd_block(blockIdx.x, gridDim.x);
    if (wi >= n_tiles) return;
    const TileGeom tg = tile_geom<BIN>(queued_tile<BIN>(wi, order), views, n_views);
    const ViewInfo& V = views[tg.vloc];
    const int ix = tg.x0 + block_px(lane, (int)kq), iy = tg.y0 + block_py(lane, (int)kq);
    const bool inside = (ix < V.width) & (iy < V.height);
    if (__builtin_amdgcn_ballot_w64(inside) == 0) return;  // whole wave
    const int64_t row = V.pixel_offset + (int64_t)iy * V.width + ix;
    float y[CCA];
#pragma unroll
    for (int c = 0; c < CC; ++c) {
        const bool use = inside && c_off + c < C;
        const float v = load_target<BF16>(targets, use ? row * C + c_off + c : 0);
        y[c] = use ? v : 0.0f;
    }
    uint2 rg = ranges[tg.bin];
    rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
    rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
    const int64_t item_base = V.item_base, slot_base = per_view ? V.vs_base : V.g_offset, g_off = V.g_offset;
    const int stride = C + 1;
    const bool first_chunk = c_off == 0;
    const float tmin = uniform_in_vgpr(bp.t_min);
    float T = inside ? 1.0f : kOutsideT;
    uint32_t cnt = 0;
    walk_block<BIN, 0>(tg, kq, lane, rg, pair_vals, rec, items, bp, lds[kq], [](bool, uint32_t, float4*) {},
                       [&](const WalkGroup<0>& g) -> bool {
        float w[kWalkEntries];
        uint32_t nh[kWalkEntries];
        uint64_t kept = 0;
#pragma unroll
        for (int u = 0; u < kWalkEntries; ++u) {
            w[u] = pixel_blend(g.ae[u], T, tmin, kept);
            nh[u] = (uint32_t)__popcll(g.cand[u] & kept);
            cnt += nh[u];
        }
        if (gcount != nullptr && first_chunk && lane == 0) {
#pragma unroll
            for (int u = 0; u < kWalkEntries; ++u)
                if (nh[u] != 0u) atomicAdd(gcount + g_off + ((int64_t)g.item[u] - item_base), nh[u]);
        }
        constexpr int NV = VPE == 1 ? kWalkEntries : 16;  // values per reduction
        constexpr int EPR = NV / VPE;                     // entries per reduction
#pragma unroll
        for (int e0 = 0; e0 < kWalkEntries; e0 += EPR) {
            uint32_t any = 0;
#pragma unroll
            for (int e = 0; e < EPR; ++e) any |= nh[e0 + e];
            if (any == 0u) continue;  // uniform
            float pend[NV];
#pragma unroll
            for (int e = 0; e < EPR; ++e) {
                pend[e * VPE] = w[e0 + e];
#pragma unroll
                for (int c = 0; c < CC; ++c) pend[e * VPE + 1 + c] = w[e0 + e] * y[c];
            }
            const float t = wave_sum_transposed<NV>(pend, lane);
            const int idx = transposed_index<NV>(lane);
            const int e = idx / VPE, v = idx % VPE;
            uint32_t item = g.item[e0], h = nh[e0];
#pragma unroll
            for (int q = 1; q < EPR; ++q) {
                item = e == q ? g.item[e0 + q] : item;
                h = e == q ? nh[e0 + q] : h;
            }
            const bool use = lane < (uint32_t)NV && h != 0u && (v == 0 ? first_chunk : c_off + v - 1 < C);
            if (use)
                unsafeAtomicAdd(VS + (slot_base + ((int64_t)item - item_base)) * (int64_t)stride + (v == 0 ? 0 : c_off + v), t);
        }
        return kept != 0;
    });
    if (c_off == 0 && lane == 0 && cnt) atomicAdd(counter, (unsigned long long)cnt);
}

// One launch: channels [c_off, c_off + CC) of C.
template <int CC, bool BF16>
static void launch_acc_blocks(const TileLists& tl, const void* targets, int C, int c_off, bool per_view,
                              BlendParams bp, float* VS, unsigned long long* counter, uint32_t* gcount,
                              hipStream_t s) {
    const uint32_t n_wt = wave_tiles(tl.n_bins, tl.bin);
    if (tl.bin == 32)
        hipLaunchKernelGGL((k_accumulate_blocks<CC, BF16, 32>), dim3(n_wt), dim3(256), 0, s, tl.views,
                           tl.n_views, n_wt, tl.ranges, tl.pair_vals, tl.rec, tl.items, targets, C, c_off,
                           (int)per_view, bp, VS, counter, gcount, tl.order);
    else
        hipLaunchKernelGGL((k_accumulate_blocks<CC, BF16, 16>), dim3(n_wt), dim3(256), 0, s, tl.views,
                           tl.n_views, n_wt, tl.ranges, tl.pair_vals, tl.rec, tl.items, targets, C, c_off,
                           (int)per_view, bp, VS, counter, gcount, tl.order);
}

template <int CC, bool BF16, int BIN, bool DET = false>
static void launch_acc_k(const TileLists& tl, const void* targets, int C, bool per_view, BlendParams bp,
                         float* VS, unsigned long long* counter, uint32_t* gcount, uint32_t* queues,
                         hipStream_t s, float2 dsc = make_float2(0.f, 0.f)) {
    const uint32_t n_wt = wave_tiles(tl.n_bins, BIN);
    const uint32_t full = (n_wt + kTileWaves - 1) / kTileWaves;
    dim3 grid(queues ? std::min(full, kPersistentBlocks * 4 / kTileWaves) : full), block(64 * kTileWaves);
    int pass = 0;
    const int step = CC > 0 ? CC : C + 1;
    for (int c_off = 0; c_off < std::max(C, 1); c_off += step, ++pass) {
        uint32_t* q = queues ? queues + pass : nullptr;
        hipLaunchKernelGGL((k_accumulate<CC, BF16, BIN, DET>), grid, block, 0, s, tl.views, tl.n_views,
                           n_wt, tl.ranges, tl.pair_vals, tl.rec, tl.items, targets, C, c_off,
                           (int)per_view, bp, VS, dsc, counter, gcount, q, tl.order);
    }
}

template <int CC>
static void launch_acc_cc(const TileLists& tl, const void* targets, int tdtype, int C, bool per_view,
                          BlendParams bp, float* VS, unsigned long long* counter, uint32_t* gcount,
                          uint32_t* queues, hipStream_t s, const float2* det) {
    const bool bf = tdtype == GSC_BF16;
#define GSC_ACCK(BFV, BINV, DETV)                                                             \
    launch_acc_k<CC, BFV, BINV, DETV>(tl, targets, C, per_view, bp, VS, counter, gcount, queues, s, \
                                      det ? *det : make_float2(0.f, 0.f))
    if (det) {
        if (tl.bin == 32) {
            if (bf) GSC_ACCK(true, 32, true); else GSC_ACCK(false, 32, true);
        } else {
            if (bf) GSC_ACCK(true, 16, true); else GSC_ACCK(false, 16, true);
        }
    } else if (tl.bin == 32) {
        if (bf) GSC_ACCK(true, 32, false); else GSC_ACCK(false, 32, false);
    } else {
        if (bf) GSC_ACCK(true, 16, false); else GSC_ACCK(false, 16, false);
    }
#undef GSC_ACCK
}

// ---- matrix-core accumulate (BF16 targets, channel blocks of 16) ----------
//
// The channel sums S_g[c] = sum_p w_gp y_p[c] of a tile are a product
// W (Gaussians x pixels) . Y (pixels x channels).  Here the blend runs as in
// accumulate_tile, but each entry's weights go to LDS as a row of W, split
// into a BF16 high part (w's upper half) and a BF16 remainder (the exact
// w - hi rounded; w = hi + lo to 2^-16 relative).  Every 8 entries,
// v_mfma_f32_16x16x32_bf16 forms (W_hi + W_lo) . [Y | 1] over the tile's 256
// pixels (eight K-steps of 32 pixels): the targets, held as B operands in
// registers for the whole tile, give S, and a block of ones gives
// V = sum_p w from the same split weights.  (Groups of 8 entries put W_hi in
// rows 0..7 of the A operand and W_lo in rows 8..15: one product per K-step.)
// K index 64 j + l is the blend's pixel of lane l in block j, so index
// 32 s + 8 q + i of K-step s (q = lane / 16) is the pixel in row 4 (s & 1) + q
// and column i of block s / 2: eight neighbours of a pixel row per lane.

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

constexpr int kWRow = 264;       // LDS row of W in BF16 elements (256 + padding against bank conflicts)
constexpr int kMfmaWaves = 2;    // waves per block

// W rows of one wave: kMfmaRows list entries per matrix product (the A operand
// holds the high parts in rows 0..7 and the remainders in rows 8..15).
constexpr int kMfmaRows = 8;
struct alignas(16) MfmaLds {
    __bf16 whi[kMfmaRows * kWRow];
    __bf16 wlo[kMfmaRows * kWRow];
    uint32_t gslot[kMfmaRows];  // local Gaussian of each group row (0xFFFFFFFF: no contribution)
    float4 crec1[64];      // the chunk's records, read back by every lane as one broadcast:
    float2 crec0[64];      // conic and opacity; the centre offset (one channel block only)
};

// Waves per SIMD the register allocation is held to (the weight rows in LDS
// allow them): the 32-channel form ran at two waves per SIMD with 208
// registers and runs at three with 168; the 16-channel and packed forms at
// four (128 registers, up from three).
template <int NBLK>
constexpr int mfma_waves_per_simd() { return NBLK == 2 ? 3 : 4; }

// YM: target layout in the B operand.  0: BF16, NBLK blocks of 16 channels,
// V from a separate product against ones.  1: BF16, C <= 15 channels packed
// with a ones column (column C) in one block.  2: FP32, C <= 7 channels
// split into BF16 high parts (columns 0..C-1) and remainders (columns
// C..2C-1), ones in column 2C.  Packed forms run in one launch (c_off = 0).
template <int NBLK, int BIN, int YM>
__device__ __forceinline__ uint32_t accumulate_tile_mfma(
    uint32_t tile, uint32_t lane, MfmaLds& L, const ViewInfo* __restrict__ views, int n_views,
    const uint2* __restrict__ ranges, const uint32_t* __restrict__ pair_vals,
    const float4* __restrict__ rec, const uint32_t* __restrict__ items,
    const void* __restrict__ targets, int C, int c_off, int per_view, const BlendParams& bp,
    const SumRows& out, uint32_t* __restrict__ gcount) {
    const TileGeom tg = tile_geom<BIN>(tile, views, n_views);
    const ViewInfo& V = views[tg.vloc];
    // view fields read once (plain values: the conditions below need no branch)
    const int vw = V.width, vh = V.height;
    const int64_t poff = V.pixel_offset;
    const uint32_t n16 = lane & 15, q4 = lane >> 4;

    uint2 rg = ranges[tg.bin];
    rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
    rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
    if (rg.x >= rg.y) return 0;
    // targets of the tile as B operands: Y[s][b] holds the eight pixels of
    // row 4 (s & 1) + q4 of block s / 2, channel c_off + 16 b + n16
    bf16x8_t Y[8][NBLK];
    // packed forms: the channel this lane's column reads, and its role
    const int pc = YM == 2 ? ((int)n16 < C ? (int)n16 : (int)n16 - C) : (int)n16;
    const bool pcol = YM == 2 ? (int)n16 < 2 * C : (int)n16 < C;   // a target column
    const bool pone = YM == 2 ? (int)n16 == 2 * C : (int)n16 == C;  // the ones column
    // Rows, columns and channels past the end read the nearest pixel of the
    // tile and the last channel instead: those pixels have weight 0
    // and those columns are not stored, so no value needs a mask (the masks of
    // 64-128 loads were spilled scalar registers).  Offsets from the tile's
    // first row fit 32 bits (16 image rows hold at most 2^25 values).
    using TY = std::conditional_t<YM == 2, float, uint16_t>;
    const int yb = min(tg.y0, vh - 1);
    const TY* trow = (const TY*)targets + (poff + (int64_t)yb * vw) * C;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const int gy = min(tg.y0 + 8 * (s >> 2) + 4 * (s & 1) + (int)q4, vh - 1);
        const int gx0 = tg.x0 + 8 * ((s >> 1) & 1);
        const uint32_t ro = (uint32_t)(gy - yb) * (uint32_t)vw * (uint32_t)C;
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            const uint32_t vo = ro + (uint32_t)(YM == 0 ? min(c_off + 16 * b + (int)n16, C - 1) : (pcol ? pc : 0));
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const TY x = (trow + (int64_t)min(gx0 + i, vw - 1) * C)[vo];
                if constexpr (YM == 2) {
                    const __bf16 hi = (__bf16)x;
                    const __bf16 v = (int)n16 < C ? hi : (__bf16)(x - (float)hi);
                    Y[s][b][i] = pone ? (__bf16)1.0f : v;
                } else {
                    const __bf16 v = __builtin_bit_cast(__bf16, x);
                    Y[s][b][i] = (YM == 1 && pone) ? (__bf16)1.0f : v;
                }
            }
        }
    }
    // the ones operand, each register made through an identity DPP move so
    // that the compiler holds it instead of rebuilding it before every product
    bf16x8_t ones;
    {
        uint32_t o4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o4[i] = (uint32_t)__builtin_amdgcn_mov_dpp(0x3F803F80, 0xE4, 0xF, 0xF, true);
        ones = __builtin_bit_cast(bf16x8_t, o4);
    }

    // transmittance of the lane's pixel in each block: four scalars (as an
    // array the compiler rebuilt it in new registers on every block update)
    float T0, T1, T2, T3;
    uint32_t alive = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool inside = (tg.x0 + block_px(lane, k) < vw) & (tg.y0 + block_py(lane, k) < vh);
        const float t = inside ? 1.0f : kOutsideT;
        if (k == 0) T0 = t;
        if (k == 1) T1 = t;
        if (k == 2) T2 = t;
        if (k == 3) T3 = t;
        alive |= (__builtin_amdgcn_ballot_w64(inside) != 0 ? 1u : 0u) << k;
    }
    alive = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive);
    uint32_t cnt = 0;
    const int64_t item_base = V.item_base;
    const int64_t slot_base = per_view ? V.vs_base : V.g_offset;
    const int64_t g_off = V.g_offset;
    const bool first_chunk = c_off == 0;
    // loop constants in vector registers (see uniform_in_vgpr)
    const float qlim = uniform_in_vgpr((float)(kExp2Scale * (double)bp.cut2));
    const float amax = uniform_in_vgpr(bp.alpha_max), amin = uniform_in_vgpr(bp.alpha_min),
                tmin = uniform_in_vgpr(bp.t_min);
    // the lane's pixel offsets from the tile's centre point; R0 below keeps,
    // per entry, the offset of that point from the projected centre
    const float lx[2] = {tile_offset_col(lane, 0), tile_offset_col(lane, 1)};
    const float ly[2] = {tile_offset_row(lane, 0), tile_offset_row(lane, 1)};
    const float ox = tile_centre(tg.x0), oy = tile_centre(tg.y0);

    // Rows are never cleared: rows past a group's count feed only output rows
    // that the flush does not use, and an entry writes zeros in the blocks its
    // footprint misses (measured faster than per-row masks that zero
    // the operand in the flush, for one and for two channel blocks).

    // one matrix product over the group's `rows` entries, then the atomics.
    // The A operand's rows 0..7 take the weights' high parts and rows 8..15
    // their remainders, so one product per K-step forms both halves; each
    // output row then adds its two halves (lanes l and l + 32).
    auto flush = [&](uint32_t rows) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        floatx4_t D[NBLK], DV;
#pragma unroll
        for (int b = 0; b < NBLK; ++b) D[b] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        DV = floatx4_t{0.f, 0.f, 0.f, 0.f};
        const __bf16* ah_p = &(n16 >= 8u ? L.wlo : L.whi)[(n16 & 7u) * kWRow + 8 * q4];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const bf16x8_t ah = *reinterpret_cast<const bf16x8_t*>(ah_p + 32 * s);
            if (YM == 0 && first_chunk) DV = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, ones, DV, 0, 0, 0);
#pragma unroll
            for (int b = 0; b < NBLK; ++b) D[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, Y[s][b], D[b], 0, 0, 0);
        }
        // Lane l adds the halves of rows 4 (q4 & 1) + i, column n16: lanes 0..31
        // of the first channel block, lanes 32..63 of the second or of V (three
        // scenes, 16 channels: 3.53 -> 3.42 ms against LDS shuffles and twice the
        // atomic instructions).
        const uint32_t half = lane >> 5;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t m = 4 * (q4 & 1u) + (uint32_t)i;
            float x, v = 0.0f, lo = 0.0f;
            if constexpr (YM != 0) {
                x = sum_xor32(D[0][i]);
                if constexpr (YM == 2) lo = __shfl(x, (int)lane + C, 64);  // remainder column
            } else if constexpr (NBLK == 1) {
                x = fold_halves(D[0][i], DV[i]);
            } else {
                x = fold_halves(D[0][i], D[1][i]);
                if (first_chunk) v = sum_xor32(DV[i]);
            }
            const uint32_t gl = L.gslot[m];
            if (m >= rows || gl == 0xFFFFFFFFu) continue;
            float* srow = out.s + (slot_base + (int64_t)gl) * (int64_t)out.s_stride;
            float* vsum = out.v + (slot_base + (int64_t)gl) * (int64_t)out.v_stride;
            if constexpr (YM != 0) {
                if (half != 0u) continue;
                if (pone) unsafeAtomicAdd(vsum, x);
                else if ((int)n16 < C) unsafeAtomicAdd(srow + n16, x + lo);
            } else if constexpr (NBLK == 1) {
                const int c = c_off + (int)n16;
                const bool put = half == 0u ? c < C : first_chunk && n16 == 0;
                if (put) unsafeAtomicAdd(half == 0u ? srow + c : vsum, x);
            } else {
                const int c = c_off + 16 * (int)half + (int)n16;
                if (c < C) unsafeAtomicAdd(srow + c, x);
                if (first_chunk && lane == (lane & 16u)) unsafeAtomicAdd(vsum, v);
            }
        }
        // the next group overwrites these rows
        __builtin_amdgcn_wave_barrier();
    };

    // list walk: chunks of 64 entries gathered one per lane; each lane also
    // forms its entry's block mask (the live blocks its footprint reaches),
    // so taking an entry costs one broadcast of that mask; the entries that
    // reach a live block are taken in order
    constexpr bool kLdsCentre = NBLK == 1;
    uint32_t rows = 0;
    for (uint32_t b = rg.x; b < rg.y && alive != 0u; b += 64) {
        const bool in_list = b + lane < rg.y;
        const uint32_t pv = in_list ? pair_vals[b + lane] : 0u;
        const uint32_t it = pv & kItemMask;
        const bool own = in_list && pair_reaches<BIN>(pv, tg.quad, alive);
        const float4 r = own ? rec[2 * (size_t)it] : make_float4(0.f, 0.f, 0.f, 0.f);
        const float2 R0 = make_float2((ox - r.x) - r.z, (oy - r.y) - r.w);
        const float4 R1 = own ? rec[2 * (size_t)it + 1] : make_float4(0.f, 0.f, 0.f, 0.f);
        const uint32_t gid = own ? items[it] : 0u;  // the entry's item
        const uint32_t BL = own ? (entry_blocks<BIN>(pv, R0, R1, bp) & alive) : 0u;
        uint64_t sm = __builtin_amdgcn_ballot_w64(BL != 0u);  // entries still to take
        // the records go through LDS: an entry then reads them with one
        // broadcast load each instead of a readlane per value (measured:
        // the centre offset too for one channel block, 5.52 -> 5.43 ms per
        // launch on the 32-scene plan; the conic and opacity only for two,
        // 8.18 -> 7.99 ms on the feature workload)
        L.crec1[lane] = R1;
        if constexpr (kLdsCentre) L.crec0[lane] = R0;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        while (sm != 0u) {
            const uint32_t j = (uint32_t)__builtin_ctzll(sm);
            sm &= sm - 1;
            const uint32_t blocks = bcast_u(BL, j) & alive;
            if (blocks == 0u) continue;
            const float2 c0 = kLdsCentre ? L.crec0[j] : make_float2(bcast(R0.x, j), bcast(R0.y, j));
            const float4 c1 = L.crec1[j];
            const float dx[2] = {c0.x + lx[0], c0.x + lx[1]}, dy[2] = {c0.y + ly[0], c0.y + ly[1]};
            const float a0[2] = {c1.x * dx[0] * dx[0], c1.x * dx[1] * dx[1]};
            const float b0[2] = {c1.y * dx[0], c1.y * dx[1]};
            uint32_t nh = 0;
            __bf16* wrow_h = &L.whi[rows * kWRow];
            __bf16* wrow_l = &L.wlo[rows * kWRow];
            auto step = [&](const int k, float& Tk) {
                if (!((blocks >> k) & 1u)) {  // uniform: no weight in this block
                    wrow_h[lane + 64 * k] = (__bf16)0.0f;
                    wrow_l[lane + 64 * k] = (__bf16)0.0f;
                    return;
                }
                const float q2 = fmaf(dy[k >> 1], fmaf(c1.z, dy[k >> 1], b0[k & 1]), a0[k & 1]);
                uint64_t taken, kept;
                const float w = pixel_step(q2, c1.w, Tk, qlim, amin, amax, tmin, taken, kept);
                // hi: w's upper half (truncated), lo: the exact remainder rounded
                // to BF16; |w - hi - lo| <= 2^-16 |w|
                const uint32_t wb = __float_as_uint(w);
                const __bf16 hi = __builtin_bit_cast(__bf16, (uint16_t)(wb >> 16));
                const __bf16 lo = (__bf16)(w - __uint_as_float(wb & 0xffff0000u));
                wrow_h[lane + 64 * k] = hi;
                wrow_l[lane + 64 * k] = lo;
                nh += (uint32_t)__popcll(taken);
                if (kept == 0) alive &= ~(1u << k);
            };
            step(0, T0);
            step(1, T1);
            step(2, T2);
            step(3, T3);
            alive = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive);
            nh = (uint32_t)__builtin_amdgcn_readfirstlane((int)nh);
            cnt += nh;
            const uint32_t gl = (uint32_t)((int64_t)bcast_u(gid, j) - item_base);
            if (lane == 0) L.gslot[rows] = nh != 0u ? gl : 0xFFFFFFFFu;
            if (nh != 0u && gcount != nullptr && first_chunk && lane == 0) atomicAdd(gcount + g_off + gl, nh);
            if (++rows == (uint32_t)kMfmaRows) {
                flush(rows);
                rows = 0;
            }
            if (alive == 0u) break;
        }
        __builtin_amdgcn_wave_barrier();  // the next chunk's records overwrite these
    }
    if (rows != 0u) flush(rows);
    return cnt;
}

template <int NBLK, int BIN, int YM>
__global__ __launch_bounds__(64 * kMfmaWaves)
__attribute__((amdgpu_waves_per_eu(mfma_waves_per_simd<NBLK>()))) void k_accumulate_mfma(
    const ViewInfo* __restrict__ views, int n_views, uint32_t n_tiles, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ pair_vals, const float4* __restrict__ rec,
    const uint32_t* __restrict__ items,
    const void* __restrict__ targets, int C, int c_off, int per_view, BlendParams bp,
    SumRows out, unsigned long long* __restrict__ counter, uint32_t* __restrict__ gcount,
    uint32_t* __restrict__ queue, const uint32_t* __restrict__ order) {
    __shared__ MfmaLds lds[kMfmaWaves];
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t cnt = 0;
    if (queue == nullptr) {
        const uint32_t wi = xcd_block(blockIdx.x, gridDim.x) * kMfmaWaves + w;
        if (wi >= n_tiles) return;  // whole wave
        const uint32_t tile = queued_tile<BIN>(wi, order);  // blocks start in index order
        cnt = accumulate_tile_mfma<NBLK, BIN, YM>(tile, lane, lds[w], views, n_views, ranges, pair_vals,
                                              rec, items, targets, C, c_off, per_view, bp, out,
                                              gcount);
    } else {
        for (;;) {
            uint32_t t = 0;
            if (lane == 0) t = atomicAdd(queue, 1u);
            const uint32_t tq = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
            if (tq >= n_tiles) break;  // uniform: every wave ends here
            const uint32_t tile = queued_tile<BIN>(tq, order);
            cnt += accumulate_tile_mfma<NBLK, BIN, YM>(tile, lane, lds[w], views, n_views, ranges,
                                                   pair_vals, rec, items, targets, C, c_off,
                                                   per_view, bp, out, gcount);
        }
    }
    if (c_off == 0 && lane == 0 && cnt) atomicAdd(counter, (unsigned long long)cnt);
}

template <int NBLK, int BIN, int YM>
static void launch_acc_mfma(const TileLists& tl, const void* targets, int C, bool per_view, BlendParams bp,
                            const SumRows& out, unsigned long long* counter, uint32_t* gcount, uint32_t* queues,
                            hipStream_t s) {
    const uint32_t n_wt = wave_tiles(tl.n_bins, BIN);
    const uint32_t full = (n_wt + kMfmaWaves - 1) / kMfmaWaves;
    dim3 grid(queues ? std::min(full, 2 * kPersistentBlocks) : full), block(64 * kMfmaWaves);
    int pass = 0;
    const int step = YM == 0 ? 16 * NBLK : C;  // packed forms: one launch
    for (int c_off = 0; c_off < C; c_off += step, ++pass) {
        uint32_t* q = queues ? queues + pass : nullptr;
        hipLaunchKernelGGL((k_accumulate_mfma<NBLK, BIN, YM>), grid, block, 0, s, tl.views, tl.n_views,
                           n_wt, tl.ranges, tl.pair_vals, tl.rec, tl.items, targets, C, c_off,
                           (int)per_view, bp, out, counter, gcount, q, tl.order);
    }
}

template <int NBLK, int YM>
static void launch_acc_mfma_bin(const TileLists& tl, const void* targets, int C, bool per_view,
                                BlendParams bp, const SumRows& out, unsigned long long* counter,
                                uint32_t* gcount, uint32_t* queues, hipStream_t s) {
    if (tl.bin == 32)
        launch_acc_mfma<NBLK, 32, YM>(tl, targets, C, per_view, bp, out, counter, gcount, queues, s);
    else
        launch_acc_mfma<NBLK, 16, YM>(tl, targets, C, per_view, bp, out, counter, gcount, queues, s);
}

// ---- 33 to 64 channels: one block per tile --------------------------------
//
// The block's four waves share a group's weight rows.  Each blends one 8x8 block
// of the tile (every pixel's weights once, where two launches of the form above
// form them twice) and multiplies the rows of all 256 pixels by 16 channels of
// its own, held as B operands in 32 registers (one wave with all 64 channels
// needs 128 and runs alone on its SIMD).  The list is gathered 256 entries at a
// time, one a thread, and those that reach a live block are put together in
// LDS in list order; groups of 16 of them share a barrier between the blend and
// the product.  A Gaussian's sums leave the tile once: splitting the tile's
// pixels over independent waves (16x8 or 8x8 pixels by 64 channels each) was
// bound by the atomics instead (25 and 44 ms; see SumRows).
// 500k Gaussians, 100 views of 960x540, 64 channels: 15.9 ms in two launches of
// 32 channels -> 8.85 ms, near the rate of the atomics (142 M requests).  Held to
// 80 registers, six blocks a CU: 8.85 ms, 96: 8.97, 125: 9.66.
constexpr int kWideRows = 16;
struct alignas(16) WideLds {
    __bf16 whi[kWideRows * kWRow];
    __bf16 wlo[kWideRows * kWRow];
    float4 rec1[256];      // the chunk's entries: conic and opacity,
    float2 rec0[256];      // offset of the tile's centre point from the centre,
    uint32_t gid[256];     // local Gaussian,
    uint32_t blocks[256];  // blocks reached
    uint32_t count[4];     // entries each wave put in
    uint32_t hit[4];       // rows of the group that got weight in each block
    uint32_t live[4];      // block has live pixels
    uint32_t next;         // tile taken from the queue
};

template <int BIN>
__device__ __forceinline__ uint32_t accumulate_tile_wide(
    uint32_t tile, uint32_t lane, uint32_t wave, WideLds& L, const ViewInfo* __restrict__ views, int n_views,
    const uint2* __restrict__ ranges, const uint32_t* __restrict__ pair_vals, const float4* __restrict__ rec,
    const uint32_t* __restrict__ items, const uint16_t* __restrict__ targets, int C, int per_view,
    const BlendParams& bp, const SumRows& out, uint32_t* __restrict__ gcount) {
    const TileGeom tg = tile_geom<BIN>(tile, views, n_views);
    const ViewInfo& V = views[tg.vloc];
    uint2 rg = ranges[tg.bin];
    rg.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.x);
    rg.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)rg.y);
    if (rg.x >= rg.y) return 0;  // the same for every wave
    const int vw = V.width, vh = V.height;
    const int64_t item_base = V.item_base, g_off = V.g_offset;
    const int64_t slot_base = per_view ? V.vs_base : V.g_offset;
    const uint32_t n16 = lane & 15, q4 = lane >> 4;
    const int c = 16 * (int)wave + (int)n16;

    // targets: as in the form above (nearest pixel, last channel past the ends)
    bf16x8_t Y[8];
    {
        const int yb = min(tg.y0, vh - 1);
        const uint16_t* trow = targets + (V.pixel_offset + (int64_t)yb * vw) * C;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int gy = min(tg.y0 + 8 * (s >> 2) + 4 * (s & 1) + (int)q4, vh - 1);
            const int gx0 = tg.x0 + 8 * ((s >> 1) & 1);
            const uint32_t vo = (uint32_t)(gy - yb) * (uint32_t)vw * (uint32_t)C + (uint32_t)min(c, C - 1);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                Y[s][i] = __builtin_bit_cast(__bf16, (trow + (int64_t)min(gx0 + i, vw - 1) * C)[vo]);
        }
    }
    bf16x8_t ones;
    {
        uint32_t o4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o4[i] = (uint32_t)__builtin_amdgcn_mov_dpp(0x3F803F80, 0xE4, 0xF, 0xF, true);
        ones = __builtin_bit_cast(bf16x8_t, o4);
    }
    const float ox = tile_centre(tg.x0), oy = tile_centre(tg.y0);
    const float lx = tile_offset_col(lane, (int)(wave & 1u)), ly = tile_offset_row(lane, (int)(wave >> 1));
    const float qlim = uniform_in_vgpr((float)(kExp2Scale * (double)bp.cut2));
    const float amax = uniform_in_vgpr(bp.alpha_max), amin = uniform_in_vgpr(bp.alpha_min),
                tmin = uniform_in_vgpr(bp.t_min);
    uint32_t alive = 0;  // blocks of the tile with pixels inside the image
#pragma unroll
    for (int k = 0; k < 4; ++k)
        alive |= (tg.x0 + 8 * (k & 1) < vw && tg.y0 + 8 * (k >> 1) < vh ? 1u : 0u) << k;
    float T = (tg.x0 + block_px(lane, (int)wave) < vw) & (tg.y0 + block_py(lane, (int)wave) < vh) ? 1.0f : kOutsideT;
    bool live = ((alive >> wave) & 1u) != 0u;
    uint32_t cnt = 0, turn = 0;
    uint32_t dirty = 0xFFFFu;  // rows whose weights of this block may be other than zero
    __bf16* wh = &L.whi[64 * wave + lane];
    __bf16* wl = &L.wlo[64 * wave + lane];

    for (uint32_t b = rg.x; b < rg.y && alive != 0u; b += 256) {
        const uint32_t e = b + 64 * wave + lane;
        const bool in_list = e < rg.y;
        const uint32_t pv = in_list ? pair_vals[e] : 0u;
        const uint32_t it = pv & kItemMask;
        const bool own = in_list && pair_reaches<BIN>(pv, tg.quad, alive);
        const float4 r = own ? rec[2 * (size_t)it] : make_float4(0.f, 0.f, 0.f, 0.f);
        const float2 R0 = make_float2((ox - r.x) - r.z, (oy - r.y) - r.w);
        const float4 R1 = own ? rec[2 * (size_t)it + 1] : make_float4(0.f, 0.f, 0.f, 0.f);
        const uint32_t gid = own ? items[it] : 0u;
        const uint32_t BL = own ? (entry_blocks<BIN>(pv, R0, R1, bp) & alive) : 0u;
        const uint64_t put = __builtin_amdgcn_ballot_w64(BL != 0u);
        if (lane == 0) {
            L.count[wave] = (uint32_t)__popcll(put);
            L.live[wave] = live ? 1u : 0u;
        }
        __syncthreads();  // the counts; the last chunk's entries are done with
        uint32_t n = 0, at = 0;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t x = L.count[k];
            at += k < wave ? x : 0u;
            n += x;
        }
        n = (uint32_t)__builtin_amdgcn_readfirstlane((int)n);
        if (BL != 0u) {
            at += __builtin_amdgcn_mbcnt_hi((uint32_t)(put >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)put, 0u));
            L.rec1[at] = R1;
            L.rec0[at] = R0;
            L.gid[at] = (uint32_t)((int64_t)gid - item_base);
            L.blocks[at] = BL;
        }
        __syncthreads();  // the entries
        for (uint32_t g = 0; g < n; g += kWideRows) {
            const uint32_t rows = min((uint32_t)kWideRows, n - g);
            const uint32_t bl = lane < rows ? L.blocks[g + lane] : 0u;
            uint32_t todo = live ? (uint32_t)__builtin_amdgcn_ballot_w64(((bl >> wave) & 1u) != 0u) : 0u;
            uint32_t hit = 0, zero = dirty & ~todo;
            dirty = todo;
            while (zero != 0u) {
                const uint32_t m = (uint32_t)__builtin_ctz(zero);
                zero &= zero - 1u;
                wh[m * kWRow] = (__bf16)0.0f;
                wl[m * kWRow] = (__bf16)0.0f;
            }
            while (todo != 0u) {
                const uint32_t m = (uint32_t)__builtin_ctz(todo);
                todo &= todo - 1u;
                const float2 c0 = L.rec0[g + m];
                const float4 c1 = L.rec1[g + m];
                const float dx = c0.x + lx, dy = c0.y + ly;
                const float q2 = fmaf(dy, fmaf(c1.z, dy, c1.y * dx), c1.x * dx * dx);
                uint64_t taken, kept;
                const float w = pixel_step(q2, c1.w, T, qlim, amin, amax, tmin, taken, kept);
                const uint32_t wb = __float_as_uint(w);
                wh[m * kWRow] = __builtin_bit_cast(__bf16, (uint16_t)(wb >> 16));
                wl[m * kWRow] = (__bf16)(w - __uint_as_float(wb & 0xffff0000u));
                const uint32_t nh = (uint32_t)__popcll(taken);
                cnt += nh;
                hit |= (nh != 0u ? 1u : 0u) << m;
                if (nh != 0u && gcount != nullptr && lane == 0) atomicAdd(gcount + g_off + L.gid[g + m], nh);
                live = kept != 0;
            }
            // (a block that has stopped gives zero weights from then on)
            if (lane == 0) {
                L.hit[wave] = hit;
                L.live[wave] = live ? 1u : 0u;
            }
            __syncthreads();  // the rows
            const uint32_t hits = (uint32_t)__builtin_amdgcn_readfirstlane((int)(L.hit[0] | L.hit[1] | L.hit[2] | L.hit[3]));
            if (hits != 0u) {
                const bool vturn = turn == wave;  // the waves form V in turn
                turn = (turn + 1u) & 3u;
                floatx4_t D = {0.f, 0.f, 0.f, 0.f}, E = D, DV = D;
                const __bf16* ah_p = &L.whi[n16 * kWRow + 8 * q4];
                const __bf16* al_p = &L.wlo[n16 * kWRow + 8 * q4];
#pragma unroll
                for (int s = 0; s < 8; ++s) {
                    const bf16x8_t ah = *reinterpret_cast<const bf16x8_t*>(ah_p + 32 * s);
                    const bf16x8_t al = *reinterpret_cast<const bf16x8_t*>(al_p + 32 * s);
                    D = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, Y[s], D, 0, 0, 0);
                    E = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, Y[s], E, 0, 0, 0);
                    if (vturn) {
                        DV = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, ones, DV, 0, 0, 0);
                        DV = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, ones, DV, 0, 0, 0);
                    }
                }
                // lane holds rows 4 q4 + i, column n16
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t m = 4 * q4 + (uint32_t)i;
                    if (!((hits >> m) & 1u)) continue;
                    const int64_t slot = slot_base + (int64_t)L.gid[g + m];
                    if (c < C) unsafeAtomicAdd(out.s + slot * out.s_stride + c, D[i] + E[i]);
                    if (vturn && n16 == 0) unsafeAtomicAdd(out.v + slot * out.v_stride, DV[i]);
                }
            }
            __syncthreads();  // the rows and the flags are done with
        }
        alive = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) alive |= L.live[k] << k;
        alive = (uint32_t)__builtin_amdgcn_readfirstlane((int)alive);
    }
    return cnt;
}

template <int BIN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_accumulate_wide(
    const ViewInfo* __restrict__ views, int n_views, uint32_t n_tiles, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ pair_vals, const float4* __restrict__ rec, const uint32_t* __restrict__ items,
    const uint16_t* __restrict__ targets, int C, int per_view, BlendParams bp, SumRows out,
    unsigned long long* __restrict__ counter, uint32_t* __restrict__ gcount, uint32_t* __restrict__ queue,
    const uint32_t* __restrict__ order) {
    __shared__ WideLds L;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint32_t cnt = 0;
    if (queue == nullptr) {
        const uint32_t tile = queued_tile<BIN>(xcd_block(blockIdx.x, gridDim.x), order);
        cnt = accumulate_tile_wide<BIN>(tile, lane, wave, L, views, n_views, ranges, pair_vals, rec, items, targets,
                                        C, per_view, bp, out, gcount);
    } else {
        for (;;) {
            if (threadIdx.x == 0) L.next = atomicAdd(queue, 1u);
            __syncthreads();
            const uint32_t tq = (uint32_t)__builtin_amdgcn_readfirstlane((int)L.next);
            if (tq >= n_tiles) break;  // the same for every wave
            cnt += accumulate_tile_wide<BIN>(queued_tile<BIN>(tq, order), lane, wave, L, views, n_views, ranges,
                                             pair_vals, rec, items, targets, C, per_view, bp, out, gcount);
            __syncthreads();  // the number is read, the tile's entries are done with
        }
    }
    if (lane == 0 && cnt) atomicAdd(counter, (unsigned long long)cnt);
}

template <int BIN>
static void launch_acc_wide(const TileLists& tl, const void* targets, int C, bool per_view, BlendParams bp,
                            const SumRows& out, unsigned long long* counter, uint32_t* gcount, uint32_t* queues,
                            hipStream_t s) {
    const uint32_t n_wt = wave_tiles(tl.n_bins, BIN);
    dim3 grid(queues ? std::min(n_wt, kPersistentBlocks) : n_wt), block(256);
    hipLaunchKernelGGL(k_accumulate_wide<BIN>, grid, block, 0, s, tl.views, tl.n_views, n_wt, tl.ranges,
                       tl.pair_vals, tl.rec, tl.items, (const uint16_t*)targets, C, (int)per_view, bp, out, counter,
                       gcount, queues, tl.order);
}

int accumulate_chunk(int C, int tdtype) {
    if (tdtype == GSC_BF16 && C >= 16) return kChunkMfma | (C <= 16 ? 16 : C <= 32 ? 32 : 64);
    return C <= 3 ? C : (C <= 4 ? 4 : (C <= 8 ? 8 : 16));
}

int resolve_chunk(int requested, int C, int tdtype) {
    if (!accumulate_chunk_valid(requested, tdtype)) return accumulate_chunk(C, tdtype);
    if (requested == kChunkPacked && C > (tdtype == GSC_BF16 ? 15 : 7)) return accumulate_chunk(C, tdtype);
    return requested;
}

bool accumulate_chunk_valid(int chunk, int tdtype) {
    if (chunk & kChunkMfma) {
        const int ch = chunk_channels(chunk);
        if (chunk != (kChunkMfma | ch)) return false;
        if (ch == 1) return true;  // packed form; fits_packed() checks C
        return tdtype == GSC_BF16 && (ch == 16 || ch == 32 || ch == 64);
    }
    return chunk == 1 || chunk == 2 || chunk == 3 || chunk == 4 || chunk == 8 || chunk == 16;
}

// Channels that the next launch of the form for few tiles takes of C that are left
// (a power of two of values an entry, with its weight).
static int block_channels(int C) { return C <= 3 ? 3 : (C <= 7 ? 7 : 15); }

AccumulateForm accumulate_form(const TileLists& tl, int C, int chunk, bool deterministic, bool persistent) {
    if (deterministic && (chunk & kChunkMfma)) chunk = accumulate_chunk(C, GSC_F32);  // vector form only
    const bool blocks = !deterministic && !persistent && few_tiles(tl) && chunk == accumulate_chunk(C, GSC_F32);
    const int ch = blocks ? block_channels(C) : chunk_channels(chunk);
    return AccumulateForm{chunk, blocks, chunk == kChunkPacked ? 1 : (C + ch - 1) / ch};
}

void launch_accumulate(const TileLists& tl, const void* targets, int tdtype, int C, bool per_view,
                       BlendParams bp, float* VS, unsigned long long* counter, uint32_t* gcount,
                       int chunk, hipStream_t s, uint32_t* queues, const float2* det, int64_t split_n) {
    if (tl.n_bins == 0) return;
    const AccumulateForm form = accumulate_form(tl, C, resolve_chunk(chunk, C, tdtype), det != nullptr, queues != nullptr);
    chunk = form.chunk;
    if (form.blocks) {
#define GSC_ACCB(CCV)                                                                                    \
    do {                                                                                                 \
        if (tdtype == GSC_BF16) launch_acc_blocks<CCV, true>(tl, targets, C, c_off, per_view, bp, VS, counter, gcount, s); \
        else launch_acc_blocks<CCV, false>(tl, targets, C, c_off, per_view, bp, VS, counter, gcount, s); \
    } while (0)
        // (the last launch as narrow as the channels that are left: 16 channels of
        // 4 views of 512x512, 100k splats, 641 us a call with two launches of 15,
        // 569 with 15 and 3; the tile form, in one launch, 556, at 2 views 510
        // against 394)
        for (int c_off = 0; c_off < C; c_off += block_channels(C - c_off)) {
            switch (block_channels(C - c_off)) {
                case 3: GSC_ACCB(3); break;
                case 7: GSC_ACCB(7); break;
                default: GSC_ACCB(15); break;
            }
        }
#undef GSC_ACCB
        return;
    }
    if (queues) launch_fill_u32(queues, 0u, (uint64_t)form.launches, s);
    if (chunk & kChunkMfma) {
        const SumRows rows = sum_rows(VS, C, split_n);
#define GSC_ACCM(NB, YMV) \
    launch_acc_mfma_bin<NB, YMV>(tl, targets, C, per_view, bp, rows, counter, gcount, queues, s)
        switch (chunk_channels(chunk)) {
            case 1:
                if (tdtype == GSC_BF16) GSC_ACCM(1, 1); else GSC_ACCM(1, 2);
                break;
            case 16: GSC_ACCM(1, 0); break;
            case 32: GSC_ACCM(2, 0); break;
            default:
                if (tl.bin == 32) launch_acc_wide<32>(tl, targets, C, per_view, bp, rows, counter, gcount, queues, s);
                else launch_acc_wide<16>(tl, targets, C, per_view, bp, rows, counter, gcount, queues, s);
                break;
        }
#undef GSC_ACCM
        return;
    }
#define GSC_ACC(CCV) \
    launch_acc_cc<CCV>(tl, targets, tdtype, C, per_view, bp, VS, counter, gcount, queues, s, det)
    switch (chunk) {
        case 1: GSC_ACC(1); break;
        case 2: GSC_ACC(2); break;
        case 3: GSC_ACC(3); break;
        case 4: GSC_ACC(4); break;
        case 8: GSC_ACC(8); break;
        default: GSC_ACC(16); break;
    }
#undef GSC_ACC
}

void launch_accumulate_weights(const TileLists& tl, bool per_view, BlendParams bp, float* V,
                               unsigned long long* counter, hipStream_t s) {
    if (tl.n_bins == 0) return;
    if (few_tiles(tl)) {
        launch_acc_blocks<0, false>(tl, nullptr, 0, 0, per_view, bp, V, counter, nullptr, s);
        return;
    }
    if (tl.bin == 32)
        launch_acc_k<0, false, 32>(tl, nullptr, 0, per_view, bp, V, counter, nullptr, nullptr, s);
    else
        launch_acc_k<0, false, 16>(tl, nullptr, 0, per_view, bp, V, counter, nullptr, nullptr, s);
}

}  // namespace gsc
