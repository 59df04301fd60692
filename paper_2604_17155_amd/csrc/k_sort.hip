// Device-wide exclusive scan and stable LSD radix sort (digits of up to 8 bits).
//
// The sorts order each view's items by depth and then the emitted (group, item)
// pairs by group of 4x4 bins.  Stability of every pass is what carries the depth
// order (and the index tie-break) into each group's, and so each bin's, list.
#include <algorithm>

#include "gsc_internal.h"

namespace gsc {

namespace {
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanBlock = kScanThreads * kScanItems;  // 2048

constexpr int kRsThreads = 512;
constexpr int kRsItems = 16;
constexpr int kRsTile = kRsThreads * kRsItems;  // 8192: runs of ~32 keys per digit
constexpr int kRsWaves = kRsThreads / 64;

// Sums that stay at 2^32 - 1 instead of wrapping (one instruction, as the plain sum).
// The pairs of a plan's run are not counted before they are placed; if its geometry
// has grown until they pass 32 bits, offsets past the end have to stay past it.
__device__ __forceinline__ uint32_t add_sat(uint32_t a, uint32_t b) { return __builtin_elementwise_add_sat(a, b); }

__device__ inline uint32_t wave_inclusive_scan(uint32_t v) {
    int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t o = __shfl_up(v, d, 64);
        if (lane >= d) v = add_sat(v, o);
    }
    return v;
}

// Exclusive scan over the NT threads of a block; returns the block total in *total.
template <int NT = kScanThreads>
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t* wsum, uint32_t* total) {
    int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = wave_inclusive_scan(v);
    if (lane == 63) wsum[w] = inc;
    uint32_t exc = __shfl_up(inc, 1, 64);
    if (lane == 0) exc = 0u;
    __syncthreads();
    uint32_t off = 0, all = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) {
        uint32_t s = wsum[k];
        if (k < w) off = add_sat(off, s);
        all = add_sat(all, s);
    }
    *total = all;
    __syncthreads();
    return add_sat(off, exc);
}
// The kScanItems = 8 consecutive elements at base: two 16-byte loads when
// they all lie below n and the array is 16-byte aligned, else one guarded
// load each (zero past the end).
__device__ inline void scan_load8(const uint32_t* in, uint64_t base, uint32_t n, uint32_t* x) {
    if (base + kScanItems <= n && (reinterpret_cast<uintptr_t>(in) & 15u) == 0) {
        const uint4 a = *reinterpret_cast<const uint4*>(in + base);
        const uint4 b = *reinterpret_cast<const uint4*>(in + base + 4);
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
        x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
    } else {
#pragma unroll
        for (int j = 0; j < kScanItems; ++j) x[j] = base + j < n ? in[base + j] : 0u;
    }
}
}  // namespace

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const uint32_t* __restrict__ in,
                                                              uint32_t n, uint32_t* __restrict__ bsums) {
    __shared__ uint32_t wsum[kScanThreads / 64];
    uint64_t base = (uint64_t)blockIdx.x * kScanBlock + (uint64_t)threadIdx.x * kScanItems;
    uint32_t x[kScanItems];
    scan_load8(in, base, n, x);
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) s = add_sat(s, x[j]);
    uint32_t tot;
    block_exclusive_scan(s, wsum, &tot);
    if (threadIdx.x == 0) bsums[blockIdx.x] = tot;
}

// Down-sweep of one 2048-element block.  The block's offset is bsums[b] when
// the block sums have been scanned already; with `raw` they have not, and the
// block adds up bsums[0 .. b) itself (a few KB read from L2 for up to 2048
// blocks, in place of a launch that scans them).
__global__ __launch_bounds__(kScanThreads) void k_scan_down(const uint32_t* in, uint32_t* out,
                                                            uint32_t n, const uint32_t* bsums,
                                                            uint32_t* total, int raw) {
    __shared__ uint32_t wsum[kScanThreads / 64];
    uint32_t off = 0u;
    if (bsums && raw) {
        uint32_t part = 0u;
        for (uint32_t i = threadIdx.x; i < blockIdx.x; i += kScanThreads) part = add_sat(part, bsums[i]);
        block_exclusive_scan(part, wsum, &off);
    } else if (bsums) {
        off = bsums[blockIdx.x];
    }
    uint64_t base = (uint64_t)blockIdx.x * kScanBlock + (uint64_t)threadIdx.x * kScanItems;
    uint32_t x[kScanItems];
    scan_load8(in, base, n, x);
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) s = add_sat(s, x[j]);
    uint32_t tot;
    uint32_t pre = block_exclusive_scan(s, wsum, &tot);
    pre = add_sat(off, pre);
    if (base + kScanItems <= n && (reinterpret_cast<uintptr_t>(out) & 15u) == 0) {
        uint32_t y[kScanItems];
#pragma unroll
        for (int j = 0; j < kScanItems; ++j) {
            y[j] = pre;
            pre = add_sat(pre, x[j]);
        }
        *reinterpret_cast<uint4*>(out + base) = make_uint4(y[0], y[1], y[2], y[3]);
        *reinterpret_cast<uint4*>(out + base + 4) = make_uint4(y[4], y[5], y[6], y[7]);
    } else {
#pragma unroll
        for (int j = 0; j < kScanItems; ++j) {
            uint64_t idx = base + j;
            if (idx < n) out[idx] = pre;
            pre = add_sat(pre, x[j]);
        }
    }
    if (total && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total = add_sat(off, tot);
}

size_t scan_scratch_words(uint64_t n) {
    size_t w = 0;
    while (n > (uint64_t)kScanBlock) {
        n = (n + kScanBlock - 1) / kScanBlock;
        w += (size_t)((n + 63) / 64) * 64;
    }
    return w + 64;
}

void launch_scan(const uint32_t* in, uint32_t* out, uint32_t n, uint32_t* total, uint32_t* scratch,
                 hipStream_t s) {
    if (n == 0) {
        if (total) launch_fill_u32(total, 0u, 1, s);
        return;
    }
    if (n <= (uint32_t)kScanBlock) {
        hipLaunchKernelGGL(k_scan_down, dim3(1), dim3(kScanThreads), 0, s, in, out, n,
                           (const uint32_t*)nullptr, total, 0);
        return;
    }
    uint32_t nb = (n + kScanBlock - 1) / kScanBlock;
    uint32_t* bs = scratch;
    uint32_t* rest = scratch + ((nb + 63) / 64) * 64;
    hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kScanThreads), 0, s, in, n, bs);
    const int raw = nb <= (uint32_t)kScanBlock ? 1 : 0;
    if (!raw) launch_scan(bs, bs, nb, nullptr, rest, s);
    hipLaunchKernelGGL(k_scan_down, dim3(nb), dim3(kScanThreads), 0, s, in, out, n,
                       (const uint32_t*)bs, total, raw);
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t v, uint64_t n) {
    uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (; i < n; i += step) p[i] = v;
}

// Fill with a kernel rather than hipMemsetAsync so that the work stays
// ordinary kernel nodes if a caller captures the stream into a graph.
void launch_fill_u32(uint32_t* p, uint32_t v, uint64_t n, hipStream_t s) {
    if (n == 0) return;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, v, n);
}

// ---- radix sort ----------------------------------------------------------
//
// Sorts run over segments: the whole array, each view's items of a batch (the
// depth sort), or each view's pairs (the group sort; their places are known on
// the device alone).  A segment is cut into tiles of 512 * ITEMS keys, one block
// each; tile counters are laid out segment by segment, digit-major within one,
// so that a scan over all of them gives output positions.

// Where a sort's keys come from and how its segments lie.
struct SortSource {
    const uint32_t* keys;    // null: depth keys of the views' items (first pass)
    const uint32_t* vals;
    const ViewInfo* views;   // null: one segment
    int n_views;
    uint32_t view_tiles;     // tiles of every view when they are alike, else 0 (views[].sort_base)
    const float* means;
    const float* opac;
    float znear, alpha_min;
    // segments on the device (null: as above): seg[v] the first key of view v,
    // seg[n_views + 1 + v] its first tile, v = n_views the ends; keys count from
    // the view's first group
    const uint32_t* seg;
};
namespace {
// The tile a block works on.
struct SortTile {
    uint64_t begin, end;  // keys of the tile
    uint64_t seg;         // first key of the segment
    uint32_t j, nb;       // tile within the segment, tiles of the segment
    uint32_t first;       // tiles before the segment
    int view;
    uint32_t base;        // subtracted from the keys (0xFFFFFFFF: none)
};
template <int ITEMS>
__device__ inline SortTile sort_tile(const SortSource& S, uint32_t t, uint32_t n, uint32_t nblocks) {
    constexpr uint32_t kTileKeys = kRsThreads * ITEMS;
    SortTile T;
    T.base = 0xFFFFFFFFu;
    if (S.seg != nullptr) {
        const uint32_t* tf = S.seg + S.n_views + 1;
        int lo = 0, hi = S.n_views - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (tf[mid] <= t) lo = mid;
            else hi = mid - 1;
        }
        const uint32_t begin = S.seg[lo], end = S.seg[lo + 1];
        T.view = lo;
        T.seg = begin;
        T.first = tf[lo];
        T.j = t - T.first;
        T.nb = (end - begin + kTileKeys - 1) / kTileKeys;
        T.begin = T.seg + (uint64_t)T.j * kTileKeys;
        T.end = min(T.begin + kTileKeys, (uint64_t)end);  // a tile past the last view's is empty
        T.base = S.views[lo].group_base;
        return T;
    }
    if (S.views == nullptr) {
        T.view = 0;
        T.seg = 0;
        T.j = t;
        T.nb = nblocks;
        T.first = 0;
        T.begin = (uint64_t)t * kTileKeys;
        T.end = min(T.begin + kTileKeys, (uint64_t)n);
        return T;
    }
    int v;
    if (S.view_tiles != 0u) {
        v = (int)(t / S.view_tiles);
        T.first = (uint32_t)v * S.view_tiles;
    } else {
        int lo = 0, hi = S.n_views - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (S.views[mid].sort_base <= t) lo = mid;
            else hi = mid - 1;
        }
        v = lo;
        T.first = S.views[v].sort_base;
    }
    const ViewInfo& V = S.views[v];
    T.view = v;
    T.seg = V.item_base;
    T.j = t - T.first;
    T.nb = (V.n_gauss + kTileKeys - 1) / kTileKeys;
    T.begin = T.seg + (uint64_t)T.j * kTileKeys;
    T.end = min(T.begin + kTileKeys, T.seg + V.n_gauss);
    return T;
}
// Depth key of Gaussian g (index within the batch's arrays) in view V: the bits
// of the camera-space depth of the mean computed in binary32 (positive floats
// order like their bit patterns), 0xFFFFFFFF for items culled by the near plane
// or too faint to pass the alpha floor anywhere.
__device__ __forceinline__ uint32_t depth_key(const SortSource& S, const ViewInfo& V, uint64_t g) {
    const float key = __fmaf_rn(V.R[6], S.means[3 * g],
                                __fmaf_rn(V.R[7], S.means[3 * g + 1], __fmaf_rn(V.R[8], S.means[3 * g + 2], V.t[2])));
    return (key > S.znear && S.opac[g] >= S.alpha_min) ? __float_as_uint(key) : 0xFFFFFFFFu;
}
// (a view's groups lie below mask; clamped, as the digit indexes LDS)
__device__ __forceinline__ uint32_t sort_digit(const SortTile& T, uint32_t key, int shift, uint32_t mask) {
    return T.base != 0xFFFFFFFFu ? min(key - T.base, mask) : (key >> shift) & mask;
}
// Keys and values of a thread's places begin + it * step (the last key's past the end).
template <int ITEMS>
__device__ __forceinline__ void sort_load(const SortSource& S, const SortTile& T, uint64_t base, uint32_t step,
                                          uint32_t (&kk)[ITEMS], uint32_t* vv) {
    if (S.keys != nullptr) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const uint64_t i = min(base + (uint64_t)it * step, T.end - 1);
            kk[it] = S.keys[i];
            if (vv) vv[it] = S.vals[i];
        }
    } else {
        const ViewInfo& V = S.views[T.view];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const uint64_t i = min(base + (uint64_t)it * step, T.end - 1);
            kk[it] = depth_key(S, V, (uint64_t)V.g_offset + (i - T.seg));
            if (vv) vv[it] = (uint32_t)i;
        }
    }
}
}  // namespace

// Digit histogram of one tile, digit-major within its segment: counter
// first * digits + d * nb + j for the digits d <= mask of the pass
// ((key >> shift) & mask).  n_dev (optional, one segment): the live key count,
// read on the device and clamped to n; the grid is sized for n.
template <int ITEMS>
__global__ __launch_bounds__(kRsThreads) void k_rs_hist(SortSource S, uint32_t n,
                                                        const uint32_t* __restrict__ n_dev,
                                                        int shift, uint32_t mask, uint32_t* __restrict__ hist,
                                                        uint32_t nblocks) {
    if (n_dev) n = min(n, *n_dev);
    // four counter sets per wave (lane % 4): keys that share a digit, as in
    // the last pass of a sort whose top digit takes few values, spread their
    // LDS atomics over four addresses, which the padded rows (264 words: a
    // shift of 8 banks from one set to the next) put in different banks
    constexpr int kSets = 4, kRow = 264;
    __shared__ uint32_t h[kRsWaves * kSets][kRow];
    const int w = (int)(threadIdx.x >> 6) * kSets + (int)(threadIdx.x & (kSets - 1));
    const SortTile T = sort_tile<ITEMS>(S, blockIdx.x, n, nblocks);
    // All loads of a thread are issued before the counters are cleared (ITEMS
    // coalesced loads in flight per wave, not one); an index past the end
    // reads the last key and is not counted.
    uint32_t kk[ITEMS];
    const bool live = T.begin < T.end;
    if (live) sort_load<ITEMS>(S, T, T.begin + threadIdx.x, kRsThreads, kk, nullptr);
    for (int k = threadIdx.x; k < kRsWaves * kSets * kRow; k += kRsThreads) (&h[0][0])[k] = 0;
    __syncthreads();
    if (live) {
#pragma unroll
        for (int it = 0; it < ITEMS; ++it)
            if (T.begin + (uint64_t)it * kRsThreads + threadIdx.x < T.end)
                atomicAdd(&h[w][sort_digit(T, kk[it], shift, mask)], 1u);
    }
    __syncthreads();
    uint32_t d = threadIdx.x;
    if (d > mask || T.j >= T.nb) return;
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kRsWaves * kSets; ++k) sum += h[k][d];
    hist[(uint64_t)T.first * (mask + 1u) + (uint64_t)d * T.nb + T.j] = sum;
}

// Stable scatter of one tile (512 threads; 16 keys per thread, 74 KB of LDS:
// two blocks and sixteen waves per CU).  Each wave ranks its keys (ITEMS
// rounds of 64) against per-wave digit counters in LDS, with no block barrier;
// the eight waves' counts then give every key its position in the tile sorted
// by digit (threads 0..255 own one digit each).  The tile is reordered through
// LDS and written out in digit order, so each digit's run of keys is stored
// contiguously at the tile's offset for that digit.
//
// MODE kScanned: the offsets are the scanned tile counters `offs`.  MODE kRaw:
// `offs` holds the counters themselves; the block adds up its segment's (at
// most kRawTiles or kRawPass tiles, a few KB from L2) instead of two launches that scan
// them.  MODE kOneSweep: a single kernel per pass (decoupled look-back).  Each
// block takes the next tile number from a ticket counter, so every lower tile
// belongs to a block that is already running.  Once ranked, it publishes its
// per-digit counts in `status`, then adds up its predecessors' (a tile that
// has published its inclusive prefix ends the walk) and publishes its own
// inclusive prefix; the digit's start comes from the global digit counts
// `gcount`.  A status word holds the value in bits 0..29, kStAgg once the
// tile's own count is there and kStInc once its inclusive prefix is.  Every
// wait is bounded: after kLookbackSpins polls a block gives up, sets *fault (a
// word of the sort's scratch, not reported further) and goes on, so no kernel
// can hang; its output is then wrong, but only a predecessor that never
// publishes could cause that, and the ticket order guarantees every
// predecessor is running.
constexpr uint32_t kStAgg = 1u << 30, kStInc = 1u << 31, kStVal = kStAgg - 1u;
constexpr uint32_t kLookbackSpins = 1u << 22;
constexpr int kScanned = 0, kRaw = 1, kOneSweep = 2;
// (a segment's tiles; of a pass of few tiles in all, that many.  us of a depth sort
// of one view, counters added up by the blocks / scanned: tiles of 2048 keys against
// scanned ones of 8192: 98 tiles 58 / 82, 157 73 / 84, 196 81 / 85, 293 113 / 92;
// tiles of 8192: 86 97 / 107, 135 113 / 114, 159 119 / 114; of two views, 160 98 / 112)
constexpr uint32_t kRawTiles = 64, kRawPass = 160;

template <int MODE, int ITEMS>
__global__ __launch_bounds__(kRsThreads) void k_rs_scatter(SortSource S, uint32_t* __restrict__ keys_out,
                                                           uint32_t* __restrict__ vals_out,
                                                           uint32_t n, const uint32_t* __restrict__ n_dev, int shift, uint32_t mask,
                                                           const uint32_t* __restrict__ offs,
                                                           uint32_t nblocks, uint32_t* status,
                                                           const uint32_t* __restrict__ gcount,
                                                           uint32_t* ticket, uint32_t* fault) {
    constexpr uint32_t kTileKeys = kRsThreads * ITEMS;
    if (n_dev) n = min(n, *n_dev);
    __shared__ uint32_t wcnt[kRsWaves][256];
    __shared__ uint32_t dstart[256];
    __shared__ uint32_t gbase[256];
    __shared__ uint32_t wsum[kRsThreads / 64];
    __shared__ uint32_t skey[kTileKeys];
    __shared__ uint32_t sval[kTileKeys];
    __shared__ uint32_t stile;
    uint32_t tile = blockIdx.x;
    if constexpr (MODE == kOneSweep) {
        if (threadIdx.x == 0) stile = atomicAdd(ticket, 1u);
        __syncthreads();
        tile = stile;
    }
    const SortTile T = sort_tile<ITEMS>(S, tile, n, nblocks);
    if (T.begin >= T.end) return;  // whole block: no live keys (no live tile of the segment follows)
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int k = lane; k < 256; k += 64) wcnt[w][k] = 0u;
    const uint64_t row = (uint64_t)T.first * (mask + 1u) + (uint64_t)threadIdx.x * T.nb;
    uint32_t before = 0u, dtot = 0u;  // kRaw: the digit's keys in earlier tiles, and in all
    if constexpr (MODE == kScanned) {
        if (threadIdx.x <= mask) gbase[threadIdx.x] = offs[row + T.j];
    } else if constexpr (MODE == kRaw) {
        if (threadIdx.x <= mask) {
#pragma unroll 8
            for (uint32_t b = 0; b < T.nb; ++b) {
                const uint32_t c = offs[row + b];
                before += b < T.j ? c : 0u;
                dtot += c;
            }
        }
    }
    const uint64_t base = T.begin + (uint64_t)w * (kTileKeys / kRsWaves);
    uint32_t kk[ITEMS], vv[ITEMS], rk[ITEMS];
    // The wave's loads are all issued before the ranking, whose wave
    // barriers would otherwise hold each round's loads until the round
    // before has been ranked; an index past the end reads the last pair.
    sort_load<ITEMS>(S, T, base + lane, 64, kk, vv);
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        const uint64_t idx = base + (uint64_t)it * 64 + lane;
        const bool valid = idx < T.end;
        const uint32_t key = kk[it];
        const uint32_t d = sort_digit(T, key, shift, mask);
        uint64_t m = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t bb = __ballot((d >> b) & 1u);
            m &= ((d >> b) & 1u) ? bb : ~bb;
        }
        const uint32_t pre = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        const uint32_t c = wcnt[w][d];
        __builtin_amdgcn_wave_barrier();
        if (valid && pre == 0) wcnt[w][d] = c + (uint32_t)__popcll(m);
        __builtin_amdgcn_wave_barrier();
        rk[it] = valid ? c + pre : 0xFFFFFFFFu;
    }
    __syncthreads();
    {
        // thread t owns digit t: prefix over the waves, then over the digits
        const uint32_t t = threadIdx.x;
        uint32_t run = 0;
        if (t < 256) {
#pragma unroll
            for (int k = 0; k < kRsWaves; ++k) {
                const uint32_t c = wcnt[k][t];
                wcnt[k][t] = run;
                run += c;
            }
        }
        uint32_t tot;
        const uint32_t ds = block_exclusive_scan<kRsThreads>(run, wsum, &tot);
        if (t < 256) dstart[t] = ds;
        if constexpr (MODE == kRaw) {
            const uint32_t gs = block_exclusive_scan<kRsThreads>(dtot, wsum, &tot);
            if (t <= mask) gbase[t] = (uint32_t)T.seg + gs + before;
        }
        if constexpr (MODE == kOneSweep) {
            // the digit's first output position, over all tiles
            const uint32_t gc = t <= mask ? gcount[t] : 0u;
            const uint32_t gstart = block_exclusive_scan<kRsThreads>(gc, wsum, &tot);
            if (t <= mask) {
                uint32_t* st = status + (uint64_t)tile * 256u + t;
                uint32_t excl = 0u;
                if (tile == 0u) {
                    __hip_atomic_store(st, kStInc | run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    __hip_atomic_store(st, kStAgg | run, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    uint64_t j = tile - 1u;
                    uint32_t spins = 0u;
                    while (true) {
                        const uint32_t v = __hip_atomic_load(status + j * 256u + t, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT);
                        if (v & kStInc) {
                            excl += v & kStVal;
                            break;
                        }
                        if (v & kStAgg) {  // tile 0 publishes its prefix at once: j stays >= 0
                            excl += v & kStVal;
                            --j;
                            continue;
                        }
                        if (++spins > kLookbackSpins) {
                            atomicOr(fault, 1u);
                            break;
                        }
                        __builtin_amdgcn_s_sleep(1);
                    }
                    __hip_atomic_store(st, kStInc | (excl + run), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                gbase[t] = gstart + excl;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
        if (rk[it] != 0xFFFFFFFFu) {
            const uint32_t d = sort_digit(T, kk[it], shift, mask);
            const uint32_t lp = dstart[d] + wcnt[w][d] + rk[it];
            skey[lp] = kk[it];
            sval[lp] = vv[it];
        }
    }
    __syncthreads();
    const uint32_t cnt = (uint32_t)(T.end - T.begin);
    for (uint32_t i = threadIdx.x; i < cnt; i += kRsThreads) {
        const uint32_t key = skey[i];
        const uint32_t d = sort_digit(T, key, shift, mask);
        const uint32_t gp = gbase[d] + (i - dstart[d]);
        keys_out[gp] = key;
        vals_out[gp] = sval[i];
    }
}

// The digit counts of every pass of a one-sweep sort, over all keys:
// gcount[p * 256 + d].  A grid of up to 2048 blocks strides over the 8192-key
// tiles; four counter sets per pass (lane mod 4) in padded rows, as in
// k_rs_hist, and one global atomic per block and non-zero count.
struct RadixDigits {
    int passes;
    int shift[4];
    uint32_t mask[4];
};
constexpr uint32_t kOneSweepHead = 1088;  // words before the status rows: gcount (1024), tickets, fault

__global__ __launch_bounds__(kRsThreads) void k_rs_counts(const uint32_t* __restrict__ keys, uint32_t n,
                                                          const uint32_t* __restrict__ n_dev, RadixDigits dg,
                                                          uint32_t* __restrict__ gcount) {
    if (n_dev) n = min(n, *n_dev);
    constexpr int kSets = 4, kRow = 264;
    __shared__ uint32_t h[4][kSets][kRow];
    for (int k = threadIdx.x; k < 4 * kSets * kRow; k += kRsThreads) (&h[0][0][0])[k] = 0u;
    __syncthreads();
    const uint32_t set = threadIdx.x & (kSets - 1);
    for (uint64_t base = (uint64_t)blockIdx.x * kRsTile; base < n; base += (uint64_t)gridDim.x * kRsTile) {
        uint32_t kk[kRsItems];
#pragma unroll
        for (int it = 0; it < kRsItems; ++it)
            kk[it] = keys[min(base + (uint64_t)it * kRsThreads + threadIdx.x, (uint64_t)n - 1)];
#pragma unroll
        for (int it = 0; it < kRsItems; ++it) {
            if (base + (uint64_t)it * kRsThreads + threadIdx.x >= n) continue;
            for (int p = 0; p < dg.passes; ++p) atomicAdd(&h[p][set][(kk[it] >> dg.shift[p]) & dg.mask[p]], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < dg.passes * 256; i += kRsThreads) {
        const int p = i >> 8, d = i & 255;
        const uint32_t c = h[p][0][d] + h[p][1][d] + h[p][2][d] + h[p][3][d];
        if (c != 0u) atomicAdd(&gcount[i], c);
    }
}

namespace {
// Tiles of 2048 keys (a short chain of ranking rounds, four times the blocks)
// for up to 2^19 keys, as long as a segment's tiles, or all, stay within the
// counters a block adds up itself; else of 8192 (runs of about 32 keys per digit in the
// scattered output).
inline int sort_items(uint64_t segment, uint64_t total) {
    constexpr uint64_t kTile = kRsThreads * 4;
    return (segment <= kRawTiles * kTile && total <= (1u << 19)) || total <= kRawPass * kTile ? 4 : kRsItems;
}

// One histogram and scatter pass; `tiles` over all segments, `seg_tiles` of the longest.
void radix_pass(const SortSource& src, uint32_t* dk, uint32_t* dv, uint32_t n, const uint32_t* n_dev, int shift,
                uint32_t mask, uint32_t tiles, uint32_t seg_tiles, int items, uint32_t* scratch, hipStream_t s) {
    uint32_t* hist = scratch;
    uint32_t* sscr = scratch + (((uint64_t)(mask + 1u) * tiles + 63) / 64) * 64;
    const dim3 grid(tiles), block(kRsThreads);
    uint32_t* nu = nullptr;
    const uint32_t* nc = nullptr;
    if (items == 4) hipLaunchKernelGGL(k_rs_hist<4>, grid, block, 0, s, src, n, n_dev, shift, mask, hist, tiles);
    else hipLaunchKernelGGL(k_rs_hist<kRsItems>, grid, block, 0, s, src, n, n_dev, shift, mask, hist, tiles);
    // (tiles of 2048 keys always: a segment has at most kRawPass of them, see sort_items)
    if (items == 4 || seg_tiles <= kRawTiles || tiles <= kRawPass) {
        if (items == 4)
            hipLaunchKernelGGL((k_rs_scatter<kRaw, 4>), grid, block, 0, s, src, dk, dv, n, n_dev, shift, mask,
                               hist, tiles, nu, nc, nu, nu);
        else
            hipLaunchKernelGGL((k_rs_scatter<kRaw, kRsItems>), grid, block, 0, s, src, dk, dv, n, n_dev, shift,
                               mask, hist, tiles, nu, nc, nu, nu);
        return;
    }
    launch_scan(hist, hist, (mask + 1u) * tiles, nullptr, sscr, s);
    hipLaunchKernelGGL((k_rs_scatter<kScanned, kRsItems>), grid, block, 0, s, src, dk, dv, n, n_dev, shift, mask,
                       hist, tiles, nu, nc, nu, nu);
}
inline size_t pass_scratch_words(uint64_t tiles) {
    const uint64_t h = 256 * (tiles > 0 ? tiles : 1);
    return (size_t)(((h + 63) / 64) * 64 + scan_scratch_words(h));
}
}  // namespace

size_t radix_scratch_words(uint32_t n) {
    const uint64_t nb = ((uint64_t)n + kRsTile - 1) / kRsTile;
    const uint64_t small = std::min<uint64_t>(((uint64_t)n + kRsThreads * 4 - 1) / (kRsThreads * 4), kRawPass);
    const size_t one_sweep = kOneSweepHead + 4 * (size_t)(256 * (nb > 0 ? nb : 1));  // up to four passes of status rows
    return std::max({pass_scratch_words(nb), pass_scratch_words(small), one_sweep});
}

void radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt, uint32_t n,
                int bits, uint32_t* scratch, hipStream_t s, const uint32_t* n_dev, bool* result_in_alt) {
    *result_in_alt = false;
    if (n <= 1 || bits <= 0) return;
    // as many passes as 8-bit digits need, with the bits spread evenly over
    // them (19 bits: 7 + 6 + 6): narrower digits leave longer runs of equal
    // digits in each tile, so the scattered writes come in fuller lines
    const int passes = (bits + 7) / 8;
    RadixDigits dg{passes, {0, 0, 0, 0}, {0u, 0u, 0u, 0u}};
    for (int p = 0, sh = 0; p < passes; ++p) {
        const int width = bits / passes + (p < bits % passes ? 1 : 0);
        dg.shift[p] = sh;
        dg.mask[p] = (1u << width) - 1u;
        sh += width;
    }
    // One sweep per pass for large sorts (where the status words can hold
    // every count); the scratch then holds [global digit counts | tickets,
    // fault | status rows].  Below 2^25 keys the look-back's waits cost more
    // than the histogram pass and scan they save (a 2^24-key sort of four
    // passes: 0.45 against 0.37 ms; 10^8 keys in two: 1.09 against 1.26).
    const bool one_sweep = n >= (1u << 25) && n < kStAgg;
    const int items = one_sweep ? kRsItems : sort_items(n, n);
    const uint32_t nb = (uint32_t)(((uint64_t)n + kRsThreads * items - 1) / (kRsThreads * items));
    uint32_t* gcount = scratch;
    uint32_t* tickets = scratch + 1024;
    uint32_t* fault = scratch + 1024 + 4;
    uint32_t* status = scratch + kOneSweepHead;
    if (one_sweep) {
        launch_fill_u32(scratch, 0u, kOneSweepHead + (uint64_t)passes * 256u * nb, s);
        hipLaunchKernelGGL(k_rs_counts, dim3(std::min<uint32_t>(nb, 2048u)), dim3(kRsThreads), 0, s, keys, n,
                           n_dev, dg, gcount);
    }
    uint32_t *sk = keys, *sv = vals, *dk = keys_alt, *dv = vals_alt;
    for (int p = 0; p < passes; ++p) {
        SortSource src{};
        src.keys = sk;
        src.vals = sv;
        if (one_sweep)
            hipLaunchKernelGGL((k_rs_scatter<kOneSweep, kRsItems>), dim3(nb), dim3(kRsThreads), 0, s, src, dk, dv,
                               n, n_dev, dg.shift[p], dg.mask[p], (const uint32_t*)nullptr, nb,
                               status + (uint64_t)p * 256u * nb, gcount + 256 * p, tickets + p, fault);
        else
            radix_pass(src, dk, dv, n, n_dev, dg.shift[p], dg.mask[p], nb, nb, items, scratch, s);
        std::swap(sk, dk);
        std::swap(sv, dv);
    }
    *result_in_alt = sk != keys;  // an odd pass count leaves the result there
}

// ---- group sort ------------------------------------------------------------
//
// The group pairs leave the emission view by view (items lie so), so a view's
// pairs need sorting by its own groups only.  Where every view has fewer than
// 256 of them that is one pass over segments, found on the device, instead of the
// passes that the groups of all views take.  100k Gaussians, 50 views (3200
// groups): a call 1624 -> 1578 us; 500k, 100 views: the sort 0.96 -> 0.41 ms, a
// call 15.65 -> 15.03 ms.  The segments' partial tiles
// have to stay within the scratch that the general form is given: one a view at
// most, so no more views than full tiles.

// One block: seg and the tile numbers of SortSource from the items' offsets.
__global__ __launch_bounds__(256) void k_pair_segments(const ViewInfo* __restrict__ views, int n_views,
                                                       uint32_t n_items, const uint32_t* __restrict__ offsets,
                                                       uint32_t n, const uint32_t* __restrict__ n_dev,
                                                       uint32_t tile_keys, uint32_t* __restrict__ seg) {
    __shared__ uint32_t wsum[4];
    if (n_dev) n = min(n, *n_dev);
    auto begin = [&](int v) {
        return v < n_views && views[v].item_base < n_items ? min(offsets[views[v].item_base], n) : n;
    };
    uint32_t run = 0;
    for (int v0 = 0; v0 < n_views; v0 += 256) {
        const int v = v0 + (int)threadIdx.x;
        const uint32_t b = begin(v), e = begin(v + 1);
        const uint32_t nt = v < n_views ? (e - b + tile_keys - 1) / tile_keys : 0u;
        uint32_t tot;
        const uint32_t at = run + block_exclusive_scan<256>(nt, wsum, &tot);
        if (v < n_views) {
            seg[v] = b;
            seg[n_views + 1 + v] = at;
        }
        run += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        seg[n_views] = n;
        seg[2 * n_views + 1] = run;
    }
}

bool group_sort_by_view(uint64_t max_groups, int bits, int n_views, uint32_t n) {
    return bits > 8 && max_groups < 256u && (uint64_t)n_views <= (uint64_t)n / kRsTile;
}

void launch_group_sort(const ViewInfo* views, int n_views, uint32_t n_items, uint64_t max_groups,
                       const uint32_t* offsets, uint32_t* keys, uint32_t* vals, uint32_t* keys_alt,
                       uint32_t* vals_alt, uint32_t n, int bits, uint32_t* scratch, hipStream_t s,
                       const uint32_t* n_dev, bool* result_in_alt) {
    if (!group_sort_by_view(max_groups, bits, n_views, n)) {
        radix_sort(keys, vals, keys_alt, vals_alt, n, bits, scratch, s, n_dev, result_in_alt);
        return;
    }
    uint32_t mask = 1u;
    while (mask < max_groups) mask = 2u * mask + 1u;  // the view's groups lie below it
    const uint32_t head = (uint32_t)((2 * (uint64_t)n_views + 2 + 63) / 64) * 64u;
    const uint32_t tiles = n / kRsTile + (uint32_t)n_views;
    hipLaunchKernelGGL(k_pair_segments, dim3(1), dim3(256), 0, s, views, n_views, n_items, offsets, n, n_dev,
                       (uint32_t)kRsTile, scratch);
    SortSource src{};
    src.keys = keys;
    src.vals = vals;
    src.views = views;
    src.n_views = n_views;
    src.seg = scratch;
    radix_pass(src, keys_alt, vals_alt, n, n_dev, 0, mask, tiles, tiles, kRsItems, scratch + head, s);
    *result_in_alt = true;
}

// ---- depth sort ------------------------------------------------------------
//
// Each view's items by depth, ties by Gaussian index; the order is view by
// view, so that a view's records lie together (3.2 MB for 100k Gaussians, less
// than an XCD's L2) for the random reads of the masks and the tile kernels.
// Views of up to kViewSort items are sorted in LDS, kRun items a block; where a
// view has several such runs, a second launch ranks each item among the others
// (binary searches in the other runs, which L2 holds).  One block a view for
// all its items left most of the chip idle: 9 views of 20000 items 77 -> 38 us.
// Six runs are where the forms meet, us of the sort in runs / segments at 24576 items:
// 1 view 38 / 43, 4 40 / 44, 9 44 / 45, 50 89 / 89; 28000 items in more runs, each of
// which every item searches, 48 / 42, 47 / 44, 52 / 46, 115 / 88.
// Larger views take four passes over segments, the first of which forms the
// keys itself.  us a call, one sort of the whole batch -> by view: 2k
// Gaussians x 8 views 220 -> 149 (13 launches of the call become one); 500k x
// 100 views 23371 -> 22795 (k_group_masks 1784 -> 1453 us, k_project 1508 ->
// 1165: their reads hit L2), 100k x 50 views 1813 -> 1816.
constexpr uint32_t kViewThreads = 1024, kViewWaves = kViewThreads / 64;
constexpr uint32_t kRun = 4096, kRuns = 6, kViewSort = kRun * kRuns;

// One run (blockIdx.y) of one view (blockIdx.x), kRun items at most.  Only the
// bits in which the run's depths differ are sorted.  keys: the run's sorted
// keys as well (views of several runs).
__global__ __launch_bounds__(kViewThreads) void k_sort_view(SortSource S, uint32_t* __restrict__ vals,
                                                            uint32_t* __restrict__ keys) {
    constexpr uint32_t IPT = kRun / kViewThreads, kCap = kRun;
    __shared__ uint32_t skey[kCap];
    __shared__ uint16_t sidx[kCap];
    __shared__ uint16_t cnt[kViewWaves][256];
    __shared__ uint32_t wsum[kViewWaves];
    __shared__ uint32_t range[2];
    const ViewInfo& V = S.views[blockIdx.x];
    const uint32_t first = blockIdx.y * kRun;
    if (first >= V.n_gauss) return;
    const uint32_t n = min(V.n_gauss - first, kRun);
    const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t rounds = (n + kViewThreads - 1) / kViewThreads;  // uniform, <= IPT
    const uint32_t base = w * rounds * 64;                          // the wave's places
    if (tid == 0) {
        range[0] = 0xFFFFFFFFu;
        range[1] = 0u;
    }
    uint32_t kk[IPT], id[IPT], rk[IPT];
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (uint32_t it = 0; it < (uint32_t)IPT; ++it) {
        if (it >= rounds) break;
        const uint32_t i = base + it * 64 + lane;
        id[it] = i;
        kk[it] = i < n ? depth_key(S, V, (uint64_t)V.g_offset + first + i) : 0xFFFFFFFFu;
        if (kk[it] != 0xFFFFFFFFu) {
            lo = min(lo, kk[it]);
            hi = max(hi, kk[it]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, 64));
    }
    if (lane == 0 && lo <= hi) {
        atomicMin(&range[0], lo);
        atomicMax(&range[1], hi);
    }
    __syncthreads();
    lo = range[0];
    hi = range[1];
    // keys relative to the nearest; culled items one past the farthest
    const uint32_t top = lo <= hi ? hi - lo + 1u : 0u;
    const int bits = top ? 32 - __clz((int)top) : 0;
#pragma unroll
    for (uint32_t it = 0; it < (uint32_t)IPT; ++it) {
        if (it >= rounds) break;
        kk[it] = kk[it] == 0xFFFFFFFFu ? top : kk[it] - lo;
    }
    const int passes = (bits + 7) / 8;
    for (int p = 0, shift = 0; p < passes; ++p) {
        const int width = bits / passes + (p < bits % passes ? 1 : 0);
        const uint32_t mask = (1u << width) - 1u;
        for (uint32_t k = lane; k < 256; k += 64) cnt[w][k] = 0u;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (uint32_t it = 0; it < (uint32_t)IPT; ++it) {
            if (it >= rounds) break;
            const bool valid = base + it * 64 + lane < n;
            const uint32_t d = (kk[it] >> shift) & mask;
            uint64_t m = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const uint64_t bb = __ballot((d >> b) & 1u);
                m &= ((d >> b) & 1u) ? bb : ~bb;
            }
            const uint32_t pre = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            const uint32_t c = cnt[w][d];
            __builtin_amdgcn_wave_barrier();
            if (valid && pre == 0) cnt[w][d] = (uint16_t)(c + (uint32_t)__popcll(m));
            __builtin_amdgcn_wave_barrier();
            rk[it] = c + pre;
        }
        __syncthreads();
        {
            // thread t owns digit t: prefix over the waves, then over the digits
            uint32_t run = 0;
            uint32_t c[kViewWaves];
            if (tid < 256) {
#pragma unroll
                for (uint32_t k = 0; k < kViewWaves; ++k) {
                    c[k] = run;
                    run += cnt[k][tid];
                }
            }
            uint32_t tot;
            const uint32_t ds = block_exclusive_scan<kViewThreads>(tid < 256 ? run : 0u, wsum, &tot);
            if (tid < 256) {
#pragma unroll
                for (uint32_t k = 0; k < kViewWaves; ++k) cnt[k][tid] = (uint16_t)(c[k] + ds);
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t it = 0; it < (uint32_t)IPT; ++it) {
            if (it >= rounds) break;
            if (base + it * 64 + lane < n) {
                const uint32_t at = cnt[w][(kk[it] >> shift) & mask] + rk[it];
                skey[at] = kk[it];
                sidx[at] = (uint16_t)id[it];
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t it = 0; it < (uint32_t)IPT; ++it) {
            if (it >= rounds) break;
            const uint32_t i = base + it * 64 + lane;
            if (i < n) {
                kk[it] = skey[i];
                id[it] = sidx[i];
            }
        }
        shift += width;
    }
#pragma unroll
    for (uint32_t it = 0; it < (uint32_t)IPT; ++it) {
        if (it >= rounds) break;
        const uint32_t i = base + it * 64 + lane;
        if (i < n) {
            vals[V.item_base + first + i] = V.item_base + first + id[it];
            if (keys) keys[V.item_base + first + i] = kk[it] == top ? 0xFFFFFFFFu : kk[it] + lo;
        }
    }
}

// Places of a view's (blockIdx.x) sorted runs' items in the view's order: an
// item's place in its run, plus the items of the other runs before it (equal keys
// in an earlier run come first: the order of the items).
__global__ __launch_bounds__(256) void k_merge_runs(const ViewInfo* __restrict__ views, const uint32_t* __restrict__ keys,
                                                    const uint32_t* __restrict__ in, uint32_t* __restrict__ out) {
    const ViewInfo& V = views[blockIdx.x];
    const uint32_t n = V.n_gauss, i = blockIdx.y * 256 + threadIdx.x;
    if (i >= n) return;
    const uint32_t* k = keys + V.item_base;
    const uint32_t key = k[i], run = i / kRun;
    uint32_t at[kRuns];  // items of each run before this one
#pragma unroll
    for (uint32_t q = 0; q < kRuns; ++q) at[q] = 0u;
    // all searches step together: at[q] items are known to come before
#pragma unroll
    for (uint32_t d = kRun; d >= 1u; d >>= 1) {
#pragma unroll
        for (uint32_t q = 0; q < kRuns; ++q) {
            const uint32_t m = min(n > q * kRun ? n - q * kRun : 0u, kRun);  // the run's items
            const uint32_t p = at[q] + d;
            if (p <= m) {
                const uint32_t x = k[q * kRun + p - 1u];
                if (x < key || (x == key && q < run)) at[q] = p;
            }
        }
    }
    uint32_t place = i - run * kRun;
#pragma unroll
    for (uint32_t q = 0; q < kRuns; ++q) place += q == run ? 0u : at[q];
    out[V.item_base + place] = in[V.item_base + i];
}

DepthSortShape depth_sort_shape(uint32_t max_n, uint64_t n_items) {
    DepthSortShape d;
    d.in_lds = max_n <= kViewSort;
    d.items = d.in_lds ? 0 : sort_items(max_n, n_items);
    d.tile = d.in_lds ? 0u : (uint32_t)(kRsThreads * d.items);
    return d;
}

size_t depth_sort_scratch_words(const DepthSortShape& d, uint64_t tiles) {
    return d.in_lds ? 0 : pass_scratch_words(tiles);
}

void launch_depth_sort(const ViewInfo* views, int n_views, uint32_t n_items, const DepthSortShape& d,
                       uint32_t max_n, uint32_t uniform_n, uint32_t tiles, const float* means, const float* opac,
                       BlendParams bp, uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                       uint32_t* scratch, hipStream_t s) {
    if (n_items == 0 || n_views <= 0) return;
    SortSource src{};
    src.views = views;
    src.n_views = n_views;
    src.means = means;
    src.opac = opac;
    src.znear = bp.znear;
    src.alpha_min = bp.alpha_min;
    if (d.in_lds) {
        const unsigned runs = (max_n + kRun - 1) / kRun;
        const dim3 grid((unsigned)n_views, runs), block(kViewThreads);
        uint32_t* none = nullptr;
        hipLaunchKernelGGL(k_sort_view, grid, block, 0, s, src, runs > 1 ? vals_alt : vals, runs > 1 ? keys : none);
        if (runs > 1)
            hipLaunchKernelGGL(k_merge_runs, dim3((unsigned)n_views, (max_n + 255) / 256), dim3(256), 0, s, views,
                               keys, vals_alt, vals);
        return;
    }
    const uint32_t seg_tiles = (max_n + d.tile - 1) / d.tile;
    src.view_tiles = uniform_n ? seg_tiles : 0u;
    uint32_t *dk = keys_alt, *dv = vals_alt, *ok = keys, *ov = vals;
    for (int p = 0; p < 4; ++p) {
        radix_pass(src, dk, dv, n_items, nullptr, 8 * p, 255u, tiles, seg_tiles, d.items, scratch, s);
        src.keys = dk;
        src.vals = dv;
        std::swap(dk, ok);
        std::swap(dv, ov);
    }
}

// ---- tile order ------------------------------------------------------------
//
// Bins by the octave of their list length, longest first, index order within
// an octave (neighbouring tiles of a view stay together and share records in
// L2): a stable counting sort over 33 classes, 4096 bins per block, the class
// taken from the ranges in both kernels (no keys or values are stored).  A
// launch of up to 4096 bins is one block, which counts and places in one
// kernel.
namespace {
constexpr uint32_t kToBins = 4096, kToClasses = 64, kToThreads = 1024, kToWaves = kToThreads / 64;
__device__ __forceinline__ uint32_t tile_class(uint2 r) { return (uint32_t)__clz((int)(r.y - r.x + 1u)); }
}  // namespace

template <bool PLACE>
__global__ __launch_bounds__(kToThreads) void k_tile_order(const uint2* __restrict__ ranges, uint32_t n_bins,
                                                           uint32_t* __restrict__ hist, uint32_t n_blocks,
                                                           uint32_t* __restrict__ out) {
    __shared__ uint32_t cnt[kToWaves][kToClasses];
    const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    for (uint32_t i = tid; i < kToWaves * kToClasses; i += kToThreads) (&cnt[0][0])[i] = 0u;
    __syncthreads();
    // wave w takes 256 consecutive bins, 64 at a time
    const uint64_t b0 = (uint64_t)blockIdx.x * kToBins + w * (kToBins / kToWaves);
    uint32_t cls[4], rank[4];
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const uint64_t b = b0 + it * 64 + lane;
        cls[it] = b < n_bins ? tile_class(ranges[b]) : 63u;
    }
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        uint64_t m = ~0ull;  // lanes of the same class
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const uint64_t bb = __ballot((cls[it] >> k) & 1u);
            m &= ((cls[it] >> k) & 1u) ? bb : ~bb;
        }
        const uint32_t pre = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        const uint32_t c = cnt[w][cls[it]];
        __builtin_amdgcn_wave_barrier();
        if (pre == 0) cnt[w][cls[it]] = c + (uint32_t)__popcll(m);
        __builtin_amdgcn_wave_barrier();
        rank[it] = c + pre;
    }
    __syncthreads();
    if (tid < kToClasses) {  // wave 0: prefix over the waves, then over the classes
        uint32_t run = 0;
        for (uint32_t k = 0; k < kToWaves; ++k) {
            const uint32_t c = cnt[k][tid];
            cnt[k][tid] = run;
            run += c;
        }
        if constexpr (!PLACE) {
            hist[(uint64_t)tid * n_blocks + blockIdx.x] = tid < 63u ? run : 0u;
        } else {
            const uint32_t base = n_blocks > 1 ? hist[(uint64_t)tid * n_blocks + blockIdx.x]
                                               : wave_inclusive_scan(run) - run;
            for (uint32_t k = 0; k < kToWaves; ++k) cnt[k][tid] += base;
        }
    }
    if constexpr (PLACE) {
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const uint64_t b = b0 + it * 64 + lane;
            if (b < n_bins) out[cnt[w][cls[it]] + rank[it]] = (uint32_t)b;
        }
    }
}

size_t tile_order_words(uint32_t n_bins) {
    const size_t nb = ((size_t)n_bins + kToBins - 1) / kToBins;
    return (size_t)n_bins + 64 + (nb > 1 ? kToClasses * nb + scan_scratch_words(kToClasses * nb) : 0);
}

void launch_tile_order(const uint2* ranges, uint32_t n_bins, uint32_t* order, hipStream_t s) {
    if (n_bins == 0) return;
    const uint32_t nb = (uint32_t)(((uint64_t)n_bins + kToBins - 1) / kToBins);
    uint32_t* hist = order + (((size_t)n_bins + 63) / 64) * 64;
    if (nb > 1) {
        hipLaunchKernelGGL(k_tile_order<false>, dim3(nb), dim3(kToThreads), 0, s, ranges, n_bins, hist, nb, order);
        launch_scan(hist, hist, kToClasses * nb, nullptr, hist + kToClasses * nb, s);
    }
    hipLaunchKernelGGL(k_tile_order<true>, dim3(nb), dim3(kToThreads), 0, s, ranges, n_bins, hist, nb, order);
}

}  // namespace gsc
