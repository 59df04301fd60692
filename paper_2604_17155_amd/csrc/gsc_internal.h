// Internal declarations shared by the HIP translation units of libgsc.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/gsc.h"

namespace gsc {

constexpr int kTile = 16;           // tile edge in pixels (16x16 = one wave, 4 pixels per lane)
constexpr int kTileShift = 4;
// Binning granularity: 16 (a bin is one tile) or 32 (a bin is 2x2 tiles).
constexpr int kMinBin = 16;
constexpr int kMaxBin = 32;
constexpr int kMaxNb = 16;          // (L+1)^2 for L <= 3
constexpr int kMaxC = 64;

// One view as the kernels see it.  A batch of views may mix scenes: each view
// names its scene's Gaussians [g_offset, g_offset + n_gauss) in the
// concatenated arrays.  The (view, Gaussian) items of a batch are numbered
// view by view: item = item_base + local Gaussian index.
struct ViewInfo {
    float R[9];
    float t[3];
    float fx, fy, cx, cy;
    double centre[3];      // camera centre -R^T t, for the SH view direction
    int32_t width, height;
    int32_t tiles_x, tiles_y;  // bins per row and column
    uint32_t tile_base;    // first global bin id of this view within its batch
    uint32_t item_base;    // first item of this view within its batch
    uint32_t group_base;   // first group (4x4 bins) of this view within its batch
    int32_t groups_x;      // groups per row
    uint32_t sort_base;    // first depth-sort tile of this view within its batch
    int64_t pixel_offset;  // first target row
    int64_t g_offset;      // first Gaussian of the view's scene
    int64_t vs_base;       // first per-view sum slot of this view (per-view layouts)
    uint32_t n_gauss;      // Gaussians of the view's scene
    uint32_t scene;        // scene index
    uint32_t uniform_n;    // n_gauss when every view of the batch has the same
                           // count (item = view * n + g), else 0
};

// View of a batch item: a division when every view has the same count,
// else a binary search on item_base (n_views >= 1).
__device__ inline int find_view_item(const ViewInfo* __restrict__ views, int n_views, uint32_t item) {
    const uint32_t un = views[0].uniform_n;
    if (un != 0u) return min((int)(item / un), n_views - 1);
    int lo = 0, hi = n_views - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (views[mid].item_base <= item) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The same lookup on the views' first items staged in LDS by the block:
// stage_view_bases fills sbase (kViewLds words) when the batch's views differ
// in size and fit, and ends with a block barrier (every thread must call it);
// view_of then searches LDS instead of the view records in global memory.
constexpr int kViewLds = 512;
__device__ inline bool stage_view_bases(const ViewInfo* __restrict__ views, int n_views, uint32_t* sbase) {
    const bool use = views[0].uniform_n == 0u && n_views <= kViewLds;
    if (use)
        for (int v = (int)threadIdx.x; v < n_views; v += (int)blockDim.x) sbase[v] = views[v].item_base;
    __syncthreads();
    return use;
}
__device__ inline int view_of(const ViewInfo* __restrict__ views, int n_views, const uint32_t* sbase,
                              bool staged, uint32_t item) {
    if (!staged) return find_view_item(views, n_views, item);
    int lo = 0, hi = n_views - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (sbase[mid] <= item) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Blend constants in the form the kernels use.
struct BlendParams {
    float alpha_min, alpha_max, t_min, cut2, dilation, znear;
};

// Splat record of the item of depth rank k, two float4 at rec[2k], rec[2k+1]
// (one 32-byte access per random gather):
//   r0 = (u_hi, v_hi, u_lo, v_lo)   projected mean as FP32 hi/lo pairs
//   r1 = (K*cxx, 2*K*cxy, K*cyy, opacity) with the conic (cxx, cxy, cyy) =
//        Sigma_2D^{-1} pre-scaled by K = -log2(e)/2, so that
//        q2 = K*q = r1.x dx^2 + r1.y dx dy + r1.z dy^2 and exp(-q/2) = exp2(q2).
constexpr double kExp2Scale = -0.72134752044448170368;  // -0.5 * log2(e)

// Bin pairs carry the depth rank in the low 26 bits and a 4-bit mask above:
// which quadrants of the bin the footprint reaches (bit 2 * row half + column
// half).  The tile kernels run one wave per 16x16 tile, which takes its pixels
// in four blocks of 8x8: for 16-pixel bins the bin is the tile and the mask
// names its blocks; for 32-pixel bins it names the bin's four tiles, and the
// blocks are found when the records are gathered (entry_blocks).
constexpr uint32_t kItemBits = 26;
constexpr uint32_t kItemMask = (1u << kItemBits) - 1u;

// ---- kernels launched from gsc_api.hip ----------------------------------
// Per-Gaussian geometry packed for the projection's gathers: one 64-byte
// record geo[g] = float (mean x, y, z, opacity), then double (Sigma xx, xy,
// xz, yy, yz, zz) with Sigma = R(q) diag(s^2) R(q)^T.
constexpr int kGeoStride = 16;  // floats per record
void launch_cov3d(const float* means, const float* opac, const float* scales, const float* quats,
                  float* geo, int64_t N, hipStream_t s);

// out[0] = sum_g mean axis scale, out[1..3] = sum_g mean (device doubles).
void launch_geometry_stats(const float* means, const float* scales, int64_t N, double* out,
                           hipStream_t s);

// Depth sort of the batch's items, view by view: vals becomes the items of
// each view in depth order (ties by Gaussian index) at the view's own places
// [item_base, item_base + n_gauss).  keys and the alternates are scratch.
// Its shape follows from the largest view and the item count; tiles: the views' ceil(n_gauss /
// tile) summed (0 when the views are sorted in LDS), numbered by sort_base;
// uniform_n: n_gauss when all views have the same, else 0.
struct DepthSortShape {
    bool in_lds;
    int items;
    uint32_t tile;
};
DepthSortShape depth_sort_shape(uint32_t max_n, uint64_t n_items);
size_t depth_sort_scratch_words(const DepthSortShape& d, uint64_t tiles);
void launch_depth_sort(const ViewInfo* views, int n_views, uint32_t n_items, const DepthSortShape& d,
                       uint32_t max_n, uint32_t uniform_n, uint32_t tiles, const float* means, const float* opac,
                       BlendParams bp, uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                       uint32_t* scratch, hipStream_t s);

// Projection in depth order: position k handles item i = order[k] (k if order
// is null) and writes counts[k], the groups of 4x4 bins its footprint is
// listed in, rects[k], how to list them (count_groups), and, when counts[k] > 0,
// the record rec[2k], rec[2k + 1] (records are only ever read through lists).
void launch_project(const ViewInfo* views, int n_views, uint32_t n_items, const uint32_t* order,
                    const float* geo, BlendParams bp, uint32_t* counts, uint32_t* rects, float4* rec,
                    int bin, hipStream_t s);

// (group, depth rank) pairs of the depth-ordered records; a rank marked kVoidPair
// reaches no bin.  Pairs at offsets >= cap are dropped and their items counted in
// *overflow (if given).
constexpr uint32_t kVoidPair = 1u << 31;
void launch_emit(const ViewInfo* views, int n_views, const uint32_t* offsets, const uint32_t* counts,
                 const uint32_t* rects, const float4* rec, BlendParams bp,
                 uint32_t n_items, uint32_t* pair_keys, uint32_t* pair_vals, int bin,
                 hipStream_t s, uint32_t cap = 0xFFFFFFFFu, uint32_t* overflow = nullptr);

// Pairs of (bin, item) over all items in any order (plan creation): adds to *out.
void launch_count_bins(const ViewInfo* views, int n_views, uint32_t n_items, const uint32_t* counts,
                       const uint32_t* rects, const float4* rec, BlendParams bp, int bin, unsigned long long* out, hipStream_t s);

// The lists of the groups of a view batch (sorted (group, rank) pairs), turned
// into bin lists in three steps.  The pairs are taken in windows of `window`,
// one per wave, whatever groups they hold, so that lists of any length spread
// evenly.  Window u's pairs of group g have row u + g of `counts` (unique, as
// both grow along the pairs).
//   launch_group_masks: every pair's blocks (mask_lo, mask_hi), each row's
//     entries per bin, and the windows' first groups; adds each group's bin
//     entries to totals[group] (zero before).
//   launch_bin_ranges: with first[group] the exclusive scan of totals, the
//     bins' ranges, and counts turned into each row's first list positions;
//     puts the next group with pairs in the place of each group's ranges.x;
//     adds *total to *sum (if given).
//   launch_bin_lists: the bins' entries, depth rank | mask << kItemBits.
// Positions past cap are cut off; the entries that lose one are counted in
// *overflow (if given).  n_dev (optional): the live pair count, clamped to
// n_pairs.
//
// A wave takes the groups of its window one after the other, each at the price of
// a dependent load or two, so the window shrinks (256 to 4, a power of two) until
// there are as many windows as groups, or as many as the chip has places for
// waves; the rows then at most double, and a window holds one or two groups.
// us a call of 1 channel, windows of 256 / by this rule: 10 splats in 20 views of
// 512x512 653 / 205, 100 splats 365 / 247, 1000 in 20 of 1024x1024 635 / 578; at
// 100k splats the windows are 256 wide again (789 / 789).  2048 or 32768 windows
// in place of 8192: within 2% from 1 to 100k splats in five sets of views.
constexpr uint32_t kWindowMax = 256, kWindowMin = 4, kWindowsWanted = 8192;
inline uint32_t group_window(uint64_t pairs, uint64_t groups) {
    uint32_t w = kWindowMax;
    while (w > kWindowMin && pairs < (uint64_t)w * (groups < kWindowsWanted ? groups : kWindowsWanted)) w /= 2;
    return w;
}
struct GroupLists {
    const ViewInfo* views;
    int n_views;
    uint32_t n_groups;
    int bin;
    uint32_t n_pairs;
    uint32_t window;  // group_window(n_pairs, n_groups), or kWindowMax to save memory
    const uint32_t* n_dev;
    uint2* ranges;
    const uint32_t* keys;
    const uint32_t* vals;
    const float4* rec;
    uint32_t* mask_lo;
    uint32_t* mask_hi;
    uint32_t* counts;       // 16 words per row
    uint32_t* first_group;  // per window
    uint32_t* totals;
};
inline uint64_t group_windows(uint64_t pairs, uint32_t window) { return (pairs + window - 1) / window; }
inline uint64_t group_count_words(uint64_t pairs, uint64_t groups, uint32_t window) {
    return 16 * (group_windows(pairs, window) + groups);
}
void launch_group_masks(const GroupLists& g, BlendParams bp, hipStream_t s);
void launch_bin_ranges(const GroupLists& g, const uint32_t* first, uint2* ranges, uint32_t cap,
                       const uint32_t* total, unsigned long long* sum, hipStream_t s);
void launch_bin_lists(const GroupLists& g, uint32_t* lists, uint32_t cap, uint32_t* overflow, hipStream_t s);

// The tile lists of a view batch, as the tile kernels read them: bin b's
// entries are pair_vals[ranges[b].x .. ranges[b].y), front to back; an entry
// names depth rank k, whose record is rec[2k], rec[2k + 1] and whose batch
// item is items[k].  order (optional): the bins in the order their tiles are
// taken (launch_tile_order).
struct TileLists {
    const ViewInfo* views;
    int n_views;
    uint32_t n_bins;
    int bin;  // bin size in pixels
    const uint2* ranges;
    const uint32_t* pair_vals;
    const float4* rec;
    const uint32_t* items;
    const uint32_t* order;
};
// 16x16 tiles of the lists.
inline uint32_t wave_tiles(uint32_t n_bins, int bin) { return bin == 32 ? 4u * n_bins : n_bins; }
// Whether the tile kernels run one wave per 8x8 block instead of one per tile
// (walk_block): launches that leave SIMDs idle and are bound by their longest
// list.  Measured, us a call, tile form against block form.  16-pixel bins:
// 100k blob Gaussians, degree 3, 4 / 6 / 8 views of 512x512 (4096 / 6144 /
// 8192 tiles): 573 / 633 / 668 against 523 / 652 / 734; an optimisation step
// on 1 / 2 / 3 views of 640x640 (1600 / 3200 / 4800): 1996 / 2139 / 2287
// against 1205 / 1757 / 2235.  The same blobs, degree 0, 2 / 4 views (2048 / 4096
// tiles): accumulate of 3 channels 342 / 394 against 278 / 409, of 15 502 / 545
// against 315 / 465; render of 3 323 / 354 against 287 / 400; a render's adjoint
// of 3 548 / 568 against 468 / 698, of 8 655 / 680 against 361 / 471.  (Short
// lists favour blocks longer: 16 views of 250x250, 4096 tiles, accumulate of 3
// 735 against 581.)  32-pixel bins (larger footprints, whose entries
// meet all four blocks, and four times the gathers): one mask channel on
// 480x320 / 640x480 / 2 x 640x480 (600 / 1200 / 2400 tiles): 253 / 260 / 268
// against 239 / 279 / 355.
inline bool few_tiles(const TileLists& tl) {
    return wave_tiles(tl.n_bins, tl.bin) <= (tl.bin == 16 ? 4096u : 1024u);
}

// Adds the sum of n uint32 counts to *out.
void launch_sum_u64(const uint32_t* counts, uint32_t n, unsigned long long* out, hipStream_t s);

// Ranges of equal keys.  Keys >= n_tiles are ignored.  n_dev (optional,
// device): live pair count, clamped to n_pairs.
void launch_tile_ranges(const uint32_t* sorted_keys, uint32_t n_pairs, uint32_t n_tiles,
                        uint2* ranges, hipStream_t s, const uint32_t* n_dev = nullptr);

void launch_fill_u32(uint32_t* p, uint32_t v, uint64_t n, hipStream_t s);

// Exclusive scan of n uint32 values (sums stay at 2^32 - 1 from there on); total
// written to *total (device). Scratch
// must hold scan_scratch_words(n) words.
size_t scan_scratch_words(uint64_t n);
void launch_scan(const uint32_t* in, uint32_t* out, uint32_t n, uint32_t* total, uint32_t* scratch,
                 hipStream_t s);

size_t radix_scratch_words(uint32_t n);
// Bins by decreasing octave of their list length (floor log2 of
// ranges[b].y - ranges[b].x + 1; bin order within an octave) to order[0 ..
// n_bins), which holds tile_order_words(n_bins) words.
size_t tile_order_words(uint32_t n_bins);
void launch_tile_order(const uint2* ranges, uint32_t n_bins, uint32_t* order, hipStream_t s);
// Stable LSD radix sort of (key, value) by the low `bits` key bits, up to 8 per
// pass.  An odd pass count leaves the result in keys_alt/vals_alt
// (*result_in_alt = true).  n_dev (optional, device): the live count, clamped to
// n (the capacity the launches are sized for).
void radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                uint32_t n, int bits, uint32_t* scratch, hipStream_t s, const uint32_t* n_dev,
                bool* result_in_alt);
// The same for the group pairs of a batch's views (keys: global groups, `bits` of
// them; offsets: the emission's places of the items; max_groups: of a view), view
// by view where group_sort_by_view says so, which is one pass.
bool group_sort_by_view(uint64_t max_groups, int bits, int n_views, uint32_t n);
void launch_group_sort(const ViewInfo* views, int n_views, uint32_t n_items, uint64_t max_groups,
                       const uint32_t* offsets, uint32_t* keys, uint32_t* vals, uint32_t* keys_alt,
                       uint32_t* vals_alt, uint32_t n, int bits, uint32_t* scratch, hipStream_t s,
                       const uint32_t* n_dev, bool* result_in_alt);

// Accumulate variants ("chunks"): the channels per launch (launches =
// ceil(C / channels)), plus kChunkMfma for the matrix-core forms: BF16
// targets in blocks of 16, 32 or 64 channels per launch, or (kChunkMfma | 1)
// all channels and a ones column packed into one block of 16 (C <= 15 for
// BF16 targets, C <= 7 for FP32 targets, split into BF16 high and low parts).
constexpr int kChunkMfma = 128;
constexpr int kChunkPacked = kChunkMfma | 1;
inline int chunk_channels(int chunk) { return chunk & (kChunkMfma - 1); }
// Default variant for C channels of targets of type tdtype.
int accumulate_chunk(int C, int tdtype);
// `requested` if it is a valid variant that applies to C channels of type
// tdtype, else the default.
int resolve_chunk(int requested, int C, int tdtype);
// What launch_accumulate makes of a resolved variant: the variant (deterministic
// sums: of the vector form), whether it runs a wave per 8x8 block (few_tiles: the
// default vector variant as a grid; other variants and the persistent grid run as
// they were asked for), and the launches that take the channels.
struct AccumulateForm {
    int chunk;
    bool blocks;
    int launches;
};
AccumulateForm accumulate_form(const TileLists& tl, int C, int chunk, bool deterministic, bool persistent);

// The sums of one slot: *(v + slot * v_stride) and the C floats at s + slot *
// s_stride.  Interleaved slots of C + 1 floats, or (split_n slots) the S rows
// first and the V after them: rows of whole 64-byte units where C is a multiple
// of 16 (from an aligned base), so that 16 channels are one atomic request and
// not two.  Atomics leave the XCDs' caches (every request reaches the fabric)
// at about 14-16 G requests/s, which bounds the wide matrix-core accumulate: 8.1
// requests a row of 64 channels interleaved, 5 split (in launches of 32
// channels, where it mattered less, 15.56 -> 14.49 ms).
struct SumRows {
    float* v;
    float* s;
    int v_stride, s_stride;
};
inline SumRows sum_rows(float* VS, int C, int64_t split_n) {
    if (split_n > 0) return SumRows{VS + split_n * C, VS, 1, C};
    return SumRows{VS, VS + 1, C + 1, C + 1};
}
// Whether sums over views (one slot a Gaussian, read by the L = 0 solve alone)
// are kept split: for the matrix-core forms and whole blocks of 16 channels.
inline bool split_sums(bool per_view, int tdtype, int C, int chunk) {
    return !per_view && tdtype == GSC_BF16 && C % 16 == 0 && (chunk & kChunkMfma) && chunk != kChunkPacked;
}

// Accumulate V_gj and S_gj into slot (view.vs_base + g) when per_view, else
// into slot (view.g_offset + g), summed over views; slots hold C+1 floats.
// chunk: the accumulate variant (1, 2, 3, 4, 8 or 16 channels per launch, or
// kChunkMfma | 16, 32 or 64 for BF16 targets; anything else picks
// accumulate_chunk(C, tdtype)).  queues (device, one word per channel pass,
// zeroed here by a fill kernel): persistent launches of kPersistentBlocks
// blocks that take tiles from a counter; nullptr: a block per kTileWaves tiles.
// split_n: the slots of split sums (see sum_rows), 0: interleaved.
// det (non-null): deterministic form.  VS holds 64-bit fixed-point words
// (zero before the first launch); each tile's share is scaled by det->x
// (visibility column) or det->y (channel columns), powers of two, and added
// with integer atomics.  Vector form only (a matrix-core chunk falls back).
constexpr uint32_t kPersistentBlocks = 2048;  // 8 blocks of 4 waves per CU
bool accumulate_chunk_valid(int chunk, int tdtype);
void launch_accumulate(const TileLists& tl, const void* targets, int tdtype, int C, bool per_view,
                       BlendParams bp, float* VS, unsigned long long* counter, uint32_t* gcount,
                       int chunk, hipStream_t s, uint32_t* queues = nullptr,
                       const float2* det = nullptr, int64_t split_n = 0);

// Colour of batch item i (view v, Gaussian g of the N): gamma[i][c] =
// sum_m coeffs[g][m][c] phi_m(dir_gv).
void launch_view_colors(const ViewInfo* views, int n_views, int64_t N, const float* means,
                        const float* coeffs, int C, int sh_deg, float* gamma, hipStream_t s);

// Targets to subtract a render from (y null: none).
struct RenderResidual {
    const void* y = nullptr;
    int bf16 = 0;
};
int render_launches(const TileLists& tl, int C);
// Whether launch_render should form the residual; else launch_residual does, over n
// values of the images from `first`.
bool residual_in_render(const TileLists& tl, int C);
void launch_residual(const RenderResidual& res, int64_t first, int64_t n, float* images, hipStream_t s);
void launch_render(const TileLists& tl, const float* gamma, int C, BlendParams bp, float* images,
                   unsigned long long* counter, hipStream_t s, const RenderResidual& res = {});

// Fold the per-view sums into the regularised normal equations and solve.
// per_view: VS holds [n_views][N][C+1] (else [N][C+1] summed over views).
// wout (optional): w_g = sum_j V_gj.  dc_scratch: N*(C+1) floats, used when
// sh_deg == 0 and per_view.
// factor (optional, sh_deg >= 1): per Gaussian the Cholesky factor of
// A_g + w_g Lambda, packed by rows (row i at i (i + 1) / 2, 1/L_ii on the
// diagonal), then w_g: refine_factor_words(sh_deg) doubles.
// obs_scratch (sh_deg >= 1): fold_obs_words(N, n_views) words, 8-byte aligned;
// the unobserved Gaussians (no view saw them) are written directly and the fold
// runs over a list of the observed ones only.
void launch_fold_solve(const ViewInfo* views, int n_views, const float* means, const float* VS,
                       bool per_view, int64_t N, int C, int sh_deg, const double* lam_nb /*host, nb*/,
                       float kappa_max, float* coeffs, uint8_t* status, float* wout,
                       float* dc_scratch, unsigned int* ill_count, hipStream_t s,
                       double* factor = nullptr, uint32_t* obs_scratch = nullptr, bool split = false);
int64_t fold_obs_words(int64_t N, int n_views);
inline int refine_factor_words(int sh_deg) {
    const int nb = (sh_deg + 1) * (sh_deg + 1);
    return nb * (nb + 1) / 2 + 1;
}

// One refinement update (Algorithm 1, step 10): with the per-view sums VS of
// the residual targets (as for launch_fold_solve; per_view when sh_deg >= 1),
//   c_g += (A_g + w_g Lambda)^{-1} (sum_j phi_gj S_gj^T - w_g Lambda c_g)
// using the stored factor (sh_deg >= 1) or w (sh_deg == 0, where the matrix is
// w_g (Y0^2 + lambda_0)).  Gaussians whose status has UNOBSERVED or FAILED
// are left alone.
void launch_refine_update(const ViewInfo* views, int n_views, const float* means, const float* VS,
                          int64_t N, int C, int sh_deg, const double* lam_nb, const double* factor,
                          const float* w, const uint8_t* status, float* coeffs, hipStream_t s);

// Weights-only accumulate: V[slot] += sum_p w (stride 1; slots as in launch_accumulate).
void launch_accumulate_weights(const TileLists& tl, bool per_view, BlendParams bp, float* V,
                               unsigned long long* counter, hipStream_t s);

// Adjoint solve: bbar = (A_g + w_g Lambda)^{-1} grad_coeffs and
// rho_g = sum lambda_m bbar[m][c] coeffs[m][c].  V holds per-view
// visibilities [n_views][N] (per_view) or their sums [N].  w_scratch: N floats
// (sh_deg == 0 with per_view); obs_scratch as for launch_fold_solve.
void launch_adjoint_solve(const ViewInfo* views, int n_views, const float* means, const float* V,
                          bool per_view, int64_t N, int C, int sh_deg, const double* lam_nb,
                          const float* grad_coeffs, const float* coeffs, float* bbar, float* rho,
                          float* w_scratch, uint32_t* obs_scratch, hipStream_t s);

// Adjoint colours of batch item i: beta[i][beta_stride(C, width)] = (beta_gj, the
// parts of delta_gj), with beta = bbar^T phi and delta = beta^T (c^T phi) + rho_g; for
// a render (bbar null) beta = c^T phi, delta = 0.  delta has one part for every
// `width` channels (their products, and rho_g in the first): the launches of the blend
// adjoint take adjoint_channels channels each and their own part.  (beta^T y and delta
// nearly cancel where the fit is good; with all of delta in one launch the sums in
// between, and the rounding of their atomics, were of delta's size.  dL/do of 24
// random scenes, 3 to 64 channels, against 64 bits, geometric mean of the relative
// errors: 1.04e-5 -> 4.5e-6; 64 channels, 131 views of 17 splats 1.2e-4 -> 4.8e-6.)
int adjoint_channels(const TileLists& tl, int C);
__host__ __device__ inline int beta_stride(int C, int width) { return C + (C + width - 1) / width; }
void launch_view_adjoint(const ViewInfo* views, int n_views, int64_t N, const float* means,
                         const float* coeffs, const float* bbar, const float* rho, int C, int width,
                         int sh_deg, float* beta, hipStream_t s);

// Blend adjoint over the binned tiles: grad_y[row][c] = sum_g w beta (every
// pixel of every view written, if grad_y) and grad_o[g] += dL/do (atomics, if grad_o).
void launch_blend_adjoint(const TileLists& tl, const void* ypix, int ydtype, int C, const float* beta,
                          BlendParams bp, float* grad_y, float* grad_o, hipStream_t s);

// grad_coeffs[g][m][c] = sum_j phi_gj[m] S_gj[c] from per-view sums [n_views][N][C+1].
void launch_fold_rhs(const ViewInfo* views, int n_views, const float* means, const float* VS,
                     bool per_view, int64_t N, int C, int sh_deg, float* out, hipStream_t s);

// Input checks and the deterministic sums.
// Over n values of dtype GSC_F32 or GSC_BF16 at p: the smallest index of a
// non-finite value (atomicMin into *first_bad, which the caller sets to
// UINT64_MAX) and the largest |value| as binary32 bits (atomicMax into
// *absmax, set to 0 by the caller; NaN counts as larger than infinity).
void launch_scan_values(const void* p, int dtype, int64_t n, unsigned long long* first_bad,
                        uint32_t* absmax, hipStream_t s);
// out[i] = in[i] / scale, scale = 1/inv_v for column 0 of every row of
// `stride` words and 1/inv_s for the others (powers of two).
void launch_det_to_float(const unsigned long long* in, int64_t n, int stride, double inv_v,
                         double inv_s, float* out, hipStream_t s);

// View selection: one bitset per view of the Gaussians it observed
// (bits[v][w], (N + 63) / 64 words per view) from per-view weights V [n_views][N].
void launch_seen_bits(const float* V, int n_views, int64_t N, unsigned long long* bits, hipStream_t s);

// Post-processing.  Linear combination of up to kCombineSets coefficient sets
// per launch: out = filter * sum_k w_k p_k elementwise (filter by channel,
// i mod C, applied when `filter`); with `accumulate` the sum continues from
// out.
constexpr int kCombineSets = 16;
struct CombineArgs {
    const float* p[kCombineSets];
    float w[kCombineSets];
    float f[kMaxC];
    int n;
    int accumulate;
    int filter;
};
void launch_combine(const CombineArgs& a, int64_t n, int C, bool vec4, float* out, hipStream_t s);

// Segmentation filter over coeffs rows of `row` floats: keep[g] (optional),
// the kept indices in increasing order (optional) and their number (device
// int64, optional).  block_scratch: mask_blocks(N) words.
int mask_blocks(int64_t N);
// Exclusive scan in place of n_blocks counts (one block of 1024 threads);
// *total (if non-null) receives the sum.
void launch_block_scan(uint32_t* counts, int n_blocks, int64_t* total, hipStream_t s);
void launch_mask_filter(const float* coeffs, int64_t N, int64_t row, int channel, float thr,
                        const uint8_t* status, uint8_t* keep, int64_t* indices, int64_t* n_kept,
                        uint32_t* block_scratch, hipStream_t s);

}  // namespace gsc
