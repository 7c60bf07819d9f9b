// Internal declarations of the gfx950 hot path: device-side view table,
// workspace layout, launch wrappers. Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/skipgs.h"

namespace sgs {

constexpr int kWave = 64;
constexpr uint32_t kMaxExtent = 1u << 24;   // |u|, |v|, radius beyond this: degenerate, culled
constexpr int kRecordFloats = 12;           // u v a b | c o rx ry | r g b clamp-mask
constexpr int kAccumFloats = 12;            // du dv da db | dc do dr dg | db - - -
constexpr int kDefaultSuperTile = 8;        // super-tile edge in tiles
constexpr int kDefaultBatch = 64;           // list entries per compositing batch
constexpr int kDefaultSplitPrefix = 8192;   // super-tile list pairs split before compositing

// Per-view constants. A call's views live in device memory (the workspace's
// view table): the first launch of the call (the projection of one view, the
// preparation of the compositing backward, a launch of its own otherwise) stores
// them there, from the call's arguments or from a camera table picked by a
// device-side view index, and the kernels after it read them through a pointer.
struct ViewDev {
    float R[9];
    float t[3];
    float fx, fy, cx, cy;
    float C[3];          // camera centre in world coordinates, -R^T t
    float lim_x, lim_y;  // clamp of tx/tz, ty/tz in the EWA Jacobian (inf: off)
    int32_t width, height, tiles_x, tiles_y;
    int32_t tile_offset; // first global tile index of the view
    int32_t sup_x, sup_y;   // super-tiles per row and column
    int32_t sup_offset;     // first global super-tile index of the view
    int64_t px_offset;   // first global pixel index of the view
};

struct Views {
    ViewDev v[SGS_MAX_VIEWS];
    int32_t n;
    int32_t total_tiles;
    int64_t total_pixels;
    int32_t total_supers;
    int32_t pad;
};

struct RasterDev {
    int32_t tile_w, tile_h;
    int32_t super_tile;    // super-tile edge in tiles
    int32_t batch;         // list entries per compositing batch (and per list chunk)
    int32_t key_bits;      // low bits of a pair key: the super-tile index
    int32_t rect_bits;     // bits per coordinate of the tile rectangle above them
    int32_t prefix_segs;   // 512-pair segments of a long super-tile list split before compositing (0: all)
    int32_t seg_log2;      // log2 of the pairs a wave of the split takes
    float bg[3];
    float near_z, dilation, alpha_min, alpha_max, t_min;
    float log2_alpha_min;  // log2(alpha_min), rounded from binary64 (-inf for 0)
};

// Adam constants: beta and 1 - beta formed in binary64, then rounded.
struct AdamDev {
    float b1, b2, c1, c2, eps;
    double beta1, beta2;  // for the bias corrections
    float lr[SGS_MAX_PLANES];
};
struct AdamStep {
    float ibc1, ibc2;  // 1 / (1 - beta^k), formed in binary64
};
AdamDev make_adam(const sgs_adam_params* p);

// Counters region of the workspace (uint32 words).
enum Counter : int {
    kStatus = 0,        // SGS_STATUS_* bits
    kVisible = 1,       // visible entries of the last forward
    kPairs = 2,         // (super-tile, entry) pairs needed by the last forward (saturating)
    kPairsWritten = 3,  // min(pairs, capacity)
    kBlended = 4,       // uint64 at words 4-5: blended (pixel, Gaussian) pairs of the last rasterize
    kEvaluated = 6,     // uint64 at words 6-7: (pixel, list entry) pairs the forward examined
    kPairsKept = 8,     // super-tile pairs left after the reach test (length of the sorted lists)
    kItems = 9,         // tile-list entries needed (saturating)
    kSegments = 10,     // super-tile list segments of the tile-list split
    kUsed = 11,         // tile-list entries up to each tile's last blended one (summed)
    kItemsRest = 12,    // tile-list entries of the completing split (saturating)
    kRedo = 13,         // 1: a tile reached the end of its list prefix with live pixels
    kNumCounters = 16
};

// A visible entry's mark (one byte; 0 for the others): this bit, and bits 0-2
// for the colour channels the forward did not clamp at 0. The same bits lie in
// the record's last word, but a backward that reads them there fetches all
// records.
constexpr uint32_t kMarkVisible = 8u;

// Pair key (uint32): the super-tile index in the low key_bits bits (a value
// below 2^key_bits - 1, so that no key has all bits set), and above them the
// entry's tile rectangle inside the super-tile, four coordinates of
// rect_bits bits (first column, last column, first row, last row, relative to
// the super-tile). Only the index is sorted on; the rectangle rides along to
// the split of the super-tile lists into tile lists. The key of an emitted
// pair whose Gaussian cannot reach alpha_min on the super-tile has all bits
// set; the first pass of the super-tile sort drops such pairs.
constexpr uint32_t kCulledTile = 0xffffffffu;
constexpr int kMaxSuperTile = 8;   // S x S tiles of a super-tile fit a 64-bit tile mask

// Emission units: each visible Gaussian (in depth order) owns kEmitHead
// header units followed by one unit per pair; a workgroup of the emission
// kernel covers a window of kEmitWindow consecutive units, so it meets at
// most kEmitWindow / (kEmitHead + 1) + 2 Gaussians.
constexpr int64_t kEmitWindow = 1024;
constexpr int64_t kEmitHead = 2;
// Super-tiles up to which the pairs are counted and placed without a sort: the
// place kernel keeps 24 bytes of LDS for each, and a wave's counts are the sparser
// the more there are. us of projection and binning, placed / sorted: 425
// super-tiles (3M Gaussians) 605 / 656, 468 (1M in 4 views) 613 / 751, 494 (2M in 8)
// 1687 / 2076; beyond the line 782 (3M) 796 / 810, 936 (2M in 8) 2265 / 2407, 936
// (300k in 8) 653 / 631.
constexpr int64_t kDirectSupers = 512;
constexpr int kPairThreads = 256;
constexpr int kPairEntries = 768;   // entries expanded at a time
constexpr int64_t kPairGroup = 32;   // blocks whose pair counts are summed up together

// Windows of an emission over `entries` entries and `capacity` pairs.
constexpr int64_t emit_windows(int64_t entries, int64_t capacity) {
    return (capacity + kEmitHead * entries + kEmitWindow - 1) / kEmitWindow;
}

// The split of the super-tile lists into tile lists. The prefix of a long list
// counts in units of kSegPairs pairs.
constexpr int64_t kSegPairs = 512;

// With a split prefix, a super-tile list longer than kCutFactor prefixes is
// split only in its first prefix_segs units before compositing (the tiles
// that composite a whole short list, often into the background, never wait
// for a second split; long lists are where the split's work is).
constexpr uint32_t kCutFactor = 4;
__host__ __device__ constexpr uint32_t list_units(uint32_t len) {
    return (uint32_t)(((uint64_t)len + kSegPairs - 1) / kSegPairs);
}
// Whether a list of at most `len` pairs can be cut, and the pairs of one that
// are split before compositing.
__host__ __device__ constexpr bool list_cut(uint32_t len, uint32_t prefix_segs) {
    return prefix_segs > 0 && list_units(len) > (uint64_t)kCutFactor * prefix_segs;
}
__host__ __device__ constexpr uint32_t split_pairs(uint32_t len, uint32_t prefix_segs) {
    return list_cut(len, prefix_segs) ? prefix_segs * (uint32_t)kSegPairs : len;
}
// A wave of the split takes a segment of 2^seg_log2 consecutive pairs (64 to
// 512) of one super-tile's list: short ones where there are few pairs, since
// every 64 pairs are a step of a chain of loads, long ones where there are many,
// since every segment adds to its super-tile's counts by atomics. us of all split
// kernels for 64 / 128 / 256 / 512 pairs: 1000 entries 16 / 22 / 32 / 51, 30k 23 /
// 26 / 39 / 66, 300k 78 / 54 / 56 / 78, 1M 105 / 72 / 64 / 84, 3M 153 / 109 / 103 /
// 109, 6M (with a completing split) 136 / 111 / 117 / 168, 16M 1168 / 712 / 555 /
// 506.
constexpr int seg_log2_for(int64_t entries) {
    return entries <= (1 << 16) ? 6 : entries <= (1 << 19) ? 7 : entries <= (1 << 23) ? 8 : 9;
}
// Slots: an upper bound on the segments of any batch with `capacity` pairs, and
// on the groups of kSegGroup segments whose tile counts are summed up together
// (group j of super-tile s: slot first segment / kSegGroup + s + j).
constexpr int64_t kSegGroup = 16;
constexpr int64_t segment_slots(int64_t capacity, int64_t supers, int seg_log2) {
    return ((capacity - 1) >> seg_log2) + 1 + supers;
}
constexpr int64_t segment_group_slots(int64_t slots, int64_t supers) {
    return slots / kSegGroup + supers + 1;
}
// Per tile (tile_state):
enum TileState : uint32_t {
    kTileWhole = 0,       // the tile's list is whole
    kTileTruncated = 1,   // its super-tile's list is longer than the prefix
    kTileIncomplete = 2,  // truncated, and a pixel was still live at the end of the list
};

struct Layout {
    int64_t entries, total_tiles, total_pixels, total_supers, capacity, seg_slots;
    int n_views;
    int64_t scan_blocks;
    int64_t pair_blocks;   // blocks of the direct pair path
    int pair_rounds;       // kPairEntries entries each there
    int seg_log2;
    int key_bits, rect_bits, key_result;  // result buffer (0/1) of the super-tile lists
    int batch;
    bool direct;           // pairs counted and placed directly (few super-tiles)
    size_t views, records, tiles, depth, dkey[2], dval[2], offsets, window_first, scan_sums,
        pair_info, pair_sorted, pair_hist, pair_groups, pair_key[2], pair_entry[2], sort_hist, sort_groups,
        pair_sort_groups, sort_weights, sup_ranges, seg_first, seg_cnt, seg_groups[2],
        sup_items[2], sup_base, pair_mask, tile_entry, tile_ranges, tile_state, tile_resume, sup_redo, tile_cost,
        marks, tile_stats, tile_order, t_final, n_last, accum, counters, total;
    // the region a binning pass accumulates into and finds cleared
    size_t clear_begin, clear_words;
};

// Whether a super-tile list of the batch can be cut by the split prefix (a list
// holds at most one view's Gaussians).
inline bool lists_cut(const RasterDev& rp, const Layout& L) {
    return list_cut((uint32_t)(L.entries / L.n_views), (uint32_t)rp.prefix_segs);
}

bool make_views(const sgs_camera* cams, int n_views, const sgs_raster_params* rp, Views* out,
                const char** err);
void make_layout(const Views& views, const RasterDev& rp, int64_t n, int64_t capacity, Layout* L);
RasterDev make_raster(const sgs_raster_params* rp);

// The call's views into the workspace's view table; the sums of compositing's
// work in counters (nullable) are cleared, step (nullable) is incremented unless
// the gate is closed.
hipError_t launch_store_views(const Views& views, Views* dst, hipStream_t s,
                              uint32_t* counters = nullptr, int32_t* step = nullptr,
                              const int32_t* gate = nullptr);
// The same for a call that bins: the views from the host (by value) or, when
// `table` is non-null, view `*d_view` of a device camera table (clamped into
// [0, n_table)) as the batch's single view; and the counters and the region of
// the workspace that binning accumulates into cleared.
hipError_t launch_begin_bin(const Views& views, const ViewDev* table, int n_table,
                            const int32_t* d_view, const Layout& L, char* ws, hipStream_t s);

// ---- launch wrappers (all asynchronous on `s`). Kernels read the views from
// the workspace's view table (ws + L.views); L carries the sizes. ----
// Projection; it also does what the first launch of its call has to (the views
// stored; with `bins` the counters and sums cleared, as launch_begin_bin).
struct CallViews {
    const Views* views;
    const ViewDev* table;   // as launch_begin_bin
    int n_table;
    int32_t* d_view;
    bool bins;
    const int32_t* seq = nullptr;   // nullable; otherwise *d_view = seq[*iter % len] first
    int64_t len = 0;
    const int64_t* iter = nullptr;
};
hipError_t launch_project(const float* planes, int64_t n, int64_t stride, int sh_degree,
                          const RasterDev& rp, const Layout& L, char* ws, const CallViews& call,
                          hipStream_t s);
hipError_t launch_load_records(const float* u, const float* v, const float* depth,
                               const int32_t* extent, const float* conic, const float* opacity,
                               const float* rgb, int64_t n, const RasterDev& rp, const Layout& L,
                               char* ws, hipStream_t s);
hipError_t launch_bin(const RasterDev& rp, int64_t n, const Layout& L, char* ws, hipStream_t s);
// After a compositing forward over list prefixes: the whole lists of the
// super-tiles that have a tile marked incomplete (tile_state 2), appended
// after the prefix lists, and the new ranges of the incomplete tiles. Every
// kernel returns at once unless counters[kRedo] is set.
hipError_t launch_split_rest(const RasterDev& rp, const Layout& L, char* ws, hipStream_t s);
// Waves that take a tile in the compositing passes of a batch.
struct TileWaves {
    int forward, backward;
};
TileWaves tile_waves(int tile_w, int64_t tiles);
hipError_t launch_rasterize(const RasterDev& rp, const Layout& L, char* ws, float* out_rgb,
                            hipStream_t s);
// What comes before the compositing backward: Adam's step count (nullable), the
// accumulators to clear (float4s), the tiles to order by their cost.
struct Prepare {
    int32_t* step;
    float4* accum;
    int64_t n4;
    const uint32_t* cost;
    int64_t tiles;
    uint32_t* order;
};
Prepare backward_preparation(const Layout& L, char* ws, int32_t* step);
// views (nullable): stored into the workspace first. step (nullable): Adam's
// step count, incremented unless the gate is closed. prepared: an earlier launch
// has done backward_preparation(L, ws, step).
hipError_t launch_rasterize_backward(const RasterDev& rp, const Layout& L, char* ws,
                                     const float* dl_drgb, const int32_t* gate, hipStream_t s,
                                     const Views* views, int32_t* step = nullptr,
                                     bool prepared = false);
hipError_t launch_project_backward(const float* planes, int64_t n, int64_t stride,
                                   int sh_degree, const RasterDev& rp, const Layout& L, char* ws,
                                   const int32_t* gate, float* grads, bool write, hipStream_t s);

// p[0..n) = v on stream s (a kernel, so that callers can be captured).
hipError_t fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s);
// Stable LSD radix sorts of (key, uint32 value) pairs. `hist`: 256 words per
// block; `groups`: radix_group_words words of zeros per call.
constexpr int64_t kSortGroup = 32;   // blocks whose digit counts are summed up together
constexpr int kDepthPasses = 4;
int radix_passes(int bits);
int64_t radix_blocks(int64_t n_max);
int64_t radix_group_words(int64_t n_max, int passes);
// The visible entries (tiles[e] != 0) of `entries` by their depth bits, ties in
// entry order, into vals[1]; their number to *n_visible and the saturated sum
// of tiles[] to *pairs. weights: a word of 8 bytes per block.
hipError_t sort_entries(const uint32_t* depth, const uint32_t* tiles, int64_t entries,
                        uint32_t* keys[2], uint32_t* vals[2], uint32_t* hist, uint32_t* groups,
                        uint64_t* weights, uint32_t* n_visible, uint32_t* pairs, hipStream_t s);
// *n_dev (<= n_max) pairs by the low `bits` bits of their keys, those with all
// bits set (kCulledTile) left out; the number of the others to *kept. The
// result is in keys[radix_passes(bits) & 1], vals likewise.
hipError_t sort_pairs(uint32_t* keys[2], uint32_t* vals[2], const uint32_t* n_dev, int64_t n_max,
                      int bits, uint32_t* hist, uint32_t* groups, uint32_t* kept, hipStream_t s);

// Adaptive density control. Thresholds as the kernels compare them (float32
// values formed in binary64 on the host).
struct DensifyDev {
    float grad_threshold;   // the statistic's mean at or above which a Gaussian densifies
    float log_size;         // log(percent_dense * scene_extent): larger max log-scale splits
    float logit_min;        // logit(min_opacity): a smaller opacity logit prunes
    float log_split;        // log(split_scale), subtracted from the children's log-scales
};
int64_t densify_blocks(int64_t n);
// Scratch words of a step over n Gaussians.
constexpr int64_t densify_scratch_words(int64_t blocks) { return 4 * blocks + 3; }
hipError_t launch_densify_stats(const Layout& L, char* ws, int64_t n, const int32_t* gate,
                                float* grad_sum, int32_t* count, hipStream_t s);
hipError_t launch_densify(const DensifyDev& d, float* params, float* m, float* v, int64_t n,
                          int64_t stride, int F, const float* grad_sum, const int32_t* count,
                          const float* normals, float* out_params, float* out_m, float* out_v,
                          int64_t out_stride, uint32_t* scratch, int64_t* n_out, hipStream_t s);

// Loss / gate / Adam
// target: the reference image, or with d_view non-null the image
// *d_view (clamped into [0, n_targets)) of an array of n_targets images.
struct TargetRef {
    const float* base;
    const int32_t* d_view;
    int32_t n_targets;
};
// What a training iteration decides once it has the loss: the gate's update or,
// without a state, an open gate.
struct GateArgs {
    double beta, eps, delta, rho_lo;
    int32_t warmup, window, calibrate, budget, n_views;
};
GateArgs gate_args(const sgs_gate_params* p);
struct LossGate {
    GateArgs args;
    char* state;            // nullable
    const int32_t* view;
    int32_t* gate;          // nullable: nothing to decide
    int64_t* iter;          // nullable: the position in the view sequence, advanced
};
hipError_t launch_loss_forward(const float* rgb, TargetRef target, int w, int h, float lambda,
                               char* ws, float* d_loss, hipStream_t s,
                               const LossGate& gate = LossGate{});
hipError_t launch_loss_backward(const float* rgb, TargetRef target, int w, int h, float lambda,
                                char* ws, const int32_t* gate, float* dl, hipStream_t s,
                                const float* scale = nullptr);
// The backward of a training iteration: the loss's gradient and the preparation
// of the compositing backward and, where no gate decides on the loss, the sum of
// the loss itself (launch_loss_forward then leaves it: gate.gate null).
hipError_t launch_train_loss(const float* rgb, TargetRef target, int w, int h, float lambda,
                             char* ws, float* d_loss, float* dl, const LossGate& gate,
                             const Prepare& prepare, hipStream_t s);
size_t loss_workspace_bytes(int w, int h);
// The loss forward with its partial sums (kLossPartials values, for any image) in
// caller-provided device memory.
constexpr int64_t kLossPartials = 2048;
hipError_t launch_loss_partials(const float* rgb, TargetRef target, int w, int h, float lambda,
                                double* partials, float* d_loss, hipStream_t s);

hipError_t launch_gate_init(const sgs_gate_params* p, void* state, hipStream_t s);
hipError_t launch_gate_update(const sgs_gate_params* p, void* state, const int32_t* view,
                              const float* loss, int32_t* gate, hipStream_t s);
size_t gate_state_bytes(const sgs_gate_params* p);
// *d_view = seq[*d_iter % len]; *d_iter += 1.
hipError_t launch_sequence_next(const int32_t* seq, int64_t len, int64_t* d_iter, int32_t* d_view,
                                hipStream_t s);

hipError_t launch_adam(const sgs_adam_params* p, float* params, float* grads, float* m, float* v,
                       int64_t n, int64_t stride, int n_planes, int32_t* step,
                       const int32_t* gate, hipStream_t s);
hipError_t launch_adam_count(int32_t* step, const int32_t* gate, hipStream_t s);
// step: the count of this step, incremented by an earlier launch.
// sparse: update only the Gaussians visible in a view of the batch (the
// others keep their parameters and moments); dense otherwise.
hipError_t launch_project_backward_adam(float* planes, int64_t n, int64_t stride, int sh_degree,
                                        const RasterDev& rp, const Layout& L, char* ws,
                                        const sgs_adam_params* prm, bool sparse, float* m,
                                        float* v, const int32_t* step, const int32_t* gate,
                                        hipStream_t s);

}  // namespace sgs
