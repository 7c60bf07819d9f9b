// Binning: the depth-ordered tile lists the tile-based rasteriser composites.
//
// The lists are built in two levels. First at the granularity of super-tiles
// (squares of S x S tiles): the stage sorts the visible entries once by depth (a
// short array) and lists them, in that order, under every super-tile they reach.
// Up to kDirectSupers super-tiles the places in these lists are counted and the
// pairs written there; beyond, the (super-tile, entry) pairs are emitted in depth
// order and sorted stably by super-tile alone, which keeps the depth order inside
// each, as a sort of 64-bit (super-tile << 32 | depth) keys would. A pair's key is
// the super-tile index and, in its upper bits, the entry's tile rectangle inside
// the super-tile. A super-tile's list holds the visible entries whose overlap box
// reaches it and that can reach alpha_min at one of its pixel centres.
//
// Then every super-tile list is split into the lists of its S x S tiles, in
// list order: per segment of a super-tile list, each pair's tile mask (the
// tiles of its rectangle on which the entry can reach alpha_min) and per-tile
// counts with their sums over groups of segments and over super-tiles, from which
// every segment finds its list positions, and a stable scatter of the entries. A
// tile's list is therefore its depth-ordered list of entries whose overlap box
// reaches it and that can reach alpha_min on it; no sort sees the (far more
// numerous) tile pairs.
//
// A tile composites only the front of its list, so a long super-tile list is
// split only in a prefix of its segments before compositing (a tile's list is
// then a prefix of its whole list). The compositing marks the tiles whose
// prefix ran out while pixels were still live; the completing split then
// splits the whole lists of their super-tiles after the prefix lists and
// points those tiles' ranges there, and the compositing resumes them.
#include <algorithm>

#include "sgs_internal.hpp"
#include "sgs_device.hpp"

namespace sgs {

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

// ---- source and sink of the emission's device-wide scan ----
// The scans add in uint32 with saturation at 2^32 - 1 (saturating addition is
// associative, so the block and grand totals are the saturated true sums): a
// batch whose pair count does not fit ends with the all-ones total, which no
// capacity (< 2^31) reaches, and every offset past the overflow saturates.
struct PairCountSrc {  // super-tiles touched, in depth order
    const uint32_t* tiles;
    const uint32_t* sorted_entry;
    const uint32_t* n_dev;
    __device__ int64_t count() const { return *n_dev; }
    __device__ uint32_t operator()(int64_t k) const { return tiles[sorted_entry[k]]; }
};
// Pair offset of every Gaussian in depth order, and for every emission window
// (kEmitWindow consecutive emission units, windows 0 .. n_windows) the
// Gaussian whose units hold the window's first unit. Gaussian k owns units
// [pos + kEmitHead k, pos + kEmitHead (k + 1) + v). A saturated offset lies
// beyond every window.
struct OffsetSink {
    uint32_t* offsets;
    uint32_t* window_first;
    uint32_t n_windows;
    __device__ void operator()(int64_t k, uint32_t v, uint32_t pos) const {
        offsets[k] = pos;
        const uint64_t first = (uint64_t)pos + (uint64_t)kEmitHead * (uint64_t)k;
        const uint64_t end = first + (uint64_t)kEmitHead + v;
        for (uint64_t w = (first + kEmitWindow - 1) / kEmitWindow;
             w <= n_windows && w * kEmitWindow < end; ++w)
            window_first[w] = (uint32_t)k;
    }
};

__device__ __forceinline__ uint32_t sat_add(uint32_t a, uint32_t b) {
    const uint32_t c = a + b;
    return c < a ? 0xffffffffu : c;
}

// Inclusive saturating prefix sum over the lanes of a wave.
__device__ __forceinline__ uint32_t wave_incl_sat_scan(uint32_t v) {
    const int l = __lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(v, d, 64);
        if (l >= d) v = sat_add(v, o);
    }
    return v;
}

// Exclusive saturating scan over a block of NT threads; *total = block sum.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_sat_scan(uint32_t v, uint32_t* smem,
                                                        uint32_t* total) {
    constexpr int NW = NT / 64;
    const int w = threadIdx.x / 64;
    const int l = __lane_id();
    const uint32_t inc = wave_incl_sat_scan(v);
    if (l == 63) smem[w] = inc;
    __syncthreads();
    if (w == 0) {
        const uint32_t x = (l < NW) ? smem[l] : 0u;
        const uint32_t xi = wave_incl_sat_scan(x);
        const uint32_t ex = __shfl_up(xi, 1, 64);
        if (l < NW) smem[l] = l == 0 ? 0u : ex;
        if (l == NW - 1) smem[NW] = xi;
    }
    __syncthreads();
    // exclusive prefix of this thread = block prefix of its wave + the wave's
    // exclusive prefix (lane l - 1's inclusive value)
    const uint32_t wex = __shfl_up(inc, 1, 64);
    const uint32_t r = sat_add(smem[w], l == 0 ? 0u : wex);
    *total = smem[NW];
    __syncthreads();
    return r;
}

// Block sums of the scan input.
template <class Src>
__global__ void __launch_bounds__(kScanThreads) scan_reduce_kernel(Src src, uint32_t* sums) {
    __shared__ uint32_t smem[kScanThreads / 64 + 1];
    const int64_t n = src.count();
    // blocks past the count (the grid covers a bound) contribute 0
    if ((int64_t)blockIdx.x * kScanTile >= n) {
        if (threadIdx.x == 0) sums[blockIdx.x] = 0u;
        return;
    }
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j)
        if (base + j < n) s = sat_add(s, src(base + j));
    uint32_t tot;
    block_excl_sat_scan<kScanThreads>(s, smem, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Second and last kernel of the scan: every block adds up the sums of the
// blocks before it (a few thousand L2-resident words), scans its own tile and
// feeds the sink; the last block writes the grand total.
template <class Src, class Sink>
__global__ void __launch_bounds__(kScanThreads) scan_down_kernel(Src src, Sink sink,
                                                                 const uint32_t* sums,
                                                                 uint32_t* total) {
    __shared__ uint32_t smem[kScanThreads / 64 + 1];
    const int64_t n = src.count();
    // blocks past the count have nothing to feed; the last one still writes
    // the total
    const bool last = blockIdx.x == gridDim.x - 1;
    if ((int64_t)blockIdx.x * kScanTile >= n && !last) return;
    uint32_t before = 0;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += kScanThreads) before = sat_add(before, sums[i]);
    uint32_t prefix;
    block_excl_sat_scan<kScanThreads>(before, smem, &prefix);
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    uint32_t v[kScanItems];
    uint32_t s = 0;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        v[j] = (base + j < n) ? src(base + j) : 0u;
        s = sat_add(s, v[j]);
    }
    uint32_t tot;
    uint32_t pos = sat_add(block_excl_sat_scan<kScanThreads>(s, smem, &tot), prefix);
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
        if (base + j < n) sink(base + j, v[j], pos);
        pos = sat_add(pos, v[j]);
    }
    if (last && threadIdx.x == 0) *total = sat_add(prefix, tot);
}

template <class Src, class Sink>
hipError_t device_scan(Src src, Sink sink, int64_t n_max, uint32_t* sums, uint32_t* total,
                       hipStream_t s) {
    const int nb = (int)((n_max + kScanTile - 1) / kScanTile);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(scan_reduce_kernel<Src>, dim3(nb), dim3(kScanThreads), 0, s, src, sums);
    hipLaunchKernelGGL((scan_down_kernel<Src, Sink>), dim3(nb), dim3(kScanThreads), 0, s, src,
                       sink, sums, total);
    return hipGetLastError();
}

// Pair emission, load balanced over emission units (a few header units per
// Gaussian, then one per pair): each workgroup takes a fixed window of
// kEmitTile consecutive units. The Gaussians (in depth order) whose units meet
// the window run from the one holding the window's first unit to the one
// holding the next window's first unit (both recorded by the offset scan); the
// header units bound their number, and so the LDS a workgroup needs (more
// workgroups in flight hide the dependent loads of each). Their super-tile
// rectangles are staged in LDS, a max-scan of their start positions gives
// every window position its Gaussian, and every thread expands its pairs to
// (key, entry) with coalesced stores. Pair q of a Gaussian is super-tile
// (x0 + q % w, y0 + q / w) of its super-tile rectangle, row-major; its key
// packs the super-tile index and the part of the Gaussian's tile rectangle
// inside that super-tile. With alpha_min > 0, pairs whose Gaussian cannot
// reach alpha_min on the super-tile's pixels in the image get the all-ones
// key (kCulledTile).
constexpr int kEmitThreads = 256;
constexpr int kEmitItems = 4;
constexpr int kEmitTile = kEmitThreads * kEmitItems;
static_assert(kEmitTile == kEmitWindow, "emission window size");
// Gaussians meeting one window: each owns at least kEmitHead + 1 units.
constexpr int kEmitMaxG = kEmitTile / (kEmitHead + 1) + 2;

__global__ void __launch_bounds__(kEmitThreads) emit_kernel(
    const uint32_t* __restrict__ sorted_entry, const uint32_t* __restrict__ offsets,
    const uint32_t* __restrict__ window_first, const float4* __restrict__ rec,
    uint32_t* __restrict__ counters, int64_t n, const Views* __restrict__ views, RasterDev rp,
    int64_t capacity, uint32_t* __restrict__ pkey, uint32_t* __restrict__ pentry) {
    __shared__ uint32_t s_off[kEmitMaxG];
    __shared__ uint32_t s_ent[kEmitMaxG];
    __shared__ uint32_t s_base[kEmitMaxG];   // global super-tile of the rectangle's first one
    __shared__ uint16_t s_w[kEmitMaxG];      // rectangle width in super-tiles
    __shared__ uint16_t s_tx[kEmitMaxG];     // super-tiles per row of the Gaussian's view
    __shared__ uint16_t s_x0[kEmitMaxG];     // first super-tile column and row of the rectangle
    __shared__ uint16_t s_y0[kEmitMaxG];
    __shared__ uint16_t s_iw[kEmitMaxG];     // image size of the Gaussian's view
    __shared__ uint16_t s_ih[kEmitMaxG];
    __shared__ uint16_t s_tr[kEmitMaxG][4];  // tile rectangle [x0, x1) x [y0, y1)
    __shared__ float s_lim[kEmitMaxG];       // reach limit on a super-tile
    __shared__ float4 s_r0[kEmitMaxG];       // record words u v a b, c o rx ry
    __shared__ float4 s_r1[kEmitMaxG];
    __shared__ uint32_t s_own[kEmitTile];    // window position -> owning Gaussian
    __shared__ uint32_t s_scan[kEmitThreads / 64 + 1];
    // pairs written = min(pairs needed, capacity); block 0 records it and
    // flags an overflow (the tile sort reads the count after this kernel)
    const uint32_t total = counters[kPairs];
    const uint32_t P = (int64_t)total > capacity ? (uint32_t)capacity : total;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        counters[kPairsWritten] = P;
        if ((int64_t)total > capacity) counters[kStatus] |= SGS_STATUS_PAIR_OVERFLOW;
    }
    const uint32_t nvis = counters[kVisible];
    const int win = blockIdx.x;
    const uint64_t c0 = (uint64_t)win * kEmitTile;   // first unit of the window
    const uint64_t units = (uint64_t)total + (uint64_t)kEmitHead * nvis;
    if (c0 >= units) return;   // uniform across the workgroup
    const int tid = threadIdx.x;
    const uint32_t k0 = window_first[win];
    // the next window's first Gaussian exists whenever units continue past
    // this window; otherwise the window ends with the last visible Gaussian
    const uint32_t k1 = c0 + kEmitTile < units ? window_first[win + 1] : nvis - 1u;
    const uint32_t cnt = k1 - k0 + 1u;
    if (k1 < k0 || cnt > (uint32_t)kEmitMaxG) return;   // cannot happen: the header bound
#pragma unroll
    for (int it = 0; it < kEmitItems; ++it) s_own[it * kEmitThreads + tid] = 0u;
    __syncthreads();
    for (uint32_t j = tid; j < cnt; j += kEmitThreads) {
        const uint32_t k = k0 + j;
        const uint32_t e = sorted_entry[k];
        const ViewDev& V = views->v[(int)(e / n)];
        const float4 r0 = rec[3 * (int64_t)e], r1 = rec[3 * (int64_t)e + 1];
        int x0, x1, y0, y1, sx0, sx1, sy0, sy1;
        tile_rect(r0.x, r0.y, (int)r1.z, (int)r1.w, rp.tile_w, rp.tile_h, V.tiles_x, V.tiles_y,
                  &x0, &x1, &y0, &y1);
        super_rect(x0, x1, y0, y1, rp.super_tile, &sx0, &sx1, &sy0, &sy1);
        const uint32_t off = offsets[k];
        s_off[j] = off;
        s_ent[j] = e;
        s_base[j] = (uint32_t)(V.sup_offset + sy0 * V.sup_x + sx0);
        s_w[j] = (uint16_t)(sx1 - sx0);
        s_tx[j] = (uint16_t)V.sup_x;
        s_x0[j] = (uint16_t)sx0;
        s_y0[j] = (uint16_t)sy0;
        s_iw[j] = (uint16_t)V.width;
        s_ih[j] = (uint16_t)V.height;
        s_tr[j][0] = (uint16_t)x0;
        s_tr[j][1] = (uint16_t)x1;
        s_tr[j][2] = (uint16_t)y0;
        s_tr[j][3] = (uint16_t)y1;
        s_lim[j] = super_limit(reach_limit(r1.y, rp));
        s_r0[j] = r0;
        s_r1[j] = r1;
        // mark where this Gaussian's units start inside the window
        const uint64_t first = (uint64_t)off + (uint64_t)kEmitHead * k;
        if (j > 0 && first - c0 < (uint64_t)kEmitTile) s_own[first - c0] = j;
    }
    __syncthreads();
    // owner of every window position = the last Gaussian starting at or
    // before it: inclusive max-scan of the start marks (thread t scans
    // positions kEmitItems t .. kEmitItems (t + 1) - 1, then the block
    // combines the per-thread maxima)
    {
        uint32_t run[kEmitItems];
        uint32_t m = 0;
#pragma unroll
        for (int i = 0; i < kEmitItems; ++i) {
            m = max(m, s_own[tid * kEmitItems + i]);
            run[i] = m;
        }
        const uint32_t before = block_excl_max_scan<kEmitThreads>(m, s_scan);
#pragma unroll
        for (int i = 0; i < kEmitItems; ++i) s_own[tid * kEmitItems + i] = max(before, run[i]);
    }
    __syncthreads();
    // test and store every item (the records were staged in LDS once per
    // Gaussian); header units and units past the written pairs do nothing
#pragma unroll
    for (int it = 0; it < kEmitItems; ++it) {
        const uint64_t c = c0 + (uint64_t)(it * kEmitThreads + tid);
        const uint32_t j = s_own[it * kEmitThreads + tid];
        const uint64_t first = (uint64_t)s_off[j] + (uint64_t)kEmitHead * (k0 + j);
        const bool is_pair = c < units && c >= first + (uint64_t)kEmitHead;
        const uint32_t q = is_pair ? (uint32_t)(c - first - (uint64_t)kEmitHead) : 0u;
        const uint32_t p = s_off[j] + q;
        if (!is_pair || p >= P) continue;
        const float4 g0 = s_r0[j], g1 = s_r1[j];
        const uint32_t w = s_w[j];
        // q / w and q % w through a float reciprocal, corrected to exact
        uint32_t qy = (uint32_t)((float)q * __builtin_amdgcn_rcpf((float)w));
        int32_t qx = (int32_t)(q - qy * w);
        while (qx < 0) { --qy; qx += (int32_t)w; }
        while (qx >= (int32_t)w) { ++qy; qx -= (int32_t)w; }
        // the super-tile's pixels inside the image
        const int sw = rp.super_tile * rp.tile_w, sh = rp.super_tile * rp.tile_h;
        const int px0 = ((int)s_x0[j] + qx) * sw, py0 = ((int)s_y0[j] + (int)qy) * sh;
        const bool keep = s_lim[j] == INFINITY ||
                          rect_reachable(g0.x, g0.y, g0.z, g0.w, g1.x, s_lim[j], g1.z, g1.w, px0,
                                         py0, min(sw, (int)s_iw[j] - px0),
                                         min(sh, (int)s_ih[j] - py0));
        // the tile rectangle inside the super-tile, relative to its first tile
        const int S = rp.super_tile;
        const int ox = ((int)s_x0[j] + qx) * S, oy = ((int)s_y0[j] + (int)qy) * S;
        const uint32_t lx0 = (uint32_t)(max((int)s_tr[j][0], ox) - ox);
        const uint32_t lx1 = (uint32_t)(min((int)s_tr[j][1], ox + S) - 1 - ox);
        const uint32_t ly0 = (uint32_t)(max((int)s_tr[j][2], oy) - oy);
        const uint32_t ly1 = (uint32_t)(min((int)s_tr[j][3], oy + S) - 1 - oy);
        const int rb = rp.rect_bits;
        const uint32_t rect = lx0 | (lx1 << rb) | (ly0 << (2 * rb)) | (ly1 << (3 * rb));
        const uint32_t sup = s_base[j] + qy * s_tx[j] + (uint32_t)qx;
        pkey[p] = keep ? (sup | (rect << rp.key_bits)) : kCulledTile;
        pentry[p] = s_ent[j];
    }
}

// ---- pairs of few super-tiles, placed without emission and sort ----
//
// The lists of at most kDirectSupers super-tiles are the result of one counting
// sort over the depth-ordered entries, each expanded in place. The projection
// leaves every visible entry's tile rectangle and, from the reach test of its
// super-tiles, which pairs are kept (the record is in registers there; read
// again in depth order it costs a cache line per entry). A count kernel gathers
// that word in depth order and counts the pairs per super-tile and block (with
// sums over groups of blocks); a place kernel expands the pairs of kPairEntries
// entries at a time in LDS, ranks them stably by super-tile with ballots, as a
// radix scatter does, and writes them out in runs. The order inside a
// super-tile is the entries' depth order.
//
// Against emitting pairs to memory by an offset scan and radix-sorting them by
// super-tile (which more super-tiles still take), the pair arrays are written
// once instead of twice and read never, and 8 launches become 2. At 3M
// Gaussians (2.05M entries, 3.8M pairs) 130 -> 112 us, 15 of them new in the
// projection; at 300k 57 -> 26 us. The count kernel is bound by its gather, a
// cache line an entry (54 us, 4.8 TB/s of lines at 3M), the place kernel by the
// latency of its LDS passes.

// Calls f(q, x, y, super-tile) for the candidates of an entry.
template <class F>
__device__ __forceinline__ void for_candidates(const ViewDev& V, int S, const uint4& info, F f) {
    int sx0, sx1, sy0, sy1;
    super_rect((int)(info.x & 0xffffu), (int)(info.x >> 16), (int)(info.y & 0xffffu),
               (int)(info.y >> 16), S, &sx0, &sx1, &sy0, &sy1);
    uint32_t q = 0;
    for (int y = sy0; y < sy1; ++y)
        for (int x = sx0; x < sx1; ++x, ++q)
            if (pair_kept(info, q)) f(x, y, (uint32_t)(V.sup_offset + y * V.sup_x + x));
}

__device__ __forceinline__ const ViewDev& view_of_entry(const Views* views, uint32_t e,
                                                        uint32_t n) {
    return views->v[views->n > 1 ? e / n : 0u];
}

// Entries with many pairs (few large Gaussians, small super-tiles) would leave the
// pairs to a few blocks and there to a few threads. So a block takes kPairEntries
// a round or, where an entry has more than kWideMean candidates in the mean, as
// many as have a chunk of them, if the grid covers all entries so; and in a round
// where a thread has more than kWideAlone candidates, the threads of the block (of
// the wave in the count, which then needs no barrier: 0.7 us at 3M) take the pairs
// of all its entries, each by its place (ten steps to its entry, five to its bit).
// us of the whole binning, every thread walking its own entries' pairs / now /
// pairs emitted and sorted: 1000 Gaussians on 41 of 117 super-tiles each 943 / 84 /
// 204, 30k 1370 / 365 / 480, 30k on 49 of 425 3090 / 196 / 261; 300k, 50 of them of
// image size 163 / 141. By kWideMean 2 / 4 / 8: 1M Gaussians with 3.9 candidates
// 297 / 276 / 278, 30k with 6.6 122 / 119 / 140; by kWideAlone 4 / 16 / 64: 3M with
// 1.9 312 / 300 / 307, 100k with 6.6 207 / 201 / 226.
constexpr int kChunkEach = 8;                            // pairs of a chunk per thread
constexpr int kChunk = kPairThreads * kChunkEach;         // pairs expanded at a time
constexpr uint32_t kWideMean = 4;
__device__ __forceinline__ int64_t block_entries(const uint32_t* counters, int rounds) {
    const uint32_t nvis = counters[kVisible], pairs = counters[kPairs];
    const int64_t most = (int64_t)kPairEntries * rounds;
    if (pairs / kWideMean <= nvis) return most;
    const uint32_t least = (nvis + gridDim.x - 1u) / gridDim.x;
    return min(most, (int64_t)max(least, max((uint32_t)kChunk / (pairs / nvis), 1u)));
}

constexpr uint32_t kWideAlone = 16;

// The entry of N that owns place p: the last one whose first place is at most p.
template <int N>
__device__ __forceinline__ int pair_owner(const uint32_t* first, uint32_t p) {
    int i = 0;
#pragma unroll
    for (int half = 512; half > 0; half >>= 1)
        if (half < N && i + half < N && first[i + half] <= p) i += half;
    return i;
}
static_assert(kPairEntries <= 1024, "ten halvings");

// Super-tile column and row of the q-th kept pair of an entry.
__device__ __forceinline__ void kept_pair_at(int S, const uint4& info, uint32_t q, int* x, int* y) {
    const uint32_t tested = (uint32_t)__builtin_popcount(info.z);
    uint32_t c = kTested + q - tested;
    if (q < tested) {   // the q-th bit set
        c = 0;
#pragma unroll
        for (int half = 16; half > 0; half >>= 1) {
            const uint32_t below =
                (uint32_t)__builtin_popcount((info.z >> c) & ((1u << half) - 1u));
            const bool up = q >= below;
            q -= up ? below : 0u;
            c += up ? (uint32_t)half : 0u;
        }
    }
    int sx0, sx1, sy0, sy1;
    super_rect((int)(info.x & 0xffffu), (int)(info.x >> 16), (int)(info.y & 0xffffu),
               (int)(info.y >> 16), S, &sx0, &sx1, &sy0, &sy1);
    // (c + 1/2 is at least 1 / (2 w) > 2^-10 from a multiple of the width w, c < 512)
    const uint32_t w = (uint32_t)(sx1 - sx0);
    const uint32_t row = (uint32_t)(((float)c + 0.5f) * __builtin_amdgcn_rcpf((float)w));
    *x = sx0 + (int)(c - row * w);
    *y = sy0 + (int)row;
}

__global__ void __launch_bounds__(kPairThreads) pair_count_kernel(
    const Views* __restrict__ views, RasterDev rp, uint32_t n,
    const uint32_t* __restrict__ sorted_entry, const uint4* __restrict__ info,
    const uint32_t* __restrict__ counters, int rounds, uint4* __restrict__ sorted_info,
    uint32_t* __restrict__ hist, uint32_t* __restrict__ groups) {
    extern __shared__ uint32_t s_cnt[];   // per super-tile
    constexpr int NW = kPairThreads / 64, kEach = kPairEntries / kPairThreads;
    constexpr int kWaveEntries = kPairEntries / NW;
    __shared__ uint4 s_info[NW][kWaveEntries];
    __shared__ uint32_t s_first[NW][kWaveEntries];
    const int tid = threadIdx.x, w = tid / 64, lane = tid % 64;
    const int ns = views->total_supers, S = rp.super_tile;
    const int64_t nvis = counters[kVisible];
    const int64_t tile = block_entries(counters, rounds);
    const int active = (int)((nvis + tile - 1) / tile);
    if ((int)blockIdx.x >= active) return;   // uniform
    const int blk = xcd_block(blockIdx.x, active);
    for (int s = tid; s < ns; s += kPairThreads) s_cnt[s] = 0u;
    __syncthreads();
    const int64_t end = min(nvis, (blk + 1) * tile);
    for (int64_t k0 = blk * tile; k0 < end; k0 += kPairEntries) {
        // the round's entries dealt out to the waves, which work on their own
        const int m = (int)min((int64_t)kPairEntries, end - k0), per = (m + NW - 1) / NW;
        const int mine = min(per, m - w * per);   // (none: not positive)
        const int64_t k1 = k0 + (int64_t)w * per;
        uint32_t e[kEach];
        uint4 c[kEach];
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            const int i = j * 64 + lane;
            e[j] = i < mine ? sorted_entry[k1 + i] : 0u;
        }
        uint32_t candidates = 0;
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            c[j] = info[e[j]];
            c[j].w = e[j];
            if (j * 64 + lane >= mine) continue;
            sorted_info[k1 + j * 64 + lane] = c[j];
            candidates += candidate_pairs(c[j], S);
        }
        if (ballot(candidates > kWideAlone) != 0ull) {
            uint32_t kept[kEach], sum = 0;
#pragma unroll
            for (int j = 0; j < kEach; ++j) {
                kept[j] = j * 64 + lane < mine ? kept_pairs(c[j], S) : 0u;
                sum += kept[j];
            }
            const uint32_t incl = wave_incl_scan(sum);
            const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
            uint32_t first = incl - sum;
#pragma unroll
            for (int j = 0; j < kEach; ++j) {
                s_first[w][lane * kEach + j] = first;
                s_info[w][lane * kEach + j] = c[j];
                first += kept[j];
            }
            wave_lds_sync();
            for (uint32_t p = lane; p < total; p += 64) {
                const int o = pair_owner<kWaveEntries>(s_first[w], p);
                const uint4 f = s_info[w][o];
                const ViewDev& V = view_of_entry(views, f.w, n);
                int x, y;
                kept_pair_at(S, f, p - s_first[w][o], &x, &y);
                atomicAdd(&s_cnt[V.sup_offset + y * V.sup_x + x], 1u);
            }
            wave_lds_sync();
            continue;
        }
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            if (j * 64 + lane >= mine) break;
            for_candidates(view_of_entry(views, e[j], n), S, c[j],
                           [&](int, int, uint32_t s) { atomicAdd(&s_cnt[s], 1u); });
        }
    }
    __syncthreads();
    for (int s = tid; s < ns; s += kPairThreads) {
        const uint32_t c = s_cnt[s];
        hist[(int64_t)blk * ns + s] = c;
        if (c != 0u) atomicAdd(&groups[(int64_t)(blk / kPairGroup) * ns + s], c);
    }
}

// Position, key and entry of every kept pair; block 0 also writes the super-tile
// ranges and the pair counts. Pairs past the capacity are not written (the
// overflow is flagged when more pairs are needed than fit).
__global__ void __launch_bounds__(kPairThreads, 4) pair_place_kernel(
    const Views* __restrict__ views, RasterDev rp, uint32_t n, uint32_t* __restrict__ counters,
    int rounds, const uint4* __restrict__ sorted_info, const uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ groups, int64_t capacity, uint32_t* __restrict__ ranges,
    uint32_t* __restrict__ pkey, uint32_t* __restrict__ pentry) {
    constexpr int NW = kPairThreads / 64;
    constexpr int kEach = kPairEntries / kPairThreads;
    constexpr int kPerWave = kChunk / NW;
    extern __shared__ uint32_t s_dyn[];   // [NW][ns] counts, [ns] next positions, [ns] starts
    __shared__ uint32_t lkey[kChunk];
    __shared__ uint32_t lent[kChunk];
    __shared__ uint32_t s_first[kPairEntries];   // first place of an entry's pairs
    __shared__ uint32_t smem[NW + 1];
    const int tid = threadIdx.x, w = tid / 64, lane = tid % 64;
    const int ns = views->total_supers, S = rp.super_tile;
    uint32_t* wcnt = s_dyn;
    uint32_t* gpos = s_dyn + NW * ns;
    uint32_t* start = gpos + ns;
    const int64_t nvis = counters[kVisible];
    const int64_t tile = block_entries(counters, rounds);
    const int active = (int)((nvis + tile - 1) / tile);
    if ((int)blockIdx.x >= max(active, 1)) return;   // uniform; block 0 always writes the ranges
    const int blk = active > 0 ? xcd_block(blockIdx.x, active) : 0;
    // positions of this block's first pairs: 2^k threads add up a row of
    // super-tile counts each, the rows' sums in LDS (lkey, lent)
    {
        int sp = 64;
        while (sp < ns && sp < kPairThreads) sp *= 2;
        const int part = tid / sp, parts = kPairThreads / sp;
        const int ng = (active + (int)kPairGroup - 1) / (int)kPairGroup, g = blk / (int)kPairGroup;
        const uint32_t cap = (uint32_t)capacity;
        uint32_t carry = 0;
        for (int s0 = 0; s0 < ns; s0 += sp) {
            const int s = s0 + (tid & (sp - 1));
            uint32_t tot = 0, before = 0;
            if (s < ns) {
                for_rows(groups + s, ns, part, ng, parts, [&](int j, uint32_t c) {
                    tot += c;
                    before += j < g ? c : 0u;
                });
                for_rows(hist + s, ns, g * (int)kPairGroup + part, blk, parts,
                         [&](int, uint32_t c) { before += c; });
            }
            lkey[tid] = tot;
            lent[tid] = before;
            __syncthreads();
            tot = before = 0;
            if (tid < sp)
                for (int k = 0; k < parts; ++k) {
                    tot += lkey[k * sp + tid];
                    before += lent[k * sp + tid];
                }
            // (saturating over the super-tiles, like the scans above, and never
            // past the capacity, below 2^31: a place that adding a chunk's pairs
            // to cannot wrap, and the ranges' lengths sum to the capacity at most)
            uint32_t all;
            const uint32_t ex = sat_add(carry, block_excl_sat_scan<kPairThreads>(tot, smem, &all));
            carry = sat_add(carry, all);
            if (tid < sp && s < ns) {
                gpos[s] = min(sat_add(ex, before), cap);
                if (blockIdx.x == 0) {
                    const uint32_t a = min(ex, cap), b = min(sat_add(ex, tot), cap);
                    ranges[2 * s] = a < b ? a : 0u;
                    ranges[2 * s + 1] = a < b ? b : 0u;
                }
            }
        }
        if (blockIdx.x == 0 && tid == 0) {
            const uint32_t needed = counters[kPairs];
            counters[kPairsWritten] = min(needed, cap);
            counters[kPairsKept] = min(carry, cap);
            if ((int64_t)needed > capacity) counters[kStatus] |= SGS_STATUS_PAIR_OVERFLOW;
        }
    }
    if (active == 0) return;
    const int rb = rp.rect_bits, kb = rp.key_bits;
    const uint32_t kmask = (1u << kb) - 1u;
    const int64_t end = min(nvis, (blk + 1) * tile);
    for (int64_t k0 = blk * tile; k0 < end; k0 += kPairEntries) {
        // thread t's entries: k0 + kEach t ...; in one scan the place of their
        // pairs and, above kPlaceBits, the threads that have many candidates
        constexpr int kPlaceBits = 20;
        static_assert(kPairEntries * kDirectSupers < 1 << kPlaceBits, "places of a round");
        uint4 c[kEach];
        uint32_t kept[kEach], mine = 0, candidates = 0;
#pragma unroll
        for (int j = 0; j < kEach; ++j) {
            const int64_t k = k0 + (int64_t)tid * kEach + j;
            c[j] = k < end ? sorted_info[k] : make_uint4(0u, 0u, 0u, 0u);
            kept[j] = k < end ? kept_pairs(c[j], S) : 0u;
            candidates += k < end ? candidate_pairs(c[j], S) : 0u;
            mine += kept[j];
        }
        uint32_t total;
        uint32_t first = block_excl_scan<kPairThreads>(
            mine | (candidates > kWideAlone ? 1u << kPlaceBits : 0u), smem, &total);
        first &= (1u << kPlaceBits) - 1u;
        const bool wide = total >> kPlaceBits != 0u;   // uniform
        total &= (1u << kPlaceBits) - 1u;
        if (wide) {
            uint32_t at = first;
#pragma unroll
            for (int j = 0; j < kEach; ++j) {
                s_first[tid * kEach + j] = at;
                at += kept[j];
            }
            __syncthreads();
        }
        for (uint32_t c0 = 0; c0 < total; c0 += (uint32_t)kChunk) {
            auto put = [&](uint32_t at, const uint4& f, int x, int y, uint32_t s) {
                // the tile rectangle inside the super-tile, relative to its first tile
                const int ox = x * S, oy = y * S;
                const uint32_t lx0 = (uint32_t)(max((int)(f.x & 0xffffu), ox) - ox);
                const uint32_t lx1 = (uint32_t)(min((int)(f.x >> 16), ox + S) - 1 - ox);
                const uint32_t ly0 = (uint32_t)(max((int)(f.y & 0xffffu), oy) - oy);
                const uint32_t ly1 = (uint32_t)(min((int)(f.y >> 16), oy + S) - 1 - oy);
                const uint32_t rect = lx0 | (lx1 << rb) | (ly0 << (2 * rb)) | (ly1 << (3 * rb));
                lkey[at] = s | (rect << kb);
                lent[at] = f.w;
            };
            if (wide) {
#pragma unroll 2
                for (uint32_t at = tid; at < (uint32_t)kChunk && c0 + at < total;
                     at += kPairThreads) {
                    const int o = pair_owner<kPairEntries>(s_first, c0 + at);
                    const uint4 f = sorted_info[k0 + o];
                    const ViewDev& V = view_of_entry(views, f.w, n);
                    int x, y;
                    kept_pair_at(S, f, c0 + at - s_first[o], &x, &y);
                    put(at, f, x, y, (uint32_t)(V.sup_offset + y * V.sup_x + x));
                }
            } else {
                uint32_t at = first - c0;   // wraps below the chunk, which no check passes
#pragma unroll
                for (int j = 0; j < kEach; ++j) {
                    if (k0 + (int64_t)tid * kEach + j >= end) break;
                    for_candidates(view_of_entry(views, c[j].w, n), S, c[j],
                                   [&](int x, int y, uint32_t s) {
                        if (at < (uint32_t)kChunk) put(at, c[j], x, y, s);
                        ++at;
                    });
                }
            }
            for (int i = tid; i < NW * ns; i += kPairThreads) wcnt[i] = 0u;
            __syncthreads();
            // stable ranking, wave by wave: lanes of one super-tile found with
            // ballots, the wave's counters carry on across its rounds
            const int have = (int)min(total - c0, (uint32_t)kChunk);
            uint32_t key[kChunkEach], ent[kChunkEach], rank[kChunkEach];
            uint32_t* cnt = wcnt + w * ns;
#pragma unroll
            for (int it = 0; it < kChunkEach; ++it) {
                const int li = w * kPerWave + it * 64 + lane;
                const bool valid = li < have;
                key[it] = valid ? lkey[li] : 0u;
                ent[it] = valid ? lent[li] : 0u;
                rank[it] = 0u;
                if (w * kPerWave + it * 64 >= have) continue;   // uniform over the wave
                const uint32_t s = key[it] & kmask;
                uint64_t peers = ballot(valid);
                for (int b = 0; b < kb; ++b) {
                    const bool bit = (s >> b) & 1u;
                    const uint64_t m = ballot(bit);
                    peers &= bit ? m : ~m;
                }
                const uint32_t before = (uint32_t)popc64(peers & lanemask_lt());
                if (valid) rank[it] = cnt[s] + before;
                // every lane has read the counters before the leaders advance them
                __builtin_amdgcn_wave_barrier();
                if (valid && before == 0) cnt[s] += (uint32_t)popc64(peers);
                __builtin_amdgcn_wave_barrier();
            }
            __syncthreads();
            uint32_t carry = 0;
            for (int s0 = 0; s0 < ns; s0 += kPairThreads) {
                const int s = s0 + tid;
                uint32_t sum = 0;
                if (s < ns) {
#pragma unroll
                    for (int k = 0; k < NW; ++k) sum += wcnt[k * ns + s];
                }
                uint32_t tot;
                uint32_t run = carry + block_excl_scan<kPairThreads>(sum, smem, &tot);
                carry += tot;
                if (s < ns) {
                    // start[s] turns a local position into the global one
                    start[s] = gpos[s] - run;
                    gpos[s] = min(gpos[s] + sum, (uint32_t)capacity);
#pragma unroll
                    for (int k = 0; k < NW; ++k) {
                        const uint32_t x = wcnt[k * ns + s];
                        wcnt[k * ns + s] = run;
                        run += x;
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int it = 0; it < kChunkEach; ++it) {
                const int li = w * kPerWave + it * 64 + lane;
                if (li >= have) break;
                const uint32_t pos = cnt[key[it] & kmask] + rank[it];
                lkey[pos] = key[it];
                lent[pos] = ent[it];
            }
            __syncthreads();
            for (int li = tid; li < have; li += kPairThreads) {
                const uint32_t k = lkey[li];
                const uint32_t out = start[k & kmask] + (uint32_t)li;
                if (out < (uint32_t)capacity) {
                    pkey[out] = k;
                    pentry[out] = lent[li];
                }
            }
            __syncthreads();
        }
    }
}

// [start, end) of every super-tile by binary search in the sorted keys
// (the super-tile index is the low key_bits bits; empty super-tiles: [0, 0)).
__global__ void __launch_bounds__(256) ranges_kernel(const uint32_t* __restrict__ pkey,
                                                     const uint32_t* __restrict__ counters,
                                                     int64_t total_supers, int key_bits,
                                                     uint32_t* __restrict__ ranges) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total_supers) return;
    const uint32_t mask = (uint32_t)((1ull << key_bits) - 1ull);
    const uint32_t P = counters[kPairsKept];
    uint32_t lo = 0, hi = P;
    while (lo < hi) {  // first key >= t
        const uint32_t mid = (lo + hi) >> 1;
        if ((pkey[mid] & mask) < (uint32_t)t) lo = mid + 1; else hi = mid;
    }
    const uint32_t a = lo;
    hi = P;
    while (lo < hi) {  // first key > t
        const uint32_t mid = (lo + hi) >> 1;
        if ((pkey[mid] & mask) <= (uint32_t)t) lo = mid + 1; else hi = mid;
    }
    const bool empty = lo == a;
    ranges[2 * t] = empty ? 0u : a;
    ranges[2 * t + 1] = empty ? 0u : lo;
}

__global__ void __launch_bounds__(64) store_views_kernel(Views v, Views* __restrict__ dst,
                                                         uint32_t* __restrict__ counters,
                                                         int32_t* step,
                                                         const int32_t* __restrict__ gate) {
    store_views(v, nullptr, 0, nullptr, dst);
    // what compositing adds up
    if (counters != nullptr && threadIdx.x < 4) counters[kBlended + threadIdx.x] = 0u;
    if (counters != nullptr && threadIdx.x == 4) counters[kUsed] = 0u;
    if (step != nullptr && threadIdx.x == 0 && !gate_closed(gate)) *step += 1;
}

// The first launch of a call that bins: block 0 stores the views and clears the
// counters binning and the compositing forward accumulate into (the status word
// stays), all blocks clear the sums binning accumulates.
constexpr int kBeginThreads = 256;
__global__ void __launch_bounds__(kBeginThreads) begin_bin_kernel(
    Views v, const ViewDev* __restrict__ table, int n_table, const int32_t* __restrict__ d_view,
    Views* __restrict__ dst, uint32_t* __restrict__ counters, uint4* __restrict__ clear,
    int64_t n4) {
    if (blockIdx.x == 0) {
        store_views(v, table, n_table, d_view, dst);
        if (threadIdx.x >= kVisible && threadIdx.x <= kRedo) counters[threadIdx.x] = 0u;
    }
    for (int64_t i = (int64_t)blockIdx.x * kBeginThreads + threadIdx.x; i < n4;
         i += (int64_t)gridDim.x * kBeginThreads)
        clear[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ void fill_u32_kernel(uint32_t* p, int64_t n, uint32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ---- the split of the super-tile lists into tile lists ----
//
// Two launches: the count kernel forms the tile masks and the counts per
// (segment, tile), their sums over groups of segments and the number of list
// entries per super-tile; the write kernel adds up what comes before a segment
// (the super-tiles in LDS, the groups and segments of its super-tile row by row,
// a tile a lane), stores the entries and the tiles' ranges. A scan over all
// (super-tile, tile, segment) counts and the ranges took three launches more.

// Pairs of super-tile s's list that a split covers: before compositing
// (kRest = false) its prefix, in the completing split the whole list of the
// super-tiles flagged in sup_redo.
template <bool kRest>
__device__ __forceinline__ uint32_t pairs_to_split(const uint32_t* ranges, const uint32_t* sup_redo,
                                                   uint32_t prefix_segs, int64_t s) {
    const uint32_t len = ranges[2 * s + 1] - ranges[2 * s];
    if (kRest) return sup_redo[s] ? len : 0u;
    return split_pairs(len, prefix_segs);
}
__device__ __forceinline__ uint32_t segments_of(uint32_t pairs, int seg_log2) {
    return (uint32_t)(((uint64_t)pairs + (1ull << seg_log2) - 1ull) >> seg_log2);
}
// Segments of every super-tile's list (the scan numbers them).
template <bool kRest>
struct SegCountSrc {
    const uint32_t* ranges;
    const uint32_t* sup_redo;
    const uint32_t* redo;
    int64_t n;
    uint32_t prefix;
    int seg_log2;
    __device__ int64_t count() const { return !kRest || *redo ? n : 0; }
    __device__ uint32_t operator()(int64_t s) const {
        return segments_of(pairs_to_split<kRest>(ranges, sup_redo, prefix, s), seg_log2);
    }
};
// List entries of every super-tile.
struct ItemCountSrc {
    const uint64_t* items;
    int64_t n;
    __device__ int64_t count() const { return n; }
    __device__ uint32_t operator()(int64_t s) const {
        return (uint32_t)min(items[s], (uint64_t)0xffffffffull);
    }
};

// Exclusive saturating scan of the counts of all super-tiles in one workgroup (a
// few hundred to a few ten thousand counts): first[s] for every super-tile and
// the total in first[n].
constexpr int kSegScanThreads = 1024;
constexpr int kSegScanItems = 4;
template <class Src>
__global__ void __launch_bounds__(kSegScanThreads) seg_scan_kernel(Src src, uint32_t* first) {
    __shared__ uint32_t smem[kSegScanThreads / 64 + 1];
    const int64_t n = src.count();
    constexpr int64_t kChunk = (int64_t)kSegScanThreads * kSegScanItems;
    uint32_t carry = 0;
    for (int64_t c0 = 0; c0 < n; c0 += kChunk) {
        const int64_t base = c0 + (int64_t)threadIdx.x * kSegScanItems;
        uint32_t v[kSegScanItems], sum = 0;
#pragma unroll
        for (int j = 0; j < kSegScanItems; ++j) {
            v[j] = base + j < n ? src(base + j) : 0u;
            sum = sat_add(sum, v[j]);
        }
        uint32_t tot;
        uint32_t pos = sat_add(carry, block_excl_sat_scan<kSegScanThreads>(sum, smem, &tot));
#pragma unroll
        for (int j = 0; j < kSegScanItems; ++j) {
            if (base + j < n) first[base + j] = pos;
            pos = sat_add(pos, v[j]);
        }
        carry = sat_add(carry, tot);
    }
    if (threadIdx.x == 0) first[src.n] = carry;
}

// The same within every workgroup of a kernel, into LDS (first[0..ns]).
template <int NT, class Src>
__device__ __forceinline__ void scan_supers(const Src& src, int ns, uint32_t* first,
                                            uint32_t* smem) {
    uint32_t carry = 0;
    for (int s0 = 0; s0 < ns; s0 += NT) {
        const int s = s0 + (int)threadIdx.x;
        const uint32_t v = s < ns ? src(s) : 0u;
        uint32_t tot;
        const uint32_t ex = sat_add(carry, block_excl_sat_scan<NT>(v, smem, &tot));
        if (s < ns) first[s] = ex;
        carry = sat_add(carry, tot);
    }
    if (threadIdx.x == 0) first[ns] = carry;
}

// Segment g of the split: super-tile s (global index), segment k of nseg in
// its list, pairs [a, b), the super-tile's first tile (tx0, ty0) in its view.
struct Segment {
    int s;
    uint32_t k, nseg, a, b;
    int tx0, ty0;
    const ViewDev* V;
};

template <bool kRest>
__device__ __forceinline__ bool locate_segment(const Views* views, const uint32_t* seg_first,
                                               const uint32_t* sup_ranges, const RasterDev& rp,
                                               uint32_t g, Segment* out) {
    const int ns = views->total_supers, S = rp.super_tile;
    if (g >= seg_first[ns]) return false;
    int lo = 0, hi = ns;   // first super-tile whose first segment lies past g
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (seg_first[mid] <= g) lo = mid + 1; else hi = mid;
    }
    const int s = lo - 1;
    int vi = 0;
    while (vi + 1 < views->n && s >= views->v[vi + 1].sup_offset) ++vi;
    const ViewDev* V = &views->v[vi];
    const int ls = s - V->sup_offset;
    out->s = s;
    out->k = g - seg_first[s];
    out->nseg = seg_first[s + 1] - seg_first[s];
    const uint32_t begin = sup_ranges[2 * s], len = sup_ranges[2 * s + 1] - begin;
    const uint32_t end = begin + (kRest ? len : split_pairs(len, (uint32_t)rp.prefix_segs));
    out->a = begin + (out->k << rp.seg_log2);
    out->b = min(end, out->a + (1u << rp.seg_log2));
    out->tx0 = (ls % V->sup_x) * S;
    out->ty0 = (ls / V->sup_x) * S;
    out->V = V;
    return true;
}

__device__ __forceinline__ uint64_t wave_or64(uint64_t m) {
    uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        lo |= (uint32_t)__shfl_xor((int)lo, d, 64);
        hi |= (uint32_t)__shfl_xor((int)hi, d, 64);
    }
    return (uint64_t)__builtin_amdgcn_readfirstlane(lo) |
           ((uint64_t)__builtin_amdgcn_readfirstlane(hi) << 32);
}

// Transpose of the 64 x 64 bit matrix whose row l is lane l's word: returns,
// in lane t, the word whose bit l is bit t of lane l's input. Six stages
// swap the off-diagonal blocks of size 32, 16, ..., 1: a lane in the upper
// half of a block pair keeps its bits of the left half and takes its
// partner's left-half bits into the right half, and the other way round.
__device__ __forceinline__ uint64_t wave_transpose64(uint64_t x) {
    const int l = __lane_id();
    uint32_t lo = (uint32_t)x, hi = (uint32_t)(x >> 32);
    {
        const uint32_t plo = (uint32_t)__shfl_xor((int)lo, 32, 64);
        const uint32_t phi = (uint32_t)__shfl_xor((int)hi, 32, 64);
        const bool up = (l & 32) != 0;
        lo = up ? phi : lo;
        hi = up ? hi : plo;
    }
    constexpr uint32_t kKeep[5] = {0x0000ffffu, 0x00ff00ffu, 0x0f0f0f0fu, 0x33333333u,
                                   0x55555555u};
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int j = 16 >> i;
        const uint32_t M = kKeep[i];
        const bool up = (l & j) != 0;
        const uint32_t plo = (uint32_t)__shfl_xor((int)lo, j, 64);
        const uint32_t phi = (uint32_t)__shfl_xor((int)hi, j, 64);
        const uint32_t slo = up ? (plo >> j) : (plo << j), shi = up ? (phi >> j) : (phi << j);
        lo = up ? ((lo & ~M) | (slo & M)) : ((lo & M) | (slo & ~M));
        hi = up ? ((hi & ~M) | (shi & M)) : ((hi & M) | (shi & ~M));
    }
    return (uint64_t)lo | ((uint64_t)hi << 32);
}

constexpr int kSplitWaves = 4;
constexpr int64_t kSplitBlocks = 2048;   // blocks of the split kernels' grid-stride loops

// Reach of one entry by rows: q = a dx^2 + 2 b dx dy + c dy^2 <= lim is, for
// dy fixed, the interval |dx - s dy| <= sqrt((lim - k dy^2) / a) (s = -b/a,
// k = det/a, det = ac - b^2), so over a band of rows its right end is largest
// at the band point nearest the dy of the ellipse's rightmost point,
// dy_r = -b sqrt(lim / (c det)) (the right end is concave in dy), and its left
// end smallest at -dy_r. Formed once per entry, in float, with margins that
// keep the test conservative: det by Kahan's fused form (error a few ulp of
// det); lim raised by a bound on the rounding of the compositing kernels' own
// float evaluation of q (16 ulp of its terms' magnitudes, at most
// 2 (a + c)^2 lim / det on the ellipse); every interval end widened by 1e-3 px
// plus the worst effect of the rounding of lim - k dy^2 near the ellipse's
// top or bottom, sqrt(4 eps lim / a), plus relative rounding.
struct Reach {
    float s, k, inv_a, lim, ym, dyr, slack;
    bool conic;   // false: no reach limit or a degenerate conic (box only)
};

// (The hardware reciprocal and square root, 1 ulp each, are covered by the
// relative margins.)
__device__ __forceinline__ Reach make_reach(float a, float b, float c, float lim) {
    Reach r;
    const float bb = b * b;
    const float det = fmaf(a, c, -bb) - fmaf(b, b, -bb);
    r.conic = lim != INFINITY && a > 0.f && c > 0.f && det > 0.f;
    const float inv_det = __builtin_amdgcn_rcpf(det);
    const float ac = a + c;
    r.lim = lim * (1.f + 2e-6f * (ac * ac * inv_det));
    r.conic = r.conic && r.lim < INFINITY;
    r.inv_a = __builtin_amdgcn_rcpf(a);
    r.s = -b * r.inv_a;
    r.k = det * r.inv_a;
    r.ym = __builtin_amdgcn_sqrtf(r.lim * a * inv_det) * (1.f + 1e-5f) + 1e-3f;
    r.dyr = -b * __builtin_amdgcn_sqrtf(r.lim * __builtin_amdgcn_rcpf(c) * inv_det);
    r.slack = 1e-3f + 2.f * __builtin_amdgcn_sqrtf(4.8e-7f * r.lim * r.inv_a);
    return r;
}

// Tile columns [*c0, *c1] (view tile indices; *c0 > *c1: none) of the tiles in
// the row band of pixel rows [py0, py0 + h) that hold a pixel centre inside
// the overlap box (widened by 1e-3 px) within the entry's reach; tile width
// 2^tw_log2.
__device__ __forceinline__ void band_columns(const Reach& R, float u, float v, float rx, float ry,
                                             int py0, int h, int tw_log2, int width, int* c0,
                                             int* c1) {
    const float m = 1e-3f;
    float lo = fmaxf((float)py0 + 0.5f - v, -ry - m);
    float hi = fminf((float)(py0 + h) - 0.5f - v, ry + m);
    float xl = -rx - m, xr = rx + m;
    if (R.conic) {
        lo = fmaxf(lo, -R.ym);
        hi = fminf(hi, R.ym);
        const float y1 = fminf(fmaxf(R.dyr, lo), hi), y2 = fminf(fmaxf(-R.dyr, lo), hi);
        const float h1 = __builtin_amdgcn_sqrtf(fmaxf(fmaf(-R.k * y1, y1, R.lim), 0.f) * R.inv_a);
        const float h2 = __builtin_amdgcn_sqrtf(fmaxf(fmaf(-R.k * y2, y2, R.lim), 0.f) * R.inv_a);
        const float t1 = R.s * y1, t2 = R.s * y2;
        const float rel = 1e-5f * (fabsf(t1) + fabsf(t2) + h1 + h2);
        xl = fmaxf(xl, t2 - h2 - R.slack - rel);
        xr = fminf(xr, t1 + h1 + R.slack + rel);
    }
    *c0 = 1;
    *c1 = 0;
    if (!(lo <= hi) || !(xl <= xr)) return;
    // pixel columns whose centre lies in [u + xl, u + xr] (the sums' rounding,
    // below an ulp of |u| + |x|, widened away)
    const float ru = 2.4e-7f * (fabsf(u) + fabsf(xl) + fabsf(xr));
    const float fl = fmaxf(ceilf(u + xl - 0.5f - ru), 0.f);
    const float fr = fminf(floorf(u + xr - 0.5f + ru), (float)(width - 1));
    if (!(fl <= fr)) return;
    *c0 = (int)fl >> tw_log2;
    *c1 = (int)fr >> tw_log2;
}

// Tile masks and per-tile counts of one segment per wave. A pair's mask has
// bit (y S + x) for tile (x, y) of its super-tile when the tile lies in the
// pair's tile rectangle and, with alpha_min > 0, the entry can reach alpha_min
// on the tile's pixels in the image (row by row of the rectangle: the tile
// columns of each row band the entry reaches).
//
// With `local` (at most kLocalSupers super-tiles) every workgroup first forms
// the segment index (the exclusive scan of src over the super-tiles) in LDS,
// and workgroup 0 also stores it for the write kernel, which saves the scan's
// own launch; otherwise seg_first holds it already.
constexpr int kLocalSupers = 1024;
template <bool kRest>
__global__ void __launch_bounds__(kSplitWaves * 64) split_count_kernel(
    const Views* __restrict__ views, RasterDev rp, SegCountSrc<kRest> src, bool local,
    uint32_t* __restrict__ seg_first_g, const uint32_t* __restrict__ sup_ranges,
    const uint32_t* __restrict__ skey, const uint32_t* __restrict__ sentry,
    const float4* __restrict__ rec, uint32_t entries, uint64_t* __restrict__ mask,
    uint32_t* __restrict__ seg_cnt, uint32_t* __restrict__ seg_groups,
    unsigned long long* __restrict__ sup_items) {
    constexpr int NT = kSplitWaves * 64;
    __shared__ uint32_t s_first[kLocalSupers + 1];
    __shared__ uint32_t s_scan[NT / 64 + 1];
    if (kRest && src.count() == 0) return;   // uniform: no tile needs more
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int S = rp.super_tile, TT = S * S;
    const uint32_t* seg_first = seg_first_g;
    if (local) {   // uniform
        const int ns = views->total_supers;
        scan_supers<NT>(src, ns, s_first, s_scan);
        __syncthreads();
        if (blockIdx.x == 0)
            for (int s = threadIdx.x; s <= ns; s += NT) seg_first_g[s] = s_first[s];
        seg_first = s_first;
    }
    // segments in a grid-stride loop (the grid is sized for the machine, not
    // for the capacity's bound on the segment count)
    for (uint32_t g = blockIdx.x * kSplitWaves + w;; g += gridDim.x * kSplitWaves) {
        Segment sg;
        if (!locate_segment<kRest>(views, seg_first, sup_ranges, rp, g, &sg)) return;   // uniform
        const ViewDev& V = *sg.V;
        const int rb = rp.rect_bits;
        const uint32_t rmask = (1u << rb) - 1u;
        const bool reach = rp.alpha_min > 0.f;
        const int tw_log2 = __builtin_ctz((unsigned)rp.tile_w);
        const float inv_th = 1.f / (float)rp.tile_h;
        uint32_t cnt = 0;   // lane t: pairs of the segment on tile t
        for (uint32_t p0 = sg.a; p0 < sg.b; p0 += 64) {
            const uint32_t p = p0 + (uint32_t)lane;
            const bool valid = p < sg.b;
            const uint32_t r = valid ? skey[p] >> rp.key_bits : 0u;
            const int x0 = (int)(r & rmask), x1 = (int)((r >> rb) & rmask);
            const int y0 = (int)((r >> (2 * rb)) & rmask), y1 = (int)((r >> (3 * rb)) & rmask);
            uint64_t M = 0;
            if (valid && !reach) {
                const uint64_t row = ((1ull << (x1 - x0 + 1)) - 1ull) << x0;
                for (int y = y0; y <= y1; ++y) M |= row << (y * S);
            } else if (valid) {
                const int64_t e = min(sentry[p], entries - 1u);
                const float4 g0 = rec[3 * e], g1 = rec[3 * e + 1];
                const Reach R = make_reach(g0.z, g0.w, g1.x, reach_limit(g1.y, rp));
                // only the rows the ellipse's height reaches
                int ya = y0, yb = y1;
                if (R.conic) {
                    const float top = fmaxf(floorf((g0.y - R.ym) * inv_th), -1e6f);
                    const float bot = fminf(floorf((g0.y + R.ym) * inv_th), 1e6f);
                    ya = max(ya, (int)top - sg.ty0 - 1);
                    yb = min(yb, (int)bot - sg.ty0 + 1);
                }
                for (int y = ya; y <= yb; ++y) {
                    const int py0 = (sg.ty0 + y) * rp.tile_h;
                    int c0, c1;
                    band_columns(R, g0.x, g0.y, g1.z, g1.w, py0, min(rp.tile_h, V.height - py0),
                                 tw_log2, V.width, &c0, &c1);
                    c0 = max(c0 - sg.tx0, x0);
                    c1 = min(c1 - sg.tx0, x1);
                    if (c0 <= c1) M |= (((1ull << (c1 - c0 + 1)) - 1ull) << c0) << (y * S);
                }
            }
            if (valid) mask[p] = M;
            // lane t counts the pairs of this step whose mask has tile t
            cnt += (uint32_t)popc64(wave_transpose64(M));
        }
        if (lane < TT) {
            seg_cnt[(size_t)g * TT + lane] = cnt;
            const size_t grp = (size_t)(seg_first[sg.s] / (uint32_t)kSegGroup) + (size_t)sg.s +
                               sg.k / (uint32_t)kSegGroup;
            if (cnt != 0u) atomicAdd(&seg_groups[grp * TT + lane], cnt);
        }
        const uint32_t items = wave_incl_scan(cnt);   // lanes past TT count nothing
        if (lane == 63 && items != 0u) atomicAdd(&sup_items[sg.s], (unsigned long long)items);
    }
}

// Stable scatter of one segment per wave into the tile lists, 64 pairs per
// step. The transposed masks give lane t the set of the step's pairs on tile
// t; the step's entries and their list positions are grouped by tile in LDS
// (tile t's after those of the tiles before it, in pair order), and the wave
// then stores the group with consecutive lanes on consecutive items, so that
// stores of neighbouring lanes mostly share cache lines. A step of more than
// kStepItems items (a few pairs covering most of their super-tile) is stored
// directly by the tile lanes.
//
// Before that, the segment's list positions: super-tile after super-tile (their
// entry counts scanned in LDS, or in sup_base beyond kLocalSupers), tile after
// tile, segment after segment. The first segment of a super-tile stores its
// tiles' ranges: before compositing (kRest = false) every tile's, with its state
// (whether its super-tile's list was cut by the prefix), in the completing split
// those of the tiles marked incomplete, which now take their whole lists. Lists
// that do not fit the capacity are left empty and flagged.
constexpr int kWriteWaves = 4;
constexpr int kStepItems = 1024;
template <bool kRest>
__global__ void __launch_bounds__(kWriteWaves * 64) split_write_kernel(
    const Views* __restrict__ views, RasterDev rp, SegCountSrc<kRest> src, bool local,
    const uint32_t* __restrict__ seg_first_g, const uint32_t* __restrict__ sup_base,
    ItemCountSrc items, const uint32_t* __restrict__ sup_ranges,
    const uint32_t* __restrict__ sentry, const uint64_t* __restrict__ mask,
    const uint32_t* __restrict__ seg_cnt, const uint32_t* __restrict__ seg_groups,
    uint32_t* __restrict__ counters, int64_t capacity, uint32_t* __restrict__ tile_entry,
    uint32_t* __restrict__ tile_ranges, uint32_t* __restrict__ tile_state,
    uint32_t* __restrict__ sup_redo) {
    constexpr int NT = kWriteWaves * 64;
    __shared__ uint32_t s_ent[kWriteWaves][64];
    __shared__ uint32_t s_item[kWriteWaves][kStepItems];
    __shared__ uint32_t s_pos[kWriteWaves][kStepItems];
    __shared__ uint32_t s_base[kLocalSupers + 1];
    __shared__ uint32_t s_scan[NT / 64 + 1];
    if (kRest && src.count() == 0) return;   // uniform: no tile needs more
    const int w = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int S = rp.super_tile, TT = S * S;
    const int ns = views->total_supers;
    const uint32_t* seg_first = seg_first_g;
    const uint32_t* base = sup_base;
    if (local) {   // uniform
        scan_supers<NT>(items, ns, s_base, s_scan);
        __syncthreads();
        base = s_base;
    }
    // the completing split's lists lie after the prefix lists
    const uint32_t origin = kRest ? counters[kItems] : 0u;
    const uint32_t total = base[ns];
    const bool overflow = (int64_t)sat_add(origin, total) > capacity;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        counters[kRest ? kItemsRest : kItems] = total;
        if (overflow) atomicOr(&counters[kStatus], (uint32_t)SGS_STATUS_PAIR_OVERFLOW);
    }
    if (!kRest) {
        // lists without a segment, and the flags the compositing sets
        uint32_t units = 0;
        for (int s = blockIdx.x * NT + threadIdx.x; s < ns; s += gridDim.x * NT) {
            sup_redo[s] = 0u;
            units += list_units(pairs_to_split<kRest>(sup_ranges, sup_redo,
                                                      (uint32_t)rp.prefix_segs, s));
            if (seg_first[s + 1] != seg_first[s]) continue;
            int vi = 0;
            while (vi + 1 < views->n && s >= views->v[vi + 1].sup_offset) ++vi;
            const ViewDev& V = views->v[vi];
            const int ls = s - V.sup_offset;
            const int tx0 = (ls % V.sup_x) * S, ty0 = (ls / V.sup_x) * S;
            for (int y = ty0; y < min(ty0 + S, V.tiles_y); ++y)
                for (int x = tx0; x < min(tx0 + S, V.tiles_x); ++x) {
                    const int t = V.tile_offset + y * V.tiles_x + x;
                    tile_ranges[2 * t] = tile_ranges[2 * t + 1] = 0u;
                    tile_state[t] = kTileWhole;
                }
        }
        units = wave_incl_scan(units);
        if (lane == 63 && units != 0u) atomicAdd(&counters[kSegments], units);
    }
    for (uint32_t g = blockIdx.x * kWriteWaves + w;; g += gridDim.x * kWriteWaves) {
        Segment sg;
        if (!locate_segment<kRest>(views, seg_first, sup_ranges, rp, g, &sg)) return;   // uniform
        // lane t: next list position of tile t
        uint32_t tot = 0, before = 0;
        if (lane < TT) {
            const int kg = (int)(sg.k / (uint32_t)kSegGroup), kr = (int)(sg.k % (uint32_t)kSegGroup);
            const size_t grp = (size_t)(seg_first[sg.s] / (uint32_t)kSegGroup) + (size_t)sg.s;
            for_rows(seg_groups + grp * TT + lane, TT, 0,
                     (int)((sg.nseg + (uint32_t)kSegGroup - 1u) / (uint32_t)kSegGroup), 1,
                     [&](int j, uint32_t c) {
                         tot += c;
                         before += j < kg ? c : 0u;
                     });
            for_rows(seg_cnt + (size_t)(g - (uint32_t)kr) * TT + lane, TT, 0, kr, 1,
                     [&](int, uint32_t c) { before += c; });
        }
        const uint32_t first = origin + base[sg.s] + wave_incl_scan(tot) - tot;
        uint32_t run = first + before;
        if (sg.k == 0u && lane < TT) {
            const ViewDev& V = *sg.V;
            const int x = sg.tx0 + lane % S, y = sg.ty0 + lane / S;
            if (x < V.tiles_x && y < V.tiles_y) {
                const int t = V.tile_offset + y * V.tiles_x + x;
                if (!kRest || tile_state[t] == kTileIncomplete) {
                    tile_ranges[2 * t] = overflow ? 0u : first;
                    tile_ranges[2 * t + 1] = overflow ? 0u : first + tot;
                }
                if (!kRest) {
                    const uint32_t len = sup_ranges[2 * sg.s + 1] - sup_ranges[2 * sg.s];
                    tile_state[t] = list_cut(len, (uint32_t)rp.prefix_segs) ? kTileTruncated
                                                                            : kTileWhole;
                }
            }
        }
        // (a second compositing of the same lists completes nothing again)
        if (kRest && sg.k == 0u && lane == 0) sup_redo[sg.s] = 0u;
        if (overflow) continue;   // the tile lists stay empty
        for (uint32_t p0 = sg.a; p0 < sg.b; p0 += 64) {
            const uint32_t p = p0 + (uint32_t)lane;
            const bool valid = p < sg.b;
            const uint64_t M = valid ? mask[p] : 0ull;
            s_ent[w][lane] = valid ? sentry[p] : 0u;
            uint64_t T = wave_transpose64(M);
            const uint32_t cnt = (uint32_t)popc64(T);
            const uint32_t incl = wave_incl_scan(cnt);
            const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
            if (total > (uint32_t)kStepItems) {
                wave_lds_sync();
                for (; T != 0ull; T &= T - 1ull) tile_entry[run++] = s_ent[w][__builtin_ctzll(T)];
                wave_lds_sync();
                continue;
            }
            wave_lds_sync();
            // group the step's entries by tile, with their list positions
            for (uint32_t o = incl - cnt; T != 0ull; T &= T - 1ull, ++o) {
                s_item[w][o] = s_ent[w][__builtin_ctzll(T)];
                s_pos[w][o] = run++;
            }
            wave_lds_sync();
            for (uint32_t i = (uint32_t)lane; i < total; i += 64)
                tile_entry[s_pos[w][i]] = s_item[w][i];
            wave_lds_sync();
        }
    }
}

}  // namespace

hipError_t launch_store_views(const Views& views, Views* dst, hipStream_t s, uint32_t* counters,
                              int32_t* step, const int32_t* gate) {
    hipLaunchKernelGGL(store_views_kernel, dim3(1), dim3(64), 0, s, views, dst, counters, step,
                       gate);
    return hipGetLastError();
}

hipError_t launch_begin_bin(const Views& views, const ViewDev* table, int n_table,
                            const int32_t* d_view, const Layout& L, char* ws, hipStream_t s) {
    const int64_t n4 = (int64_t)(L.clear_words / 4);   // regions are 256-byte aligned
    const int64_t nb = std::min<int64_t>(std::max<int64_t>(1, n4 / (2 * kBeginThreads)), 1024);
    hipLaunchKernelGGL(begin_bin_kernel, dim3((unsigned)nb), dim3(kBeginThreads), 0, s, views, table,
                       n_table, d_view, reinterpret_cast<Views*>(ws + L.views),
                       reinterpret_cast<uint32_t*>(ws + L.counters),
                       reinterpret_cast<uint4*>(ws + L.clear_begin), n4);
    return hipGetLastError();
}

hipError_t fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// The split of the sorted super-tile lists into tile lists: of the prefixes of
// the long ones, the others whole, before compositing (kRest = false), or of the
// whole lists of the super-tiles flagged by that compositing, placed after the
// prefix lists (kRest = true; predicated on counters[kRedo]).
template <bool kRest>
static hipError_t launch_split(const RasterDev& rp, const Layout& L, char* ws, hipStream_t s) {
    if (L.total_supers == 0 || L.total_tiles == 0) return hipSuccess;
    const Views* views = reinterpret_cast<const Views*>(ws + L.views);
    uint32_t* counters = reinterpret_cast<uint32_t*>(ws + L.counters);
    const uint32_t* ranges = reinterpret_cast<const uint32_t*>(ws + L.sup_ranges);
    const uint32_t* skey = reinterpret_cast<const uint32_t*>(ws + L.pair_key[L.key_result]);
    const uint32_t* sentry = reinterpret_cast<const uint32_t*>(ws + L.pair_entry[L.key_result]);
    const float4* rec = reinterpret_cast<const float4*>(ws + L.records);
    uint32_t* seg_first = reinterpret_cast<uint32_t*>(ws + L.seg_first);
    uint32_t* seg_cnt = reinterpret_cast<uint32_t*>(ws + L.seg_cnt);
    uint32_t* seg_groups = reinterpret_cast<uint32_t*>(ws + L.seg_groups[kRest]);
    uint64_t* mask = reinterpret_cast<uint64_t*>(ws + L.pair_mask);
    uint32_t* sup_redo = reinterpret_cast<uint32_t*>(ws + L.sup_redo);
    uint32_t* sup_base = reinterpret_cast<uint32_t*>(ws + L.sup_base);
    const SegCountSrc<kRest> src{ranges, sup_redo, counters + kRedo, L.total_supers,
                                 (uint32_t)rp.prefix_segs, rp.seg_log2};
    const ItemCountSrc items{reinterpret_cast<const uint64_t*>(ws + L.sup_items[kRest]),
                             L.total_supers};
    hipError_t err;
    // segments to split; their total -> seg_first[total_supers] (formed by
    // the count kernel itself when the super-tiles are few)
    const bool local = L.total_supers <= kLocalSupers;
    if (!local) {
        hipLaunchKernelGGL(seg_scan_kernel<SegCountSrc<kRest>>, dim3(1), dim3(kSegScanThreads), 0, s,
                           src, seg_first);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    // grid-stride over the segments: at most a few resident waves per SIMD
    // (the completing split, usually idle and otherwise a few super-tiles,
    // on a quarter of the grid)
    static_assert(kSplitWaves == kWriteWaves, "one grid");
    const int64_t blocks = kRest ? kSplitBlocks / 4 : kSplitBlocks;
    const dim3 grid((unsigned)std::min<int64_t>((L.seg_slots + kSplitWaves - 1) / kSplitWaves,
                                                blocks));
    const uint32_t entries = (uint32_t)std::max<int64_t>(1, L.entries);
    hipLaunchKernelGGL(split_count_kernel<kRest>, grid, dim3(kSplitWaves * 64), 0, s, views, rp, src,
                       local, seg_first, ranges, skey, sentry, rec, entries, mask, seg_cnt,
                       seg_groups, reinterpret_cast<unsigned long long*>(ws + L.sup_items[kRest]));
    if ((err = hipGetLastError()) != hipSuccess) return err;
    if (!local) {
        hipLaunchKernelGGL(seg_scan_kernel<ItemCountSrc>, dim3(1), dim3(kSegScanThreads), 0, s, items,
                           sup_base);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    }
    hipLaunchKernelGGL(split_write_kernel<kRest>, grid, dim3(kWriteWaves * 64), 0, s, views, rp, src,
                       local, seg_first, sup_base, items, ranges, sentry, mask, seg_cnt, seg_groups,
                       counters, L.capacity, reinterpret_cast<uint32_t*>(ws + L.tile_entry),
                       reinterpret_cast<uint32_t*>(ws + L.tile_ranges),
                       reinterpret_cast<uint32_t*>(ws + L.tile_state), sup_redo);
    return hipGetLastError();
}

hipError_t launch_split_rest(const RasterDev& rp, const Layout& L, char* ws, hipStream_t s) {
    return launch_split<true>(rp, L, ws, s);
}

hipError_t launch_bin(const RasterDev& rp, int64_t n, const Layout& L, char* ws, hipStream_t s) {
    const int64_t E = L.entries;
    const Views* views = reinterpret_cast<const Views*>(ws + L.views);
    uint32_t* counters = reinterpret_cast<uint32_t*>(ws + L.counters);
    uint32_t* tiles = reinterpret_cast<uint32_t*>(ws + L.tiles);
    const float4* rec = reinterpret_cast<const float4*>(ws + L.records);
    uint32_t* dkey[2] = {reinterpret_cast<uint32_t*>(ws + L.dkey[0]),
                         reinterpret_cast<uint32_t*>(ws + L.dkey[1])};
    uint32_t* dval[2] = {reinterpret_cast<uint32_t*>(ws + L.dval[0]),
                         reinterpret_cast<uint32_t*>(ws + L.dval[1])};
    uint32_t* hist = reinterpret_cast<uint32_t*>(ws + L.sort_hist);
    uint32_t* ranges = reinterpret_cast<uint32_t*>(ws + L.sup_ranges);
    uint32_t* pkey[2] = {reinterpret_cast<uint32_t*>(ws + L.pair_key[0]),
                         reinterpret_cast<uint32_t*>(ws + L.pair_key[1])};
    uint32_t* pentry[2] = {reinterpret_cast<uint32_t*>(ws + L.pair_entry[0]),
                           reinterpret_cast<uint32_t*>(ws + L.pair_entry[1])};
    hipError_t err;
    if (E > 0) {
        // visible entries by depth, ties in entry order; their number and the
        // number of their pairs -> counters[kVisible], [kPairs]
        err = sort_entries(reinterpret_cast<const uint32_t*>(ws + L.depth), tiles, E, dkey, dval,
                           hist, reinterpret_cast<uint32_t*>(ws + L.sort_groups),
                           reinterpret_cast<uint64_t*>(ws + L.sort_weights), counters + kVisible,
                           counters + kPairs, s);
        if (err != hipSuccess) return err;
    }
    const uint32_t* sorted = dval[1];
    if (E > 0 && L.direct) {
        const uint4* info = reinterpret_cast<const uint4*>(ws + L.pair_info);
        uint4* sinfo = reinterpret_cast<uint4*>(ws + L.pair_sorted);
        uint32_t* phist = reinterpret_cast<uint32_t*>(ws + L.pair_hist);
        uint32_t* pgroups = reinterpret_cast<uint32_t*>(ws + L.pair_groups);
        const dim3 grid((unsigned)L.pair_blocks);
        const size_t ns = (size_t)L.total_supers;
        hipLaunchKernelGGL(pair_count_kernel, grid, dim3(kPairThreads), ns * sizeof(uint32_t), s,
                           views, rp, (uint32_t)n, sorted, info, counters, L.pair_rounds, sinfo,
                           phist, pgroups);
        hipLaunchKernelGGL(pair_place_kernel, grid, dim3(kPairThreads),
                           (kPairThreads / 64 + 2) * ns * sizeof(uint32_t), s, views, rp,
                           (uint32_t)n, counters, L.pair_rounds, sinfo, phist, pgroups, L.capacity,
                           ranges, pkey[0], pentry[0]);
        if ((err = hipGetLastError()) != hipSuccess) return err;
    } else if (E > 0) {
        uint32_t* offsets = reinterpret_cast<uint32_t*>(ws + L.offsets);
        uint32_t* window_first = reinterpret_cast<uint32_t*>(ws + L.window_first);
        uint32_t* sums = reinterpret_cast<uint32_t*>(ws + L.scan_sums);
        // pair offsets in depth order; total -> counters[kPairs]
        const uint32_t n_windows = (uint32_t)emit_windows(E, L.capacity);
        err = device_scan(PairCountSrc{tiles, sorted, counters + kVisible},
                          OffsetSink{offsets, window_first, n_windows}, E, sums,
                          counters + kPairs, s);
        if (err != hipSuccess) return err;
        // at least one workgroup: block 0 also records the written pair count
        const dim3 egrid((unsigned)std::max<int64_t>(1, emit_windows(E, L.capacity)));
        hipLaunchKernelGGL(emit_kernel, egrid, dim3(kEmitThreads), 0, s, sorted, offsets,
                           window_first, rec, counters, n, views, rp, L.capacity, pkey[0],
                           pentry[0]);
        if ((err = hipGetLastError()) != hipSuccess) return err;
        // stable sort of the pairs by super-tile; the first pass drops culled
        // pairs and counts the rest into counters[kPairsKept]
        err = sort_pairs(pkey, pentry, counters + kPairsWritten, L.capacity, L.key_bits, hist,
                         reinterpret_cast<uint32_t*>(ws + L.pair_sort_groups),
                         counters + kPairsKept, s);
        if (err != hipSuccess) return err;
    }
    const dim3 rgrid((unsigned)((L.total_supers + 255) / 256));
    if (L.total_supers > 0 && (E == 0 || !L.direct))
        hipLaunchKernelGGL(ranges_kernel, rgrid, dim3(256), 0, s, pkey[L.key_result], counters,
                           L.total_supers, L.key_bits, ranges);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    return launch_split<false>(rp, L, ws, s);
}

}  // namespace sgs
