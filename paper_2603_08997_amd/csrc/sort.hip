// Stable least-significant-digit radix sort of (key, uint32 value) pairs over
// the low bits of uint32 keys, digits of at most 8 bits, two launches a pass:
//   hist:    per-block digit counts [blocks][256], and their sums over groups
//            of kSortGroup blocks [groups][256] by atomics;
//   scatter: each block adds up the groups and the blocks before it (a digit a
//            thread, whole rows of counts at a time), ranks its keys stably
//            (each wave ranks a contiguous part of the block with ballots and
//            its own digit counters; per-wave counts give the order across
//            waves), sorts them into LDS, and writes digit runs out coalesced.
// Each block owns a contiguous range of keys, so equal digits keep their input
// order and the sort is stable; no pass waits on another block.
//
// The depth sort's first pass reads the uncompacted entries and drops the
// invisible ones, which makes the compaction of the visible entries part of
// it, and its last pass leaves the keys out.
//
// What bounds a pass: latency, the chain of loads, LDS passes and scattered
// stores of a block; its 32 bytes a key take a sixth of its time. Before, a
// scan kernel between the two walked the counts digit by digit and a separate
// scan compacted the entries: 12 + 2 launches for the depth sort instead of 8,
// and on sets that do not fill the chip a launch is most of a kernel's time.
#include <algorithm>

#include "sgs_internal.hpp"
#include "sgs_device.hpp"

namespace sgs {

namespace {

// Keys per block: us a pass of the 1M, 3M and 6M scenes (0.7, 2.05 and 4.1M
// keys) with 2048 12.4 / 20.5 / 44.5, with 4096 11.6 / 19.5 / 35.3, with 8192
// 14.2 / 29.2 / 45.4 (one block per compute unit is left); 21k keys 10.2 / 10.8 /
// 12.6.
constexpr int kThreads = 512;
constexpr int kKeys = 8;
constexpr int kTile = kThreads * kKeys;
constexpr int kWaves = kThreads / 64;
constexpr int kRadix = 256;
constexpr int kHistCopies = 4;

// What a pass sorts: key and value of input i, and whether it is kept.
struct EntrySrc {   // the visible entries, by depth bits
    const uint32_t* depth;
    const uint32_t* tiles;
    int64_t n;
    __device__ int64_t count() const { return n; }
    __device__ bool load(int64_t i, uint32_t& key, uint32_t& val) const {
        key = depth[i];
        val = (uint32_t)i;
        return tiles[i] != 0u;
    }
    __device__ uint32_t weight(int64_t i) const { return tiles[i]; }
};
template <bool kDrop>   // kDrop: keys with all bits set (culled pairs) are left out
struct PairSrc {
    const uint32_t* keys;
    const uint32_t* vals;
    const uint32_t* n;
    __device__ int64_t count() const { return *n; }
    __device__ bool load(int64_t i, uint32_t& key, uint32_t& val) const {
        key = keys[i];
        val = vals[i];
        return !kDrop || key != kCulledTile;
    }
};

__device__ __forceinline__ uint32_t digit_of(uint32_t k, int shift, uint32_t mask) {
    return (k >> shift) & mask;
}

// Mask of the lanes whose (valid) digit equals this lane's digit.
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid, int bits) {
    uint64_t peers = ballot(valid);
    for (int b = 0; b < bits; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t m = ballot(bit);
        peers &= bit ? m : ~m;
    }
    return peers;
}

// Digit counts of one block's kept keys (counting does not depend on order).
// kWeights: also the block's sum of the inputs' weights, to weights[block].
template <class Src, bool kWeights>
__global__ void __launch_bounds__(kThreads) radix_hist_kernel(Src src, int shift, int bits,
                                                        uint32_t* __restrict__ hist,
                                                        uint32_t* __restrict__ groups,
                                                        uint64_t* __restrict__ weights) {
    // kHistCopies counters per digit, lane l counting into copy l % kHistCopies,
    // so that fewer lanes of one atomic instruction hit the same address
    __shared__ uint32_t cnt[kHistCopies][kRadix];
    __shared__ uint64_t wsum[kThreads / 64];
    const int tid = threadIdx.x;
    const int64_t n = src.count();
    // the grid covers a bound; the first ceil(n / kTile) workgroups work
    const int active = (int)((n + kTile - 1) / kTile);
    if ((int)blockIdx.x >= active) return;
    const int blk = xcd_block(blockIdx.x, active);
    const int64_t base = (int64_t)blk * kTile;
    for (int i = tid; i < kHistCopies * kRadix; i += kThreads) cnt[i / kRadix][i % kRadix] = 0;
    // all loads first, then the counts
    uint32_t key[kKeys], val;
    bool ok[kKeys];
    uint64_t w = 0;
#pragma unroll
    for (int it = 0; it < kKeys; ++it) {
        const int64_t i = base + it * kThreads + tid;
        ok[it] = i < n && src.load(i, key[it], val);
        if constexpr (kWeights)
            if (i < n) w += src.weight(i);
    }
    __syncthreads();
    const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
    for (int it = 0; it < kKeys; ++it)
        if (ok[it]) atomicAdd(&cnt[tid % kHistCopies][digit_of(key[it], shift, mask)], 1u);
    if constexpr (kWeights) {
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) w += __shfl_xor(w, d, 64);
        if (tid % 64 == 0) wsum[tid / 64] = w;
    }
    __syncthreads();
    if (tid < kRadix) {
        uint32_t total = 0;
#pragma unroll
        for (int k = 0; k < kHistCopies; ++k) total += cnt[k][tid];
        hist[(int64_t)blk * kRadix + tid] = total;
        if (total != 0u) atomicAdd(&groups[(int64_t)(blk / kSortGroup) * kRadix + tid], total);
    }
    if constexpr (kWeights) {
        if (tid == 0) {
            w = 0;
            for (int k = 0; k < kThreads / 64; ++k) w += wsum[k];
            weights[blk] = w;
        }
    }
}

// Scatter of one block's keys. Wave w owns the contiguous key range
// [w kPerWave, (w+1) kPerWave) and ranks it in kKeys rounds of 64
// consecutive keys with its own LDS digit counters, so ranking needs no
// block barrier: within a round, lanes with the same digit are found with
// ballots and ordered by lane; across rounds the wave's counter carries the
// count. One barrier later, the digit's start in the block plus the counts of
// the earlier waves give every key its block-local position; keys are sorted
// into LDS and written out in digit runs. Block 0 also writes the number of
// kept keys (kept, nullable) and, with kWeights, the saturated sum of the
// weights.
template <class Src, bool kWeights, bool kKeysOut>
__global__ void __launch_bounds__(kThreads) radix_scatter_kernel(
    Src src, uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out, int shift, int bits,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ groups,
    const uint64_t* __restrict__ weights, uint32_t* __restrict__ kept,
    uint32_t* __restrict__ weight_sum) {
    constexpr int kPerWave = kTile / kWaves;
    constexpr int kParts = kThreads / kRadix;         // threads adding up a digit's counts
    __shared__ uint32_t lkeys[kTile];
    __shared__ uint32_t lvals[kTile];
    __shared__ uint32_t gbase[kRadix];          // global start of this block's digit run
    __shared__ uint32_t wcnt[kWaves][kRadix];   // keys of each digit per wave
    __shared__ uint32_t smem[kThreads / 64 + 1];

    const int64_t n = src.count();
    const int active = (int)((n + kTile - 1) / kTile);
    const int tid = threadIdx.x, w = tid / 64, lane = tid % 64;
    if ((int)blockIdx.x >= active) {   // uniform across the block
        if (active == 0 && blockIdx.x == 0 && tid == 0) {
            if (kept != nullptr) *kept = 0u;
            if (kWeights) *weight_sum = 0u;
        }
        return;
    }
    const int blk = xcd_block(blockIdx.x, active);
    const int64_t base = (int64_t)blk * kTile;
    const uint32_t mask = (1u << bits) - 1u;

    // all loads first: wave w, round it, lane l holds key w*kPerWave + 64*it + l
    uint32_t key[kKeys], val[kKeys];
    uint32_t ok = 0;
#pragma unroll
    for (int it = 0; it < kKeys; ++it) {
        const int64_t i = base + w * kPerWave + it * 64 + lane;
        key[it] = val[it] = 0u;
        if (i < n && src.load(i, key[it], val[it])) ok |= 1u << it;
    }
    {
        // lkeys serves as scratch: [part][digit] totals, lvals: counts before
        const int d = tid % kRadix, part = tid / kRadix;
        const int ng = (active + kSortGroup - 1) / kSortGroup, g = blk / kSortGroup;
        uint32_t tot = 0, before = 0;
        for_rows(groups + d, kRadix, part, ng, kParts, [&](int j, uint32_t c) {
            tot += c;
            before += j < g ? c : 0u;
        });
        for_rows(hist + d, kRadix, g * (int)kSortGroup + part, blk, kParts,
                 [&](int, uint32_t c) { before += c; });
        lkeys[tid] = tot;
        lvals[tid] = before;
        __syncthreads();
        tot = before = 0;
        if (tid < kRadix) {
#pragma unroll
            for (int k = 0; k < kParts; ++k) {
                tot += lkeys[k * kRadix + tid];
                before += lvals[k * kRadix + tid];
            }
        }
        uint32_t all;
        const uint32_t ex = block_excl_scan<kThreads>(tot, smem, &all);
        if (tid < kRadix) gbase[tid] = ex + before;
        if (blockIdx.x == 0 && tid == 0 && kept != nullptr) *kept = all;
    }
    if (kWeights && blockIdx.x == 0 && w == 0) {
        uint64_t s = 0;
        for (int j = lane; j < active; j += 64) s += weights[j];
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d, 64);
        if (lane == 0) *weight_sum = (uint32_t)min(s, (uint64_t)0xffffffffull);
    }
    for (int i = tid; i < kWaves * kRadix; i += kThreads) wcnt[i / kRadix][i % kRadix] = 0;
    __syncthreads();

    // wave-private stable ranking (dropped keys take no position)
    uint32_t rank[kKeys];
#pragma unroll
    for (int it = 0; it < kKeys; ++it) {
        const bool valid = (ok >> it) & 1u;
        const uint32_t d = digit_of(key[it], shift, mask);
        const uint64_t peers = match_digit(d, valid, bits);
        const uint32_t before = (uint32_t)popc64(peers & lanemask_lt());
        uint32_t r = 0;
        if (valid) r = wcnt[w][d] + before;
        rank[it] = r;
        // every lane has read the counters before the leaders advance them
        __builtin_amdgcn_wave_barrier();
        if (valid && before == 0) wcnt[w][d] += (uint32_t)popc64(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // per digit (thread tid): start in the block and the counts of earlier waves
    int nkept;
    {
        uint32_t sum = 0;
        if (tid < kRadix) {
#pragma unroll
            for (int k = 0; k < kWaves; ++k) sum += wcnt[k][tid];
        }
        uint32_t tot;
        uint32_t start = block_excl_scan<kThreads>(sum, smem, &tot);
        if (tid < kRadix) {
#pragma unroll
            for (int k = 0; k < kWaves; ++k) {
                const uint32_t c = wcnt[k][tid];
                wcnt[k][tid] = start;
                start += c;
            }
        }
        nkept = (int)tot;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kKeys; ++it) {
        if ((ok >> it) & 1u) {
            const uint32_t pos = wcnt[w][digit_of(key[it], shift, mask)] + rank[it];
            lkeys[pos] = key[it];
            lvals[pos] = val[it];
        }
    }
    __syncthreads();
    // wcnt[0][d] is now the block-local start of digit d
#pragma unroll 4
    for (int li = tid; li < nkept; li += kThreads) {
        const uint32_t k = lkeys[li];
        const uint32_t d = digit_of(k, shift, mask);
        const uint32_t out = gbase[d] + (uint32_t)li - wcnt[0][d];
        if (kKeysOut) keys_out[out] = k;
        vals_out[out] = lvals[li];
    }
}

// The depth sort of a set that one workgroup holds: every pass in LDS, in one
// launch instead of eight that each last a launch's latency (a few us). Wave w
// ranks positions [w 64 R, (w+1) 64 R) as in the scatter above. 1000 entries: 49 us
// before, 8.9 now. The whole binning of 2000 entries: 45 us, 51 by sorted runs,
// 77 in eight launches; with 8 keys a thread 4k / 8k entries took 62 / 67 us where
// runs take 53 / 54.
//
// kRuns: every workgroup sorts its own range of inputs into a run (keys and
// values at the range's start), for merge_runs_kernel; run_count and run_weight
// get the number of its visible entries and their weights' sum.
constexpr int64_t kSmallSort = 2048;
template <int T, int R, bool kRuns>
__global__ void __launch_bounds__(T) small_sort_kernel(
    EntrySrc src, uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out,
    uint32_t* __restrict__ kept, uint32_t* __restrict__ weight_sum,
    uint32_t* __restrict__ run_count, uint64_t* __restrict__ run_weight) {
    constexpr int NW = T / 64;
    static_assert(T >= kRadix, "a digit a thread");
    __shared__ uint32_t lkeys[T * R];
    __shared__ uint32_t lvals[T * R];
    __shared__ uint32_t wcnt[NW][kRadix];   // keys of each digit per wave
    __shared__ uint32_t smem[NW + 1];
    __shared__ uint64_t wsum[NW];
    const int tid = threadIdx.x, w = tid / 64, lane = tid % 64;
    const int64_t base = kRuns ? (int64_t)blockIdx.x * (T * R) : 0;
    int n = (int)min(src.n - base, (int64_t)(T * R));
    uint32_t key[R], val[R], rank[R];
    uint32_t ok = 0;
    uint64_t sum = 0;
#pragma unroll
    for (int it = 0; it < R; ++it) {
        const int i = (w * R + it) * 64 + lane;
        key[it] = val[it] = 0u;
        if (i < n) {
            if (src.load(base + i, key[it], val[it])) ok |= 1u << it;
            sum += src.weight(base + i);
        }
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) wsum[w] = sum;
    for (int pass = 0; pass < kDepthPasses; ++pass) {
        const int shift = 8 * pass;
#pragma unroll
        for (int k = 0; k < kRadix / 64; ++k) wcnt[w][64 * k + lane] = 0;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < R; ++it) {
            const bool valid = (ok >> it) & 1u;
            const uint32_t d = digit_of(key[it], shift, kRadix - 1u);
            const uint64_t peers = match_digit(d, valid, 8);
            const uint32_t before = (uint32_t)popc64(peers & lanemask_lt());
            uint32_t r = 0;
            if (valid) r = wcnt[w][d] + before;
            rank[it] = r;
            __builtin_amdgcn_wave_barrier();
            if (valid && before == 0) wcnt[w][d] += (uint32_t)popc64(peers);
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // per digit (thread tid): the start of every wave's keys
        uint32_t c[NW], total = 0, all;
        if (tid < kRadix) {
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                c[k] = wcnt[k][tid];
                total += c[k];
            }
        }
        uint32_t start = block_excl_scan<T>(total, smem, &all);
        if (tid < kRadix) {
#pragma unroll
            for (int k = 0; k < NW; ++k) {
                wcnt[k][tid] = start;
                start += c[k];
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < R; ++it) {
            if ((ok >> it) & 1u) {
                const uint32_t pos = wcnt[w][digit_of(key[it], shift, kRadix - 1u)] + rank[it];
                lkeys[pos] = key[it];
                lvals[pos] = val[it];
            }
        }
        __syncthreads();
        n = (int)all;   // (after the first pass the invisible are gone)
        if (pass == kDepthPasses - 1) break;
        ok = 0;
#pragma unroll
        for (int it = 0; it < R; ++it) {
            const int i = (w * R + it) * 64 + lane;
            if (i < n) {
                key[it] = lkeys[i];
                val[it] = lvals[i];
                ok |= 1u << it;
            }
        }
    }
    for (int i = tid; i < n; i += T) {
        if (kRuns) keys_out[base + i] = lkeys[i];
        vals_out[base + i] = lvals[i];
    }
    if (tid == 0) {
        sum = 0;
        for (int k = 0; k < NW; ++k) sum += wsum[k];
        if (kRuns) {
            run_count[blockIdx.x] = (uint32_t)n;
            run_weight[blockIdx.x] = sum;
        } else {
            *kept = (uint32_t)n;
            *weight_sum = (uint32_t)min(sum, (uint64_t)0xffffffffull);
        }
    }
}

// Merge of all runs in one launch: a thread an entry, whose place is its place
// in its run and, in every other run, the number of entries before it (equal
// keys: those of earlier runs, whose inputs come first). A workgroup takes
// kMergeThreads neighbouring entries of a run: it finds the stretches of the
// other runs between its smallest and its largest key, brings them into LDS, and
// its threads search there (stretches that don't fit are searched where they
// are).
//
// What bounds it: latency, and with the number of runs the searches, which grow
// with the square of the set. The whole binning, two launches / eight: 8k entries
// 54 / 86 us, 16k 58 / 87, 30k 66 / 90, 65k 81 / 94, 131k 153 / 101 (64 runs). With
// every search in global memory 30k took 80 us and 65k 119.
constexpr int kRunThreads = 1024;
constexpr int kRunKeys = 2;
constexpr int kRun = kRunThreads * kRunKeys;
constexpr int kMergeThreads = 256;
constexpr int kMaxRuns = 32;
constexpr int kSearches = 4;        // at a time
constexpr int kStretch = 10240;     // keys in LDS
constexpr int64_t kRunSort = (int64_t)kRun * kMaxRuns;   // entries up to which runs are merged
__global__ void __launch_bounds__(kMergeThreads) merge_runs_kernel(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals, int runs,
    const uint32_t* __restrict__ run_count, const uint64_t* __restrict__ run_weight,
    uint32_t* __restrict__ vals_out, uint32_t* __restrict__ kept,
    uint32_t* __restrict__ weight_sum) {
    constexpr int kParts = kRun / kMergeThreads;
    __shared__ uint32_t s_keys[kStretch];
    __shared__ int s_end[2][kMaxRuns];   // per run: first and past the last key of the stretch
    __shared__ int s_at[kMaxRuns];       // its place in s_keys, or -1
    const int tid = threadIdx.x;
    const int run = blockIdx.x / kParts, first = (int)(blockIdx.x % kParts) * kMergeThreads;
    if (blockIdx.x == 0 && tid < 64) {
        uint32_t n = 0;
        uint64_t w = 0;
        if (tid < runs) {
            n = run_count[tid];
            w = run_weight[tid];
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            n += (uint32_t)__shfl_xor((int)n, d, 64);
            w += __shfl_xor(w, d, 64);
        }
        if (tid == 0) {
            *kept = n;
            *weight_sum = (uint32_t)min(w, (uint64_t)0xffffffffull);
        }
    }
    const int mine = (int)run_count[run] - first;   // entries of this workgroup and after
    if (mine <= 0) return;                          // uniform
    const uint32_t* own = keys + (int64_t)run * kRun + first;
    const uint32_t lo = own[0], hi = own[min(mine, kMergeThreads) - 1];
    {
        // keys below lo and up to hi in every run, runs side by side: of 64 evenly
        // spaced keys, then of the 32 from the last such key that counts
        constexpr int NQ = kMaxRuns / (kMergeThreads / 64), kStep = kRun / 64;
        static_assert(2 * kStep == 64, "two searches a wave");
        const int w = tid / 64, lane = tid % 64;
        int n[NQ], from[NQ];
        uint32_t k[NQ];
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            const int q = w + j * (kMergeThreads / 64), at = (lane + 1) * kStep - 1;
            n[j] = q < runs && q != run ? (int)run_count[min(q, runs - 1)] : 0;
            k[j] = at < n[j] ? keys[(int64_t)q * kRun + at] : 0u;
        }
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            const int q = w + j * (kMergeThreads / 64), at = (lane + 1) * kStep - 1;
            const int a = kStep * popc64(ballot(at < n[j] && k[j] < lo));
            const int b = kStep * popc64(ballot(at < n[j] && k[j] <= hi));
            from[j] = lane < kStep ? a : b;
            const int i = from[j] + lane % kStep;
            k[j] = i < n[j] ? keys[(int64_t)q * kRun + i] : 0u;
        }
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            const int q = w + j * (kMergeThreads / 64), i = from[j] + lane % kStep;
            const uint64_t m =
                ballot(i < n[j] && (lane < kStep ? k[j] < lo : k[j] <= hi));
            if (lane % kStep == 0)
                s_end[lane / kStep][q] = from[j] + popc64(lane ? m >> kStep : m & 0xffffffffull);
        }
    }
    __syncthreads();
    if (tid < kMaxRuns) {
        const int n = s_end[1][tid] - s_end[0][tid];
        const int at = (int)wave_incl_scan((uint32_t)n) - n;
        s_at[tid] = at + n <= kStretch ? at : -1;
    }
    __syncthreads();
    for (int q = tid / 64; q < runs; q += kMergeThreads / 64) {
        const int a = s_end[0][q], n = s_end[1][q] - a, at = s_at[q];
        if (at < 0) continue;
        for (int k = tid % 64; k < n; k += 64) s_keys[at + k] = keys[(int64_t)q * kRun + a + k];
    }
    __syncthreads();
    if (tid >= mine) return;
    const uint32_t key = own[tid];
    int place = first + tid;
    for (int q0 = 0; q0 < runs; q0 += kSearches) {
        int pos[kSearches], n[kSearches], at[kSearches], longest = 0;
        bool fits = true;
#pragma unroll
        for (int u = 0; u < kSearches; ++u) {
            const int q = min(q0 + u, kMaxRuns - 1);
            const int a = __builtin_amdgcn_readfirstlane(s_end[0][q]);
            n[u] = __builtin_amdgcn_readfirstlane(s_end[1][q]) - a;   // (0 past the last run)
            at[u] = __builtin_amdgcn_readfirstlane(s_at[q]);
            place += a;
            pos[u] = 0;
            longest = max(longest, n[u]);
            fits &= at[u] >= 0;
        }
        if (longest == 0) continue;
        auto search = [&](auto key_at) {
            for (int half = 1 << (31 - __builtin_clz((unsigned)longest)); half > 0; half >>= 1) {
#pragma unroll
                for (int u = 0; u < kSearches; ++u) {
                    const int i = pos[u] + half - 1;
                    const uint32_t k = key_at(u, max(min(i, n[u] - 1), 0));
                    const bool before = k < key || (q0 + u < run && k == key);
                    pos[u] += i < n[u] && before ? half : 0;
                }
            }
        };
        if (fits)   // uniform
            search([&](int u, int i) { return s_keys[min(at[u] + i, kStretch - 1)]; });
        else
            search([&](int u, int i) {
                const int q = min(q0 + u, runs - 1);
                return keys[(int64_t)q * kRun + min(s_end[0][q] + i, kRun - 1)];
            });
#pragma unroll
        for (int u = 0; u < kSearches; ++u) place += pos[u];
    }
    vals_out[place] = vals[(int64_t)run * kRun + first + tid];
}

struct Pass {
    int shift, bits;
    uint32_t *hist, *groups;
    uint64_t* weights;
    uint32_t *kept, *weight_sum;
};

template <class Src, bool kWeights = false, bool kKeysOut = true>
void run_pass(const Src& src, const Pass& p, uint32_t* keys_out, uint32_t* vals_out, int64_t n_max,
              hipStream_t s) {
    const dim3 grid((unsigned)radix_blocks(n_max)), block(kThreads);
    hipLaunchKernelGGL((radix_hist_kernel<Src, kWeights>), grid, block, 0, s, src, p.shift, p.bits,
                       p.hist, p.groups, p.weights);
    hipLaunchKernelGGL((radix_scatter_kernel<Src, kWeights, kKeysOut>), grid, block, 0, s, src,
                       keys_out, vals_out, p.shift, p.bits, p.hist, p.groups, p.weights, p.kept,
                       p.weight_sum);
}

}  // namespace

int64_t radix_blocks(int64_t n_max) {
    return std::max<int64_t>(1, (n_max + kTile - 1) / kTile);
}

int64_t radix_group_words(int64_t n_max, int passes) {
    return passes * kRadix * ((radix_blocks(n_max) + kSortGroup - 1) / kSortGroup);
}

int radix_passes(int bits) { return bits <= 0 ? 0 : (bits + 7) / 8; }

// Bits of pass p when `bits` are sorted in radix_passes(bits) passes of
// near-equal width (13 bits: 7 + 6).
static int pass_bits(int bits, int p, int* shift) {
    const int passes = radix_passes(bits);
    const int base = bits / passes, extra = bits % passes;
    int sh = 0;
    for (int q = 0; q < p; ++q) sh += base + (q < extra ? 1 : 0);
    *shift = sh;
    return base + (p < extra ? 1 : 0);
}

hipError_t sort_entries(const uint32_t* depth, const uint32_t* tiles, int64_t entries,
                        uint32_t* keys[2], uint32_t* vals[2], uint32_t* hist, uint32_t* groups,
                        uint64_t* weights, uint32_t* n_visible, uint32_t* pairs, hipStream_t s) {
    if (entries <= kSmallSort) {
        const EntrySrc src{depth, tiles, entries};
        if (entries <= 1024)
            hipLaunchKernelGGL((small_sort_kernel<1024, 1, false>), dim3(1), dim3(1024), 0, s, src,
                               nullptr, vals[1], n_visible, pairs, nullptr, nullptr);
        else
            hipLaunchKernelGGL((small_sort_kernel<1024, 2, false>), dim3(1), dim3(1024), 0, s, src,
                               nullptr, vals[1], n_visible, pairs, nullptr, nullptr);
        return hipGetLastError();
    }
    if (entries <= kRunSort) {
        const EntrySrc src{depth, tiles, entries};
        const int runs = (int)((entries + kRun - 1) / kRun);
        uint64_t* run_weight = reinterpret_cast<uint64_t*>(hist);
        uint32_t* run_count = hist + 2 * runs;
        hipLaunchKernelGGL((small_sort_kernel<kRunThreads, kRunKeys, true>), dim3(runs),
                           dim3(kRunThreads), 0, s, src, keys[0], vals[0], nullptr, nullptr,
                           run_count, run_weight);
        hipLaunchKernelGGL(merge_runs_kernel, dim3(runs * (kRun / kMergeThreads)),
                           dim3(kMergeThreads), 0, s, keys[0], vals[0], runs, run_count, run_weight,
                           vals[1], n_visible, pairs);
        return hipGetLastError();
    }
    const int64_t gw = radix_group_words(entries, 1);
    Pass p{0, 8, hist, groups, weights, n_visible, pairs};
    run_pass<EntrySrc, true>(EntrySrc{depth, tiles, entries}, p, keys[0], vals[0], entries, s);
    p.weights = nullptr;
    p.kept = p.weight_sum = nullptr;
    for (int k = 1; k < kDepthPasses; ++k) {
        p.shift = 8 * k;
        p.groups = groups + k * gw;
        const int in = (k - 1) & 1;
        const PairSrc<false> src{keys[in], vals[in], n_visible};
        if (k == kDepthPasses - 1)
            run_pass<PairSrc<false>, false, false>(src, p, nullptr, vals[in ^ 1], entries, s);
        else
            run_pass<PairSrc<false>>(src, p, keys[in ^ 1], vals[in ^ 1], entries, s);
    }
    return hipGetLastError();
}

hipError_t sort_pairs(uint32_t* keys[2], uint32_t* vals[2], const uint32_t* n_dev, int64_t n_max,
                      int bits, uint32_t* hist, uint32_t* groups, uint32_t* kept, hipStream_t s) {
    const int passes = radix_passes(bits);
    const int64_t gw = radix_group_words(n_max, 1);
    for (int k = 0; k < passes; ++k) {
        Pass p{0, 0, hist, groups + k * gw, nullptr, k == 0 ? kept : nullptr, nullptr};
        p.bits = pass_bits(bits, k, &p.shift);
        const int in = k & 1;
        if (k == 0)
            run_pass(PairSrc<true>{keys[0], vals[0], n_dev}, p, keys[1], vals[1], n_max, s);
        else
            run_pass(PairSrc<false>{keys[in], vals[in], kept}, p, keys[in ^ 1], vals[in ^ 1],
                     n_max, s);
    }
    return hipGetLastError();
}

}  // namespace sgs
