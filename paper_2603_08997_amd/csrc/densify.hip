// Adaptive density control of the densification phase (Sec. 3): the
// view-space positional gradient statistic gathered after each backward, and
// one clone / split / prune step over all Gaussians.
//
// Statistic: for every Gaussian visible in a view of the last render, the
// norm of dL/d(u, v) in normalised device units (the image spans [-1, 1] on
// each axis), || (dL/du W / 2, dL/dv H / 2) ||, added to a running sum and
// the view counted; dL/du and dL/dv are the first two floats of the entry's
// record-gradient accumulator the compositing backward left.
//
// Step: a Gaussian whose opacity is below min_opacity produces nothing; one
// whose mean statistic reaches grad_threshold is cloned (exact copy added)
// when its largest scale is at most percent_dense * scene_extent and split
// otherwise (replaced by two children centred at mu + R(q) diag(s) z_j, z_j
// drawn by the caller, with scales s / split_scale); every other Gaussian is
// kept. The new set is written as the kept Gaussians in index order, then the
// clones, then the children (two per split Gaussian), into separate output
// planes; kept Gaussians keep their Adam moments, new ones start at zero. The
// decisions compare the float32 log-scale and opacity logit with float32
// thresholds formed in binary64 on the host, and the statistic's sum with
// threshold * count in binary64, so they are exact for the given inputs.
//
// Two launches: per-block counts of the three outcomes (packed in one word
// per thread), and the write, which adds up the counts, repeats the decisions,
// scans them within the block and streams every plane of every output Gaussian;
// all outputs of one segment from one block are consecutive. An output set larger than the output planes' stride is reported
// and nothing is written.
#include <algorithm>

#include "sgs_internal.hpp"
#include "sgs_device.hpp"

namespace sgs {

namespace {

constexpr uint32_t kNoClone = 0xffffu;
constexpr int kLineWords = 32;
constexpr int kGroup = 8;   // planes whose loads are in flight together
// outcome counts packed in one word: keep in bits 0-9, clone 10-19, split 20-29
// (up to a workgroup's threads of each)
constexpr int kClonePos = 10, kSplitPos = 20;
constexpr uint32_t kField = (1u << 10) - 1u;

__global__ void __launch_bounds__(256) densify_stats_kernel(
    const Views* __restrict__ views, int64_t n, const uint32_t* __restrict__ tiles,
    const float* __restrict__ accum, const int32_t* __restrict__ gate, float* __restrict__ grad_sum,
    int32_t* __restrict__ count) {
    if (gate_closed(gate)) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float s = 0.f;
    int c = 0;
    for (int v = 0; v < views->n; ++v) {
        const int64_t e = (int64_t)v * n + i;
        if (tiles[e] == 0u) continue;
        const float du = accum[kAccumFloats * e] * (0.5f * (float)views->v[v].width);
        const float dv = accum[kAccumFloats * e + 1] * (0.5f * (float)views->v[v].height);
        s += sqrtf(fmaf(du, du, dv * dv));
        ++c;
    }
    if (c > 0) {
        grad_sum[i] += s;
        count[i] += c;
    }
}

// Output stores through L2 with the default policy: the lines at the ends of a
// workgroup's outputs, and those of clones and children, are filled by several
// waves and are best merged in L2 before they go to HBM.
__device__ __forceinline__ void put(const PlaneBuf& B, int j, uint32_t lane_off, float x) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), B.rsrc(j), (int)lane_off, 0, 0);
}

__device__ __forceinline__ uint32_t outcome(const PlaneBuf& P, uint32_t off, float g, int32_t c,
                                            const DensifyDev& d) {
    const float logit = P.load(10, off);
    const float ls = fmaxf(fmaxf(P.load(3, off), P.load(4, off)), P.load(5, off));
    if (logit < d.logit_min) return 0u;
    const bool cand = c > 0 && (double)g >= (double)d.grad_threshold * (double)c;
    if (!cand) return 1u;                       // keep
    return ls > d.log_size ? (1u << kSplitPos)  // split
                           : (1u | (1u << kClonePos));   // keep and clone
}

// Outcomes of each workgroup of the write: counts[k nblocks + b], k = kept,
// clones, split.
template <int T, int kParts>
__global__ void __launch_bounds__(T) densify_count_kernel(
    PlaneBuf P, int64_t n, const float* __restrict__ grad_sum, const int32_t* __restrict__ count,
    DensifyDev d, uint32_t* __restrict__ counts) {
    constexpr int kWriteInputs = T * kParts;
    __shared__ uint32_t s_sum[3];
    if (threadIdx.x < 3) s_sum[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * kWriteInputs + threadIdx.x;
    uint32_t o = 0;   // (at most kParts of each)
#pragma unroll
    for (int part = 0; part < kParts; ++part) {
        const int64_t i = first + part * T;
        if (i < n) o += outcome(P, (uint32_t)i * 4u, grad_sum[i], count[i], d);
    }
#pragma unroll
    for (int k = 32; k > 0; k >>= 1) o += (uint32_t)__shfl_xor((int)o, k, 64);
    if (threadIdx.x % 64 == 0) {
        atomicAdd(&s_sum[0], o & kField);
        atomicAdd(&s_sum[1], (o >> kClonePos) & kField);
        atomicAdd(&s_sum[2], (o >> kSplitPos) & kField);
    }
    __syncthreads();
    if (threadIdx.x < 3)
        counts[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = s_sum[threadIdx.x];
}

// The write. A workgroup adds up the counts of all workgroups (its outputs' places
// and the size of the new set), repeats the decisions of its inputs and lists
// its outputs in LDS (the input of each kept output and the rank of its clone,
// the inputs that split). The kept outputs are then walked in positions aligned
// to the cache line, so that a line is written by one wave but at the ends of
// the workgroup's range, and loads, which then straddle lines, go through L2, in
// groups of kGroup planes whose loads are all issued before their stores; a
// clone's store takes its parent's value from the same lane. Children take two
// threads a split Gaussian, and the zero moments of all new Gaussians are one
// range, cleared in whole lines.
//
// What bounds it: HBM (3M Gaussians, SH 3: 4.5 GB). One input a thread with its
// outputs stored where they fell took 1483 us, every line in parts from several
// waves on different XCDs; now 1026 (4.3 TB/s). Of the same with cached stores
// 1171, with streamed loads 1488 (1.5 lines fetched for each one used), in
// workgroups of 256 threads and 4096 inputs 1057, of 512 and 4096 1045. Adding up
// 1465 counts in every workgroup replaces a scan launch of 28 us.
template <int T, int kParts>
__global__ void __launch_bounds__(T) densify_write_kernel(
    PlaneBuf P, PlaneBuf M, PlaneBuf V, int64_t n, int F,
    const float* __restrict__ grad_sum, const int32_t* __restrict__ count,
    const float* __restrict__ normals, DensifyDev d, const uint32_t* __restrict__ counts,
    int64_t* __restrict__ n_out, int64_t out_stride, PlaneBuf PO, PlaneBuf MO, PlaneBuf VO) {
    constexpr int kWaves = T / 64, kWriteInputs = T * kParts;
    // (three counts a workgroup: the scratch has four words per 256 inputs)
    static_assert(T * kParts >= 256 && T <= 512, "scratch and packed counts");
    __shared__ uint32_t smem[kWaves + 1];
    __shared__ uint32_t s_sum[6];
    __shared__ uint16_t s_kept[kWriteInputs];    // input (within the workgroup) of a kept output
    __shared__ uint16_t s_clone[kWriteInputs];   // rank of its clone, or kNoClone
    __shared__ uint16_t s_split[kWriteInputs];
    const int tid = threadIdx.x;
    // neighbouring workgroups on one XCD: the lines they share meet in its L2
    const int nblocks = (int)gridDim.x;
    const int blk = xcd_block(blockIdx.x, nblocks);
    // totals of the three outcomes and those of the workgroups before
    if (tid < 6) s_sum[tid] = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        uint32_t all = 0, before = 0;
        for_rows(counts + (int64_t)k * nblocks, 1, tid, nblocks, T,
                 [&](int j, uint32_t c) {
                     all += c;
                     before += j < blk ? c : 0u;
                 });
#pragma unroll
        for (int x = 32; x > 0; x >>= 1) {
            all += (uint32_t)__shfl_xor((int)all, x, 64);
            before += (uint32_t)__shfl_xor((int)before, x, 64);
        }
        if (tid % 64 == 0) {
            atomicAdd(&s_sum[k], all);
            atomicAdd(&s_sum[3 + k], before);
        }
    }
    __syncthreads();
    const uint32_t K = s_sum[0], Cn = s_sum[1];
    const int64_t out = (int64_t)K + (int64_t)Cn + 2 * (int64_t)s_sum[2];
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) *n_out = out;
    if (out > out_stride) return;   // the caller provides larger planes and calls again
    const uint32_t k0 = s_sum[3], c0 = K + s_sum[4], s0 = K + Cn + 2u * s_sum[5];
    const int64_t first = (int64_t)blk * kWriteInputs;
    uint32_t kept = 0, clones = 0, splits = 0;
    for (int r = 0; r < kParts; ++r) {
        const int local = r * T + tid;
        const int64_t i = first + local;
        const uint32_t o = i < n ? outcome(P, (uint32_t)i * 4u, grad_sum[i], count[i], d) : 0u;
        uint32_t tot;
        const uint32_t ex = block_excl_scan<T>(o, smem, &tot);
        if (o & kField) {
            const uint32_t at = kept + (ex & kField);
            s_kept[at] = (uint16_t)local;
            s_clone[at] = (uint16_t)((o >> kClonePos) & kField
                                         ? clones + ((ex >> kClonePos) & kField) : kNoClone);
        }
        if ((o >> kSplitPos) & kField)
            s_split[splits + ((ex >> kSplitPos) & kField)] = (uint16_t)local;
        kept += tot & kField;
        clones += (tot >> kClonePos) & kField;
        splits += (tot >> kSplitPos) & kField;
    }
    __syncthreads();
    const int part = blockIdx.y, parts = gridDim.y;   // which groups of planes
    // kept Gaussians and clones
    for (uint32_t p0 = k0 & ~(uint32_t)(kLineWords - 1); p0 < k0 + kept; p0 += T) {
        const uint32_t p = p0 + (uint32_t)tid;
        if (p < k0 || p >= k0 + kept) continue;
        const uint32_t off = (uint32_t)(first + s_kept[p - k0]) * 4u;
        const uint32_t clone = s_clone[p - k0];
        const uint32_t pc = (c0 + clone) * 4u;
        for (int f0 = part * kGroup; f0 < F; f0 += parts * kGroup) {
            float x[kGroup], mm[kGroup], vv[kGroup];
#pragma unroll
            for (int k = 0; k < kGroup; ++k) {
                const int f = min(f0 + k, F - 1);
                x[k] = P.load<0>(f, off);
                mm[k] = M.load<0>(f, off);
                vv[k] = V.load<0>(f, off);
            }
#pragma unroll
            for (int k = 0; k < kGroup; ++k) {
                const int f = f0 + k;
                if (f >= F) break;
                PO.store(f, p * 4u, x[k]);
                MO.store(f, p * 4u, mm[k]);
                VO.store(f, p * 4u, vv[k]);
                if (clone != kNoClone) put(PO, f, pc, x[k]);
            }
        }
    }
    // children
    for (uint32_t c = tid; c < 2u * splits; c += T) {
        const int64_t i = first + s_split[c / 2u];
        const uint32_t off = (uint32_t)i * 4u, po = (s0 + c) * 4u;
        if (part == 0) {
            float mu[3], ls[3], s[3], q[4];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                mu[k] = P.load(k, off);
                ls[k] = P.load(3 + k, off);
                s[k] = expf(ls[k]);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) q[k] = P.load(6 + k, off);
            const float qn = 1.f / sqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
            const float w = q[0] * qn, x = q[1] * qn, y = q[2] * qn, z = q[3] * qn;
            const float R[9] = {1.f - 2.f * (y * y + z * z), 2.f * (x * y - w * z), 2.f * (x * z + w * y),
                                2.f * (x * y + w * z), 1.f - 2.f * (x * x + z * z), 2.f * (y * z - w * x),
                                2.f * (x * z - w * y), 2.f * (y * z + w * x), 1.f - 2.f * (x * x + y * y)};
            const float* zj = normals + 6 * i + 3 * (c % 2u);
            const float t[3] = {s[0] * zj[0], s[1] * zj[1], s[2] * zj[2]};
#pragma unroll
            for (int r = 0; r < 3; ++r)
                put(PO, r, po, mu[r] + (R[3 * r] * t[0] + R[3 * r + 1] * t[1] + R[3 * r + 2] * t[2]));
#pragma unroll
            for (int k = 0; k < 3; ++k) put(PO, 3 + k, po, ls[k] - d.log_split);
        }
        for (int f0 = 6 + part * kGroup; f0 < F; f0 += parts * kGroup) {
            float v[kGroup];
#pragma unroll
            for (int k = 0; k < kGroup; ++k) v[k] = P.load(min(f0 + k, F - 1), off);
#pragma unroll
            for (int k = 0; k < kGroup; ++k)
                if (f0 + k < F) put(PO, f0 + k, po, v[k]);
        }
    }
    // the moments of the new Gaussians: workgroup after workgroup takes a stretch
    // of whole lines of every plane
    const int64_t z0 = K & ~63u;
    const int64_t each = ((out - z0 + nblocks - 1) / nblocks + 63) & ~(int64_t)63;
    const int64_t a = z0 + blk * each;
    for (int64_t p = a + tid % 64; p < min(a + each, out); p += 64) {
        if (p < (int64_t)K) continue;
        for (int f = tid / 64 + part * (T / 64); f < F; f += parts * (T / 64)) {
            MO.store(f, (uint32_t)p * 4u, 0.f);
            VO.store(f, (uint32_t)p * 4u, 0.f);
        }
    }
}

}  // namespace

// (what a caller's scratch is sized by)
int64_t densify_blocks(int64_t n) { return (n + 255) / 256; }

hipError_t launch_densify_stats(const Layout& L, char* ws, int64_t n, const int32_t* gate,
                                float* grad_sum, int32_t* count, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const Views* views = reinterpret_cast<const Views*>(ws + L.views);
    const uint32_t* tiles = reinterpret_cast<const uint32_t*>(ws + L.tiles);
    const float* acc = reinterpret_cast<const float*>(ws + L.accum);
    hipLaunchKernelGGL(densify_stats_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                       views, n, tiles, acc, gate, grad_sum, count);
    return hipGetLastError();
}

// Inputs up to which a workgroup takes 256 of them, 2048 beyond: fewer leave
// the chip idle, more share fewer lines (SH 3, us of a step with 256 / 2048:
// 120k inputs 58 / 121, 250k 94 / 137, 500k 203 / 178, 2M 792 / 691). And
// workgroups from which the planes are no longer dealt out to several workgroups
// of the same inputs: below, a workgroup's chain of groups of planes is the time
// (5k inputs 34 us without, 14 with; 30k 36 / 21, 120k 58 / 53). With one scan
// launch and a thread an input: 5k 42, 30k 92, 120k 123, 500k 342, 2M 1041.
constexpr int64_t kDensifySmall = 1 << 18;
constexpr int64_t kDensifyBlocks = 1024;

hipError_t launch_densify(const DensifyDev& d, float* params, float* m, float* v, int64_t n,
                          int64_t stride, int F, const float* grad_sum, const int32_t* count,
                          const float* normals, float* out_params, float* out_m, float* out_v,
                          int64_t out_stride, uint32_t* scratch, int64_t* n_out, hipStream_t s) {
    const PlaneBuf P{params, stride}, M{m, stride}, V{v, stride};
    const PlaneBuf PO{out_params, out_stride}, MO{out_m, out_stride}, VO{out_v, out_stride};
    const int64_t groups = (F + kGroup - 1) / kGroup;
#define SGS_DENSIFY(T, PARTS, SPLIT)                                                             \
    do {                                                                                         \
        const int64_t nb = std::max<int64_t>(1, (n + T * PARTS - 1) / (T * PARTS));              \
        const int64_t py = SPLIT ? std::clamp<int64_t>(kDensifyBlocks / nb, 1, groups) : 1;      \
        hipLaunchKernelGGL((densify_count_kernel<T, PARTS>), dim3((unsigned)nb), dim3(T), 0, s, P, \
                           n, grad_sum, count, d, scratch);                                      \
        hipLaunchKernelGGL((densify_write_kernel<T, PARTS>), dim3((unsigned)nb, (unsigned)py),   \
                           dim3(T), 0, s, P, M, V, n, F, grad_sum, count, normals, d, scratch,   \
                           n_out, out_stride, PO, MO, VO);                                       \
    } while (0)
    if (n <= kDensifySmall)
        SGS_DENSIFY(256, 1, true);
    else
        SGS_DENSIFY(512, 4, false);
#undef SGS_DENSIFY
    return hipGetLastError();
}

}  // namespace sgs
