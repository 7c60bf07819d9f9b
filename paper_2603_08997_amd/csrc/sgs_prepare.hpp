// What the compositing backward needs done before it, for the launch of its own
// that a backward call makes (raster.hip) and for the loss backward of a training
// iteration (loss.hip).
#pragma once

#include "sgs_device.hpp"
#include "sgs_internal.hpp"

namespace sgs {

constexpr int kOrderSlots = 1024;

// Workgroup `block` of `blocks`, NT threads each: block 0 counts Adam's step
// (nullable) and orders the tiles by the forward's measured work, largest first
// (a counting sort in LDS: bucket counts, their exclusive scan, then every tile
// takes the next slot of its bucket), the others clear the accumulators.
// slot: kOrderSlots words of LDS, smem: NT / 64 + 1.
template <int NT>
__device__ __forceinline__ void prepare_backward(const Prepare& p, int block, int blocks,
                                                 uint32_t* slot, uint32_t* smem) {
    const int tid = threadIdx.x;
    if (block > 0) {
        for (int64_t i = (int64_t)(block - 1) * NT + tid; i < p.n4; i += (int64_t)(blocks - 1) * NT)
            p.accum[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        return;
    }
    if (p.step != nullptr && tid == 0) *p.step += 1;
    auto bucket = [&](int64_t t) {
        return (uint32_t)(kOrderSlots - 1) - min(p.cost[t], (uint32_t)(kOrderSlots - 1));
    };
    constexpr int kEach = (kOrderSlots + NT - 1) / NT;   // neighbouring slots a thread
    for (int k = tid; k < kOrderSlots; k += NT) slot[k] = 0;
    __syncthreads();
    for (int64_t t = tid; t < p.tiles; t += NT) atomicAdd(&slot[bucket(t)], 1u);
    __syncthreads();
    uint32_t c[kEach], sum = 0;
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const int at = tid * kEach + k;
        c[k] = at < kOrderSlots ? slot[at] : 0u;
        sum += c[k];
    }
    uint32_t tot;
    uint32_t first = block_excl_scan<NT>(sum, smem, &tot);
#pragma unroll
    for (int k = 0; k < kEach; ++k) {
        const int at = tid * kEach + k;
        if (at < kOrderSlots) slot[at] = first;
        first += c[k];
    }
    __syncthreads();
    for (int64_t t = tid; t < p.tiles; t += NT)
        p.order[atomicAdd(&slot[bucket(t)], 1u)] = (uint32_t)t;
}

}  // namespace sgs
