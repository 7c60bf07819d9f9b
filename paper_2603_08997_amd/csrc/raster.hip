// Front-to-back compositing (paper Sec. 3, Eqs. 4-5) over the per-tile
// depth-ordered lists, and its reverse-order adjoint.
//
// One or several wavefronts (64 lanes) per tile, each owning a part of it, SW x
// SH pixels (a launch rule on the number of tiles picks 1, 2 or 4 parts); lane l
// owns column l % SW of the part and the rows l / SW + k * 64 / SW, so every
// per-pixel load or store of the wave is a run of contiguous row segments. The
// tile's list is staged through LDS B records at a time, each wave for itself;
// while staging, each lane turns one record into the coefficients the inner
// loop needs, and a wave of a part leaves out the entries that cannot take
// part in its pixels. Every lane then walks the batch with broadcast LDS reads.
//
// The exponent of Eq. 5 is evaluated in base 2 with the opacity folded in,
// E = log2(o) + A dx^2 + B dx dy + C dy^2 (A = -a log2(e)/2, B = -b log2(e),
// C = -c log2(e)/2), so that o exp(P) = 2^E. The part that depends on dx only
// is formed once per lane and Gaussian (the lane's pixels share a column);
// each pixel then costs two fused multiply-adds. A pixel takes part when it
// lies in the overlap box (bit masks over the part's columns and rows, formed
// exactly at staging), E >= log2(alpha_min) (alpha' >= alpha_min;
// alpha_min <= alpha_max) and E <= log2(o) (P <= 0); only then is 2^E
// evaluated. Forward and backward share these functions, so their skip
// decisions agree bit for bit.
//
// The forward keeps, per pixel, only the final transmittance and the list
// position of the last blended Gaussian. The backward walks the list again
// from that position towards the front, recovering T_i = T_{i+1} / (1 -
// alpha'_i) and, per pixel, G.S = sum over channels of dL/dC times the colour
// accumulated behind the Gaussian, so no per-pixel blend list is stored. A
// Gaussian's gradient is gathered per lane as moments of dL/dP over its
// pixels, turned into the 9 parameter gradients per lane, summed over the 64
// lanes reduce-scatter style (lane 8 k ends with gradient k), and added with one
// hardware float atomic instruction over 9 lanes for that (part, Gaussian)
// pair; Gaussians that touch no pixel of the part skip both.
//
// All tiles of a launch are resident at once, so a launch lasts as long as
// its busiest SIMD. The forward records each tile's work for the backward
// (the longest prefix of the list any pixel blends), and the backward takes
// the tiles in decreasing order of it: consecutive workgroups land on
// different SIMDs, so every SIMD gets a mix of long and short tiles.
#include <algorithm>

#include "sgs_prepare.hpp"

namespace sgs {

namespace {

constexpr int kLanes = 64;

// Width of the part of a TW x TH tile that each of W waves takes: parts as
// square as they can be, which the fewest Gaussians reach (4 parts of 8x8 pixels
// against 16x4: forward 51.4 -> 46.9 us at 16 tiles, 37.0 -> 34.6 at 1200, 100
// -> 96 at 4056, backward 78.7 -> 76.8 at 1200).
constexpr int part_width(int tw, int w) { return w == 4 ? 8 : (w == 2 ? 16 : tw); }
constexpr float kNegHalfLog2e = -0.721347520444481703680f;  // -log2(e) / 2
constexpr float kNegLog2e = -1.44269504088896340736f;       // -log2(e)

// Bit q set iff the pixel origin + q (centre origin + q + 0.5) of an n-pixel
// tile span lies in the overlap box |p - centre| <= r (r an integer). With
// f = floor(centre) and t = centre - f (both exact in FP32, |centre| < 2^24),
// the first such pixel is f - r + [t > 1/2] and the last f + r - [t < 1/2]:
// the box test of the reals in integer arithmetic.
__device__ __forceinline__ uint32_t box_mask(float centre, float r, int origin, int n) {
    const float f = floorf(centre);
    const float t = centre - f;
    const int fi = (int)f, ri = (int)r;
    const int lo = fi - ri + (t > 0.5f ? 1 : 0) - origin;
    const int hi = fi + ri - (t < 0.5f ? 1 : 0) - origin;
    const int l = max(lo, 0), h = min(hi, n - 1);
    if (l > h) return 0u;
    return (0xffffffffu >> (31 - h)) & (0xffffffffu << l);
}

// The overlap box over a rectangle of TW x TH pixels as bit masks: columns in
// the low TW bits and rows above them where both fit one word (a pixel then
// takes one AND and one compare against its own two bits), columns and rows in
// a word each otherwise.
template <int TW, int TH>
struct BoxBits {
    static constexpr bool kOneWord = TW + TH <= 32;
    uint32_t c, r;   // the pixel's bits
    __device__ __forceinline__ BoxBits() : c(0), r(0) {}
    __device__ __forceinline__ BoxBits(int col, int row) {
        c = (1u << col) | (kOneWord ? 1u << ((TW + row) & 31) : 0u);
        r = kOneWord ? 0u : 1u << row;
    }
    __device__ __forceinline__ bool in(float z, float w) const {
        if constexpr (kOneWord) return (__float_as_uint(z) & c) == c;
        return (__float_as_uint(z) & c) != 0u && (__float_as_uint(w) & r) != 0u;
    }
};

// Staged record of one list entry for one wave's rectangle: geo = (u, v, A, B),
// aux = (C, log2 o, box bits). Returns whether the box holds a pixel of it.
template <int TW, int TH>
__device__ __forceinline__ bool stage_entry(const float4& r0, const float4& r1, int x0, int y0,
                                            float4& geo, float4& aux) {
    geo = make_float4(r0.x, r0.y, r0.z * kNegHalfLog2e, r0.w * kNegLog2e);
    const uint32_t c = box_mask(r0.x, r1.z, x0, TW), r = box_mask(r0.y, r1.w, y0, TH);
    const uint32_t z = BoxBits<TW, TH>::kOneWord ? c | (r << (TW & 31)) : c;
    aux = make_float4(r1.x * kNegHalfLog2e, __builtin_amdgcn_logf(r1.y), __uint_as_float(z),
                      __uint_as_float(r));
    return c != 0u && r != 0u;
}

// Whether an entry can take part in a pixel of the rectangle: its box holds
// one and, for a part of a tile (the tile lists hold no entry that fails on
// the whole tile), it can reach alpha_min there.
template <bool kPart>
__device__ __forceinline__ bool entry_reaches(bool box, const float4& r0, const float4& r1,
                                              const RasterDev& rp, int x0, int y0, int w, int h) {
    if constexpr (kPart) {
        // (the test needs a convex exponent: a, c and det = ac - b^2 > 0, det
        // by Kahan's fused form; other conics keep their box)
        const float a = r0.z, b = r0.w, c = r1.x, bb = b * b;
        const bool convex = a > 0.f && c > 0.f && fmaf(a, c, -bb) - fmaf(b, b, -bb) > 0.f;
        return box && (!convex || rect_reachable(r0.x, r0.y, a, b, c, reach_limit(r1.y, rp), r1.z,
                                                 r1.w, x0, y0, w, h));
    }
    return box;
}

// Per lane and Gaussian: the dx-only part of E.
struct LaneTerms {
    float dx, bx, base;
};

__device__ __forceinline__ LaneTerms lane_terms(const float4& geo, const float4& aux, float px) {
    LaneTerms t;
    t.dx = px - geo.x;
    t.base = fmaf(geo.z * t.dx, t.dx, aux.y);
    t.bx = geo.w * t.dx;
    return t;
}

// E at the pixel row offset dy = py - v.
__device__ __forceinline__ float exponent2(const LaneTerms& t, const float4& aux, float dy) {
    return fmaf(dy, fmaf(aux.x, dy, t.bx), t.base);
}

__device__ __forceinline__ bool takes_part(bool in_box, float e, const float4& aux, float lmin) {
    return in_box & (e >= lmin) & (e <= aux.y);
}

template <int kCtrl>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, false));
}

// One exchange step of the reduce-scatter: lanes with `hi` set keep b and
// send a, the others keep a and send b; the kept value adds what the partner
// lane (the DPP source, which differs in that bit) sent, the sum of the same
// value over both lanes.
template <int kCtrl>
__device__ __forceinline__ float rs_step(float a, float b, bool hi) {
    const float keep = hi ? b : a, send = hi ? a : b;
    return keep + dpp_f<kCtrl>(send);
}

// Reduce-scatter of a pair over rows of 16 lanes: exchanging the odd rows of a
// with the even rows of b leaves the even rows with a's and the odd rows with
// b's two terms, one add apart (row16: rows 1 apart, row32: rows 2 apart).
__device__ __forceinline__ float rs_row16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float rs_row32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sums of x[0..8] over the 64 lanes of a (fully active) wave. Returns, in
// lanes 8 v .. 8 v + 7, the total of x[v], v < 8; *t8 gets the total of x[8]
// in lane 63. The row swaps come first: a swap and an add halve a pair of
// values where a DPP exchange takes two selects and an add, so the four pairs
// and the two pairs go through the swaps and one pair is left to the selects
// (18 instructions for the eight values, 6 for the ninth).
__device__ __forceinline__ float wave_sum9_scatter(const float (&x)[9], int lane, float* t8) {
    // row r = 2 h + g of the wave ends with values 2 r and 2 r + 1
    float y[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) y[k] = rs_row16(x[(k & 1) + 4 * (k >> 1)], x[(k & 1) + 4 * (k >> 1) + 2]);
    const float z0 = rs_row32(y[0], y[2]), z1 = rs_row32(y[1], y[3]);
    float w = rs_step<0x128>(z0, z1, (lane & 8) != 0);   // row rotate 8: the other half-row
    w += dpp_f<0xb1>(w);    // xor 1
    w += dpp_f<0x4e>(w);    // xor 2
    w += dpp_f<0x141>(w);   // the other quad of the half-row
    float t = wave_sum_to_lane63(x[8]);
    // (both sums formed here: sunk into the branch that adds them, their last
    // steps lose the fused DPP form)
    asm volatile("" : "+v"(w), "+v"(t));
    *t8 = t;
    return w;
}

__device__ __forceinline__ int view_of_tile(const Views* views, int tile) {
    int vi = 0;
    while (vi + 1 < views->n && tile >= views->v[vi + 1].tile_offset) ++vi;
    return vi;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, d, 64));
    return v;
}

__device__ __forceinline__ uint32_t wave_add_u32(uint32_t v) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) v += (uint32_t)__shfl_xor((int)v, d, 64);
    return v;
}

// Where the tiles' work is summed into counters[kBlended], [kEvaluated] (uint64)
// and [kUsed] (uint32). An addition to one address takes 8 ns and three of them
// a tile, so a few tiles add their own (16 tiles: nothing to be seen, against
// the 4.6 us of a launch; 2170 tiles: +27 us); otherwise one more block of the
// resuming launch does it, and resumed tiles add what they did there; a launch of
// its own where there is no second pass.
enum class SumBy { kTile, kRedo, kLaunch };
constexpr int64_t kTileSums = 128;

__device__ __forceinline__ void add_work(uint32_t* counters, unsigned long long blended,
                                         unsigned long long evaluated, uint32_t used) {
    unsigned long long* sum = reinterpret_cast<unsigned long long*>(counters + kBlended);
    atomicAdd(&sum[0], blended);
    atomicAdd(&sum[1], evaluated);
    atomicAdd(&counters[kUsed], used);
}

// Sums of {blended, evaluated, used} over the tiles by one workgroup, added to
// the counters (kAdd) or written to them.
template <int NT, bool kAdd>
__device__ __forceinline__ void sum_tiles(const uint4* __restrict__ tile_stats, int64_t tiles,
                                          uint32_t* counters) {
    __shared__ unsigned long long s_sum[3][NT / 64];
    unsigned long long b = 0, e = 0, u = 0;
#pragma unroll 4
    for (int64_t t = threadIdx.x; t < tiles; t += NT) {
        const uint4 v = tile_stats[t];
        b += v.x;
        e += v.y;
        u += v.z;
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        b += __shfl_xor(b, d, 64);
        e += __shfl_xor(e, d, 64);
        u += __shfl_xor(u, d, 64);
    }
    const int w = threadIdx.x / 64;
    if (threadIdx.x % 64 == 0) {
        s_sum[0][w] = b;
        s_sum[1][w] = e;
        s_sum[2][w] = u;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        b = e = u = 0;
        for (int k = 0; k < NT / 64; ++k) {
            b += s_sum[0][k];
            e += s_sum[1][k];
            u += s_sum[2][k];
        }
        if (kAdd) {
            add_work(counters, b, e, (uint32_t)u);
        } else {
            reinterpret_cast<unsigned long long*>(counters + kBlended)[0] = b;
            reinterpret_cast<unsigned long long*>(counters + kEvaluated)[0] = e;
            counters[kUsed] = (uint32_t)u;
        }
    }
}

// Forward of one tile by W waves: each composites its SW x SH pixels
// front to back over the tile's list in batches of B entries (records
// gathered and staged in LDS per batch, each wave for itself) and stops when
// every pixel of the part has terminated. A wave leaves the entries that
// cannot take part in its pixels out at staging.
template <int TW, int TH, int B, int W>
__global__ void __launch_bounds__(kLanes * W) raster_forward_kernel(
    const Views* __restrict__ views, RasterDev rp, const uint32_t* __restrict__ tile_ranges,
    const uint32_t* __restrict__ tile_entry, const float4* __restrict__ rec,
    float* __restrict__ out_rgb, float* __restrict__ t_final, uint32_t* __restrict__ n_last,
    uint4* __restrict__ tile_stats, uint32_t* __restrict__ tile_cost, uint32_t entries,
    uint32_t* __restrict__ tile_state, uint32_t* __restrict__ tile_resume,
    uint32_t* __restrict__ sup_redo, uint32_t* __restrict__ counters, SumBy sum_by, bool redo) {
    constexpr int SW = part_width(TW, W);     // a wave's part of the tile
    constexpr int SH = TW * TH / (W * SW);
    constexpr int PIX = SW * SH / kLanes;
    constexpr int RS = kLanes / SW;           // row step between a lane's pixels
    static_assert(B % 32 == 0 && B >= 32 && B <= 256, "batch size");
    static_assert(PIX >= 1 && PIX * kLanes * W == TW * TH && TW % SW == 0, "whole waves");
    // (the last entries: padding and the read ahead past it)
    __shared__ float4 s_geo[W][B + 4];
    __shared__ float4 s_aux[W][B + 4];
    __shared__ float4 s_col[W][B + 4];   // r, g, b, list position (bits)
    __shared__ uint32_t s_tile[W][4];

    const int tile = blockIdx.x;
    if (redo && tile == views->total_tiles) {   // (one block more with SumBy::kRedo)
        sum_tiles<kLanes * W, true>(tile_stats, tile, counters);
        return;
    }
    // the second pass goes on with the tiles the first left incomplete
    if (redo && tile_state[tile] != kTileIncomplete) return;
    const ViewDev& V = views->v[view_of_tile(views, tile)];
    const int local = tile - V.tile_offset;
    const int tx = local % V.tiles_x, ty = local / V.tiles_x;
    const int wv = W > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes) : 0;
    const int tid = threadIdx.x % kLanes;
    const int col = tid % SW, row0 = tid / SW;
    const uint32_t start = tile_ranges[2 * tile], end = tile_ranges[2 * tile + 1];
    const float lmin = rp.log2_alpha_min, amax = rp.alpha_max, tmin = rp.t_min;
    const int px0 = tx * TW + wv % (TW / SW) * SW, py0 = ty * TH + wv / (TW / SW) * SH;
    float4* geo = s_geo[wv];
    float4* aux = s_aux[wv];
    float4* rgb = s_col[wv];

    const float px = (float)(px0 + col) + 0.5f;
    const int64_t plane = (int64_t)V.width * V.height;
    float* img = out_rgb + 3 * V.px_offset;
    // a pixel outside the view or stopped has py = NaN: its E is NaN and takes
    // part in nothing
    float py[PIX], T[PIX], C0[PIX], C1[PIX], C2[PIX];
    BoxBits<SW, SH> bits[PIX];
    uint32_t last[PIX];
    // the second pass resumes each pixel where the first stopped, at the end
    // of the tile's list prefix (which begins its whole list): transmittance,
    // colour sums (stored without the background), last blended position and
    // whether the pixel is still live (bit 31 of that position)
#pragma unroll
    for (int k = 0; k < PIX; ++k) {
        const int y = py0 + row0 + RS * k;
        py[k] = __builtin_nanf("");
        bits[k] = BoxBits<SW, SH>(col, row0 + RS * k);
        T[k] = 1.f;
        C0[k] = C1[k] = C2[k] = 0.f;
        last[k] = 0;
        if (px0 + col < V.width && y < V.height) {
            py[k] = (float)y + 0.5f;
            if (redo) {
                const int64_t pix = (int64_t)y * V.width + px0 + col;
                T[k] = t_final[V.px_offset + pix];
                C0[k] = img[pix];
                C1[k] = img[plane + pix];
                C2[k] = img[2 * plane + pix];
                const uint32_t nl = n_last[V.px_offset + pix];
                last[k] = nl & 0x7fffffffu;
                if (!(nl >> 31)) py[k] = __builtin_nanf("");
            }
        }
    }
    const uint32_t begin = redo ? min(start + tile_resume[tile], end) : start;
    // examined entries: a pixel that stops at list position p examined p of
    // them (of this pass: p - resume), one that never stops the whole list
    const uint32_t skipped = begin - start;
    uint32_t n_blend = 0;
    uint32_t stop_pos[PIX];
#pragma unroll
    for (int k = 0; k < PIX; ++k) stop_pos[k] = 0;
    auto any_live = [&]() {
        uint64_t l = 0;
#pragma unroll
        for (int k = 0; k < PIX; ++k) l |= ballot(py[k] == py[k]);
        return l != 0;
    };
    bool alive = any_live();   // uniform
    // Software pipeline over the batches: the entry indices are loaded two
    // batches ahead and (one entry per lane, B <= 64) the records one batch
    // ahead, so the gathers of a batch run while the previous one composites
    // (a tile whose pixels stay live walks its whole list, and its time is
    // otherwise a chain of two memory round trips per batch).
    constexpr int NE = (B + kLanes - 1) / kLanes;   // entries per lane per batch
    auto entry_at = [&](uint32_t b, int i) -> uint32_t {
        const uint32_t k = b + (uint32_t)(i * kLanes + tid);
        return k < end ? min(tile_entry[k], entries - 1u) : 0u;
    };
    uint32_t e_cur[NE], e_next[NE];
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        e_cur[i] = entry_at(begin, i);
        e_next[i] = entry_at(begin + (uint32_t)B, i);
    }
    float4 q0, q1, q2;   // records of the lane's entry of the current batch (NE == 1)
    if constexpr (NE == 1) {
        q0 = rec[3 * (int64_t)e_cur[0]];
        q1 = rec[3 * (int64_t)e_cur[0] + 1];
        q2 = rec[3 * (int64_t)e_cur[0] + 2];
    }
    for (uint32_t b0 = begin; b0 < end && alive; b0 += (uint32_t)B) {
        wave_lds_sync();
        const int in_batch = (int)min((uint32_t)B, end - b0);
        int cnt = 0;   // staged entries
        auto stage = [&](int j, const float4& r0, const float4& r1, const float4& r2) {
            float4 g, x;
            const bool box = stage_entry<SW, SH>(r0, r1, px0, py0, g, x);
            const bool keep =
                j < in_batch && entry_reaches<(W > 1)>(box, r0, r1, rp, px0, py0,
                                                       min(SW, V.width - px0),
                                                       min(SH, V.height - py0));
            const uint64_t m = ballot(keep);
            if (keep) {
                const int o = cnt + popc64(m & lanemask_lt());
                geo[o] = g;
                aux[o] = x;
                rgb[o] = make_float4(r2.x, r2.y, r2.z,
                                     __uint_as_float(b0 - start + (uint32_t)j + 1u));
            }
            cnt += popc64(m);
        };
        if constexpr (NE == 1) {
            stage(tid, q0, q1, q2);
            const uint32_t e2 = entry_at(b0 + 2u * (uint32_t)B, 0);
            q0 = rec[3 * (int64_t)e_next[0]];
            q1 = rec[3 * (int64_t)e_next[0] + 1];
            q2 = rec[3 * (int64_t)e_next[0] + 2];
            e_next[0] = e2;
        } else {
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int64_t e = e_cur[i];
                stage(i * kLanes + tid, rec[3 * e], rec[3 * e + 1], rec[3 * e + 2]);
                e_cur[i] = e_next[i];
                e_next[i] = entry_at(b0 + 2u * (uint32_t)B, i);
            }
        }
        if (cnt == 0) continue;
        // the batch padded to whole groups with entries outside every box
        constexpr int U = 4;
        if (tid < U - 1) {
            geo[cnt + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
            aux[cnt + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
            rgb[cnt + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        wave_lds_sync();
        // the next entry's LDS reads are issued before the current entry is
        // processed, so a wave running alone does not wait on them
        float4 Gn = geo[0], Xn = aux[0], Cn = rgb[0];
        for (int j = 0; j < cnt && alive; j += U) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float4 G = Gn, X = Xn, c = Cn;
                Gn = geo[j + u + 1];
                Xn = aux[j + u + 1];
                Cn = rgb[j + u + 1];
                const LaneTerms L = lane_terms(G, X, px);
#pragma unroll
                for (int k = 0; k < PIX; ++k) {
                    const float e = exponent2(L, X, py[k] - G.y);
                    const bool take = takes_part(bits[k].in(X.z, X.w), e, X, lmin);
                    if (take) {
                        // a pixel whose transmittance would fall below t_min stops
                        // before this Gaussian; otherwise the Gaussian is blended
                        const float alpha = __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(e), 0.f, amax);
                        const float wgt = alpha * T[k];
                        const float tn = T[k] - wgt;
                        const bool stop = tn < tmin;
                        py[k] = stop ? __builtin_nanf("") : py[k];
                        stop_pos[k] = stop ? __float_as_uint(c.w) : stop_pos[k];
                        if (!stop) {
                            C0[k] = fmaf(c.x, wgt, C0[k]);
                            C1[k] = fmaf(c.y, wgt, C1[k]);
                            C2[k] = fmaf(c.z, wgt, C2[k]);
                            T[k] = tn;
                            last[k] = __float_as_uint(c.w);
                            ++n_blend;
                        }
                    }
                }
            }
            alive = any_live();
        }
    }
    uint32_t n_eval = 0;
#pragma unroll
    for (int k = 0; k < PIX; ++k)
        n_eval += stop_pos[k] != 0u ? stop_pos[k] - skipped : (py[k] == py[k] ? end - begin : 0u);

    // the backward walks every pixel's list up to its last blended Gaussian:
    // the tile's longest such prefix is its work (where its counters are summed
    // up: SumBy)
    uint32_t my_last = 0;
#pragma unroll
    for (int k = 0; k < PIX; ++k) my_last = max(my_last, last[k]);
    uint32_t tile_last = wave_max_u32(my_last);
    uint32_t nb = wave_add_u32(n_blend), ne2 = wave_add_u32(n_eval);
    bool tile_live = alive;
    if constexpr (W > 1) {
        if (tid == 0) {
            s_tile[wv][0] = tile_last;
            s_tile[wv][1] = nb;
            s_tile[wv][2] = ne2;
            s_tile[wv][3] = tile_live ? 1u : 0u;
        }
        __syncthreads();
        tile_last = nb = ne2 = 0;
        uint32_t al = 0;
#pragma unroll
        for (int k = 0; k < W; ++k) {
            tile_last = max(tile_last, s_tile[k][0]);
            nb += s_tile[k][1];
            ne2 += s_tile[k][2];
            al |= s_tile[k][3];
        }
        tile_live = al != 0u;
    }
    // a pixel still live at the end of a list cut by the split prefix: the
    // tile is resumed by the second pass over its whole list, after the whole
    // lists of its super-tile have been split; until then its pixels hold the
    // state to resume from
    const bool suspend =
        !redo && tile_state != nullptr && tile_live && tile_state[tile] == kTileTruncated;
    const int x = px0 + col;
#pragma unroll
    for (int k = 0; k < PIX; ++k) {
        const int y = py0 + row0 + RS * k;
        if (x >= V.width || y >= V.height) continue;
        const int64_t pix = (int64_t)y * V.width + x;
        const bool lk = py[k] == py[k];
        img[pix] = suspend ? C0[k] : fmaf(T[k], rp.bg[0], C0[k]);
        img[plane + pix] = suspend ? C1[k] : fmaf(T[k], rp.bg[1], C1[k]);
        img[2 * plane + pix] = suspend ? C2[k] : fmaf(T[k], rp.bg[2], C2[k]);
        t_final[V.px_offset + pix] = T[k];
        n_last[V.px_offset + pix] = suspend && lk ? last[k] | 0x80000000u : last[k];
    }
    if (W > 1) __syncthreads();   // every wave has read the tile's state
    if (threadIdx.x == 0) {
        const uint32_t before = redo ? tile_cost[tile] : 0u;
        if (sum_by == SumBy::kTile || (redo && sum_by == SumBy::kRedo)) {   // uniform
            add_work(counters, nb, ne2, tile_last - before);
        } else {
            const uint4 first = redo ? tile_stats[tile] : make_uint4(0u, 0u, 0u, 0u);
            tile_stats[tile] = make_uint4(nb + first.x, ne2 + first.y, tile_last, 0u);
        }
        tile_cost[tile] = tile_last;
        if (redo) {
            tile_state[tile] = kTileWhole;
        } else if (suspend) {
            const int S = rp.super_tile;
            tile_state[tile] = kTileIncomplete;
            tile_resume[tile] = end - start;
            sup_redo[V.sup_offset + (ty / S) * V.sup_x + tx / S] = 1u;
            counters[kRedo] = 1u;
        }
    }
}

// The sums alone, where the compositing launches cannot take them (also clears).
constexpr int kStatThreads = 1024;
__global__ void __launch_bounds__(kStatThreads) sum_tile_stats_kernel(
    const uint4* __restrict__ tile_stats, int64_t tiles, uint32_t* __restrict__ counters) {
    sum_tiles<kStatThreads, false>(tile_stats, tiles, counters);
}

// At most 72 VGPRs (batches of 64), so that 7 waves fit on each SIMD: the
// 6700 tiles of a 1600x1060 view (16x16 tiles) then all run at once on the
// 1024 SIMDs of the chip instead of leaving a second round for the last tiles.
//
// Gradient of one (tile, Gaussian) pair from per-lane moments of dL/dP over
// the lane's pixels (dP = dL/dP, dy per pixel, dx per lane): with
// P = -(a dx^2 + c dy^2)/2 - b dx dy, dx = px - u, dy = py - v,
//   dL/du = a M1 + b M2,  dL/dv = b M1 + c M2,  dL/da = -M3/2,
//   dL/db = -M4,  dL/dc = -M5/2,  dL/do = M6 / o  (unclamped alpha' = o e^P),
// M1 = sum dP dx, M2 = sum dP dy, M3 = sum dP dx^2, M4 = sum dP dx dy,
// M5 = sum dP dy^2, M6 = sum dP.
// Waves per SIMD the LDS of a batch allows (64 B per staged entry).
constexpr int backward_waves(int batch) { return batch <= 64 ? 7 : (batch == 128 ? 5 : 3); }

template <int TW, int TH, int B, int W>
__global__ void __launch_bounds__(kLanes, backward_waves(B)) raster_backward_kernel(
    const Views* __restrict__ views, RasterDev rp, const uint32_t* __restrict__ tile_ranges,
    const uint32_t* __restrict__ tile_entry, const float4* __restrict__ rec,
    const float* __restrict__ t_final, const uint32_t* __restrict__ n_last,
    const float* __restrict__ dl_drgb, const int32_t* __restrict__ gate,
    float* __restrict__ accum, const uint32_t* __restrict__ order, int total_tiles,
    uint32_t entries) {
    constexpr int SW = part_width(TW, W);   // a wave's part of the tile
    constexpr int SH = TW * TH / (W * SW);
    constexpr int PIX = SW * SH / kLanes;
    constexpr int RS = kLanes / SW;
    static_assert(PIX >= 1 && PIX * kLanes * W == TW * TH && TW % SW == 0, "whole waves");
    __shared__ float4 s_geo[B + 1];
    __shared__ float4 s_aux[B + 1];
    __shared__ float4 s_col[B + 1];   // r, g, b, entry (bits)
    __shared__ float4 s_con[B];       // a, b, c, 1 / o
    __shared__ uint32_t s_rel[B + 1];
    if (gate_closed(gate)) return;

    // the W parts of a tile are consecutive workgroups
    const int tile = (int)order[blockIdx.x / W];
    if (tile >= total_tiles) return;   // order is a permutation of the tiles
    const ViewDev& V = views->v[view_of_tile(views, tile)];
    const int local = tile - V.tile_offset;
    const int tx = local % V.tiles_x, ty = local / V.tiles_x;
    const int tid = threadIdx.x;
    const int col = tid % SW, row0 = tid / SW;
    const float lmin = rp.log2_alpha_min, amax = rp.alpha_max;

    const int64_t plane = (int64_t)V.width * V.height;
    const float* dl = dl_drgb + 3 * V.px_offset;
    const int wv = (int)(blockIdx.x % W);
    const int px0 = tx * TW + wv % (TW / SW) * SW, py0 = ty * TH + wv / (TW / SW) * SH;
    const int x = px0 + col;
    const float px = (float)x + 0.5f;
    float py[PIX], T[PIX], G0[PIX], G1[PIX], G2[PIX], GS[PIX];
    BoxBits<SW, SH> bits[PIX];
    uint32_t last[PIX];
    uint32_t my_max = 0;
#pragma unroll
    for (int k = 0; k < PIX; ++k) {
        const int y = py0 + row0 + RS * k;
        py[k] = (float)y + 0.5f;
        bits[k] = BoxBits<SW, SH>(col, row0 + RS * k);
        T[k] = 1.f;
        G0[k] = G1[k] = G2[k] = 0.f;
        last[k] = 0;
        if (x < V.width && y < V.height) {
            const int64_t pix = (int64_t)y * V.width + x;
            G0[k] = dl[pix];
            G1[k] = dl[plane + pix];
            G2[k] = dl[2 * plane + pix];
            T[k] = t_final[V.px_offset + pix];
            last[k] = n_last[V.px_offset + pix];
        }
        // dL/dC . (colour composited behind the current Gaussian), background included
        GS[k] = fmaf(G0[k], rp.bg[0], fmaf(G1[k], rp.bg[1], G2[k] * rp.bg[2])) * T[k];
        my_max = max(my_max, last[k]);
    }
    const uint32_t start = tile_ranges[2 * tile], end = tile_ranges[2 * tile + 1];
    const uint32_t stop =
        min((uint32_t)__builtin_amdgcn_readfirstlane((int)wave_max_u32(my_max)), end - start);

    // the lane that adds gradient v of a pair: 8 v for v < 8, 63 for the ninth
    const int slot = tid == 63 ? 8 : tid / 8;
    const bool adds = tid == 63 || tid % 8 == 0;

    // the list from the last blended position towards the front, B entries
    // at a time (list positions [b0, b_end), staged last first)
    for (uint32_t b_end = stop; b_end > 0u;) {
        const uint32_t b0 = b_end > (uint32_t)B ? b_end - (uint32_t)B : 0u;
        const int in_batch = (int)(b_end - b0);
        int cnt = 0;   // staged entries
        __syncthreads();
        for (int k0 = 0; k0 < in_batch; k0 += kLanes) {
            const int k = k0 + tid;
            const uint32_t p = b_end - 1u - (uint32_t)min(k, in_batch - 1);   // list position
            const uint32_t e = min(tile_entry[start + p], entries - 1u);
            const float4 r0 = rec[3 * (int64_t)e], r1 = rec[3 * (int64_t)e + 1],
                         r2 = rec[3 * (int64_t)e + 2];
            float4 g, xm;
            const bool box = stage_entry<SW, SH>(r0, r1, px0, py0, g, xm);
            const bool keep =
                k < in_batch && entry_reaches<(W > 1)>(box, r0, r1, rp, px0, py0,
                                                       min(SW, V.width - px0),
                                                       min(SH, V.height - py0));
            const uint64_t m = ballot(keep);
            if (keep) {
                const int o = cnt + popc64(m & lanemask_lt());
                s_geo[o] = g;
                s_aux[o] = xm;
                s_col[o] = make_float4(r2.x, r2.y, r2.z, __uint_as_float(e));
                // 1/o capped at FLT_MAX: an opacity that underflowed to 0 can only
                // take part with alpha' = 0 (alpha_min = 0), where M6 = 0
                s_con[o] = make_float4(r0.z, r0.w, r1.x, fminf(1.f / r1.y, 3.402823466e38f));
                s_rel[o] = p;
            }
            cnt += popc64(m);
        }
        __syncthreads();
        // With few waves on a SIMD (parts) the next entry's LDS reads are
        // issued before the current entry is processed (the last one reads
        // ahead into the spare element); with one wave per tile the other
        // waves cover them, and the registers are worth more.
        constexpr bool kAhead = W > 1;
        uint32_t rel_n;
        float4 Gn, Xn, Cn;
        auto fetch = [&](int j) {
            rel_n = s_rel[j];
            Gn = s_geo[j];
            Xn = s_aux[j];
            Cn = s_col[j];
        };
        if (kAhead) fetch(0);
        for (int j = 0; j < cnt; ++j) {
            if (!kAhead) fetch(j);
            const uint32_t rel = rel_n;   // list position
            const float4 G = Gn, X = Xn, c = Cn;
            if (kAhead) fetch(j + 1);
            // read once per Gaussian with the coefficients (the compiler would
            // otherwise re-read it inside each pixel's branch)
            if (!kAhead) asm volatile("" ::"v"(c.x), "v"(c.y), "v"(c.z));
            const LaneTerms L = lane_terms(G, X, px);
            // -0 is the additive identity for every float, so the first
            // accumulation into each sum folds away
            float sdp = -0.f, sdy = -0.f, sdy2 = -0.f, d_r = -0.f, d_g = -0.f, d_bl = -0.f;
            bool contrib = false;
#pragma unroll
            for (int k = 0; k < PIX; ++k) {
                const float dy = py[k] - G.y;
                const float e = exponent2(L, X, dy);
                if ((rel < last[k]) & takes_part(bits[k].in(X.z, X.w), e, X, lmin)) {
                    const float raw = __builtin_amdgcn_exp2f(e);
                    const bool clamped = raw > amax;
                    const float alpha = __builtin_amdgcn_fmed3f(raw, 0.f, amax);
                    // 1 - alpha' >= 1 - alpha_max > 0: one hardware reciprocal
                    // (1 ulp) serves the transmittance recovery and dC/dalpha'
                    const float inv_om = __builtin_amdgcn_rcpf(1.f - alpha);
                    const float Ti = T[k] * inv_om;
                    const float w = alpha * Ti;
                    d_r = fmaf(G0[k], w, d_r);
                    d_g = fmaf(G1[k], w, d_g);
                    d_bl = fmaf(G2[k], w, d_bl);
                    // dL/dalpha' = T_i (dL/dC . c_i) - (dL/dC . S_i) / (1 - alpha'_i)
                    const float gc = fmaf(G0[k], c.x, fmaf(G1[k], c.y, G2[k] * c.z));
                    const float d_alpha = fmaf(Ti, gc, -(inv_om * GS[k]));
                    GS[k] = fmaf(w, gc, GS[k]);
                    T[k] = Ti;
                    // alpha' = o exp(P) unless clamped at alpha_max (then it
                    // depends on neither o nor the geometry); dalpha'/dP = alpha'
                    const float dP = clamped ? 0.f : d_alpha * alpha;
                    sdp += dP;
                    const float t = dP * dy;
                    sdy += t;
                    sdy2 = fmaf(t, dy, sdy2);
                    contrib = true;
                }
            }
            if (ballot(contrib) == 0) continue;
            // per-lane parameter gradients (the moments scaled by the
            // Gaussian's a, b, c, 1/o), summed over the wave reduce-scatter
            // style: lane 8 k ends with the total of gradient k < 8, lane 63
            // with that of gradient 8; one atomic instruction adds all 9
            const float4 Q = s_con[j];
            const float m1 = L.dx * sdp;
            float x[9];
            x[0] = fmaf(Q.x, m1, Q.y * sdy);   // dL/du
            x[1] = fmaf(Q.y, m1, Q.z * sdy);   // dL/dv
            x[2] = (-0.5f * L.dx) * m1;        // dL/da
            x[3] = -(L.dx * sdy);              // dL/db
            x[4] = -0.5f * sdy2;               // dL/dc
            x[5] = Q.w * sdp;                  // dL/do
            x[6] = d_r;
            x[7] = d_g;
            x[8] = d_bl;
            float t8;
            const float t = wave_sum9_scatter(x, tid, &t8);
            if (adds)
                unsafeAtomicAdd(accum + (int64_t)kAccumFloats *
                                            __float_as_uint(kAhead ? c.w : s_col[j].w) + slot,
                                slot == 8 ? t8 : t);
        }
        b_end = b0;
    }
}

// What the compositing backward needs done before it, in one launch: the call's
// views stored (nullable) and prepare_backward, on a grid sized for the machine
// (a closed gate then costs a launch of a few hundred blocks). As launches of
// their own the order took 9 us at 6700 tiles, the count and the views 4.6 us each.
constexpr int kPrepareThreads = 1024;
constexpr int64_t kPrepareBlocks = 512;
__global__ void __launch_bounds__(kPrepareThreads) prepare_backward_kernel(
    Views v, Views* __restrict__ dst, const int32_t* __restrict__ gate, Prepare p) {
    __shared__ uint32_t slot[kOrderSlots];
    __shared__ uint32_t smem[kPrepareThreads / 64 + 1];
    if (blockIdx.x == 0 && dst != nullptr) store_views(v, nullptr, 0, nullptr, dst);
    if (gate_closed(gate)) return;
    prepare_backward<kPrepareThreads>(p, (int)blockIdx.x, (int)gridDim.x, slot, smem);
}

}  // namespace

// Waves per tile. A wave's time is its instruction count (a wave alone on a
// SIMD issues one instruction every 4 cycles), so a launch with fewer waves
// than the chip's 1024 SIMDs hold ends with its longest tile, and cutting a
// tile into parts shortens exactly that; parts also drop the entries that miss
// them. 8x8 tiles have one pixel per lane already.
//
// Forward: parts win at every size, the finer ones until the per-part work
// (LDS broadcasts, 24 cycles an entry and wave) catches up. us for 1 / 2 / 4
// waves: 16 tiles 74 / 45 / 27 (one pass), 1200 tiles 89 / 55 / 35, 2170 tiles
// 124 / 73 / 58, 4056 tiles 149 / 105 / 96, 6700 tiles 167 / 135 / 137 (many
// Gaussians a pixel: 2 x 74 / 68), 28000 tiles 746 / 562 / 570.
//
// Backward: each part repeats the wave reduction and the atomic of a pair, so
// parts pay only while SIMDs would idle: 16 tiles 68 / 42 / 29, 1200 tiles
// 135 / 88 / 75, 2170 tiles 188 / 131 / 144, 4056 tiles 228 / 222 / 249, 6700
// tiles 284 / 290 / 403, 28000 tiles 910 / 1177 / 1704. Gaussians that cover much
// of a tile have more pairs with every part: 1000 of a third of the image take 80 /
// 114 with 2 / 4 waves at 1200 tiles, 85 / 112 with 1 / 2 at 2170 and 131 / 202 at
// 4056, where their forward gains 40 to 70 from its parts; where between 3000 and
// 5120 tiles one wave or two are better depends on the view (4056 tiles, 1M small
// Gaussians: 214 / 238 in one, 244 / 211 in another).
constexpr int64_t kForwardFine = 5120;    // tiles up to which the forward takes 4 waves, else 2
constexpr int64_t kBackwardFine = 1536;   // tiles up to which the backward takes 4 waves
constexpr int64_t kBackwardHalf = 5120;   // ... 2 waves, else 1
TileWaves tile_waves(int tile_w, int64_t tiles) {
    if (tile_w == 8) return {1, 1};
    return {tiles <= kForwardFine ? 4 : 2,
            tiles <= kBackwardFine ? 4 : (tiles <= kBackwardHalf ? 2 : 1)};
}

// Kernel instantiations: tile shapes 16x16, 8x8, 32x8; the batches 32, 64,
// 128, 256 the raster parameters accept where one wave takes a tile, batches
// of 64 in parts (us of the forward with 32 / 64 / 128 / 256: 2170 tiles 86 / 77 /
// 80 / 105, 4056 131 / 116 / 124 / 177, 6700 168 / 155 / 160 / 214: every wave
// holds a batch of its own).
#define SGS_RASTER_BATCHES(KERNEL, TW, TH, ...)                                       \
    do {                                                                             \
        if (rp.batch == 32) SGS_LAUNCH((KERNEL<TW, TH, 32, 1>), 1, __VA_ARGS__);       \
        else if (rp.batch == 128) SGS_LAUNCH((KERNEL<TW, TH, 128, 1>), 1, __VA_ARGS__); \
        else if (rp.batch == 256) SGS_LAUNCH((KERNEL<TW, TH, 256, 1>), 1, __VA_ARGS__); \
        else SGS_LAUNCH((KERNEL<TW, TH, 64, 1>), 1, __VA_ARGS__);                      \
    } while (0)
#define SGS_RASTER_PARTS(KERNEL, W, ...)                                             \
    do {                                                                             \
        if (rp.tile_w == 16) SGS_LAUNCH((KERNEL<16, 16, 64, W>), W, __VA_ARGS__);      \
        else SGS_LAUNCH((KERNEL<32, 8, 64, W>), W, __VA_ARGS__);                       \
    } while (0)

hipError_t launch_rasterize(const RasterDev& rp, const Layout& L, char* ws, float* out_rgb,
                            hipStream_t s) {
    if (L.total_tiles == 0) return hipSuccess;
    const Views* views = reinterpret_cast<const Views*>(ws + L.views);
    const uint32_t* ranges = reinterpret_cast<const uint32_t*>(ws + L.tile_ranges);
    const uint32_t* entry = reinterpret_cast<const uint32_t*>(ws + L.tile_entry);
    const float4* rec = reinterpret_cast<const float4*>(ws + L.records);
    float* tf = reinterpret_cast<float*>(ws + L.t_final);
    uint32_t* nl = reinterpret_cast<uint32_t*>(ws + L.n_last);
    uint32_t* cnt = reinterpret_cast<uint32_t*>(ws + L.counters);
    uint32_t* cost = reinterpret_cast<uint32_t*>(ws + L.tile_cost);
    uint4* stats = reinterpret_cast<uint4*>(ws + L.tile_stats);
    const uint32_t entries = (uint32_t)std::max<int64_t>(1, L.entries);
    // (no second pass where no list can be cut)
    uint32_t* state = lists_cut(rp, L) ? reinterpret_cast<uint32_t*>(ws + L.tile_state) : nullptr;
    uint32_t* sup_redo = reinterpret_cast<uint32_t*>(ws + L.sup_redo);
    uint32_t* resume = reinterpret_cast<uint32_t*>(ws + L.tile_resume);
    // (the sum of the used entries stays below the capacity, below 2^31)
    const SumBy sum_by = L.total_tiles <= kTileSums ? SumBy::kTile
                         : state != nullptr         ? SumBy::kRedo
                                                    : SumBy::kLaunch;
    // the waves of a tile are one workgroup
#define SGS_LAUNCH(K, W, ...) \
    hipLaunchKernelGGL(K, dim3(blocks), dim3(kLanes * W), 0, s, __VA_ARGS__)
    const int waves = tile_waves(rp.tile_w, L.total_tiles).forward;
    auto composite = [&](bool redo) {
        const unsigned blocks =
            (unsigned)L.total_tiles + (redo && sum_by == SumBy::kRedo ? 1u : 0u);
        if (waves == 1)
            SGS_RASTER_BATCHES(raster_forward_kernel, 8, 8, views, rp, ranges, entry, rec, out_rgb,
                               tf, nl, stats, cost, entries, state, resume, sup_redo, cnt,
                               sum_by, redo);
        else if (waves == 4)
            SGS_RASTER_PARTS(raster_forward_kernel, 4, views, rp, ranges, entry, rec, out_rgb, tf,
                              nl, stats, cost, entries, state, resume, sup_redo, cnt, sum_by, redo);
        else
            SGS_RASTER_PARTS(raster_forward_kernel, 2, views, rp, ranges, entry, rec, out_rgb, tf,
                              nl, stats, cost, entries, state, resume, sup_redo, cnt, sum_by, redo);
        return hipGetLastError();
    };
    if (hipError_t err = composite(false); err != hipSuccess) return err;
    if (state != nullptr) {
        // tiles whose list prefix ran out with live pixels: the whole lists of
        // their super-tiles, then their compositing resumed
        if (hipError_t err = launch_split_rest(rp, L, ws, s); err != hipSuccess) return err;
        if (hipError_t err = composite(true); err != hipSuccess) return err;
    }
    if (sum_by == SumBy::kLaunch)
        hipLaunchKernelGGL(sum_tile_stats_kernel, dim3(1), dim3(kStatThreads), 0, s, stats,
                           L.total_tiles, cnt);
    return hipGetLastError();
#undef SGS_LAUNCH
}

Prepare backward_preparation(const Layout& L, char* ws, int32_t* step) {
    return {step,
            reinterpret_cast<float4*>(ws + L.accum),
            L.entries * kAccumFloats / 4,
            reinterpret_cast<const uint32_t*>(ws + L.tile_cost),
            L.entries > 0 ? L.total_tiles : 0,
            reinterpret_cast<uint32_t*>(ws + L.tile_order)};
}

hipError_t launch_rasterize_backward(const RasterDev& rp, const Layout& L, char* ws,
                                     const float* dl_drgb, const int32_t* gate, hipStream_t s,
                                     const Views* store, int32_t* step, bool prepared) {
    const Prepare prep = backward_preparation(L, ws, step);
    if (!prepared) {
        const int64_t clear = (prep.n4 + kPrepareThreads - 1) / kPrepareThreads;
        hipLaunchKernelGGL(prepare_backward_kernel,
                           dim3((unsigned)(1 + std::min<int64_t>(clear, kPrepareBlocks))),
                           dim3(kPrepareThreads), 0, s, store != nullptr ? *store : Views{},
                           store != nullptr ? reinterpret_cast<Views*>(ws + L.views) : nullptr,
                           gate, prep);
    }
    float* acc = reinterpret_cast<float*>(ws + L.accum);
    const uint32_t* order = prep.order;
    if (L.total_tiles == 0 || L.entries == 0) return hipGetLastError();
    const Views* views = reinterpret_cast<const Views*>(ws + L.views);
    const uint32_t* ranges = reinterpret_cast<const uint32_t*>(ws + L.tile_ranges);
    const uint32_t* entry = reinterpret_cast<const uint32_t*>(ws + L.tile_entry);
    const float4* rec = reinterpret_cast<const float4*>(ws + L.records);
    const float* tf = reinterpret_cast<const float*>(ws + L.t_final);
    const uint32_t* nl = reinterpret_cast<const uint32_t*>(ws + L.n_last);
    const int tiles = (int)L.total_tiles;
    // every part is a workgroup of its own
#define SGS_LAUNCH(K, W, ...)                                                                  \
    hipLaunchKernelGGL(K, dim3((unsigned)(L.total_tiles * W)), dim3(kLanes), 0, s, __VA_ARGS__)
#define SGS_ARGS                                                                              \
    views, rp, ranges, entry, rec, tf, nl, dl_drgb, gate, acc, order, tiles, (uint32_t)L.entries
    const int waves = tile_waves(rp.tile_w, L.total_tiles).backward;
    if (waves == 4)
        SGS_RASTER_PARTS(raster_backward_kernel, 4, SGS_ARGS);
    else if (waves == 2)
        SGS_RASTER_PARTS(raster_backward_kernel, 2, SGS_ARGS);
    else if (rp.tile_w == 8)
        SGS_RASTER_BATCHES(raster_backward_kernel, 8, 8, SGS_ARGS);
    else if (rp.tile_w == 16)
        SGS_RASTER_BATCHES(raster_backward_kernel, 16, 16, SGS_ARGS);
    else
        SGS_RASTER_BATCHES(raster_backward_kernel, 32, 8, SGS_ARGS);
#undef SGS_ARGS
#undef SGS_LAUNCH
    return hipGetLastError();
}

#undef SGS_RASTER_PARTS
#undef SGS_RASTER_BATCHES

}  // namespace sgs
