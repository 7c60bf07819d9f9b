// Photometric loss (paper Eq. 6): L = (1 - lambda) L1 + lambda (1 - SSIM),
// SSIM with an 11x11 Gaussian window (sigma 1.5), zero-padded same-size
// filtering, both terms averaged over the 3 H W values.
//
// One wave filters one channel of a strip of 54 columns (64 lanes less the
// window's halo) and walks down its rows. A row of values (x, y and their three
// products, formed once per pixel) goes through LDS, a float4 and a float per
// lane, for the horizontal taps; the filtered row is then added to the ten
// output rows in the making, whose partial sums each lane holds in registers:
// one fused multiply-add per moment and tap, and since every partial sum moves
// one place with its update, no shift and no LDS. Strips are cut into as few
// rows as it takes to fill the chip, since every strip repeats ten rows of the
// filters.
//
// What bounds it: vector issue, 113 operations per pixel and channel in the
// filters, times 1.19 for the halo columns and 1.36 for the halo rows (28 to a
// strip at 1600x1060), and 60 for S and the maps. The tiled form before it
// (16x16 pixels per workgroup, 26x26 staged values, the products formed again at
// every tap, both passes through LDS) issued twice as many instructions. The
// order of every sum and the rounding of every quotient are the tiled form's,
// so the maps and the gradient are the same bit for bit. Repeated on the same
// 1600x1060 images: forward 90 -> 53 us, backward 72 -> 41 us (122 MB of images,
// maps and gradient, 3 TB/s); at 980x545 38 -> 27 and 30 -> 21 us; at 640x480 and
// below the forward alone is 1 to 2 us slower than the tiled one (25 and 23 us
// with its reduction at 640x480) and the backward 4 faster. In a training iteration
// of 3M Gaussians, which leaves little of the images in the caches, the forward
// takes 71 us and the backward, with the clearing it takes along, 69. (Vertical
// pass first takes 7% off both, as the halo rows skip the horizontal taps, but
// rounds differently: 3e-6 of the gradient, as far as either is from 64 bits.)
//
// A lane adds the values of its column in FP32 over kFold rows and these in
// binary64, as all sums after it are: a strip has the more rows the larger the
// image (32 at 1600x1060, 1366 at 8192x8192), and FP32 over all of them is off by
// 2e-5 there for a flat difference. Per-strip sums go to a partials array that a
// one-workgroup kernel reduces in index order, so the loss is bit-reproducible.
//
// Backward: per pixel p the SSIM value S(p) depends on x through mu_x(p),
// E[x^2](p) and E[xy](p); the map derivatives dS/dmu_x, dS/dE[x^2],
// dS/dE[xy] are written by the forward (when a workspace holds them) and
// filtered again by the backward (the window is symmetric):
//   dSSIM/dx(q) = F[dS/dmu_x](q) + 2 x(q) F[dS/dE[x^2]](q) + y(q) F[dS/dE[xy]](q).
#include <algorithm>

#include "sgs_gate.hpp"
#include "sgs_prepare.hpp"

namespace sgs {

namespace {

constexpr int kR = 5;                   // window radius
constexpr int kTaps = 2 * kR + 1;
constexpr int kCols = 64 - 2 * kR;      // output columns of a wave
constexpr int kThreads = 3 * 64;        // one wave a channel
constexpr int kFold = 8;                // rows added up in FP32
constexpr float kC1 = 0.01f * 0.01f;
constexpr float kC2 = 0.03f * 0.03f;

struct Window {
    float g[kTaps];
};

Window make_window() {
    Window w;
    double s = 0.0, v[kTaps];
    for (int k = 0; k < kTaps; ++k) {
        const double d = k - kR;
        v[k] = std::exp(-(d * d) / (2.0 * 1.5 * 1.5));
        s += v[k];
    }
    for (int k = 0; k < kTaps; ++k) w.g[k] = (float)(v[k] / s);
    return w;
}

// The image cut into strips of kCols columns and `rows` rows, one workgroup
// each: as many as make 4 workgroups (3 waves per SIMD) on every compute unit,
// of kLeast rows at least. us of the forward with its reduction / of the
// backward by the bound on the strips: 1600x1060 800 71.7 / 46.9, 1024 57.4 /
// 40.7, 1152 60.9 / 43.9, 1400 (a second round) 72.7 / 44.6; 980x545 800 34.3
// / 22.0, 1024 31.2 / 20.5, 1280 32.4 / 22.6, 1400 38.3 / 24.0. At 64x64 twice
// the rows cost a quarter more.
constexpr int64_t kResident = 1024;
constexpr int64_t kLeast = 4;
struct Strips {
    int rows;
    dim3 grid;
};
Strips strips(int w, int h) {
    const int64_t nx = (w + kCols - 1) / kCols;
    const int64_t ny = std::max<int64_t>(1, kResident / nx);
    const int64_t rows = std::max<int64_t>((h + ny - 1) / ny, kLeast);
    return {(int)rows, dim3((unsigned)nx, (unsigned)((h + rows - 1) / rows))};
}

// Loss workspace: [partials: kLossPartials doubles][maps: 9 * H * W floats].
// There are at most kResident strips (images of up to 32768 columns have fewer
// strips side by side).
static_assert(32768 / kCols + 1 <= kResident && kLossPartials == 2 * kResident, "two sums a strip");
struct LossLayout {
    size_t partials, maps, total;
};

LossLayout loss_layout(int w, int h) {
    LossLayout L;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    L.partials = 0;
    L.maps = al(sizeof(double) * kLossPartials);
    L.total = al(L.maps + sizeof(float) * 9 * (size_t)w * h);
    return L;
}

// Sum of a binary64 value over the wave, in lane 63, in the DPP steps of
// wave_sum_to_lane63 (by shuffles the two sums add 0.7 us to a 64x64 image).
template <int kCtrl>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, kCtrl, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), kCtrl, 0xf, 0xf, false);
    return v + __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}
__device__ __forceinline__ double wave_sum_to_lane63(double v) {
    return dpp_add<0x143>(dpp_add<0x142>(dpp_add<0x128>(dpp_add<0x124>(dpp_add<0x4e>(dpp_add<0xb1>(v))))));
}

// The reference image of a call: the given one, or image *d_view (clamped)
// of an array of n_targets images of 3 H W floats.
__device__ __forceinline__ const float* target_of(const TargetRef& t, int64_t image_floats) {
    if (t.d_view == nullptr) return t.base;
    const int i = min(max(*t.d_view, 0), t.n_targets - 1);
    return t.base + (int64_t)i * image_floats;
}

// Quotients by one divisor, each rounded as an IEEE division rounds it: the
// reciprocal is refined to the nearest float (two Newton steps), and a quotient
// a r corrected once by its exact remainder is then the nearest one (Markstein
// 1990), without the scaling of the general sequence. That needs divisors and
// quotients far from the ends of the float range: B1 >= C1, and B2 is C2 plus
// multiples of the last places of the squared means, so with 0 < |B1 B2| < 2^40
// (pixel values into the thousands) nothing here comes near them. Other pixels
// are divided in full (NaN, infinities, zero and subnormal reciprocals included).
constexpr float kDivisorEnd = 0x1p40f;
struct Divisor {
    float d, r;
    __device__ __forceinline__ explicit Divisor(float x) : d(x) {
        const float r0 = __builtin_amdgcn_rcpf(x);
        const float r1 = fmaf(fmaf(-x, r0, 1.f), r0, r0);
        r = fmaf(fmaf(-x, r1, 1.f), r1, r1);
    }
    __device__ __forceinline__ float of(float a) const {
        const float q = a * r;
        return fmaf(fmaf(-d, q, a), r, q);
    }
};

// The partial sums of one field over rows: after input row r, sum[j] holds
// output row r - kR + 1 + j less the rows still to come.
struct Column {
    float sum[kTaps - 1];
    __device__ __forceinline__ Column() {
#pragma unroll
        for (int j = 0; j < kTaps - 1; ++j) sum[j] = 0.f;
    }
    // Adds a row's value and returns the output row it completes.
    __device__ __forceinline__ float add(const Window& W, float v) {
        const float done = fmaf(W.g[kTaps - 1], v, sum[0]);
#pragma unroll
        for (int j = 1; j < kTaps - 1; ++j) sum[j - 1] = fmaf(W.g[kTaps - 1 - j], v, sum[j]);
        sum[kTaps - 2] = W.g[0] * v;
        return done;
    }
};

// One workgroup's strip: this wave's channel and this lane's column.
struct Place {
    int ch, lane, cx, first, end;   // output rows [first, end)
    bool out;                       // the lane's column is an output column
    bool in_image;
    int tap0;                       // LDS index of the lane's first horizontal tap
    __device__ __forceinline__ Place(int w, int h, int rows, int row) {
        lane = threadIdx.x % 64;
        ch = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
        cx = (int)blockIdx.x * kCols - kR + lane;
        first = row * rows;
        end = min(first + rows, h);
        in_image = cx >= 0 && cx < w;
        out = lane >= kR && lane < kR + kCols && cx < w;
        tap0 = min(max(lane, kR), kR + kCols - 1) - kR;
    }
};

// Forward: sums of |x - y| and of S over the strip into partials[2 blk] and,
// with kMaps, the maps dS/dmu_x, dS/dE[x^2], dS/dE[xy] the backward filters.
// The maps are written on every forward: forming them again in the backward
// would repeat the whole moment pass, which costs more than the writes it
// saves on iterations whose backward is skipped.
// (4 waves per SIMD: at most 128 registers.)
template <bool kMaps>
__global__ void __launch_bounds__(kThreads, 4) ssim_forward_kernel(
    const float* __restrict__ x, TargetRef target, int w, int h, int rows, Window W,
    double* __restrict__ partials, float* __restrict__ maps) {
    __shared__ float4 s_m4[3][64];
    __shared__ float s_m1[3][64];
    __shared__ double red[2][3];
    const Place p(w, h, rows, (int)blockIdx.y);
    const int64_t plane = (int64_t)w * h;
    const float* __restrict__ xc = x + p.ch * plane + p.cx;
    const float* __restrict__ yc = target_of(target, 3 * plane) + p.ch * plane + p.cx;
    float4* m4 = s_m4[p.ch];
    float* m1 = s_m1[p.ch];
    Column cx_, cy_, cxx, cyy, cxy;
    float s_l1 = 0.f, s_ssim = 0.f;
    double l1 = 0.0, ssim = 0.0;
    auto fold = [&]() {
        l1 += (double)s_l1;
        ssim += (double)s_ssim;
        s_l1 = s_ssim = 0.f;
    };
    // rows are loaded kAhead rows before they are used
    constexpr int kAhead = 2;
    float a[kAhead], b[kAhead];
    auto load = [&](int r, float& av, float& bv) {
        const bool ok = p.in_image && r >= 0 && r < h;
        av = ok ? xc[(int64_t)r * w] : 0.f;
        bv = ok ? yc[(int64_t)r * w] : 0.f;
    };
#pragma unroll
    for (int k = 0; k < kAhead; ++k) load(p.first - kR + k, a[k], b[k]);
    for (int r = p.first - kR; r < p.end + kR; ++r) {
        if (r % kFold == 0) fold();   // uniform
        const float av = a[0], bv = b[0];
#pragma unroll
        for (int k = 0; k + 1 < kAhead; ++k) {
            a[k] = a[k + 1];
            b[k] = b[k + 1];
        }
        load(r + kAhead, a[kAhead - 1], b[kAhead - 1]);
        if (p.out && r >= p.first && r < p.end) s_l1 += fabsf(av - bv);
        m4[p.lane] = make_float4(av, bv, av * av, bv * bv);
        m1[p.lane] = av * bv;
        wave_lds_sync();
        float h0 = 0.f, h1 = 0.f, h2 = 0.f, h3 = 0.f, h4 = 0.f;
#pragma unroll
        for (int k = 0; k < kTaps; ++k) {
            const float4 q = m4[p.tap0 + k];
            const float g = W.g[k];
            h0 = fmaf(g, q.x, h0);
            h1 = fmaf(g, q.y, h1);
            h2 = fmaf(g, q.z, h2);
            h3 = fmaf(g, q.w, h3);
            h4 = fmaf(g, m1[p.tap0 + k], h4);
        }
        wave_lds_sync();
        const float mx = cx_.add(W, h0), my = cy_.add(W, h1), exx = cxx.add(W, h2),
                    eyy = cyy.add(W, h3), exy = cxy.add(W, h4);
        const int o = r - kR;
        if (o < p.first) continue;   // uniform
        if (p.out) {
            const float sxx = exx - mx * mx, syy = eyy - my * my, sxy = exy - mx * my;
            const float A1 = 2.f * mx * my + kC1, A2 = 2.f * sxy + kC2;
            const float B1 = mx * mx + my * my + kC1, B2 = sxx + syy + kC2;
            const float D = B1 * B2;
            float S = 0.f, m0 = 0.f, m1 = 0.f, m2 = 0.f;
            auto quotients = [&](float r1, float r2, auto by_d, auto by_2) {
                S = by_d(A1 * A2);
                if (kMaps) {
                    m0 = by_d(2.f * my * (A2 - A1)) - 2.f * mx * S * (r1 - r2);
                    m1 = by_2(-S);
                    m2 = by_d(2.f * A1);
                }
            };
            if (fabsf(D) < kDivisorEnd && D != 0.f) {
                const Divisor d1(B1), d2(B2), dd(D);
                quotients(d1.r, d2.r, [&](float a) { return dd.of(a); },
                          [&](float a) { return d2.of(a); });
            } else {
                quotients(1.f / B1, 1.f / B2, [&](float a) { return a / D; },
                          [&](float a) { return a / B2; });
            }
            s_ssim += S;
            if (kMaps) {
                const int64_t pix = (int64_t)o * w + p.cx;
                maps[(0 * 3 + p.ch) * plane + pix] = m0;
                maps[(1 * 3 + p.ch) * plane + pix] = m1;
                maps[(2 * 3 + p.ch) * plane + pix] = m2;
            }
        }
    }
    // fixed-order workgroup sum
    fold();
    l1 = wave_sum_to_lane63(l1);
    ssim = wave_sum_to_lane63(ssim);
    if (p.lane == 63) {
        red[0][p.ch] = l1;
        red[1][p.ch] = ssim;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const int64_t blk = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
        partials[2 * blk] = (red[0][0] + red[0][1]) + red[0][2];
        partials[2 * blk + 1] = (red[1][0] + red[1][1]) + red[1][2];
    }
}

// Sum of the per-strip partials in index order (binary64), then Eq. 6 and, in a
// training iteration, the gate's decision (a launch of its own otherwise) and
// the step of the view sequence. One workgroup of NT threads.
struct LossSum {
    const double* partials;
    int64_t nb;
    double count;
    float lambda;
    float* d_loss;
    LossGate gate;
};
constexpr int kSumSlots = 1024;
template <int NT>
__device__ __forceinline__ void loss_sum(const LossSum& p, double (*dred)[kSumSlots]) {
    const int tid = threadIdx.x;
    for (int k = tid; k < kSumSlots; k += NT) {
        double a = 0.0, b = 0.0;
        for (int64_t i = k; i < p.nb; i += kSumSlots) {
            a += p.partials[2 * i];
            b += p.partials[2 * i + 1];
        }
        dred[0][k] = a;
        dred[1][k] = b;
    }
    __syncthreads();
    for (int st = kSumSlots / 2; st > 0; st >>= 1) {
        for (int k = tid; k < st; k += NT) {
            dred[0][k] += dred[0][k + st];
            dred[1][k] += dred[1][k + st];
        }
        __syncthreads();
    }
    if (tid == 0) {
        const double l1 = dred[0][0] / p.count, ssim = dred[1][0] / p.count;
        const float loss =
            (float)((1.0 - (double)p.lambda) * l1 + (double)p.lambda * (1.0 - ssim));
        *p.d_loss = loss;
        const LossGate& g = p.gate;
        if (g.gate != nullptr) {
            if (g.state != nullptr)
                gate_step(g.args, g.state, g.view, loss, g.gate);
            else
                *g.gate = 1;
        }
        if (g.iter != nullptr) *g.iter += 1;
    }
}

__global__ void __launch_bounds__(kSumSlots) loss_reduce_kernel(LossSum p) {
    __shared__ double dred[2][kSumSlots];
    loss_sum<kSumSlots>(p, dred);
}

// Besides the gradient, the backward of a training iteration (kTrain) takes
// along, in its first t.rows rows of workgroups, the preparation of the
// compositing backward and, where no gate waits for it, the sum of the loss: 4.6
// us each as launches of their own, and the accumulators (25 us at 3M Gaussians)
// are cleared while the filters keep the vector units busy (the 64x64 step 177 ->
// 174 us with the view of the sequence picked by the projection, the 3M one 1977
// -> 1966).
struct LossTrain {
    Prepare prepare;
    LossSum sum;   // d_loss nullable: summed before
    int rows;
};
template <bool kTrain>
__global__ void __launch_bounds__(kThreads) ssim_backward_kernel(
    LossTrain t, const float* __restrict__ x, TargetRef target, int w, int h, int rows, float lambda,
    Window W, const float* __restrict__ maps, const int32_t* __restrict__ gate,
    const float* __restrict__ scale, float* __restrict__ dl) {
    if (gate_closed(gate)) return;
    if constexpr (kTrain) {
        __shared__ double s_sum[2][kSumSlots];
        __shared__ uint32_t s_scan[kThreads / 64 + 1];
        if ((int)blockIdx.y < t.rows) {   // uniform
            const int block = (int)(blockIdx.y * gridDim.x + blockIdx.x);
            if (block == 0 && t.sum.d_loss != nullptr) loss_sum<kThreads>(t.sum, s_sum);
            if (block > 0)
                prepare_backward<kThreads>(t.prepare, block - 1, t.rows * (int)gridDim.x - 1,
                                           reinterpret_cast<uint32_t*>(s_sum), s_scan);
            return;
        }
    }
    __shared__ float4 s_m[3][64];   // a row of the three maps
    const Place p(w, h, rows, (int)blockIdx.y - (kTrain ? t.rows : 0));
    const int64_t plane = (int64_t)w * h;
    const float* __restrict__ xc = x + p.ch * plane + p.cx;
    const float* __restrict__ yc = target_of(target, 3 * plane) + p.ch * plane + p.cx;
    const float* __restrict__ mc = maps + p.ch * plane + p.cx;
    float* __restrict__ dc = dl + p.ch * plane + p.cx;
    float4* m = s_m[p.ch];
    Column c0, c1, c2;
    const float inv = 1.f / (3.f * (float)w * (float)h);
    const float outer = scale != nullptr ? *scale : 1.f;   // (times 1 is exact)
    // map rows are loaded kAhead rows before they are used, the output row's
    // pixels one row before
    constexpr int kAhead = 3;
    float q[kAhead][3];
    auto load = [&](int r, float (&v)[3]) {
        const bool ok = p.in_image && r >= 0 && r < h;
#pragma unroll
        for (int f = 0; f < 3; ++f) v[f] = ok ? mc[3 * f * plane + (int64_t)r * w] : 0.f;
    };
    float an = 0.f, bn = 0.f;
    auto pixel = [&](int o) {
        const bool ok = p.out && o >= p.first && o < p.end;
        an = ok ? xc[(int64_t)o * w] : 0.f;
        bn = ok ? yc[(int64_t)o * w] : 0.f;
    };
#pragma unroll
    for (int k = 0; k < kAhead; ++k) load(p.first - kR + k, q[k]);
    for (int r = p.first - kR; r < p.end + kR; ++r) {
        float v[3];
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            v[f] = q[0][f];
#pragma unroll
            for (int k = 0; k + 1 < kAhead; ++k) q[k][f] = q[k + 1][f];
        }
        load(r + kAhead, q[kAhead - 1]);
        const int o = r - kR;
        const float a = an, b = bn;
        pixel(o + 1);
        m[p.lane] = make_float4(v[0], v[1], v[2], 0.f);
        wave_lds_sync();
        float h0 = 0.f, h1 = 0.f, h2 = 0.f;
#pragma unroll
        for (int k = 0; k < kTaps; ++k) {
            const float4 t = m[p.tap0 + k];
            h0 = fmaf(W.g[k], t.x, h0);
            h1 = fmaf(W.g[k], t.y, h1);
            h2 = fmaf(W.g[k], t.z, h2);
        }
        wave_lds_sync();
        const float F0 = c0.add(W, h0), F1 = c1.add(W, h1), F2 = c2.add(W, h2);
        if (o < p.first) continue;   // uniform
        if (p.out) {
            const float d_ssim = F0 + 2.f * a * F1 + b * F2;
            const float sgn = a > b ? 1.f : (a < b ? -1.f : 0.f);
            dc[(int64_t)o * w] =
                ((1.f - lambda) * sgn * inv - lambda * d_ssim * inv) * outer;
        }
    }
}

}  // namespace

size_t loss_workspace_bytes(int w, int h) { return loss_layout(w, h).total; }

static LossSum loss_sum_of(const Strips& st, int w, int h, float lambda, const double* partials,
                           float* d_loss, const LossGate& gate) {
    return {partials, (int64_t)st.grid.x * st.grid.y, 3.0 * (double)w * (double)h, lambda, d_loss,
            gate};
}

hipError_t launch_loss_partials(const float* rgb, TargetRef target, int w, int h, float lambda,
                                double* partials, float* d_loss, hipStream_t s) {
    const Strips st = strips(w, h);
    hipLaunchKernelGGL((ssim_forward_kernel<false>), st.grid, dim3(kThreads), 0, s, rgb, target, w,
                       h, st.rows, make_window(), partials, nullptr);
    hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(kSumSlots), 0, s,
                       loss_sum_of(st, w, h, lambda, partials, d_loss, LossGate{}));
    return hipGetLastError();
}

hipError_t launch_loss_forward(const float* rgb, TargetRef target, int w, int h, float lambda,
                               char* ws, float* d_loss, hipStream_t s, const LossGate& gate) {
    const LossLayout L = loss_layout(w, h);
    const Strips st = strips(w, h);
    double* partials = reinterpret_cast<double*>(ws + L.partials);
    float* maps = reinterpret_cast<float*>(ws + L.maps);
    hipLaunchKernelGGL((ssim_forward_kernel<true>), st.grid, dim3(kThreads), 0, s, rgb, target, w,
                       h, st.rows, make_window(), partials, maps);
    if (d_loss != nullptr)
        hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(kSumSlots), 0, s,
                           loss_sum_of(st, w, h, lambda, partials, d_loss, gate));
    return hipGetLastError();
}

hipError_t launch_loss_backward(const float* rgb, TargetRef target, int w, int h, float lambda,
                                char* ws, const int32_t* gate, float* dl, hipStream_t s,
                                const float* scale) {
    const LossLayout L = loss_layout(w, h);
    const Strips st = strips(w, h);
    const float* maps = reinterpret_cast<const float*>(ws + L.maps);
    hipLaunchKernelGGL(ssim_backward_kernel<false>, st.grid, dim3(kThreads), 0, s, LossTrain{}, rgb,
                       target, w, h, st.rows, lambda, make_window(), maps, gate, scale, dl);
    return hipGetLastError();
}

hipError_t launch_train_loss(const float* rgb, TargetRef target, int w, int h, float lambda,
                             char* ws, float* d_loss, float* dl, const LossGate& gate,
                             const Prepare& prepare, hipStream_t s) {
    const bool gated = gate.state != nullptr;
    hipError_t err = launch_loss_forward(rgb, target, w, h, lambda, ws, gated ? d_loss : nullptr, s, gate);
    if (err != hipSuccess) return err;
    const LossLayout L = loss_layout(w, h);
    const Strips st = strips(w, h);
    const double* partials = reinterpret_cast<const double*>(ws + L.partials);
    const float* maps = reinterpret_cast<const float*>(ws + L.maps);
    LossTrain t{prepare, loss_sum_of(st, w, h, lambda, partials, gated ? nullptr : d_loss, gate), 0};
    // the sum, the order, and a workgroup for every kClearEach float4s, up to
    // kClearBlocks (us of the launch at 1M / 3M Gaussians with 64 40.2 / 75.5, 128
    // 39.4 / 71.4, 256 37.6 / 69.4, 1024 40.7 / 70.4, 4096 46.0 / 71.3: more stores
    // in flight hold up the filters' loads)
    constexpr int64_t kClearEach = 4 * kThreads, kClearBlocks = 256;
    const int64_t blocks =
        2 + std::min<int64_t>((prepare.n4 + kClearEach - 1) / kClearEach, kClearBlocks);
    t.rows = (int)((blocks + st.grid.x - 1) / st.grid.x);
    hipLaunchKernelGGL(ssim_backward_kernel<true>, dim3(st.grid.x, st.grid.y + (unsigned)t.rows),
                       dim3(kThreads), 0, s, t, rgb, target, w, h, st.rows, lambda, make_window(),
                       maps, gated ? gate.gate : nullptr, nullptr, dl);
    return hipGetLastError();
}

}  // namespace sgs
