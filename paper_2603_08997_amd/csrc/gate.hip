// SkipGS backward gate (paper Sec. 4, Algorithm 1, Eqs. 7-13) on the device.
// One thread updates the state in binary64, so the decision never leaves the
// GPU: the backward and Adam kernels read the flag it writes, and the view
// index itself is read from device memory, so a captured iteration can be
// replayed over a device-side view sequence. The library is built without
// floating-point contraction, so every operation rounds once, in the order
// written.
//
// The update separates what the gate observes (the score of Eq. 8 and the
// ratio of Eq. 10, both against the state before this iteration), what it
// decides (a pure function of the proposal of Eq. 9, the phase and the budget
// test of Eq. 11) and how its state moves (warmup statistic and calibration,
// Eqs. 12-13; the backward count; the EMA of Eq. 7, on every iteration).
#include "sgs_gate.hpp"

namespace sgs {

namespace {

__global__ void gate_init_kernel(GateArgs p, char* state) {
    GateView S(state, p.n_views);
    for (int i = threadIdx.x; i < p.n_views; i += blockDim.x) {
        S.ema[i] = 0.0;
        S.has[i] = 0;
    }
    if (threadIdx.x == 0) {
        sgs_gate_snapshot* h = S.h;
        h->t = h->b = h->t_w = h->b_w = h->warm_hits = h->warm_count = 0;
        h->rho_min = p.rho_lo;
        h->last_s = 0.0;
        h->last_rho = 0.0;
        h->calibrated = 0;
        h->flags = 0;
        h->last_g = h->last_proposed = h->last_forced = 0;
        h->last_view = -1;
    }
}

__global__ void gate_update_kernel(GateArgs p, char* state, const int32_t* d_view,
                                   const float* d_loss, int32_t* d_gate) {
    if (threadIdx.x == 0 && blockIdx.x == 0) gate_step(p, state, d_view, *d_loss, d_gate);
}

__global__ void sequence_next_kernel(const int32_t* seq, int64_t len, int64_t* iter,
                                     int32_t* view) {
    if (threadIdx.x != 0) return;
    const int64_t k = *iter;
    *view = seq[k % len];
    *iter = k + 1;
}

}  // namespace

GateArgs gate_args(const sgs_gate_params* p) {
    return GateArgs{p->beta, p->eps, p->delta, p->rho_lo, p->warmup, p->window, p->calibrate,
                    p->budget, p->n_views};
}

size_t gate_state_bytes(const sgs_gate_params* p) {
    return sizeof(sgs_gate_snapshot) + sizeof(double) * (size_t)p->n_views + (size_t)p->n_views;
}

hipError_t launch_gate_init(const sgs_gate_params* p, void* state, hipStream_t s) {
    hipLaunchKernelGGL(gate_init_kernel, dim3(1), dim3(256), 0, s, gate_args(p),
                       static_cast<char*>(state));
    return hipGetLastError();
}

hipError_t launch_sequence_next(const int32_t* seq, int64_t len, int64_t* d_iter, int32_t* d_view,
                                hipStream_t s) {
    hipLaunchKernelGGL(sequence_next_kernel, dim3(1), dim3(64), 0, s, seq, len, d_iter, d_view);
    return hipGetLastError();
}

hipError_t launch_gate_update(const sgs_gate_params* p, void* state, const int32_t* view,
                              const float* loss, int32_t* gate, hipStream_t s) {
    hipLaunchKernelGGL(gate_update_kernel, dim3(1), dim3(64), 0, s, gate_args(p),
                       static_cast<char*>(state), view, loss, gate);
    return hipGetLastError();
}

}  // namespace sgs
