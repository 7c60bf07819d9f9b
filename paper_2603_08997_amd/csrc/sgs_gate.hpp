// The SkipGS gate's state and its update (gate.hip says what it does), for the
// kernel of a gate call and for the loss reduction of a training iteration.
#pragma once

#include "sgs_device.hpp"
#include "sgs_internal.hpp"

namespace sgs {

// Device state: this header, then double ema[n_views], then uint8 has_ema[n_views].
static_assert(sizeof(sgs_gate_snapshot) % 8 == 0, "header must keep the EMA array aligned");

struct GateView {
    sgs_gate_snapshot* h;
    double* ema;
    uint8_t* has;
    __device__ GateView(char* state, int n_views)
        : h(reinterpret_cast<sgs_gate_snapshot*>(state)),
          ema(reinterpret_cast<double*>(state + sizeof(sgs_gate_snapshot))),
          has(reinterpret_cast<uint8_t*>(state + sizeof(sgs_gate_snapshot) +
                                         sizeof(double) * (size_t)n_views)) {}
};

// g of one iteration (Eqs. 9 and 11): warmup iterations always run the
// backward; afterwards the proposal stands unless the budget floor is
// enforced and the backward ratio is below it.
__device__ __forceinline__ int gate_decision(int proposal, bool in_warmup, bool budget, double rho,
                                             double rho_min) {
    if (in_warmup) return 1;
    if (budget && rho < rho_min) return 1;
    return proposal;
}

// Eqs. 12-13: the floor from the warmup statistic, once, after the warmup;
// with no scored warmup iteration the floor stays at rho_lo.
__device__ __forceinline__ void calibrate_floor(const GateArgs& p, sgs_gate_snapshot* h) {
    if (h->calibrated || !p.calibrate || p.warmup <= 0) return;
    if (h->warm_count > 0)
        h->rho_min = p.rho_lo + (1.0 - p.rho_lo) * ((double)h->warm_hits / (double)h->warm_count);
    h->calibrated = 1;
}

// One iteration with loss `loss` (one thread).
__device__ __forceinline__ void gate_step(const GateArgs& p, char* state, const int32_t* d_view,
                                          float loss, int32_t* d_gate) {
    GateView S(state, p.n_views);
    sgs_gate_snapshot* h = S.h;
    const int view = *d_view;
    if (view < 0 || view >= p.n_views) {
        // not an iteration: the state keeps its clock, counts and EMAs
        h->flags |= (int32_t)SGS_STATUS_BAD_VIEW;
        h->last_g = h->last_proposed = h->last_forced = 0;
        h->last_view = view;
        *d_gate = 0;
        return;
    }
    const double L = (double)loss;
    // the clock (and the tumbling window) advance on every iteration
    h->t += 1;
    if (p.window > 0 && (h->t - 1) % p.window == 0) {
        h->t_w = 0;
        h->b_w = 0;
    }
    h->t_w += 1;
    h->last_view = view;
    if (!isfinite(L)) {
        h->flags |= (int32_t)SGS_STATUS_NONFINITE_LOSS;
        h->last_g = h->last_proposed = h->last_forced = 0;
        h->last_s = __builtin_nan("");
        h->last_rho = __builtin_nan("");
        *d_gate = 0;
        return;
    }
    // observation: score (Eq. 8; +inf for a view with no EMA yet, which
    // always proposes) and ratio (Eq. 10) against the state before this
    // iteration
    const bool scored = S.has[view] != 0;
    const double s = scored ? L / (S.ema[view] + p.eps) : __builtin_inf();
    const int proposal = s > 1.0 + p.delta ? 1 : 0;
    const double rho = p.window > 0 ? (double)h->b_w / (double)max(h->t_w - 1, (int64_t)1)
                                    : (double)h->b / (double)max(h->t - 1, (int64_t)1);
    const bool in_warmup = h->t <= p.warmup;
    if (in_warmup) {
        if (scored) {
            h->warm_count += 1;
            h->warm_hits += proposal;
        }
    } else {
        calibrate_floor(p, h);
    }
    const int g = gate_decision(proposal, in_warmup, p.budget != 0, rho, h->rho_min);
    h->b += g;
    h->b_w += g;
    S.ema[view] = scored ? p.beta * S.ema[view] + (1.0 - p.beta) * L : L;
    S.has[view] = 1;
    h->last_g = g;
    h->last_proposed = proposal;
    h->last_forced = (g == 1 && proposal == 0) ? 1 : 0;
    h->last_s = s;
    h->last_rho = rho;
    *d_gate = g;
}

}  // namespace sgs
