// Device pieces of the draw of k_t (Sec. 3.4) shared by the draw's own kernels and the
// launch that runs several iterations of a search (kb_ucb.hip).
#pragma once
#include "kb_internal.h"
#include "kb_rng_dev.h"

namespace kb {

constexpr int kNoCandidate = 0x7fffffff;

struct SampleArgs {
    int G, Ksum;
    int64_t N;
    const int32_t* seg_off;
    const int32_t* koff;
    const int32_t* assign;
    const uint8_t* alive;      // may be NULL: every candidate alive
    const float* bound;
    const float* incumbent;
    const int32_t* sel;        // [G,3]
    // paper-form potential (mode 1): V = theta_sat - h[k, target[S*]]
    const float* h;
    const int32_t* target;
    int R, S, mode;
    float theta_sat;
    unsigned seed_lo, seed_hi, draw_lo, draw_hi;
    double tau;
    int32_t* ksel;             // [G]
    double* slot_key;          // [2 * ranges]  left slot of range r at 2r, right slot at 2r+1
    int32_t* slot_idx;         // [2 * ranges]
    int short_n;               // sample_short() of the batch
    int mixed;                 // 1: searches of at most short_n candidates go to the wave form of sample_search, longer
                               //    ones to the range kernels, in the same call
};

// (key, index) pairs ordered by larger key, then lower index; index kNoCandidate = empty
__device__ __forceinline__ bool better(double ka, int ia, double kb_, int ib) {
    return ia != kNoCandidate && (ib == kNoCandidate || ka > kb_ || (ka == kb_ && ia < ib));
}

__device__ __forceinline__ double sample_key(const SampleArgs& a, int k, double pot_scale,
                                             int tcol) {
    double V;
    if (a.mode == 0) {
        V = 1.0 - (double)a.bound[k] / pot_scale;
    } else {
        V = (double)a.theta_sat - (double)a.h[(size_t)k * a.R + tcol];
    }
    return V / a.tau + gumbel_variate(a.seed_lo, a.seed_hi, a.draw_lo, a.draw_hi, k);
}

inline SampleArgs make_sample_args(const kb_batch& b, const SampleCall& c) {
    SampleArgs a;
    a.G = b.G; a.Ksum = b.Ksum; a.N = b.N; a.seg_off = b.seg_off; a.koff = b.koff;
    a.assign = c.assign; a.alive = c.alive; a.bound = c.bound; a.incumbent = c.incumbent;
    a.sel = c.sel; a.h = c.h; a.target = c.target; a.R = c.R; a.S = b.S; a.mode = c.h ? 1 : 0;
    a.theta_sat = c.theta_sat;
    a.seed_lo = (unsigned)c.seed; a.seed_hi = (unsigned)(c.seed >> 32);
    a.draw_lo = (unsigned)c.draw; a.draw_hi = (unsigned)(c.draw >> 32);
    a.tau = (double)c.tau;
    a.ksel = c.ksel; a.slot_key = c.slot_key; a.slot_idx = c.slot_idx;
    a.short_n = 0; a.mixed = 0;
    return a;
}

}  // namespace kb
