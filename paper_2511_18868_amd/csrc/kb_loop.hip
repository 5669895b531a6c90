// The small steps that close the loop of Alg. 1 around the scoring pass:
// the strategy mask in the paper's own form (Eq. 5) and the statistics update
// that ends an iteration.  Both touch a few bytes per cluster arm or per search.
#include "kb_internal.h"

namespace kb {

namespace {

constexpr int kThreads = 256;

// M[i,s] = [ h(rep_i)[target(s)] < theta_sat ]; nvalid[g] = number of valid cluster arms of
// the search.  NT threads per search: a wave, or a workgroup where a search may have more
// than kMaskWave arms.  Bound by the dependent loads rep -> h: a thread of a workgroup has U of
// its arms in flight, so a search is a few such chains (a wave per search went through its
// 2048 arms in 32 chains: 512 searches of up to 64 clusters and 32 strategies 37.5 us, now 6 us).
// Where many searches share the chip they hide each other's loads, and a wave each, one arm
// per lane, gets through more of them (whole calls, wave / workgroup: 4000 searches of 1024 arms
// 13.1 / 12.4 us, 20000 of 272 14.8 / 25.6, of 1024 34.7 / 38.2, of 8192 235 / 212).
constexpr int kMaskWave = 256;
constexpr int kMaskFewG = 4096;           // more searches: a workgroup each only for kMaskMany arms on average
constexpr int kMaskMany = 4096;

template <int NT, int U>
__global__ void __launch_bounds__(kThreads)
strategy_mask_kernel(int G, int S, int R, int Ksum, int64_t N, const int32_t* __restrict__ koff,
                     const float* __restrict__ h, const int32_t* __restrict__ target,
                     const int32_t* __restrict__ rep, float theta_sat, uint8_t* __restrict__ M,
                     int32_t* __restrict__ nvalid) {
    __shared__ int part[kThreads / kWave];
    const int lane = threadIdx.x & (NT - 1);
    const int g = blockIdx.x * (kThreads / NT) + threadIdx.x / NT;
    if (g >= G) return;                   // (whole waves; with NT = 256 never)
    const int k0 = clampi(koff[g], 0, Ksum);
    const int k1 = clampi(koff[g + 1], k0, Ksum);
    const int arms = (k1 - k0) * S;
    int n = 0;
    for (int q0 = lane; q0 < arms; q0 += NT * U) {
        int r[U], col[U];
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u * NT;
            r[u] = -1;
            if (q < arms) {
                const int i = q / S;
                r[u] = rep[k0 + i];
                col[u] = clampi(target[q - i * S], 0, R - 1);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (r[u] >= 0 && (int64_t)r[u] < N) v[u] = h[(size_t)r[u] * R + col[u]];
            else r[u] = -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = q0 + u * NT;
            if (q < arms) {
                const int m = r[u] >= 0 && v[u] < theta_sat ? 1 : 0;
                M[(size_t)k0 * S + q] = (uint8_t)m;
                n += m;
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    if constexpr (NT > kWave) {
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
        __syncthreads();
        n = 0;
#pragma unroll
        for (int w = 0; w < NT / kWave; ++w) n += part[w];
    }
    if (lane == 0) nvalid[g] = n;
}

// One thread per search.  Searches own disjoint cluster arms and candidates, so
// the read-modify-write steps need no atomics.
__global__ void __launch_bounds__(kThreads)
update_stats_kernel(int G, int S, int Ksum, int64_t N, const int32_t* __restrict__ seg_off,
                    const int32_t* __restrict__ koff, const int32_t* __restrict__ sel,
                    const int32_t* __restrict__ ksel, const float* __restrict__ reward,
                    const uint8_t* __restrict__ ok, double prior_n, int32_t* __restrict__ visits,
                    float* __restrict__ rsum, int32_t* __restrict__ Ncs, float* __restrict__ mu,
                    int64_t* __restrict__ t, const int32_t* __restrict__ assign,
                    const uint8_t* __restrict__ alive, unsigned* __restrict__ gN,
                    unsigned long long* __restrict__ gR) {
    const int g = blockIdx.x * kThreads + threadIdx.x;
    if (g >= G) return;
    t[g] += 1;
    int n0, ng, k0, K;
    search_bounds(seg_off, koff, g, N, Ksum, n0, ng, k0, K);
    const int I = sel[(size_t)g * 3], s = sel[(size_t)g * 3 + 1], k = ksel[g];
    if (!ok[g] || I < 0 || I >= K || s < 0 || s >= S || k < n0 || k >= n0 + ng) return;
    const size_t arm = ((size_t)k0 + I) * S + s;
    const int nn = Ncs[arm] + 1;
    Ncs[arm] = nn;
    const double r = (double)reward[g];
    const double m = (double)mu[arm];
    mu[arm] = (float)(m + (r - m) / ((double)nn + prior_n));
    const size_t cell = (size_t)k * S + s;
    visits[cell] += 1;
    const float r_old = rsum[cell];
    const float r_new = (float)((double)r_old + r);
    rsum[cell] = r_new;
    if (gN && (!alive || alive[k])) {
        // the tables an aggregation over the alive candidates would now give: one more
        // visit and the change of this cell's fixed-point image, in the candidate's cluster
        int j = assign[k];
        j = (j >= 0 && j < K) ? j : 0;
        const size_t tarm = ((size_t)k0 + j) * S + s;
        gN[tarm] += 1u;
        gR[tarm] += reward_fixed(r_new) - reward_fixed(r_old);
    }
}

}  // namespace

hipError_t launch_strategy_mask(const kb_batch& b, int R, const float* h, const int32_t* target,
                                const int32_t* rep, float theta_sat, uint8_t* M, int32_t* nvalid,
                                hipStream_t st) {
    const auto go = [&](auto kern, int per) {
        hipLaunchKernelGGL(kern, dim3((unsigned)((b.G + per - 1) / per)), dim3(kThreads), 0, st, b.G, b.S, R,
                           b.Ksum, b.N, b.koff, h, target, rep, theta_sat, M, nvalid);
    };
    const bool groups = b.G <= kMaskFewG ? (int64_t)b.Kmax * b.S > kMaskWave
                                         : (int64_t)b.Ksum * b.S >= (int64_t)kMaskMany * b.G;
    if (groups) go(strategy_mask_kernel<kThreads, 4>, 1);
    else go(strategy_mask_kernel<kWave, 1>, kThreads / kWave);
    return hipGetLastError();
}

hipError_t launch_update_stats(const kb_batch& b, float prior_n, const int32_t* sel,
                               const int32_t* ksel, const float* reward, const uint8_t* ok,
                               int32_t* visits, float* rsum, int32_t* Ncs, float* mu, int64_t* t,
                               hipStream_t st, const int32_t* assign, const uint8_t* alive,
                               unsigned* gN, unsigned long long* gR) {
    if (gN && (!gR || !assign)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(update_stats_kernel, dim3((unsigned)((b.G + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, st, b.G, b.S, b.Ksum, b.N, b.seg_off, b.koff, sel, ksel,
                       reward, ok, (double)prior_n, visits, rsum, Ncs, mu, t, assign, alive, gN, gR);
    return hipGetLastError();
}

}  // namespace kb
