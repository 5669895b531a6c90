// Draw of k_t inside the chosen cluster (Sec. 3.4; Alg. 1 "Sample k_t"):
// P(k) proportional to exp(V(k)/tau) over the alive members of cluster I_t, with
// V the candidate's remaining headroom.  The draw is a deterministic argmax: the
// Gumbel-max identity turns the softmax into argmax_k (V(k)/tau - ln(-ln u_k)),
// and u_k comes from the counter-based generator Philox4x32-10 (Salmon, Moraes,
// Dror, Shaw, SC'11) keyed by the seed and addressed by (candidate, draw), so
// a draw depends on nothing but its arguments.
//
// One pass over assign (and over alive / bound of the members only).  The
// candidate axis is cut into flat ranges of kSampleRange candidates, one workgroup
// each; a workgroup walks the searches that intersect its range.  A search that
// lies inside one range is finished there.  A search that crosses range borders
// leaves one partial (key, index) per range in the workspace - the piece that
// starts before the range in its "left" slot, the piece that starts inside and
// runs past the end in its "right" slot - and sample_final merges the slots of
// each such search in index order.  Keys are fp64 and compared exactly, lowest
// index on ties, so the result does not depend on the cutting.
#include "kb_internal.h"
#include "kb_sample_dev.h"

namespace kb {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
// Which threads draw for a search (sample_search where nothing else is said; range kernels or a wave
// each / 256 threads / 1024, us):
//   up to 256 candidates: a wave.
//   up to 4096: 256 threads.  1024 searches of 512 11.8 / 7.5 / 14.6, 300 of 70-1900 23.2 / 9.2 / 9.7, 512 of
//     64-4096 32.7 / 10.1 / 11.8, 4096 of them 34.1 / 18.5 / 58.3, 2000 of 1500 43.9 / 19.5 / 40.9.
//   few that may be longer than 2048, up to 11000, or to 16384 where a cluster has few members: 1024 threads.
//     One of 4096 10.8 / 5.8 / 4.9, 8 of 4000 29.5 / 16.2 / 8.9.  Every member of the chosen cluster is two
//     logarithms, which the ranges spread over the chip: the longest searches take the ranges from 1200 members on
//     (range kernels / 1024: 30 of up to 15132, K = 2 26.6 / 60.8, K = 4 34.5 / 62.7, 8 of up to 13880, K = 1
//     25.7 / 32.7; 100 of 35-12445, K = 16 34 / 13.6, of 256-9689, K = 1 36 / 25; over random searches with more
//     members, of 8192-11000 rows 1.18, of 12300-16384 0.83 times as fast in 1024 threads).
//   very many with few candidates on average: a wave (4000 of 300 15.8 / 16.1 / 54.3).
//   otherwise the range kernels, and in a batch of several searches a wave for those of up to
//     short_n (4096 where searches have 1024 candidates or fewer on average, else 256) in the same call.
constexpr int kGroupN = 4096, kGroupMaxG = 4096, kGroupMeanN = 512;
constexpr int kWideFewG = 256, kWideFewN = 2048, kWideMaxG = 512, kWideN = 11000, kWideMembersN = 16384, kWideMembers = 1200;
constexpr int kSampleShortMany = 4096;
static int sample_short(const kb_batch& b) {
    return b.N <= (int64_t)1024 * b.G ? kSampleShortMany : kShortSearch;
}

__global__ void __launch_bounds__(kThreads) sample_range(SampleArgs a) {
    __shared__ double redk[kWaves];
    __shared__ int redi[kWaves];
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * kSampleRange;
    if (r0 >= a.N) return;
    const int64_t r1 = r0 + kSampleRange < a.N ? r0 + kSampleRange : a.N;
    if (tid == 0) {
        a.slot_idx[2 * (size_t)blockIdx.x] = kNoCandidate;
        a.slot_idx[2 * (size_t)blockIdx.x + 1] = kNoCandidate;
    }
    // largest g with seg_off[g] <= r0
    int lo = 0, hi = a.G;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)a.seg_off[mid] <= r0) lo = mid; else hi = mid;
    }
    const auto mine = [&](int n0, int ng, int k0, int K) {
        return n0 >= r1 || (ng > 0 && !(a.mixed && ng <= a.short_n));
    };
    for (int g = lo; (g = next_search(a.seg_off, a.koff, g, a.G, a.N, a.Ksum, mine)) < a.G; ++g) {
        int n0, ng, k0, K;
        search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
        if (n0 >= r1) break;
        if (ng <= 0) continue;
        if (a.mixed && ng <= a.short_n) continue;      // (uniform) a wave of sample_search takes this search
        const int n1 = n0 + ng;
        const int q0 = r0 > n0 ? (int)r0 : n0;
        const int q1 = r1 < n1 ? (int)r1 : n1;
        if (q0 >= q1) continue;
        const int I = a.sel[(size_t)g * 3];
        double bk = 0.0;
        int bi = kNoCandidate;
        if (I >= 0) {
            double pot_scale = 1.0;
            int tcol = 0;
            if (a.mode == 0) {
                pot_scale = (double)a.incumbent[g];
            } else {
                const int s = clampi(a.sel[(size_t)g * 3 + 1], 0, a.S - 1);
                tcol = clampi(a.target[s], 0, a.R - 1);
            }
            constexpr int U = 4;
            for (int pb = q0 + tid; pb < q1; pb += kThreads * U) {
                int jj[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int p = pb + u * kThreads;
                    jj[u] = p < q1 ? a.assign[p] : -1;
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int p = pb + u * kThreads;
                    if (jj[u] != I) continue;
                    if (a.alive && !a.alive[p]) continue;
                    const double key = sample_key(a, p, pot_scale, tcol);
                    if (better(key, p, bk, bi)) { bk = key; bi = p; }
                }
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const double ok = __shfl_xor(bk, o);
                const int oi = __shfl_xor(bi, o);
                if (better(ok, oi, bk, bi)) { bk = ok; bi = oi; }
            }
            if ((tid & 63) == 0) { redk[tid >> 6] = bk; redi[tid >> 6] = bi; }
            __syncthreads();
            if (tid == 0) {
                for (int w = 1; w < kWaves; ++w)
                    if (better(redk[w], redi[w], bk, bi)) { bk = redk[w]; bi = redi[w]; }
            }
        }
        if (tid == 0) {
            if (n0 >= r0 && n1 <= r1) {
                a.ksel[g] = bi == kNoCandidate ? -1 : bi;
            } else {
                const size_t slot = 2 * (size_t)blockIdx.x + (n0 < r0 ? 0 : 1);
                a.slot_key[slot] = bk;
                a.slot_idx[slot] = bi;
            }
        }
        __syncthreads();
    }
}

// One thread per search: searches without candidates get -1; searches that
// cross range borders merge their slots in increasing range order.
__global__ void __launch_bounds__(kThreads) sample_final(SampleArgs a) {
    const int g = blockIdx.x * kThreads + threadIdx.x;
    if (g >= a.G) return;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (ng <= 0) { a.ksel[g] = -1; return; }
    if (a.mixed && ng <= a.short_n) return;
    const int rf = n0 / kSampleRange, rl = (n0 + ng - 1) / kSampleRange;
    if (rf == rl) return;
    double bk = a.slot_key[2 * (size_t)rf + 1];
    int bi = a.slot_idx[2 * (size_t)rf + 1];
    for (int r = rf + 1; r <= rl; ++r) {
        const double ok = a.slot_key[2 * (size_t)r];
        const int oi = a.slot_idx[2 * (size_t)r];
        if (better(ok, oi, bk, bi)) { bk = ok; bi = oi; }
    }
    a.ksel[g] = bi == kNoCandidate ? -1 : bi;
}

// A search to NT threads: a wave (four searches per workgroup) or a workgroup of its own, one launch.
// (A workgroup of sample_range walks the searches of its range one after
// the other, a barrier per search; with a few dozen candidates per search that is
// hundreds of searches in a row.)  Same keys, same exact comparison, so the same draw.
template <int NT>
__global__ void __launch_bounds__(NT < kThreads ? kThreads : NT) sample_search(SampleArgs a) {
    constexpr int W = NT / kWave;
    __shared__ double redk[W];
    __shared__ int redi[W];
    const int tid = NT == kWave ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
    const int g = NT == kWave ? (int)blockIdx.x * kWaves + (int)(threadIdx.x >> 6) : (int)blockIdx.x;
    if (g >= a.G) return;                  // (whole waves)
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (ng <= 0) {
        if (tid == 0) a.ksel[g] = -1;
        return;
    }
    if (a.mixed && ng > a.short_n) return;         // the range kernels take this search
    const int I = a.sel[(size_t)g * 3];
    double bk = 0.0;
    int bi = kNoCandidate;
    if (I >= 0) {                                  // (uniform over the search's threads)
        double pot_scale = 1.0;
        int tcol = 0;
        if (a.mode == 0) {
            pot_scale = (double)a.incumbent[g];
        } else {
            const int s = clampi(a.sel[(size_t)g * 3 + 1], 0, a.S - 1);
            tcol = clampi(a.target[s], 0, a.R - 1);
        }
        constexpr int U = NT == kWave ? 1 : 4;     // clusters of a thread's candidates requested together
        const int n1 = n0 + ng;
        for (int pb = n0 + tid; pb < n1; pb += NT * U) {
            int jj[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int p = pb + u * NT;
                jj[u] = p < n1 ? a.assign[p] : -1;
            }
#pragma unroll 1
            for (int u = 0; u < U; ++u) {
                const int p = pb + u * NT;
                int j = jj[0];
#pragma unroll
                for (int v = 1; v < U; ++v) j = u == v ? jj[v] : j;
                if (j != I) continue;
                if (a.alive && !a.alive[p]) continue;
                const double key = sample_key(a, p, pot_scale, tcol);
                if (better(key, p, bk, bi)) { bk = key; bi = p; }
            }
        }
        auto merge = [&](double ok, int oi) {
            if (better(ok, oi, bk, bi)) { bk = ok; bi = oi; }
        };
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) merge(__shfl_xor(bk, o), __shfl_xor(bi, o));
        if constexpr (NT > kWave) {
            if ((tid & 63) == 0) { redk[tid >> 6] = bk; redi[tid >> 6] = bi; }
            __syncthreads();
            if (tid == 0)
                for (int w = 1; w < W; ++w) merge(redk[w], redi[w]);
        }
    }
    if (tid == 0) a.ksel[g] = bi == kNoCandidate ? -1 : bi;
}

}  // namespace

hipError_t launch_sample(const kb_batch& b, const SampleCall& c, hipStream_t st) {
    SampleArgs a = make_sample_args(b, c);
    // a batch of short searches only: a wave per search, one launch; a batch of several
    // searches with longer ones among them: both kernels, each skipping the other's searches
    // (an empty launch of the other kernel costs a few microseconds)
    const auto workgroup = [&](auto kern, int threads) {
        hipLaunchKernelGGL(kern, dim3((unsigned)b.G), dim3((unsigned)threads), 0, st, a);
        return hipGetLastError();
    };
    a.mixed = 0;
    if (b.Nmax > kShortSearch &&
        (b.Nmax <= kWideN || (b.Nmax <= kWideMembersN && b.Nmax <= (int64_t)kWideMembers * b.Kmax))) {
        if (b.Nmax > (b.G <= kWideFewG ? kWideFewN : kGroupN) && b.G <= kWideMaxG) return workgroup(sample_search<1024>, 1024);
        if (b.Nmax <= kGroupN && (b.G <= kGroupMaxG || b.N >= (int64_t)kGroupMeanN * b.G))
            return workgroup(sample_search<kThreads>, kThreads);
    }
    a.short_n = sample_short(b);
    a.mixed = b.Nmax > a.short_n && b.G > 1;
    if ((b.Nmax <= a.short_n || a.mixed) && b.G > 0) {
        hipLaunchKernelGGL(sample_search<kWave>, dim3((unsigned)((b.G + kWaves - 1) / kWaves)), dim3(kThreads), 0, st, a);
        if (!a.mixed) return hipGetLastError();
    }
    const unsigned ranges = (unsigned)((b.N + kSampleRange - 1) / kSampleRange);
    if (ranges) hipLaunchKernelGGL(sample_range, dim3(ranges), dim3(kThreads), 0, st, a);
    hipLaunchKernelGGL(sample_final, dim3((unsigned)((b.G + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, st, a);
    return hipGetLastError();
}

}  // namespace kb
