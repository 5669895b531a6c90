// Very short searches: batches in which every search has at most 64 candidates and 16
// clusters - the size of a search in the paper's own runs (Sec. 3.6: a frontier of a few
// dozen kernels, K = 3).  Such a search is one wave's work: lane l keeps candidate l's row in
// registers, centroids and fixed-point sums sit in the wave's own piece of LDS, and since
// nothing is shared with another wave no step needs a workgroup barrier or a block-wide
// reduction (what a step of a short search mostly consists of in the kernels that give a
// search a workgroup).
//
// What bounds it is one wave's chain of dependent instructions, so a Lloyd step is kept to the
// pieces that it cannot do without:
//   score    every lane forms the fp32 direct-difference distances of its candidate to all
//            centroids, two or four centroids at a time (independent chains); no distance bounds, since
//            a step without a move ends the search anyway (below) and in every other step some
//            lane has to score, which costs the wave the same as all lanes.
//   decide   relative error <= (D + 2) 2^-24, sums of non-negative terms: if the two smallest are
//            further apart than twice that bound allows, the smallest is the unique nearest
//            centroid; otherwise fp64, summed over the features in index order with separate
//            multiply and add (the plain definition), lowest index on ties.
//   move     a lane whose cluster changed moves its row between the fixed-point sums (integer
//            LDS atomics: any order gives the same sums).
//   renew    one lane per centroid coordinate: the mean, in fp64, rounded once to fp32.
// Same fixed-point grid and same rounding as in the workgroup kernels, so the same centroid bytes.
// A search stops at its first step without a move: such a step leaves sums, sizes and centroids
// as they were, so every later step would repeat it and all outputs are the same bytes as
// after the full count of steps.
//
// Measured against the form with distance bounds, four lanes per centroid and a centroid at a time
// in the score: ten steps of 183 searches of 12-41 candidates (D = 5, K = 3) 22.8 -> 12.1 us, the
// whole round 26.9 -> 14.3 us; rounds of 20000 searches of 1-40 112 -> 55 us, of 4000 searches of 64
// candidates, K = 16, D = 64 (20 steps) 334 -> 205 us, of 20000 with D = 32 474 -> 280 us.  What a lane
// could keep over the steps beside its row - its fixed-point image, its fp64 form - is formed
// again in each: kept, the registers leave one wave per SIMD (D = 32: three times as long).
#include "kb_cluster_dev.h"
#include "kb_ucb_dev.h"
#include "kb_wave_dev.h"
#include "kb_sample_dev.h"
#include <type_traits>

namespace kb {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;     // searches per workgroup
constexpr int kShortMaxN = 64, kShortMaxK = 16;

struct ShortArgs {
    int G, D, Ksum, Kmax;
    int64_t N;
    const int32_t* seg_off;
    const int32_t* koff;
    const float* X;
    const float* cent_init;     // NULL: the first K_g rows
    int iters;
    int guard;                  // leave searches with N_g < 2 K_g as they are (re-clustering rule of Alg. 1)
    int32_t* assign;
    float* cent_out;
    int32_t* counts;
    float* objective;
};

__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// A wave's piece of LDS.  NC: 16-byte pieces of a row.
struct ShortLds {
    size_t sums, cent, cnt, touched, total;
};
__host__ __device__ inline ShortLds short_lds_layout(int Kmax, int D, int NC) {
    ShortLds l;
    size_t off = 0;
    l.sums = off; off += (size_t)Kmax * (D | 1) * 8;      // odd row stride: clusters spread over the LDS banks
    off = (off + 15) & ~(size_t)15;
    l.cent = off; off += (size_t)((Kmax + 3) & ~3) * (4 * NC + 4) * 4;      // (rows are read four at a time)
    l.cnt = off;  off += (size_t)Kmax * 4;
    l.touched = off; off += (size_t)Kmax;                 // a byte per cluster: moves in this step
    l.total = (off + 15) & ~(size_t)15;
    return l;
}

// This lane's row, zero-padded to 4 NC features (a lane without a candidate holds zeros).
template <int NC>
__device__ __forceinline__ void short_row(const float* __restrict__ xr, int D, bool valid, float (&x)[4 * NC]) {
#pragma unroll
    for (int d = 0; d < 4 * NC; ++d) x[d] = 0.f;
    if (!valid) return;
    if (D >= 4) {
        float4 v[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = row_piece_load(xr, 4 * c, D);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const float4 w = row_piece_shift(v[c], 4 * c, D);
            x[4 * c] = w.x; x[4 * c + 1] = w.y; x[4 * c + 2] = w.z; x[4 * c + 3] = w.w;
        }
    } else {
        x[0] = xr[0];
        if (D > 1) x[1] = xr[1];
        if (D > 2) x[2] = xr[2];
    }
}

// The initial centroids - from memory, (init == NULL) the rows of the first K lanes, or (keep) the
// present ones -; sums and sizes 0.
template <int NC>
__device__ __forceinline__ void short_begin(const float* __restrict__ init, bool keep, int D, int ng, int K,
                                            const float (&x)[4 * NC], int lane, long long* sums, float* cent,
                                            int* cnt, unsigned char* touched) {
    constexpr int DP = 4 * NC + 4;
    if (keep) {
    } else if (init) {
        for (int i = lane; i < K * DP; i += kWave) {
            const int j = i / DP, d = i - j * DP;
            cent[i] = d < D ? init[(size_t)j * D + d] : 0.f;
        }
    } else {
        // (a malformed search of fewer candidates than clusters repeats its last row)
        for (int j = lane; j < K && (j == lane || lane == ng - 1); ++j) {
            if (j != lane && j < ng) continue;
            if (lane < ng) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    *reinterpret_cast<float4*>(cent + (size_t)j * DP + 4 * c) =
                        make_float4(x[4 * c], x[4 * c + 1], x[4 * c + 2], x[4 * c + 3]);
            }
        }
    }
    for (int i = lane; i < K * (D | 1); i += kWave) sums[i] = 0;
    if (lane < K) { cnt[lane] = 0; touched[lane] = 0; }
    wave_sync();
}

// `iters` >= 1 Lloyd steps of one search by one wave, from the centroids in `cent`; returns the
// objective (in every lane) and leaves new centroids, sizes and this lane's cluster.
template <int NC>
__device__ __forceinline__ float short_cluster(int iters, int D, int ng, int K, const float (&x)[4 * NC],
                                               bool valid, int lane, long long* sums, float* cent, int* cnt,
                                               unsigned char* touched, int& mine) {
    constexpr int DP = 4 * NC + 4;
    const int SP = D | 1;
    float am = 0.f;
    double tsq = 0.0;
#pragma unroll
    for (int d = 0; d < 4 * NC; ++d) {
        am = fmaxf(am, fabsf(x[d]));
        tsq = fma((double)x[d], (double)x[d], tsq);
    }
    am = wave_max_f(am);
    tsq = wave_sum_d(tsq);
    const int sh = fixed_shift(am, ng);
    const int fsh = sh - 32;
    const double inv = ldexp(1.0, -sh);
    const float eps = 2.f * (float)(D + 2) * 5.9604644775390625e-08f;
    // coordinate e of the centroids: feature e mod 2^lg of cluster e / 2^lg (2^lg >= D)
    const int lg = D > 1 ? 32 - __clz(D - 1) : 0;
    const int E = K << lg, dmask = (1 << lg) - 1;

    // Centroids scored side by side.  A step runs through its code once, so of rows of 17 to 48 features
    // only two: their chains keep the unit busy, and four rows' worth of unrolled code took longer to fetch
    // than it saved (four / two, 20 steps: 183 searches of 64 rows of 40, K = 16 82 / 75 us, 1500 of 17-64 rows of
    // 24, K = 6 33 / 28, 20000 of 12-64 rows of 32 123 / 109).  Of longer rows four: a round of 500 searches of 64
    // rows of 64, K = 16, ten steps 94 / 101.
    constexpr int U = NC == 8 || NC == 12 ? 2 : 4;
    mine = -1;
    double J = 0.0;
    for (int it = 0;; ++it) {
        float b32 = INFINITY, s32 = INFINITY;
        int bj = 0;
        for (int j0 = 0; j0 < K; j0 += U) {
            float acc[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                // (one address for all lanes; rows and centroids are zero-padded: the extra terms are +0.0)
                const float4* cr = reinterpret_cast<const float4*>(cent + (size_t)(j0 + u) * DP);
                float a0 = 0.f, a1 = 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const float4 cv = cr[c];
                    const float e0 = x[4 * c] - cv.x, e1 = x[4 * c + 1] - cv.y;
                    const float e2 = x[4 * c + 2] - cv.z, e3 = x[4 * c + 3] - cv.w;
                    a0 = fmaf(e0, e0, a0);
                    a1 = fmaf(e1, e1, a1);
                    a0 = fmaf(e2, e2, a0);
                    a1 = fmaf(e3, e3, a1);
                }
                acc[u] = a0 + a1;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float v = j0 + u < K ? acc[u] : INFINITY;
                const bool lt = v < b32;
                s32 = lt ? b32 : (v < s32 ? v : s32);
                bj = lt ? j0 + u : bj;
                b32 = lt ? v : b32;
            }
        }
        if (valid && !(s32 * (1.f - eps) > b32 * (1.f + eps) + 1.0e-35f)) {
            double bd = INFINITY;
            bj = 0;
            for (int j = 0; j < K; ++j) {
                // (Four of the centroid's values are under way.  With a trip to LDS for each, one step of 183
                // searches of 64 rows of 64, K = 16, some candidate in doubt, took 61 us, now 41.  The empty asm
                // keeps the fp64 forms of the row, twice its registers, from being held over the steps.)
                const float* cr = cent + (size_t)j * DP;
                float cv[4] = {cr[0], cr[1], cr[2], cr[3]};
                double acc = 0.0;
#pragma unroll
                for (int d = 0; d < 4 * NC; ++d) {
                    float xv = x[d];
                    asm volatile("" : "+v"(xv));
                    const double diff = __dsub_rn((double)xv, (double)cv[d & 3]);
                    acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                    cv[d & 3] = cr[d + 4 < 4 * NC ? d + 4 : d];
                }
                if (acc < bd) { bd = acc; bj = j; }
            }
        }
        const bool move = valid && bj != mine;
        const bool moved = __ballot(move) != 0;
        if (move) {
            // (formed again in every step: kept over the loop, the images take twice a row's registers)
            int f = fsh;
            asm volatile("" : "+v"(f));
            auto shift = [&](int d) __attribute__((always_inline)) {
                const long long q = to_fixed(x[d], f);
                atomicAdd(reinterpret_cast<unsigned long long*>(sums + bj * SP + d), (unsigned long long)q);
                if (it > 0)
                    atomicAdd(reinterpret_cast<unsigned long long*>(sums + mine * SP + d), (unsigned long long)-q);
            };
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (4 * c + 4 <= D) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) shift(4 * c + e);
                } else if (4 * c < D) {
                    shift(4 * c);
                    if (4 * c + 1 < D) shift(4 * c + 1);
                    if (4 * c + 2 < D) shift(4 * c + 2);
                }
            }
            atomicAdd(&cnt[bj], 1);
            if (it > 0) atomicSub(&cnt[mine], 1);
            touched[bj] = 1;
            if (it > 0) touched[mine] = 1;
            mine = bj;
        }
        wave_sync();
        const bool last = it == iters - 1 || !moved;
        if (last) {
            // Objective relative to the centroids c_j that entered this step: with S_j the exact sum
            // and n_j the size of cluster j, sum |x|^2 - sum_j c_j . (2 S_j - n_j c_j) in fp64;
            // member by member when the subtraction leaves less than 1e-7 of the first term.
            double part = 0.0;
            for (int e = lane; e < E; e += kWave) {
                const int j = e >> lg, d = e & dmask;
                if (d < D) {
                    const double cj = (double)cent[(size_t)j * DP + d];
                    const double Sj = (double)sums[j * SP + d] * inv;
                    part += cj * (2.0 * Sj - (double)cnt[j] * cj);
                }
            }
            J = tsq - wave_sum_d(part);
            if (!(J >= 1.0e-7 * tsq)) {
                double acc = 0.0;
                if (valid) {
                    const float4* cr = reinterpret_cast<const float4*>(cent + (size_t)mine * DP);
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        const float4 cv = cr[c];
                        const float e0 = x[4 * c] - cv.x, e1 = x[4 * c + 1] - cv.y;
                        const float e2 = x[4 * c + 2] - cv.z, e3 = x[4 * c + 3] - cv.w;
                        acc += (double)fmaf(e0, e0, fmaf(e1, e1, fmaf(e2, e2, e3 * e3)));
                    }
                }
                J = wave_sum_d(acc);
            }
            wave_sync();
        }
        if (moved) {
            // (an empty cluster keeps its centroid)
            if (E <= kWave) {
                // a lane per coordinate, reciprocals and all
                const int j = lane >> lg, d = lane & dmask;
                if (lane < E && d < D) {
                    const int c = cnt[j];
                    const double t = (double)sums[j * SP + d] * inv;
                    const double cd = (double)(c > 0 ? c : 1);
                    const float v = mean_f32(t, cd, 1.0 / cd);
                    if (c > 0) cent[(size_t)j * DP + d] = v;
                }
            } else {
                // several passes: a cluster's reciprocal is formed once, clusters without a move
                // are left out (a pass covers whole clusters)
                const int cl = lane < K ? cnt[lane] : 0;
                const double rl = 1.0 / (double)(cl > 0 ? cl : 1);
                const unsigned dirty = (unsigned)__ballot(lane < K && touched[lane] != 0);
                const int per = kWave >> lg;                 // clusters per pass (lg <= 6)
                for (int j0 = 0; j0 < K; j0 += per) {
                    if (!((dirty >> j0) & ((1u << per) - 1u))) continue;      // (uniform)
                    const int j = j0 + (lane >> lg), d = lane & dmask;
                    const double rc = __shfl(rl, j);
                    const int c = __shfl(cl, j);
                    if (j < K && d < D && c > 0) {
                        const double t = (double)sums[j * SP + d] * inv;
                        cent[(size_t)j * DP + d] = mean_f32(t, (double)c, rc);
                    }
                }
                if (lane < K) touched[lane] = 0;
            }
            wave_sync();
        }
        if (last) break;
    }
    return (float)J;
}

// What the whole-round kernel needs beyond the clustering arguments: the pruning
// step's inputs and outputs (Eq. 2 and the mask of Eq. 5) and the selection call.
struct ShortRound {
    const float* flops;
    const float* bytes;
    const float* incumbent;
    float peak_flops, peak_bw;
    float* bound;
    uint8_t* alive;
    UcbArgs u;
};

// bytes of the selection tables of a wave
__host__ __device__ inline size_t arm_lds_bytes(int Kmax, int S) {
    return ((size_t)Kmax * S * 12 + (size_t)Kmax * 12 + 15) & ~(size_t)15;
}

constexpr int kHeldS = 8;      // strategies whose visits and rewards a lane holds from the start of the call

// ROUND: the whole round of the search in this one wave - the roofline bound and the
// mask of every candidate first (the same correctly rounded divisions and strict
// compare as the pruning kernel), the clustering, then the cluster-arm statistics
// from the lanes' own clusters (integer LDS atomics, as in the selection kernel, so
// the same tables), scores and selection.  (The host takes this path with a.iters >= 1
// and a.guard = 0.)  Everything that comes from memory is requested before the clustering: on
// fresh inputs a trip to memory costs as much as two steps.
template <int NC, bool ROUND>
__device__ __forceinline__ void short_search(const ShortArgs& a, const ShortRound* rd, unsigned char* smem) {
    constexpr int DP = 4 * NC + 4;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = (int)blockIdx.x * kWaves + wv;
    if (g >= a.G) return;                 // (a whole wave leaves: nothing in this kernel waits for another wave)
    const int D = a.D;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (K > a.Kmax) K = a.Kmax;
    if (ng > kShortMaxN) ng = kShortMaxN;   // (the host launches this kernel only for such batches)
    const bool valid = lane < ng;
    const size_t row = (size_t)n0 + (valid ? lane : 0);
    float x[4 * NC];
    short_row<NC>(a.X + row * D, D, valid && K > 0, x);
    bool live = true;                     // this lane's candidate passed the pruning step
    float rbound = 0.f;
    int hv[kHeldS];
    float hr[kHeldS];
    long long tg = 1;
    bool held = false;
    if constexpr (ROUND) {
        const UcbArgs& u = rd->u;
        float fl = 0.f, by = 0.f;
        if (valid) { fl = rd->flops[row]; by = rd->bytes[row]; }
        const float inc = rd->incumbent[g];
        tg = u.t[g];
        held = u.S <= kHeldS;             // (uniform)
        if (held && valid) {
#pragma unroll
            for (int s = 0; s < kHeldS; ++s) {
                if (s < u.S) { hv[s] = u.visits[row * u.S + s]; hr[s] = u.rsum[row * u.S + s]; }
            }
        }
        if (valid) {
            const float t_compute = fl / rd->peak_flops;
            const float t_memory = by / rd->peak_bw;
            rbound = t_compute > t_memory ? t_compute : t_memory;
            live = rbound < inc;
            rd->bound[row] = rbound;
            rd->alive[row] = live ? 1 : 0;
        }
    }
    if (ng <= 0 || K <= 0) {
        if (lane == 0 && a.iters > 0 && a.objective) a.objective[g] = 0.f;
        if constexpr (ROUND) {
            if (lane < 3) rd->u.sel[(size_t)g * 3 + lane] = -1;
        }
        return;
    }
    if (a.guard && ng < 2 * K) return;

    const ShortLds L = short_lds_layout(a.Kmax, D, NC);
    const size_t arm = ROUND ? arm_lds_bytes(a.Kmax, rd->u.S) : 0;
    unsigned char* base = smem + (size_t)wv * (L.total + arm);
    long long* sums = reinterpret_cast<long long*>(base + L.sums);      // [Kmax][D | 1]
    float* cent = reinterpret_cast<float*>(base + L.cent);              // [Kmax][DP]
    int* cnt = reinterpret_cast<int*>(base + L.cnt);                    // [Kmax]
    unsigned char* touched = base + L.touched;                          // [Kmax]

    short_begin<NC>(a.cent_init ? a.cent_init + (size_t)k0 * D : nullptr, false, D, ng, K, x, lane, sums, cent, cnt, touched);
    int mine = 0;
    if (a.iters > 0) {
        const float J = short_cluster<NC>(a.iters, D, ng, K, x, valid, lane, sums, cent, cnt, touched, mine);
        if (lane == 0) a.objective[g] = J;
        if (valid) a.assign[row] = mine;
        if (lane < K) a.counts[k0 + lane] = cnt[lane];
    }
    for (int i = lane; i < K * D; i += kWave) {
        const int j = i / D, d = i - j * D;
        a.cent_out[(size_t)(k0 + j) * D + d] = cent[(size_t)j * DP + d];
    }

    if constexpr (ROUND) {
        const UcbArgs& u = rd->u;
        const int S = u.S, KS = K * S;
        unsigned long long* R = reinterpret_cast<unsigned long long*>(base + L.total);       // [Kmax*S]
        unsigned long long* kmin = R + (size_t)a.Kmax * S;                                   // [Kmax]
        unsigned* Ncnt = reinterpret_cast<unsigned*>(kmin + a.Kmax);                         // [Kmax*S]
        unsigned* nalive = Ncnt + (size_t)a.Kmax * S;                                        // [Kmax]
        for (int i = lane; i < KS; i += kWave) { R[i] = 0ull; Ncnt[i] = 0u; }
        if (lane < K) { kmin[lane] = ~0ull; nalive[lane] = 0u; }
        wave_sync();
        if (valid && live) {      // (iters >= 1: every candidate has a cluster)
            if (held) {
#pragma unroll
                for (int s = 0; s < kHeldS; ++s) {
                    if (s < S) {
                        atomicAdd(&Ncnt[mine * S + s], (unsigned)hv[s]);
                        atomicAdd(&R[mine * S + s], reward_fixed(hr[s]));
                    }
                }
                ucb_count_candidate(lane, mine, rbound, nalive, kmin);
            } else {
                ucb_add_candidate(u, row, lane, mine, rbound, Ncnt, R, nalive, kmin);
            }
        }
        wave_sync();
        ucb_finish<kWave>(u, g, n0, k0, K, Ncnt, R, nalive, kmin, nullptr, nullptr, lane, tg);
    }
}

template <int NC>
__global__ void __launch_bounds__(kThreads) cluster_wave_kernel(ShortArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    short_search<NC, false>(a, nullptr, smem);
}

template <int NC>
__global__ void __launch_bounds__(kThreads) round_wave_kernel(ShortArgs a, ShortRound rd) {
    extern __shared__ __align__(16) unsigned char smem[];
    short_search<NC, true>(a, &rd, smem);
}

// ---- whole iterations of Alg. 1 in one launch ------------------------------------------
// Nothing of an iteration - re-clustering, representatives and mask every tau-th time, masked
// selection, draw of k_t, statistics update - touches another search, so a search runs all of
// them on its own, in a workgroup of four waves.  The first wave carries the search: its rows,
// centroids, clusters and cluster arms (A arms per lane) stay in registers and LDS from the first
// iteration to the last, the history (visits and reward sums) in LDS, written back at the end.  The other three form the Gumbel variates of the draws, which depend on
// nothing but the draw's number and the candidate, kAhead iterations ahead in one of two buffers;
// one barrier per kAhead iterations hands them over.  What is left of an iteration for the first
// wave is the dependent chain score - argmax - key - argmax - one cell of the history: no
// logarithm, no trip to memory, no shuffle through LDS.
//
// What bounds it is one wave's chain of fp64 instructions, 1.1 us an iteration.  With eight launches and
// a wave per search twenty iterations of 183 searches of 12-41 candidates (D = 5, K = 3, S = 6) with two
// re-clusterings took 122 us, now 48 us.
//
// NW = 1: one wave does both, the variates of the next kAhead iterations after every kAhead.  A search
// takes a fifth longer, but no wave waits for another: beyond the searches that fit the chip with
// four waves each (three workgroups per compute unit with rows of at most 16 features and an arm per
// lane, one otherwise) the batch is done sooner (four waves / one, us: 768 searches above 56 / 68, 4000, D = 12,
// K = 6, S = 10 400 / 222; 300 of 40-64 candidates, D = 40, K = S = 16 373 / 304).
constexpr int kAhead = 8;
constexpr int kIterateMaxR = 8, kIterateMaxArms = 256;
constexpr size_t kIterateMaxLds = 40 * 1024, kLdsPerUnit = 160 * 1024;
constexpr int kComputeUnits = 256;

struct IterateArgs {
    ShortArgs c;
    UcbArgs u;                  // sel unused
    SampleArgs s;               // sel, ksel unused
    int rounds, tau, first_due, warm;     // the first re-clustering comes before iteration first_due (tau <= 0: never)
    unsigned long long draw0;
    const float* reward;        // [rounds][G]
    const uint8_t* ok;          // [rounds][G]
    int32_t* visits;
    float* rsum;
    int64_t* t;
    int32_t* sel_log;           // [rounds][G][3]
    int32_t* ksel_log;          // [rounds][G]
    uint8_t* M;
    int32_t* nvalid;
    int32_t* rep;
    float* radius;
    int Nmax;
};

struct IterateLds {
    ShortLds c;
    size_t gum, pot, R, gmin, gmax, N, grep, vis, rs, total;
};
__host__ __device__ inline IterateLds iterate_lds_layout(int Kmax, int D, int NC, int S, int R, int Nmax) {
    IterateLds l;
    l.c = short_lds_layout(Kmax, D, NC);
    size_t off = l.c.total;
    l.gum = off;  off += (size_t)2 * kAhead * Nmax * 8;
    l.pot = off;  off += (size_t)R * Nmax * 8;           // (theta_sat - h) / tau, [resource][candidate]
    l.R = off;    off += (size_t)Kmax * S * 8;
    l.gmin = off; off += (size_t)Kmax * 8;
    l.gmax = off; off += (size_t)Kmax * 8;
    l.N = off;    off += (size_t)Kmax * S * 4;
    l.grep = off; off += (size_t)Kmax * 4;
    l.vis = off;  off += (size_t)Nmax * S * 4;
    l.rs = off;   off += (size_t)Nmax * S * 4;
    l.total = (off + 15) & ~(size_t)15;
    return l;
}

constexpr int kNoMember = 0x7fffffff;

template <int NC, int A, int NW>
__global__ void __launch_bounds__(NW * kWave, NW == 1 ? (NC <= 4 ? 4 : 2) : 1) iterate_kernel(IterateArgs r) {
    constexpr int kThreads = NW * kWave;
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int DP = 4 * NC + 4;
    const ShortArgs& a = r.c;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = NW > 1 ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    const int g = (int)blockIdx.x;
    const int D = a.D, S = r.u.S, T = r.rounds, NM = r.Nmax;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    const bool due = r.tau > 0 && r.first_due < T;         // some iteration of this launch re-clusters
    if (K > a.Kmax) K = a.Kmax;
    if (ng > NM) ng = NM;                 // (LDS is sized from the host copies)
    if (ng <= 0 || K <= 0) {
        // nothing to choose from (the workgroup leaves as a whole)
        for (int it = tid; it < T; it += kThreads) {
            const size_t at = (size_t)it * a.G + g;
            for (int q = 0; q < 3; ++q) r.sel_log[at * 3 + q] = -1;
            r.ksel_log[at] = -1;
        }
        if (due) {
            for (int i = tid; i < K; i += kThreads) { r.rep[k0 + i] = -1; r.radius[k0 + i] = 0.f; }
            for (int i = tid; i < K * S; i += kThreads) r.M[(size_t)k0 * S + i] = 0;
            if (tid == 0) { a.objective[g] = 0.f; r.nvalid[g] = 0; }
        }
        if (tid == 0) r.t[g] += T;
        return;
    }
    const int KS = K * S;
    const IterateLds L = iterate_lds_layout(a.Kmax, D, NC, S, r.s.R, NM);
    long long* sums = reinterpret_cast<long long*>(smem + L.c.sums);
    float* cent = reinterpret_cast<float*>(smem + L.c.cent);
    int* cnt = reinterpret_cast<int*>(smem + L.c.cnt);
    unsigned char* touched = smem + L.c.touched;
    double* gum = reinterpret_cast<double*>(smem + L.gum);              // [2][kAhead][NM]
    double* pot = reinterpret_cast<double*>(smem + L.pot);              // [R][NM]
    unsigned long long* tR = reinterpret_cast<unsigned long long*>(smem + L.R);          // [KS]
    unsigned long long* gmin = reinterpret_cast<unsigned long long*>(smem + L.gmin);     // [K]
    unsigned long long* gmax = reinterpret_cast<unsigned long long*>(smem + L.gmax);     // [K]
    unsigned* tN = reinterpret_cast<unsigned*>(smem + L.N);             // [KS]
    int* grep = reinterpret_cast<int*>(smem + L.grep);                  // [K]
    int* vis = reinterpret_cast<int*>(smem + L.vis);                    // [ng][S]
    float* rs = reinterpret_cast<float*>(smem + L.rs);                  // [ng][S]

    // the first wave's candidate and arms
    const bool valid = wv == 0 && lane < ng;
    const size_t row = (size_t)n0 + (valid ? lane : 0);
    float x[4 * NC];
    bool live = false;
    int raw = 0;                          // this lane's cluster as the arrays have it
    long long t = 0;
    int cl[A], st[A], col[A];             // cluster, strategy and resource of this lane's arms
    bool allowed[A];                      // by the mask
    if (wv == 0) {
        short_row<NC>(a.X + row * D, D, valid && due, x);
        live = valid && (!r.u.alive || r.u.alive[row] != 0);
        if (valid) raw = r.u.assign[row];
        t = r.t[g];
#pragma unroll
        for (int q = 0; q < A; ++q) {
            const int i = lane + q * kWave;
            cl[q] = i / S;
            st[q] = i - cl[q] * S;
            col[q] = clampi(r.s.target[st[q]], 0, r.s.R - 1);
            allowed[q] = i < KS && r.M[(size_t)k0 * S + i] != 0;
        }
    }
    {
        const int R = r.s.R;
        for (int i = tid; i < ng * S; i += kThreads) {
            vis[i] = r.visits[(size_t)n0 * S + i];
            rs[i] = r.rsum[(size_t)n0 * S + i];
        }
        for (int i = tid; i < ng * R; i += kThreads) {
            const int k = i / R;
            pot[(i - k * R) * NM + k] = ((double)r.s.theta_sat - (double)r.s.h[(size_t)n0 * R + i]) / r.s.tau;
        }
    }
    if (NW > 1) __syncthreads();
    else wave_sync();

    unsigned n[A];
    unsigned long long Rw[A];
    double mean[A];
    bool arm[A];
    int mine = 0;                         // this lane's cluster, 0 where the array names none of the search
    double lnl = 0.0;                     // lane l: ln t, reward and verification of iteration 64 i + l
    float rwl = 0.f;
    int okl = 0;
    int rd = 0;
    int64_t next = r.tau > 0 ? r.first_due : (int64_t)T;
    bool fresh = true, have = false;      // tables to be built; centroids in LDS
    // the last iteration, for the arms' outputs
    double u[A];
    int bf = -1;
    bool updated = false;
    double rw = 0.0;
    int log_I = -1, log_s = -1, log_lead = -1, log_k = -1;     // lane l: the log of iteration 64 i + l
    const int chunks = (T + kAhead - 1) / kAhead;
    auto variates = [&](int c, int first, int stride) __attribute__((always_inline)) {
        double* out = gum + (c & 1) * kAhead * NM;
        const int left = T - c * kAhead, m = (left < kAhead ? left : kAhead) * ng;
        for (int i = first; i < m; i += stride) {
            const int it = i / ng, k = i - it * ng;
            const unsigned long long draw = r.draw0 + (unsigned long long)(c * kAhead + it);
            out[it * NM + k] = gumbel_variate(r.s.seed_lo, r.s.seed_hi, (unsigned)draw, (unsigned)(draw >> 32),
                                              n0 + k);
        }
    };
    for (int c = 0; c <= chunks; ++c) {
        if (NW > 1 && wv > 0) {
            if (c < chunks) variates(c, tid - kWave, kThreads - kWave);
        } else {
            const int stop = c * kAhead < T ? c * kAhead : T;
            const double* gb = gum + ((c - 1) & 1) * kAhead * NM;
            while (true) {
                if (fresh) {
                    fresh = false;
                    if (rd == next) {
                        next += r.tau;
                        if (ng >= 2 * K) {
                            short_begin<NC>(r.warm ? a.cent_out + (size_t)k0 * D : nullptr, r.warm && have, D, ng, K,
                                            x, lane, sums, cent, cnt, touched);
                            const float J = short_cluster<NC>(a.iters, D, ng, K, x, valid, lane, sums, cent, cnt,
                                                              touched, raw);
                            if (lane == 0) a.objective[g] = J;
                            if (valid) a.assign[row] = raw;
                            if (lane < K) a.counts[k0 + lane] = cnt[lane];
                            for (int i = lane; i < K * D; i += kWave) {
                                const int j = i / D;
                                a.cent_out[(size_t)k0 * D + i] = cent[(size_t)j * DP + i - j * D];
                            }
                        } else if (!have) {
                            short_begin<NC>(a.cent_out + (size_t)k0 * D, false, D, ng, K, x, lane, sums, cent, cnt,
                                            touched);
                        }
                        have = true;
                        // representatives and radii: fp64 distances as the definition forms them
                        const int j = raw >= 0 && raw < K ? raw : 0;
                        if (lane < K) { gmin[lane] = ~0ull; gmax[lane] = 0ull; grep[lane] = kNoMember; }
                        wave_sync();
                        double acc = 0.0;
                        const float* cr = cent + (size_t)j * DP;
#pragma unroll
                        for (int d = 0; d < 4 * NC; ++d) {
                            float xv = x[d];
                            asm volatile("" : "+v"(xv));          // (its fp64 form is not kept over the loop)
                            const double diff = __dsub_rn((double)xv, (double)cr[d]);
                            acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                        }
                        const unsigned long long bits = (unsigned long long)__double_as_longlong(acc);
                        if (valid) { atomicMin(&gmin[j], bits); atomicMax(&gmax[j], bits); }
                        wave_sync();
                        if (valid && bits == gmin[j]) atomicMin(&grep[j], lane);
                        wave_sync();
                        if (lane < K) {
                            r.rep[k0 + lane] = grep[lane] == kNoMember ? -1 : n0 + grep[lane];
                            r.radius[k0 + lane] = (float)sqrt(__longlong_as_double((long long)gmax[lane]));
                        }
                        // Eq. 5: h < theta_sat exactly where theta_sat - h is above 0
                        int nv = 0;
#pragma unroll
                        for (int q = 0; q < A; ++q) {
                            const int i = lane + q * kWave;
                            allowed[q] = false;
                            if (i < KS) {
                                const int rp = grep[cl[q]];
                                allowed[q] = rp != kNoMember && pot[col[q] * NM + rp] > 0.0;
                                r.M[(size_t)k0 * S + i] = allowed[q] ? 1 : 0;
                            }
                            nv += __popcll(__ballot(allowed[q]));
                        }
                        if (lane == 0) r.nvalid[g] = nv;
                    }
                    // tables of the history under the present clusters
                    mine = raw >= 0 && raw < K ? raw : 0;
                    for (int i = lane; i < KS; i += kWave) { tR[i] = 0ull; tN[i] = 0u; }
                    wave_sync();
                    if (live) {
                        for (int s = 0; s < S; ++s) {
                            atomicAdd(&tN[mine * S + s], (unsigned)vis[lane * S + s]);
                            atomicAdd(&tR[mine * S + s], reward_fixed(rs[lane * S + s]));
                        }
                    }
                    wave_sync();
#pragma unroll
                    for (int q = 0; q < A; ++q) arm[q] = false;
                    for (int j = 0; j < K; ++j) {
                        const bool any = __ballot(live && mine == j) != 0;
#pragma unroll
                        for (int q = 0; q < A; ++q) arm[q] = cl[q] == j ? any : arm[q];
                    }
#pragma unroll
                    for (int q = 0; q < A; ++q) {
                        const int i = lane + q * kWave;
                        n[q] = i < KS ? tN[i] : 0u;
                        Rw[q] = i < KS ? tR[i] : 0ull;
                        mean[q] = ucb_mean(r.u, n[q], Rw[q]);
                        arm[q] = i < KS && arm[q] && allowed[q];
                    }
                }
                if (rd >= stop) break;

                const bool last = rd == T - 1;
                const int l64 = rd & 63;
                if (l64 == 0) {
                    const long long tt = t + rd + lane;
                    lnl = log((double)(tt < 1 ? 1 : tt));
                    if (rd + lane < T) {
                        const size_t al = (size_t)(rd + lane) * a.G + g;
                        rwl = r.reward[al];
                        okl = r.ok[al];
                    }
                }
                const double lnt = lane_d(lnl, l64);
                double bu = -INFINITY;
                bf = -1;
#pragma unroll
                for (int q = 0; q < A; ++q) {
                    u[q] = ucb_index(r.u, n[q], arm[q], lnt, mean[q]);
                    if (arm[q] && (bf < 0 || u[q] > bu)) { bu = u[q]; bf = lane + q * kWave; }
                }
                wave_best_arm<(A > 1)>(bu, bf);
                bf = __builtin_amdgcn_readfirstlane(bf);
                int I = -1, s = -1, lead = -1, k = -1;
                if (bf >= 0) {
                    const int ow = bf & 63;
                    int tc = 0;
#pragma unroll
                    for (int q = 0; q < A; ++q) {
                        if (bf >> 6 == q) {
                            I = __builtin_amdgcn_readlane(cl[q], ow);
                            s = __builtin_amdgcn_readlane(st[q], ow);
                            tc = __builtin_amdgcn_readlane(col[q], ow);
                        }
                    }
                    lead = __ffsll((long long)__ballot(live && mine == I)) - 1;
                    const bool member = live && raw == I;
                    double key = -INFINITY;
                    if (member) {
                        key = pot[tc * NM + lane] + gb[(rd & (kAhead - 1)) * NM + lane];
                        // A key that is not a number loses to every other, except that of the first
                        // member, which then stays chosen: the result of scanning the members in order.
                        if (!(key == key)) key = lane == lead ? INFINITY : -INFINITY;
                    }
                    k = wave_top_lane(key, member);           // (lowest candidate on ties)
                }
                const bool log_here = lane == l64;
                log_I = log_here ? I : log_I;
                log_s = log_here ? s : log_s;
                log_lead = log_here ? lead : log_lead;
                log_k = log_here ? k : log_k;
                updated = k >= 0 && __builtin_amdgcn_readlane(okl, l64) != 0;
                if (updated) {
                    rw = (double)lane_f(rwl, l64);
                    const int cell = k * S + s;
                    const float r_old = rs[cell];
                    const float r_new = (float)((double)r_old + rw);
                    if (lane == 0) { vis[cell] += 1; rs[cell] = r_new; }
                    wave_sync();
                    if (!last) {
                        const unsigned long long step = reward_fixed(r_new) - reward_fixed(r_old);
#pragma unroll
                        for (int q = 0; q < A; ++q) {
                            if (lane + q * kWave == bf) {
                                n[q] += 1u;
                                Rw[q] += step;
                                mean[q] = ucb_mean(r.u, n[q], Rw[q]);
                            }
                        }
                    }
                }
                if (l64 == 63 || last) {
                    // 64 iterations' logs, one per lane
                    const int it = rd - l64 + lane;
                    if (it <= rd) {
                        const size_t at = (size_t)it * a.G + g;
                        r.sel_log[at * 3 + 0] = log_I;
                        r.sel_log[at * 3 + 1] = log_s;
                        r.sel_log[at * 3 + 2] = log_lead >= 0 ? n0 + log_lead : -1;
                        r.ksel_log[at] = log_k >= 0 ? n0 + log_k : -1;
                    }
                }
                ++rd;
                fresh = rd < T && rd == next;
            }
            if (NW == 1 && c < chunks) variates(c, lane, kWave);
        }
        if (NW > 1) __syncthreads();
        else wave_sync();
    }
    if (wv == 0) {
        // counts, means and scores as the last iteration saw them, with its update of one arm
#pragma unroll
        for (int q = 0; q < A; ++q) {
            const int i = lane + q * kWave;
            if (i < KS) {
                const size_t o = (size_t)k0 * S + i;
                const bool up = updated && i == bf;
                const int nn = (int32_t)n[q] + (up ? 1 : 0);
                const double mo = (double)(float)mean[q];
                r.u.Ncs[o] = nn;
                r.u.mu[o] = up ? (float)(mo + (rw - mo) / ((double)nn + (double)r.u.prior_n)) : (float)mean[q];
                r.u.ucb[o] = (float)u[q];
            }
        }
    }
    for (int i = tid; i < ng * S; i += kThreads) {
        r.visits[(size_t)n0 * S + i] = vis[i];
        r.rsum[(size_t)n0 * S + i] = rs[i];
    }
    if (tid == 0) r.t[g] = t + T;
}

// 16-byte pieces of a row that a kernel is compiled for, from the feature count
int row_pieces(int D) {
    const int n = (D + 3) / 4;
    return n <= 4 ? (n < 2 ? 2 : n) : n <= 8 ? 8 : n <= 12 ? 12 : 16;
}

// go(std::integral_constant<int, NC>) for the batch's NC
template <class F>
hipError_t with_pieces(int D, F go) {
    switch (row_pieces(D)) {
        case 2: return go(std::integral_constant<int, 2>{});
        case 3: return go(std::integral_constant<int, 3>{});
        case 4: return go(std::integral_constant<int, 4>{});
        case 8: return go(std::integral_constant<int, 8>{});
        case 12: return go(std::integral_constant<int, 12>{});
        default: return go(std::integral_constant<int, 16>{});
    }
}

template <class K, class... A>
hipError_t launch(K kern, unsigned grid, unsigned threads, size_t lds, hipStream_t st, const A&... args) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, st, args...);
    return hipGetLastError();
}

int kmax_of(const kb_batch& b) { return b.Kmax > 0 ? b.Kmax : 1; }
unsigned wave_grid(const kb_batch& b) { return (unsigned)((b.G + kWaves - 1) / kWaves); }

ShortArgs short_args(const kb_batch& b, const ClusterCall& c) {
    ShortArgs a;
    a.G = b.G; a.D = b.D; a.Ksum = b.Ksum; a.Kmax = kmax_of(b); a.N = b.N;
    a.seg_off = b.seg_off; a.koff = b.koff; a.X = c.X; a.cent_init = c.cent_init;
    a.iters = c.iters; a.guard = c.guard; a.assign = c.assign; a.cent_out = c.cent_out;
    a.counts = c.counts; a.objective = c.objective;
    return a;
}

}  // namespace

bool cluster_wave_per_search(const kb_batch& b, int scorer) {
    return scorer == KB_SCORER_DEFAULT && b.Nmax <= kShortMaxN && b.Kmax <= kShortMaxK;
}

hipError_t launch_cluster_wave(const kb_batch& b, const ClusterCall& c, hipStream_t st) {
    if (!cluster_wave_per_search(b, c.scorer) || c.mixed) return hipErrorInvalidValue;
    const ShortArgs a = short_args(b, c);
    return with_pieces(b.D, [&](auto nc) {
        constexpr int NC = decltype(nc)::value;
        return launch(cluster_wave_kernel<NC>, wave_grid(b), kThreads, kWaves * short_lds_layout(a.Kmax, a.D, NC).total, st, a);
    });
}

// A batch of searches of at most 64 candidates and 16 clusters each, in the default
// mode: the whole round (Sec. 3.5: prune, cluster, select) is one launch, a wave per
// search.  (The selection tables share the wave's piece of LDS; strategy counts that
// would leave fewer than two workgroups per compute unit take the three-stage path.)
bool round_in_one_launch(const kb_batch& b, int scorer) {
    if (!cluster_wave_per_search(b, scorer)) return false;
    return kWaves * (short_lds_layout(kmax_of(b), b.D, row_pieces(b.D)).total + arm_lds_bytes(kmax_of(b), b.S)) <=
           64 * 1024;
}

hipError_t launch_round_wave(const kb_batch& b, const ClusterCall& c, const UcbCall& uc,
                             const float* flops, const float* bytes, const float* incumbent,
                             float peak_flops, float peak_bw, float* bound, uint8_t* alive,
                             hipStream_t st) {
    if (!round_in_one_launch(b, c.scorer) || c.mixed || c.guard || c.iters < 1 || c.cent_init)
        return hipErrorInvalidValue;
    const ShortArgs a = short_args(b, c);
    ShortRound rd;
    rd.flops = flops; rd.bytes = bytes; rd.incumbent = incumbent;
    rd.peak_flops = peak_flops; rd.peak_bw = peak_bw; rd.bound = bound; rd.alive = alive;
    rd.u = make_ucb_args(b, uc);
    return with_pieces(b.D, [&](auto nc) {
        constexpr int NC = decltype(nc)::value;
        const size_t lds = kWaves * (short_lds_layout(a.Kmax, a.D, NC).total + arm_lds_bytes(a.Kmax, b.S));
        return launch(round_wave_kernel<NC>, wave_grid(b), kThreads, lds, st, a, rd);
    });
}

// `kb_iterate` on a batch of such searches can be one launch per 1024 iterations, provided that the
// resources and strategies are few enough for the tables of a search (a lane holds one or four
// cluster arms; at least four workgroups' tables fit a compute unit).
static size_t iterate_lds(const kb_batch& b, int R) {
    return iterate_lds_layout(kmax_of(b), b.D, row_pieces(b.D), b.S, R, b.Nmax).total;
}
static bool iterate_fits(const kb_batch& b, int scorer, int R) {
    return cluster_wave_per_search(b, scorer) && b.G > 0 && R <= kIterateMaxR &&
           (int64_t)kmax_of(b) * b.S <= kIterateMaxArms && b.Nmax > 0 && iterate_lds(b, R) <= kIterateMaxLds;
}

// Whether that is faster than the launches one by one (their time / one launch's, us).  What it saves grows with
// the iterations; a re-clustering, three launches more, counts as four of them: w in all.
//   Up to one search per compute unit: always (1.1 to 2.5 times over 1500 random shapes).
//   As long as the chip holds all searches at once - by LDS, and by registers 16 waves per unit with rows
//     of up to 16 features, else 8 -: always (1.0 to 2.0 times), except that the four arms per lane spill beside
//     short rows: beyond five searches per unit from w = 15 on (1500 searches of 12-41, K = 6, S = 16: one iteration
//     37 / 40, four 47.5 / 47.7, twenty 136 / 113; 768 of 40-64, D = 40, K = S = 16, twenty 308 / 302).
//   Beyond, the launches keep more waves in flight than the tables leave room for, and with an arm per lane the
//     line falls with the waves that a unit holds: at 16 always (20000 of 12-41, K = 3, S = 6, one iteration
//     113 / 108), at 8 from w = 20 on (4000 of 40-64, D = 3, S = 16, ten iterations 99 / 113, twenty 198 / 200; of 64
//     rows of 64, S = 2, ten iterations with four re-clusterings 715 / 541).  With four arms the launches win (12000
//     of 40-64, D = 16, K = 16, S = 10, ten iterations 307 / 542) but for rows of 17 to 32 features, which
//     neither spill nor fill the registers, from w = 15 on if LDS holds as many (4000 of 40-64, D = 32, K = 10, S = 8,
//     ten iterations with four re-clusterings 372 / 264).
constexpr int kIterateWaves = 16, kIterateWavesLong = 8, kIterateShortRows = 16, kIterateMiddleRows = 32;
bool iterate_in_one_launch(const kb_batch& b, int scorer, int R, int64_t rounds, int64_t reclusterings) {
    if (!iterate_fits(b, scorer, R)) return false;
    if (b.G <= kComputeUnits) return true;
    const bool short_rows = b.D <= kIterateShortRows, one_arm = kmax_of(b) * b.S <= kWave;
    const int by_lds = (int)(kLdsPerUnit / ((iterate_lds(b, R) + 1279) / 1280 * 1280));
    const int by_registers = short_rows ? kIterateWaves : kIterateWavesLong;
    const int waves = by_lds < by_registers ? by_lds : by_registers;
    const int64_t w = rounds + 4 * reclusterings;
    if (b.G <= kComputeUnits * waves) return one_arm || !short_rows || b.G <= 5 * kComputeUnits || w >= 15;
    if (one_arm) return 2 * w >= 5 * (kIterateWaves - waves);
    return !short_rows && b.D <= kIterateMiddleRows && waves == by_registers && w >= 15;
}

hipError_t launch_iterate(const kb_batch& b, const ClusterCall& c, const UcbCall& uc, const SampleCall& sc,
                          const RoundsCall& rc, const IterateCall& ic, hipStream_t st) {
    if (!iterate_fits(b, c.scorer, sc.R) || c.mixed || uc.bound || !sc.h || rc.rounds < 1)
        return hipErrorInvalidValue;
    IterateArgs r;
    r.c = short_args(b, c);
    r.u = make_ucb_args(b, uc);
    r.s = make_sample_args(b, sc);
    r.rounds = rc.rounds; r.tau = ic.tau; r.first_due = ic.first_due; r.warm = ic.warm;
    r.draw0 = sc.draw; r.reward = rc.reward; r.ok = rc.ok; r.visits = rc.visits; r.rsum = rc.rsum; r.t = rc.t;
    r.sel_log = rc.sel_log; r.ksel_log = rc.ksel_log;
    r.M = ic.M; r.nvalid = ic.nvalid; r.rep = ic.rep; r.radius = ic.radius;
    r.Nmax = b.Nmax;
    return with_pieces(b.D, [&](auto nc) {
        constexpr int NC = decltype(nc)::value;
        const size_t lds = iterate_lds(b, sc.R);
        const auto go = [&](auto kern, int waves) { return launch(kern, (unsigned)b.G, waves * kWave, lds, st, r); };
        const bool one = r.c.Kmax * b.S <= kWave;
        const bool few = b.G <= (one && NC <= 4 ? 768 : kComputeUnits);      // (the line: see above)
        return few ? (one ? go(iterate_kernel<NC, 1, 4>, 4) : go(iterate_kernel<NC, 4, 4>, 4))
                   : (one ? go(iterate_kernel<NC, 1, 1>, 1) : go(iterate_kernel<NC, 4, 1>, 1));
    });
}

}  // namespace kb
