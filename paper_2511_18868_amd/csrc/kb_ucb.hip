// Cluster-arm statistics, masked UCB index and arm selection (Eq. 6, Sec. 3.4).
//
// One workgroup per search streams the search's visits / reward-sum rows once
// (flat, coalesced 16-byte loads) and scatters them into K x S accumulators in
// LDS keyed by the candidate's cluster.  All accumulators are integers - visit
// counts as they are, reward sums in 2^-30 fixed point (a cluster's reward sum
// is below its visit count, which is below 2^31) - so the LDS atomics commute
// and the statistics are bit-identical from run to run.  The per-cluster "most
// headroom" candidate is a 64-bit atomic min over (ordered bound bits, index).
// Scores are formed in fp64 from the accumulators, compared in fp64, and
// rounded to fp32 on output.
#include "kb_internal.h"
#include "kb_ucb_dev.h"
#include "kb_sample_dev.h"
#include <cmath>

namespace kb {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kWideThreads = 1024;
constexpr int kUcbHead = (8 + 4) * kWideThreads / kWave;      // reduction scratch ahead of the tables in LDS
constexpr int kUcbLong = 16384;     // searches longer than this are cut into candidate ranges

// Scatter the visits / reward sums of the alive candidates [q0, q1) of a search
// (indices local to the search) into K x S tables keyed by cluster.
//
// A candidate's two rows are cut into pieces of E values - 16 bytes when S is a
// multiple of 4, 8 bytes when it is even, single values otherwise (the rows start at
// multiples of 4 S bytes, so that is the alignment they have) - and T threads, the
// next power of two at or above the number of pieces, share a candidate: the
// thread-to-piece mapping is fixed, so no index arithmetic per step (with S = 6, the
// paper's own count, a loop over single values that divides every index by S ran at a
// quarter of the rate of S = 8).  Four candidates per thread are in flight: mask and
// cluster first, then the rows of the alive ones, then the atomics.
// EXACT: the pieces of a row are a power of two in number, one per thread of its group
// (no idle threads and no loop over pieces).
template <int E, bool EXACT, int NT>
__device__ __forceinline__ void ucb_accumulate_pieces(const UcbArgs& a, int n0, int K, int q0, int q1,
                                                      unsigned* Ncnt, unsigned long long* R,
                                                      unsigned* nalive, unsigned long long* kmin) {
    const int tid = threadIdx.x;
    const int S = a.S;
    const int pieces = S / E;
    int T = 1;
    while (T < pieces && T < NT) T <<= 1;
    const int rpp = NT / T;                   // candidates per pass of the workgroup
    const int sq = tid & (T - 1), row = tid / T;
    constexpr int U = 4;
    for (int pb = q0 + row; pb < q1; pb += rpp * U) {
        bool al[U];
        int jj[U];
        float bd[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = pb + u * rpp;
            const int pc = p < q1 ? p : q1 - 1;
            al[u] = (a.alive ? a.alive[(size_t)n0 + pc] != 0 : true) && p < q1;
            jj[u] = a.assign[(size_t)n0 + pc];
            bd[u] = a.bound ? a.bound[(size_t)n0 + pc] : 0.f;
        }
        const auto piece = [&](int c) {
            int v[U][E];
            float r[U][E];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int p = pb + u * rpp;
#pragma unroll
                for (int e = 0; e < E; ++e) { v[u][e] = 0; r[u][e] = 0.f; }
                if (al[u]) {
                    const size_t at = ((size_t)n0 + p) * pieces + c;
                    if constexpr (E == 4) {
                        const int4 vv = reinterpret_cast<const int4*>(a.visits)[at];
                        const float4 rv = reinterpret_cast<const float4*>(a.rsum)[at];
                        v[u][0] = vv.x; v[u][1] = vv.y; v[u][2] = vv.z; v[u][3] = vv.w;
                        r[u][0] = rv.x; r[u][1] = rv.y; r[u][2] = rv.z; r[u][3] = rv.w;
                    } else if constexpr (E == 2) {
                        const int2 vv = reinterpret_cast<const int2*>(a.visits)[at];
                        const float2 rv = reinterpret_cast<const float2*>(a.rsum)[at];
                        v[u][0] = vv.x; v[u][1] = vv.y;
                        r[u][0] = rv.x; r[u][1] = rv.y;
                    } else {
                        v[u][0] = a.visits[at];
                        r[u][0] = a.rsum[at];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (!al[u]) continue;
                const int j = (jj[u] >= 0 && jj[u] < K) ? jj[u] : 0;
                unsigned* nc = Ncnt + (size_t)j * S + c * E;
                unsigned long long* rr = R + (size_t)j * S + c * E;
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    atomicAdd(nc + e, (unsigned)v[u][e]);
                    atomicAdd(rr + e, reward_fixed(r[u][e]));
                }
                if (c == 0) {         // the thread with a row's first piece also counts the candidate
                    atomicAdd(&nalive[j], 1u);
                    const unsigned long long key =
                        ((unsigned long long)ordered_bits(bd[u]) << 32) | (unsigned)(pb + u * rpp);
                    atomicMin(&kmin[j], key);
                }
            }
        };
        if constexpr (EXACT) {
            piece(sq);
        } else {
            for (int c = sq; c < pieces; c += T) piece(c);     // (one round unless a row has more than NT pieces)
        }
    }
}


// E, EXACT: how the rows are cut (ucb_accumulate_pieces); instantiations of their own,
// so that each form has the registers it needs and no more (in one kernel the forms for
// odd strategy counts raised the count from 64 to 99 and halved the resident waves of all)
template <int E, bool EXACT, int NT>
__global__ void __launch_bounds__(NT) ucb_kernel(UcbArgs a) {
    constexpr int kThreads = NT;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int S = a.S;

    int g = a.order ? a.order[blockIdx.x] : (int)blockIdx.x;
    g = clampi(g, 0, a.G - 1);
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (K > a.Kmax) K = a.Kmax;
    if (ng <= 0 || K <= 0) {
        if (tid < 3) a.sel[(size_t)g * 3 + tid] = -1;
        return;
    }
    if (a.mixed && ng > a.longer) return;     // the range kernels take this search
    const int KS = K * S;

    double* redv = reinterpret_cast<double*>(smem);                                      // [waves]
    int* redi = reinterpret_cast<int*>(smem + 8 * (kWideThreads / kWave));               // [waves]
    unsigned long long* R = reinterpret_cast<unsigned long long*>(smem + kUcbHead);      // [Kmax*S]
    unsigned long long* kmin = R + (size_t)a.Kmax * S;                                   // [Kmax]
    unsigned* Ncnt = reinterpret_cast<unsigned*>(kmin + a.Kmax);                         // [Kmax*S]
    unsigned* nalive = Ncnt + (size_t)a.Kmax * S;                                        // [Kmax]

    for (int i = tid; i < KS; i += kThreads) { R[i] = 0ull; Ncnt[i] = 0u; }
    for (int i = tid; i < K; i += kThreads) { kmin[i] = ~0ull; nalive[i] = 0u; }
    __syncthreads();

    ucb_accumulate_pieces<E, EXACT, kThreads>(a, n0, K, 0, ng, Ncnt, R, nalive, kmin);
    __syncthreads();

    if (a.keep) {
        // (a search is owned by this workgroup: plain stores)
        for (int i = tid; i < KS; i += kThreads) {
            a.gN[(size_t)k0 * S + i] = Ncnt[i];
            a.gR[(size_t)k0 * S + i] = R[i];
        }
        for (int i = tid; i < K; i += kThreads) { a.gnalive[k0 + i] = nalive[i]; a.gkmin[k0 + i] = kmin[i]; }
    }
    ucb_finish<kThreads>(a, g, n0, k0, K, Ncnt, R, nalive, kmin, redv, redi, tid, a.t[g]);
}


// ---- short searches: a wave per search, four searches per workgroup, no barrier.
// A lane owns a candidate and adds its two rows to the wave's own tables; the same
// integer tables as above, so the same scores and the same selection.
__global__ void __launch_bounds__(kThreads) ucb_wave(UcbArgs a, int per) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = (int)blockIdx.x * kWaves + wv;
    if (g >= a.G) return;                 // (a whole wave leaves: no wave waits for another in this kernel)
    const int S = a.S;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (K > a.Kmax) K = a.Kmax;
    if (ng <= 0 || K <= 0) {
        if (lane < 3) a.sel[(size_t)g * 3 + lane] = -1;
        return;
    }
    const int KS = K * S;
    unsigned char* base = smem + (size_t)wv * per;
    unsigned long long* R = reinterpret_cast<unsigned long long*>(base);                 // [Kmax*S]
    unsigned long long* kmin = R + (size_t)a.Kmax * S;                                   // [Kmax]
    unsigned* Ncnt = reinterpret_cast<unsigned*>(kmin + a.Kmax);                         // [Kmax*S]
    unsigned* nalive = Ncnt + (size_t)a.Kmax * S;                                        // [Kmax]
    for (int i = lane; i < KS; i += kWave) { R[i] = 0ull; Ncnt[i] = 0u; }
    for (int i = lane; i < K; i += kWave) { kmin[i] = ~0ull; nalive[i] = 0u; }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (int p = lane; p < ng; p += kWave) {
        if (a.alive && !a.alive[(size_t)n0 + p]) continue;
        int j = a.assign[(size_t)n0 + p];
        j = (j >= 0 && j < K) ? j : 0;
        ucb_add_candidate(a, (size_t)n0 + p, p, j, a.bound ? a.bound[(size_t)n0 + p] : 0.f, Ncnt, R, nalive, kmin);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    ucb_finish<kWave>(a, g, n0, k0, K, Ncnt, R, nalive, kmin, nullptr, nullptr, lane, a.t[g]);
}


// ---- several iterations of a search in one launch ----------------------------------
// Between two re-clusterings an iteration of Alg. 1 is selection, draw of k_t and
// statistics update, each a few microseconds of launch and one search's worth of work;
// an iteration touches nothing of another search.  So a search runs all of them on its
// own: the cluster-arm tables are aggregated once into LDS (integer tables: advanced by
// the update they equal a fresh aggregation bit for bit), the alive members of every
// cluster are listed once, and an iteration is then a pass over the K S arms, a draw over
// the members of the chosen cluster, and one cell of the tables - two barriers'
// worth of latency, bound by the dependent chain (logarithms, square roots, the gathers of
// h and of the updated cell) and no longer by launches.  Scores, means and counts of
// all arms are written in the last iteration only; the ones before would be overwritten.
//
// Launch by launch an iteration of 183 paper-size searches took 13.5 us and one of 512
// searches of 64-4096 candidates 34 us; twenty and ten such iterations with their two
// re-clusterings went 331 -> 147 us and 1779 -> 1422 us.
//
// NT threads per search, a workgroup each; or, for short searches, one wave (NT = 64) per
// search and four searches per workgroup, without any barrier.
struct RoundsArgs {
    UcbArgs u;
    SampleArgs s;               // .sel / .ksel unused (the logs below); draw number of the first iteration
    int rounds;
    unsigned long long draw0;
    const float* reward;        // [rounds][G]
    const uint8_t* ok;          // [rounds][G]
    int32_t* visits;            // the history (u.visits, u.rsum), advanced
    float* rsum;
    int64_t* t;
    int32_t* sel_log;           // [rounds][G][3]
    int32_t* ksel_log;          // [rounds][G]
    int Nmax;
    int means;                  // 1: the arms' mean rewards are kept in LDS beside the tables
};

struct RoundsLds {
    size_t R, mean, kmin, N, nalive, first, cursor, target, valid, member, total;
};
__host__ __device__ inline RoundsLds rounds_lds_layout(int Kmax, int S, int Nmax, bool means) {
    const size_t KS = (size_t)Kmax * S;
    RoundsLds l;
    size_t off = 0;
    l.R = off;      off += KS * 8;
    l.mean = off;   off += means ? KS * 8 : 0;
    l.kmin = off;   off += (size_t)Kmax * 8;
    l.N = off;      off += KS * 4;
    l.nalive = off; off += (size_t)Kmax * 4;
    l.first = off;  off += ((size_t)Kmax + 1) * 4;      // first member of every cluster in `member`
    l.cursor = off; off += (size_t)Kmax * 4;
    l.target = off; off += (size_t)S * 4;
    l.valid = off;  off += (KS + 3) & ~(size_t)3;       // arm allowed by mask and members
    l.member = off; off += (size_t)Nmax * 2;            // alive members grouped by cluster (N_g <= 16384)
    l.total = (off + 15) & ~(size_t)15;
    return l;
}

template <int NT>
__device__ __forceinline__ void rounds_sync() {
    if constexpr (NT > kWave) __syncthreads();
    else __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// E = 0: a lane owns a whole candidate in the aggregation (the wave form)
template <int E, bool EXACT, int NT>
__device__ __forceinline__ void rounds_search(const RoundsArgs& r, int g, unsigned char* smem, double* redv,
                                              int* redi, int tid) {
    constexpr int NW = NT / kWave;
    const UcbArgs& a = r.u;
    const int S = a.S;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (K > a.Kmax) K = a.Kmax;
    if (ng > r.Nmax) ng = r.Nmax;       // (LDS is sized from the host copy)
    if (ng <= 0 || K <= 0) {
        for (int it = tid; it < r.rounds; it += NT) {
            const size_t at = (size_t)it * a.G + g;
            for (int q = 0; q < 3; ++q) r.sel_log[at * 3 + q] = -1;
            r.ksel_log[at] = -1;
        }
        if (tid == 0) r.t[g] += r.rounds;
        return;
    }
    const int KS = K * S;
    const RoundsLds L = rounds_lds_layout(a.Kmax, S, r.Nmax, r.means != 0);
    double* mean = r.means ? reinterpret_cast<double*>(smem + L.mean) : nullptr;
    unsigned long long* R = reinterpret_cast<unsigned long long*>(smem + L.R);
    unsigned long long* kmin = reinterpret_cast<unsigned long long*>(smem + L.kmin);
    unsigned* Ncnt = reinterpret_cast<unsigned*>(smem + L.N);
    unsigned* nalive = reinterpret_cast<unsigned*>(smem + L.nalive);
    int* first = reinterpret_cast<int*>(smem + L.first);
    int* cursor = reinterpret_cast<int*>(smem + L.cursor);
    int* target = reinterpret_cast<int*>(smem + L.target);
    unsigned char* valid = smem + L.valid;
    unsigned short* member = reinterpret_cast<unsigned short*>(smem + L.member);

    for (int i = tid; i < KS; i += NT) { R[i] = 0ull; Ncnt[i] = 0u; }
    for (int i = tid; i < K; i += NT) { kmin[i] = ~0ull; nalive[i] = 0u; cursor[i] = 0; }
    for (int i = tid; i < S; i += NT) target[i] = clampi(r.s.target[i], 0, r.s.R - 1);
    rounds_sync<NT>();
    // tables of the history, and the sizes of the member lists
    if constexpr (E == 0) {
        for (int p = tid; p < ng; p += NT) {
            if (a.alive && !a.alive[(size_t)n0 + p]) continue;
            int j = a.assign[(size_t)n0 + p];
            j = (j >= 0 && j < K) ? j : 0;
            ucb_add_candidate(a, (size_t)n0 + p, p, j, 0.f, Ncnt, R, nalive, kmin);
        }
    } else {
        ucb_accumulate_pieces<E, EXACT, NT>(a, n0, K, 0, ng, Ncnt, R, nalive, kmin);
    }
    for (int p = tid; p < ng; p += NT) {
        const int j = a.assign[(size_t)n0 + p];
        if (j >= 0 && j < K && (!a.alive || a.alive[(size_t)n0 + p])) atomicAdd(&cursor[j], 1);
    }
    long long t = a.t[g];
    rounds_sync<NT>();
    for (int i = tid; i < KS; i += NT) {
        valid[i] = nalive[i / S] > 0u && (!a.M || a.M[(size_t)k0 * S + i] != 0);
        if (mean) mean[i] = ucb_mean(a, Ncnt[i], R[i]);
    }
    if (tid < kWave) {
        // exclusive prefix sums of the sizes (K <= 256: four clusters per lane)
        int c[4], sum = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) { c[e] = 4 * tid + e < K ? cursor[4 * tid + e] : 0; sum += c[e]; }
        int inc = sum;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int up = __shfl_up(inc, o);
            if (tid >= o) inc += up;
        }
        int at = inc - sum;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int j = 4 * tid + e;
            if (j < K) { first[j] = at; cursor[j] = at; at += c[e]; if (j == K - 1) first[K] = at; }
        }
    }
    rounds_sync<NT>();
    for (int p = tid; p < ng; p += NT) {
        const int j = a.assign[(size_t)n0 + p];
        if (j >= 0 && j < K && (!a.alive || a.alive[(size_t)n0 + p]))
            member[atomicAdd(&cursor[j], 1)] = (unsigned short)p;    // (in any order: the draw compares indices)
    }
    rounds_sync<NT>();

    double lnl = 0.0;             // lane l: ln t of iteration 64 i + l
    for (int it = 0; it < r.rounds; ++it) {
        const bool last = it == r.rounds - 1;
        const size_t at = (size_t)it * a.G + g;
        const float reward = r.reward[at];           // (requested before they are needed)
        const bool ok = r.ok[at] != 0;
        if ((it & 63) == 0) {
            const long long tg = t + it + (tid & 63);
            lnl = log((double)(tg < 1 ? 1 : tg));
        }
        const double lnt = lane_d(lnl, it & 63);
        double bu = -INFINITY;
        int bf = -1;
        for (int i = tid; i < KS; i += NT) {
            const unsigned n = Ncnt[i];
            const double m = mean ? mean[i] : ucb_mean(a, n, R[i]);
            const double u = ucb_index(a, n, valid[i] != 0, lnt, m);
            if (last) {
                const size_t o = (size_t)k0 * S + i;
                a.Ncs[o] = (int32_t)n;
                a.mu[o] = (float)m;
                a.ucb[o] = (float)u;
            }
            if (valid[i] && (bf < 0 || u > bu)) { bu = u; bf = i; }
        }
        // argmax, lowest flat index on ties; every thread gets it
        auto merge_arm = [&](double ou, int of) {
            if (of >= 0 && (bf < 0 || ou > bu || (ou == bu && of < bf))) { bu = ou; bf = of; }
        };
        wave_best_arm<true>(bu, bf);
        if constexpr (NT > kWave) {
            if ((tid & 63) == 0) { redv[tid >> 6] = bu; redi[tid >> 6] = bf; }
            __syncthreads();
            bu = redv[0]; bf = redi[0];
            for (int w = 1; w < NW; ++w) merge_arm(redv[w], redi[w]);
        } else {
            // scores that are not numbers (c = +inf at t = 1) leave the lanes with different
            // arms: lane 0 decides, as in a selection call of its own
            bf = __builtin_amdgcn_readfirstlane(bf);
        }
        const int I = bf >= 0 ? bf / S : -1, s = bf >= 0 ? bf - I * S : -1;
        if (tid == 0) {
            r.sel_log[at * 3 + 0] = I;
            r.sel_log[at * 3 + 1] = s;
            r.sel_log[at * 3 + 2] = bf >= 0 ? n0 + (int)(unsigned)(kmin[I] & 0xffffffffull) : -1;
        }
        int k = kNoCandidate;
        if (I >= 0) {                                // (uniform over the search's threads)
            // A key that is not a number loses to every other, except that of the first
            // member, which then stays chosen: the result of scanning the members in order.
            const int lead = n0 + (int)(unsigned)(kmin[I] & 0xffffffffull);
            SampleArgs sa = r.s;
            const unsigned long long draw = r.draw0 + (unsigned long long)it;
            sa.draw_lo = (unsigned)draw; sa.draw_hi = (unsigned)(draw >> 32);
            const int tcol = target[s];
            const int m1 = first[I + 1];
            double bk = 0.0;
            for (int q = first[I] + tid; q < m1; q += NT) {
                const int p = n0 + member[q];
                double key = sample_key(sa, p, 1.0, tcol);
                if (!(key == key)) key = p == lead ? INFINITY : -INFINITY;
                if (better(key, p, bk, k)) { bk = key; k = p; }
            }
            auto merge_key = [&](double ok2, int oi) {
                if (better(ok2, oi, bk, k)) { bk = ok2; k = oi; }
            };
            {
                // (keys are numbers by now)
                const int top = wave_top_lane(bk, k != kNoCandidate);
                if (top >= 0) {
                    const double best = lane_d(bk, top);
                    k = wave_min_i(k != kNoCandidate && bk == best ? k : kNoCandidate);
                    bk = best;
                }
            }
            if constexpr (NT > kWave) {
                // (slots of their own: the first reduction's may still be read)
                if ((tid & 63) == 0) { redv[NW + (tid >> 6)] = bk; redi[NW + (tid >> 6)] = k; }
                __syncthreads();
                bk = redv[NW]; k = redi[NW];
                for (int w = 1; w < NW; ++w) merge_key(redv[NW + w], redi[NW + w]);
            }
        }
        if (tid == 0) r.ksel_log[at] = k == kNoCandidate ? -1 : k;
        // statistics update (as in update_stats_kernel): by the thread that wrote the arm's
        // score, so that its stores to an arm and to the arm's cells stay in order
        if (ok && k != kNoCandidate && tid == bf % NT) {
            const double rw = (double)reward;
            if (last) {
                const size_t arm = (size_t)k0 * S + bf;
                const int nn = (int32_t)Ncnt[bf] + 1;
                const double m = (double)a.mu[arm];
                a.Ncs[arm] = nn;
                a.mu[arm] = (float)(m + (rw - m) / ((double)nn + (double)a.prior_n));
            }
            const size_t cell = (size_t)k * S + s;
            r.visits[cell] += 1;
            const float r_old = r.rsum[cell];
            const float r_new = (float)((double)r_old + rw);
            r.rsum[cell] = r_new;
            Ncnt[bf] += 1u;
            R[bf] += reward_fixed(r_new) - reward_fixed(r_old);
            if (mean) mean[bf] = ucb_mean(a, Ncnt[bf], R[bf]);
        }
        rounds_sync<NT>();
    }
    if (tid == 0) r.t[g] = t + r.rounds;
}

template <int E, bool EXACT, int NT>
__global__ void __launch_bounds__(NT) rounds_kernel(RoundsArgs r) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double redv[2 * NT / kWave];
    __shared__ int redi[2 * NT / kWave];
    int g = r.u.order ? r.u.order[blockIdx.x] : (int)blockIdx.x;
    g = clampi(g, 0, r.u.G - 1);
    rounds_search<E, EXACT, NT>(r, g, smem, redv, redi, (int)threadIdx.x);
}

__global__ void __launch_bounds__(kThreads) rounds_wave(RoundsArgs r, int per) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = (int)blockIdx.x * kWaves + wv;
    if (g >= r.u.G) return;               // (a whole wave leaves: no wave waits for another in this kernel)
    rounds_search<0, false, kWave>(r, g, smem + (size_t)wv * per, nullptr, nullptr, (int)(threadIdx.x & 63));
}

// ---- searches too long for one workgroup: partial tables per candidate range,
// ---- merged in global memory with integer atomics (still order-independent)

__global__ void __launch_bounds__(kThreads) ucb_zero(UcbArgs a) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = t0; i < (int64_t)a.Ksum * a.S; i += stride) { a.gN[i] = 0u; a.gR[i] = 0ull; }
    for (int64_t i = t0; i < a.Ksum; i += stride) { a.gnalive[i] = 0u; a.gkmin[i] = ~0ull; }
}

template <int E, bool EXACT>
__global__ void __launch_bounds__(kThreads) ucb_partial(UcbArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    const int S = a.S;
    const int64_t r0 = (int64_t)blockIdx.x * a.range;
    if (r0 >= a.N) return;
    const int64_t r1 = r0 + a.range < a.N ? r0 + a.range : a.N;
    unsigned long long* R = reinterpret_cast<unsigned long long*>(smem + kUcbHead);
    unsigned long long* kmin = R + (size_t)a.Kmax * S;
    unsigned* Ncnt = reinterpret_cast<unsigned*>(kmin + a.Kmax);
    unsigned* nalive = Ncnt + (size_t)a.Kmax * S;
    // largest g with seg_off[g] <= r0
    int lo = 0, hi = a.G;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)a.seg_off[mid] <= r0) lo = mid; else hi = mid;
    }
    const auto mine = [&](int n0, int ng, int k0, int K) {
        return n0 >= r1 || (ng > 0 && K > 0 && !(a.mixed && ng <= a.longer));
    };
    for (int g = lo; (g = next_search(a.seg_off, a.koff, g, a.G, a.N, a.Ksum, mine)) < a.G; ++g) {
        int n0, ng, k0, K;
        search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
        if (K > a.Kmax) K = a.Kmax;
        if (n0 >= r1) break;
        if (ng <= 0 || K <= 0) continue;
        if (a.mixed && ng <= a.longer) continue;     // one workgroup takes this search whole
        const int64_t q0 = r0 > n0 ? r0 : n0;
        const int64_t q1 = r1 < (int64_t)n0 + ng ? r1 : (int64_t)n0 + ng;
        if (q0 >= q1) continue;
        const int KS = K * S;
        for (int i = tid; i < KS; i += kThreads) { R[i] = 0ull; Ncnt[i] = 0u; }
        for (int i = tid; i < K; i += kThreads) { kmin[i] = ~0ull; nalive[i] = 0u; }
        __syncthreads();
        ucb_accumulate_pieces<E, EXACT, kThreads>(a, n0, K, (int)(q0 - n0), (int)(q1 - n0), Ncnt, R, nalive, kmin);
        __syncthreads();
        for (int i = tid; i < KS; i += kThreads) {
            if (Ncnt[i]) atomicAdd(&a.gN[(size_t)k0 * S + i], Ncnt[i]);
            if (R[i]) atomicAdd(&a.gR[(size_t)k0 * S + i], R[i]);
        }
        for (int i = tid; i < K; i += kThreads) {
            if (nalive[i]) {
                atomicAdd(&a.gnalive[k0 + i], nalive[i]);
                atomicMin(&a.gkmin[k0 + i], kmin[i]);
            }
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kThreads) ucb_final(UcbArgs a) {
    __shared__ double redv[kWaves];
    __shared__ int redi[kWaves];
    const int g = blockIdx.x;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (K > a.Kmax) K = a.Kmax;
    if (a.mixed && ng <= a.longer) return;       // (uniform) done by ucb_kernel, empty searches included
    if (ng <= 0 || K <= 0) {
        if (threadIdx.x < 3) a.sel[(size_t)g * 3 + threadIdx.x] = -1;
        return;
    }
    ucb_finish<kThreads>(a, g, n0, k0, K, a.gN + (size_t)k0 * a.S, a.gR + (size_t)k0 * a.S,
                         a.gnalive + k0, a.gkmin + k0, redv, redi, (int)threadIdx.x, a.t[g]);
}

}  // namespace

// bytes of one search's tables in ucb_wave
static int wave_table_bytes(const kb_batch& b) {
    const size_t kmax = b.Kmax > 0 ? b.Kmax : 1;
    return (int)(((kmax * b.S * 12 + kmax * 12) + 15) & ~(size_t)15);
}

bool ucb_wave_per_search(const kb_batch& b) {
    return b.G > 0 && b.Nmax <= kShortSearch && (size_t)wave_table_bytes(b) * kWaves <= 64 * 1024;
}

// Few searches get 1024 threads each, so that one with a compute unit to itself keeps more rows in
// flight (256 / 1024 threads, us: one search of 4096 candidates, S = 16 36.9 / 16.6, of 16000 147 / 50, of
// 300 5.2 / 4.8; 256 of 512, S = 32 15.0 / 10.2, 200 of 4096 90 / 36, 512 of 1000 32.6 / 30.4, 300 of 1900, S = 6
// 25.9 / 21.0); beyond the compute units only for long ones (512 of 600, S = 3 11.2 / 12.4, of 512, S = 32
// 18.0 / 18.5), and where there is little to a row - its pieces (ucb_accumulate_pieces) a power of two, a thread
// each - only from 6000 pieces on (512 of 201-1118, S = 1 11.4 / 13.9, 512 of 1227-2752, S = 8 29 / 34) or beside
// much shorter ones, when the longest decide (300 of 22-2853, S = 8 21.9 / 15.7, 512 of 134-5551, S = 1 21.3 / 17.5).
constexpr int kUcbWideFewG = 256, kUcbWideMaxG = 512, kUcbWideMinN = 1000, kUcbWidePieces = 6000;

// pieces of a candidate's row, see ucb_accumulate_pieces
static int ucb_pieces(int S) { return (S & 3) == 0 ? S / 4 : (S & 1) == 0 ? S / 2 : S; }

namespace {

// the aggregation kernels in the form that fits the strategy count (see ucb_accumulate_pieces)
template <int E, bool EXACT, int NT>
hipError_t launch_search_kernel_nt(const UcbArgs& a, size_t lds, hipStream_t st) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(ucb_kernel<E, EXACT, NT>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((ucb_kernel<E, EXACT, NT>), dim3((unsigned)a.G), dim3(NT), lds, st, a);
    return hipGetLastError();
}
template <int E, bool EXACT>
hipError_t launch_search_kernel(const UcbArgs& a, bool wide, size_t lds, hipStream_t st) {
    return wide ? launch_search_kernel_nt<E, EXACT, kWideThreads>(a, lds, st)
                : launch_search_kernel_nt<E, EXACT, kThreads>(a, lds, st);
}
template <int E, bool EXACT>
hipError_t launch_range_kernel(const UcbArgs& a, unsigned ranges, size_t lds, hipStream_t st) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(ucb_partial<E, EXACT>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((ucb_partial<E, EXACT>), dim3(ranges), dim3(kThreads), lds, st, a);
    return hipGetLastError();
}
// form 0: 16-byte pieces, a power of two of them per row; 1: 16-byte pieces; 2: 8-byte; 3: single values
int row_form(int S) {
    if ((S & 3) == 0) {
        const int pieces = S >> 2;
        return ((pieces & (pieces - 1)) == 0 && pieces <= kThreads) ? 0 : 1;
    }
    return (S & 1) == 0 ? 2 : 3;
}
hipError_t launch_search_kernel(const UcbArgs& a, bool wide, size_t lds, hipStream_t st) {
    switch (row_form(a.S)) {
        case 0: return launch_search_kernel<4, true>(a, wide, lds, st);
        case 1: return launch_search_kernel<4, false>(a, wide, lds, st);
        case 2: return launch_search_kernel<2, false>(a, wide, lds, st);
        default: return launch_search_kernel<1, false>(a, wide, lds, st);
    }
}
hipError_t launch_range_kernel(const UcbArgs& a, unsigned ranges, size_t lds, hipStream_t st) {
    switch (row_form(a.S)) {
        case 0: return launch_range_kernel<4, true>(a, ranges, lds, st);
        case 1: return launch_range_kernel<4, false>(a, ranges, lds, st);
        case 2: return launch_range_kernel<2, false>(a, ranges, lds, st);
        default: return launch_range_kernel<1, false>(a, ranges, lds, st);
    }
}

}  // namespace

// (Scores that are not numbers - possible only with an infinite parameter - have no order, and the arm chosen
// among them follows from how the arms are dealt to the threads: always 256 then, so that a search's choice
// does not depend on how many others the batch holds.)
static bool ucb_wide(const kb_batch& b, const UcbArgs& a) {
    if (!std::isfinite(a.c) || !std::isfinite(a.prior_n) || !std::isfinite(a.prior_mu)) return false;
    if (b.G <= kUcbWideFewG) return true;
    const int pieces = ucb_pieces(b.S);
    return b.G <= kUcbWideMaxG && b.Nmax >= kUcbWideMinN &&
           ((pieces & (pieces - 1)) != 0 || (int64_t)b.Nmax * pieces >= kUcbWidePieces ||
            3 * (int64_t)b.Nmax * b.G >= 8 * b.N);
}

// Long searches: ranges that give every compute unit a workgroup, of 512 candidates at least and not
// below a quarter of a search's cluster arms, whose tables every range adds to the global ones.  (Ranges
// of 8192 / these, the kernels of a call, us: one search of 20000, S = 32, K = 64 164 / 28, S = 3, K = 4 74 / 16,
// of 200000, S = 8, K = 100 57 / 22, three of 60000, S = 32, K = 64 174 / 45, one of 2^20, S = 4, K = 256 37 / 30.)
// In a batch of a few searches the ranges pay from 6000 candidates on (one workgroup of 1024 threads /
// ranges: one of 16000 50 / 17.6, of 8000 18.0 / 15.4, of 4096 16.0 / 18.0), where a row is one piece later (S = 1: one of
// 6277 12.8 / 14.1, of 8201 15.9 / 14.8, two of up to 9307 16.6 / 17.4, of up to 10834 19.5 / 17.0; S = 4: eight of up to
// 9616 31 / 36, of up to 14890 51 / 27).
constexpr int kUcbFewG = 8, kUcbFewN = 6000, kUcbRanges = 256, kUcbRangeMin = 512, kUcbRangeMax = 8192;
constexpr int kUcbFewOneN = 8000, kUcbFewOnesN = 12000;
static int ucb_few_n(const kb_batch& b) {
    return ucb_pieces(b.S) > 1 ? kUcbFewN : b.G == 1 ? kUcbFewOneN : kUcbFewOnesN;
}

hipError_t launch_ucb(const kb_batch& b, const UcbCall& c, hipStream_t st) {
    UcbArgs a = make_ucb_args(b, c);
    const size_t lds = kUcbHead + (size_t)a.Kmax * b.S * 12 + (size_t)a.Kmax * 12;
    if (lds > 160 * 1024) return hipErrorInvalidValue;
    if (c.from_tables) {
        if (!c.gN) return hipErrorInvalidValue;
        hipLaunchKernelGGL(ucb_final, dim3((unsigned)b.G), dim3(kThreads), 0, st, a);
        return hipGetLastError();
    }
    if (c.keep_tables && !c.gN) return hipErrorInvalidValue;
    a.keep = c.keep_tables ? 1 : 0;
    // (the tables in global memory are there unless the caller has none to give)
    const bool can = c.gN && b.G <= kUcbFewG, few = can && b.Nmax > ucb_few_n(b);
    if (c.chunked || few) {
        if (!c.gN) return hipErrorInvalidValue;
        a.longer = can ? kUcbFewN : kUcbLong;        // (with the launches of the ranges paid for)
        a.range = kUcbRangeMin;
        while (a.range < kUcbRangeMax &&
               (b.N > (int64_t)kUcbRanges * a.range || (int64_t)a.Kmax * b.S > 4 * a.range))
            a.range *= 2;
        // long searches: candidate ranges -> partial tables -> global tables -> scores;
        // in a batch of several searches the short ones get a workgroup each as usual
        const size_t items = (size_t)b.Ksum * b.S;
        unsigned zb = (unsigned)((items + kThreads - 1) / kThreads);
        if (zb > 4096u) zb = 4096u;
        if (zb == 0) zb = 1;
        hipLaunchKernelGGL(ucb_zero, dim3(zb), dim3(kThreads), 0, st, a);
        if (b.G > 1) {
            a.mixed = 1;
            const hipError_t e = launch_search_kernel(a, ucb_wide(b, a), lds, st);
            if (e != hipSuccess) return e;
        }
        const unsigned ranges = (unsigned)((b.N + a.range - 1) / a.range);
        if (ranges) {
            const hipError_t e = launch_range_kernel(a, ranges, lds, st);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(ucb_final, dim3((unsigned)b.G), dim3(kThreads), 0, st, a);
        return hipGetLastError();
    }
    // a batch of short searches only: a wave per search (if four searches' tables fit the
    // 64 KB of LDS a kernel gets without asking); needs no scheduling order
    if (ucb_wave_per_search(b)) {
        if (a.keep) return hipErrorInvalidValue;      // ucb_wave leaves no tables (rounds_in_one_launch holds for
                                                      // every such batch, so kb_iterate does not ask for them)
        const int per = wave_table_bytes(b);
        hipLaunchKernelGGL(ucb_wave, dim3((unsigned)((b.G + kWaves - 1) / kWaves)), dim3(kThreads),
                           (size_t)per * kWaves, st, a, per);
        return hipGetLastError();
    }
    return launch_search_kernel(a, ucb_wide(b, a), lds, st);
}

static size_t rounds_lds(const kb_batch& b, bool means = false) {
    return rounds_lds_layout(b.Kmax > 0 ? b.Kmax : 1, b.S, b.Nmax, means).total;
}
static bool rounds_wave_per_search(const kb_batch& b) {
    return b.Nmax <= kShortSearch && rounds_lds(b) * kWaves <= 64 * 1024;
}
// One workgroup draws over all members of the chosen cluster.  Where that is most of a long
// search (a single cluster), launches that spread the draw over the chip are faster, the sooner the
// fewer searches there are: ten iterations, launches / one launch, one search of 8192 rows 291 / 264 us,
// of 12000 310 / 361, of 16384 329 / 476; 100 searches of 12000 482 / 386, of 16384 499 / 511; 300 of
// 12000 780 / 783, of 16384 903 / 1022.  (Two clusters: one search of 16384 318 / 281.)
constexpr int kRoundsFew = 8, kRoundsMembersFew = 9000, kRoundsMembers = 14000;
bool rounds_in_one_launch(const kb_batch& b) {
    const int64_t members = b.G <= kRoundsFew ? kRoundsMembersFew : kRoundsMembers;
    return b.G > 0 && b.Nmax <= kUcbLong && b.Nmax <= members * (b.Kmax > 0 ? b.Kmax : 1) &&
           rounds_lds(b) + 1024 <= 160 * 1024;
}
bool rounds_need_order(const kb_batch& b) { return order_matters(b) && !rounds_wave_per_search(b); }

// Batches of up to two searches per compute unit give every search 1024 threads, larger ones 256.
constexpr int kRoundsWideMaxG = 512;

template <int NT>
static hipError_t launch_rounds_nt(const RoundsArgs& r, size_t lds, hipStream_t st) {
    const auto go = [&](auto kern) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)r.u.G), dim3(NT), lds, st, r);
        return hipGetLastError();
    };
    switch (row_form(r.u.S)) {
        case 0: return go(rounds_kernel<4, true, NT>);
        case 1: return go(rounds_kernel<4, false, NT>);
        case 2: return go(rounds_kernel<2, false, NT>);
        default: return go(rounds_kernel<1, false, NT>);
    }
}

hipError_t launch_rounds(const kb_batch& b, const UcbCall& c, const SampleCall& sc, const RoundsCall& rc,
                         hipStream_t st) {
    if (!rounds_in_one_launch(b) || c.bound || !sc.h || rc.rounds < 1) return hipErrorInvalidValue;
    RoundsArgs r;
    r.u = make_ucb_args(b, c);
    r.s = make_sample_args(b, sc);
    r.rounds = rc.rounds; r.draw0 = sc.draw; r.reward = rc.reward; r.ok = rc.ok;
    r.visits = rc.visits; r.rsum = rc.rsum; r.t = rc.t; r.sel_log = rc.sel_log; r.ksel_log = rc.ksel_log;
    r.Nmax = b.Nmax;
    // (means beside the tables where two searches per compute unit still fit)
    r.means = rounds_lds(b, true) <= (rounds_wave_per_search(b) ? 16 * 1024 : 78 * 1024);
    const size_t lds = rounds_lds(b, r.means != 0);
    if (rounds_wave_per_search(b)) {
        hipLaunchKernelGGL(rounds_wave, dim3((unsigned)((b.G + kWaves - 1) / kWaves)), dim3(kThreads),
                           lds * kWaves, st, r, (int)lds);
        return hipGetLastError();
    }
    return b.G <= kRoundsWideMaxG ? launch_rounds_nt<1024>(r, lds, st) : launch_rounds_nt<256>(r, lds, st);
}

}  // namespace kb
