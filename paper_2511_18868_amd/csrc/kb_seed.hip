// Farthest-point initial centroids (greedy cover of a search's frontier): the
// first centroid is the search's first row, every further one the candidate
// farthest from the centroids chosen so far.  The largest cluster radius of this
// cover is within a factor two of the smallest possible one - the covering
// radius that the approximation term of Theorem 1 is linear in.
//
// One workgroup per search, K_g passes over the search's rows.  A thread owns the
// rows tid, tid + 512, ...  The first R of them are read once and stay in
// registers for all passes (R x 512 rows, 1536 at 48 features), the next ones in LDS;
// rows beyond that are streamed again in every pass.
//
// The definition is in fp64: squared distances from direct differences, summed over the
// features in index order with separate multiply and add, the largest running minimum
// (or, for the D^2-weighted draw, the largest ln(minimum) + Gumbel variate), lowest
// index on ties.  A pass forms all of that in fp32 only - a sum of non-negative terms
// is good to (D + 2) 2^-24 of itself, a key to 5e-5 - and keeps best and second best.
// If no other row comes within a margin of several times those errors, the best is the
// definition's choice.  Otherwise ("contested", about one pass in a thousand on data
// without repeated rows) the rows within the margin get their fp64 values, unless they are
// all the same row.  A contest of many rows, or contests in most passes, are the mark of
// coarsely quantised or often repeated rows, where a pass in fp64 throughout costs less: the
// search then goes through the centroids chosen so far once more, and on, in such passes.
// (One-hot rows, farthest point, 1024 searches of 64-4096 rows of 48 features: 3500 us with
// a contest in every pass, 1070 us now, 980 us in fp64 from the start; each row five times:
// 1220, 760 and 1040 us.)
// In fp64 throughout a row and pass was 48 conversions, 144 fp64 operations and three
// fp64 logarithms; in fp32 it is 96 operations, the counter-based generator (17 32-bit
// multiplications, a quarter of the rate each) and two hardware logarithms.  1024 searches
// of 64-4096 rows of 48 features, D^2-weighted: 1850 -> 705 us; what bounds it now is the
// latency of a pass in short searches (2.6 us: two barriers, the reduction, the generator)
// and the streamed rows in the longest.  The register share R is as large as fits without
// spilling (one more row per thread: 256 searches of 2048 rows 320 -> 455 us).
//
// Searches longer than kBigRows rows would keep one compute unit busy for K_g
// passes over memory; they take one launch per centroid instead.  The candidate
// axis is cut into flat ranges of kRange rows, one workgroup each; a workgroup
// first finds the newest centroid of its search - the best of the (key, row)
// pairs that the ranges of the previous launch left in the workspace - then does
// the pass over its own rows and leaves its pair for the next launch.  Two sets of
// pairs alternate between launches.
#include "kb_internal.h"
#include "kb_rng_dev.h"
#include "kb_wave_dev.h"

namespace kb {

namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / kWave;
constexpr int kBigRows = 4096;     // longer searches take the launch-per-centroid path
constexpr int kRange = 1024;       // its rows per workgroup (at most kBigRows, so that a range
                                   // meets at most two long searches: one that began before
                                   // it, one that begins inside)
constexpr int kBigThreads = 256;
constexpr int kNone = 0x7fffffff;
constexpr int kListed = 64;        // rows of a contest that are listed
constexpr int kSettled = 16;       // more of them, unless all are the same row: the search goes on in fp64
constexpr int kContests = 4;       // or after so many contests, in most passes
// rows a workgroup keeps in LDS after the registers are full: padded to 16 DS + 4
// words (16-byte reads of consecutive rows fall into different banks), at most
// two per thread, within 140 KB; the fp32 minima of the streamed rows lie behind them
constexpr int lds_stride(int DS) { return 16 * DS + 4; }
constexpr int lds_rows(int DS) {
    return 143360 / (4 * lds_stride(DS)) < 2 * kThreads ? 143360 / (4 * lds_stride(DS)) : 2 * kThreads;
}
constexpr int streamed_rows(int DS, int R) {
    return kBigRows > R * kThreads + lds_rows(DS) ? kBigRows - R * kThreads - lds_rows(DS) : 0;
}
// Fast keys are log2(minimum) - log2(-log2 u).  Outside these bounds of the largest one
// an fp32 minimum may have lost its relative accuracy to underflow or overflow (a variate
// lies between -6 and 53): every row is then formed in fp64.  The margin is ten times the
// 5e-5 of a key (log2_exponential 3e-5; the minimum's (D + 2) 2^-24, its logarithm and the
// difference 1.7e-5), of which two compare.
constexpr float kKeyLow = -40.f, kKeyHigh = 100.f, kKeyMargin = 0x1p-11f;
constexpr float kFarLow = 0x1p-100f, kFarHigh = 0x1p100f;

struct SeedArgs {
    int G, D, Ksum;
    int64_t N;
    const int32_t* seg_off;
    const int32_t* koff;
    const float* X;
    float* cent;
    int32_t* pick;       // may be NULL
    double* mind;        // [N] running minimum of every candidate
    const int32_t* order;
    // randomised (D^2-weighted) seeding instead of the farthest point
    int dsquared;
    unsigned seed_lo, seed_hi;
    unsigned long long draw0;
    // launch-per-centroid path: pair (key, row in its search) of range r, slot s
    // (0: the search that began before the range, 1: the one that begins inside),
    // set b at index (b * nranges + r) * 2 + s
    double* skey;
    int32_t* sidx;
    int nranges;
};

// exact squared difference added to a running sum, the three roundings kept apart
__device__ __forceinline__ double add_sq(double acc, float x, double c) {
    const double diff = __dsub_rn((double)x, c);
    return __dadd_rn(acc, __dmul_rn(diff, diff));
}

// Features d .. d + 3 of a row, zeros beyond D: one 16-byte load whatever D is (rows
// start at multiples of 4 bytes: load4).  `inside`: the piece ends inside the row.
__device__ __forceinline__ float4 row_piece(const float* row, int d, int D, bool inside) {
    if (inside) return load4(row + d);
    if (D >= 4) return row_piece_shift(row_piece_load(row, d, D), d, D);
    return d > 0 ? make_float4(0.f, 0.f, 0.f, 0.f)
                 : make_float4(row[0], D > 1 ? row[1] : 0.f, D > 2 ? row[2] : 0.f, 0.f);
}
__device__ __forceinline__ float add_sq4(float acc, const float4& x, const float4& c) {
    const float e0 = x.x - c.x, e1 = x.y - c.y, e2 = x.z - c.z, e3 = x.w - c.w;
    return fmaf(e3, e3, fmaf(e2, e2, fmaf(e1, e1, fmaf(e0, e0, acc))));
}

// log2(E) of the exponential variate E = -ln u behind gumbel_variate, up to the constant
// log2(ln 2), to 3e-5: u from its 32 leading bits, with a series where u is so close to 1
// that its logarithm would cancel, and in fp64 for the 9 variates in 10^6 whose leading
// bits do not determine it well enough.  The bits left out are worth up to 2^-33 of u: beside
// 1 - u >= kNearOne 2^-32 that is 2^-16 of E, 2.2e-5 on log2(E); beside u >= kNearZero 2^-32 it is
// 2^-13 of u, that much of an E of 13.8 nats, 1.3e-5.  (Series, logarithms and fp32 roundings
// add 4e-6.)  These are the variates that win draws, so the lines are generous.
constexpr unsigned kNearZero = 1u << 12, kNearOne = 1u << 15;
__device__ __forceinline__ float log2_exponential(unsigned seed_lo, unsigned seed_hi, unsigned draw_lo,
                                                  unsigned draw_hi, int k) {
    unsigned x0, x1;
    philox4x32_10((unsigned)k, 0u, draw_lo, draw_hi, seed_lo, seed_hi, x0, x1);
    const unsigned nx = ~x0;
    const float u = fmaf((float)x0, 0x1p-32f, 0x1p-33f), v = fmaf((float)nx, 0x1p-32f, 0x1p-33f);
    const float near1 = v * fmaf(v, fmaf(v, 0.333333343f, 0.5f), 1.f) * 1.44269502f;
    const float E = nx < 0x04000000u ? near1 : -__builtin_amdgcn_logf(u);
    float l = __builtin_amdgcn_logf(E);
    if (x0 < kNearZero || nx < kNearOne)
        l = (float)((-gumbel_variate(seed_lo, seed_hi, draw_lo, draw_hi, k) - log(M_LN2)) * M_LOG2E);
    return l;
}

// DS: features padded to 16 DS (zeros add +0.0 to a sum); R: rows per thread kept in registers
template <int DS, int R, bool DSQ>
__global__ void __launch_bounds__(kThreads) seed_farthest_kernel(SeedArgs a) {
    constexpr int Q = 4 * DS;
    constexpr int RS = lds_stride(DS), LROWS = lds_rows(DS), LV = (LROWS + kThreads - 1) / kThreads;
    constexpr int FIRST = R * kThreads + LROWS;        // first streamed row
    extern __shared__ __align__(16) float lx[];        // [LROWS][RS]
    float* ms = lx + (size_t)LROWS * RS;               // [streamed_rows] minima of the streamed rows
    __shared__ __align__(16) float c[16 * DS];
    __shared__ unsigned short picks[kBigRows];         // rows chosen so far (K <= N_g)
    __shared__ float redf[kWaves];
    __shared__ int redk[kWaves];                       // the row, or -1 - row if contested inside the wave
    __shared__ double redv[kWaves];
    __shared__ int redi[kWaves];
    __shared__ int nlist, differ;                      // rows of a contest; not all of them the same row
    __shared__ unsigned short list[kListed];
    const int tid = threadIdx.x;
    const int D = a.D;
    int g = a.order ? a.order[blockIdx.x] : (int)blockIdx.x;
    g = clampi(g, 0, a.G - 1);
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (ng <= 0 || K <= 0 || ng > kBigRows) return;
    if (K > kBigRows) K = kBigRows;      // (more clusters than candidates: not a consistent batch)
    const float* Xg = a.X + (size_t)n0 * D;
    double* mind = a.mind + n0;
    const float far_keep = 1.f - 4.f * (float)(D + 4) * 0x1p-24f;     // farthest point: margin of a contest

    // what a row offers in draw `drawn`: its minimum (farthest point) or its fast key
    auto offer = [&](float m, int k, unsigned long long drawn) {
        if constexpr (!DSQ) return m;
        // (opaque: the generator's first products, the same in every pass, would be kept
        // in registers for every row)
        asm volatile("" : "+v"(k));
        return __builtin_amdgcn_logf(m) - log2_exponential(a.seed_lo, a.seed_hi, (unsigned)drawn,
                                                           (unsigned)(drawn >> 32), n0 + k);
    };
    float best, second;         // this thread's best and second best offer
    int arg;
    auto take = [&](float v, int k) {
        const bool gt = v > best;               // (false for a NaN, which is never chosen)
        second = gt ? best : fmaxf(second, v);
        arg = gt ? k : arg;
        best = gt ? v : best;
    };
    // The row to choose: the one with the best offer, if nothing else comes close.  Every
    // thread returns the row, or -1 for a contest over the rows that offer `thr` or more.
    // (One barrier: every thread merges the waves' results itself.  The slots are written
    // again only after the barrier that follows the staging of the next centroid.)
    auto keep_from = [&](float m) { return DSQ ? m - kKeyMargin : m * far_keep; };
    auto choose = [&](float& thr) {
        const float m = wave_max_f(best);
        const float t = keep_from(m);
        const unsigned long long same = __ballot(best >= t);
        const unsigned long long most = __ballot(best == m);
        const bool alone = __popcll(same) == 1 && !__any(second >= t);
        const int row = __builtin_amdgcn_readlane(arg, most ? __ffsll((long long)most) - 1 : 0);
        if ((tid & 63) == 0) { redf[tid >> 6] = m; redk[tid >> 6] = alone ? row : -1 - row; }
        __syncthreads();
        float bm = redf[0];
        int bk = redk[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            const float om = redf[w];
            bk = om > bm ? redk[w] : bk;
            bm = om > bm ? om : bm;
        }
        thr = keep_from(bm);
        int close = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) close += redf[w] >= thr ? 1 : 0;
        const bool sane = DSQ ? (bm > kKeyLow && bm < kKeyHigh) : (bm > kFarLow && bm < kFarHigh);
        if (!sane) thr = -INFINITY;             // every row
        return sane && close == 1 && bk >= 0 && bk < ng ? bk : -1;
    };
    // A contest: the definition's choice among the rows that offer thr or more, listed by
    // the threads that own them.  They take a wave each, lanes over the j + 1 centroids
    // chosen so far (none for the first draw, whose keys are the variates alone).
    double far;
    int farg;
    auto sq_dist = [&](const float* row, const float* cr) {
        double acc = 0.0;
        for (int d0 = 0; d0 < D; d0 += 16) {
            float4 xv[4], cv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int d = d0 + 4 * q;
                xv[q] = row_piece(row, d, D, false);
                cv[q] = row_piece(cr, d, D, false);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {                // (+0.0 beyond D)
                acc = add_sq(acc, xv[q].x, (double)cv[q].x);
                acc = add_sq(acc, xv[q].y, (double)cv[q].y);
                acc = add_sq(acc, xv[q].z, (double)cv[q].z);
                acc = add_sq(acc, xv[q].w, (double)cv[q].w);
            }
        }
        return acc;
    };
    auto settle = [&](double mn, int k, int j, unsigned long long drawn) {
        double key = mn;
        if constexpr (DSQ) {
            asm volatile("" : "+v"(k));          // (as in `offer`)
            key = (j >= 0 ? log(mn) : 0.0) + gumbel_variate(a.seed_lo, a.seed_hi, (unsigned)drawn,
                                                             (unsigned)(drawn >> 32), n0 + k);
        }
        if (key > far || (key == far && k < farg)) { far = key; farg = k; }
    };
    // minima are formed as m = m < d ? m : d centroid by centroid, so a NaN is forgotten
    // with the next centroid's distance
    auto contest_wave = [&](int k, int j, unsigned long long drawn) {
        const int lane = tid & 63;
        double mn = INFINITY;
        for (int i0 = 0; i0 <= j; i0 += 64) {
            const bool in = i0 + lane <= j;
            const double acc = sq_dist(Xg + (size_t)k * D, Xg + (size_t)picks[in ? i0 + lane : j] * D);
            const unsigned long long nan = __ballot(in && acc != acc);
            const int last = nan ? 63 - __clzll((long long)nan) : -1;
            double m = in && lane > last ? acc : INFINITY;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                const double om = __shfl_xor(m, o);
                m = om < m ? om : m;
            }
            if (nan) mn = NAN;
            if (!nan || i0 + last < (j < i0 + 63 ? j : i0 + 63)) mn = mn < m ? mn : m;
        }
        settle(mn, k, j, drawn);
    };
    // largest (value, lowest index) of the workgroup; every thread returns the index.
    // (The slots are read before the barrier that follows the next staging.)
    auto block_argmax = [&]() {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double of = __shfl_xor(far, o);
            const int oa = __shfl_xor(farg, o);
            if (of > far || (of == far && oa < farg)) { far = of; farg = oa; }
        }
        if ((tid & 63) == 0) { redv[tid >> 6] = far; redi[tid >> 6] = farg; }
        __syncthreads();
        far = redv[0]; farg = redi[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) {
            const double of = redv[w];
            const int oa = redi[w];
            if (of > far || (of == far && oa < farg)) { far = of; farg = oa; }
        }
        return (farg >= 0 && farg < ng) ? farg : 0;
    };

    // (`minimum(k)`: the fp32 minimum of a row of this thread; -1: to be decided in fp64 passes)
    int contests = 0;
    auto resolve = [&](int j, unsigned long long drawn, float thr, auto minimum) {
        far = -INFINITY; farg = kNone;
#pragma unroll 1
        for (int k = tid; k < ng; k += kThreads) {
            if (offer(minimum(k), k, drawn) >= thr) {
                const int at = atomicAdd(&nlist, 1);
                if (at < kListed) list[at] = (unsigned short)k;
            }
        }
        __syncthreads();
        const int n = nlist, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
        if (n > kListed) {                       // (uniform over the workgroup)
            if (j >= 0) return -1;
            for (int k = tid; k < ng; k += kThreads) settle(0.0, k, -1, drawn);
            return block_argmax();
        }
        if constexpr (!DSQ) {
            // rows that are copies of one: the lowest, whatever their distance is
            const float* first = Xg + (size_t)list[0] * D;
            bool other = false;
            for (int i = w; i < n; i += kWaves)
                if (lane < D) other |= __float_as_uint(first[lane]) != __float_as_uint(Xg[(size_t)list[i] * D + lane]);
            if (__any(other) && lane == 0) differ = 1;
            __syncthreads();
            if (!differ) {
                int k = lane < n ? (int)list[lane] : kNone;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) {
                    const int ok = __shfl_xor(k, o);
                    k = ok < k ? ok : k;
                }
                return k < ng ? k : 0;
            }
        }
        if (j >= 0 && n > kSettled) return -1;
        ++contests;
        for (int i = w; i < n; i += kWaves) contest_wave(list[i], j, drawn);
        return block_argmax();
    };

    // the rows that stay in registers; `ru`: how many of them any lane of this wave has
    float4 xr[R][Q];
    float mk[R];
    int ru = 0;
#pragma unroll
    for (int u = 0; u < R; ++u) {
        if ((tid & ~63) + u * kThreads < ng) ru = u + 1;
        const int k = tid + u * kThreads;
        const bool ex = k < ng;
        const float* row = Xg + (size_t)(ex ? k : 0) * D;      // (D > 16 (DS - 1))
#pragma unroll
        for (int q = 0; q < Q; ++q) xr[u][q] = row_piece(row, 4 * q, D, q < Q - 4);
        mk[u] = INFINITY;
    }
    // the next LROWS rows go to LDS, row R * 512 + tid + 512 v to thread tid
    float ml[LV];
#pragma unroll
    for (int v = 0; v < LV; ++v) {
        const int sl = tid + v * kThreads, k = R * kThreads + sl;
        ml[v] = INFINITY;
        if (sl < LROWS && k < ng) {
            const float* row = Xg + (size_t)k * D;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                *reinterpret_cast<float4*>(lx + (size_t)sl * RS + 4 * q) = row_piece(row, 4 * q, D, q < Q - 4);
        }
    }
    for (int k = FIRST + tid; k < ng; k += kThreads) ms[k - FIRST] = INFINITY;

    float thr;
    int chosen = 0;
    if (tid == 0) { nlist = 0; differ = 0; }     // (before the barrier of the first choice)
    if constexpr (DSQ) {
        // first centroid: a uniform draw, i.e. the largest variate of draw number draw0
        best = -INFINITY; second = -INFINITY; arg = kNone;
        for (int k = tid; k < ng; k += kThreads) take(offer(1.f, k, a.draw0), k);
        chosen = choose(thr);
        if (chosen < 0) {                        // (uniform over the workgroup)
            chosen = resolve(-1, a.draw0, thr, [](int) { return 1.f; });
        }
    }
    // The chosen row becomes the centroid: out of its owner's registers, from LDS, or from
    // memory if it is one of the streamed rows.
    auto stage = [&](int row) {
        if (row < R * kThreads) {
#pragma unroll
            for (int u = 0; u < R; ++u) {
                if (u == row / kThreads && tid == (row & (kThreads - 1))) {
#pragma unroll
                    for (int q = 0; q < Q; ++q) reinterpret_cast<float4*>(c)[q] = xr[u][q];
                }
            }
        } else if (tid < 16 * DS) {
            c[tid] = row < FIRST ? lx[(size_t)(row - R * kThreads) * RS + tid]
                     : tid < D   ? Xg[(size_t)row * D + tid]
                                 : 0.f;
        }
    };
    int known = K;                     // (known < K: so many centroids are chosen, the rest in fp64 passes)
    for (int j = 0; j < K; ++j) {
        const unsigned long long drawn = a.draw0 + (unsigned long long)j + 1ull;
        chosen = __builtin_amdgcn_readfirstlane(chosen);     // (the same in every thread)
        if (tid == 0) { picks[j] = (unsigned short)chosen; nlist = 0; differ = 0; }
        if (j + 1 == K) break;         // the last centroid is followed by no choice
        stage(chosen);
        __syncthreads();
        best = -INFINITY; second = -INFINITY; arg = kNone;
        // rows in registers and in LDS, one walk over the centroid; its next two pieces are
        // requested while two are worked on (all of them at once, as the compiler would
        // have it, do not fit beside the rows)
        if (ru > 0) {
            const bool inlds = (tid & ~63) + R * kThreads < ng;       // (uniform over the wave)
            float acc[R], accl[LV];
            const float* lrow[LV];
#pragma unroll
            for (int u = 0; u < R; ++u) acc[u] = 0.f;
#pragma unroll
            for (int v = 0; v < LV; ++v) {
                accl[v] = 0.f;
                // (a slot beyond the search's rows is read all the same: inside the array)
                lrow[v] = lx + (size_t)(tid + v * kThreads < LROWS ? tid + v * kThreads : tid) * RS;
            }
            float4 cv[2];
            cv[0] = *reinterpret_cast<const float4*>(c);
            cv[1] = *reinterpret_cast<const float4*>(c + 4);
#pragma unroll
            for (int q = 0; q < Q; q += 2) {
                if (q <= Q - 4 || 4 * q < D) {
                    float4 cn[2];
                    cn[0] = cv[0]; cn[1] = cv[1];
                    if (q + 2 < Q) {
                        cn[0] = *reinterpret_cast<const float4*>(c + 4 * q + 8);
                        cn[1] = *reinterpret_cast<const float4*>(c + 4 * q + 12);
                    }
                    if (inlds) {
#pragma unroll
                        for (int v = 0; v < LV; ++v) {
                            const float4 x0 = *reinterpret_cast<const float4*>(lrow[v] + 4 * q);
                            const float4 x1 = *reinterpret_cast<const float4*>(lrow[v] + 4 * q + 4);
                            accl[v] = add_sq4(add_sq4(accl[v], x0, cv[0]), x1, cv[1]);
                        }
                    }
#pragma unroll
                    for (int u = 0; u < R; ++u)
                        if (u < ru) acc[u] = add_sq4(add_sq4(acc[u], xr[u][q], cv[0]), xr[u][q + 1], cv[1]);
                    cv[0] = cn[0]; cv[1] = cn[1];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const int k = tid + u * kThreads;
                if (u < ru) {
                    mk[u] = mk[u] < acc[u] ? mk[u] : acc[u];
                    const float v = offer(mk[u], k, drawn);
                    take(k < ng ? v : -INFINITY, k);
                }
            }
            if (inlds) {
#pragma unroll
                for (int v = 0; v < LV; ++v) {
                    const int sl = tid + v * kThreads, k = R * kThreads + sl;
                    if (sl < LROWS && k < ng) {
                        ml[v] = ml[v] < accl[v] ? ml[v] : accl[v];
                        take(offer(ml[v], k, drawn), k);
                    }
                }
            }
        }
        // Rows beyond the registers' and the LDS's share: four lanes per row, so that a
        // load takes 64 consecutive bytes of each of 16 rows.  (A lane per row took 16
        // bytes of each of 64 rows and the cache line had left the vector cache by the
        // next piece: a pass over 4096 rows of 48 features was 12.1 us and is 9.2 us.)  Lane
        // l then offers row 16 (l & 3) + l / 4 of the wave's 64.
        if constexpr (FIRST < kBigRows) {
            const int lane = tid & 63, quad = lane & 3;
            for (int kb = FIRST + (tid & ~63); kb < ng; kb += kThreads) {     // (uniform over the wave)
                float mine = 0.f;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    float4 xs[2][DS];
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const int k = kb + 16 * (2 * half + u) + (lane >> 2);
                        const float* row = Xg + (size_t)(k < ng ? k : kb) * D;
#pragma unroll
                        for (int i = 0; i < DS; ++i)
                            xs[u][i] = row_piece(row, 16 * i + 4 * quad, D, i + 1 < DS);
                    }
                    float acc[2] = {0.f, 0.f};
#pragma unroll
                    for (int i = 0; i < DS; ++i) {
                        const float4 cv = *reinterpret_cast<const float4*>(c + 16 * i + 4 * quad);
#pragma unroll
                        for (int u = 0; u < 2; ++u) acc[u] = add_sq4(acc[u], xs[u][i], cv);
                    }
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        acc[u] += dpp_f<0xB1>(acc[u]);
                        acc[u] += dpp_f<0x4E>(acc[u]);
                        mine = quad == 2 * half + u ? acc[u] : mine;
                    }
                }
                const int k = kb + 16 * quad + (lane >> 2);
                if (k < ng) {
                    const float old = ms[k - FIRST];
                    const float m = old < mine ? old : mine;
                    ms[k - FIRST] = m;
                    take(offer(m, k, drawn), k);
                }
            }
        }
        chosen = choose(thr);
        if (__builtin_expect(chosen < 0, 0)) {   // (uniform over the workgroup)
            chosen = resolve(j, drawn, thr, [&](int k) {
                float m = 0.f;
                const int u0 = k / kThreads;     // (a register array is not indexed by a variable)
#pragma unroll
                for (int u = 0; u < R; ++u) m = u == u0 ? mk[u] : m;
#pragma unroll
                for (int v = 0; v < LV; ++v) m = u0 == R + v ? ml[v] : m;
                return k >= FIRST ? ms[k - FIRST] : m;
            });
            if (chosen < 0 || (contests >= kContests && 2 * contests > j + 1)) {
                known = j + 1;
                if (chosen >= 0) {
                    if (tid == 0) picks[known] = (unsigned short)chosen;
                    ++known;
                }
                break;
            }
        }
    }
    if (known < K) {
        // fp64 passes over the centroids chosen so far and on from there
        // Minima of the rows on chip stay in registers where they are the offers themselves.  For
        // the draw they go to memory like those of the streamed rows, and the variates, eight
        // sets of fp64 logarithms in one pass, come one at a time from there.
        double m64[DSQ ? 1 : R], l64[DSQ ? 1 : LV];
        const auto keep = [&](double d, int k, int j) {
            if (j > 0) {
                const double old = mind[k];
                d = old < d ? old : d;
            }
            mind[k] = d;
            return d;
        };
        __syncthreads();
        for (int j = 0; j < K; ++j) {
            const unsigned long long drawn = a.draw0 + (unsigned long long)j + 1ull;
            chosen = __builtin_amdgcn_readfirstlane(j < known ? (int)picks[j] : chosen);
            if (tid == 0 && j >= known) picks[j] = (unsigned short)chosen;
            if (j + 1 == K) break;
            stage(chosen);
            __syncthreads();
            const bool choosing = j + 1 >= known;
            far = -INFINITY; farg = kNone;
            if (ru > 0) {
                const bool inlds = (tid & ~63) + R * kThreads < ng;       // (uniform over the wave)
                double acc[R], accl[LV];
                const float* lrow[LV];
#pragma unroll
                for (int u = 0; u < R; ++u) acc[u] = 0.0;
#pragma unroll
                for (int v = 0; v < LV; ++v) {
                    accl[v] = 0.0;
                    lrow[v] = lx + (size_t)(tid + v * kThreads < LROWS ? tid + v * kThreads : tid) * RS;
                }
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    if (4 * q < D) {
                        const float4 cv = *reinterpret_cast<const float4*>(c + 4 * q);
                        const double cx = (double)cv.x, cy = (double)cv.y, cz = (double)cv.z, cw = (double)cv.w;
#pragma unroll
                        for (int u = 0; u < R; ++u) {
                            if (u < ru) {
                                // (opaque to the compiler, which would otherwise widen every
                                // row to fp64 once, outside the passes, at twice the registers)
                                asm volatile("" : "+v"(xr[u][q].x), "+v"(xr[u][q].y), "+v"(xr[u][q].z),
                                                  "+v"(xr[u][q].w));
                                acc[u] = add_sq(acc[u], xr[u][q].x, cx);
                                acc[u] = add_sq(acc[u], xr[u][q].y, cy);
                                acc[u] = add_sq(acc[u], xr[u][q].z, cz);
                                acc[u] = add_sq(acc[u], xr[u][q].w, cw);
                            }
                        }
                        if (inlds) {
#pragma unroll
                            for (int v = 0; v < LV; ++v) {
                                const float4 x4 = *reinterpret_cast<const float4*>(lrow[v] + 4 * q);
                                accl[v] = add_sq(accl[v], x4.x, cx);
                                accl[v] = add_sq(accl[v], x4.y, cy);
                                accl[v] = add_sq(accl[v], x4.z, cz);
                                accl[v] = add_sq(accl[v], x4.w, cw);
                            }
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    const int k = tid + u * kThreads;
                    if constexpr (DSQ) {
                        if (k < ng) keep(acc[u], k, j);
                    } else {
                        m64[u] = j > 0 && m64[u] < acc[u] ? m64[u] : acc[u];
                        if (k < ng) settle(m64[u], k, j, drawn);
                    }
                }
                if (inlds) {
#pragma unroll
                    for (int v = 0; v < LV; ++v) {
                        const int sl = tid + v * kThreads, k = R * kThreads + sl;
                        if constexpr (DSQ) {
                            if (sl < LROWS && k < ng) keep(accl[v], k, j);
                        } else {
                            l64[v] = j > 0 && l64[v] < accl[v] ? l64[v] : accl[v];
                            if (sl < LROWS && k < ng) settle(l64[v], k, j, drawn);
                        }
                    }
                }
            }
            if constexpr (FIRST < kBigRows) {
                constexpr int U = 2;      // rows in flight per thread
                // (row k to thread k mod 512, as all others)
                const int k0s = FIRST + ((tid + kThreads - FIRST % kThreads) & (kThreads - 1));
                for (int kb = k0s; kb < ng; kb += U * kThreads) {
                    double acc[U];
                    const float* row[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        acc[u] = 0.0;
                        row[u] = Xg + (size_t)(kb + u * kThreads < ng ? kb + u * kThreads : kb) * D;
                    }
                    for (int d0 = 0; d0 < D; d0 += 8) {
                        float4 xv[U][2];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            xv[u][0] = row_piece(row[u], d0, D, false);
                            xv[u][1] = row_piece(row[u], d0 + 4, D, false);
                        }
#pragma unroll
                        for (int q = 0; q < 2; ++q) {                // (zeros beyond D, also in c)
                            const float4 cv = *reinterpret_cast<const float4*>(c + d0 + 4 * q);
#pragma unroll
                            for (int u = 0; u < U; ++u) {
                                acc[u] = add_sq(acc[u], xv[u][q].x, (double)cv.x);
                                acc[u] = add_sq(acc[u], xv[u][q].y, (double)cv.y);
                                acc[u] = add_sq(acc[u], xv[u][q].z, (double)cv.z);
                                acc[u] = add_sq(acc[u], xv[u][q].w, (double)cv.w);
                            }
                        }
                    }
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int k = kb + u * kThreads;
                        if (k < ng) {
                            const double m = keep(acc[u], k, j);
                            if constexpr (!DSQ) settle(m, k, j, drawn);
                        }
                    }
                }
            }
            if (choosing) {
                if constexpr (DSQ) {
                    // (a thread reads back what it wrote)
#pragma unroll 1
                    for (int k = tid; k < ng; k += kThreads) settle(mind[k], k, j, drawn);
                }
                chosen = block_argmax();
            } else {
                __syncthreads();                 // (every thread has read the centroid)
            }
        }
    }
    // the chosen rows (written at the end: a store on the way would be waited for at the
    // next barrier)
    __syncthreads();
    for (int idx = tid; idx < K * D; idx += kThreads) {
        const int j = idx / D, d = idx - j * D;
        a.cent[(size_t)k0 * D + idx] = Xg[(size_t)picks[j] * D + d];
    }
    if (a.pick)
        for (int j = tid; j < K; j += kThreads) a.pick[k0 + j] = n0 + (int)picks[j];
}

// One launch per centroid for the searches of more than kBigRows rows.  `j`: the
// centroid this launch places (-1: only the keys of the uniform first draw);
// `wset`: the set of pairs this launch writes, the other one holds the previous
// launch's.
template <bool DSQ>
__global__ void __launch_bounds__(kBigThreads) seed_big_pass(SeedArgs a, int j, int wset) {
    constexpr int kW = kBigThreads / kWave;
    __shared__ __align__(16) float c[KB_MAX_D];
    __shared__ double redv[kW];
    __shared__ int redi[kW];
    __shared__ int chosen_s;
    const int tid = threadIdx.x;
    const int D = a.D;
    const bool vec = (D & 3) == 0;
    const int r = blockIdx.x;
    const int64_t r0 = (int64_t)r * kRange;
    if (r >= a.nranges || r0 >= a.N) return;
    const int64_t r1 = r0 + kRange < a.N ? r0 + kRange : a.N;
    double* wkey = a.skey + ((size_t)wset * a.nranges + r) * 2;
    int32_t* widx = a.sidx + ((size_t)wset * a.nranges + r) * 2;
    const double* pkey = a.skey + (size_t)(wset ^ 1) * a.nranges * 2;
    const int32_t* pidx = a.sidx + (size_t)(wset ^ 1) * a.nranges * 2;
    if (tid == 0) { widx[0] = kNone; widx[1] = kNone; }
    auto block_argmax = [&](double far, int arg) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const double of = __shfl_xor(far, o);
            const int oa = __shfl_xor(arg, o);
            if (of > far || (of == far && oa < arg)) { far = of; arg = oa; }
        }
        if ((tid & 63) == 0) { redv[tid >> 6] = far; redi[tid >> 6] = arg; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < kW; ++w)
                if (redv[w] > far || (redv[w] == far && redi[w] < arg)) { far = redv[w]; arg = redi[w]; }
            redv[0] = far;
            chosen_s = arg;
        }
        __syncthreads();
        const int res = chosen_s;
        return res;
    };
    // largest g with seg_off[g] <= r0
    int lo = 0, hi = a.G;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)a.seg_off[mid] <= r0) lo = mid; else hi = mid;
    }
    for (int g = lo; g < a.G; ++g) {
        int n0, ng, k0, K;
        search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
        if (n0 >= r1) break;
        if (ng <= kBigRows || K <= 0 || j >= K) continue;
        const int n1 = n0 + ng;
        const int q0 = r0 > n0 ? (int)r0 : n0;
        const int q1 = r1 < n1 ? (int)r1 : n1;
        if (q0 >= q1) continue;
        const float* Xg = a.X + (size_t)n0 * D;
        double* mind = a.mind + n0;
        const int slot = n0 < r0 ? 0 : 1;
        double far = -INFINITY;
        int arg = kNone;
        if (j < 0) {
            for (int k = q0 - n0 + tid; k < q1 - n0; k += kBigThreads) {
                const double key = gumbel_variate(a.seed_lo, a.seed_hi, (unsigned)a.draw0,
                                                  (unsigned)(a.draw0 >> 32), n0 + k);
                if (key > far || (key == far && k < arg)) { far = key; arg = k; }
            }
        } else {
            int chosen = 0;
            if (DSQ || j > 0) {
                // the newest centroid: best pair of the previous launch over the search's ranges
                const int rf = n0 / kRange, rl = (n1 - 1) / kRange;
                double bk = -INFINITY;
                int bi = kNone;
                for (int q = rf + tid; q <= rl; q += kBigThreads) {
                    const int sl = n0 < q * kRange ? 0 : 1;
                    const double ok = pkey[2 * (size_t)q + sl];
                    const int oi = pidx[2 * (size_t)q + sl];
                    if (oi != kNone && (ok > bk || (ok == bk && oi < bi))) { bk = ok; bi = oi; }
                }
                chosen = block_argmax(bk, bi);
                chosen = (chosen >= 0 && chosen < ng) ? chosen : 0;
            }
            if (tid < KB_MAX_D) {
                const float v = tid < D ? Xg[(size_t)chosen * D + tid] : 0.f;
                c[tid] = v;
                if (slot == 1 && tid < D) a.cent[((size_t)k0 + j) * D + tid] = v;
            }
            if (slot == 1 && tid == 0 && a.pick) a.pick[k0 + j] = n0 + chosen;
            __syncthreads();
            if (j + 1 < K) {
                const unsigned long long drawn = a.draw0 + (unsigned long long)j + 1ull;
                constexpr int U = kRange / kBigThreads;     // this thread's rows, all in flight
                const int kb = q0 - n0 + tid, ke = q1 - n0;
                double acc[U];
#pragma unroll
                for (int u = 0; u < U; ++u) acc[u] = 0.0;
                if (vec) {
                    for (int d0 = 0; d0 < D; d0 += 16) {
                        float4 xv[U][4];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int k = kb + u * kBigThreads;
                            const float* row = Xg + (size_t)(k < ke ? k : q0 - n0) * D + d0;
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                xv[u][q] = d0 + 4 * q < D ? *reinterpret_cast<const float4*>(row + 4 * q)
                                                          : make_float4(0.f, 0.f, 0.f, 0.f);
                        }
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            if (d0 + 4 * q < D) {
                                const float4 cv = *reinterpret_cast<const float4*>(c + d0 + 4 * q);
                                const double cx = (double)cv.x, cy = (double)cv.y, cz = (double)cv.z,
                                             cw = (double)cv.w;
#pragma unroll
                                for (int u = 0; u < U; ++u) {
                                    acc[u] = add_sq(acc[u], xv[u][q].x, cx);
                                    acc[u] = add_sq(acc[u], xv[u][q].y, cy);
                                    acc[u] = add_sq(acc[u], xv[u][q].z, cz);
                                    acc[u] = add_sq(acc[u], xv[u][q].w, cw);
                                }
                            }
                        }
                    }
                } else {
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int k = kb + u * kBigThreads;
                        const float* row = Xg + (size_t)(k < ke ? k : q0 - n0) * D;
                        for (int d = 0; d < D; ++d) acc[u] = add_sq(acc[u], row[d], (double)c[d]);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int k = kb + u * kBigThreads;
                    if (k < ke) {
                        double m = acc[u];
                        if (j > 0) {
                            const double old = mind[k];
                            m = old < acc[u] ? old : acc[u];
                        }
                        mind[k] = m;
                        double v = m;
                        if constexpr (DSQ)
                            v = log(m) + gumbel_variate(a.seed_lo, a.seed_hi, (unsigned)drawn,
                                                        (unsigned)(drawn >> 32), n0 + k);
                        if (v > far || (v == far && k < arg)) { far = v; arg = k; }
                    }
                }
            }
        }
        arg = block_argmax(far, arg);
        if (tid == 0) { wkey[slot] = redv[0]; widx[slot] = arg; }
        __syncthreads();
    }
}

}  // namespace

size_t seed_ranges(const kb_batch& b) { return (size_t)((b.N + kRange - 1) / kRange) + 1; }

hipError_t launch_seed(const kb_batch& b, const float* X, float* cent, int32_t* pick, double* mind,
                       double* skey, int32_t* sidx, const int32_t* order, int dsquared, uint64_t seed,
                       uint64_t draw0, hipStream_t st) {
    SeedArgs a;
    a.dsquared = dsquared; a.seed_lo = (unsigned)seed; a.seed_hi = (unsigned)(seed >> 32);
    a.draw0 = draw0;
    a.G = b.G; a.D = b.D; a.Ksum = b.Ksum; a.N = b.N; a.seg_off = b.seg_off; a.koff = b.koff;
    a.X = X; a.cent = cent; a.pick = pick; a.mind = mind; a.order = order;
    a.skey = skey; a.sidx = sidx; a.nranges = (int)seed_ranges(b);
    const dim3 grid((unsigned)b.G), block(kThreads);
    hipError_t err = hipSuccess;
    auto go = [&](auto far, auto dsq, int DS, int R) {
        const size_t lds = (size_t)4 * (lds_stride(DS) * lds_rows(DS) + streamed_rows(DS, R));
        auto kern = dsquared ? dsq : far;
        err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err == hipSuccess) hipLaunchKernelGGL(kern, grid, block, lds, st, a);
    };
    if (b.D <= 16) go(seed_farthest_kernel<1, 8, false>, seed_farthest_kernel<1, 8, true>, 1, 8);
    else if (b.D <= 32) go(seed_farthest_kernel<2, 4, false>, seed_farthest_kernel<2, 4, true>, 2, 4);
    else if (b.D <= 48) go(seed_farthest_kernel<3, 3, false>, seed_farthest_kernel<3, 3, true>, 3, 3);
    else go(seed_farthest_kernel<4, 2, false>, seed_farthest_kernel<4, 2, true>, 4, 2);
    if (err != hipSuccess) return err;
    if (b.Nmax > kBigRows) {
        const dim3 bgrid((unsigned)a.nranges), bblock(kBigThreads);
        int launches = 0;
        if (dsquared) hipLaunchKernelGGL(seed_big_pass<true>, bgrid, bblock, 0, st, a, -1, launches++ & 1);
        for (int j = 0; j < b.Kmax; ++j) {
            if (dsquared) hipLaunchKernelGGL(seed_big_pass<true>, bgrid, bblock, 0, st, a, j, launches++ & 1);
            else hipLaunchKernelGGL(seed_big_pass<false>, bgrid, bblock, 0, st, a, j, launches++ & 1);
        }
    }
    return hipGetLastError();
}

}  // namespace kb
