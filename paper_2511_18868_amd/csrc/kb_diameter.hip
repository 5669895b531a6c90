// Cluster diameters: diam(C_i) = the largest distance between two members of
// cluster i, the quantity in the approximation term L * max_i diam(C_i) of
// Theorem 1.
//
//   dia_zero     per-cluster counters and maxima <- 0
//   dia_group    one workgroup per search: sizes, grouped indices, unit numbers; or, in batches
//                with searches of more than kGroupMax candidates,
//   dia_walk<false>
//                cluster sizes: flat candidate ranges walk the searches that
//                intersect them, LDS histogram per search piece, one global atomic
//                per touched cluster and piece
//   dia_bsum / dia_bscan / dia_apply
//                exclusive prefix sums of the sizes and of the unit counts,
//                counters reset
//   dia_walk<true>
//                candidate indices grouped by cluster (same walk; a piece reserves
//                its slots per cluster with one global atomic, positions inside the
//                piece come from LDS atomics).  The order inside a cluster varies
//                from run to run; the maximum over its pairs does not.
//   dia_pairs    the squares of 64 x 64 member pairs of all clusters are numbered and
//                every wave takes an equal share; the matrix cores form the distances of
//                32 x 32 pairs at a time in fp32, and the pairs that may be the farthest
//                are evaluated from direct differences in fp32 (relative error at most
//                (D + 2) 2^-24 each, being sums of non-negative terms)
//   dia_final    square root
#include "kb_internal.h"
#include "kb_wave_dev.h"

namespace kb {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kRange = 4096;     // candidates per workgroup of the histogram / scatter walks
constexpr int kDiaShort = 64;    // searches of at most this many candidates: all pairs by one wave (dia_wave);
                                 // beyond, a lane's loop over the later members gets long (a search of 256
                                 // candidates took 0.34 ms that way against 0.03 ms through the tiles)

constexpr int kGroupMax = 16384; // batches without longer searches: members grouped by dia_group, a
                                 // workgroup per search
constexpr int kGroupThreads = 512;
constexpr int kGroupMany = 4096, kGroupSearches = 8;     // batches of so many searches: 8 per workgroup
constexpr int kUnitBits = 40;    // units of a batch < 2^40 (fewer than 2^31 candidates in searches of at
                                 // most 16384), searches <= 2^20

// consecutive unit numbers: clusters c0 .. c1 - 1 from unit `first` on
struct DiaSlot {
    long long first;
    int c0, c1;
};

struct DiaArgs {
    int G, D, Ksum, Kmax;
    int64_t N;
    const int32_t* seg_off;
    const int32_t* koff;
    const float* X;
    const int32_t* assign;
    float* diam;          // [Ksum] out
    int32_t* cnt;         // [Ksum] sizes, then cursors
    int32_t* off;         // [Ksum + 1] first slot of every cluster in perm
    int32_t* toff;        // [Ksum + 1] first unit of every cluster in the numbering of its slot
    long long* bsum;      // [2 * blocks of the prefix sum] (members, units) per block
    DiaSlot* slots;       // [max_slots] one per search with units (dia_group); null: one slot, the whole batch
    long long max_slots;  // N / 2: such a search has two candidates or more of its own
    unsigned long long* reserved;   // slots (upper bits) and units (lower kUnitBits) handed out so far
    unsigned* dmax;       // [Ksum] bits of the largest squared distance (aliases diam)
    int32_t* perm;        // [N]
    int mixed;            // 1: searches of at most kDiaShort candidates go to dia_wave, longer ones
                          //    through the grouping and the pair tiles, in the same call
};

__global__ void __launch_bounds__(kThreads) dia_zero(DiaArgs a) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < a.Ksum) { a.cnt[i] = 0; a.dmax[i] = 0u; }
    if (i == 0 && a.slots) *a.reserved = 0ull;
}

// SCATTER = false: sizes; true: grouped indices
template <bool SCATTER>
__global__ void __launch_bounds__(kThreads) dia_walk(DiaArgs a) {
    __shared__ int lcnt[KB_MAX_K];
    __shared__ int lbase[KB_MAX_K];
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * kRange;
    if (r0 >= a.N) return;
    const int64_t r1 = r0 + kRange < a.N ? r0 + kRange : a.N;
    int lo = 0, hi = a.G;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)a.seg_off[mid] <= r0) lo = mid; else hi = mid;
    }
    const auto mine = [&](int n0, int ng, int k0, int K) {
        return n0 >= r1 || (ng > 0 && K > 0 && !(a.mixed && ng <= kDiaShort));
    };
    for (int g = lo; (g = next_search(a.seg_off, a.koff, g, a.G, a.N, a.Ksum, mine)) < a.G; ++g) {
        int n0, ng, k0, K;
        search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
        if (K > KB_MAX_K) K = KB_MAX_K;
        if (n0 >= r1) break;
        if (ng <= 0 || K <= 0) continue;
        if (a.mixed && ng <= kDiaShort) continue;         // (uniform) a wave of dia_wave takes this search:
                                                          // its clusters keep size 0 here and get no units
        const int q0 = r0 > n0 ? (int)r0 : n0;
        const int q1 = r1 < (int64_t)n0 + ng ? (int)r1 : n0 + ng;
        if (q0 >= q1) continue;
        for (int j = tid; j < K; j += kThreads) lcnt[j] = 0;
        __syncthreads();
        for (int p = q0 + tid; p < q1; p += kThreads) {
            int j = a.assign[p];
            j = (j >= 0 && j < K) ? j : 0;
            atomicAdd(&lcnt[j], 1);
        }
        __syncthreads();
        if (!SCATTER) {
            for (int j = tid; j < K; j += kThreads)
                if (lcnt[j]) atomicAdd(&a.cnt[k0 + j], lcnt[j]);
        } else {
            for (int j = tid; j < K; j += kThreads) {
                lbase[j] = lcnt[j] ? a.off[k0 + j] + atomicAdd(&a.cnt[k0 + j], lcnt[j]) : 0;
                lcnt[j] = 0;
            }
            __syncthreads();
            for (int p = q0 + tid; p < q1; p += kThreads) {
                int j = a.assign[p];
                j = (j >= 0 && j < K) ? j : 0;
                const int64_t pos = (int64_t)lbase[j] + atomicAdd(&lcnt[j], 1);
                if (pos >= 0 && pos < a.N) a.perm[pos] = p;
            }
        }
        __syncthreads();
    }
}

// Units of member pairs of a cluster of n members: none below two members, otherwise the
// squares of 64 x 64 pairs on and above the diagonal.
__device__ __forceinline__ long long units_of(int n) {
    if (n < 2) return 0;
    const long long T = (n + 63) >> 6;
    return T * (T + 1) / 2;
}

// off = exclusive prefix sum of cnt, toff = that of the unit counts, cnt <- 0, in
// three launches with coalesced accesses: sums of blocks of kScanBlock entries,
// their prefix sums (one workgroup), then the entries of every block.
constexpr int kScanBlock = 4096;
constexpr int kScanU = kScanBlock / kThreads;

// (members, units) summed over the workgroup; every thread gets the result
__device__ __forceinline__ void block_sum2(long long& m, long long& t, long long* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { m += __shfl_xor(m, o); t += __shfl_xor(t, o); }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) { red[2 * (threadIdx.x >> 6)] = m; red[2 * (threadIdx.x >> 6) + 1] = t; }
    __syncthreads();
    m = 0; t = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) { m += red[2 * w]; t += red[2 * w + 1]; }
}

__global__ void __launch_bounds__(kThreads) dia_bsum(DiaArgs a) {
    __shared__ long long red[2 * kWaves];
    const int i0 = blockIdx.x * kScanBlock + threadIdx.x;
    long long m = 0, t = 0;
#pragma unroll
    for (int u = 0; u < kScanU; ++u) {
        const int i = i0 + u * kThreads;
        const int v = i < a.Ksum ? a.cnt[i] : 0;
        m += v;
        t += units_of(v);
    }
    block_sum2(m, t, red);
    if (threadIdx.x == 0) { a.bsum[2 * blockIdx.x] = m; a.bsum[2 * blockIdx.x + 1] = t; }
}

// exclusive prefix sums of the block sums, in place; one workgroup, blocks in order
__global__ void __launch_bounds__(kThreads) dia_bscan(DiaArgs a, int nblocks) {
    __shared__ long long red[2 * kWaves];
    __shared__ long long carry[2];
    const int tid = threadIdx.x;
    if (tid == 0) { carry[0] = 0; carry[1] = 0; }
    __syncthreads();
    for (int b0 = 0; b0 < nblocks; b0 += kThreads) {
        const int b = b0 + tid;
        const long long m = b < nblocks ? a.bsum[2 * b] : 0, t = b < nblocks ? a.bsum[2 * b + 1] : 0;
        // inclusive scan over the workgroup: inside the waves, then over the wave totals
        long long im = m, it = t;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const long long um = __shfl_up(im, o), ut = __shfl_up(it, o);
            if ((tid & 63) >= o) { im += um; it += ut; }
        }
        if ((tid & 63) == 63) { red[2 * (tid >> 6)] = im; red[2 * (tid >> 6) + 1] = it; }
        __syncthreads();
        long long pm = carry[0], pt = carry[1];
        for (int w = 0; w < (tid >> 6); ++w) { pm += red[2 * w]; pt += red[2 * w + 1]; }
        if (b < nblocks) { a.bsum[2 * b] = pm + im - m; a.bsum[2 * b + 1] = pt + it - t; }
        __syncthreads();
        if (tid == kThreads - 1) { carry[0] = pm + im; carry[1] = pt + it; }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kThreads) dia_apply(DiaArgs a) {
    __shared__ long long red[2 * kWaves];
    const int tid = threadIdx.x;
    const int i0 = blockIdx.x * kScanBlock + tid;
    int v[kScanU];
#pragma unroll
    for (int u = 0; u < kScanU; ++u) {
        const int i = i0 + u * kThreads;
        v[u] = i < a.Ksum ? a.cnt[i] : 0;
    }
    long long cm = a.bsum[2 * blockIdx.x], ct = a.bsum[2 * blockIdx.x + 1];
    const long long tcap = 0x7fffffffll;
    // entries i0 + u * 256: one pass of the workgroup per u keeps the index order
#pragma unroll
    for (int u = 0; u < kScanU; ++u) {
        const int i = i0 + u * kThreads;
        const long long m = v[u], t = units_of(v[u]);
        long long im = m, it = t;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const long long um = __shfl_up(im, o), ut = __shfl_up(it, o);
            if ((tid & 63) >= o) { im += um; it += ut; }
        }
        __syncthreads();
        if ((tid & 63) == 63) { red[2 * (tid >> 6)] = im; red[2 * (tid >> 6) + 1] = it; }
        __syncthreads();
        long long pm = cm, pt = ct, tm = 0, tt = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (w < (tid >> 6)) { pm += red[2 * w]; pt += red[2 * w + 1]; }
            tm += red[2 * w]; tt += red[2 * w + 1];
        }
        if (i < a.Ksum) {
            const long long om = pm + im - m, ot = pt + it - t;
            a.off[i] = (int)(om < a.N ? om : a.N);
            a.toff[i] = (int)(ot < tcap ? ot : tcap);
            a.cnt[i] = 0;
            if (i == a.Ksum - 1) {
                a.off[a.Ksum] = (int)(om + m < a.N ? om + m : a.N);
                a.toff[a.Ksum] = (int)(ot + t < tcap ? ot + t : tcap);
            }
        }
        cm += tm; ct += tt;
    }
}

// Batches whose searches all have at most kGroupMax candidates: one workgroup per search
// does in one launch what the walks and the prefix sums do in five.  The members of a
// search are grouped inside its own part of `perm`, so no prefix sum over the batch is
// needed; a workgroup reserves its unit numbers and slots of the slot list together with one
// 64-bit atomic, so the slots are in the order of their first units whatever the order of
// the workgroups.  (1024 searches of 64-4096 candidates: 19 us, the five launches 71 us.)
// The atomics of all workgroups queue up, 12 ns each, so in a batch of many searches a
// workgroup takes B = 8 of them with one reservation (20000 searches of 100 candidates
// 244 -> 47 us).
// Malformed offsets (overlapping searches) can ask for more slots or units than there can
// be: lengths are cut to what the host announced, slots beyond the list are dropped.
template <int B>
__global__ void __launch_bounds__(kGroupThreads) dia_group(DiaArgs a) {
    __shared__ int lcnt[B][KB_MAX_K];
    __shared__ int units[B];
    const int tid = threadIdx.x, g0 = blockIdx.x * B;
    int n0[B], ng[B], k0[B], K[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        n0[b] = ng[b] = k0[b] = K[b] = 0;
        if (g0 + b < a.G) search_bounds(a.seg_off, a.koff, g0 + b, a.N, a.Ksum, n0[b], ng[b], k0[b], K[b]);
        if (K[b] > KB_MAX_K) K[b] = KB_MAX_K;
        if (ng[b] > kGroupMax) ng[b] = kGroupMax;
        for (int j = tid; j < K[b]; j += kGroupThreads) lcnt[b][j] = 0;
    }
    __syncthreads();
    constexpr int U = 4;
#pragma unroll
    for (int b = 0; b < B; ++b) {
        if (K[b] <= 0) continue;
        const int32_t* as = a.assign + n0[b];
        for (int p0 = tid; p0 < ng[b]; p0 += U * kGroupThreads) {
            int j[U];
#pragma unroll
            for (int u = 0; u < U; ++u) j[u] = p0 + u * kGroupThreads < ng[b] ? as[p0 + u * kGroupThreads] : 0;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (p0 + u * kGroupThreads < ng[b]) atomicAdd(&lcnt[b][(j[u] >= 0 && j[u] < K[b]) ? j[u] : 0], 1);
        }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < B; ++b) {
        if ((tid >> 6) == b) {                           // (B <= 8 waves: one search each)
            // exclusive prefix sums of members and units, four clusters per lane (K <= 256)
            const int lane = tid & 63;
            int n[4], m = 0, t = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = 4 * lane + e;
                n[e] = j < K[b] && ng[b] > 0 ? lcnt[b][j] : 0;
                m += n[e];
                t += (int)units_of(n[e]);
            }
            int im = m, it = t;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int um = __shfl_up(im, o), ut = __shfl_up(it, o);
                if (lane >= o) { im += um; it += ut; }
            }
            if (lane == kWave - 1) units[b] = it;
            int om = n0[b] + im - m, ot = it - t;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = 4 * lane + e;
                if (j < K[b] && ng[b] > 0) {
                    a.cnt[k0[b] + j] = n[e]; a.off[k0[b] + j] = om; a.toff[k0[b] + j] = ot;
                    lcnt[b][j] = om - n0[b];
                }
                om += n[e];
                ot += (int)units_of(n[e]);
            }
        }
    }
    __syncthreads();
    if (tid == 0) {
        unsigned long long want = 0;
#pragma unroll
        for (int b = 0; b < B; ++b)
            if (units[b] > 0) want += (1ull << kUnitBits) | (unsigned long long)units[b];
        if (want) {
            const unsigned long long old = atomicAdd(a.reserved, want);
            long long at = (long long)(old >> kUnitBits);
            DiaSlot s;
            s.first = (long long)(old & ((1ull << kUnitBits) - 1));
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (units[b] <= 0) continue;
                s.c0 = k0[b]; s.c1 = k0[b] + K[b];
                if (at < a.max_slots) a.slots[at] = s;
                ++at;
                s.first += units[b];
            }
        }
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
        if (K[b] <= 0) continue;
        const int32_t* as = a.assign + n0[b];
        for (int p0 = tid; p0 < ng[b]; p0 += U * kGroupThreads) {
            int j[U];
#pragma unroll
            for (int u = 0; u < U; ++u) j[u] = p0 + u * kGroupThreads < ng[b] ? as[p0 + u * kGroupThreads] : 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (p0 + u * kGroupThreads < ng[b]) {
                    const int pos = atomicAdd(&lcnt[b][(j[u] >= 0 && j[u] < K[b]) ? j[u] : 0], 1);
                    if (pos < ng[b]) a.perm[(size_t)n0[b] + pos] = n0[b] + p0 + u * kGroupThreads;
                }
            }
        }
    }
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// 32 members of a cluster in the operand layout of v_mfma_f32_32x32x2_f32: lanes l and
// l + 32 share member l, the first holds features 8c .. 8c + 3, the second 8c + 4 .. 8c + 7
// of every chunk c (the order of the features inside a product is free as long as both
// operands have the same); zeros beyond D.
template <int CH>
struct DiaBlock {
    float v[4 * CH];
    float norm;          // |x|^2
    int row;
};
// Piece of chunk c of CH = ceil(D / 8): only the last chunk can reach beyond the row.
__device__ __forceinline__ float4 dia_piece(const float* x, int c, int CH, int half, int D) {
    const int d0 = 8 * c + 4 * half;
    if (c < CH - 1) return load4(x + d0);
    if (D >= 4) return row_piece_shift(row_piece_load(x, d0, D), d0, D);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (half == 0) {
        v.x = x[0];
        if (D > 1) v.y = x[1];
        if (D > 2) v.z = x[2];
    }
    return v;
}
// (all loads before the first use: the norms are formed by dia_finish)
template <int CH>
__device__ __forceinline__ void dia_load(const DiaArgs& a, DiaBlock<CH>& b, int base, int n, int m0, int lane) {
    int m = m0 + (lane & 31);
    m = m < n ? m : n - 1;           // rows beyond the cluster: its last member, whose distances are genuine ones
    int row = a.perm[base + m];
    row = (row >= 0 && row < a.N) ? row : 0;
    b.row = row;
    const float* x = a.X + (size_t)row * a.D;
    __builtin_assume(CH == 1 || a.D >= 4);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const float4 p = dia_piece(x, c, CH, lane >> 5, a.D);
        b.v[4 * c + 0] = p.x; b.v[4 * c + 1] = p.y; b.v[4 * c + 2] = p.z; b.v[4 * c + 3] = p.w;
    }
}
// the norms; before that, if `centred`, the rows relative to the row `ctr`
template <int CH>
__device__ __forceinline__ void dia_finish(DiaBlock<CH>& b, const float* ctr, bool centred, int D, int lane) {
    if (centred) {
        __builtin_assume(CH == 1 || D >= 4);
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const float4 o = dia_piece(ctr, c, CH, lane >> 5, D);
            b.v[4 * c + 0] -= o.x; b.v[4 * c + 1] -= o.y; b.v[4 * c + 2] -= o.z; b.v[4 * c + 3] -= o.w;
            if (c & 1) asm volatile("" ::: "memory");    // (two pieces of the centre at a time: registers)
        }
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4 * CH; ++i) s = fmaf(b.v[i], b.v[i], s);
    b.norm = s + __shfl_xor(s, 32);
}

// The squared distance of two rows, direct differences in fp32: fused multiply-adds over
// the features in index order.
__device__ __forceinline__ float dia_exact(const float* x, const float* y, int D) {
    float acc = 0.f;
    int d = 0;
#pragma unroll 4
    for (; d + 4 <= D; d += 4) {
        const float4 u = load4(x + d), v = load4(y + d);
        float e = u.x - v.x; acc = fmaf(e, e, acc);
        e = u.y - v.y; acc = fmaf(e, e, acc);
        e = u.z - v.z; acc = fmaf(e, e, acc);
        e = u.w - v.w; acc = fmaf(e, e, acc);
    }
    for (; d < D; ++d) {
        const float e = x[d] - y[d];
        acc = fmaf(e, e, acc);
    }
    return acc;
}

// The farthest of 32 x 32 pairs.  The matrix cores give -d^2 / 2 = x.y - |x|^2 / 2 - |y|^2 / 2 in
// fp32; with M the largest |x|^2 in the tile, that and the value of dia_exact differ by at most
// err = M (10 D + 40) 2^-23 on d^2:
//   - the accumulation, at most 2 D + 8 roundings (taken as 2^-23 each, truncation included) of
//     partial sums of at most 2 M, and the norms' own inside that count:  2 (2 D + 8) 2 M 2^-23
//   - where the rows are centred, 2^-24 of every component of both:        8 M 2^-24
//   - the chain of dia_exact, (D + 2) 2^-24 of at most 4 M:                (D + 2) 4 M 2^-24
// So the pair with the largest dia_exact lies within 2 err of the largest matrix value and, where
// the cluster's maximum is known to be `least` or more, above least - err.  Those pairs, nearly
// always one or none per tile, wait in the wave's queue until 64 can be evaluated side by side
// (or the wave ends), so the result is the maximum of dia_exact over all pairs, bit for bit.
struct DiaQueue {
    int row[kWave], col[kWave], cluster[kWave];
};

// evaluates the waiting pairs, one per lane.  Pairs of a cluster wait side by side, so each run of
// them sends its largest alone to the cluster's maximum, and only if it is larger than what is there:
// a line of 16 maxima takes atomics one after the other.  (40000 candidates in 16 clusters of 16
// features, the pair kernel: 137 us with an atomic per pair, 69 us.)
__device__ __noinline__ void dia_drain(const float* X, int D, unsigned* dmax, const DiaQueue* q, int count) {
    const int lane = threadIdx.x & 63;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    float d2 = 0.f;
    int cid = -1;
    if (lane < count) {
        cid = q->cluster[lane];
        const unsigned have = __hip_atomic_load(&dmax[cid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        d2 = dia_exact(X + (size_t)q->row[lane] * D, X + (size_t)q->col[lane] * D, D);
        if (!(d2 > __uint_as_float(have))) d2 = 0.f;     // (a NaN does not count)
    }
    if (__ballot(d2 > 0.f) != 0ull) {
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {            // the largest from this lane to the end of its run
            const float od = __shfl_down(d2, o);
            const int oc = __shfl_down(cid, o);
            if (lane + o < kWave && oc == cid) d2 = fmaxf(d2, od);
        }
        const int before = __shfl_up(cid, 1);
        if (d2 > 0.f && (lane == 0 || before != cid)) atomicMax(&dmax[cid], __float_as_uint(d2));
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}

// All pairs of a unit from direct differences, for units with many contenders (equal distances:
// rows of few distinct values, rows that occur many times).  Rows and columns stay in registers, one
// of each per lane.  Every group of 16 lanes takes the pairs of 16 columns and 16 rows; the rows are
// turned through the group (a modifier of the subtraction, no instruction of its own), so a pair and
// feature is two vector instructions, as in a kernel that forms every pair this way.  Four group
// squares at a time: four passes, three on the diagonal, one for 32 members or fewer.
template <int S>
__device__ __forceinline__ float dia_turned(float v) {
    if constexpr (S == 0) return v;
    else return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + S, 0xf, 0xf, true));
}
template <int S = 0>
__device__ __forceinline__ void dia_turn(float (&acc)[16], float x, float y) {
    const float e = dia_turned<S>(x) - y;
    acc[S] = fmaf(e, e, acc[S]);
    if constexpr (S < 15) dia_turn<S + 1>(acc, x, y);
}
// Members m0 .. m0 + 63, one per lane (beyond the cluster: its last member), features in order.
// Lanes l and l + 32 load halves of the rows l and 32 + l, so a load takes 32 consecutive bytes of
// a row, and trade them.
template <int CH>
__device__ __forceinline__ void dia_load_rows(float (&v)[8 * CH], const float* X, const int32_t* perm, int N, int D,
                                              int base, int n, int m0, int lane) {
    const auto row_of = [&](int m) {
        const int row = perm[(size_t)base + (m < n ? m : n - 1)];
        return X + (size_t)((row >= 0 && row < N) ? row : 0) * D;
    };
    const float* lo = row_of(m0 + (lane & 31));
    const float* hi = row_of(m0 + 32 + (lane & 31));
    __builtin_assume(CH == 1 || D >= 4);
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const float4 p = dia_piece(lo, c, CH, lane >> 5, D), q = dia_piece(hi, c, CH, lane >> 5, D);
        v[8 * c + 0] = p.x; v[8 * c + 1] = p.y; v[8 * c + 2] = p.z; v[8 * c + 3] = p.w;
        v[8 * c + 4] = q.x; v[8 * c + 5] = q.y; v[8 * c + 6] = q.z; v[8 * c + 7] = q.w;
    }
#pragma unroll
    for (int c = 0; c < CH; ++c) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const auto w = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[8 * c + e]),
                                                            __float_as_uint(v[8 * c + 4 + e]), false, false);
            v[8 * c + e] = __uint_as_float(w[0]);
            v[8 * c + 4 + e] = __uint_as_float(w[1]);
        }
    }
}
// Returns the largest squared distance of the unit.
template <int CH>
__device__ __noinline__ float dia_unit_direct(const float* X, const int32_t* perm, int N, int D, int base, int n,
                                              int ma, int mb) {
    const int lane = threadIdx.x & 63, group = lane >> 4;
    D = __builtin_amdgcn_readfirstlane(D);
    const bool one = ma == mb && n - ma <= 32;
    const int passes = __builtin_amdgcn_readfirstlane(one ? 1 : (ma == mb ? 3 : 4));
    float x[8 * CH], y[8 * CH];
    dia_load_rows<CH>(y, X, perm, N, D, base, n, mb, lane);
    dia_load_rows<CH>(x, X, perm, N, D, base, n, ma, lane);
    if (one) {
        // group squares (columns, rows) of the one pass: (0,0) (1,1) (1,0) and (0,0) once more
        const int from = group == 1 || group == 2 ? 16 + (lane & 15) : lane & 15;
#pragma unroll
        for (int i = 0; i < 8 * CH; ++i) {
            y[i] = __shfl(y[i], from);
            x[i] = __shfl(x[i], group == 1 ? lane : lane & 15);
        }
    }
    float far = 0.f;
    for (int p = 0;; ++p) {
        float acc[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        // (a branch for every four features: in one block the compiler turns the values of all of
        // them ahead of their use, into registers that there are not)
#pragma unroll
        for (int q = 0; q < 2 * CH; ++q) {
            if (4 * q < D) {
#pragma unroll
                for (int i = 4 * q; i < 4 * q + 4; ++i) dia_turn(acc, x[i], y[i]);
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) far = fmaxf(far, acc[r]);
        if (p + 1 >= passes) break;
#pragma unroll
        for (int i = 0; i < 8 * CH; ++i) x[i] = __shfl(x[i], (lane + 16) & 63);
    }
    return wave_max_f(far);
}

// Pair of C/D element r: column lane & 31, row dia_row(r, lane / 32) of the tile.
__device__ __forceinline__ int dia_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// Appends the pairs of the lanes' mask bits; `same`: both operands are the same rows, only
// the pairs above the diagonal count.  Returns the new number of waiting pairs.  If a tile has
// more than kFlood, none of them stay and the unit and what is left of the cluster's share are
// evaluated whole (dia_unit_direct).  64: fewer, and continuous rows come near it (16: clusters of 350
// members of 32 features 93 -> 147 us).  One-hot rows, every distance the same, without / with
// the line: 1024 searches of 64-4096 rows of 48 features 3.5 / 0.40 ms, one of 40000 rows of 16
// features in 16 clusters 537 / 0.11 ms (every pair directly, as the kernel before the matrix
// cores did: 0.28 and 0.12 ms).
constexpr int kFlood = 64, kFloodBit = 1 << 16;
__device__ __forceinline__ int dia_push(const float* X, int D, unsigned* dmax, DiaQueue* q, int count, unsigned mask,
                                        int ra, int rb, int cid, bool same, int lane) {
    int pushed = 0, others = count;          // (waiting pairs of other tiles)
    while (__ballot(mask != 0u) != 0ull) {
        const int r = mask ? __builtin_ctz(mask) : 0;
        const int i = dia_row(r, lane >> 5), row = __shfl(ra, i);
        const bool take = mask != 0u && !(same && i >= (lane & 31));
        mask &= mask - 1u;
        const unsigned long long takers = __ballot(take);
        const int n = __popcll(takers);
        pushed += n;
        if (pushed > kFlood) return others | kFloodBit;
        if (count + n > kWave) { dia_drain(X, D, dmax, q, count); count = 0; others = 0; }
        if (take) {
            const int at = count + __popcll(takers & ((1ull << lane) - 1ull));
            q->row[at] = row; q->col[at] = rb; q->cluster[at] = cid;
        }
        count += n;
    }
    return count;
}

__device__ __forceinline__ f32x16 dia_norms(float na, float nb, f32x16 acc, int half) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(half ? 1.f : -0.5f * na, half ? -0.5f * nb : 1.f, acc, 0, 0, 0);
}
__device__ __forceinline__ float dia_min(const f32x16& acc) {
    float v = acc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) v = fminf(v, acc[r]);
    return wave_min_f(v);
}
__device__ __forceinline__ float dia_err(float M, int D) { return M * ((float)(10 * D + 40) * 0x1p-23f); }
// bits of the elements at or below -lim / 2
__device__ __forceinline__ unsigned dia_contenders(const f32x16& acc, float lim) {
    const float at = -0.5f * lim;
    unsigned mask = 0u;
#pragma unroll
    for (int r = 0; r < 16; ++r) mask |= acc[r] <= at ? 1u << r : 0u;
    return mask;
}

// What the fast form leaves: err not small against the largest value (a tight cluster far from
// the origin) - the tile is formed again relative to the cluster's first member `ctr`; rows that
// are not finite, or whose norms could overflow or vanish - every pair is evaluated.  Not
// inlined: its registers would cost dia_pairs a resident wave.  Returns `least` and the
// number of waiting pairs, kFloodBit beside it as in dia_push.
__device__ __noinline__ float2 dia_tile_slow(const float* X, int D, unsigned* dmax, DiaQueue* q, int count,
                                             const float* ctr, int ra, int rb, int cid, bool same, float least) {
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const float* x = X + (size_t)ra * D;
    const float* y = X + (size_t)rb * D;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    float na = 0.f, nb = 0.f;
    bool differ = false;
    const int chunks = (D + 7) >> 3;
    for (int c = 0; c < chunks; ++c) {
        const float4 o = dia_piece(ctr, c, chunks, half, D), u = dia_piece(x, c, chunks, half, D),
                     v = dia_piece(y, c, chunks, half, D);
        const float ov[4] = {o.x, o.y, o.z, o.w}, uv[4] = {u.x, u.y, u.z, u.w}, vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float xa = uv[e] - ov[e], xb = vv[e] - ov[e];
            differ = differ || !(uv[e] == ov[e] && vv[e] == ov[e]);
            na = fmaf(xa, xa, na);
            nb = fmaf(xb, xb, nb);
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(xa, xb, acc, 0, 0, 0);
        }
    }
    if (__ballot(differ) != 0ull) {                      // (all rows equal: no distance to add)
        na += __shfl_xor(na, 32);
        nb += __shfl_xor(nb, 32);
        acc = dia_norms(na, nb, acc, half);
        unsigned mask = 0xffffu;
        const float M = wave_max_f(fmaxf(na, nb));
        if (__ballot(!(na < 1e37f && nb < 1e37f)) == 0ull && M >= 1e-30f) {
            const float err = dia_err(M, D), far = -2.f * dia_min(acc);
            mask = dia_contenders(acc, fmaxf(far - 2.f * err, least - err));
            least = fmaxf(least, far - err);
        }
        count = dia_push(X, D, dmax, q, count, mask, ra, rb, cid, same, lane);
    }
    return make_float2(least, __int_as_float(count));
}

// One tile: pairs that may be the farthest go to the queue; returns the cluster's new `least`.
template <int CH>
__device__ __forceinline__ float dia_tile(const DiaArgs& a, DiaQueue* q, int& count, bool& tight, bool& flood,
                                          const DiaBlock<CH>& A, const DiaBlock<CH>& B, bool same, const float* ctr,
                                          int cid, float least, int lane) {
    if (flood) return least;
    const int half = lane >> 5;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    acc = dia_norms(A.norm, B.norm, acc, half);
#pragma unroll
    for (int i = 0; i < 4 * CH; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(A.v[i], B.v[i], acc, 0, 0, 0);
    const bool odd = __ballot(!(A.norm < 1e37f && B.norm < 1e37f)) != 0ull;
    const float M = wave_max_f(fmaxf(A.norm, B.norm)), far = -2.f * dia_min(acc), err = dia_err(M, a.D);
    if (odd || M < 1e-30f || err > 0.03f * fmaxf(far, least)) {
        const float2 r = dia_tile_slow(a.X, a.D, a.dmax, q, count, ctr, A.row, B.row, cid, same, least);
        count = __builtin_amdgcn_readfirstlane(__float_as_int(r.y));
        flood = flood || (count & kFloodBit) != 0;
        count &= kFloodBit - 1;
        tight = true;
        return lane_f(r.x, 0);
    }
    if (far < least - err) return least;
    const unsigned mask = dia_contenders(acc, fmaxf(far - 2.f * err, least - err));
    count = dia_push(a.X, a.D, a.dmax, q, count, mask, A.row, B.row, cid, same, lane);
    flood = flood || (count & kFloodBit) != 0;
    count &= kFloodBit - 1;
    return fmaxf(least, far - err);
}

// Units t .. t1 - 1.  Rows as they are need no centre to be read; CENTRED: rows relative to the
// first member of their cluster.  Returns where it stopped: at t1 or, without CENTRED,
// after a unit too tight for rows as they are.
template <int CH, bool CENTRED>
__device__ __forceinline__ long long dia_share(const DiaArgs& a, DiaQueue* q, int& waiting, long long t, long long t1,
                                               long long total, int nslots, int lane) {
    bool tight = false;
    int s = 0;                            // slot of the first unit: the last with first <= t
    for (int hi = nslots; hi - s > 1;) {
        const int mid = (s + hi) >> 1;
        if (a.slots[mid].first <= t) s = mid; else hi = mid;
    }
    for (; s < nslots && t < t1; ++s) {
        long long first = 0, next = total;
        int c0 = 0, c1 = a.Ksum;
        if (a.slots) {
            first = a.slots[s].first; c0 = a.slots[s].c0; c1 = a.slots[s].c1;
            if (s + 1 < nslots) next = a.slots[s + 1].first;
        }
        long long u = t - first;
        const long long uend = (t1 < next ? t1 : next) - first;
        if (c1 - c0 > kWave) {            // a cluster at or before that of unit u
            for (int hi = c1; hi - c0 > 1;) {
                const int mid = (c0 + hi) >> 1;
                if ((long long)a.toff[mid] <= u) c0 = mid; else hi = mid;
            }
        }
        for (; c0 < c1 && u < uend; c0 += kWave) {
            // 64 clusters at a time, one per lane
            const int cl = c0 + lane;
            const int wn = cl < c1 ? a.cnt[cl] : 0;
            const int wbase = cl < c1 ? a.off[cl] : 0;
            const int wfirst = cl < c1 ? a.toff[cl] : 0;
            const long long wend = wfirst + units_of(wn);
            while (u < uend) {
                const unsigned long long at = __ballot(wfirst <= u && u < wend);
                if (at == 0ull) break;
                const int l = (int)__builtin_ctzll(at);
                const int n = __builtin_amdgcn_readlane(wn, l);
                const int base = __builtin_amdgcn_readlane(wbase, l);
                const long long cf = __builtin_amdgcn_readlane(wfirst, l);
                long long ce = cf + units_of(n);
                ce = ce < uend ? ce : uend;
                if (base < 0 || (long long)base + n > a.N) { u = ce; continue; }
                const int cid = c0 + l;
                int r0 = __builtin_amdgcn_readfirstlane(a.perm[base]);
                r0 = (r0 >= 0 && r0 < a.N) ? r0 : 0;
                const float* ctr = a.X + (size_t)r0 * a.D;
                float least = lane_f(__uint_as_float(__hip_atomic_load(&a.dmax[cid], __ATOMIC_RELAXED,
                                                                       __HIP_MEMORY_SCOPE_AGENT)), 0);
                // units are numbered row by row over the upper triangle
                const int T = (n + 63) >> 6;
                int ta = 0;
                long long rem = u - cf;
                if (rem >= T) {
                    // rows before unit rem: ta T - ta (ta - 1) / 2 <= rem
                    const double h = (double)T + 0.5;
                    ta = (int)(h - sqrt(h * h - 2.0 * (double)rem));
                    ta = ta < 0 ? 0 : (ta > T - 1 ? T - 1 : ta);
                    const auto before = [T](long long r) { return r * T - r * (r - 1) / 2; };
                    while (ta > 0 && before(ta) > rem) --ta;
                    while (ta < T - 1 && before(ta + 1) <= rem) ++ta;
                    rem -= before(ta);
                }
                DiaBlock<CH> A0, A1, B;
                int held = -1;
                bool flood = false;
                for (; u < ce && ta < T; ++u) {
                    const int ma = 64 * ta, mb = 64 * (ta + (int)rem);
                    const bool two = ma + 32 < n;
                    if (held != ta) {
                        dia_load<CH>(a, A0, base, n, ma, lane);
                        dia_load<CH>(a, A1, base, n, ma + 32, lane);
                        dia_finish<CH>(A0, ctr, CENTRED, a.D, lane);
                        dia_finish<CH>(A1, ctr, CENTRED, a.D, lane);
                        held = ta;
                    }
                    for (int h = 0; h < 2 && mb + 32 * h < n; ++h) {
                        if (rem > 0) {
                            dia_load<CH>(a, B, base, n, mb + 32 * h, lane);
                            dia_finish<CH>(B, ctr, CENTRED, a.D, lane);
                        } else {
                            B = h ? A1 : A0;
                        }
                        least = dia_tile<CH>(a, q, waiting, tight, flood, A0, B, rem == 0 && h == 0, ctr, cid, least, lane);
                        // (on the diagonal the tile of A1 and the first half mirrors that of A0 and the second)
                        if (two && rem + h > 0)
                            least = dia_tile<CH>(a, q, waiting, tight, flood, A1, B, rem == 0, ctr, cid, least, lane);
                    }
                    if (flood) break;
                    if (!CENTRED && tight) { ce = u + 1; break; }
                    if (++rem >= T - ta) { rem = 0; ++ta; }
                }
                if (flood) {
                    // many contenders: this unit and the rest of the cluster's share whole
                    float whole = 0.f;
                    for (; u < ce && ta < T; ++u) {
                        whole = fmaxf(whole, dia_unit_direct<CH>(a.X, a.perm, (int)a.N, a.D, base, n, 64 * ta,
                                                                 64 * (ta + (int)rem)));
                        if (++rem >= T - ta) { rem = 0; ++ta; }
                    }
                    if (lane == 0 && __float_as_uint(whole) >
                                         __hip_atomic_load(&a.dmax[cid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                        atomicMax(&a.dmax[cid], __float_as_uint(whole));
                }
                if (!CENTRED && tight) return first + ce;
                u = ce;
            }
        }
        t = first + uend;
    }
    return t1;
}

// The units of member pairs (units_of) of all clusters are numbered in one sequence and every wave
// takes an equal, contiguous share, so the work is balanced whatever the cluster sizes are.
// A wave keeps the 64 rows of a unit in the operand registers (no LDS, no barrier) and the
// 64 columns beside them; the row side stays for the next unit of the same rows.  The
// maximum of a run of units of one cluster goes to the cluster's maximum with an integer
// atomic max on the float's bits (non-negative floats order like their bit patterns).
//
// 43000 units of 36000 clusters of 48 features, mostly below 64 members (1024 searches of 64-4096
// candidates): 144 us, of which the matrix instructions are 50 us and the vector ones about as
// much; 16 x 16 threads with 4 x 4 pairs each of direct differences through LDS, two barriers
// per 16 features, took 247 us.  Representatives and diameters of that batch
// 390 -> 269 us; clusters of 100-1000 members twice as fast.
template <int CH>
__global__ void __launch_bounds__(kThreads, CH <= 6 ? 3 : 2) dia_pairs(DiaArgs a) {
    __shared__ DiaQueue queue[kWaves];
    const int lane = threadIdx.x & 63;
    DiaQueue* q = &queue[threadIdx.x >> 6];
    int waiting = 0;
    const long long wave = (long long)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long long waves = (long long)gridDim.x * kWaves;
    const unsigned long long res = a.slots ? *a.reserved : 0ull;
    const long long total = a.slots ? (long long)(res & ((1ull << kUnitBits) - 1)) : (long long)a.toff[a.Ksum];
    const long long taken = (long long)(res >> kUnitBits);
    const int nslots = a.slots ? (int)(taken < a.max_slots ? taken : a.max_slots) : 1;
    const long long per = (total + waves - 1) / waves;
    const long long t0 = per * wave;
    const long long t1 = t0 + per < total ? t0 + per : total;
    if (t0 >= t1) return;
    const long long t = dia_share<CH, false>(a, q, waiting, t0, t1, total, nslots, lane);
    if (t < t1) dia_share<CH, true>(a, q, waiting, t, t1, total, nslots, lane);
    dia_drain(a.X, a.D, a.dmax, q, waiting);
}

// Short searches: one wave per search, four searches per workgroup.  (The walks above
// take the searches of a range one after the other with barriers around each, and the
// grouping, the prefix sums and the tile numbering are seven launches: 0.34 ms for 183
// searches of a few dozen candidates.)  Lane l takes candidates l, l + 64, ... and
// compares each with the later members of its cluster; a pair's squared distance is
// the same chain of fused multiply-adds over the features in index order as in the
// tiles above, so the maxima are the same bits.
__global__ void __launch_bounds__(kThreads) dia_wave(DiaArgs a) {
    extern __shared__ unsigned wmax[];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = (int)blockIdx.x * kWaves + wv;
    if (g >= a.G) return;                 // (a whole wave leaves: no wave waits for another in this kernel)
    const int D = a.D;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (K > a.Kmax) K = a.Kmax;
    if (K <= 0) return;
    if (a.mixed && ng > kDiaShort) return;            // the tile kernels take this search
    unsigned* lmax = wmax + (size_t)wv * a.Kmax;      // [Kmax] bits of the largest squared distance
    for (int j = lane; j < K; j += kWave) lmax[j] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    const bool vec = (D & 3) == 0;
    for (int p = lane; p < ng; p += kWave) {
        int jp = a.assign[(size_t)n0 + p];
        jp = (jp >= 0 && jp < K) ? jp : 0;
        const float* xp = a.X + ((size_t)n0 + p) * D;
        float far = 0.f;
        for (int q = p + 1; q < ng; ++q) {
            int jq = a.assign[(size_t)n0 + q];
            jq = (jq >= 0 && jq < K) ? jq : 0;
            if (jq != jp) continue;
            const float* xq = a.X + ((size_t)n0 + q) * D;
            float acc = 0.f;
            if (vec) {
                for (int d = 0; d < D; d += 4) {
                    const float4 u = *reinterpret_cast<const float4*>(xp + d);
                    const float4 v = *reinterpret_cast<const float4*>(xq + d);
                    float e = u.x - v.x; acc = fmaf(e, e, acc);
                    e = u.y - v.y; acc = fmaf(e, e, acc);
                    e = u.z - v.z; acc = fmaf(e, e, acc);
                    e = u.w - v.w; acc = fmaf(e, e, acc);
                }
            } else {
                for (int d = 0; d < D; ++d) {
                    const float e = xp[d] - xq[d];
                    acc = fmaf(e, e, acc);
                }
            }
            far = fmaxf(far, acc);
        }
        if (far > 0.f) atomicMax(&lmax[jp], __float_as_uint(far));
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (int j = lane; j < K; j += kWave) {
        if (a.mixed) a.dmax[k0 + j] = lmax[j];        // dia_final takes the root of every cluster
        else a.diam[k0 + j] = sqrtf(__uint_as_float(lmax[j]));
    }
}

__global__ void __launch_bounds__(kThreads) dia_final(DiaArgs a) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < a.Ksum) a.diam[i] = sqrtf(__uint_as_float(a.dmax[i]));
}

}  // namespace

// As many workgroups as the chip holds at once (three or two per compute unit); each wave takes an
// equal share of the units, whose number is only known on the device.  (1024 searches of
// 64-4096 candidates: 144 us; twice as many workgroups 150 us, 2048 156 us, 4096 161 us.)
static void launch_pairs(const DiaArgs& a, hipStream_t st) {
    const dim3 grid(a.D <= 48 ? 768 : 512), block(kThreads);
    switch ((a.D + 7) / 8) {
        case 1: hipLaunchKernelGGL(dia_pairs<1>, grid, block, 0, st, a); break;
        case 2: hipLaunchKernelGGL(dia_pairs<2>, grid, block, 0, st, a); break;
        case 3: hipLaunchKernelGGL(dia_pairs<3>, grid, block, 0, st, a); break;
        case 4: hipLaunchKernelGGL(dia_pairs<4>, grid, block, 0, st, a); break;
        case 5: hipLaunchKernelGGL(dia_pairs<5>, grid, block, 0, st, a); break;
        case 6: hipLaunchKernelGGL(dia_pairs<6>, grid, block, 0, st, a); break;
        case 7: hipLaunchKernelGGL(dia_pairs<7>, grid, block, 0, st, a); break;
        default: hipLaunchKernelGGL(dia_pairs<8>, grid, block, 0, st, a); break;      // (KB_MAX_D = 64)
    }
}

hipError_t launch_diameter(const kb_batch& b, const DiameterCall& c, hipStream_t st) {
    if (b.Ksum <= 0) return hipSuccess;
    DiaArgs a;
    a.G = b.G; a.D = b.D; a.Ksum = b.Ksum; a.Kmax = b.Kmax > 0 ? b.Kmax : 1; a.N = b.N;
    a.seg_off = b.seg_off; a.koff = b.koff; a.X = c.X; a.assign = c.assign; a.diam = c.diam;
    a.cnt = c.cnt; a.off = c.off; a.toff = c.toff; a.bsum = c.bsum; a.dmax = reinterpret_cast<unsigned*>(c.diam); a.perm = c.perm;
    a.slots = nullptr; a.reserved = nullptr; a.max_slots = b.N / 2;
    const unsigned kblocks = (unsigned)((b.Ksum + kThreads - 1) / kThreads);
    const unsigned ranges = (unsigned)((b.N + kRange - 1) / kRange);
    // a batch of short searches only: a wave per search, one launch; a batch of mostly
    // short searches (256 candidates or fewer on average) with longer ones among them: the
    // wave kernel after the maxima are zeroed, then the grouping and the tiles, which leave
    // the short searches out
    a.mixed = b.Nmax > kDiaShort && b.G > 1 && b.N <= (int64_t)kShortSearch * b.G;
    const size_t wlds = (size_t)kWaves * 4 * (b.Kmax > 0 ? b.Kmax : 1);
    const dim3 wgrid((unsigned)((b.G + kWaves - 1) / kWaves));
    if (b.Nmax <= kDiaShort && b.G > 0) {
        hipLaunchKernelGGL(dia_wave, wgrid, dim3(kThreads), wlds, st, a);
        return hipGetLastError();
    }
    // (dia_group takes the short searches in passing: 3000 searches of 20-90 candidates 139 us with
    // the wave kernel, the walks and the prefix sums, 73 us here)
    if (b.Nmax <= kGroupMax) {
        a.slots = reinterpret_cast<DiaSlot*>(c.slots);
        a.reserved = reinterpret_cast<unsigned long long*>(c.bsum);
        hipLaunchKernelGGL(dia_zero, dim3(kblocks), dim3(kThreads), 0, st, a);
        if (b.G >= kGroupMany)
            hipLaunchKernelGGL(dia_group<kGroupSearches>, dim3((unsigned)((b.G + kGroupSearches - 1) / kGroupSearches)),
                               dim3(kGroupThreads), 0, st, a);
        else
            hipLaunchKernelGGL(dia_group<1>, dim3((unsigned)b.G), dim3(kGroupThreads), 0, st, a);
        launch_pairs(a, st);
        hipLaunchKernelGGL(dia_final, dim3(kblocks), dim3(kThreads), 0, st, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(dia_zero, dim3(kblocks), dim3(kThreads), 0, st, a);
    if (a.mixed) hipLaunchKernelGGL(dia_wave, wgrid, dim3(kThreads), wlds, st, a);
    if (ranges) hipLaunchKernelGGL(dia_walk<false>, dim3(ranges), dim3(kThreads), 0, st, a);
    const int nscan = (b.Ksum + kScanBlock - 1) / kScanBlock;
    hipLaunchKernelGGL(dia_bsum, dim3((unsigned)nscan), dim3(kThreads), 0, st, a);
    hipLaunchKernelGGL(dia_bscan, dim3(1), dim3(kThreads), 0, st, a, nscan);
    hipLaunchKernelGGL(dia_apply, dim3((unsigned)nscan), dim3(kThreads), 0, st, a);
    if (ranges) hipLaunchKernelGGL(dia_walk<true>, dim3(ranges), dim3(kThreads), 0, st, a);
    launch_pairs(a, st);
    hipLaunchKernelGGL(dia_final, dim3(kblocks), dim3(kThreads), 0, st, a);
    return hipGetLastError();
}

}  // namespace kb
