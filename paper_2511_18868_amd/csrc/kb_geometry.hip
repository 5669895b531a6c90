// Cluster representatives and radii (Sec. 3.3 "Representative profiling"; Alg. 1
// "Update centroids k_c"; covering term of Theorem 1).
//
// For every candidate the squared distance to its own centroid is formed exactly
// as the plain definition does - fp64, direct differences, summed over the
// features in index order with separate multiply and add - so the per-cluster
// minimum (the representative, lowest index on ties) and maximum (the radius)
// are exact and need no tolerance.
//
//   geo_dist and geo_merge, or in batches with searches of more than kGeoMergeMax candidates and
//   in mixed ones geo_init, geo_dist, geo_rep, geo_final:
//   geo_init   per-cluster tables: min = all ones, max = 0, rep = none
//   geo_dist   one workgroup per flat range of candidates walks the searches that
//              intersect it.  Per search piece the centroids are staged in LDS;
//              tiles of 256 rows are fetched with coalesced 16-byte loads (the
//              next tile is requested before the current one is worked on),
//              transposed through LDS (padded row stride: conflict-free) so
//              that each thread owns one candidate, and the distances are reduced
//              per cluster with 64-bit integer LDS atomics on their bit patterns
//              (non-negative doubles order like unsigned integers), then merged
//              into the global tables.  The distance of every candidate is kept.
//              With geo_merge to follow, the workgroup itself finds the representatives
//              of its pieces: a search that lies inside the range is finished, of the at
//              most two others (one that began before it, one that goes on after it) the
//              results per cluster wait in a slot of the range.
//   geo_merge  a wave per search merges the slots of a search that crosses a border.
//   geo_rep    second, light pass (12 bytes per candidate): the candidates whose
//              distance equals their cluster's minimum compete for the lowest
//              index with an integer atomic min.
//   geo_final  rep = -1 for empty clusters, radius = sqrt(max) rounded to fp32.
#include "kb_internal.h"

namespace kb {

namespace {

constexpr int kThreads = 256;
constexpr int kNone = 0x7fffffff;
constexpr int kGeoRangeMin = 512, kGeoFill = 300, kGeoFillRagged = 600;
constexpr int kGeoMergeMax = 16384;    // longer searches: a wave of geo_merge would walk many slots

struct GeoArgs {
    int G, D, Ksum, Kmax;
    int64_t N;
    const int32_t* seg_off;
    const int32_t* koff;
    const float* X;
    const float* cent;
    const int32_t* assign;
    int32_t* rep;
    float* radius;
    double* d2;                    // [N]
    unsigned long long* gmin;      // [Ksum]
    unsigned long long* gmax;      // [Ksum]
    unsigned char* spare;          // [4 N] bytes: slots of searches that began before a range
    int range;                     // candidates per workgroup
    int merged;                    // 1: geo_merge follows, gmin / gmax are not used
    int mixed;                     // 1: searches of at most kShortSearch candidates go to geo_wave, longer
                                   //    ones to the range kernels, in the same call
};

// Slot of a range: what one piece of a search gives, per cluster.  A piece that began before
// range r: slot in the 4 bytes per candidate of range r - 1 in `spare` (r >= 1, so that range
// is whole); a piece that goes on after range r: in the 8 bytes per candidate of range r in
// d2, whose distances only this workgroup reads, and it has.
struct GeoSlot {
    unsigned long long* least;     // [Kmax] bits of the smallest squared distance
    unsigned long long* most;      // [Kmax] and of the largest
    int32_t* rep;                  // [Kmax] lowest candidate at the smallest, kNone
};
static_assert(20 * KB_MAX_K <= 4 * kGeoRange, "a slot fits the bytes of a range");     // (range_of: of a shorter one)
__device__ __forceinline__ GeoSlot geo_slot(const GeoArgs& a, int64_t range, bool began_before) {
    unsigned char* base = began_before ? a.spare + (range - 1) * (4 * (int64_t)a.range)
                                       : reinterpret_cast<unsigned char*>(a.d2) + range * (8 * (int64_t)a.range);
    GeoSlot s;
    s.least = reinterpret_cast<unsigned long long*>(base);
    s.most = s.least + a.Kmax;
    s.rep = reinterpret_cast<int32_t*>(s.most + a.Kmax);
    return s;
}

__global__ void __launch_bounds__(kThreads) geo_init(GeoArgs a) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < a.Ksum) { a.gmin[i] = ~0ull; a.gmax[i] = 0ull; a.rep[i] = kNone; }
}

// VEC = 4: D is a multiple of 4 and pieces of 16 bytes stay inside a row; VEC = 1: any D, the tile is
// one run of floats all the same, fetched in 16-byte pieces that may cross from row to row.
// kPieces: pieces of a thread (4 times as many features at most).  They are its registers, and with them
// the workgroups of a unit: as many forms as make a difference (one for all rows of 17 features and more / these:
// 300 searches of 4489-9820 rows of 17 82 / 50 us, 256 of 4395-7118 of 33 103 / 62).
template <int VEC, int kPieces>
__global__ void __launch_bounds__(kThreads, VEC == 4 ? 1 : kPieces <= 8 ? 4 : kPieces <= 12 ? 3 : 2) geo_dist(GeoArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x;
    // row stride of the transposed tile: D + 4 words keeps 16-byte pieces aligned and
    // spreads consecutive rows over the banks (conflict-free 16-byte reads whenever
    // D/4 is even); the next odd number for the scalar path
    const int D = a.D, DP = VEC == 4 ? D + 4 : (D | 1);
    unsigned long long* lmin = reinterpret_cast<unsigned long long*>(smem);          // [Kmax]
    unsigned long long* lmax = lmin + a.Kmax;                                         // [Kmax]
    float* lc = reinterpret_cast<float*>(lmax + a.Kmax);                              // [Kmax * D]
    float* lx = lc + (size_t)a.Kmax * D;                                              // [256 * DP]

    const int64_t r0 = (int64_t)blockIdx.x * a.range;
    if (r0 >= a.N) return;
    const int64_t r1 = r0 + a.range < a.N ? r0 + a.range : a.N;

    // position of this thread's pieces inside a tile: piece i of the thread begins at
    // element 4 (tid + 256 i) of the tile = (row, col); advancing i adds
    // (qd, rd) with a carry
    const int step = 4 * kThreads;
    const int qd = step / D, rd = step - qd * D;
    const int row0 = (4 * tid) / D, col0 = 4 * tid - row0 * D;
    const int npieces = (D + 3) / 4;              // pieces per thread of a full tile

    int lo = 0, hi = a.G;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)a.seg_off[mid] <= r0) lo = mid; else hi = mid;
    }
    const auto mine = [&](int n0, int ng, int k0, int K) {
        return n0 >= r1 || (ng > 0 && K > 0 && !(a.mixed && ng <= kShortSearch));
    };
    for (int g = lo; (g = next_search(a.seg_off, a.koff, g, a.G, a.N, a.Ksum, mine)) < a.G; ++g) {
        int n0, ng, k0, K;
        search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
        if (K > a.Kmax) K = a.Kmax;
        if (n0 >= r1) break;
        if (ng <= 0 || K <= 0) continue;
        if (a.mixed && ng <= kShortSearch) continue;      // (uniform) a wave of geo_wave takes this search
        const int q0 = r0 > n0 ? (int)r0 : n0;
        const int q1 = r1 < (int64_t)n0 + ng ? (int)r1 : n0 + ng;
        if (q0 >= q1) continue;

        // centroids of the search -> LDS
        {
            const float* cg = a.cent + (size_t)k0 * D;
            const int total = K * D;
            if constexpr (VEC == 4) {
                for (int i = tid; i < total / 4; i += kThreads)
                    reinterpret_cast<float4*>(lc)[i] = reinterpret_cast<const float4*>(cg)[i];
            } else {
                for (int i = tid; i < total; i += kThreads) lc[i] = cg[i];
            }
            for (int j = tid; j < K; j += kThreads) { lmin[j] = ~0ull; lmax[j] = 0ull; }
        }

        float xr[kPieces][4];
        auto fetch = [&](int tb) {
            const int cnt = q1 - tb < kThreads ? q1 - tb : kThreads;
            const int total = cnt * D;
            const float* src = a.X + (size_t)tb * D;
#pragma unroll
            for (int i = 0; i < kPieces; ++i) {
                const int at = 4 * (tid + i * kThreads);
                if (i < npieces && at < total) {
                    // (the last piece is moved back so that it ends with the tile, and shifted when it is stored)
                    float4 v;
                    if constexpr (VEC == 4) {
                        v = *reinterpret_cast<const float4*>(src + at);
                    } else if (total >= 4) {
                        v = load4(src + (at + 4 <= total ? at : total - 4));
                    } else {
                        v = make_float4(0.f, total > 2 ? src[0] : 0.f, total > 1 ? src[total - 2] : 0.f, src[total - 1]);
                    }
                    xr[i][0] = v.x; xr[i][1] = v.y; xr[i][2] = v.z; xr[i][3] = v.w;
                }
            }
        };
        fetch(q0);
        for (int tb = q0; tb < q1; tb += kThreads) {
            const int cnt = q1 - tb < kThreads ? q1 - tb : kThreads;
            const int total = cnt * D;
            // registers -> LDS, one row per candidate
            {
                int row = row0, col = col0;
#pragma unroll
                for (int i = 0; i < kPieces; ++i) {
                    const int at = 4 * (tid + i * kThreads);
                    if (i < npieces && at < total) {
                        float* dst = lx + row * DP + col;
                        if constexpr (VEC == 4) {
                            *reinterpret_cast<float4*>(dst) = make_float4(xr[i][0], xr[i][1], xr[i][2], xr[i][3]);
                        } else {
                            // (from the end of a row to the start of the next: DP - D words are skipped)
                            float v[4] = {xr[i][0], xr[i][1], xr[i][2], xr[i][3]};
                            const int over = at + 4 - total;          // values of the last piece that came before it
                            if (over > 0) {
                                if (over & 1) { v[0] = v[1]; v[1] = v[2]; v[2] = v[3]; }
                                if (over & 2) { v[0] = v[2]; v[1] = v[3]; }
                            }
                            int c = col;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                if (e + over < 4) *dst = v[e];
                                ++dst;
                                if (++c == D) { c = 0; dst += DP - D; }
                            }
                        }
                    }
                    row += qd; col += rd;
                    if (col >= D) { col -= D; row += 1; }
                }
            }
            const int p = tb + tid;
            int j = p < q1 ? a.assign[p] : 0;
            j = (j >= 0 && j < K) ? j : 0;
            __syncthreads();
            if (tb + kThreads < q1) fetch(tb + kThreads);
            if (tid < cnt) {
                const float* xrow = lx + tid * DP;
                const float* crow = lc + (size_t)j * D;
                double acc = 0.0;
                if constexpr (VEC == 4) {
                    // 16-byte LDS reads, eight features in flight; the sum itself stays
                    // in index order
#pragma unroll 2
                    for (int d = 0; d < D; d += 4) {
                        const float4 xv = *reinterpret_cast<const float4*>(xrow + d);
                        const float4 cv = *reinterpret_cast<const float4*>(crow + d);
                        double diff = __dsub_rn((double)xv.x, (double)cv.x);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                        diff = __dsub_rn((double)xv.y, (double)cv.y);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                        diff = __dsub_rn((double)xv.z, (double)cv.z);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                        diff = __dsub_rn((double)xv.w, (double)cv.w);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                    }
                } else {
                    // eight features' values requested before the first is used; the sum
                    // itself stays in index order
                    int d = 0;
                    for (; d + 8 <= D; d += 8) {
                        float xv[8], cv[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) { xv[u] = xrow[d + u]; cv[u] = crow[d + u]; }
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const double diff = __dsub_rn((double)xv[u], (double)cv[u]);
                            acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                        }
                    }
                    for (; d < D; ++d) {
                        const double diff = __dsub_rn((double)xrow[d], (double)crow[d]);
                        acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                    }
                }
                a.d2[p] = acc;
                const unsigned long long bits = (unsigned long long)__double_as_longlong(acc);
                atomicMin(&lmin[j], bits);
                atomicMax(&lmax[j], bits);
            }
            __syncthreads();
        }
        if (a.merged) {
            int* lrep = reinterpret_cast<int*>(lx);       // (the tile is done with)
            for (int j = tid; j < K; j += kThreads) lrep[j] = kNone;
            __syncthreads();
            // (a thread reads back the distances it wrote itself)
            for (int p = q0 + tid; p < q1; p += kThreads) {
                int j = a.assign[p];
                j = (j >= 0 && j < K) ? j : 0;
                if ((unsigned long long)__double_as_longlong(a.d2[p]) == lmin[j]) atomicMin(&lrep[j], p);
            }
            __syncthreads();
            const bool before = n0 < r0, after = (int64_t)n0 + ng > r1;
            if (before || after) {
                const GeoSlot o = geo_slot(a, blockIdx.x, before);
                for (int j = tid; j < K; j += kThreads) {
                    o.least[j] = lmin[j]; o.most[j] = lmax[j]; o.rep[j] = lrep[j];
                }
            } else {
                for (int j = tid; j < K; j += kThreads) {
                    a.rep[k0 + j] = lrep[j] == kNone ? -1 : lrep[j];
                    a.radius[k0 + j] = (float)sqrt(__longlong_as_double((long long)lmax[j]));
                }
            }
            __syncthreads();
            continue;
        }
        for (int j = tid; j < K; j += kThreads) {
            if (lmin[j] != ~0ull) {
                atomicMin(&a.gmin[k0 + j], lmin[j]);
                atomicMax(&a.gmax[k0 + j], lmax[j]);
            }
        }
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kThreads) geo_rep(GeoArgs a) {
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * a.range;
    if (r0 >= a.N) return;
    const int64_t r1 = r0 + a.range < a.N ? r0 + a.range : a.N;
    int lo = 0, hi = a.G;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)a.seg_off[mid] <= r0) lo = mid; else hi = mid;
    }
    const auto mine = [&](int n0, int ng, int k0, int K) {
        return n0 >= r1 || (ng > 0 && K > 0 && !(a.mixed && ng <= kShortSearch));
    };
    for (int g = lo; (g = next_search(a.seg_off, a.koff, g, a.G, a.N, a.Ksum, mine)) < a.G; ++g) {
        int n0, ng, k0, K;
        search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
        if (K > a.Kmax) K = a.Kmax;
        if (n0 >= r1) break;
        if (ng <= 0 || K <= 0) continue;
        if (a.mixed && ng <= kShortSearch) continue;
        const int q0 = r0 > n0 ? (int)r0 : n0;
        const int q1 = r1 < (int64_t)n0 + ng ? (int)r1 : n0 + ng;
        for (int p = q0 + tid; p < q1; p += kThreads) {
            int j = a.assign[p];
            j = (j >= 0 && j < K) ? j : 0;
            const unsigned long long bits = (unsigned long long)__double_as_longlong(a.d2[p]);
            if (bits == a.gmin[k0 + j]) atomicMin(&a.rep[k0 + j], p);
        }
    }
}

__global__ void __launch_bounds__(kThreads) geo_final(GeoArgs a) {
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= a.Ksum) return;
    if (a.rep[i] == kNone) a.rep[i] = -1;
    a.radius[i] = (float)sqrt(__longlong_as_double((long long)a.gmax[i]));
}

// Searches that cross a border of ranges, and the clusters of searches without candidates: a
// wave for every 64 clusters of a search, four slots' values in flight.
// (With it one light launch follows geo_dist in place of two, one of them over all candidates,
// and one before it: representatives and diameters of 1024 searches of 64-4096 candidates 269 -> 255 us,
// ten iterations of 512 such searches with two re-clusterings 1359 -> 1337 us.  With a wave for all
// clusters of a search, slot by slot, one search of 16384 candidates and 256 clusters took 50 us in
// place of the 43 us before; now 37.)
__global__ void __launch_bounds__(kThreads) geo_merge(GeoArgs a, int parts) {
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t)blockIdx.x * (kThreads / kWave) + (int64_t)(threadIdx.x >> 6);
    const int g = (int)(w / parts), part = (int)(w - (int64_t)g * parts);
    if (g >= a.G) return;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    const int Kc = ng <= 0 ? 0 : (K > a.Kmax ? a.Kmax : K);
    for (int j = Kc + kWave * part + lane; j < K; j += kWave * parts) { a.rep[k0 + j] = -1; a.radius[k0 + j] = 0.f; }
    const int j = kWave * part + lane;
    if (j >= Kc) return;
    const int64_t ra = n0 / a.range, rb = ((int64_t)n0 + ng - 1) / a.range;
    if (ra == rb) return;                                // finished by its range
    unsigned long long least = ~0ull, most = 0ull;
    int rep = kNone;
#pragma unroll 4
    for (int64_t r = ra; r <= rb; ++r) {                 // (ascending: the lowest candidate on ties)
        const GeoSlot o = geo_slot(a, r, r != ra);
        const unsigned long long m = o.least[j], x = o.most[j];
        const int p = o.rep[j];
        rep = m < least ? p : rep;
        least = m < least ? m : least;
        most = x > most ? x : most;
    }
    a.rep[k0 + j] = rep == kNone ? -1 : rep;
    a.radius[k0 + j] = (float)sqrt(__longlong_as_double((long long)most));
}

// Batches of short searches: one wave per search, four searches per workgroup, the
// whole pass in one launch.  (A workgroup of the range kernels above walks the
// searches of its range one after the other with barriers around each; with a few
// dozen candidates per search that is hundreds of searches in a row.)  Same distances
// - the same fp64 operations in the same order - and the same exact comparisons, so
// the same representatives and radii.  Any search length is handled (the distances
// wait in d2 between the two sweeps); short ones are what it is launched for.
template <int VEC>
__global__ void __launch_bounds__(kThreads) geo_wave(GeoArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = (int)blockIdx.x * (kThreads / kWave) + wv;
    if (g >= a.G) return;                 // (a whole wave leaves: no wave waits for another in this kernel)
    const int D = a.D;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (K > a.Kmax) K = a.Kmax;
    if (K <= 0) return;
    if (a.mixed && ng > kShortSearch) return;         // the range kernels take this search
    unsigned long long* lmin = reinterpret_cast<unsigned long long*>(smem) + (size_t)wv * 2 * a.Kmax;   // [Kmax]
    unsigned long long* lmax = lmin + a.Kmax;                                                            // [Kmax]
    int* lrep = reinterpret_cast<int*>(smem + (size_t)(kThreads / kWave) * 16 * a.Kmax) + (size_t)wv * a.Kmax;   // [Kmax]
    for (int j = lane; j < K; j += kWave) { lmin[j] = ~0ull; lmax[j] = 0ull; lrep[j] = kNone; }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (int p = n0 + lane; p < n0 + ng; p += kWave) {
        int j = a.assign[p];
        j = (j >= 0 && j < K) ? j : 0;
        const float* xrow = a.X + (size_t)p * D;
        const float* crow = a.cent + (size_t)(k0 + j) * D;
        double acc = 0.0;
        if constexpr (VEC == 4) {
            for (int d = 0; d < D; d += 4) {
                const float4 xv = *reinterpret_cast<const float4*>(xrow + d);
                const float4 cv = *reinterpret_cast<const float4*>(crow + d);
                double diff = __dsub_rn((double)xv.x, (double)cv.x);
                acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                diff = __dsub_rn((double)xv.y, (double)cv.y);
                acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                diff = __dsub_rn((double)xv.z, (double)cv.z);
                acc = __dadd_rn(acc, __dmul_rn(diff, diff));
                diff = __dsub_rn((double)xv.w, (double)cv.w);
                acc = __dadd_rn(acc, __dmul_rn(diff, diff));
            }
        } else {
            for (int d = 0; d < D; ++d) {
                const double diff = __dsub_rn((double)xrow[d], (double)crow[d]);
                acc = __dadd_rn(acc, __dmul_rn(diff, diff));
            }
        }
        a.d2[p] = acc;
        const unsigned long long bits = (unsigned long long)__double_as_longlong(acc);
        atomicMin(&lmin[j], bits);
        atomicMax(&lmax[j], bits);
    }
    // (a lane reads back only the distances it wrote itself)
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (int p = n0 + lane; p < n0 + ng; p += kWave) {
        int j = a.assign[p];
        j = (j >= 0 && j < K) ? j : 0;
        const unsigned long long bits = (unsigned long long)__double_as_longlong(a.d2[p]);
        if (bits == lmin[j]) atomicMin(&lrep[j], p);
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    for (int j = lane; j < K; j += kWave) {
        if (a.mixed) {
            // geo_final finishes every cluster of the batch from the global tables
            a.rep[k0 + j] = lrep[j];
            a.gmax[k0 + j] = lmax[j];
        } else {
            a.rep[k0 + j] = lrep[j] == kNone ? -1 : lrep[j];
            a.radius[k0 + j] = (float)sqrt(__longlong_as_double((long long)lmax[j]));
        }
    }
}

}  // namespace

size_t geometry_lds_bytes(int Kmax, int D) {
    return (size_t)16 * Kmax + (size_t)4 * Kmax * D + (size_t)4 * kThreads * (D + 4);
}

// Candidates per workgroup: as many as leave every compute unit the workgroups that its LDS holds, two, or
// one where centroids and rows of whole pieces take half of it (more where a piece crosses rows and takes longer), if the slots
// of the shorter ranges hold a search's clusters.  geo_dist, 2048 / this (us): 512 searches of 64-4096 rows of 48
// features 44 / 35 (in ranges of 512 42), 200 of them 44 / 23, one of 10000 rows of 32 18 / 7.5; 1000 of 70-1900
// rows of 50 97 / 64 with pieces that cross rows (value by value 120), 300 of them 111 / 31; 1000 of 284-839
// rows of 64, K = 52, whose workgroups have a unit to themselves, 64 as if two fitted and 59.
static int range_of(const kb_batch& b) {
    const bool two = geometry_lds_bytes(b.Kmax, b.D) <= 80 * 1024;
    const int fill = (b.D & 3) != 0 ? kGeoFillRagged : two ? kGeoFill : kGeoFill / 2;
    int range = kGeoRange;
    while (range > kGeoRangeMin && b.N < (int64_t)fill * range && 5 * (int64_t)b.Kmax <= range / 2) range /= 2;
    return range;
}

hipError_t launch_geometry(const kb_batch& b, const GeoCall& c, hipStream_t st) {
    GeoArgs a;
    a.G = b.G; a.D = b.D; a.Ksum = b.Ksum; a.Kmax = b.Kmax > 0 ? b.Kmax : 1; a.N = b.N;
    a.seg_off = b.seg_off; a.koff = b.koff; a.X = c.X; a.cent = c.cent; a.assign = c.assign;
    a.rep = c.rep; a.radius = c.radius; a.d2 = c.d2; a.gmin = c.gmin; a.gmax = c.gmax;
    a.spare = reinterpret_cast<unsigned char*>(c.spare); a.merged = 0;
    a.range = range_of(b);
    if (b.Ksum <= 0) return hipSuccess;
    // a batch of short searches only: a wave per search, one launch; a batch of mostly
    // short searches (256 candidates or fewer on average) with longer ones among them: the
    // wave kernel after the tables are initialised, then the range kernels, each skipping
    // the other's searches.  (Where short searches are the exception the range kernels
    // take them in passing: on the largest benchmark the extra launch cost more than it saved.)
    a.mixed = b.Nmax > kShortSearch && b.G > 1 && b.N <= (int64_t)kShortSearch * b.G;
    const size_t wlds = (size_t)(kThreads / kWave) * 20 * a.Kmax;
    const dim3 wgrid((unsigned)((b.G + kThreads / kWave - 1) / (kThreads / kWave)));
    if (wlds > 64 * 1024) return hipErrorInvalidValue;
    if (b.Nmax <= kShortSearch && b.G > 0) {
        if ((b.D & 3) == 0) hipLaunchKernelGGL(geo_wave<4>, wgrid, dim3(kThreads), wlds, st, a);
        else hipLaunchKernelGGL(geo_wave<1>, wgrid, dim3(kThreads), wlds, st, a);
        return hipGetLastError();
    }
    const unsigned kblocks = (unsigned)((b.Ksum + kThreads - 1) / kThreads);
    a.merged = !a.mixed && b.Nmax <= kGeoMergeMax;
    if (!a.merged) hipLaunchKernelGGL(geo_init, dim3(kblocks), dim3(kThreads), 0, st, a);
    if (a.mixed) {
        if ((b.D & 3) == 0) hipLaunchKernelGGL(geo_wave<4>, wgrid, dim3(kThreads), wlds, st, a);
        else hipLaunchKernelGGL(geo_wave<1>, wgrid, dim3(kThreads), wlds, st, a);
    }
    const unsigned ranges = (unsigned)((b.N + a.range - 1) / a.range);
    if (ranges) {
        const size_t lds = geometry_lds_bytes(a.Kmax, b.D);
        if (lds > 160 * 1024) return hipErrorInvalidValue;
        const auto go = [&](auto kern) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(kern, dim3(ranges), dim3(kThreads), lds, st, a);
            return hipSuccess;
        };
        const hipError_t e = (b.D & 3) == 0 ? go(geo_dist<4, 16>) : b.D <= 16 ? go(geo_dist<1, 4>)
                             : b.D <= 32 ? go(geo_dist<1, 8>) : b.D <= 48 ? go(geo_dist<1, 12>) : go(geo_dist<1, 16>);
        if (e != hipSuccess) return e;
        if (!a.merged) hipLaunchKernelGGL(geo_rep, dim3(ranges), dim3(kThreads), 0, st, a);
    }
    if (a.merged) {
        const int parts = (a.Kmax + kWave - 1) / kWave;
        const unsigned waves = (unsigned)((int64_t)b.G * parts);      // (G <= 2^20, parts <= 4)
        hipLaunchKernelGGL(geo_merge, dim3((waves + kThreads / kWave - 1) / (kThreads / kWave)), dim3(kThreads), 0, st,
                           a, parts);
    }
    if (!a.merged) hipLaunchKernelGGL(geo_final, dim3(kblocks), dim3(kThreads), 0, st, a);
    return hipGetLastError();
}

}  // namespace kb
