// K-Means (Lloyd) clustering of searches whose rows fit the registers of one workgroup: searches of at most 512
// candidates (256 with more than 32 clusters) in batches of up to 256, one per compute unit; with fewer
// features two per unit, in batches of up to 512, and with fewer still in turns, in batches of up to 1024
// (cluster_resident says which).
//
// What a step of such a search costs in the kernel of kb_cluster_lloyd.h is not its scoring but
// what decides which candidates have to be scored and fetches them: the clocks of the drift
// bounds, the walk over limits and queue, a trip to memory for rows, one for the rows that move - 2.4
// us a step however short the search.  Here a wave keeps the rows of its T tiles of 32 candidates in
// registers from the first step to the last, as fp32 (for the sums) and as the matrix cores' bf16
// operands, and scores them in every step: matrix instructions, exact pass for the doubtful, moves
// between the fixed-point sums straight from the registers, a barrier, the renewal of the centroids, a
// barrier.  Same scores, same exact pass, same fixed-point grid and renewal, so the same bytes of
// assignments, sizes and centroids (the objective, a sum in fp64, takes another order).
//
// A step after one in which no candidate moved scores nothing: no centroid has moved, so nobody's
// nearest has changed (what the drift bounds say there, too).  A doubtful candidate's row goes through LDS
// to lanes over features: read again, it cost a trip to L2 each.
//
// A round of one search / of 200, 20 steps, rows fetched again / resident (us): 256 rows of 16 features, K = 8
// 62 / 33 and 103 / 56; 256 of 64, K = 4 86 / 56 and 189 / 111; 512 of 32, K = 16 88 / 53 and 157 / 99; 512 of 64,
// K = 32 85 / 54 and 188 / 87; one search of 274 rows of 53, K = 3, 30 steps 94 / 56, of 178 of 50, K = 2 63 / 36,
// of 382 of 16, K = 15 69 / 39.  Two tiles of rows against two of centroids are slower than the bounds (500 of
// 50, K = 40 92 / 95 and 122 / 131, without the two points above), hence 256 rows where a search may have more
// than 32 clusters.
//
// What the first step costs more - all rows move, most of them into the same sums - only later steps
// bring back: with two tiles of rows of more than 32 features and at most 4 clusters not fewer than ten do
// (one search of 512 rows of 64, K = 2, two steps 39.6 / 43.1 us, twenty 73 / 54; 256 of 200-512 rows of 48,
// K = 3 44.5 / 51.0 and 180 / 125).
//
// Two searches per compute unit, in 128 registers (which rows of up to 16 features, and one tile of up to 32
// against one of centroids, never exceed).  512 / 300 searches, 20 steps: 256 rows of 16, K = 16
// 97 / 58 and 93 / 55; of 32, K = 32 117 / 69 and 117 / 68; of 48, K = 16 108 / 67 and 94 / 59; 512 rows of 16
// 163 / 103 and 155 / 92 (around well-separated centres 115 / 75 and 111 / 67), of 32 199 / 140 and 188 / 123
// (121 / 97 and 104 / 81) although 27 registers spill there.  Not with 64 features, nor with 48 and more than 32
// clusters or 512 rows, whose registers spill and which lose (100 / 112, 118 / 134, 241 / 251, before the first
// point above).
// Up to 1024 searches, in turns, where a step is shortest: 256 rows of 16 103 / 87, of 32, K = 32 109 / 90, K <= 64 147 /
// 112; 512 rows of 16 193 / 160 (145 / 122), but of 32 142 / 152, hence 16 features there.  Beyond, batches of even
// lengths gain as much (2000 of 512 rows 1.15 to 1.4 times, 3000 of 256 1.2 to 1.4), but those in which most
// searches are far shorter than the longest lose: 1500 of 8-512 rows down to 0.88, 3000 of 4-256 to 0.86.
// 1024 and 1200 searches lost in none of 170 random shapes.
#include "kb_cluster_lloyd.h"

namespace kb {

namespace {

constexpr int kThreads = 512, kWaves = kThreads / kWave;
constexpr int kResidentTurnsG = 1024;     // searches that take turns on the compute units, two at a time
constexpr int kResidentFewK = 4, kResidentFewIters = 10;

struct ResidentLds {
    size_t flags, row, sums, cent, cn, cnt, dirty, aop, total;
};
__host__ __device__ constexpr ResidentLds resident_lds_layout(int Kmax, int D, int DP) {
    ResidentLds l{};
    size_t off = (size_t)kWaves * 16;                       // reduction scratch: two slots of one double per wave
    l.flags = off; off += 16;                               // whether any candidate moved in an even / odd step
    l.row = off; off += (size_t)kWaves * 16 * ((DP - 4) / 16) * 4;      // a wave's row for the exact pass
    l.sums = off; off += (size_t)Kmax * (D | 1) * 8;        // odd row stride: clusters spread over the LDS banks
    off = (off + 15) & ~(size_t)15;
    l.cent = off; off += (size_t)Kmax * DP * 4;
    l.cn = off;   off += (size_t)((Kmax + 31) & ~31) * 4;
    l.cnt = off;  off += (size_t)Kmax * 4;
    l.dirty = off; off += (size_t)Kmax;
    off = (off + 15) & ~(size_t)15;
    l.aop = off;  off += (size_t)((Kmax + 31) / 32) * ((DP - 4) / 16) * 2 * 64 * 16;
    l.total = off;
    return l;
}
// Everything that is moved in pieces of 16 bytes begins on such a piece, whatever the number of clusters.
constexpr bool resident_lds_aligned() {
    for (int Kmax = 1; Kmax <= 64; ++Kmax)
        for (int D = 1; D <= KB_MAX_D; ++D) {
            const ResidentLds l = resident_lds_layout(Kmax, D, 16 * ((D + 15) / 16) + 4);
            if ((l.row | l.cent | l.cn | l.aop) & 15 || (l.sums & 7)) return false;
        }
    return true;
}
static_assert(resident_lds_aligned(), "16-byte pieces of the LDS layout");

// Two waves per SIMD: 256 registers a lane, of which the rows take 16 * DS * T.  PAIR: two searches per
// compute unit, 128 registers.
template <int DS, int MT, int T, bool PAIR>
__global__ void __launch_bounds__(kThreads, PAIR ? 4 : 2) cluster_resident_kernel(ClusterArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int DP = 16 * DS + 4;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 31, h = lane >> 5;
    const int D = a.D, SP = D | 1;
    const int g = (int)blockIdx.x;
    int n0, ng, k0, K;
    search_bounds(a.seg_off, a.koff, g, a.N, a.Ksum, n0, ng, k0, K);
    if (K > a.Kmax) K = a.Kmax;                     // LDS is sized from the host copies
    if (K > 32 * MT) K = 32 * MT;
    if (ng > 32 * T * kWaves) ng = 32 * T * kWaves; // (the host launches this kernel only for such batches)
    if (ng <= 0 || K <= 0) {
        if (tid == 0) a.objective[g] = 0.f;
        return;
    }
    if (a.guard && ng < 2 * K) return;              // too few candidates to re-cluster: nothing is touched

    const ResidentLds L = resident_lds_layout(a.Kmax, D, DP);
    double* red = reinterpret_cast<double*>(smem);
    long long* sums = reinterpret_cast<long long*>(smem + L.sums);      // [Kmax][SP]
    float* cent = reinterpret_cast<float*>(smem + L.cent);              // [Kmax][DP]
    float* cn = reinterpret_cast<float*>(smem + L.cn);                  // [Kmax]
    int* cnt = reinterpret_cast<int*>(smem + L.cnt);                    // [Kmax]
    unsigned char* dirty = smem + L.dirty;                              // [Kmax]
    int* flags = reinterpret_cast<int*>(smem + L.flags);
    float* row = reinterpret_cast<float*>(smem + L.row) + 16 * DS * wid;
    bf16x8* aop = reinterpret_cast<bf16x8*>(smem + L.aop);
    const float* Xg = a.X + (size_t)n0 * D;
    const int mtiles = (K + 31) >> 5;
    const float kappa = mfma_kappa(DS);

    // Tile wid + kWaves * t: lane (m, h) holds the features 16 s + 8 h + i of row m, zeros beyond D (and in
    // rows that do not exist).
    float x[T][DS][8];
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int p = (wid + kWaves * t) * 32 + m;
        const float* xr = Xg + (size_t)(p < ng ? p : 0) * D;
        float4 v[DS][2];
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            const int d0 = 16 * s + 8 * h;
            v[s][0] = make_float4(0.f, 0.f, 0.f, 0.f);
            v[s][1] = v[s][0];
            if (p < ng) {
                if (D >= 4) {
                    v[s][0] = row_piece_load(xr, d0, D);
                    v[s][1] = row_piece_load(xr, d0 + 4, D);
                } else if (d0 == 0) {
                    v[s][0].x = xr[0];
                    if (D > 1) v[s][0].y = xr[1];
                    if (D > 2) v[s][0].z = xr[2];
                }
            }
        }
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            const int d0 = 16 * s + 8 * h;
            if (D >= 4) {
                v[s][0] = row_piece_shift(v[s][0], d0, D);
                v[s][1] = row_piece_shift(v[s][1], d0 + 4, D);
            }
            x[t][s][0] = v[s][0].x; x[t][s][1] = v[s][0].y; x[t][s][2] = v[s][0].z; x[t][s][3] = v[s][0].w;
            x[t][s][4] = v[s][1].x; x[t][s][5] = v[s][1].y; x[t][s][6] = v[s][1].z; x[t][s][7] = v[s][1].w;
        }
    }
    for (int idx = tid; idx < K * DP; idx += kThreads) {
        const int j = idx / DP, d = idx - j * DP;
        float v = 0.f;
        if (d < D)
            v = a.cent_init ? a.cent_init[(size_t)(k0 + j) * D + d]
                            : Xg[(size_t)(j < ng ? j : ng - 1) * D + d];
        cent[idx] = v;
    }
    for (int idx = tid; idx < K * SP; idx += kThreads) sums[idx] = 0;
    for (int j = tid; j < K; j += kThreads) { cnt[j] = 0; dirty[j] = 0; }
    for (int j = K + tid; j < ((a.Kmax + 31) & ~31); j += kThreads) cn[j] = kBig;
    if (tid < 2) flags[tid] = 0;

    bf16x8 Bh[T][DS], Bm[T][DS];
    float xn[T];
    float am = 0.f;
    double tsq = 0.0;         // sum of x^2, exact products
#pragma unroll
    for (int t = 0; t < T; ++t) {
        xn[t] = 0.f;
#pragma unroll
        for (int s = 0; s < DS; ++s) {
            split8(x[t][s], Bh[t][s], Bm[t][s]);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                xn[t] = fmaf(x[t][s][i], x[t][s][i], xn[t]);
                am = fmaxf(am, fabsf(x[t][s][i]));
                tsq = fma((double)x[t][s][i], (double)x[t][s][i], tsq);
            }
        }
        xn[t] += __shfl_xor(xn[t], 32);
    }
    int phase = 0;
    am = block_max_f<kWaves>(am, red, phase);
    tsq = block_sum_d<kWaves>(tsq, red, phase);
    const int sh = fixed_shift(am, ng);
    const int fsh = sh - 32;
    const double inv = ldexp(1.0, -sh);

    (void)renew_rows<DS, true, kThreads, renew_lanes(DS, MT, kThreads), false>(cent, cn, aop, sums, cnt, dirty, nullptr, K,
                                                                               D, SP, inv, true, true);
    __syncthreads();
    float cm = wave_max_f(lane < K ? cn[lane] : 0.f);       // largest |c_j|^2 (K <= 64: every wave for itself)

    int mine[T];
#pragma unroll
    for (int t = 0; t < T; ++t) mine[t] = -1;
    bool still = false;       // no candidate moved in the last step: no centroid did, so nobody's nearest has changed
    for (int it = 0; it < a.iters; ++it) {
        int moved = 0;
        if (!still) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int base = (wid + kWaves * t) * 32;
            if (base < ng) {                                 // (uniform)
                const bool valid = base + m < ng;
                float best, second;
                int bi;
                tile_scores<DS, MT>(Bh[t], Bm[t], cn, aop, mtiles, lane, best, second, bi);
                bi = bi < K ? bi : 0;
                const float E = kappa * (xn[t] + cm);
                // (a best score next to zero may have lost its position bits to a flush of
                // subnormal numbers: that candidate goes to the exact pass)
                const bool certain = (K == 1) || (((second - best) > 2.f * E) && fabsf(best) > 1.0e-30f);
                unsigned doubt = (unsigned)__ballot(valid && !certain && h == 0);
                while (doubt) {
                    const int b = __ffs((int)doubt) - 1;
                    doubt &= doubt - 1;
                    // (its row to lanes over features, zeros beyond D)
                    if (m == b) {
#pragma unroll
                        for (int s = 0; s < DS; ++s) {
                            float4* to = reinterpret_cast<float4*>(row + 16 * s + 8 * h);
                            to[0] = make_float4(x[t][s][0], x[t][s][1], x[t][s][2], x[t][s][3]);
                            to[1] = make_float4(x[t][s][4], x[t][s][5], x[t][s][6], x[t][s][7]);
                        }
                    }
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    const float xv = lane < 16 * DS ? row[lane] : 0.f;
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    float ub, lbd;
                    int bj = exact_nearest<DS>(xv, cent, K, D, DP, ub, lbd);
                    bj = bj < K ? bj : 0;
                    bi = m == b ? bj : bi;
                }
                const bool chg = valid && bi != mine[t];
                if (__any(chg)) {
                    moved = 1;
                    if (chg) {
                        // (formed again in every step: kept over the loop, the images take twice a row's registers)
                        int f = fsh;
                        asm volatile("" : "+v"(f));
                        const int old = mine[t];
                        long long* to = sums + bi * SP + 8 * h;
                        long long* from = sums + (old >= 0 ? old : 0) * SP + 8 * h;
#pragma unroll
                        for (int s = 0; s < DS; ++s) {
                            if (16 * s + 8 * h + 8 <= D) {
#pragma unroll
                                for (int i = 0; i < 8; ++i) {
                                    const long long q = to_fixed(x[t][s][i], f);
                                    lds_add(to + 16 * s + i, q);
                                    if (old >= 0) lds_add(from + 16 * s + i, -q);
                                }
                            } else {
#pragma unroll
                                for (int i = 0; i < 7; ++i) {
                                    if (16 * s + 8 * h + i < D) {
                                        const long long q = to_fixed(x[t][s][i], f);
                                        lds_add(to + 16 * s + i, q);
                                        if (old >= 0) lds_add(from + 16 * s + i, -q);
                                    }
                                }
                            }
                        }
                        if (h == 0) {
                            atomicAdd(&cnt[bi], 1);
                            dirty[bi] = 1;
                            if (old >= 0) { atomicSub(&cnt[old], 1); dirty[old] = 1; }
                        }
                        mine[t] = bi;
                    }
                }
            }
        }
        }
        int changed;
        if (a.early_exit) changed = block_or_i<kWaves>(moved, red, phase) & 1;
        else {
            if (moved && lane == 0) flags[it & 1] = 1;
            __syncthreads();
            changed = __builtin_amdgcn_readfirstlane(flags[it & 1]);
            if (tid == 0) flags[(it + 1) & 1] = 0;      // (read before the last barrier, set after the next)
        }
        still = !changed;

        const bool last = (it == a.iters - 1) || (a.early_exit && !changed);
        if (last) {
            // Objective relative to the centroids c_j that entered this step, as in the kernel for longer
            // searches: from the exact sums, member by member (four squares in fp32, their sums in fp64) where
            // the subtraction cancels.
            double part = 0.0;
            for (int j0 = 0; j0 < K; j0 += kThreads / 16) {
                const int j = j0 + (tid >> 4);
                if (j < K) {
                    const double nj = (double)cnt[j];
                    for (int d = tid & 15; d < D; d += 16) {
                        const double cj = (double)cent[(size_t)j * DP + d];
                        const double Sj = (double)sums[(size_t)j * SP + d] * inv;
                        part += cj * (2.0 * Sj - nj * cj);
                    }
                }
            }
            part = block_sum_d<kWaves>(part, red, phase);
            double J = tsq - part;
            if (!(J >= 1.0e-7 * tsq)) {
                double acc = 0.0;
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    if ((wid + kWaves * t) * 32 + m < ng) {
                        const float* cr = cent + (size_t)mine[t] * DP + 8 * h;
#pragma unroll
                        for (int s = 0; s < DS; ++s) {
#pragma unroll
                            for (int i = 0; i < 8; i += 4) {
                                const float e0 = x[t][s][i] - cr[16 * s + i], e1 = x[t][s][i + 1] - cr[16 * s + i + 1];
                                const float e2 = x[t][s][i + 2] - cr[16 * s + i + 2], e3 = x[t][s][i + 3] - cr[16 * s + i + 3];
                                acc += (double)fmaf(e0, e0, fmaf(e1, e1, fmaf(e2, e2, e3 * e3)));
                            }
                        }
                    }
                }
                J = block_sum_d<kWaves>(acc, red, phase);
            }
            if (tid == 0) a.objective[g] = (float)J;
        }
        (void)renew_rows<DS, true, kThreads, renew_lanes(DS, MT, kThreads), false>(cent, cn, aop, sums, cnt, dirty, nullptr,
                                                                                   K, D, SP, inv, false, !last);
        __syncthreads();
        if (last) break;
        cm = wave_max_f(lane < K ? cn[lane] : 0.f);
    }

#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int p = (wid + kWaves * t) * 32 + m;
        if (h == 0 && p < ng) a.assign[(size_t)n0 + p] = mine[t];
    }
    for (int idx = tid; idx < K * D; idx += kThreads) {
        const int j = idx / D, d = idx - j * D;
        a.cent_out[(size_t)(k0 + j) * D + d] = cent[(size_t)j * DP + d];
    }
    for (int j = tid; j < K; j += kThreads) a.counts[k0 + j] = cnt[j];
}

// (PAIR where the rows leave 128 registers unfilled anyway: one kernel for both kinds of batches)
template <int DS, int MT, int T, bool PAIR = false>
hipError_t launch(const ClusterArgs& a, hipStream_t st) {
    constexpr bool kPair = PAIR || DS == 1 || (DS == 2 && MT == 1 && T == 1);
    const size_t lds = resident_lds_layout(a.Kmax, a.D, 16 * DS + 4).total;
    return launch_one(cluster_resident_kernel<DS, MT, T, kPair>, kThreads, a, lds, st);
}

}  // namespace

bool cluster_resident(const kb_batch& b, int scorer, int iters) {
    if (scorer != KB_SCORER_DEFAULT || iters <= 1 || b.Kmax < 1 || b.Kmax > 64) return false;
    const bool two = b.Nmax > 32 * kWaves;                  // tiles of a wave
    if (b.Nmax > 64 * kWaves || (two && b.Kmax > 32)) return false;
    if (two && b.D > 32 && b.Kmax <= kResidentFewK && iters < kResidentFewIters) return false;
    if (b.G <= kResidentMaxG) return true;
    if (b.G <= kResidentPairG) return b.D <= (!two && b.Kmax <= 32 ? 48 : 32);
    return b.G <= kResidentTurnsG && b.D <= (two ? 16 : 32);
}

hipError_t launch_cluster_resident(const ClusterArgs& a, int Nmax, hipStream_t st) {
    const int ds = (a.D + 15) / 16, mt = a.Kmax <= 32 ? 1 : 2, t = Nmax <= 32 * kWaves ? 1 : 2;
    const auto go = [&](auto d) {
        constexpr int DS = decltype(d)::value;
        if (a.G > kResidentMaxG) {
            if constexpr (DS <= 3) {
                if (t == 1 && mt == 1) return launch<DS, 1, 1, true>(a, st);
            }
            if constexpr (DS <= 2) {        // (two tiles of rows: one of centroids, cluster_resident)
                return t == 1 ? launch<DS, 2, 1, true>(a, st) : launch<DS, 1, 2, true>(a, st);
            }
            return hipErrorInvalidValue;
        }
        if (mt == 2) return t == 1 ? launch<DS, 2, 1>(a, st) : hipErrorInvalidValue;
        return t == 1 ? launch<DS, 1, 1>(a, st) : launch<DS, 1, 2>(a, st);
    };
    switch (ds) {
        case 1: return go(std::integral_constant<int, 1>{});
        case 2: return go(std::integral_constant<int, 2>{});
        case 3: return go(std::integral_constant<int, 3>{});
        default: return go(std::integral_constant<int, 4>{});
    }
}

}  // namespace kb
