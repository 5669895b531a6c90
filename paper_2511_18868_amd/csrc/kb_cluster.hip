// K-Means (Lloyd) clustering of searches that one workgroup holds: which form of the kernel
// (kb_cluster_lloyd.h) a batch takes, and its launch.
#include "kb_cluster_lloyd.h"

namespace kb {

extern template hipError_t launch_lloyd<1>(const ClusterArgs&, const LloydForm&, hipStream_t);
extern template hipError_t launch_lloyd<2>(const ClusterArgs&, const LloydForm&, hipStream_t);
extern template hipError_t launch_lloyd<3>(const ClusterArgs&, const LloydForm&, hipStream_t);
extern template hipError_t launch_lloyd<4>(const ClusterArgs&, const LloydForm&, hipStream_t);

constexpr size_t kMaxLds = 160 * 1024;
constexpr int kWideMaxG = 256;     // most searches of a batch that takes the wide shape whatever it holds

// sizes the one-workgroup kernel is laid out for: the largest search it will take
static int one_wg_kmax(const kb_batch& b) { return b.Kmax > kOneWgMaxK ? kOneWgMaxK : (b.Kmax > 0 ? b.Kmax : 1); }
static int one_wg_nmax(const kb_batch& b) { return b.Nmax > one_wg_limit_n(b) ? one_wg_limit_n(b) : b.Nmax; }

bool cluster_supported(const kb_batch& b) {
    const int ds = (b.D + 15) / 16;
    return lds_layout(one_wg_kmax(b), b.D, 16 * ds + 4, one_wg_nmax(b), kThreadsNarrow / kWave, false).total <= kMaxLds;
}

static ClusterArgs cluster_args(const kb_batch& b, const ClusterCall& c) {
    ClusterArgs a;
    a.G = b.G; a.D = b.D; a.Ksum = b.Ksum; a.Kmax = one_wg_kmax(b); a.N = b.N;
    a.seg_off = b.seg_off; a.koff = b.koff; a.X = c.X; a.cent_init = c.cent_init;
    a.iters = c.iters; a.early_exit = c.stop_early ? 1 : 0; a.assign = c.assign; a.cent_out = c.cent_out;
    a.counts = c.counts; a.objective = c.objective; a.a_new = c.a_new;
    a.order = c.order;
    a.use_bounds = c.scorer != 2;
    a.guard = c.guard;
    a.mixed = c.mixed;
    a.limit_n = one_wg_limit_n(b);
    a.lim = reinterpret_cast<float2*>(c.lim);
    a.Nmax = one_wg_nmax(b);
    return a;
}

// Which shape a batch takes.  A search runs 1.7 times as fast with 768 threads and a
// compute unit to itself, but the chip then gets through 30-40 % fewer rows per second
// than with three or four 256-thread searches per unit, and through fewer searches: each
// costs a unit its steps' barriers whatever its length.  So the wide shape pays while
// the launch lasts as long as its longest search, i.e. while all searches together hold
// only so many times the rows of the longest one (N / Nmax), and are not many beside it
// (G / Nmax).  Both shapes measured, 20 steps, narrow / wide (us); rows around centres of
// different width and weight, in brackets around well-separated ones:
//   lengths 64-4096, D = 48, K <= 64:   N/Nmax  67: 757 / 421   232: 1001 / 611   346: 1065 / 907
//                                       592: 1244 / 1512
//   lengths 70-1900, D = 50, K <= 24:   141: 504 / 305   240: 712 / 440 (290 / 306)   278: 545 / 483
//                                       (296 / 355)   357: 555 / 588
//   lengths 70-1900, D = 48, K <= 64:   239: 439 / 378 (291 / 296)   294: 396 / 435 (245 / 336)
//   lengths 100-500, D = 48, K <= 64:   154: 139 / 136   291: 174 / 226
//   one of 4096 and G of 70, D = 48:    1200: 661 / 362 (483 / 298)  1638: 613 / 401 (420 / 350)
//                                       2048: 945 / 528 (391 / 434)  8000: (573 / 1515)
//   one of 4096 and G of 300:           1200: 829 / 486 (377 / 360)  2048: 649 / 680 (416 / 573)
//   one of 2000 and G of 100, D = 32:   800: 279 / 229 (183 / 183)   1000: 235 / 244 (168 / 215)
//   one of 600 and G of 100, D = 48:    300: 133 / 135   600: 113 / 190   1000: 143 / 262
// Short searches gain less from more threads (a step is barriers and reductions), hence
// the lower line for them, and so does a single step, whose narrow form holds more searches per
// unit (64-4096, N/Nmax 148: 112 / 79, 182: 114 / 93, 227: 117 / 110, 340: 142 / 179).  Rows of no
// whole 16-byte pieces cost the narrow shape more, hence their higher line in G.  Batches of long searches
// only (2048 rows or more on average) are 13-20 % faster in the wide shape however many they are -
// but for a single step, where they have the line of the long ones only (3000-8000, N/Nmax 368: 289 /
// 258; 2048-2500, 543: 122 / 138, 2700: 434 / 547).
// In a batch that holds searches of the multi-workgroup path as well, the longest is one of
// those and the others' longest is not known: four times their average is taken, the ratio
// of lengths that are spread evenly over their logarithm (4000 searches of 64-4096 rows
// beside one of 100000, by the longest of all: 3666 / 3776).
constexpr int kWideLoad = 400, kWideLoadStep = 250, kWideLoadShort = 200, kWideShortN = 1024;
static bool wide_shape(const kb_batch& b, bool one, bool mixed) {
    if (b.G <= kWideMaxG) return true;
    int64_t N = b.N, longest = b.Nmax;
    if (mixed) {
        N -= b.Nmax;
        longest = 4 * N / b.G;
        if (longest > one_wg_limit_n(b)) longest = one_wg_limit_n(b);
    }
    const bool all_long = N >= (int64_t)2048 * b.G;
    const int load = longest < kWideShortN ? kWideLoadShort : (one && !all_long ? kWideLoadStep : kWideLoad);
    const int many = (b.D & 3) == 0 ? 9 : 11;
    return (N <= load * longest && 20 * (int64_t)b.G <= many * longest) || (all_long && !one);
}

// Workgroups of a kernel that a compute unit holds by their LDS, which is handed out in pieces of 1280 bytes.
static int resident(size_t lds) { return (int)(kMaxLds / ((lds + 1279) / 1280 * 1280)); }

hipError_t launch_cluster(const kb_batch& b, const ClusterCall& c, hipStream_t st) {
    const ClusterArgs a = cluster_args(b, c);
    const int ds = (b.D + 15) / 16;   // 1..4 K-steps of 16 features
    // a batch of very short searches, in the library's default mode: one wave per search
    if (!c.mixed && cluster_wave_per_search(b, c.scorer)) return launch_cluster_wave(b, c, st);
    if (!c.mixed && cluster_resident(b, c.scorer, c.iters)) return launch_cluster_resident(a, b.Nmax, st);
    const auto lds = [&](bool wide, bool state) {
        return lds_layout(a.Kmax, b.D, 16 * ds + 4, a.Nmax, (wide ? kThreadsWide : kThreadsNarrow) / kWave, state).total;
    };
    LloydForm f;
    f.mt = a.Kmax <= 32 ? 1 : (a.Kmax <= 64 ? 2 : 0);
    if (c.scorer == 1) f.mt = 0;
    f.rows = (b.D & 3) == 0 ? kRowsWhole : b.D >= 4 ? kRowsRagged : kRowsTiny;
    const bool one = f.mt > 0 && c.iters == 1;
    f.wide = wide_shape(b, one, c.mixed != 0) && lds(true, false) <= kMaxLds;
    // The candidates' states stay in LDS where that costs no resident workgroup: a step of a short
    // search then has a trip to L2 less (a round of one search of 4096 rows 243 -> 235 us, of 1024 of 512
    // 171 -> 170, ten iterations of 512 searches of 64-4096 1283 -> 1270).
    const int most = f.wide ? 1 : narrow_workgroups_per_cu(ds, f.mt);
    const auto fits = [&](bool state) { const int n = resident(lds(f.wide, state)); return n < most ? n : most; };
    f.state = f.mt > 0 && c.iters > 1 && lds(f.wide, true) <= kMaxLds && fits(true) >= fits(false);
    f.one = one && !f.wide;
    f.lds = f.one ? lds_layout(a.Kmax, b.D, 16 * ds + 4, a.Nmax, kThreadsNarrow / kWave, false, true).total
                  : lds(f.wide, f.state);
    if (f.lds > kMaxLds) return hipErrorInvalidValue;
    switch (ds) {
        case 1: return launch_lloyd<1>(a, f, st);
        case 2: return launch_lloyd<2>(a, f, st);
        case 3: return launch_lloyd<3>(a, f, st);
        default: return launch_lloyd<4>(a, f, st);
    }
}

}  // namespace kb
