"""Measured cases of the arm-scoring library: what a search service has it do, through the
C ABI as the binding exposes it, on seeded synthetic traces of the shapes that
`paper_2511_18868_amd.synth` describes (drawn here on the GPU, so that making them is quick).

A case is one call (or the short sequence of calls a caller always makes together):

  round      kb_round; with draw also kb_sample, which picks k_t for the next generation
  iterate    kb_iterate: `rounds` iterations of Alg. 1 with a re-clustering every `tau`-th
  step       kb_cluster_step from given centroids: the unit of the Lloyd step
  recluster  seeding, kb_cluster from those seeds, kb_cluster_geometry: a clustering renewed
             as the paper's scikit-learn default does it
  diagnose   kb_cluster_geometry and kb_cluster_diameter of a finished clustering: the
             covering terms of Theorem 1

A batch holds G searches of nmin .. nmax candidates (log-uniform), K_g = min(kcap, N_g // kdiv)
clusters each, D features, S strategies, `iters` Lloyd steps.
"""
import math

import numpy as np
import torch

from paper_2511_18868_amd import binding as kb

PEAK_FLOPS, PEAK_BW = 2.5e15, 8.0e12
ROOT2 = float(np.float32(math.sqrt(2.0)))
RESOURCES = 3          # DRAM, L2 and compute shares of a hardware signature
THETA = 0.75           # the paper's saturation threshold


def _case(entry, G, nmin, nmax, D, S, kcap, kdiv, iters, **more):
    c = dict(entry=entry, G=G, nmin=nmin, nmax=nmax, D=D, S=S, kcap=kcap, kdiv=kdiv, iters=iters,
             features="gauss")
    c.update(more)
    return c


def listed():
    varlen = dict(nmin=64, nmax=4096, D=48, S=32, kcap=64, kdiv=16, iters=20, features="mixture")
    return [
        # one search per benchmark kernel at the sizes the paper runs (a frontier of a few
        # dozen kernels, 3 clusters, 6 strategies): a round and the draw of the next kernel
        _case("round", 183, 12, 41, 5, 6, 3, 4, 10, name="paper_round", draw=True, features="mixture"),
        # the same searches through twenty whole iterations, re-clustered every tenth
        _case("iterate", 183, 12, 41, 5, 6, 3, 4, 10, name="paper_iterate", rounds=20, tau=10,
              features="mixture"),
        # one small search, log-normal counters (benchmark configuration 1)
        _case("round", 1, 256, 256, 16, 8, 8, 1, 20, name="one_256", features="lognormal"),
        # one search of a few thousand candidates (benchmark configuration 2)
        _case("round", 1, 4096, 4096, 32, 16, 32, 1, 30, name="one_4096"),
        # a thousand equal searches in one call (benchmark configuration 3)
        _case("round", 1024, 512, 512, 32, 16, 16, 1, 25, name="batch_512"),
        # ragged batch with a feature count that fills no 16-byte row, the paper's six
        # strategies, and the draw
        _case("round", 300, 70, 1900, 50, 6, 24, 16, 20, name="batch_odd", draw=True,
              features="mixture"),
        # the full round of four thousand searches of very different length (configuration 5)
        _case("round", 4096, name="batch_varlen", **varlen),
        # one very large search with outliers, 256 clusters (configuration 4)
        _case("round", 1, 1 << 20, 1 << 20, 64, 4, 256, 1, 10, name="one_1m", features="outliers"),
        # ten iterations of a batch of such searches, re-clustered every fifth
        _case("iterate", 512, name="iterate_varlen", rounds=10, tau=5, **varlen),
        # a clustering renewed from randomised seeds until it stands still
        _case("recluster", 1024, name="recluster", seeding="dsquared", stop_early=True, **varlen),
        # one Lloyd step of the large batch from its present centroids
        _case("step", 4096, name="lloyd_step", **varlen),
        # representatives, radii and diameters of a finished clustering
        _case("diagnose", 1024, name="diagnose", **varlen),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["short", "short", "single", "single", "batch", "batch", "batch", "large"])
    if kind == "short":       # a service over the paper's own sizes
        entry = rng.choice(["round", "iterate"])
        nmin = rng.randint(8, 16)
        more = dict(rounds=rng.randint(4, 24), tau=rng.randint(3, 12)) if entry == "iterate" \
            else dict(draw=rng.random() < 0.5)
        return _case(entry, _log(rng, 1, 4000), nmin, rng.randint(nmin + 4, 60), rng.randint(3, 12),
                     rng.randint(3, 10), rng.randint(2, 6), 4, rng.randint(5, 20),
                     features="mixture", **more)
    if kind == "single":      # one search, latency
        n = _log(rng, 100, 20000)
        return _case("round", 1, n, n, rng.randint(5, 64), rng.randint(3, 32),
                     min(64, max(2, n // rng.randint(16, 130))), 1, rng.randint(10, 30),
                     draw=rng.random() < 0.3)
    if kind == "large":       # one large search with many clusters
        n = _log(rng, 100000, 1000000)
        return _case("round", 1, n, n, rng.randint(16, 64), rng.randint(2, 8), rng.randint(65, 256), 1,
                     rng.randint(4, 10), features="outliers")
    entry = rng.choice(["round", "round", "round", "iterate", "recluster", "step", "diagnose"])
    nmin = _log(rng, 40, 400)
    nmax = _log(rng, nmin + 10, 4096)
    most = 4_000_000 if entry in ("round", "step") else 600_000
    G = _log(rng, 24, max(30, min(6000, most // nmax)))
    more = {}
    if entry == "round":
        more = dict(draw=rng.random() < 0.3, stop_early=rng.random() < 0.3)
    elif entry == "iterate":
        more = dict(rounds=rng.randint(4, 12), tau=rng.randint(3, 12))
    elif entry == "recluster":
        more = dict(seeding=rng.choice(["dsquared", "farthest"]), stop_early=True)
    return _case(entry, G, nmin, nmax, rng.randint(5, 64), rng.randint(3, 32), rng.randint(4, 64), 16,
                 rng.randint(10, 25), features="mixture", **more)


def _sizes(case):
    """N_g and K_g of every search: part of the case, the same for every seed."""
    rng = np.random.default_rng([case[k] for k in ("G", "nmin", "nmax", "kcap")])
    n = np.rint(np.exp(rng.uniform(math.log(case["nmin"]), math.log(case["nmax"]), case["G"])))
    n = np.clip(n, case["nmin"], case["nmax"]).astype(np.int64)
    return n, np.maximum(1, np.minimum(case["kcap"], n // case["kdiv"]))


def _segment_mean(x, n, equal):
    """Mean over every search's rows, the same bits in every run."""
    if equal:
        return x.view(len(n), -1, x.shape[1]).mean(1)
    return torch.segment_reduce(x, "mean", lengths=torch.from_numpy(n).to(x.device), axis=0)


def _features(case, rng, gen, n, k, sid):
    """Rows around seeded centres, z-scored per feature and search (the normalised phi)."""
    dev, D, kind = sid.device, case["D"], case["features"]
    N, ksum = int(n.sum()), int(k.sum())
    koff = np.concatenate([[0], np.cumsum(k)])
    u = torch.rand(N, generator=gen, device=dev, dtype=torch.float64)
    if kind == "mixture":     # Dirichlet(1) weights, a width per centre
        w = rng.exponential(size=ksum)
        cs = np.concatenate([[0.0], np.cumsum(w)])
        tot = np.diff(cs[koff])
        inside = (cs[1:] - np.repeat(cs[koff[:-1]], k)) / np.repeat(tot, k)
        inside[koff[1:] - 1] = 1.0
        flat = torch.from_numpy(np.repeat(np.arange(len(k)), k) + inside).to(dev)
        lab = torch.searchsorted(flat, sid + u, right=True)
        lab = torch.minimum(lab, torch.from_numpy(koff[1:] - 1).to(dev)[sid])
        sigma = torch.from_numpy(rng.uniform(0.5, 1.5, ksum).astype(np.float32)).to(dev)
    else:
        lab = torch.from_numpy(koff[:-1]).to(dev)[sid] + (u * torch.from_numpy(k).to(dev)[sid]).long()
        sigma = None
    spread = 1.0 if kind == "lognormal" else 3.0
    centres = spread * torch.randn(ksum, D, generator=gen, device=dev)
    x = torch.randn(N, D, generator=gen, device=dev)
    if sigma is not None:
        x *= sigma[lab][:, None]
    x += centres[lab]
    if kind == "lognormal":
        x = x.exp()
    elif kind == "outliers":  # one row in ten anywhere in the box
        lo, hi = x.min(0).values, x.max(0).values
        out = torch.rand(N, generator=gen, device=dev) < 0.1
        x = torch.where(out[:, None], lo + (hi - lo) * torch.rand(N, D, generator=gen, device=dev), x)
    equal = bool((n == n[0]).all())
    x -= _segment_mean(x, n, equal)[sid]
    sd = _segment_mean(x * x, n, equal).sqrt()
    x /= torch.where(sd > 0, sd, torch.ones_like(sd))[sid]
    return x.contiguous()


class _State:
    pass


def prepare(case, seed):
    dev = torch.device("cuda:0")
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    n, k = _sizes(case)
    G, D, S, N, ksum = case["G"], case["D"], case["S"], int(n.sum()), int(k.sum())
    s = _State()
    s.case = case
    off = np.concatenate([[0], np.cumsum(n)])
    s.seg_off = torch.from_numpy(off.astype(np.int32)).to(dev)
    s.koff = torch.from_numpy(np.concatenate([[0], np.cumsum(k)]).astype(np.int32)).to(dev)
    sid = torch.repeat_interleave(torch.arange(G, device=dev), torch.from_numpy(n).to(dev), output_size=N)
    s.X = _features(case, rng, gen, n, k, sid)

    new = lambda shape, dt: torch.zeros(shape, dtype=dt, device=dev)  # noqa: E731
    s.assign, s.counts = new(N, torch.int32), new(ksum, torch.int32)
    s.cent, s.objective = new((ksum, D), torch.float32), new(G, torch.float32)
    s.batch = kb.make_batch(G, D, S, N, int(k.max()), ksum, int(n.max()), s.seg_off, s.koff)
    prior = case["entry"] == "iterate"           # Alg. 1 starts its statistics at N = 1, mu = 0.5
    s.params = kb.make_params(PEAK_FLOPS, PEAK_BW, 2.0 if prior else ROOT2, 1.0 if prior else 0.0, 0.5,
                              case["iters"], kb.KB_SCORER_DEFAULT, int(case.get("stop_early", False)))
    s.ws_bytes = kb.kb_workspace_bytes(s.batch, s.params)
    s.ws = torch.empty(max(s.ws_bytes, 256), dtype=torch.uint8, device=dev)

    if case["entry"] in ("round", "iterate"):
        s.visits = torch.poisson(torch.full((N, S), 5.0, device=dev), generator=gen) + 1.0
        p = torch.rand(N, S, generator=gen, device=dev)
        s.rsum = torch.binomial(s.visits, p, generator=gen)
        s.visits = s.visits.int()
        rows = torch.zeros(N + 1, dtype=torch.int64, device=dev)
        rows[1:] = s.visits.sum(1, dtype=torch.int64).cumsum(0)
        s.t = (rows[s.seg_off[1:].long()] - rows[s.seg_off[:-1].long()]).clamp_min(1)
        s.Ncs, s.mu, s.ucb = new((ksum, S), torch.int32), new((ksum, S), torch.float32), new((ksum, S), torch.float32)
    if case["entry"] == "round":
        s.flops = 10.0 ** (6.0 + 6.0 * torch.rand(N, generator=gen, device=dev))
        s.bytes = 10.0 ** (6.0 + 6.0 * torch.rand(N, generator=gen, device=dev))
        # incumbent: the lower median of the search's own roofline runtimes
        runtime = torch.maximum(s.flops / PEAK_FLOPS, s.bytes / PEAK_BW)
        key = (sid << 32 | runtime.view(torch.int32).long()).sort().values
        mid = torch.from_numpy(off[:-1] + (n - 1) // 2).to(dev)
        s.incumbent = (key[mid] & 0xFFFFFFFF).int().view(torch.float32).contiguous()
        s.bound, s.alive, s.sel = new(N, torch.float32), new(N, torch.uint8), new((G, 3), torch.int32)
        s.io = kb.kb_round_io(*[x.data_ptr() for x in (
            s.X, s.flops, s.bytes, s.incumbent, s.visits, s.rsum, s.t, s.bound, s.alive, s.assign, s.cent,
            s.counts, s.objective, s.Ncs, s.mu, s.ucb, s.sel)])
        if case.get("draw"):
            s.ksel, s.sp = new(G, torch.int32), kb.kb_sample_params(seed, 1, 1.0)
    elif case["entry"] == "iterate":
        T = case["rounds"]
        s.h = torch.from_numpy(rng.beta(2.0, 2.0, size=(N, RESOURCES)).astype(np.float32)).to(dev)
        s.target = torch.arange(S, dtype=torch.int32, device=dev) % RESOURCES
        s.ok = (torch.rand(T, G, generator=gen, device=dev) < 0.8).to(torch.uint8)
        s.reward = torch.rand(T, G, generator=gen, device=dev) * s.ok
        s.rep, s.nvalid, s.M = new(ksum, torch.int32), new(G, torch.int32), new((ksum, S), torch.uint8)
        s.radius = new(ksum, torch.float32)
        s.sel_log, s.ksel_log = new((T, G, 3), torch.int32), new((T, G), torch.int32)
        s.ip = kb.kb_iterate_params(T, case["tau"], 0, 0, RESOURCES, THETA, kb.kb_sample_params(seed, 1, 1.0))
        s.io = kb.kb_iterate_io(*[x.data_ptr() if x is not None else None for x in (
            s.X, s.h, s.target, None, s.reward, s.ok, s.visits, s.rsum, s.t, s.assign, s.cent, s.counts,
            s.objective, s.rep, s.radius, s.M, s.nvalid, s.Ncs, s.mu, s.ucb, s.sel_log, s.ksel_log)])
    elif case["entry"] == "step":
        # present centroids: what two steps from the first rows give
        s.cent_in = new((ksum, D), torch.float32)
        two = kb.make_params(PEAK_FLOPS, PEAK_BW, ROOT2, 0.0, 0.5, 2)
        kb.kb_cluster(s.batch, two, s.X, None, s.assign, s.cent_in, s.counts, s.objective, s.ws, s.ws_bytes)
    elif case["entry"] == "recluster":
        s.seeds, s.pick = new((ksum, D), torch.float32), new(ksum, torch.int32)
        s.rep, s.radius, s.seed = new(ksum, torch.int32), new(ksum, torch.float32), seed
    elif case["entry"] == "diagnose":
        kb.kb_cluster(s.batch, s.params, s.X, None, s.assign, s.cent, s.counts, s.objective, s.ws, s.ws_bytes)
        s.rep, s.radius, s.diam = new(ksum, torch.int32), new(ksum, torch.float32), new(ksum, torch.float32)
    return s


def run(s):
    case, ws = s.case, (s.ws, s.ws_bytes)
    if case["entry"] == "round":
        kb.kb_round(s.batch, s.params, s.io, *ws)
        out = dict(bound=s.bound, alive=s.alive, assign=s.assign, cent=s.cent, counts=s.counts,
                   objective=s.objective, Ncs=s.Ncs, mu=s.mu, ucb=s.ucb, sel=s.sel)
        if case.get("draw"):
            kb.kb_sample(s.batch, s.sp, s.assign, s.alive, s.bound, s.incumbent, s.sel, s.ksel, *ws)
            out["ksel"] = s.ksel
        return out
    if case["entry"] == "iterate":
        kb.kb_iterate(s.batch, s.params, s.ip, s.io, *ws)
        return dict(sel_log=s.sel_log, ksel_log=s.ksel_log, visits=s.visits, rsum=s.rsum, t=s.t,
                    assign=s.assign, cent=s.cent, counts=s.counts, objective=s.objective, rep=s.rep,
                    radius=s.radius, M=s.M, nvalid=s.nvalid, Ncs=s.Ncs, mu=s.mu, ucb=s.ucb)
    if case["entry"] == "step":
        kb.kb_cluster_step(s.batch, s.X, s.cent_in, s.assign, s.cent, s.counts, s.objective, *ws)
        return dict(assign=s.assign, cent=s.cent, counts=s.counts, objective=s.objective)
    if case["entry"] == "recluster":
        if case["seeding"] == "dsquared":
            kb.kb_seed_dsquared(s.batch, s.X, s.seed, 0, s.seeds, s.pick, *ws)
        else:
            kb.kb_seed_farthest(s.batch, s.X, s.seeds, s.pick, *ws)
        kb.kb_cluster(s.batch, s.params, s.X, s.seeds, s.assign, s.cent, s.counts, s.objective, *ws)
        kb.kb_cluster_geometry(s.batch, s.X, s.cent, s.assign, s.rep, s.radius, *ws)
        return dict(seeds=s.seeds, pick=s.pick, assign=s.assign, cent=s.cent, counts=s.counts,
                    objective=s.objective, rep=s.rep, radius=s.radius)
    kb.kb_cluster_geometry(s.batch, s.X, s.cent, s.assign, s.rep, s.radius, *ws)
    kb.kb_cluster_diameter(s.batch, s.X, s.assign, s.diam, *ws)
    return dict(rep=s.rep, radius=s.radius, diam=s.diam)


def _counts(case):
    """Candidates, clusters, (candidate, cluster) pairs, pairs of members of equal clusters."""
    n, k = _sizes(case)
    return float(n.sum()), float(k.sum()), float((n * k).sum()), float((n * n / k).sum()) / 2


def work(case):
    """Every input read once and every output written once; one full assignment of the rows to
    the centroids (what no clustering can do without - how often a candidate has to be scored
    again depends on the data), for the diameters every pair of members of equal clusters."""
    N, K, NK, pairs = _counts(case)
    D, S, G, entry = case["D"], case["S"], case["G"], case["entry"]
    clustering = 4 * N * D + 4 * N + K * (4 * D + 4) + 4 * G      # rows in; assignment and centroids out
    if entry == "round":
        return {"bytes": clustering + 13 * N + 8 * N * S + 12 * K * S + 28 * G, "flops": 2 * NK * D}
    if entry == "iterate":
        # rewards, draws and statistics of every round beside one aggregation of the history
        return {"bytes": clustering + 8 * N * S + 4 * N * RESOURCES + 13 * K * S + 25 * G * case["rounds"],
                "flops": 2 * NK * D}
    if entry == "step":
        return {"bytes": clustering + 4 * K * D, "flops": 2 * NK * D}
    if entry == "recluster":
        # seeds: every row against every chosen row; then an assignment
        return {"bytes": clustering + K * (4 * D + 12), "flops": 4 * NK * D}
    return {"bytes": 4 * N * D + 4 * N + K * (4 * D + 12), "flops": 2 * N * D + 3 * pairs * D}


def tolerance(case):
    """Masks, assignments, counts, visit sums and choices are whole numbers, equal on every
    input; the scores, means and objectives come from 64-bit sums rounded once to 32 bits
    (against the same path in fp64: rel 2.7e-8, max 6.0e-8).  Diameters are fp32 sums over the
    features, within (D + 2) 2^-24 of a distance."""
    if case["entry"] == "diagnose":
        return {"rel": 4e-6, "max": 4e-6}
    return {"rel": 1.2e-7, "max": 2.4e-7}
