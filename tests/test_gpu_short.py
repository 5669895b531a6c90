"""The kernels for batches of very short searches (at most 64 candidates and 16 clusters, a wave
per search) at the edges of their forms: row lengths on both sides of the compiled numbers of
16-byte pieces, one to sixteen clusters (a coordinate per lane in one pass and in several), searches
of one and of 64 candidates, against the workgroup kernels, which share no step with them."""
import numpy as np
import pytest

from paper_2511_18868_amd import synth
from kbcheck import assert_rel_close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_18868_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("D", [1, 3, 4, 5, 8, 9, 12, 13, 16, 17, 32, 33, 48, 49, 64])
@pytest.mark.parametrize("kcap,kdiv", [(1, 1), (5, 2), (16, 1)])
def test_clustering_by_a_wave_equals_the_workgroup_kernel(kb, D, kcap, kdiv):
    import torch
    b = synth.config5(G=61, nmin=1, nmax=64, D=D, S=3, iters=6, kcap=kcap, kdiv=kdiv, seed=500 + D)
    if D % 2:          # rows on a grid: equal distances, which the fp64 distances and the lowest index decide
        b.X[:] = np.rint(2.0 * b.X) / 2.0
    out = []
    for mode, init in ((0, False), (2, False), (0, True), (2, True)):
        d = kb.DeviceBatch(b, scorer=mode)
        start = None
        if init:       # caller-supplied centroids: every row of the search's own, from the back
            rows = np.concatenate([np.arange(e - 1, e - 1 - k, -1) for e, k in
                                   zip(b.seg_off[1:], np.diff(b.koff))]).astype(np.int64)
            start = torch.from_numpy(b.X[rows].copy()).to(d.device)
        kb.kb_cluster(d.batch, d.params, d.X, start, d.assign, d.cent, d.counts, d.objective, d.ws, d.ws_bytes)
        torch.cuda.synchronize()
        out.append({k: d.host(k).copy() for k in ("assign", "cent", "counts", "objective")})
    for one, other in ((out[0], out[1]), (out[2], out[3])):
        for k in ("assign", "cent", "counts"):
            np.testing.assert_array_equal(one[k].view(np.uint8), other[k].view(np.uint8), err_msg=k)
        assert_rel_close(one["objective"], other["objective"], what="objective")
    assert not np.array_equal(out[0]["cent"], out[2]["cent"]) or kcap == 1


SHAPES = {
    # G, nmin, nmax, D, S, kcap, kdiv, rounds: four waves a search, then one; one arm per lane, then four
    "paper": (61, 12, 41, 5, 6, 3, 4, 70),
    "many": (800, 1, 64, 5, 6, 3, 4, 19),
    "edge": (37, 1, 64, 33, 16, 16, 1, 19),
    "manyedge": (770, 1, 30, 13, 16, 16, 1, 9),
    "onearm": (5, 1, 64, 64, 1, 1, 1, 19),
    "morethanalaunch": (3, 20, 41, 8, 6, 4, 4, 1030),
}


@pytest.mark.parametrize("variant", ["cold", "warm", "masked", "notanumber"])
@pytest.mark.parametrize("shape", list(SHAPES))
def test_iterations_in_one_launch_equal_the_launches_one_by_one(kb, shape, variant):
    """A signature of at most eight resources lets a batch run its iterations in one launch; with a
    ninth, which no strategy works on, the same call goes through the launches of the stages.  Every
    output byte for byte, searches too short to be clustered again (N_g < 2 K_g) among them."""
    import torch
    G, nmin, nmax, D, S, kcap, kdiv, T = SHAPES[shape]
    b = synth.config5(G=G, nmin=nmin, nmax=nmax, D=D, S=S, kcap=kcap, kdiv=kdiv, iters=4, seed=600 + G)
    R = 8 if shape == "edge" else 3
    h, target, theta = synth.signatures(b, R)
    fb = [synth.feedback(b, seed=r) for r in range(T)]
    rw, ok = np.stack([f[0] for f in fb]), np.stack([f[1] for f in fb])
    alive = (np.arange(b.N) % 3 != 1).astype(np.uint8) if variant == "masked" else None
    if variant == "notanumber":       # inf * sqrt(ln 1 / n), beside untried arms
        b.t[:] = 1
        b.visits[:, ::2] = 0
        b.rsum[:, ::2] = 0.0
    got = []
    for cols in (R, 9):
        d = kb.DeviceBatch(b)
        if variant == "notanumber":
            d.params.c, d.params.prior_n = float("inf"), 0.0
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(d.device)  # noqa: E731
        hp = np.zeros((b.N, cols), np.float32)
        hp[:, :R] = h
        dh, dt = up(hp), up(target)
        d.cluster()
        d.cluster_geometry()
        kb.kb_strategy_mask(d.batch, cols, dh, dt, d.rep, theta, d.M, d.nvalid)
        sel_log = torch.full((T, b.G, 3), -7, dtype=torch.int32, device=d.device)
        ksel_log = torch.full((T, b.G), -7, dtype=torch.int32, device=d.device)
        ip = kb.kb_iterate_params(T, 5, 3, int(variant == "warm"), cols, theta, kb.kb_sample_params(9, 77, 0.8))
        d.iterate(ip, dh, dt, up(rw), up(ok), sel_log, ksel_log, alive=None if alive is None else up(alive))
        torch.cuda.synchronize()
        out = {k: d.host(k).copy() for k in ("visits", "rsum", "t", "assign", "cent", "counts", "objective", "rep",
                                             "radius", "M", "nvalid", "Ncs", "mu", "ucb")}
        out["sel_log"], out["ksel_log"] = sel_log.cpu().numpy(), ksel_log.cpu().numpy()
        got.append(out)
    for k in got[0]:
        np.testing.assert_array_equal(got[0][k].view(np.uint8), got[1][k].view(np.uint8), err_msg=k)
    assert (got[0]["ksel_log"] >= 0).any()


@pytest.mark.parametrize("G", [100, 300])
def test_round_of_short_searches_with_many_strategies(kb, G):
    """Strategy counts whose tables leave no room for four searches in a workgroup: clustering by a wave
    per search, selection by a workgroup each, with a workspace that holds anything."""
    import torch
    b = synth.config5(G=G, nmin=1, nmax=60, D=6, S=110, iters=5, kcap=16, kdiv=2, seed=31)
    outs = ("bound", "alive", "assign", "cent", "counts", "Ncs", "mu", "ucb", "sel")
    one, three = kb.DeviceBatch(b), kb.DeviceBatch(b)
    one.ws.fill_(0x5a)
    one.round()
    three.prune()
    three.cluster()
    three.ucb_select()
    torch.cuda.synchronize()
    for k in outs:
        np.testing.assert_array_equal(one.host(k).view(np.uint8), three.host(k).view(np.uint8), err_msg=k)
