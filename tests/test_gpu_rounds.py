"""The iterations between two re-clusterings, which kb_iterate runs in one launch, against
the same stages called one by one (masked selection, draw, update): every output of
every round byte for byte, over the strategy counts that select the forms of the
aggregation and over the batch sizes that select wave, narrow and wide workgroups."""
import numpy as np
import pytest

from paper_2511_18868_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_18868_amd import binding
    binding.lib()
    return binding


def _batch(shape, S):
    if shape == "wave":           # a wave per search; 183 searches fill no whole workgroup at the end
        return synth.config5(G=183, nmin=2, nmax=70, D=8, S=S, kcap=6, kdiv=2, iters=3, seed=301)
    if shape == "waveedge":       # the longest searches a wave takes, and searches of one candidate
        return synth.config5(G=37, nmin=1, nmax=256, D=8, S=S, kcap=16, kdiv=1, iters=3, seed=302)
    if shape == "wide":           # 257 candidates and more, few searches
        return synth.config5(G=9, nmin=200, nmax=4100, D=8, S=S, kcap=64, kdiv=16, iters=3, seed=303)
    if shape == "narrow":         # more searches than the wide form takes
        return synth.config5(G=520, nmin=40, nmax=600, D=8, S=S, kcap=24, kdiv=16, iters=3, seed=304)
    if shape == "onecluster":     # too many members for the draw of one workgroup: launches of their own
        return synth.config2(seed=307, N=12000, D=8, K=1, S=S, iters=3)
    return synth.config2(seed=305, N=16384, D=8, K=2, S=S, iters=3)     # the longest search of one workgroup


def _compare_with_the_stages(kb, b, T, **params):
    """T iterations of one kb_iterate call against the stages called one by one."""
    import torch
    R = 3
    h, target, _ = synth.signatures(b, R)
    theta = 0.9                   # (few arms masked)
    fb = [synth.feedback(b, seed=r) for r in range(T)]
    rw, ok = np.stack([f[0] for f in fb]), np.stack([f[1] for f in fb])
    alive = (np.arange(b.N) % 4 != 1).astype(np.uint8)

    def start():
        d = kb.DeviceBatch(b)
        for name, value in params.items():
            setattr(d.params, name, value)
        up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(d.device)  # noqa: E731
        d.cluster()
        d.cluster_geometry()
        arr = dict(h=up(h), target=up(target), rw=up(rw), ok=up(ok), alive=up(alive))
        kb.kb_strategy_mask(d.batch, R, arr["h"], arr["target"], d.rep, theta, d.M, d.nvalid)
        return d, arr

    d, x = start()
    sel_log = torch.full((T, b.G, 3), -7, dtype=torch.int32, device=d.device)
    ksel_log = torch.full((T, b.G), -7, dtype=torch.int32, device=d.device)
    ip = kb.kb_iterate_params(T, 0, 0, 0, R, theta, kb.kb_sample_params(5, 40, 0.7))
    d.iterate(ip, x["h"], x["target"], x["rw"], x["ok"], sel_log, ksel_log, alive=x["alive"])

    e, y = start()
    for r in range(T):
        kb.kb_ucb_select_masked(e.batch, e.params, e.assign, y["alive"], None, e.M, e.visits, e.rsum, e.t,
                                e.Ncs, e.mu, e.ucb, e.sel, e.ws, e.ws_bytes)
        kb.kb_sample_signature(e.batch, kb.kb_sample_params(5, 40 + r, 0.7), e.assign, y["alive"], R,
                               y["h"], y["target"], theta, e.sel, e.ksel, e.ws, e.ws_bytes)
        torch.testing.assert_close(sel_log[r], e.sel, rtol=0, atol=0)
        torch.testing.assert_close(ksel_log[r], e.ksel, rtol=0, atol=0)
        kb.kb_update_stats(e.batch, e.params, e.sel, e.ksel, y["rw"][r], y["ok"][r], e.visits, e.rsum,
                           e.Ncs, e.mu, e.t)
    assert (ksel_log >= 0).any()
    for name in ("visits", "rsum", "t", "Ncs", "mu", "ucb"):
        a, c = d.host(name), e.host(name)
        np.testing.assert_array_equal(a.view(np.uint8), c.view(np.uint8), err_msg=name)


@pytest.mark.parametrize("S", [1, 6, 12, 32])
@pytest.mark.parametrize("shape", ["wave", "waveedge", "wide", "narrow", "longest", "onecluster"])
def test_rounds_in_one_launch_equal_the_stages_one_by_one(kb, shape, S):
    _compare_with_the_stages(kb, _batch(shape, S), 5)


@pytest.mark.parametrize("prior_n", [0.0, 1.0])
@pytest.mark.parametrize("shape", ["wave", "narrow"])
def test_scores_that_are_not_numbers_choose_one_arm(kb, shape, prior_n):
    """c = +inf passes the checks and gives inf * sqrt(ln 1 / n) = NaN in a search's first
    iteration (beside +inf for untried arms when there are no pseudo-visits), +inf later."""
    b = _batch(shape, 6)
    b.t[:] = 1
    b.visits[:, ::2] = 0
    b.rsum[:, ::2] = 0.0
    _compare_with_the_stages(kb, b, 3, c=float("inf"), prior_n=prior_n)


@pytest.mark.parametrize("nmax", [40, 600], ids=["wave", "workgroup"])
def test_more_rounds_than_one_launch_runs(kb, nmax):
    """A launch runs 1024 iterations at most: the next one rebuilds its tables from the
    advanced history and goes on with the logs, rewards, draws and t where the first ended."""
    b = synth.config5(G=3, nmin=nmax // 2, nmax=nmax, D=8, S=6, kcap=4, kdiv=4, iters=3, seed=306)
    _compare_with_the_stages(kb, b, 1030)
