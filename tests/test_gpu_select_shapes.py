"""The selection of a search by 1024 threads (batches of few searches) against the same searches by
256 threads (behind enough others): every output byte for byte, over the forms of the rows."""
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


@pytest.mark.parametrize("S", [1, 6, 12, 32, 40])
def test_selection_by_wide_and_by_narrow_workgroups(kb, S):
    import torch
    few = synth.config5(G=5, nmin=1, nmax=1100, D=4, S=S, kcap=64, kdiv=8, iters=2, seed=700 + S)
    rest = synth.config5(G=520, nmin=1, nmax=300, D=4, S=S, kcap=8, kdiv=8, iters=2, seed=800 + S)
    both = synth.concat(few, rest, "few then many")
    out = []
    for b in (few, both):
        d = kb.DeviceBatch(b)
        d.prune()
        d.cluster()
        d.ucb_select()
        torch.cuda.synchronize()
        out.append({k: d.host(k).copy() for k in ("assign", "Ncs", "mu", "ucb", "sel")})
    for k, n in (("assign", few.N), ("Ncs", few.Ksum), ("mu", few.Ksum), ("ucb", few.Ksum), ("sel", few.G)):
        np.testing.assert_array_equal(out[0][k].view(np.uint8), out[1][k][:n].view(np.uint8), err_msg=k)


def test_scores_that_are_not_numbers_choose_the_same_arm(kb):
    """c = +inf at t = 1: inf * sqrt(0) in every arm that was tried.  Such scores have no order, and which of
    them a search ends with follows from how its arms are dealt to the threads: the same whatever else the
    batch holds."""
    import torch
    few = synth.config5(G=5, nmin=1000, nmax=1100, D=4, S=32, kcap=64, kdiv=8, iters=2, seed=71)
    rest = synth.config5(G=520, nmin=1, nmax=30, D=4, S=32, kcap=8, kdiv=8, iters=2, seed=72)
    out = []
    for b in (few, synth.concat(few, rest, "few then many")):
        b.t[:] = 1
        d = kb.DeviceBatch(b)
        d.params.c = float("inf")
        d.prune()
        d.cluster()
        d.alive.copy_((d.assign > 0).to(torch.uint8))     # no alive member in the clusters of the first arms
        d.ucb_select()
        torch.cuda.synchronize()
        out.append(d.host("sel")[:few.G].copy())
    assert (out[0][:, 0] > 0).all()
    np.testing.assert_array_equal(out[0], out[1])
