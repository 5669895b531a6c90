"""The selection of long searches cut into ranges, in batches of few and of more searches and next to
searches that a workgroup takes whole, against the oracle: candidates on both sides of the lines, more
cluster arms than a range has candidates, arms beyond those of the shortest ranges."""
import numpy as np
import pytest

from kbcheck import assert_rel_close
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


@pytest.mark.parametrize("sizes,K,S", [((6000,), 4, 3), ((6001,), 4, 6), ((6001, 40, 9000), 64, 32),
                                       ((16385, 3), 8, 5), ((7000,) * 9, 4, 4), ((8000,), 4, 4), ((8001,), 4, 1),
                                       ((12000, 50), 8, 2), ((12001, 7000, 12000), 8, 4), ((20000,), 256, 32), ((70000,), 3, 12)])
def test_selection_in_ranges(kb, sizes, K, S):
    import torch
    parts = [synth.config2(N=n, D=4, K=min(K, n), S=S, iters=1, seed=40 + i) for i, n in enumerate(sizes)]
    b = parts[0]
    for i, p in enumerate(parts[1:]):
        b = synth.concat(b, p, f"ranges{i}")
    d = kb.DeviceBatch(b)
    d.ws.fill_(0x37)
    d.prune()
    rng = np.random.default_rng(3)
    kg = np.repeat(np.diff(b.koff), np.diff(b.seg_off))
    assign = rng.integers(0, kg).astype(np.int32)
    d.assign.copy_(torch.from_numpy(assign))
    d.ucb_select()
    torch.cuda.synchronize()
    Ncs = np.zeros((b.Ksum, S), np.int64)
    Rs = np.zeros((b.Ksum, S))
    alive = d.host("alive") != 0
    row = assign + np.repeat(b.koff[:-1], np.diff(b.seg_off))
    np.add.at(Ncs, row[alive], b.visits[alive])
    np.add.at(Rs, row[alive], b.rsum[alive].astype(np.float64))
    np.testing.assert_array_equal(d.host("Ncs"), Ncs)
    nt = Ncs + float(b.prior_n)
    mu = np.where(nt > 0, (Rs + b.prior_n * b.prior_mu) / np.where(nt > 0, nt, 1), np.nan)
    assert_rel_close(d.host("mu"), mu, rel=1e-6, what="mu")
    # k*: the alive member of the chosen cluster with the smallest bound
    sel, bound = d.host("sel"), d.host("bound")
    for g in range(b.G):
        lo, hi = b.seg_off[g], b.seg_off[g + 1]
        mem = np.nonzero(alive[lo:hi] & (assign[lo:hi] == sel[g, 0]))[0] + lo
        assert sel[g, 2] == mem[np.argmin(bound[mem])]
        u = d.host("ucb")[b.koff[g]:b.koff[g + 1]]
        assert u[sel[g, 0], sel[g, 1]] == u.max()
