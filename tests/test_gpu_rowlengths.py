"""Rows whose length is no multiple of 4 features, in both workgroup shapes of the
one-workgroup Lloyd kernel: the last 16-byte piece of a row is loaded so that it ends
with the row and is shifted into place (rows of fewer than 4 features value by
value).  Whole rounds against the oracle, bit for bit on the searches it saw no
near-tie in."""
import numpy as np
import pytest

import oracle
from paper_2511_18868_amd import synth
from kbcheck import assert_cent_close, assert_rel_close, search_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_18868_amd import binding
    binding.lib()
    return binding


def batch(D, K, G, seed):
    """Searches of 65 candidates and more: ragged last tiles, the last one ending with X."""
    rng = np.random.default_rng(seed)
    b = None
    for i in range(G):
        n = int(rng.integers(65, (10 if G > 256 else 40) * K + 70))
        one = synth.config2(seed=seed * 1000 + i, N=n, D=D, K=K, S=3, iters=5)
        b = one if b is None else synth.concat(b, one, f"D{D}")
    return b


def compare_round(kb, b, scorer, few_clean):
    import torch
    d = kb.DeviceBatch(b, scorer=scorer)
    d.round()
    torch.cuda.synchronize()
    ora = oracle.round_(b)
    clean = ora.dirty == 0
    assert clean.sum() >= few_clean
    cp, ck = clean[search_of(b.seg_off)], np.repeat(clean, np.diff(b.koff))
    np.testing.assert_array_equal(d.host("bound").view(np.uint32), ora.bound.view(np.uint32))
    np.testing.assert_array_equal(d.host("alive"), ora.alive)
    np.testing.assert_array_equal(d.host("assign")[cp], ora.assign[cp])
    np.testing.assert_array_equal(d.host("counts")[ck], ora.counts[ck])
    assert_cent_close(d.host("cent")[ck], ora.cent[ck])
    assert_rel_close(d.host("objective")[clean], ora.objective[clean], what="objective")
    np.testing.assert_array_equal(d.host("Ncs")[ck], ora.Ncs[ck])
    ok = clean & (ora.near == 0)
    np.testing.assert_array_equal(d.host("sel")[ok], ora.sel[ok])


@pytest.mark.parametrize("D", [1, 2, 3, 5, 7, 15, 17, 30, 33, 47, 49, 62, 63])
@pytest.mark.parametrize("K", [5, 40], ids=["onetile", "twotiles"])
@pytest.mark.parametrize("G", [6, 450], ids=["wide", "narrow"])
def test_row_lengths(kb, D, K, G):
    b = batch(D, K, G, seed=40 + D)
    # (the oracle sees a near-tie in at most 4 of these 450 searches)
    compare_round(kb, b, 0, G - max(1, G // 90))
