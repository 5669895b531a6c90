"""The draw by a wave, by 256 and by 1024 threads per search and by ranges of candidates: the same
searches behind batches that select each, at the lengths where the forms change, both potentials.  The
variates belong to global indices, so the searches come first and the fillers behind them."""
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


def _draw(kb, b, signature):
    import torch
    rng = np.random.default_rng(5)
    h = rng.random((120000, 3), dtype=np.float32)          # (the first searches' rows are the same in every batch)
    d = kb.DeviceBatch(b)
    d.round()
    sp = kb.kb_sample_params(77, 5, 0.9)
    if signature:
        assert b.N <= len(h)
        dh = torch.from_numpy(h[:b.N].copy()).to(d.device)
        dt = (torch.arange(b.S, dtype=torch.int32) % 3).to(d.device)
        kb.kb_sample_signature(d.batch, sp, d.assign, None, 3, dh, dt, 0.75, d.sel, d.ksel, d.ws, d.ws_bytes)
    else:
        kb.kb_sample(d.batch, sp, d.assign, d.alive, d.bound, d.incumbent, d.sel, d.ksel, d.ws, d.ws_bytes)
    torch.cuda.synchronize()
    return d.host("ksel").copy()


@pytest.mark.parametrize("signature", [False, True])
@pytest.mark.parametrize("longest", [257, 2048, 2049, 4096, 11001])
def test_every_form_of_the_draw_chooses_alike(kb, longest, signature):
    first = synth.config5(G=9, nmin=1, nmax=longest, D=4, S=4, iters=1, kcap=8, kdiv=8, seed=60)
    first = synth.concat(first, synth.config2(N=longest, D=4, K=2, S=4, iters=1, seed=61), "draw")
    want = _draw(kb, first, signature)
    assert (want >= 0).any()
    fillers = (synth.config2(N=17000, D=4, K=2, S=4, iters=1, seed=62),                         # ranges
               synth.config2(N=5000, D=4, K=2, S=4, iters=1, seed=63),                          # 1024 threads
               synth.config2(N=5000, D=4, K=32, S=4, iters=1, seed=66),                         # beyond 11000, too
               synth.config5(G=300, nmin=1, nmax=200, D=4, S=4, iters=1, kcap=4, kdiv=8, seed=64),      # 256
               synth.config5(G=5000, nmin=1, nmax=30, D=4, S=4, iters=1, kcap=2, kdiv=8, seed=65))      # a wave
    for f in fillers:
        got = _draw(kb, synth.concat(first, f, "draw behind"), signature)
        np.testing.assert_array_equal(got[:first.G], want)
