"""The form of the Lloyd kernel for a single step (256 threads per search: many searches beside the
longest) against the vector-ALU scorer, which takes the general form: one and two centroid tiles, row
lengths at the edges of K-steps and of 16-byte pieces, searches of fewer rows than centroids, equal
distances, more doubtful candidates than the list holds, rows larger than the first ones."""
import numpy as np
import pytest

from paper_2511_18868_amd import synth
from kbcheck import assert_rel_close, takes_256_threads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def kb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_18868_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("D", [1, 3, 5, 16, 17, 31, 33, 48, 49, 64])
@pytest.mark.parametrize("kcap", [17, 32, 33, 64])
@pytest.mark.parametrize("rows", ["plain", "grid", "late"])
def test_single_step(kb, D, kcap, rows):
    import torch
    b = synth.config5(G=900, nmin=1, nmax=100, D=D, S=3, iters=1, kcap=kcap, kdiv=2, seed=70 + D)
    long = synth.config2(N=1500, D=D, K=kcap, S=3, iters=1, seed=5)
    b = synth.concat(b, long, "step")
    assert takes_256_threads(b)
    if rows == "grid":          # equal distances
        b.X[:] = np.rint(b.X)
    if rows == "late":          # beyond the rows from which the scale is estimated
        b.X[b.seg_off[-1] - 100:] *= 1.0e4
    first = np.concatenate([np.minimum(np.arange(s, s + k), e - 1) for s, e, k in
                            zip(b.seg_off[:-1], b.seg_off[1:], np.diff(b.koff))]).astype(np.int64)
    given = torch.from_numpy(b.X[first][::-1].copy())
    for init in (False, True):
        out = []
        for mode in (0, 1):
            d = kb.DeviceBatch(b, iters=1, scorer=mode)
            d.ws.fill_(0x37)
            start = given.to(d.device) if init else None
            kb.kb_cluster(d.batch, d.params, d.X, start, d.assign, d.cent, d.counts, d.objective, d.ws, d.ws_bytes)
            torch.cuda.synchronize()
            out.append({k: d.host(k).copy() for k in ("assign", "cent", "counts", "objective")})
        for k in ("assign", "cent", "counts"):
            np.testing.assert_array_equal(out[0][k].view(np.uint8), out[1][k].view(np.uint8), err_msg=k)
        assert_rel_close(out[0]["objective"], out[1]["objective"], what="objective")
