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
