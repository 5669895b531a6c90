"""The Lloyd kernel that keeps a search's rows in registers (at most 256 searches, up to 512 candidates,
256 with more than 32 clusters; two searches per compute unit, up to 1024
searches of few features) against the kernel that fetches them, which scorer mode 2 takes: row
lengths at the edges of K-steps and 16-byte pieces, tiles and pairs of tiles filled exactly and by one,
equal distances, caller-supplied centroids, stopping early."""
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


@pytest.mark.parametrize("D", [1, 2, 4, 7, 16, 17, 33, 48, 50, 64])
@pytest.mark.parametrize("nmax,kcap,kdiv", [(256, 64, 2), (257, 32, 4), (512, 32, 8), (100, 3, 4)])
@pytest.mark.parametrize("stop", [0, 1])
def test_resident_rows_give_the_bytes_of_fetched_rows(kb, D, nmax, kcap, kdiv, stop):
    import torch
    b = synth.config5(G=24, nmin=1, nmax=nmax, D=D, S=3, iters=9, kcap=kcap, kdiv=kdiv, seed=900 + D)
    longest = synth.config2(N=nmax, D=D, K=min(kcap, nmax // kdiv), S=3, iters=9, seed=3)
    b = synth.concat(b, longest, "resident")
    if D % 2:          # rows on a grid: equal distances
        b.X[:] = np.rint(2.0 * b.X) / 2.0
    rows = np.concatenate([np.arange(e - 1, e - 1 - k, -1) for e, k in
                           zip(b.seg_off[1:], np.diff(b.koff))]).astype(np.int64)
    for init in (False, True):
        out = []
        for mode in (0, 2):
            d = kb.DeviceBatch(b, iters=9, scorer=mode, stop_early=stop)
            start = torch.from_numpy(b.X[rows].copy()).to(d.device) if init else None
            kb.kb_cluster(d.batch, d.params, d.X, start, d.assign, d.cent, d.counts, d.objective, d.ws, d.ws_bytes)
            torch.cuda.synchronize()
            out.append({k: d.host(k).copy() for k in ("assign", "cent", "counts", "objective")})
        for k in ("assign", "cent", "counts"):
            np.testing.assert_array_equal(out[0][k].view(np.uint8), out[1][k].view(np.uint8), err_msg=k)
        assert_rel_close(out[0]["objective"], out[1]["objective"], what="objective")


@pytest.mark.parametrize("G,nmax", [(256, 256), (511, 256), (256, 512), (512, 257), (1023, 256), (700, 512)])  # (and one)
@pytest.mark.parametrize("D,kcap", [(1, 32), (6, 64), (16, 32), (17, 32), (32, 33), (33, 5), (48, 32)])
@pytest.mark.parametrize("stop,init", [(0, False), (1, True)])
def test_two_searches_per_compute_unit(kb, G, nmax, D, kcap, stop, init):
    import torch
    b = synth.config5(G=G, nmin=1, nmax=nmax, D=D, S=3, iters=6, kcap=kcap, kdiv=2, seed=30 + D)
    b = synth.concat(b, synth.config2(N=nmax, D=D, K=kcap, S=3, iters=6, seed=4), "pair")
    if D % 2:          # rows on a grid: equal distances
        b.X[:] = np.rint(2.0 * b.X) / 2.0
    rows = np.concatenate([np.arange(e - 1, e - 1 - k, -1) for e, k in
                           zip(b.seg_off[1:], np.diff(b.koff))]).astype(np.int64)
    out = []
    for mode in (0, 2):
        d = kb.DeviceBatch(b, iters=6, scorer=mode, stop_early=stop)
        d.ws.fill_(0x37)
        start = torch.from_numpy(b.X[rows].copy()).to(d.device) if init else None
        kb.kb_cluster(d.batch, d.params, d.X, start, d.assign, d.cent, d.counts, d.objective, d.ws, d.ws_bytes)
        torch.cuda.synchronize()
        out.append({k: d.host(k).copy() for k in ("assign", "cent", "counts", "objective")})
    for k in ("assign", "cent", "counts"):
        np.testing.assert_array_equal(out[0][k].view(np.uint8), out[1][k].view(np.uint8), err_msg=k)
    assert_rel_close(out[0]["objective"], out[1]["objective"], what="objective")


@pytest.mark.parametrize("G,n", [(3, 128), (3, 512), (300, 128), (300, 512)])   # tiles of a wave; searches per unit
def test_objective_member_by_member_sums_in_fp64(kb, G, n):
    """Rows at c + d and c - d, c so far from the origin that sum |x|^2 leaves nothing to subtract from:
    the squares are added member by member.  d^2 = 2^24 in the first four features together and 4 in the
    next four - every group of four is exact in fp32, all eight together are not: fp64 takes them from there."""
    import torch
    b = synth.config5(G=G, nmin=n, nmax=n, D=8, S=3, iters=3, kcap=1, kdiv=1, seed=8)
    sign = np.where(np.arange(b.N) % 2 == 0, 1.0, -1.0)[:, None]
    b.X[:] = 2.0 ** 23 + sign * np.array([4096, 0, 0, 0, 1, 1, 1, 1])
    for mode in (0, 2):
        d = kb.DeviceBatch(b, iters=3, scorer=mode)
        kb.kb_cluster(d.batch, d.params, d.X, None, d.assign, d.cent, d.counts, d.objective, d.ws, d.ws_bytes)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(d.host("cent"), np.float32(2.0 ** 23))
        np.testing.assert_array_equal(d.host("objective"), np.float32(n * (2.0 ** 24 + 4)), err_msg=str(mode))
