"""Representatives and radii over the candidates-per-workgroup choices and over row lengths whose 16-byte
pieces cross from row to row: first and last tiles of one row and of fewer than four values, searches that
cross borders of 512, 1024 and 2048, against the oracle (both exact)."""
import numpy as np
import pytest

import oracle
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


def _run(kb, b):
    import torch
    cl = oracle.cluster(b.seg_off, b.koff, b.X, 1)
    d = kb.DeviceBatch(b)
    d.cent.copy_(torch.from_numpy(np.ascontiguousarray(cl.cent, np.float32)))
    d.assign.copy_(torch.from_numpy(np.ascontiguousarray(cl.assign, np.int32)))
    d.cluster_geometry()
    torch.cuda.synchronize()
    geo = oracle.cluster_geometry(b.seg_off, b.koff, b.X, d.host("cent"), d.host("assign"))
    np.testing.assert_array_equal(d.host("rep"), geo.rep)
    np.testing.assert_array_equal(d.host("radius"), geo.radius.astype(np.float32))


@pytest.mark.parametrize("D", [1, 2, 3, 5, 6, 15, 16, 17, 31, 33, 47, 50, 63])
@pytest.mark.parametrize("kcap", [4, 64, 200])
def test_geometry_over_ranges_and_row_lengths(kb, D, kcap):
    # one row alone, then rows enough for several ranges of 512 (kcap 64), 1024 (200) and for whole ones
    one = synth.config2(N=1, D=D, K=1, S=2, iters=1, seed=1)
    few = synth.config2(N=3, D=D, K=1, S=2, iters=1, seed=2)
    long_ = synth.config2(N=2600, D=D, K=kcap, S=2, iters=1, seed=3)
    some = synth.config5(G=7, nmin=250, nmax=700, D=D, S=2, iters=1, kcap=kcap, kdiv=3, seed=4)
    b = one
    for i, other in enumerate((few, long_, some, one)):
        b = synth.concat(b, other, f"ranges{i}")
    _run(kb, b)
