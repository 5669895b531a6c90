"""How many kernels a call enqueues: the scheduling order (longest search first) is a launch of its own and
is formed only where a kernel of the call reads it.  Counted as the nodes of the HIP graph the call records
(nothing runs)."""
import ctypes

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


def recorded(call):
    import torch
    hip = ctypes.CDLL("libamdhip64.so")
    stream = torch.cuda.Stream()
    handle, graph, n = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(handle, 2) == 0
    call(stream)
    assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


@pytest.mark.parametrize("G,nmax,cluster,round_", [
    (200, 256, 1, 3),      # as many searches as compute units or fewer: none
    (300, 256, 1, 3),      # rows in registers, a wave per search in the selection: nobody reads it
    (300, 512, 1, 4),      # rows in registers; the selection reads it
    (300, 800, 2, 4),      # the Lloyd kernel and the selection read the same
])
def test_order_only_where_it_is_read(kb, G, nmax, cluster, round_):
    import torch
    b = synth.config5(G=G, nmin=nmax // 2, nmax=nmax, D=16, S=4, kcap=16, kdiv=8, iters=3, seed=9)
    b = synth.concat(b, synth.config2(N=nmax, D=16, K=16, S=4, iters=3, seed=9), "launches")
    d = kb.DeviceBatch(b)
    d.round()                     # (the library's code is loaded outside of the recording)
    torch.cuda.synchronize()
    assert recorded(lambda st: d.cluster(stream=st)) == cluster
    assert recorded(lambda st: d.round(stream=st)) == round_
