"""How many kernels a call enqueues - the scheduling order (longest search first), a launch of its own, only
where a kernel of the call reads it; iterations of short searches in one launch only where that is faster -
counted as the nodes of the HIP graph that the call records (nothing of it runs)."""
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


@pytest.mark.parametrize("G,D,S,K,rounds,one", [
    (256, 5, 16, 8, 1, True),         # a compute unit each: always one launch
    (1500, 5, 6, 3, 1, True),         # all on the chip at once, an arm per lane
    (1280, 5, 16, 8, 1, True),
    (1500, 5, 16, 8, 10, False),      # four arms per lane beside short rows: too few iterations ...
    (1500, 5, 16, 8, 11, True),       # ... and enough
    (1500, 17, 16, 8, 1, True),       # four arms beside longer rows
    (5000, 5, 3, 2, 1, True),         # more than the chip holds, sixteen waves per unit
    (5000, 40, 3, 2, 15, False),      # ... and eight: too few iterations
    (5000, 40, 3, 2, 16, True),
    (5000, 5, 16, 8, 60, False),      # four arms on a full chip
    (5000, 20, 16, 8, 10, False),
    (5000, 20, 16, 8, 11, True),
])
def test_iterations_in_one_launch_where_that_is_faster(kb, G, D, S, K, rounds, one):
    """Both sides of every line of the rule, with a re-clustering in the first iteration."""
    import torch
    b = synth.config5(G=G, nmin=18, nmax=20, D=D, S=S, kcap=K, kdiv=2, iters=2, seed=7)
    d = kb.DeviceBatch(b)
    h, target, theta = synth.signatures(b, 3)
    dh, dt = torch.from_numpy(h).to(d.device), torch.from_numpy(target).to(d.device)
    new = lambda *shape, dtype=torch.int32: torch.zeros(shape, dtype=dtype, device=d.device)      # noqa: E731
    rw, ok, sel, ksel = new(rounds, G, dtype=torch.float32), new(rounds, G, dtype=torch.uint8), new(rounds, G, 3), new(rounds, G)
    ip = kb.kb_iterate_params(rounds, 1000, 0, 0, 3, theta, kb.kb_sample_params(1, 1, 1.0))
    d.iterate(ip, dh, dt, rw, ok, sel, ksel)
    torch.cuda.synchronize()
    assert (recorded(lambda st: d.iterate(ip, dh, dt, rw, ok, sel, ksel, stream=st)) == 1) == one
