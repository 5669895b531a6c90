"""Seeding where the fp32 pass cannot decide alone: repeated rows, features on a coarse
grid (exact ties everywhere), values so small or large that squares leave the fp32 range,
and searches at the borders of the register, LDS and streamed shares of a workgroup.
Farthest points are exact and compared exactly; the randomised picks wherever the oracle
sees no near-tie."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import oracle  # noqa: E402


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_18868_amd import binding
    return binding


def _features(kind, N, D, rng):
    x = rng.standard_normal((N, D)).astype(np.float32)
    if kind == "grid":
        return np.rint(x).astype(np.float32)
    if kind == "repeated":
        return x[rng.integers(0, max(1, N // 40), N)].copy()
    if kind == "equal":
        return np.ones((N, D), np.float32)
    if kind == "tiny":
        return (x * np.float32(1e-21)).astype(np.float32)
    if kind == "huge":
        return (x * np.float32(3e19)).astype(np.float32)
    if kind == "mixed_scale":
        return (x * (10.0 ** rng.uniform(-22, 2, (N, 1)))).astype(np.float32)
    return x


@pytest.mark.parametrize("D", [2, 13, 32, 47, 64])
@pytest.mark.parametrize("kind", ["plain", "grid", "repeated", "equal", "tiny", "huge", "mixed_scale"])
def test_seeds_where_fp32_cannot_decide(kb, kind, D):
    rng = np.random.default_rng(1000 * D + len(kind))
    n = np.array([1, 63, 64, 65, 511, 513, 1537, 2120, 2771, 3100, 4095, 4096])
    k = np.minimum(np.maximum(1, n // 40), 24)
    seg_off = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    koff = np.concatenate([[0], np.cumsum(k)]).astype(np.int32)
    G, N, ksum = len(n), int(n.sum()), int(k.sum())
    X = _features(kind, N, D, rng)
    dev = torch.device("cuda:0")
    so, ko, Xd = (torch.from_numpy(v).to(dev) for v in (seg_off, koff, X))
    batch = kb.make_batch(G, D, 4, N, int(k.max()), ksum, int(n.max()), so, ko)
    wsb = kb.kb_workspace_bytes(batch, kb.make_params(1.0, 1.0, 1.0, 0.0, 0.5, 1))
    ws = torch.empty(wsb, dtype=torch.uint8, device=dev)
    cent = torch.zeros(ksum, D, device=dev)
    pick = torch.zeros(ksum, dtype=torch.int32, device=dev)
    kb.kb_seed_farthest(batch, Xd, cent, pick, ws, wsb)
    torch.cuda.synchronize()
    want = oracle.seed_farthest(seg_off, koff, X)
    np.testing.assert_array_equal(pick.cpu().numpy(), want.pick)
    np.testing.assert_array_equal(cent.cpu().numpy(), want.cent)
    for draw0 in (0, 77):
        kb.kb_seed_dsquared(batch, Xd, 12345, draw0, cent, pick, ws, wsb)
        torch.cuda.synchronize()
        want = oracle.seed_dsquared(seg_off, koff, X, 12345, draw0)
        clear = np.repeat(want.near == 0, k)
        assert clear.mean() > 0.5
        np.testing.assert_array_equal(pick.cpu().numpy()[clear], want.pick[clear])
