"""Seeding where the fp32 pass cannot decide alone: repeated rows, features on a coarse
grid (exact ties everywhere), values so small or large that squares leave the fp32 range,
searches at the borders of the register, LDS and streamed shares of a workgroup, and
variates that their leading bits do not determine.
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
    if kind == "binary":
        return (x > 0).astype(np.float32)
    if kind == "onehot":
        return np.eye(D, dtype=np.float32)[rng.integers(0, D, N)]
    if kind == "few":
        return x[rng.integers(0, min(8, N), N)].copy()
    if kind == "late":                   # a few rows far apart, chosen first, then ties everywhere
        return np.where(rng.random((N, 1)) < 0.004, 100 * x, np.float32(0.1) * (x > 0)).astype(np.float32)
    if kind == "equal":
        return np.ones((N, D), np.float32)
    if kind == "tiny":
        return (x * np.float32(1e-21)).astype(np.float32)
    if kind == "huge":
        return (x * np.float32(3e19)).astype(np.float32)
    if kind == "mixed_scale":
        return (x * (10.0 ** rng.uniform(-22, 2, (N, 1)))).astype(np.float32)
    return x


@pytest.mark.parametrize("D", [2, 13, 32, 47, 48, 64])
@pytest.mark.parametrize("kind", ["plain", "grid", "repeated", "binary", "onehot", "few", "late", "equal", "tiny", "huge",
                                  "mixed_scale"])
def test_seeds_where_fp32_cannot_decide(kb, kind, D):
    rng = np.random.default_rng(1000 * D + len(kind))
    n = np.array([1, 63, 64, 65, 511, 513, 1537, 2120, 2225, 2226, 2771, 3100, 4095, 4096])
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


def _first_words(k, draw, seed):
    """The first two words of Philox4x32-10 for the candidates `k` (draw and seed below 2^32)."""
    k = np.asarray(k, np.uint64)
    c = [k, np.zeros_like(k), np.full_like(k, draw), np.zeros_like(k)]
    k0, k1, low, half = seed, 0, np.uint64(0xFFFFFFFF), np.uint64(32)
    for _ in range(10):
        p, q = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(q >> half) ^ c[1] ^ np.uint64(k0), q & low, (p >> half) ^ c[3] ^ np.uint64(k1), p & low]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c[0], c[1]


# (seed, row whose variate in draw 1 is that close to 1: ~x0 of a few hundred to a few thousand)
NEAR_ONE = [(8427, 2374), (17473, 947), (6731, 2548), (25550, 391), (35594, 2480), (9907, 283), (28013, 976),
            (38008, 1197), (2769, 573)]


@pytest.mark.parametrize("D", [1, 48])
@pytest.mark.parametrize("seed,row", NEAR_ONE)
def test_a_variate_close_to_one_beside_a_close_rival(kb, seed, row, D):
    """Two rows away from all others, one with a variate u so close to 1 that its 32 leading bits
    leave ln(-ln u) uncertain by 3e-4 to 2e-3, the other 1e-4 behind or ahead of it: the side on
    which the leading bits alone name the wrong winner."""
    N = 2600
    x0, x1 = _first_words(np.arange(N), 1, seed)
    near = 0xFFFFFFFF - int(x0[row])
    assert 256 <= near < 1 << 15
    # 1 - u in units of 2^-32, exactly and with the middle of the interval for the bits left out
    exact, middle = near + ((0xFFFFFFFF - int(x1[row]) >> 12) + 0.5) * 2.0 ** -20, near + 0.5
    u = ((x0.astype(np.float64) * 2.0 ** 20 + (x1 >> np.uint64(12)).astype(np.float64)) + 0.5) * 2.0 ** -52
    gumbel = -np.log(-np.log(u))
    gumbel[row] = -np.log(-np.log1p(-exact * 2.0 ** -32))
    first = oracle.seed_dsquared(np.array([0, N], np.int32), np.array([0, 1], np.int32),
                                 np.zeros((N, D), np.float32), seed, 0).pick[0]
    rival = next(k for k in range(row // 2, N) if 0.3 < u[k] < 0.7 and k not in (row, first))
    ahead = 1e-4 if exact > middle else -1e-4
    X = np.zeros((N, D), np.float32)
    X[row, 0] = 1.0
    X[rival, 0] = np.exp(0.5 * (gumbel[row] + ahead - gumbel[rival]))
    seg_off, koff = np.array([0, N], np.int32), np.array([0, 2], np.int32)
    want = oracle.seed_dsquared(seg_off, koff, X, seed, 0)
    assert want.near[0] == 0 and want.pick[1] == (rival if ahead > 0 else row)
    dev = torch.device("cuda:0")
    so, ko, Xd = (torch.from_numpy(v).to(dev) for v in (seg_off, koff, X))
    batch = kb.make_batch(1, D, 4, N, 2, 2, N, so, ko)
    wsb = kb.kb_workspace_bytes(batch, kb.make_params(1.0, 1.0, 1.0, 0.0, 0.5, 1))
    ws = torch.empty(wsb, dtype=torch.uint8, device=dev)
    cent = torch.zeros(2, D, device=dev)
    pick = torch.zeros(2, dtype=torch.int32, device=dev)
    kb.kb_seed_dsquared(batch, Xd, seed, 0, cent, pick, ws, wsb)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(pick.cpu().numpy(), want.pick)
