"""Cluster diameters where the matrix-core tiles can go wrong: cluster sizes around 32, 64 and
their multiples, row lengths that fill no chunk, repeated rows and equal distances, tight clusters
far from the origin, magnitudes whose squares leave the safe range, rows that are not finite.
Every diameter against fp64 with the bound of the definition's fp32 chain (relative (D + 2) 2^-24
on the squared distance), and bit for bit against the wave-per-search kernel, which forms the
same chain for every pair, wherever a search is short enough for it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHORT = [1, 2, 3, 31, 32, 33, 47, 63, 64]          # one cluster each, searches of at most 64
LONG = [65, 96, 97, 128, 129, 200, 321]


@pytest.fixture(scope="module")
def kb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2511_18868_amd import binding
    return binding


def _rows(kind, N, D, rng):
    x = rng.standard_normal((N, D)).astype(np.float32)
    if kind == "grid":
        return np.rint(x)
    if kind == "repeated":
        return x[rng.integers(0, max(1, N // 40), N)].copy()
    if kind == "few":                     # eight distinct rows
        return x[rng.integers(0, min(8, N), N)].copy()
    if kind == "onehot":                  # all distances 0 or sqrt(2)
        return np.eye(D, dtype=np.float32)[rng.integers(0, D, N)]
    if kind == "equal":
        return np.ones((N, D), np.float32)
    if kind == "far":
        return np.float32(1000.0) + np.float32(0.05) * x
    if kind == "tiny":
        return x * np.float32(1e-17)
    if kind == "huge":
        return x * np.float32(1e18)
    if kind == "infinite":
        x[rng.random(N) < 0.1, D // 2] = np.inf
        x[rng.random(N) < 0.1, 0] = np.nan
    return x


def _diameters(kb, sizes_of_clusters, X):
    """sizes_of_clusters: per search the members of its clusters, listed round robin by rows."""
    dev = torch.device("cuda:0")
    n = np.array([sum(c) for c in sizes_of_clusters])
    k = np.array([len(c) for c in sizes_of_clusters])
    off, koff = np.concatenate([[0], np.cumsum(n)]), np.concatenate([[0], np.cumsum(k)])
    assign = np.empty(len(X), np.int32)
    for g, c in enumerate(sizes_of_clusters):
        a = np.repeat(np.arange(len(c)), c)
        assign[off[g]:off[g + 1]] = np.random.default_rng(g).permutation(a)
    up = lambda v, t: torch.from_numpy(np.ascontiguousarray(v.astype(t))).to(dev)  # noqa: E731
    seg, ko, xd, ad = up(off, np.int32), up(koff, np.int32), up(X, np.float32), up(assign, np.int32)
    b = kb.make_batch(len(n), X.shape[1], 4, len(X), int(k.max()), int(k.sum()), int(n.max()), seg, ko)
    p = kb.make_params(1e15, 1e12, 1.0, 0.0, 0.5, 1)
    wb = kb.kb_workspace_bytes(b, p)
    ws = torch.randint(0, 255, (max(wb, 256),), dtype=torch.uint8, device=dev)
    diam = torch.full((int(k.sum()),), -1.0, device=dev)
    kb.kb_cluster_diameter(b, xd, ad, diam, ws, wb)
    torch.cuda.synchronize()
    return diam.cpu().numpy(), assign, off, koff


def _want(X, assign, off, koff):
    out = np.zeros(koff[-1])
    for g in range(len(off) - 1):
        for j in range(koff[g + 1] - koff[g]):
            m = X[off[g]:off[g + 1]][assign[off[g]:off[g + 1]] == j].astype(np.float64)
            best = 0.0
            for i in range(len(m) - 1):
                with np.errstate(invalid="ignore"):
                    d2 = ((m[i + 1:] - m[i]) ** 2).sum(1)
                d2 = d2[~np.isnan(d2)]               # a distance that is no number does not count
                if len(d2):
                    best = max(best, d2.max())
            out[koff[g] + j] = np.sqrt(best)
    return out


@pytest.mark.parametrize("kind", ["plain", "grid", "repeated", "few", "onehot", "equal", "far", "tiny", "huge",
                                  "infinite"])
@pytest.mark.parametrize("D", [1, 3, 4, 7, 8, 9, 21, 40, 48, 50, 64])
def test_diameters_at_the_edges_of_the_tiles(kb, D, kind):
    rng = np.random.default_rng([D, len(kind)])
    short, long_ = [[n] for n in SHORT] + [[5, 30, 1, 20]], [[n] for n in LONG] + [[40, 70, 1, 33, 2] * 3]
    n_short = sum(map(sum, short))
    X = _rows(kind, n_short + sum(map(sum, long_)), D, rng)
    got, assign, off, koff = _diameters(kb, short + long_, X)
    want = _want(X, assign, off, koff)
    fin = np.isfinite(want)
    np.testing.assert_array_equal(got[~fin], want[~fin])
    assert (np.abs(got[fin] - want[fin]) <= (D + 4) * 2.0 ** -24 * want[fin]).all()
    alone, _, _, _ = _diameters(kb, short, X[:n_short])          # a wave per search
    np.testing.assert_array_equal(got[:len(alone)].view(np.uint32), alone.view(np.uint32))


@pytest.mark.parametrize("D", [5, 48])
def test_diameters_beside_a_search_too_long_for_one_workgroup(kb, D):
    # more than 16384 candidates: grouped by the range walks, units numbered over the whole batch
    rng = np.random.default_rng(D)
    sizes = [[n] for n in LONG] + [[100] * 170] + [[64, 65, 2]]
    X = _rows("plain", sum(map(sum, sizes)), D, rng)
    got, assign, off, koff = _diameters(kb, sizes, X)
    want = _want(X, assign, off, koff)
    assert (np.abs(got - want) <= (D + 4) * 2.0 ** -24 * want).all()
    parts, _, _, _ = _diameters(kb, sizes[:len(LONG)], X[:sum(LONG)])
    np.testing.assert_array_equal(got[:len(LONG)].view(np.uint32), parts.view(np.uint32))


@pytest.mark.parametrize("D", [3, 8, 30, 50])
@pytest.mark.parametrize("sizes", [[[16384]], [[5000, 70, 40], [9000, 31], [12000]], [[20000, 64]]],
                         ids=["one", "several", "long"])
def test_equal_distances_in_clusters_of_many_units(kb, sizes, D):
    """Distances of 0 and sqrt(2) everywhere, so that every unit is evaluated whole, several in a
    row by one wave - and one pair farther apart in each search's first cluster."""
    rng = np.random.default_rng(D)
    X = _rows("onehot", sum(map(sum, sizes)), D, rng)
    _, assign, off, _ = _diameters(kb, sizes, X)
    want = []
    for g, c in enumerate(sizes):
        first = off[g] + np.flatnonzero(assign[off[g]:off[g + 1]] == 0)
        i, j = rng.choice(first, 2, replace=False)
        X[i], X[j] = 0.0, 0.0
        X[i, D - 1], X[j, D - 1] = 3.0, -2.5
        want += [5.5] + [np.sqrt(np.float32(2.0))] * (len(c) - 1)
    got, _, _, _ = _diameters(kb, sizes, X)
    np.testing.assert_array_equal(got, np.array(want, np.float32))


@pytest.mark.parametrize("G", [4095, 4096, 4101])
def test_diameters_of_many_searches(kb, G):
    """From 4096 searches on a workgroup groups eight of them; the last one has fewer.  Empty
    searches, searches without a pair and one long search among them."""
    rng = np.random.default_rng(G)
    D, sizes = 6, [[int(v)] if v < 12 else [int(v) // 2, 1, int(v) - int(v) // 2] for v in rng.integers(0, 90, G)]
    sizes[G // 2] = [3000, 40, 2]
    X = _rows("plain", sum(map(sum, sizes)), D, rng)
    got, assign, off, koff = _diameters(kb, sizes, X)
    want = _want(X, assign, off, koff)
    assert (np.abs(got - want) <= (D + 4) * 2.0 ** -24 * want).all()


def test_overlapping_searches_stay_inside_the_workspace(kb):
    """Offsets that go up and down (a violated precondition) make every second search the whole
    batch: far more searches with pairs than the workspace has slots for.  The numbers are then
    meaningless, but nothing beside the workspace and the output is written."""
    dev = torch.device("cuda:0")
    N, G = 200, 200_000
    off = torch.zeros(G + 1, dtype=torch.int32, device=dev)
    off[1::2] = N
    koff = torch.zeros(G + 1, dtype=torch.int32, device=dev)
    koff[1::2] = 1
    X = torch.randn(N, 8, device=dev)
    assign = torch.zeros(N, dtype=torch.int32, device=dev)
    b = kb.make_batch(G, 8, 4, N, 1, 1, N, off, koff)
    wb = kb.kb_workspace_bytes(b, kb.make_params(1e15, 1e12, 1.0, 0.0, 0.5, 1))
    wb = (wb + 255) // 256 * 256
    ws = torch.full((wb + 32 * G,), 0xA5, dtype=torch.uint8, device=dev)
    diam = torch.full((256,), -1.0, device=dev)
    kb.kb_cluster_diameter(b, X, assign, diam, ws, wb)
    torch.cuda.synchronize()
    assert (ws[wb:] == 0xA5).all()
    assert (diam[1:] == -1.0).all()
