"""Prediction with the ensemble in LDS at the edges of its rule (rows per
block, row width, depth, trees per chunk, shallow and truncated trees), bit
for bit against a numpy walk that adds the leaves in tree order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gbt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_09148_amd import gbt as g
    return g


def ensemble(gbt, depths, m, bins, seed, cut=0):
    """Trees with early leaves; cut > 0 drops that many nodes of each table's end."""
    r = np.random.default_rng(seed)
    out = []
    for D in depths:
        nn = max((2 << D) - 1 - cut, 1)
        t = np.zeros(nn, gbt.NODE_DTYPE)
        live = np.zeros(nn, bool)
        live[0] = True
        for i in range(nn):
            if not live[i]:
                t["feature"][i] = -7  # never read
                continue
            t["flags"][i] = gbt.NODE_PRESENT
            t["leaf_value"][i] = r.normal()
            if 2 * i + 2 < nn and r.random() < 0.9:
                t["feature"][i] = r.integers(0, m)
                t["threshold"][i] = r.normal()
                t["split_bin"][i] = r.integers(-1, bins + 2)
                t["flags"][i] |= gbt.NODE_DEFAULT_LEFT * int(r.integers(0, 2))
                live[2 * i + 1] = live[2 * i + 2] = True
            else:
                t["flags"][i] |= gbt.NODE_LEAF
        out.append(gbt.TreeOut(t, 0, 0, D))
    return out


def walk(gbt, trees, X, base, binned=None):
    acc = np.full(len(X), base, np.float32)
    at = np.arange(len(X))
    for t in trees:
        nodes, node = t.nodes, np.zeros(len(X), np.int64)
        while True:
            nd = nodes[node]
            go = ((nd["flags"] & gbt.NODE_LEAF) == 0) & (2 * node + 2 < len(nodes))
            if not go.any():
                break
            f = np.where(go, nd["feature"], 0)
            with np.errstate(invalid="ignore"):
                left = X[at, f] <= nd["threshold"] if binned is None else binned[at, f] < nd["split_bin"]
            left = np.where(np.isnan(X[at, f]), (nd["flags"] & gbt.NODE_DEFAULT_LEFT) != 0, left)
            node = np.where(go, 2 * node + 2 - left, node)
        acc = acc + nodes["leaf_value"][node]
    return acc


@pytest.mark.parametrize("n,m,depths,cut", [
    (1, 1, [3], 0), (63, 5, [0, 1, 2, 0], 0), (65, 28, [6] * 10, 0), (1000, 29, [8, 8, 8, 8, 8, 7, 8, 8, 8, 8], 0),
    (32_769, 28, [8] * 13, 0), (32_768, 33, [5, 5, 5, 5, 11, 4], 0), (40_001, 64, [4] * 3, 0), (300, 480, [7] * 5, 0),
    (300, 700, [5] * 5, 0), (500, 9, [12, 3], 0), (500, 9, [4] * 9, 3), (35_000, 3, [11, 10, 9], 1)])
@pytest.mark.parametrize("kind", ["raw", "binned"])
def test_predict_matches_walk(gbt, n, m, depths, cut, kind):
    predict_and_walk(gbt, n, m, depths, cut, kind)


@pytest.mark.parametrize("n,m,depths", [
    (400, 90, [4] * 5 + [2]), (400, 90, [4] * 5 + [3]), (33_000, 40, [5]), (33_000, 40, [6]),
    (33_000, 5, [0, 1, 3, 0]), (33_000, 5, [0, 1, 2, 0]), (33_000, 90, [6] * 9), (33_000, 90, [6] * 8 + [5]), (300, 480, [8] * 72),
    (500, 28, [4] * 3), (500, 28, [5, 4, 4]), (500, 28, [5]), (500, 28, [6])])
@pytest.mark.parametrize("kind", ["raw", "binned"])
def test_predict_around_the_step_rule(gbt, n, m, depths, kind):
    """Both sides of the line in steps from which rows are staged in LDS."""
    predict_and_walk(gbt, n, m, depths, 0, kind)


def predict_and_walk(gbt, n, m, depths, cut, kind):
    r = np.random.default_rng(n + m)
    X = r.normal(size=(n, m)).astype(np.float32)
    X[r.random(X.shape) < 0.1] = np.nan
    ctx = gbt.Context(0)
    trees = ensemble(gbt, depths, m, 64, n + len(depths), cut)
    Xd = torch.from_numpy(X).cuda()
    if kind == "raw":
        got = gbt.gbt_predict(ctx, trees, 0.25, raw=Xd)
        want = walk(gbt, trees, X, 0.25)
    else:
        mx = gbt.gbt_quantize(ctx, Xd, max_bin=64)
        cp, cv = mx.cuts()
        binned = np.stack([np.searchsorted(cv[cp[j]:cp[j + 1]], X[:, j]) for j in range(m)], 1)
        got = gbt.gbt_predict(ctx, trees, 0.25, binned=mx)
        want = walk(gbt, trees, X, 0.25, binned)
    assert got.cpu().numpy().tobytes() == want.tobytes()
    ctx.close()


def test_predict_leading_dimension(gbt):
    r = np.random.default_rng(4)
    X = r.normal(size=(777, 40)).astype(np.float32)
    trees = ensemble(gbt, [6] * 5, 13, 8, 4)
    ctx = gbt.Context(0)
    Xd = torch.from_numpy(X).cuda()
    inp, _ = gbt.dense_input(Xd)
    inp.n_cols = 13
    out = torch.empty(777, device="cuda")
    arr = (gbt.Tree * 5)(*[t.as_struct() for t in trees])
    gbt._check(gbt.lib().gbt_predict(ctx.h, arr, 5, gbt.C.byref(inp), None, 0.0, out.data_ptr()))
    assert out.cpu().numpy().tobytes() == walk(gbt, trees, X, 0.0).tobytes()
    ctx.close()


def test_wide_rows_cost_what_the_trees_read(gbt):
    """One shallow tree over 1 M x 400 rows reads a few values of each row:
    less than a copy of the rows (staging whole rows took ten copies)."""
    import time
    X = torch.randn(1_000_000, 400, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    trees = ensemble(gbt, [3], 400, 8, 1)
    ctx = gbt.Context(0)
    best = {"copy": 1e9, "predict": 1e9}
    for _ in range(6):
        for what in best:
            torch.cuda.synchronize()
            t = time.perf_counter()
            X.clone() if what == "copy" else gbt.gbt_predict(ctx, trees, 0.0, raw=X)
            torch.cuda.synchronize()
            best[what] = min(best[what], time.perf_counter() - t)
    assert best["predict"] < 3 * best["copy"]
    ctx.close()


def test_first_and_later_calls_of_a_context(gbt):
    """The first 16 calls' trees go up from ordinary memory, later ones from
    pinned memory, and more than 4 MB of them from ordinary memory again."""
    r = np.random.default_rng(8)
    X = r.normal(size=(300, 9)).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    ctx = gbt.Context(0)
    few = ensemble(gbt, [6] * 12, 9, 8, 3)
    more = ensemble(gbt, [8] * 40, 9, 8, 4)
    large = ensemble(gbt, [11], 9, 8, 5) * 180  # 4.4 MB
    for trees in (few, more, large) + (few,) * 13 + (more, few, large, more, few):
        got = gbt.gbt_predict(ctx, trees, 0.5, raw=Xd)
        assert got.cpu().numpy().tobytes() == walk(gbt, trees, X, 0.5).tobytes()
    ctx.close()


def test_first_call_takes_no_pinned_memory(gbt):
    """A fresh context's first call against its next ones: 1.3 times as long;
    with an allocation of pinned memory in it, 2.3 to 2.9."""
    import time
    X = torch.randn(1000, 28, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    trees = ensemble(gbt, [6] * 10, 28, 8, 1)
    warm = gbt.Context(0)
    gbt.gbt_predict(warm, trees, 0.0, raw=X)
    first, later, ctxs = [], [], []
    for _ in range(21):
        ctxs.append(gbt.Context(0))
        torch.cuda.synchronize()
        for k in range(6):
            t = time.perf_counter()
            gbt.gbt_predict(ctxs[-1], trees, 0.0, raw=X)
            (later if k else first).append(time.perf_counter() - t)
    assert np.median(first) < 1.9 * np.median(later)
    for c in ctxs + [warm]:
        c.close()
