"""Trees that every row trains, whose fixed-point pairs come straight from
margins and labels: arrays at any 4-byte alignment and odd row counts give
the same trees and margins."""
import numpy as np
import pytest

from paper_2005_09148_amd import datagen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,loss", [(1, 1), (2, 0), (513, 0), (5001, 1)])
@pytest.mark.parametrize("off", [(1, 0), (0, 1), (1, 1)])
def test_unaligned_rows(n, loss, off):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_09148_amd import gbt
    d = datagen.config1(n=n)
    ctx = gbt.Context(0)
    mx = gbt.gbt_quantize(ctx, d["X"], max_bin=32)
    P = gbt.make_train_params(loss=loss, max_depth=4, eta=0.3)
    outs = []
    for a, b in ((0, 0), off):
        label = torch.zeros(n + 1, device="cuda")[a:a + n]
        margin = torch.full((n + 1,), 0.1, device="cuda")[b:b + n]
        label.copy_(torch.from_numpy(d["y"]))
        trees = gbt.gbt_train_trees(ctx, mx, label, margin, P, 3)
        outs.append([t.nodes.tobytes() for t in trees] + [margin.cpu().numpy().tobytes()])
    assert outs[0] == outs[1]
    ctx.close()


@pytest.mark.parametrize("n,m,max_bin,depth,f", [
    (16_384, 5, 256, 5, 1.0), (16_385, 5, 256, 5, 1.0), (32_768, 3, 64, 6, 1.0), (32_769, 3, 64, 6, 1.0),
    (40_000, 29, 256, 4, 0.4), (1025, 130, 32, 4, 1.0), (3000, 70, 17, 8, 1.0), (255, 2, 2, 3, 1.0),
    (20_000, 4, 300, 4, 0.5)])
@pytest.mark.parametrize("loss", [0, 1])
def test_small_levels(n, m, max_bin, depth, f, loss):
    """The one-kernel histogram and evaluation of levels of few rows around its
    limits (rows, blocks of 1024 or 256 threads, above 128 features, above
    256 bins), against the chunked passes with the histogram kernel forced."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_09148_amd import gbt
    r = np.random.default_rng(n + m)
    X = r.normal(size=(n, m)).astype(np.float32)
    X[r.random(X.shape) < 0.1] = np.nan
    X[:, -1] = np.floor(X[:, -1])
    y = torch.from_numpy((np.nan_to_num(X[:, 0]) + r.normal(size=n) > 0).astype(np.float32)).cuda()
    ctx = gbt.Context(0)
    mx = gbt.gbt_quantize(ctx, X, max_bin=max_bin)
    P = gbt.make_train_params(loss=loss, max_depth=depth, eta=0.3, f=f)
    outs = []
    for kernel in (ctx.HIST_AUTO, ctx.HIST_PLAIN):
        ctx.set_hist_kernel(kernel)
        margin = torch.zeros(n, device="cuda")
        trees = gbt.gbt_train_trees(ctx, mx, y, margin, P, 2)
        stats = [(t.stats.hist_updates, t.stats.hist_rows, t.stats.hist_bytes, t.stats.hist_launches,
                  t.stats.hist_cols) for t in trees]
        outs.append([t.nodes.tobytes() for t in trees] + [margin.cpu().numpy().tobytes(), stats])
    assert outs[0] == outs[1]
    ctx.close()


@pytest.mark.parametrize("n,m,max_bin,depth", [(4096, 512, 16, 4), (4097, 512, 16, 4), (300, 512, 256, 3),
                                               (300, 513, 256, 3), (900, 200, 16, 9), (700, 60, 40, 11)])
def test_wide_small_trees_match_oracle(n, m, max_bin, depth):
    """Trees of few rows on both sides of the column and cell limits of the
    one-kernel levels, and deep ones whose lower levels pass the limit on
    their blocks, bit for bit against the CPU oracle."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle as orc
    from paper_2005_09148_amd import gbt
    from tests.gpu_helpers import node_diff, oracle_quantize
    r = np.random.default_rng(n + m)
    X = r.normal(size=(n, m)).astype(np.float32)
    X[r.random(X.shape) < 0.05] = np.nan
    y = (np.nan_to_num(X[:, 1]) + r.normal(size=n) > 0).astype(np.float32)
    ctx = gbt.Context(0)
    trees, margin = gbt.train(ctx, gbt.gbt_quantize(ctx, X, max_bin=max_bin), torch.from_numpy(y).cuda(),
                              gbt.make_train_params(loss=1, max_depth=depth, eta=0.3), 2, 0.0)
    _, b, _, _ = oracle_quantize(X, max_bin)
    want, want_margin = orc.train(b, y, orc.Params(loss=1, max_depth=depth, eta=0.3), 2, 0.0)
    for g, o in zip(trees, want):
        assert node_diff(g.nodes, o.nodes) is None
    assert margin.cpu().numpy().tobytes() == want_margin.tobytes()
    ctx.close()


@pytest.mark.parametrize("n,m,depth", [(16_384, 2000, 6), (4000, 500, 12)])
def test_wide_small_trees_take_no_longer(n, m, depth):
    """The chosen path takes no longer than the chunked passes (one-kernel
    levels took 1.9 times as long without a bound on the columns, 1.4 times
    without one on a level's blocks; 1.2 allows for the spread of one run)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import time
    from paper_2005_09148_amd import gbt
    X = torch.randn(n, m, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    y = (X[:, 0] > 0).float()
    ctx = gbt.Context(0)
    mx = gbt.gbt_quantize(ctx, X, max_bin=32)
    P = gbt.make_train_params(loss=0, max_depth=depth, eta=0.1)
    best = {}
    for _ in range(6):
        for kernel in (ctx.HIST_AUTO, ctx.HIST_PLAIN):
            ctx.set_hist_kernel(kernel)
            margin = torch.zeros(n, device="cuda")
            torch.cuda.synchronize()
            t = time.perf_counter()
            gbt.gbt_train_trees(ctx, mx, y, margin, P, 3)
            best[kernel] = min(best.get(kernel, 1e9), time.perf_counter() - t)
    assert best[ctx.HIST_AUTO] < 1.2 * best[ctx.HIST_PLAIN]
    ctx.close()


@pytest.mark.parametrize("n,forced,kind", [(10_000, False, 3), (10_000, True, 1), (20_000, False, 1)])
def test_stats_name_the_root_kernel(n, forced, kind):
    """The stats of a tree whose root level is one kernel (HIST_LEVEL), of
    the forced plain kernel and of a tree above the root's row limit."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_09148_amd import gbt
    X = torch.randn(n, 20, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    ctx = gbt.Context(0)
    ctx.set_timing(1)
    if forced:
        ctx.set_hist_kernel(ctx.HIST_PLAIN)
    mx = gbt.gbt_quantize(ctx, X)
    st = gbt.gbt_train_tree(ctx, mx, (X[:, 0] > 0).float(), torch.zeros(n, device="cuda"),
                            gbt.make_train_params(loss=0, max_depth=5)).stats
    assert st.hist_kernel == kind and st.hist_launches == 5
    assert 0 < st.ms_hist < st.ms_total and st.ms_split == 0
    ctx.close()


@pytest.mark.parametrize("n,m,density", [(1500, 3000, 0.01), (14_000, 1500, 0.01), (22_000, 1000, 0.01),
                                         (40_000, 600, 0.02)])
def test_sparse_passes_of_few_items_match_oracle(n, m, density):
    """Sparse passes with fewer work items than XCDs (2048 rows each), with
    more that are short of a multiple of eight or nearly one, and of several
    kinds in one tree, over several feature groups."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle as orc
    from paper_2005_09148_amd import gbt
    from tests.gpu_helpers import node_diff, oracle_quantize
    r = np.random.default_rng(n + m)
    lens = r.binomial(m, density, n)
    d = {"kind": "csr", "indptr": np.concatenate([[0], np.cumsum(lens)]).astype(np.int64),
         "indices": np.concatenate([np.sort(r.choice(m, k, replace=False)) for k in lens]).astype(np.int32), "m": m}
    d["values"] = np.exp(r.normal(size=len(d["indices"]))).astype(np.float32)
    y = (r.random(n) < 0.5).astype(np.float32)
    ctx = gbt.Context(0)
    mx = gbt.gbt_quantize(ctx, d, max_bin=32)
    trees, margin = gbt.train(ctx, mx, torch.from_numpy(y).cuda(), gbt.make_train_params(loss=0, max_depth=4, eta=0.3),
                              2, 0.0)
    _, b, _, _ = oracle_quantize(d, 32)
    want, want_margin = orc.train(b, y, orc.Params(loss=0, max_depth=4, eta=0.3), 2, 0.0)
    for g, o in zip(trees, want):
        assert node_diff(g.nodes, o.nodes) is None
    assert margin.cpu().numpy().tobytes() == want_margin.tobytes()
    ctx.close()
