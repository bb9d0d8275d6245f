"""The device selection of the quantile cuts at the edges of its branches
(segments sorted whole by 256 or 1024 threads, split and gathered segments,
buckets above one block's sort), bit for bit against the CPU oracle."""
import numpy as np
import pytest

from tests.gpu_helpers import oracle_quantize, same_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gbt():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_09148_amd import gbt as g
    return g


def columns(n, seed):
    """One column per distribution the selection can meet."""
    r = np.random.default_rng(seed)
    normal = r.normal(size=n)
    zeros = np.where(r.random(n) < 0.7, 0.0, normal)  # one heavy value
    huge = np.where(r.random(n) < 0.5, 1.0, -1.0) * 10.0 ** r.uniform(-44, 38, n)  # subnormals to near the largest
    cols = [normal, r.random(n), r.integers(0, 5, n), zeros, np.full(n, -2.5), np.exp(4 * normal), huge,
            np.arange(n) % 1000, 3e38 * np.where(np.arange(n) % 2, 1, -1), np.where(np.arange(n) % 97, np.nan, normal),
            np.full(n, np.nan), np.where(r.random(n) < 0.999, 1e-3 * normal, 1e30 * normal)]
    with np.errstate(over="ignore"):
        X = np.stack(cols, 1).astype(np.float32)
    X[np.isinf(X)] = np.float32(3e38)
    X[r.random(n) < 0.01, 0] = np.float32(-0.0)
    return X


@pytest.mark.parametrize("n,max_bin", [(1, 256), (2, 2), (255, 16), (4096, 256), (4097, 256), (16384, 64),
                                       (16385, 256), (16385, 2560), (65537, 3), (300_001, 256), (300_001, 2560)])
def test_cuts_match_oracle(gbt, n, max_bin):
    X = columns(n, n + max_bin)
    cuts, _, _, page = oracle_quantize(X, max_bin)
    ctx = gbt.Context(0)
    mx = gbt.gbt_quantize(ctx, torch.from_numpy(X).cuda(), max_bin=max_bin)
    cp, cv = mx.cuts()
    assert same_bits(cp, cuts.cut_ptr) and same_bits(cv, cuts.cut_values)
    assert same_bits(mx.page(0), page)
    ctx.close()


@pytest.mark.parametrize("n,m,max_bin,ld,page_rows", [
    (1, 1, 2, 1, 0), (255, 15, 256, 15, 0), (257, 17, 256, 19, 0), (511, 16, 300, 16, 200), (513, 33, 1100, 40, 0),
    (1025, 31, 2560, 31, 512), (3000, 32, 2, 32, 0), (700, 100, 64, 101, 513), (2049, 47, 5, 48, 0)])
def test_pages_match_oracle(gbt, n, m, max_bin, ld, page_rows):
    """Edges of the encoder's tiles (rows, feature chunks, cuts per chunk),
    a leading dimension above the columns, pages cut within a tile."""
    r = np.random.default_rng(n + m)
    X = r.normal(size=(n, ld)).astype(np.float32)
    X[r.random(X.shape) < 0.1] = np.nan
    X[:, 0] = np.floor(X[:, 0])
    _, _, _, page = oracle_quantize(np.ascontiguousarray(X[:, :m]), max_bin)
    ctx = gbt.Context(0)
    Xd = torch.from_numpy(X).cuda()
    q = gbt.Quantizer(ctx, m, n, max_bin=max_bin, page_rows=page_rows)
    inp, _ = gbt.dense_input(Xd)
    inp.n_cols = m
    lib = gbt.lib()
    gbt._check(lib.gbt_quantize_sketch_batch(q.h, gbt.C.byref(inp)))
    q.finalize()
    gbt._check(lib.gbt_quantize_encode_batch(q.h, gbt.C.byref(inp)))
    assert same_bits(q.end().pages(), page)
    ctx.close()


def sample_places(n, feature):
    """Places of the selection's sample of a segment of n keys (cuts.hip):
    one scrambled place in each of 16384 equal strata."""
    i = np.arange(16384, dtype=np.uint64)
    lo, hi = i * n // 16384, (i + 1) * n // 16384
    h = (i * 0x9e3779b9 + feature) & 0xffffffff
    for shift, mul in ((16, 0x7feb352d), (15, 0x846ca68b), (16, 1)):
        h = (h ^ (h >> np.uint64(shift))) * np.uint64(mul) & np.uint64(0xffffffff)
    return (lo + h % (hi - lo)).astype(np.int64)


def rank_buckets(x, max_bin):
    """Keys and ranks of the selection's buckets that hold a rank, for a
    column x of positive values of which none is frequent in its sample."""
    q = np.sort(x[sample_places(len(x), 0)])[np.arange(1, 4096) * 4]
    assert (np.diff(q) > 0).all()
    v = np.sort(x)
    ranks = (np.arange(1, max_bin, dtype=np.int64) * len(x) + max_bin - 1) // max_bin - 1
    ends = np.concatenate([np.searchsorted(v, q, side="right"), [len(x)]])
    holds = np.searchsorted(ends, np.concatenate([ranks, [len(x) - 1]]), side="right")
    at, per = np.unique(holds, return_counts=True)
    return np.diff(np.concatenate([[0], ends]))[at], per, np.unique(v[ranks])


def test_uneven_buckets(gbt):
    """Every size of bucket: 20,000 close keys at places that are not in the
    sample share a bucket with several ranks (searched digit by digit: more
    than one block sorts), others hold up to 1024 keys and up to 4096."""
    n, bins = 4_000_000, 1024
    r = np.random.default_rng(3)
    x = r.integers(1, 16_000_000, n)
    x[(x >= 9_000_000) & (x < 9_040_000)] -= 5_000_000
    free = np.setdiff1d(np.arange(n), sample_places(n, 0))
    x[r.choice(free, 20_000, replace=False)] = 9_010_000 + r.permutation(20_000)
    x = x.astype(np.float32)
    keys, ranks, cuts = rank_buckets(x, bins)
    assert (keys <= 1024).any() and ((keys > 1024) & (keys <= 4096)).any()
    assert (ranks[keys > 4096] > 2).any()
    ctx = gbt.Context(0)
    mx = gbt.gbt_quantize(ctx, torch.from_numpy(x[:, None]).cuda(), max_bin=bins)
    assert same_bits(mx.cuts()[1], cuts[cuts < x.max()])
    ctx.close()


@pytest.mark.parametrize("max_bin", [16, 256])
def test_cuts_without_room_for_the_selection(gbt, max_bin):
    """A budget that holds the keys but not the selection's workspace."""
    n = 60_000
    X = columns(n, 5)
    m = X.shape[1]
    cuts, _, _, page = oracle_quantize(X, max_bin)
    ctx = gbt.Context(0, budget_bytes=n * m * 4 + 500_000)
    q = gbt.Quantizer(ctx, m, n, max_bin=max_bin, page_home=gbt.HOME_PINNED_HOST)
    q.sketch(torch.from_numpy(X).cuda())
    q.finalize()
    for lo in range(0, n, 7001):
        q.encode(torch.from_numpy(X[lo:lo + 7001]).cuda())
    mx = q.end()
    cp, cv = mx.cuts()
    assert same_bits(cp, cuts.cut_ptr) and same_bits(cv, cuts.cut_values)
    assert same_bits(mx.pages(), page)
    ctx.close()


def test_kept_blocks(gbt):
    """Large blocks that a context keeps and hands out again: the pages of
    matrices alive meanwhile stay as a context with a budget (which keeps
    none) makes them, and the bytes held are the same."""
    plain = gbt.Context(0, budget_bytes=64 << 30)
    ctx = gbt.Context(0)
    g = torch.Generator(device="cuda").manual_seed(9)
    kept, want = [], []
    for n in (2_500_000, 2_300_000, 3_000_000, 2_499_999):
        X = torch.randn(n, 28, generator=g, device="cuda")
        mx = gbt.gbt_quantize(ctx, X)
        if n != 2_300_000:
            kept.append(mx)
            ref = gbt.gbt_quantize(plain, X)
            want.append(ref.page(0))
            assert same_bits(ref.cuts()[1], mx.cuts()[1])
            ref.free()
        else:
            mx.free()
    for mx, page in zip(kept, want):
        assert same_bits(mx.page(0), page)
        mx.free()
    assert ctx.memory()[0] == plain.memory()[0]
    ctx.close()
    plain.close()


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_kept_blocks_make_room_for_other_contexts(gbt):
    """An allocation that fails in one context returns the blocks that the
    others keep."""
    X = torch.randn(4_000_000, 28, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    ctx, other = gbt.Context(0), gbt.Context(0, budget_bytes=1 << 50)
    gbt.gbt_quantize(ctx, X).free()
    kept = free_bytes()
    with pytest.raises(gbt.GbtError) as err:  # 1 TiB of keys: more than the card holds
        gbt.Quantizer(other, 64, 1 << 32, sketch_max_rows=1 << 40)
    assert err.value.code == gbt.GBT_E_OOM
    assert free_bytes() - kept >= 4_000_000 * 28 * 4
    cuts = gbt.gbt_quantize(ctx, X).cuts()[1]  # the context goes on
    assert same_bits(cuts, gbt.gbt_quantize(other, X).cuts()[1])
    ctx.close()
    other.close()


def test_kept_blocks_are_bounded_over_contexts(gbt):
    X = torch.randn(12_000_000, 28, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    before = free_bytes()
    ctxs = [gbt.Context(0) for _ in range(4)]
    for ctx in ctxs:  # 1.3 GB of keys and more each
        gbt.gbt_quantize(ctx, X).free()
        gbt.gbt_quantize(ctx, X[:len(X) // (1 + ctxs.index(ctx))]).free()  # of several sizes
    held = before - free_bytes()
    assert held < (4 << 30) + (256 << 20)
    for ctx in ctxs:  # the contexts share the kept blocks
        gbt.gbt_quantize(ctx, X).free()
    assert before - free_bytes() < held + (64 << 20)
    for ctx in ctxs:
        ctx.close()
    assert before - free_bytes() < 256 << 20


def test_kept_blocks_between_threads_and_streams(gbt):
    """Contexts on streams of their own, used by threads at the same time,
    hand large blocks to one another: every page stays as one context alone
    makes it."""
    import threading
    sizes = (2_700_000, 3_000_000, 2_500_000)
    g = torch.Generator(device="cuda").manual_seed(11)
    data = [torch.randn(n, 28, generator=g, device="cuda") for n in sizes]
    alone = gbt.Context(0, budget_bytes=64 << 30)  # keeps no blocks
    want = []
    for X in data:
        mx = gbt.gbt_quantize(alone, X)
        want.append((mx.cuts()[1].tobytes(), mx.page(0).tobytes()))
        mx.free()
    torch.cuda.synchronize()
    wrong, errors = [], []

    def work(k):
        try:
            ctx = gbt.Context(0, stream=torch.cuda.Stream())
            for i in range(5):
                mx = gbt.gbt_quantize(ctx, data[(k + i) % 3])
                if (mx.cuts()[1].tobytes(), mx.page(0).tobytes()) != want[(k + i) % 3]:
                    wrong.append((k, i))
                mx.free()
            ctx.close()
        except Exception as e:  # shown below: a thread's exception would pass unseen
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors and not wrong
    alone.close()


def csr_rows(n, m, density, seed, nan=0.0, empty=0.0):
    r = np.random.default_rng(seed)
    lens = np.minimum(r.binomial(m, density, n), m)
    lens[r.random(n) < empty] = 0
    cols = [np.sort(r.choice(m, k, replace=False)) for k in lens]
    indptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    idx = np.concatenate(cols + [np.zeros(0, np.int64)]).astype(np.int32)
    val = np.exp(r.normal(size=len(idx))).astype(np.float32)
    val[r.random(len(val)) < nan] = np.nan
    return {"kind": "csr", "indptr": indptr, "indices": idx, "values": val, "m": m}


@pytest.mark.parametrize("n,m,density,nan,empty,max_rows,device", [
    (1, 3, 1.0, 0.0, 0.0, 0, True), (255, 20, 0.3, 0.1, 0.3, 0, True), (513, 7, 0.9, 0.5, 0.1, 0, False),
    (700, 2000, 0.6, 0.02, 0.05, 0, True), (300, 40, 0.0, 0.0, 0.0, 0, True), (5003, 30, 0.2, 0.1, 0.2, 1000, True),
    (400, 20_000, 0.003, 0.1, 0.1, 0, True), (60_001, 12, 0.7, 0.0, 0.0, 0, True)])
def test_csr_matches_oracle(gbt, n, m, density, nan, empty, max_rows, device):
    """Edges of the CSR kernels: ragged and empty rows, missing values stored,
    rows past the LDS tile, skipped sketch rows, more features than the
    grouping's LDS counters."""
    d = csr_rows(n, m, density, n + m, nan, empty)
    cuts, _, _, page = oracle_quantize(d, 16, max_rows or 1 << 24)
    ctx = gbt.Context(0)
    dd = dict(d, **{k: torch.from_numpy(d[k]).cuda() for k in ("indptr", "indices", "values")}) if device else d
    mx = gbt.gbt_quantize(ctx, dd, max_bin=16, sketch_max_rows=max_rows)
    cp, cv = mx.cuts()
    assert same_bits(cp, cuts.cut_ptr) and same_bits(cv, cuts.cut_values)
    assert same_bits(mx.page(0), page)
    ctx.close()


def test_csr_blocks_of_fewer_rows(gbt):
    """Above 2^22 columns a block takes fewer than 256 rows (here 107)."""
    n, m = 700, 10_000_000
    r = np.random.default_rng(6)
    lens = r.integers(0, 60, n)
    d = {"kind": "csr", "indptr": np.concatenate([[0], np.cumsum(lens)]).astype(np.int64), "m": m,
         "indices": np.concatenate([np.sort(r.choice(10_000_000 // 50, k, replace=False) * 50) for k in lens])}
    d["indices"] = d["indices"].astype(np.int32)
    d["values"] = r.normal(size=len(d["indices"])).astype(np.float32)
    d["values"][r.random(len(d["values"])) < 0.1] = np.nan
    cuts, _, _, page = oracle_quantize(d, 2)
    ctx = gbt.Context(0)
    mx = gbt.gbt_quantize(ctx, d, max_bin=2)
    cp, cv = mx.cuts()
    assert same_bits(cp, cuts.cut_ptr) and same_bits(cv, cuts.cut_values)
    assert same_bits(mx.page(0), page)
    ctx.close()


def test_csr_without_room_for_the_count_tables(gbt):
    """A budget that holds the pairs, the grouped keys and 8 bytes per
    feature, but not the grouping's count tables (98 blocks x 2000 features)."""
    d = csr_rows(20_000, 2000, 0.01, 8)
    m, nk = 2000, len(d["values"])
    cuts, _, _, page = oracle_quantize(d, 16)

    def sketched(budget):
        ctx = gbt.Context(0, budget_bytes=budget)
        q = gbt.Quantizer(ctx, m, 20_000, max_bin=16, kind=gbt.INPUT_CSR, page_home=gbt.HOME_PINNED_HOST)
        q.sketch(d)
        return ctx, q

    ctx, q = sketched(1 << 30)
    held = ctx.memory()[0]
    ctx.close()
    # 98 x 2000 counts are 784 kB; the selection of short segments takes 210 kB
    ctx, q = sketched(held + 4 * nk + 400_000)
    q.finalize()
    q.encode(d)
    mx = q.end()
    cp, cv = mx.cuts()
    assert same_bits(cp, cuts.cut_ptr) and same_bits(cv, cuts.cut_values)
    assert same_bits(mx.pages(), page)
    ctx.close()


@pytest.mark.parametrize("what", ["equal", "descending", "negative", "large", "indptr"])
def test_csr_refuses_bad_indices(gbt, what):
    d = csr_rows(600, 30, 0.4, 1)
    row = int(np.flatnonzero(np.diff(d["indptr"]) >= 3)[-1])
    e = int(d["indptr"][row])
    if what == "equal":
        d["indices"][e + 1] = d["indices"][e]
    elif what == "descending":
        d["indices"][e:e + 2] = d["indices"][e:e + 2][::-1]
    elif what == "negative":
        d["indices"][e] = -1
    elif what == "large":
        d["indices"][int(d["indptr"][row + 1]) - 1] = 30
    else:
        d["indptr"][row] = d["indptr"][row + 1] + 1
    ctx = gbt.Context(0)
    with pytest.raises(gbt.GbtError) as err:
        gbt.gbt_quantize(ctx, d, max_bin=16)
    assert err.value.code == gbt.GBT_E_INVALID
    ctx.close()


def test_more_keys_than_31_bits(gbt):
    """Ranks above 2^31 of one feature's keys: the values are i mod 1000, so
    every rank's value is known."""
    n, bins = (1 << 31) + 1001, 8
    X = torch.arange(1000, dtype=torch.float32, device="cuda").repeat(n // 1000 + 1)[:n, None]
    ctx = gbt.Context(0)
    mx = gbt.gbt_quantize(ctx, X, max_bin=bins, sketch_max_rows=n)
    counts = np.full(1000, n // 1000, np.int64)
    counts[:n % 1000] += 1
    ranks = (np.arange(1, bins, dtype=np.int64) * n + bins - 1) // bins - 1
    want = np.searchsorted(np.cumsum(counts), ranks, side="right").astype(np.float32)
    assert np.array_equal(mx.cuts()[1], np.unique(want))
    mx.free()
    ctx.close()
