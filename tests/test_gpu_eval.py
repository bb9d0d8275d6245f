"""The fused reduction and evaluation of a level in each of its forms (a
block per feature and node, a wave per few features and node, a wave for a
node and its sibling) and feature widths, against the CPU oracle: equal
trees and margins, bit for bit."""
import numpy as np
import pytest

from oracle import oracle as orc
from tests.gpu_helpers import node_diff, oracle_quantize, same_bits

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# more rows than the one-kernel small levels take; the last three reach 64
# nodes of 29 feature blocks
@pytest.mark.parametrize("m,max_bin,depth", [
    (1, 2, 3), (5, 17, 5), (37, 64, 6), (37, 65, 6), (9, 128, 6), (9, 129, 6), (3, 256, 7),
    (460, 64, 8), (230, 128, 8), (115, 256, 8)])
def test_evaluation_forms(m, max_bin, depth):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2005_09148_amd import gbt
    n = 33_001
    r = np.random.default_rng(m + max_bin)
    X = r.normal(size=(n, m)).astype(np.float32)
    X[:, 0] = np.floor(2 * X[:, 0])
    X[r.random(X.shape) < 0.1] = np.nan
    y = np.nan_to_num(X).sum(1) + r.normal(size=n).astype(np.float32)
    y = (y > 0).astype(np.float32)
    _, b, _, _ = oracle_quantize(X, max_bin)
    otrees, omargin = orc.train(b, y, orc.Params(loss=0, max_depth=depth, eta=0.3), 2, 0.0)[:2]
    ctx = gbt.Context(0)
    mx = gbt.gbt_quantize(ctx, X, max_bin=max_bin)
    margin = torch.zeros(n, device="cuda")
    trees = gbt.gbt_train_trees(ctx, mx, torch.from_numpy(y).cuda(), margin,
                                gbt.make_train_params(loss=0, max_depth=depth, eta=0.3), 2)
    for t, (a, o) in enumerate(zip(trees, otrees)):
        d = node_diff(a.nodes, o.nodes)
        assert d is None, f"tree {t} node {d[0]}: {d[1]}, oracle {d[2]}"
    assert same_bits(margin.cpu().numpy(), omargin)
    ctx.close()
