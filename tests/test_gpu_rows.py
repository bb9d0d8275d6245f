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
