"""The launch search on small and ordinary batches of every layout: it starts
from the launch that fp_predict makes without a record, and goes down to tiles
of one row.  What it records predicts as the oracle does."""
import numpy as np
import pytest

import oracle
import paper_1806_07300_amd as fp
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [fp.FP_LAYOUT_PACKED, fp.FP_LAYOUT_COMPACT, fp.FP_LAYOUT_BLOCKED, fp.FP_LAYOUT_CLUSTERED])
@pytest.mark.parametrize("threads,cursors", [(0, 0), (256, 2), (1024, 4)])
def test_records_of_small_batches(layout, threads, cursors):
    import torch
    Xt, y = synth.gaussian_mixture(4000, 14, 3, seed=71)
    f = synth.train_forest(Xt, y, n_trees=90, n_classes=3, mtry=3, max_depth=12, bootstrap=True, seed=72)
    X, _ = synth.gaussian_mixture(5000, 14, 3, seed=73)
    want = oracle.predict(f, X)
    p = fp.fp_pack_forest(f, layout=layout, bin_size=16, interleave_depth=3)
    fp.fp_packed_upload(p)
    for n in (1, 300, 5000):
        Xd = torch.from_numpy(X[:n]).cuda()
        t = fp.fp_tune_launch(p, Xd, block_threads=threads, cursors=cursors)
        assert t["rows_per_block"] > 0 and t["tree_groups"] > 0 and t["refill_lanes"] > 0
        assert t["block_threads"] == threads or (threads == 0 and t["block_threads"] > 0)
        v, c = fp.fp_predict_tuned(p, t, Xd)
        torch.cuda.synchronize()
        assert np.array_equal(v.cpu().numpy(), want[0][:n]) and np.array_equal(c.cpu().numpy(), want[1][:n]), (n, t)
