"""Classes taken from a tile's votes, four at a time and the rest one by one:
class counts around multiples of four, many ties (the lowest class wins).
Equal to the oracle's."""
import numpy as np
import pytest

import oracle
import paper_1806_07300_amd as fp
from handmade import depth3_forest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [fp.FP_LAYOUT_PACKED, fp.FP_LAYOUT_COMPACT, fp.FP_LAYOUT_BLOCKED])
@pytest.mark.parametrize("n_classes", [1, 2, 4, 5, 6, 8, 9, 12, 100, 1001])
def test_ties_and_remainders(layout, n_classes):
    import torch
    f = depth3_forest(6, [[(5 * t + k) % 9 for k in range(7)] for t in range(6)], n_classes, 0.3)
    X = np.random.default_rng(n_classes).random((777, f.n_features), dtype=np.float32)
    want = oracle.predict(f, X)
    p = fp.fp_pack_forest(f, layout=layout, bin_size=3, interleave_depth=1)
    fp.fp_packed_upload(p)
    for tune in ({}, {"rows_per_block": 7, "block_threads": 64}):
        v, c = fp.fp_predict_tuned(p, tune, torch.from_numpy(X).cuda())
        torch.cuda.synchronize()
        assert np.array_equal(v.cpu().numpy(), want[0]) and np.array_equal(c.cpu().numpy(), want[1])
