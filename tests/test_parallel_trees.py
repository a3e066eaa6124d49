"""Validation and node statistics run over a forest's trees on several threads
from 64K nodes on: the same results and the same first error as in order."""
import numpy as np
import pytest

import paper_1806_07300_amd as fp
from handmade import depth3_forest


def forest(n_trees):
    return depth3_forest(n_trees, [[(3 * t + k) % 9 for k in range(7)] for t in range(n_trees)], 4)


@pytest.mark.parametrize("n_trees", [4369, 4370, 9000])  # 65,535 nodes and more
def test_first_faulty_tree_is_reported(n_trees):
    for faults in ([n_trees - 1], [n_trees - 1, 17], [n_trees // 2, n_trees // 2 + 1, n_trees - 3]):
        f = forest(n_trees)
        for t in faults:
            f.left[15 * t + 2] = 99  # out of the tree's range
        with pytest.raises(fp.FPError) as e:
            fp.fp_pack_forest(f, layout=fp.FP_LAYOUT_CLUSTERED)
        assert e.value.code == fp.FP_ECORRUPT
        assert f"tree {min(faults)} node 2:" in str(e.value)


@pytest.mark.gpu
@pytest.mark.parametrize("n_trees", [3, 4369, 4370, 9000])
def test_inferred_counts(n_trees):
    import torch
    f = forest(n_trees)
    X = np.random.default_rng(n_trees).random((257, f.n_features), dtype=np.float32)
    X[::9, 1] = np.nan
    card = fp.fp_infer_cardinality(f, torch.from_numpy(X).cuda())
    want = np.zeros((n_trees, 15), np.int64)
    go = ~(X[:, :] <= np.float32(0.5))  # right
    for t in range(n_trees):
        at = np.zeros(len(X), int)
        for _ in range(3):
            want[t] += np.bincount(at, minlength=15)
            at = 2 * at + 1 + go[np.arange(len(X)), f.feature[15 * t + at]]
        want[t] += np.bincount(at, minlength=15)
    assert np.array_equal(card.reshape(n_trees, 15), want)
