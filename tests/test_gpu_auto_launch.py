"""The launch that fp_predict picks when every parameter is left at its
default: batch sizes and forests on each side of the lines the rule draws
(a tile per CU, 16,384 walks and 512 or 256 rows a tile, 512 trees, 2^18
walks, 4 MB of nodes, the LDS budget), and explicit tiles spread over full rounds.  Whole numbers: equal
to the CPU checker's."""
import numpy as np
import pytest

import oracle
import paper_1806_07300_amd as fp
import synth
from handmade import depth3_forest

pytestmark = pytest.mark.gpu


def check(f, n, layout, tune=None, bin_size=16):
    import torch
    X = np.random.default_rng(n).random((n, f.n_features), dtype=np.float32)
    X[::13, 0] = np.nan
    want = oracle.predict(f, X)
    p = fp.fp_pack_forest(f, layout=layout, bin_size=bin_size, interleave_depth=3)
    fp.fp_packed_upload(p)
    if tune:
        fp.fp_packed_set_tune(p, tune)
    votes, cls = fp.fp_predict(p, torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(votes.cpu().numpy(), want[0])
    assert np.array_equal(cls.cpu().numpy(), want[1])


def forest(n_trees, n_used, n_classes=5, thr=0.1):
    return depth3_forest(n_trees, [[(7 * t + k) % n_used for k in range(7)] for t in range(n_trees)], n_classes, thr)


@pytest.mark.parametrize("layout", [fp.FP_LAYOUT_PACKED, fp.FP_LAYOUT_COMPACT, fp.FP_LAYOUT_BLOCKED,
                                    fp.FP_LAYOUT_CLUSTERED])
@pytest.mark.parametrize("n_trees,n_used,n", [
    (3, 7, 1), (3, 7, 255), (3, 7, 256), (3, 7, 257), (9, 20, 131073), (40, 20, 200_001),
    (511, 30, 514), (512, 30, 511), (512, 30, 512), (512, 30, 513), (1100, 30, 5000), (1100, 30, 3),
    (200, 700, 20_001), (130, 1000, 4000),
])
def test_default_launch(layout, n_trees, n_used, n):
    check(forest(n_trees, n_used), n, layout)


@pytest.fixture(scope="module")
def noise_forest():
    """256 trees grown to purity on random labels: over 4 MB of PACKED nodes."""
    rng = np.random.default_rng(3)
    X = rng.random((5000, 6), dtype=np.float32)
    y = rng.integers(0, 4, 5000).astype(np.int32)
    f = synth.train_forest(X, y, n_trees=256, n_classes=4, mtry=2, max_depth=-1, bootstrap=True, seed=8)
    assert f.n_internal() * 16 > 4 << 20
    return f


@pytest.mark.parametrize("layout", [fp.FP_LAYOUT_PACKED, fp.FP_LAYOUT_COMPACT])
@pytest.mark.parametrize("n", [1023, 1024, 3001])
def test_node_layouts_larger_than_an_l2(noise_forest, layout, n):
    """2^18 walks from 1,024 rows on."""
    check(noise_forest, n, layout)


@pytest.mark.parametrize("cursors", [1, 2, 4, 8])
@pytest.mark.parametrize("D", [0, 1, 3])
def test_packed_runs_to_the_last_node(cursors, D):
    """Two nodes are loaded at a time: the last one of the section, on its own
    or as a run's second, with top nodes in LDS and without."""
    f = forest(5, 7)
    for top in (-1, 2, 0):
        check(f, 333, fp.FP_LAYOUT_PACKED, {"cursors": cursors, "lds_top_nodes": top}, bin_size=5)
    import torch
    X = np.random.default_rng(1).random((64, f.n_features), dtype=np.float32)
    want = oracle.predict(f, X)
    p = fp.fp_pack_forest(f, layout=fp.FP_LAYOUT_PACKED, bin_size=2, interleave_depth=D)
    fp.fp_packed_upload(p)
    v, _ = fp.fp_predict_tuned(p, {"cursors": cursors, "lds_top_nodes": -1}, torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    assert np.array_equal(v.cpu().numpy(), want[0])


@pytest.mark.parametrize("rows,n", [(768, 100_000), (768, 262_145), (33, 40_001), (4096, 2_000_003)])
def test_explicit_tiles_over_full_rounds(rows, n):
    check(forest(12, 9), n, fp.FP_LAYOUT_CLUSTERED,
          {"rows_per_block": rows, "block_threads": 1024, "lds_bytes": 163840, "tree_passes": 2}, bin_size=4)


def test_many_classes_shrink_the_automatic_tile():
    """600 classes: the vote counters of a 512-row tile would not fit LDS."""
    check(forest(100, 9, n_classes=600), 150_000, fp.FP_LAYOUT_BLOCKED)
