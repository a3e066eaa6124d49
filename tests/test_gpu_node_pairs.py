"""PACKED nodes fetched in pairs: forests on both sides of the depths from
which they are (7 levels below the bin tops for busy launches, 8.5 for small
ones), top regions staged whole and in part, features in LDS and in memory,
one walk per lane to four.  Whole numbers: equal to the oracle's."""
import numpy as np
import pytest

import oracle
import paper_1806_07300_amd as fp
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def forest():
    """12 trees grown to purity on random labels: walks of about 16 nodes."""
    rng = np.random.default_rng(2)
    X = rng.random((4000, 9), dtype=np.float32)
    y = rng.integers(0, 3, 4000).astype(np.int32)
    f = synth.train_forest(X, y, n_trees=12, n_classes=3, mtry=3, max_depth=-1, bootstrap=True, seed=8)
    rows = rng.random((22_000, 9), dtype=np.float32)
    rows[::17, ::3] = np.nan
    return f, rows, oracle.predict(f, rows)


@pytest.mark.parametrize("below", [6.5, 7.5, 9.0, 99.0])
@pytest.mark.parametrize("n", [500, 22_000])
@pytest.mark.parametrize("cursors", [1, 2, 4])
def test_both_sides_of_the_depths(forest, below, n, cursors):
    import torch
    f, rows, want = forest
    depth = fp.fp_pack_forest(f, layout=fp.FP_LAYOUT_PACKED, bin_size=5, interleave_depth=3).info["expected_depth"]
    D = max(0, round(depth - 1 - below))
    p = fp.fp_pack_forest(f, layout=fp.FP_LAYOUT_PACKED, bin_size=5, interleave_depth=D)
    fp.fp_packed_upload(p)
    X = torch.from_numpy(rows[:n]).cuda()
    for tune in ({}, {"rows_per_block": 32}, {"rows_per_block": 32, "lds_top_nodes": 7}, {"feature_lds": -1},
                 {"rows_per_block": 16, "block_threads": 256}):
        v, c = fp.fp_predict_tuned(p, dict(tune, cursors=cursors), X)
        torch.cuda.synchronize()
        assert np.array_equal(v.cpu().numpy(), want[0][:n]) and np.array_equal(c.cpu().numpy(), want[1][:n]), tune
    votes = torch.full((n, 3), -7, dtype=torch.int32, device="cuda")
    fp.fp_predict_batched_noalloc([(p, X, votes, None)], cursors=cursors)
    torch.cuda.synchronize()
    assert np.array_equal(votes.cpu().numpy(), want[0][:n])


@pytest.mark.parametrize("cursors", [2, 4, 8])
@pytest.mark.parametrize("n_features,pad", [(8, 0), (9, 3), (10, 0), (40, 4)])
def test_first_and_later_tiles(cursors, n_features, pad):
    """A workgroup's first tile, of which some kernels fetch the first quads ahead, and those after it."""
    import torch
    rng = np.random.default_rng(n_features)
    X = rng.random((900, n_features), dtype=np.float32)
    f = synth.train_forest(X, rng.integers(0, 5, 900).astype(np.int32), n_trees=7, n_classes=5, mtry=3, max_depth=-1,
                           bootstrap=True, seed=6)
    rows = rng.random((9_001, n_features + pad), dtype=np.float32)
    want = oracle.predict(f, np.ascontiguousarray(rows[:, :n_features]))
    Xd = torch.from_numpy(rows).cuda()[:, :n_features]
    p = fp.fp_pack_forest(f, layout=fp.FP_LAYOUT_PACKED, bin_size=3, interleave_depth=3)
    fp.fp_packed_upload(p)
    for tune in ({"rows_per_block": 4}, {"rows_per_block": 7, "block_threads": 64}, {"rows_per_block": 64, "block_threads": 1024}):
        v, c = fp.fp_predict_tuned(p, dict(tune, cursors=cursors), Xd)
        torch.cuda.synchronize()
        assert np.array_equal(v.cpu().numpy(), want[0]) and np.array_equal(c.cpu().numpy(), want[1]), tune
