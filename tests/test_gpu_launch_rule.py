"""Launches with some parameters given and the rest left to the rule: groups
that would hold no bin, groups for idle CUs and for wide rows, smaller
workgroups, features in memory, small shares of LDS.  Whole numbers: equal to
the oracle's."""
import numpy as np
import pytest

import oracle
import paper_1806_07300_amd as fp
import synth
from handmade import depth3_forest

pytestmark = pytest.mark.gpu

LAYOUTS = [fp.FP_LAYOUT_PACKED, fp.FP_LAYOUT_COMPACT, fp.FP_LAYOUT_BLOCKED, fp.FP_LAYOUT_CLUSTERED]
TUNES = [{}, {"rows_per_block": 64}, {"rows_per_block": 16, "block_threads": 256}, {"block_threads": 256},
         {"block_threads": 64}, {"cursors": 4}, {"feature_lds": -1}, {"feature_lds": -1, "rows_per_block": 64},
         {"lds_bytes": 40000}, {"lds_bytes": 12000}, {"lds_top_nodes": -1}, {"tree_groups": 8}, {"tree_passes": 4},
         {"tree_groups": 5, "tree_passes": 3}]


@pytest.fixture(scope="module")
def many():
    """520 trees grown to purity on random labels: over 4 MB in every layout."""
    rng = np.random.default_rng(3)
    X = rng.random((3000, 6), dtype=np.float32)
    y = rng.integers(0, 4, 3000).astype(np.int32)
    f = synth.train_forest(X, y, n_trees=520, n_classes=4, mtry=2, max_depth=-1, bootstrap=True, seed=8)
    rows = rng.random((4100, 6), dtype=np.float32)
    rows[::13, 0] = np.nan
    return f, rows, oracle.predict(f, rows)


def check(f, rows, want, layout, bin_size, tunes, sizes):
    import torch
    p = fp.fp_pack_forest(f, layout=layout, bin_size=bin_size, interleave_depth=3)
    fp.fp_packed_upload(p)
    for n in sizes:
        X = torch.from_numpy(rows[:n]).cuda()
        for tune in tunes:
            if tune.get("rows_per_block", 0) * f.n_classes * 4 > 80 << 10:  # the given tile's votes do not fit LDS
                with pytest.raises(fp.FPError) as e:
                    fp.fp_predict_tuned(p, tune, X)
                assert e.value.code == fp.FP_E2BIG
                continue
            v, c = fp.fp_predict_tuned(p, tune, X)
            torch.cuda.synchronize()
            assert np.array_equal(v.cpu().numpy(), want[0][:n]) and np.array_equal(c.cpu().numpy(), want[1][:n]), (n, tune)
    return p


@pytest.mark.parametrize("layout", LAYOUTS)
@pytest.mark.parametrize("bin_size", [16, 58, 31])  # 33, 9 and 17 bins
def test_given_and_automatic_parameters(many, layout, bin_size):
    f, rows, want = many
    p = check(f, rows, want, layout, bin_size, TUNES, (1, 505, 4100))
    assert p.info["bytes"] > 4 << 20


@pytest.mark.parametrize("n_used,n_classes,layout", [(3000, 3, lay) for lay in LAYOUTS] + [
    (u, c, lay) for u, c in ((700, 40), (40, 900)) for lay in LAYOUTS[:3]])  # a clustered block holds 32 classes
def test_wide_rows_and_many_classes(n_used, n_classes, layout):
    T = 530
    f = depth3_forest(T, [[(7 * t + k) % n_used for k in range(7)] for t in range(T)], n_classes, 0.1)
    rows = np.random.default_rng(1).random((600, f.n_features), dtype=np.float32)
    check(f, rows, oracle.predict(f, rows), layout, 16, [t for t in TUNES if t.get("lds_bytes") != 12000], (3, 600))


@pytest.mark.parametrize("layout", [fp.FP_LAYOUT_BLOCKED, fp.FP_LAYOUT_CLUSTERED])
def test_small_tiles_on_long_walks(layout):
    """Over 128 MB of long walks: tiles of fewer than 224 rows refill earlier, passes of fewer bytes and larger tiles do not."""
    rng = np.random.default_rng(12)
    X = rng.random((600_000, 6), dtype=np.float32)
    y = rng.integers(0, 2, len(X)).astype(np.int32)
    f = synth.train_forest(X, y, n_trees=4, n_classes=2, mtry=2, max_depth=-1, bootstrap=True, seed=9)
    f = synth.concat_forests([f] * 24)
    rows = rng.random((1100, 6), dtype=np.float32)
    p = check(f, rows, oracle.predict(f, rows), layout, 16,
              [{"rows_per_block": r, "block_threads": t, "tree_passes": passes}
               for r, t, passes in ((1, 512, 1), (96, 512, 1), (223, 1024, 1), (224, 1024, 1), (128, 512, 4), (0, 0, 1))], (1, 1100))
    assert p.info["bytes"] > 140 << 20 and p.info["expected_depth"] > 21.5, p.info
