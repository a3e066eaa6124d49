"""The walk form that fp_packed_upload gives blocks on the device: every form
and each side of the limits that choose it (classes, used features, fp16
thresholds), block counts around the chunks of its in-place conversion, and
the two properties of a packed buffer it relies on, which the verifier checks.
Votes are whole numbers: they equal the CPU checker's exactly."""
import numpy as np
import pytest

import oracle
import paper_1806_07300_amd as fp
import synth
from handmade import depth3_forest
from packed_format import decode, reseal


def feats(n_used, n_trees):
    return [[(7 * t + k) % n_used for k in range(7)] for t in range(n_trees)]


def rows_for(f, n, seed):
    X = np.random.default_rng(seed).random((n, f.n_features), dtype=np.float32)
    X[::17, ::3] = np.nan
    X[5::19, 1::4] = np.inf
    X[7::23, ::5] = -np.inf
    X[3::11] = np.where(X[3::11] < 0.3, np.float32(0.5), X[3::11])  # ties with the 0.5 thresholds
    return X


def gpu_votes(p, X, tune=None):
    import torch
    v, c = fp.fp_predict(p, torch.from_numpy(X).cuda()) if tune is None else \
        fp.fp_predict_tuned(p, tune, torch.from_numpy(X).cuda())
    torch.cuda.synchronize()
    return v.cpu().numpy(), c.cpu().numpy()


# (layout, used features, classes, threshold): 0.5 is an fp16 value, 0.1 is not
LIMITS = [
    ("CLUSTERED", 512, 16, 0.5), ("CLUSTERED", 40, 17, 0.5), ("CLUSTERED", 513, 32, 0.5),
    ("CLUSTERED", 1024, 8, 0.1), ("CLUSTERED", 1025, 8, 0.1), ("CLUSTERED", 60, 9, 0.1), ("CLUSTERED", 4096, 32, 0.1),
    ("BLOCKED", 16, 32, 0.1), ("BLOCKED", 16, 33, 0.1), ("BLOCKED", 1024, 2, 0.1), ("BLOCKED", 1025, 2, 0.1),
    ("BLOCKED", 5000, 8, 0.1), ("BLOCKED", 600, 128, 0.1), ("BLOCKED", 600, 129, 0.1),
]


@pytest.mark.gpu
@pytest.mark.parametrize("layout,n_used,n_classes,thr", LIMITS)
def test_forms_at_their_limits(layout, n_used, n_classes, thr):
    f = depth3_forest(-(-n_used // 7) + 3, feats(n_used, -(-n_used // 7) + 3), n_classes, thr)
    X = rows_for(f, 150, n_used + n_classes)
    want = oracle.predict(f, X)
    p = fp.fp_pack_forest(f, layout=getattr(fp, "FP_LAYOUT_" + layout), bin_size=16, interleave_depth=3)
    fp.fp_packed_upload(p)
    for tune in (None, {"feature_lds": -1}, {"feature_lds": -1, "lds_top_nodes": -1, "block_threads": 64}):
        got = gpu_votes(p, X, tune)
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), tune


@pytest.mark.gpu
@pytest.mark.parametrize("thr", [0.5, 0.1])
@pytest.mark.parametrize("n_blocks", [1, 2, 255, 256, 257, 341, 342, 384, 385, 1500])
def test_conversion_chunks(n_blocks, thr):
    """One block per tree, one bin: the conversion's first workgroup, its
    edges and the growing chunks behind it."""
    f = depth3_forest(n_blocks, feats(24, n_blocks), 5, thr)
    X = rows_for(f, 64, n_blocks)
    want = oracle.predict(f, X)
    p = fp.fp_pack_forest(f, layout=fp.FP_LAYOUT_CLUSTERED, bin_size=n_blocks, interleave_depth=3)
    fp.fp_packed_upload(p)
    got = gpu_votes(p, X, {"rows_per_block": 8, "lds_top_nodes": 40})
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.gpu
@pytest.mark.parametrize("layout", ["CLUSTERED", "BLOCKED"])
@pytest.mark.parametrize("integer", [False, True])
def test_deep_forest_with_part_of_its_blocks_in_lds(layout, integer):
    """Blocks whose children are in LDS, partly there, and in memory."""
    X, y = synth.gaussian_mixture(4000, 12, 6, seed=3)
    if integer:
        X = np.rint(X * 8).astype(np.float32)
    f = synth.train_forest(X, y, n_trees=9, n_classes=6, mtry=3, max_depth=-1, bootstrap=True, seed=4)
    want = oracle.predict(f, X)
    for B in (1, 4, 9):
        p = fp.fp_pack_forest(f, layout=getattr(fp, "FP_LAYOUT_" + layout), bin_size=B, interleave_depth=3)
        fp.fp_packed_upload(p)
        for top in (-1, 3, 50, 333, 2000):
            got = gpu_votes(p, X, {"rows_per_block": 64, "block_threads": 512, "lds_top_nodes": top, "lds_bytes": 163840})
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), (B, top)


def test_verifier_refuses_exits_that_are_no_tree():
    """Five exits that cover all outcomes once but are no tree's leaves."""
    X, y = synth.gaussian_mixture(3000, 8, 3, seed=5)
    f = synth.train_forest(X, y, n_trees=4, n_classes=3, mtry=3, max_depth=8, bootstrap=True, seed=6)
    good = fp.fp_packed_host_bytes(fp.fp_pack_forest(f, layout=fp.FP_LAYOUT_CLUSTERED, bin_size=4, interleave_depth=0))
    dec = decode(good)
    assert dec["h"]["block_bytes"] == 64
    fp.fp_packed_from_bytes(reseal(good))
    first = dec["h"]["nodes_offset"] + 8 * int(dec["bins"][0]["node_base"])
    for k in range(int(dec["bins"][0]["deep_len"])):
        at = first + 64 * k
        if (good[at + 28:at + 36] != 0x80).sum() == 5:
            break
    else:
        raise AssertionError("no block with five exits")
    bad = good.copy()
    bad[at + 28:at + 33] = [0b111, 0b111, 0b011, 0b110, 0b101]
    bad[at + 36:at + 41] = [0b000, 0b111, 0b010, 0b100, 0b001]
    cover = np.zeros(16, int)
    for care, val in zip(bad[at + 28:at + 33], bad[at + 36:at + 41]):
        cover += [((g ^ int(val)) & int(care)) == 0 for g in range(16)]
    assert (cover == 1).all()
    with pytest.raises(fp.FPError) as e:
        fp.fp_packed_from_bytes(reseal(bad))
    assert e.value.code == fp.FP_ECORRUPT


def test_verifier_refuses_overlapping_bins():
    f = depth3_forest(8, feats(20, 8), 3, 0.1)
    good = fp.fp_packed_host_bytes(fp.fp_pack_forest(f, layout=fp.FP_LAYOUT_CLUSTERED, bin_size=4, interleave_depth=3))
    dec = decode(good)
    bad = good.copy()
    at = dec["h"]["table_offset"] + 32  # bin 1's first node: bin 0's
    bad[at:at + 8] = good[at - 32:at - 24]
    with pytest.raises(fp.FPError) as e:
        fp.fp_packed_from_bytes(reseal(bad))
    assert e.value.code == fp.FP_ECORRUPT
