"""PACKED buffers whose alignment gaps (node slots behind a bin that no
reference reaches) hold anything at all: the verifier accepts them, and a walk
that loads a node together with the slot behind it takes nothing from a gap,
whatever feature it names.  Votes are whole numbers: equal to the
oracle's."""
import numpy as np
import pytest

import oracle
import paper_1806_07300_amd as fp
import synth
from packed_format import NODE, decode, reseal


@pytest.fixture(scope="module")
def deep():
    """9 trees grown to purity on random labels: walks of a dozen nodes."""
    rng = np.random.default_rng(3)
    X = rng.random((6000, 8), dtype=np.float32)
    y = rng.integers(0, 3, 6000).astype(np.int32)
    return synth.train_forest(X, y, n_trees=9, n_classes=3, mtry=3, max_depth=-1, bootstrap=True, seed=8)


def planted(f, bin_size, D):
    """The packed bytes with every slot outside the bins overwritten, and how many there were."""
    good = fp.fp_packed_host_bytes(fp.fp_pack_forest(f, layout=fp.FP_LAYOUT_PACKED, bin_size=bin_size, interleave_depth=D))
    dec = decode(good)
    used = np.zeros(dec["h"]["n_nodes"], bool)
    for be in dec["bins"]:
        used[be["node_base"]:be["node_base"] + be["top_len"] + be["deep_len"]] = True
    bad = good.copy()
    at = dec["h"]["nodes_offset"]
    nodes = bad[at:at + 16 * len(used)].view(NODE)
    gaps = np.flatnonzero(~used)
    nodes["feat"][gaps] = np.resize(np.array([900, -1, 2**31 - 1, -2**31, dec["h"]["n_used_features"]], np.int32), len(gaps))
    nodes["thr"][gaps] = np.nan
    nodes["left"][gaps], nodes["right"][gaps] = 2**31 - 1, -2**31
    return reseal(bad), len(gaps)


@pytest.mark.parametrize("bin_size,D", [(1, 0), (2, 1), (5, 3)])
def test_gaps_are_not_verified(deep, bin_size, D):
    buf, n = planted(deep, bin_size, D)
    assert n > 0
    assert fp.fp_packed_from_bytes(buf).info["expected_depth"] > 11


@pytest.mark.gpu
@pytest.mark.parametrize("bin_size,D", [(1, 0), (2, 1), (5, 3)])
@pytest.mark.parametrize("cursors", [1, 2, 4])
def test_gaps_decide_nothing(deep, bin_size, D, cursors):
    import torch
    f = deep
    X = np.random.default_rng(bin_size).random((333, f.n_features), dtype=np.float32)
    X[::17, ::3] = np.nan
    want = oracle.predict(f, X)
    p = fp.fp_packed_from_bytes(planted(f, bin_size, D)[0])
    fp.fp_packed_upload(p)
    Xd = torch.from_numpy(X).cuda()
    for feature_lds in (1, -1):
        for top in (0, 2, -1):
            v, c = fp.fp_predict_tuned(p, {"cursors": cursors, "feature_lds": feature_lds, "lds_top_nodes": top}, Xd)
            torch.cuda.synchronize()
            assert np.array_equal(v.cpu().numpy(), want[0]) and np.array_equal(c.cpu().numpy(), want[1]), (feature_lds, top)
    votes = torch.full((333, 3), -7, dtype=torch.int32, device="cuda")
    fp.fp_predict_batched_noalloc([(p, Xd, votes, None)], cursors=cursors)
    torch.cuda.synchronize()
    assert np.array_equal(votes.cpu().numpy(), want[0])
