"""What the no-alloc call's fixed scratch has to hold: a full table of 4,096
jobs with 11,092 work items, and the two work lists of block-layout and
node-layout jobs where one list over both would fit.  Whole numbers: equal to
the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_1806_07300_amd as fp
from handmade import depth3_forest

pytestmark = pytest.mark.gpu


def packed(n_trees, layout, **tune):
    f = depth3_forest(n_trees, [[(3 * t + k) % 8 for k in range(7)] for t in range(n_trees)], 4, 0.1)
    p = fp.fp_pack_forest(f, layout=layout, bin_size=2, interleave_depth=3)
    fp.fp_packed_upload(p)
    fp.fp_packed_set_tune(p, tune)
    return f, p


def test_full_job_table():
    f, three = packed(6, fp.FP_LAYOUT_CLUSTERED, tree_groups=3, rows_per_block=16)
    _, two = packed(6, fp.FP_LAYOUT_CLUSTERED, tree_groups=2, rows_per_block=16)
    X = np.random.default_rng(0).random((4096, 8), dtype=np.float32)
    Xd = torch.from_numpy(X).cuda()
    votes = torch.full((4096, 4), -7, dtype=torch.int32, device="cuda")
    cls = torch.full((4096,), -7, dtype=torch.int32, device="cuda")
    jobs = [(three if i < 2900 else two, Xd[i:i + 1], votes[i:i + 1], cls[i:i + 1]) for i in range(4096)]
    fp.fp_predict_batched_noalloc(jobs)
    torch.cuda.synchronize()
    want = oracle.predict(f, X)
    assert np.array_equal(votes.cpu().numpy(), want[0]) and np.array_equal(cls.cpu().numpy(), want[1])


def test_lists_of_both_layout_classes():
    """51,000 and 20,000 tiles; at 100 items a workgroup one list would chunk the cheap ones."""
    jobs, want = [], []
    for n, trees, layout in ((408_000, 20, fp.FP_LAYOUT_BLOCKED), (160_000, 6, fp.FP_LAYOUT_PACKED)):
        f, p = packed(trees, layout, rows_per_block=8, tree_groups=1)
        X = np.random.default_rng(n).random((n, 8), dtype=np.float32)
        jobs.append((p, torch.from_numpy(X).cuda(), torch.full((n, 4), -7, dtype=torch.int32, device="cuda"), None))
        want.append(oracle.predict(f, X)[0])
    fp.fp_predict_batched_noalloc(jobs, items_per_block=100)
    torch.cuda.synchronize()
    for (_, _, votes, _), w in zip(jobs, want):
        assert np.array_equal(votes.cpu().numpy(), w)


def test_one_list_too_long_is_refused():
    _, p = packed(6, fp.FP_LAYOUT_BLOCKED, rows_per_block=1, tree_groups=1)
    n = 70_000
    job = (p, torch.zeros((n, 8), device="cuda"), torch.empty((n, 4), dtype=torch.int32, device="cuda"), None)
    with pytest.raises(fp.FPError) as e:
        fp.fp_predict_batched_noalloc([job], items_per_block=1000)
    assert e.value.code == fp.FP_E2BIG
