"""Batched launches whose jobs are partly in block and partly in node layouts
(a kernel each over its part of the work list), with and without tree groups
that add into the same votes, replayed: the work counters are zero again after
every run.  Whole numbers: equal to the CPU checker's."""
import numpy as np
import pytest

import oracle
import paper_1806_07300_amd as fp
from handmade import depth3_forest

pytestmark = pytest.mark.gpu

L = fp


def make(layouts, groups):
    import torch
    jobs, want = [], []
    for i, layout in enumerate(layouts):
        n_trees, n = (5, 40, 130)[i % 3], (1, 700, 70, 9001)[i % 4]
        f = depth3_forest(n_trees, [[(3 * t + k + i) % 11 for k in range(7)] for t in range(n_trees)], 3 + i, 0.1)
        X = np.random.default_rng(i).random((n, f.n_features), dtype=np.float32)
        p = fp.fp_pack_forest(f, layout=layout, bin_size=4, interleave_depth=3)
        fp.fp_packed_upload(p)
        if groups > 1 and i % 2:
            fp.fp_packed_set_tune(p, {"tree_groups": groups})
        votes = torch.full((n, f.n_classes), -7, dtype=torch.int32, device="cuda")
        cls = torch.full((n,), -7, dtype=torch.int32, device="cuda") if i != 2 else None
        jobs.append((p, torch.from_numpy(X).cuda(), votes, cls))
        want.append(oracle.predict(f, X))
    return jobs, want


def check(jobs, want):
    import torch
    torch.cuda.synchronize()
    for (_, _, votes, cls), (wv, wc) in zip(jobs, want):
        assert np.array_equal(votes.cpu().numpy(), wv)
        if cls is not None:
            assert np.array_equal(cls.cpu().numpy(), wc)
        votes.fill_(-7)
        if cls is not None:
            cls.fill_(-7)
    torch.cuda.synchronize()


MIXES = [[L.FP_LAYOUT_BLOCKED, L.FP_LAYOUT_PACKED, L.FP_LAYOUT_CLUSTERED, L.FP_LAYOUT_COMPACT],
         [L.FP_LAYOUT_PACKED, L.FP_LAYOUT_COMPACT], [L.FP_LAYOUT_CLUSTERED, L.FP_LAYOUT_BLOCKED],
         [L.FP_LAYOUT_COMPACT, L.FP_LAYOUT_CLUSTERED, L.FP_LAYOUT_CLUSTERED, L.FP_LAYOUT_PACKED, L.FP_LAYOUT_BLOCKED]]


@pytest.mark.parametrize("groups", [1, 3])
@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("mix", range(len(MIXES)))
def test_mixed_plan(mix, use_graph, groups):
    jobs, want = make(MIXES[mix], groups)
    plan = fp.fp_plan_create(jobs, use_graph=use_graph)
    for _ in range(3):
        fp.fp_predict_batched(plan)
        check(jobs, want)


@pytest.mark.parametrize("groups", [1, 3])
@pytest.mark.parametrize("cursors", [1, 2, 4, 8])
def test_mixed_noalloc(cursors, groups):
    jobs, want = make(MIXES[3], groups)
    for _ in range(3):
        fp.fp_predict_batched_noalloc(jobs, cursors=cursors, block_threads=512)
        check(jobs, want)
