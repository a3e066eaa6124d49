"""The work counters of batched launches are kept between runs (plans) or
copied with each call: runs that overlapped on two streams leave nothing
behind that a later run, alone, would suffer from.  Whole numbers: equal to
the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_1806_07300_amd as fp
from handmade import depth3_forest

pytestmark = pytest.mark.gpu


def make(layouts):
    jobs, want = [], []
    for i, layout in enumerate(layouts):
        f = depth3_forest(40 + i, [[(5 * t + 3 * k + i) % 30 for k in range(7)] for t in range(40 + i)], 4, 0.1)
        X = np.random.default_rng(i).random((20_000 + 777 * i, f.n_features), dtype=np.float32)
        p = fp.fp_pack_forest(f, layout=layout, bin_size=16, interleave_depth=3)
        fp.fp_packed_upload(p)
        n = X.shape[0]
        jobs.append((p, torch.from_numpy(X).cuda(), torch.empty((n, 4), dtype=torch.int32, device="cuda"),
                     torch.empty((n,), dtype=torch.int32, device="cuda")))
        want.append(oracle.predict(f, X))
    return jobs, want


LAYOUTS = {"blocks": (fp.FP_LAYOUT_BLOCKED, fp.FP_LAYOUT_CLUSTERED), "nodes": (fp.FP_LAYOUT_PACKED, fp.FP_LAYOUT_COMPACT),
           "mixed": (fp.FP_LAYOUT_BLOCKED, fp.FP_LAYOUT_PACKED)}


@pytest.mark.parametrize("which", ["blocks", "nodes", "mixed"])
@pytest.mark.parametrize("how", ["plan", "noalloc"])
@pytest.mark.parametrize("threads", [64, 1024])
def test_a_run_after_overlapping_ones_is_whole(which, how, threads):
    jobs, want = make(LAYOUTS[which])
    if how == "plan":
        plan = fp.fp_plan_create(jobs, use_graph=False, block_threads=threads)
        run = lambda s=None: fp.fp_predict_batched(plan, stream=s)
    else:  # the same jobs on both streams: the tables that the calls overwrite hold the same bytes
        run = lambda s=None: fp.fp_predict_batched_noalloc(jobs, block_threads=threads, stream=s)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for rep in range(6):
        for k in range(8):
            run(streams[k % 2])
        torch.cuda.synchronize()
        for _, _, votes, cls in jobs:
            votes.fill_(-7)
            cls.fill_(-7)
        run()
        torch.cuda.synchronize()
        for i, (_, _, votes, cls) in enumerate(jobs):
            assert np.array_equal(votes.cpu().numpy(), want[i][0]), (rep, i)
            assert np.array_equal(cls.cpu().numpy(), want[i][1]), (rep, i)
