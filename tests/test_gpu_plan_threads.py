"""Plans and no-alloc calls whose tiles are left to the library, over workgroup
sizes: 16 to 64 rows, 64 tiles of 1,024 threads or more.  Whole numbers: equal
to the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_1806_07300_amd as fp
from handmade import depth3_forest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [64, 256, 512, 768, 1024])
@pytest.mark.parametrize("layouts", [(3, 4), (1, 2), (1, 2, 3, 4)])
def test_automatic_tiles(threads, layouts):
    jobs, want = [], []
    for i, (layout, n) in enumerate(zip(layouts * 2, (1, 1023, 1025, 4097, 63, 2000, 3100, 16))):
        f = depth3_forest(30 + i, [[(5 * t + 3 * k + i) % 24 for k in range(7)] for t in range(30 + i)], 5, 0.1)
        X = np.random.default_rng(i).random((n, f.n_features), dtype=np.float32)
        p = fp.fp_pack_forest(f, layout=layout, bin_size=8, interleave_depth=3)
        fp.fp_packed_upload(p)
        jobs.append((p, torch.from_numpy(X).cuda(), torch.full((n, 5), -7, dtype=torch.int32, device="cuda"),
                     torch.full((n,), -7, dtype=torch.int32, device="cuda")))
        want.append(oracle.predict(f, X))
    plan = fp.fp_plan_create(jobs, block_threads=threads)
    for run in (lambda: fp.fp_predict_batched(plan), lambda: fp.fp_predict_batched_noalloc(jobs, block_threads=threads)):
        for _, _, v, c in jobs:
            v.fill_(-7)
            c.fill_(-7)
        run()
        torch.cuda.synchronize()
        for (_, _, v, c), w in zip(jobs, want):
            assert np.array_equal(v.cpu().numpy(), w[0]) and np.array_equal(c.cpu().numpy(), w[1])
