"""Walks of many blocks in every walk form and in both host forms, with part
of the blocks in LDS, none, features in LDS and in memory, one forest at a
time and in a batched launch; and, on the CPU, the form that each header
takes on both sides of every limit.  Whole numbers: equal to the
oracle's."""
import os
import subprocess

import numpy as np
import pytest

import oracle
import paper_1806_07300_amd as fp
import synth
from packed_format import decode

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"
NONE, W64, W48H, W48B, W48F, W32H = range(6)
B, K = fp.FP_LAYOUT_BLOCKED, fp.FP_LAYOUT_CLUSTERED

# (layout, features, classes, integer rows) -> (bytes of a packed block, walk form)
FORESTS = {
    "64 clustered": (K, 12, 12, False, 64, W64), "64 blocked": (B, 40, 40, False, 64, W64),
    "48h": (K, 12, 20, True, 48, W48H), "48b": (B, 12, 6, False, 48, W48B), "48b of 64": (B, 300, 20, False, 64, W48B),
    "48f": (K, 12, 6, False, 64, W48F), "32h": (K, 12, 6, True, 48, W32H),
    "host 48": (B, 12, 40, False, 48, NONE), "host 64": (B, 40, 130, False, 64, NONE),
}


def deep_forest(features, classes, integer):
    """9 trees grown to purity on random labels."""
    rng = np.random.default_rng(features + classes)
    X = rng.random((3000, features), dtype=np.float32)
    if integer:
        X = np.rint(X * 200).astype(np.float32)
    y = rng.integers(0, classes, 3000).astype(np.int32)
    f = synth.train_forest(X, y, n_trees=9, n_classes=classes, mtry=3, max_depth=-1, bootstrap=True, seed=4)
    return f, X[:700].copy()


@pytest.fixture(scope="module")
def forests():
    return {k: (*deep_forest(*v[1:4]), v) for k, v in FORESTS.items()}


def forms(rows, tmp_path):
    exe = str(tmp_path / "walk_form")
    csrc = os.path.join(ROOT, "paper_1806_07300_amd", "csrc")
    subprocess.run([CLANG, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                    "-I" + csrc, os.path.join(ROOT, "tests", "native", "walk_form.cpp"), "-o", exe], check=True)
    text = "\n".join(" ".join(str(int(x)) for x in r) for r in rows)
    return [int(x) for x in subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.split()]


@pytest.mark.skipif(not os.path.exists(CLANG) or not os.path.exists(os.path.join(ROOT, "tests", "native")),
                    reason="host compiler or the native sources not here")
def test_forms_of_the_forests_and_on_both_sides_of_the_limits(forests, tmp_path):
    rows, want = [], []
    for f, _, (layout, _, classes, _, block, form) in forests.values():
        p = fp.fp_pack_forest(f, layout=layout, bin_size=4, interleave_depth=3)
        h = decode(fp.fp_packed_host_bytes(p))["h"]
        assert h["block_bytes"] == block
        rows.append((layout, block, classes, h["n_used_features"], h["total_bytes"] - h["nodes_offset"]))
        want.append(form)
    most = 32 * ((1 << 20) - (1 << 14))  # the references of the 32-byte form
    for row, form in (((K, 48, 16, 512, most - 32), W32H), ((K, 48, 16, 512, most), W48H), ((K, 48, 17, 512, 4096), W48H),
                      ((K, 64, 8, 1024, 4096), W48F), ((K, 64, 9, 1024, 4096), W64), ((K, 64, 8, 1025, 4096), W64),
                      ((K, 64, 32, 4096, 4096), W64), ((B, 48, 32, 1024, 4096), W48B), ((B, 48, 33, 1024, 4096), NONE),
                      ((B, 64, 32, 1024, 4096), W48B), ((B, 64, 33, 1024, 4096), W64), ((B, 64, 32, 1025, 4096), W64),
                      ((B, 64, 128, 65535, 4096), W64), ((B, 64, 129, 65535, 4096), NONE), ((B, 64, 128, 65536, 4096), NONE),
                      ((fp.FP_LAYOUT_PACKED, 0, 2, 4, 4096), NONE), ((fp.FP_LAYOUT_COMPACT, 0, 2, 4, 4096), NONE)):
        rows.append(row)
        want.append(form)
    assert forms(rows, tmp_path) == want


@pytest.mark.gpu
@pytest.mark.parametrize("which", list(FORESTS))
def test_deep_walks(forests, which):
    import torch
    f, X, (layout, *_) = forests[which]
    X[::17, ::3] = np.nan
    X[5::19, 1::4] = np.inf
    want = oracle.predict(f, X)
    Xd = torch.from_numpy(X).cuda()
    for bins in (1, 4, 9):
        p = fp.fp_pack_forest(f, layout=layout, bin_size=bins, interleave_depth=3)
        fp.fp_packed_upload(p)
        for top in (-1, 3, 333, 2000, 0):
            for feature_lds in (1, 2, -1):
                v, c = fp.fp_predict_tuned(p, {"rows_per_block": 32, "block_threads": 512, "lds_top_nodes": top,
                                               "feature_lds": feature_lds}, Xd)
                torch.cuda.synchronize()
                assert np.array_equal(v.cpu().numpy(), want[0]), (bins, top, feature_lds)
                assert np.array_equal(c.cpu().numpy(), want[1]), (bins, top, feature_lds)


@pytest.mark.gpu
@pytest.mark.parametrize("feature_lds", [0, 2, -1])
@pytest.mark.parametrize("groups", [1, 2])
def test_deep_walks_in_one_batched_launch(forests, feature_lds, groups):
    import torch
    jobs, want = [], []
    for f, X, (layout, *_) in forests.values():
        p = fp.fp_pack_forest(f, layout=layout, bin_size=4, interleave_depth=3)
        fp.fp_packed_upload(p)
        fp.fp_packed_set_tune(p, {"feature_lds": feature_lds, "tree_groups": groups})
        jobs.append((p, torch.from_numpy(X).cuda(), torch.full((len(X), f.n_classes), -7, dtype=torch.int32, device="cuda"),
                     torch.full((len(X),), -7, dtype=torch.int32, device="cuda")))
        want.append(oracle.predict(f, X))
    plan = fp.fp_plan_create(jobs)
    for _ in range(2):
        fp.fp_predict_batched(plan)
        torch.cuda.synchronize()
        for (name, _), (_, _, v, c), w in zip(forests.items(), jobs, want):
            assert np.array_equal(v.cpu().numpy(), w[0]) and np.array_equal(c.cpu().numpy(), w[1]), name
            v.fill_(-7)
            c.fill_(-7)
