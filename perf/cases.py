"""Timed cases of the library: what programs that classify with packed forests do.

A case is a dict of plain values.  `kind` says which entry points it goes
through:

  predict  fp_pack_forest, fp_packed_upload once; fp_predict per pass
  plan     fp_plan_create once over several forests; fp_predict_batched per pass
  noalloc  fp_predict_batched_noalloc per pass over several forests
  serve    a server with resident forests; fp_serve_submit / fp_serve_poll per pass, on host rows
  infer    fp_infer_cardinality per pass (node statistics from observations, taken before packing)

Forests and rows are made from the seed on the GPU.  `data` is the shape of the
rows: "tabular" (standard normals and, in the last quarter of the columns,
products of pairs of them; two classes), "mixture" (Gaussian classes with
shifted means) or "image" (integer pixels 0..255, about 80% zeros, 10
classes).  A forest is grown on `train` rows per tree: at every node a few
random splits, the one with the best Gini score kept, to pure leaves or to
`depth`, so its node counts, depths and hot paths follow the data.  The
library's results are whole numbers (votes and classes); exact() walks the
forests node by node in 64 bits.
"""
import math

import numpy as np
import torch

import paper_1806_07300_amd as fp
from paper_1806_07300_amd import presets

DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # one observation at a time: a caller in a loop, a forest of 32 trees
        # x depth 12 over 16 features, packed and launched with the defaults
        dict(name="one_row", kind="predict", data="mixture", features=16, classes=10, trees=32, train=10_000, depth=12,
             rows=1, layout="default", launch="default", ld_pad=0, missing=0.0),
        # the small two-class forest's ordinary batch, with its preset
        dict(name="small_10k", kind="predict", data="mixture", features=16, classes=2, trees=32, train=10_000,
             depth=12, rows=10_000, layout="preset", launch="preset", ld_pad=0, missing=0.0),
        # a request-sized batch of images, library default launch
        dict(name="image_300", kind="predict", data="image", features=784, classes=10, trees=128, train=60_000,
             depth=0, rows=300, layout="clustered", launch="default", ld_pad=0, missing=0.0),
        # the image workload: 1M rows of 784 pixels through 128 trees, its preset
        dict(name="image_1m", kind="predict", data="image", features=784, classes=10, trees=128, train=60_000,
             depth=0, rows=1_000_000, layout="preset", launch="preset", ld_pad=0, missing=0.0),
        # a request-sized batch for a forest of many trees
        dict(name="trees_1024", kind="predict", data="tabular", features=28, classes=2, trees=1024, train=10_000,
             depth=12, rows=4_096, layout="clustered", launch="default", ld_pad=0, missing=0.0),
        # everything left at its default (node layout): a mid-sized forest of
        # about 24,000 nodes per tree, an odd number of rows, missing values
        dict(name="defaults_100k", kind="predict", data="tabular", features=28, classes=2, trees=64, train=70_000,
             depth=0, rows=100_003, layout="default", launch="default", ld_pad=0, missing=0.01),
        # wide real-valued rows of a table with more columns, 10 classes,
        # complete-subtree blocks
        dict(name="wide_20k", kind="predict", data="mixture", features=784, classes=10, trees=256, train=10_000,
             depth=12, rows=20_001, layout="blocked", launch="default", ld_pad=16, missing=0.0),
        # the large tabular workload: a forest beyond the last-level cache,
        # walked in passes, with its preset
        dict(name="tabular_2m", kind="predict", data="tabular", features=28, classes=2, trees=160, train=400_000,
             depth=0, rows=2_000_000, layout="preset", launch="preset", ld_pad=0, missing=0.0),
        # many uneven forests in one graph launch
        dict(name="plan_16", kind="plan", jobs=16, trees=512, features=256, train=10_000, depth=12, rows=60_000),
        # a few small forests without device allocations (code under capture, tight loops)
        dict(name="noalloc_6", kind="noalloc", jobs=6, trees=128, features=64, train=10_000, depth=12, rows=4_000),
        # 48 requests of 1 to 4,096 rows to four resident forests, from host memory
        dict(name="serve_48", kind="serve", jobs=4, trees=256, features=256, train=10_000, depth=12, requests=48,
             rows=4_096),
        # access statistics of a forest from 65,536 observations
        dict(name="infer_65k", kind="infer", data="tabular", features=28, classes=2, trees=64, train=70_000, depth=0,
             rows=65_536, missing=0.0),
    ]


def draw(rng):
    def logu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["predict"] * 6 + ["plan", "noalloc", "serve", "infer"])
    if kind in ("plan", "noalloc", "serve"):
        c = dict(kind=kind, jobs=rng.randint(2, 16 if kind == "plan" else 8), trees=logu(16, 512 if kind == "plan" else 256),
                 features=logu(8, 256), train=10_000, depth=rng.randint(6, 12))
        if kind == "serve":
            c.update(requests=rng.randint(8, 60))
        c["rows"] = logu(500, {"plan": 60_000, "noalloc": 10_000, "serve": 4_096}[kind])
        return c
    data = rng.choice(["tabular", "mixture", "image"])
    if data == "image":
        features, classes = 784, 10
    elif data == "tabular":
        features, classes = rng.randint(8, 64), 2
    else:
        features, classes = logu(4, 784), rng.randint(2, 10)
    deep = data != "mixture" and rng.random() < 0.5
    c = dict(kind=kind, data=data, features=features, classes=classes, trees=logu(8, 96 if deep else 1024),
             train=logu(10_000, 100_000) if deep else 10_000, depth=0 if deep else rng.randint(5, 12))
    most = min(1_000_000, 30_000_000 // c["trees"], 200_000_000 // features)
    if kind == "infer":
        return dict(c, trees=min(c["trees"], 128), rows=logu(100, min(most, 200_000)),
                    missing=rng.choice([0.0, 0.0, 0.02]) if data != "image" else 0.0)
    layout = rng.choice(["default", "compact", "blocked", "clustered", "clustered", "preset"])
    if layout == "preset" and data == "tabular":
        c["features"] = min(features, 28)
    return dict(c, rows=logu(4, most), layout=layout, launch="preset" if layout == "preset" else "default",
                ld_pad=rng.choice([0, 0, 1, 4, 7]), missing=rng.choice([0.0, 0.0, 0.02]) if data != "image" else 0.0)


# ---------------------------------------------------------------------------
# rows and forests from a seed
# ---------------------------------------------------------------------------
def _gen(*seed):
    g = torch.Generator(device=DEV)
    h = 0x9E3779B97F4A7C15
    for s in seed:
        h = ((h ^ int(s)) * 0x100000001B3 + 0x632BE59BD9B4E019) % (1 << 62)
    g.manual_seed(h)
    return g


def _image_means(g):
    """Per class a mean image on 30% of the pixels, inside a shared 45% pool."""
    pool = torch.randperm(784, generator=g, device=DEV)[:353]
    mean = torch.zeros(10, 784, device=DEV)
    for k in range(10):
        at = pool[torch.randperm(353, generator=g, device=DEV)[:235]]
        mean[k, at] = 255.0 * torch.rand(235, generator=g, device=DEV) + 1.0
    return mean


def _rows(data, n, features, classes, gm, g, ld_pad=0, missing=0.0):
    """n observations and their classes: the population from gm, the draws from g."""
    X = torch.zeros(n, features + ld_pad, device=DEV)[:, :features]
    y = torch.empty(n, dtype=torch.int64, device=DEV)
    if data == "image":
        mean = _image_means(gm)
    elif data == "tabular":
        nz = features - features // 4
        pair = torch.randint(nz, (2, features - nz), generator=gm, device=DEV)
        w = torch.randn(features, generator=gm, device=DEV, dtype=torch.float64) / math.sqrt(features)
    for lo in range(0, n, 1 << 17):
        hi = min(n, lo + (1 << 17))
        m = hi - lo
        if data == "image":
            k = torch.randint(10, (m,), generator=g, device=DEV)
            v = (mean[k] + 48.0 * torch.randn(m, 784, generator=g, device=DEV)).round_().clamp_(0.0, 255.0)
            v *= (mean[k] > 0) & (torch.rand(m, 784, generator=g, device=DEV) < 0.72)
            X[lo:hi] = v
            other = torch.randint(10, (m,), generator=g, device=DEV)
            y[lo:hi] = torch.where(torch.rand(m, generator=g, device=DEV) < 0.08, other, k)
        elif data == "tabular":
            z = torch.randn(m, nz, generator=g, device=DEV)
            X[lo:hi, :nz] = z
            X[lo:hi, nz:] = z[:, pair[0]] * z[:, pair[1]]
            q = (X[lo:hi].double() * w).sum(1)
            y[lo:hi] = (q + 0.7 * torch.randn(m, generator=g, device=DEV) > 0).long()
        else:
            k = torch.randint(classes, (m,), generator=g, device=DEV)
            y[lo:hi] = k
            X[lo:hi] = torch.randn(m, features, generator=g, device=DEV) + (k.float() / max(classes - 1, 1))[:, None]
    if missing:
        X.masked_fill_(torch.rand(n, features, generator=g, device=DEV) < missing, float("nan"))
    return X, y


class Forest:
    """Trees as concatenated node arrays in breadth-first order (what a trainer hands to fp_pack_forest)."""


def _grow(X, y, classes, trees, n, depth, tries, g):
    """Grows `trees` trees on n rows each, drawn with replacement, level by level for all trees at once."""
    N, F = X.shape
    samp = torch.randint(N, (trees * n,), generator=g, device=DEV)
    off = torch.arange(trees + 1, device=DEV) * n           # samples of frontier node m: [off[m], off[m + 1])
    tree = torch.arange(trees, device=DEV)
    levels, first = [], 0                                   # per level: (tree, feature, thr, left, right, class, count)
    while tree.numel():
        M = tree.numel()
        cnt = off[1:] - off[:-1]
        seg = torch.repeat_interleave(torch.arange(M, device=DEV), cnt)
        lab = y[samp]
        hist = torch.zeros(M * classes, dtype=torch.int32, device=DEV)
        hist.scatter_add_(0, seg * classes + lab, torch.ones_like(seg, dtype=torch.int32))
        hist = hist.view(M, classes)
        top, _ = hist.max(1)
        # the most frequent class, the lowest on ties
        label = (hist.long() * classes + torch.arange(classes - 1, -1, -1, device=DEV)).argmax(1)
        split = (top < cnt) & (cnt >= 2) & (depth == 0 or len(levels) < depth)
        best = torch.full((M,), -1.0, dtype=torch.float64, device=DEV)
        feat = torch.zeros(M, dtype=torch.int64, device=DEV)
        thr = torch.zeros(M, device=DEV)
        keep = split[seg]
        samp, seg, lab = samp[keep], seg[keep], lab[keep]
        off = torch.zeros(M + 1, dtype=torch.int64, device=DEV)
        off[1:] = torch.cumsum(cnt * split, 0)
        if not samp.numel():
            split = torch.zeros_like(split)
        else:
            total = hist.double()
            last = samp.numel() - 1
            for _ in range(tries):
                f = torch.randint(F, (M,), generator=g, device=DEV)
                u = torch.rand(2, M, generator=g, device=DEV, dtype=torch.float64)
                at = (off[:-1] + (u * cnt).long().clamp_(max=cnt - 1)).clamp_(max=last)
                a, b = X[samp[at[0]], f], X[samp[at[1]], f]
                lo, hi = torch.minimum(a, b), torch.maximum(a, b)
                t = (lo + hi) * 0.5
                t = torch.where(t >= hi, lo, t)
                left = X[samp, f[seg]] <= t[seg]
                lh = torch.zeros(M * classes, dtype=torch.int32, device=DEV)
                lh.scatter_add_(0, seg * classes + lab, left.int())
                L = lh.view(M, classes).double()
                R = total - L
                nl, nr = L.sum(1), R.sum(1)
                score = torch.where((lo < hi) & split, (L * L).sum(1) / nl.clamp(min=1) + (R * R).sum(1) / nr.clamp(min=1),
                                    torch.full_like(best, -1.0))
                better = score > best
                best = torch.where(better, score, best)
                feat = torch.where(better, f, feat)
                thr = torch.where(better, t, thr)
            split = best > 0
            keep = split[seg]
            if not bool(keep.all()):
                samp, seg = samp[keep], seg[keep]
                off[1:] = torch.cumsum(cnt * split, 0)
        S = int(split.sum())
        rank = torch.cumsum(split, 0) - 1                   # split nodes in order: children 2 rank, 2 rank + 1
        child = first + M + 2 * rank
        levels.append((tree, torch.where(split, feat, -1), thr, torch.where(split, child, -1),
                       torch.where(split, child + 1, -1), label, cnt))
        first += M
        if not S:
            break
        # the samples of each split node, left ones first, both in their order
        left = X[samp, feat[seg]] <= thr[seg]
        cl = torch.cumsum(left, 0)
        base = torch.cat([cl.new_zeros(1), cl])[off]        # left samples before each node
        nl = base[1:] - base[:-1]
        i = torch.arange(samp.numel(), device=DEV)
        lrank = cl - left.long() - base[seg]
        pos = off[seg] + torch.where(left, lrank, nl[seg] + (i - off[seg]) - lrank)
        moved = torch.empty_like(samp)
        moved[pos] = samp
        samp = moved
        sizes = torch.stack([nl, (off[1:] - off[:-1]) - nl], 1)[split].view(-1)
        off = torch.zeros(2 * S + 1, dtype=torch.int64, device=DEV)
        off[1:] = torch.cumsum(sizes, 0)
        tree = tree[split].repeat_interleave(2)
    cols = [torch.cat([lv[c] for lv in levels]) for c in range(7)]
    order = torch.sort(cols[0], stable=True)[1]             # per tree, levels in order: breadth-first
    at = torch.empty_like(order)
    at[order] = torch.arange(order.numel(), device=DEV)
    sizes = torch.bincount(cols[0], minlength=trees)
    start = torch.zeros(trees + 1, dtype=torch.int64, device=DEV)
    start[1:] = torch.cumsum(sizes, 0)
    shift = start[cols[0]]

    def out(v, dtype):
        return v[order].to(dtype).cpu().numpy()

    f = Forest()
    f.n_trees, f.n_features, f.n_classes = trees, F, classes
    f.tree_node_offset = start.cpu().numpy()
    f.feature, f.threshold = out(cols[1], torch.int32), out(cols[2], torch.float32)
    inner = cols[1] >= 0
    f.left = out(torch.where(inner, at[cols[3].clamp(min=0)] - shift, -1), torch.int32)
    f.right = out(torch.where(inner, at[cols[4].clamp(min=0)] - shift, -1), torch.int32)
    f.leaf_class = out(torch.where(inner, -1, cols[5]), torch.int32)
    f.cardinality = out(cols[6], torch.int64)
    f.n_levels = len(levels)
    return f


def _forest(c, seed, job=0):
    X, y = _rows(c["data"], c["train"], c["features"], c["classes"], _gen(seed, job, 1), _gen(seed, job, 2))
    return _grow(X, y, c["classes"], c["trees"], c["train"], c["depth"], 12 if c["data"] == "image" else 3,
                 _gen(seed, job, 3))


def _inputs(c, seed, job=0):
    return _rows(c["data"], c["rows"], c["features"], c["classes"], _gen(seed, job, 1), _gen(seed, job, 4),
                 c.get("ld_pad", 0), c.get("missing", 0.0))[0]


def _jobs(c):
    """The forests of a plan, a batched call or a server: sizes spread below the case's largest."""
    rng = np.random.Generator(np.random.PCG64([c["jobs"], c["trees"], c["features"], c["rows"]]))
    out = []
    for i in range(c["jobs"]):
        def logu(lo, hi):
            return int(round(math.exp(rng.uniform(math.log(lo), math.log(max(lo, hi))))))
        j = dict(data="mixture", train=c["train"], depth=c["depth"], trees=logu(16, c["trees"]),
                 features=logu(4, c["features"]), classes=int(rng.integers(2, 11)), rows=logu(1, c["rows"]),
                 layout="clustered" if i % 4 == 3 else "blocked")
        if i == 0:
            j.update(trees=c["trees"], features=c["features"], rows=c["rows"])
        out.append(j)
    return out


def _requests(c):
    """(forest, rows) of each request of a serving pass."""
    rng = np.random.Generator(np.random.PCG64([c["requests"], c["rows"]]))
    return [(int(rng.integers(c["jobs"])), int(math.exp(rng.uniform(0.0, math.log(c["rows"] + 1)))))
            for _ in range(c["requests"])]


# ---------------------------------------------------------------------------
# what a program has in hand, and one pass
# ---------------------------------------------------------------------------
def _pack(c, forest):
    layout = c["layout"]
    if layout == "default":
        p = fp.fp_pack_forest(forest)
    elif layout == "preset":
        p = fp.fp_pack_forest(forest, **_preset(c)["pack"])
    else:
        p = fp.fp_pack_forest(forest, layout={"compact": fp.FP_LAYOUT_COMPACT, "blocked": fp.FP_LAYOUT_BLOCKED,
                                              "clustered": fp.FP_LAYOUT_CLUSTERED}[layout],
                              bin_size=16, interleave_depth=3)
    fp.fp_packed_upload(p)
    if c.get("launch") == "preset":
        tune = dict(_preset(c)["tune"])
        if tune.get("tree_passes", 0) > 1:  # about one pass per 176 MB of forest
            tune["tree_passes"] = -(-p.info["bytes"] // (176 << 20))
        fp.fp_packed_set_tune(p, tune)
    return p


def _preset(c):
    return {"image": presets.IMAGE, "tabular": presets.TABULAR, "mixture": presets.SMALL}[c["data"]]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "predict":
        return dict(kind=kind, packed=_pack(case, _forest(case, seed)), X=_inputs(case, seed))
    if kind == "infer":
        # one forest for every seed (a count per node comes back); the observations are the seed's
        return dict(kind=kind, forest=_forest(case, 0), X=_inputs(case, seed))
    jobs = _jobs(case)
    packed = [_pack(j, _forest(j, seed, i)) for i, j in enumerate(jobs)]
    if kind == "serve":
        server = fp.fp_server_create(hbm_budget_bytes=256 << 20, max_inflight=4)
        ids = [fp.fp_server_add_forest(server, p) for p in packed]
        reqs = []
        for r, (i, n) in enumerate(_requests(case)):
            X = _inputs(dict(jobs[i], rows=n), seed * 1000 + r, i)
            reqs.append((ids[i], X.cpu().numpy(), np.zeros((n, jobs[i]["classes"]), np.int32)))
        return dict(kind=kind, server=server, reqs=reqs, packed=packed)
    table = []
    for i, (j, p) in enumerate(zip(jobs, packed)):
        X = _inputs(j, seed, i)
        table.append((p, X, torch.zeros(j["rows"], j["classes"], dtype=torch.int32, device=DEV),
                      torch.zeros(j["rows"], dtype=torch.int32, device=DEV)))
    state = dict(kind=kind, jobs=table)
    if kind == "plan":
        state["plan"] = fp.fp_plan_create(table)
    return state


def run(state):
    kind = state["kind"]
    if kind == "predict":
        return fp.fp_predict(state["packed"], state["X"])
    if kind == "infer":
        return fp.fp_infer_cardinality(state["forest"], state["X"])
    if kind == "serve":
        server = state["server"]
        tickets = [fp.fp_serve_submit(server, f, X, votes) for f, X, votes in state["reqs"]]
        for t in tickets:
            fp.fp_serve_poll(server, t)
        return [votes for _, _, votes in state["reqs"]]
    if kind == "plan":
        fp.fp_predict_batched(state["plan"])
    else:
        fp.fp_predict_batched_noalloc(state["jobs"])
    return [(votes, cls) for _, _, votes, cls in state["jobs"]]


# ---------------------------------------------------------------------------
# what a pass cannot do without, and its exact result
# ---------------------------------------------------------------------------
def _one_work(c, rows, cls=True):
    """One forest: rows, votes and classes once, the forest once at 8 bytes
    (a threshold, a feature and a reference) per split, about one split per
    three training rows up to a full tree of the given depth; one comparison
    per tree and level of a balanced tree."""
    splits = c["trees"] * min(c["train"] / 3.0, 2.0 ** c["depth"] if c["depth"] else math.inf)
    out = 4.0 * rows * (c["classes"] + bool(cls))
    levels = min(math.log2(c["train"] / 3.0), c["depth"] or math.inf)
    return 4.0 * rows * c["features"] + out + 8.0 * splits, rows * c["trees"] * levels


def work(case):
    kind = case["kind"]
    if kind in ("predict", "infer"):
        b, f = _one_work(case, case["rows"])
    elif kind == "serve":
        jobs = _jobs(case)
        got = [_one_work(jobs[i], n, False) for i, n in _requests(case)]
        b, f = sum(x[0] for x in got), sum(x[1] for x in got)
    else:
        got = [_one_work(j, j["rows"]) for j in _jobs(case)]
        b, f = sum(x[0] for x in got), sum(x[1] for x in got)
    return {"bytes": float(b), "flops": float(f)}


def _walk(forest, X):
    """Votes and classes of rows X, in 64 bits, a tree and a level at a time."""
    n, C = X.shape[0], forest.n_classes
    votes = torch.zeros(n, C, dtype=torch.int64, device=DEV)
    row = torch.arange(n, device=DEV)
    off = forest.tree_node_offset
    feature, left, right, label = (torch.from_numpy(a).to(DEV).long() for a in
                                   (forest.feature, forest.left, forest.right, forest.leaf_class))
    thr = torch.from_numpy(forest.threshold).to(DEV).double()
    for t in range(forest.n_trees):
        lo, hi = int(off[t]), int(off[t + 1])
        f, l, r, h = feature[lo:hi], left[lo:hi], right[lo:hi], thr[lo:hi]
        at = torch.zeros(n, dtype=torch.int64, device=DEV)
        for _ in range(forest.n_levels):
            x = X[row, f[at].clamp(min=0)].double()
            go = torch.where(x <= h[at], l[at], r[at])
            at = torch.where(f[at] >= 0, go, at)
        votes[row, label[lo:hi][at]] += 1
    order = torch.arange(C - 1, -1, -1, device=DEV)
    return votes.int(), (votes * C + order).argmax(1).int()


def exact(case, seed):
    kind = case["kind"]
    if kind == "predict":
        return _walk(_forest(case, seed), _inputs(case, seed))
    if kind == "infer":
        return None  # counts of visits: whole numbers
    jobs = _jobs(case)
    if kind == "serve":
        forests = [_forest(j, seed, i) for i, j in enumerate(jobs)]
        return [_walk(forests[i], _inputs(dict(jobs[i], rows=n), seed * 1000 + r, i))[0]
                for r, (i, n) in enumerate(_requests(case))]
    return [_walk(_forest(j, seed, i), _inputs(j, seed, i)) for i, j in enumerate(jobs)]
