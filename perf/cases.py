"""The work that users of this framework have it do, as cases to be timed.

Each case is a tree ensemble, a block of rows and one public call on them:
first-order Shapley values, a training step on the leaf values (values and
their adjoint, through autograd), pairwise interactions, or third-order
interactions.  The ensembles are of the two kinds that boosting libraries
grow: full trees of a fixed depth, and trees grown into their larger child
first under a cap on leaves (deep, ragged).  Rows are standard normal columns
with some integer columns 0..9 (ties with thresholds) and, where the case says
so, missing values.

A case's fields: kind (values, train, pairs, triples), rows, trees, depth (the
deepest a tree may grow), min_depth (trees draw their depth limit from
[min_depth, depth]; 0: all the same), leaves (cap per tree; 0: none, full
trees), features, integers and missing (shares of columns and of values),
outputs (1, or several with a tree each in turn), precision, traversal (of the
interactions calls).
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2605_04497_amd as qts

TRAIN_ROWS = 100_000  # rows that the covers count
LEAF_SIGMA = 0.05


def _case(name, kind, rows, trees, depth, features, *, min_depth=0, leaves=0, integers=0.2,
          missing=0.0, outputs=1, precision="fp32", traversal="auto"):
    c = {"kind": kind, "rows": rows, "trees": trees, "depth": depth, "min_depth": min_depth,
         "leaves": leaves, "features": features, "integers": integers, "missing": missing,
         "outputs": outputs, "precision": precision, "traversal": traversal}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one row explained while a request waits: a usual boosted model
        _case("one_row", "values", 1, 500, 6, 50),
        # a notebook's or a monitor's small block on a small model
        _case("small_model", "values", 1000, 10, 4, 8, integers=0.0),
        # a large table explained on the usual large model (the benchmark's rows, half its trees)
        _case("table", "values", 100000, 500, 8, 100),
        # the same in double precision, with missing values, a ragged number of rows
        _case("table_fp64_missing", "values", 5003, 300, 8, 100, missing=0.02, precision="fp64"),
        # deep trees grown under a cap on leaves: paths of up to 32 features
        _case("deep_trees", "values", 10000, 100, 32, 64, leaves=512, integers=0.0),
        # wide tables (image-like, one-hot): features past one sample tile
        _case("wide", "values", 3001, 200, 8, 784),
        # a multi-class model, one output per class, with missing values
        _case("multi_class", "values", 4099, 350, 6, 54, outputs=7, missing=0.05),
        # a training step on the leaf values: values and their adjoint
        _case("train_step", "train", 20000, 200, 6, 50, integers=0.0),
        # pairwise interactions of a few rows, for a page that shows them
        _case("pairs_few_rows", "pairs", 16, 300, 6, 30),
        # pairwise interactions of a sample of rows, trees of many depths
        _case("pairs_table", "pairs", 512, 100, 20, 200, min_depth=3, leaves=1024, integers=0.0),
        # pairwise interactions of deep trees, by the walk of the trees
        _case("pairs_deep", "pairs", 1003, 100, 32, 64, leaves=512, integers=0.0,
              traversal="dfs"),
        # third-order indices of a sample of rows
        _case("triples", "triples", 1000, 200, 6, 50, integers=0.0),
    ]


def _spread(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# the most method flops that a drawn case of each kind has: its listed cases' largest
def _most(kind):
    return max(work(c)["flops"] for c in listed() if c["kind"] == kind)


def draw(rng):
    kind = rng.choice(["values", "values", "values", "values", "train", "train", "pairs", "pairs",
                       "triples"])
    deep = kind != "triples" and rng.random() < 0.3
    c = _case(None, kind, 1, 1, 1, 1)
    c["precision"] = "fp64" if rng.random() < 0.25 else "fp32"
    c["integers"] = rng.choice([0.0, 0.2])
    c["missing"] = rng.choice([0.0, 0.0, 0.02, 0.05])
    if deep:
        c["depth"] = rng.randint(10, 32)
        c["min_depth"] = rng.choice([0, 3])
        c["leaves"] = _spread(rng, 64, 1024)
        c["trees"] = _spread(rng, 10, 100)
        if kind == "pairs" and c["depth"] >= 16 and rng.random() < 0.5:
            c["traversal"] = "dfs"
    else:
        c["depth"] = rng.randint(3, 6 if kind == "triples" else 8)
        c["trees"] = _spread(rng, 10, 200 if kind == "triples" else 1000)
    if kind in ("values", "train"):
        c["features"] = _spread(rng, 8, 200)
        if not deep and rng.random() < 0.15:
            c["features"] = rng.randint(211, 784)
            c["trees"] = min(c["trees"], 200)
        if rng.random() < 0.2:
            c["outputs"] = rng.randint(2, 10)
            c["trees"] = max(c["trees"], 2 * c["outputs"])
        c["rows"] = _spread(rng, 1, 50000)
    elif kind == "pairs":
        c["features"] = _spread(rng, 8, 200)
        c["rows"] = _spread(rng, 1, 1024)
    else:
        c["features"] = _spread(rng, 8, 50)
        c["rows"] = _spread(rng, 1, 1000)
    # no more work than the kind's largest listed case: fewer rows, then fewer trees
    over = work(c)["flops"] / _most(kind)
    if over > 1:
        c["rows"] = max(1, int(c["rows"] / over))
    while work(c)["flops"] > _most(kind) and c["trees"] > 10:
        c["trees"] = max(10, c["trees"] * 2 // 3)
    return c


# ------------------------------------------------------------------- the model

def _grow(case, rng):
    """The trees of a case, all at once, tree by tree and node by node in the
    order in which they are grown: parent (local), side, depth and cover."""
    T, D = case["trees"], case["depth"]
    limit = rng.integers(case["min_depth"], D + 1, T) if case["min_depth"] else np.full(T, D)
    cap = case["leaves"] or 1 << D
    most = 2 * min(cap, 1 << min(D, 20)) - 1
    left = np.full((T, most), -1, np.int32)
    parent = np.full((T, most), -1, np.int32)
    depth = np.zeros((T, most), np.int32)
    cover = np.zeros((T, most))
    cover[:, 0] = TRAIN_ROWS
    share = rng.uniform(0.05, 0.95, (T, most))  # of a node's rows that go left
    stack = np.zeros((T, D + 2), np.int32)
    top = np.ones(T, np.int32)  # entries on each tree's stack
    count = np.ones(T, np.int32)
    leaves = np.ones(T, np.int32)
    t = np.arange(T)
    while t.size:
        v = stack[t, top[t] - 1]
        top[t] -= 1
        ok = (depth[t, v] < limit[t]) & (cover[t, v] >= 2) & (leaves[t] < cap)
        s, v = t[ok], v[ok]
        if s.size:
            a = count[s]  # the left child; the right one follows
            count[s] += 2
            leaves[s] += 1
            left[s, v] = a
            n = np.clip(np.round(cover[s, v] * share[s, v]), 1, cover[s, v] - 1)
            cover[s, a], cover[s, a + 1] = n, cover[s, v] - n
            parent[s, a] = parent[s, a + 1] = v
            depth[s, a] = depth[s, a + 1] = depth[s, v] + 1
            large = n * 2 >= cover[s, v]
            stack[s, top[s]] = np.where(large, a + 1, a)
            stack[s, top[s] + 1] = np.where(large, a, a + 1)  # the larger child next
            top[s] += 2
        t = t[top[t] > 0]
    real = np.arange(most)[None, :] < count[:, None]
    off = np.concatenate([[0], np.cumsum(count)]).astype(np.int64)
    return SimpleNamespace(off=off, left=left[real], parent=parent[real], depth=depth[real],
                           cover=cover[real], share=share[real],
                           tree=np.repeat(np.arange(T), count))


def _model(case, seed):
    # the trees' shapes are the case's, everything else the seed's
    g = _grow(case, np.random.default_rng(1))
    rng = np.random.default_rng([seed, 1])
    F = case["features"]
    N = g.left.size
    base = g.off[g.tree]
    up = np.where(g.parent >= 0, base + g.parent, -1)
    is_left = np.zeros(N, bool)
    inner = np.flatnonzero(g.left >= 0)
    is_left[base[inner] + g.left[inner]] = True
    feature = rng.integers(0, F, N).astype(np.int32)
    whole = feature < int(F * case["integers"])
    # the share of the column's values below each threshold, inside what the splits above left
    q = np.zeros(N)
    for level in range(int(g.depth.max()) + 1):
        v = inner[g.depth[inner] == level]
        lo, hi = np.zeros(v.size), np.ones(v.size)
        at = v.copy()
        for _ in range(level):
            from_left = is_left[at]
            at = up[at]
            same = feature[at] == feature[v]
            hi = np.where(same & from_left, np.minimum(hi, q[at]), hi)
            lo = np.where(same & ~from_left, np.maximum(lo, q[at]), lo)
        x = lo + g.share[v] * (hi - lo)
        near = np.round(10 * x) / 10
        x = np.where(whole[v] & (near > lo + 0.05) & (near < hi - 0.05), near, x)
        q[v] = x
    normal = torch.special.ndtri(torch.from_numpy(np.clip(q, 1e-12, 1 - 1e-12))).numpy()
    leaf = g.left < 0
    m = SimpleNamespace(
        tree_offsets=g.off, left=g.left, right=np.where(leaf, -1, g.left + 1).astype(np.int32),
        feature=np.where(leaf, -1, feature).astype(np.int32),
        threshold=np.where(leaf, 0, np.where(whole, 10 * q, normal)).astype(np.float32),
        default_left=rng.integers(0, 2, N).astype(np.uint8), cover=g.cover,
        value=np.where(leaf, rng.normal(0, LEAF_SIGMA, N), 0.0), n_features=F, base_score=0.5)
    if case["outputs"] > 1:
        m.n_groups = case["outputs"]
        m.tree_group = (np.arange(case["trees"]) % case["outputs"]).astype(np.int32)
    m.up, m.is_left, m.tree, m.depth = up, is_left, g.tree, g.depth
    return m


def _rows(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 2 + 1)
    M, F = case["rows"], case["features"]
    X = torch.randn((M, F), generator=g, device="cuda", dtype=torch.float32)
    n = int(F * case["integers"])
    if n:
        X[:, :n] = torch.randint(0, 10, (M, n), generator=g, device="cuda").float()
    if case["missing"]:
        X[torch.rand((M, F), generator=g, device="cuda") < case["missing"]] = float("nan")
    shape = (M, case["outputs"], F) if case["outputs"] > 1 else (M, F)
    target = 0.1 * torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
    return X, target.to(torch.float64 if case["precision"] == "fp64" else torch.float32)


# ------------------------------------------------------------------- the calls

def prepare(case, seed):
    m = _model(case, seed)
    X, target = _rows(case, seed)
    ens = qts.Ensemble(m)
    if case["traversal"] != "auto":
        ens.set_pair_traversal(case["traversal"])
    s = SimpleNamespace(kind=case["kind"], precision=case["precision"], ens=ens, X=X)
    if case["kind"] == "train":
        s.target = target
        s.leaf_values = torch.from_numpy(m.value[m.left < 0]).cuda().requires_grad_()
    return s


def run(s):
    if s.kind == "values":
        return s.ens.shap_values(s.X, s.precision)
    if s.kind == "train":
        # the gradient of half the squared distance to the target
        phi = qts.ShapValues.apply(s.leaf_values, s.X, s.ens, s.precision)
        grad, = torch.autograd.grad(phi, s.leaf_values, phi.detach() - s.target)
        return [phi.detach(), grad]
    if s.kind == "pairs":
        return list(s.ens.shap_interactions(s.X, s.precision, with_phi=True))
    return s.ens.shap_interactions3(s.X, s.precision)


def work(case):
    """What a pass cannot do without.  Bytes: rows and model in, results out.
    Flops: the tree walk at the method's 8 nodes, per sample and tree edge the
    factor, its product down, the sum up and the edge's node sum (7 per node);
    with pairs and triples one node sum more per update of a split with the
    features (pairs of features) split above it."""
    M, F, K = case["rows"], case["features"], case["outputs"]
    D = (case["depth"] + (case["min_depth"] or case["depth"])) / 2
    per_tree = min(2.0 ** D, case["leaves"] or 2.0 ** D)
    leaves = case["trees"] * per_tree
    edges = 2 * leaves
    mean = math.log2(per_tree) if per_tree == 2.0 ** D else 0.7 * D  # splits above a leaf
    above = F * (1 - (1 - 1 / F) ** max(0.0, mean - 1))  # other features split above a node
    size = 8 if case["precision"] == "fp64" else 4
    ops = {"values": 56 * edges, "train": 112 * edges,
           "pairs": 56 * edges + 16 * leaves * above,
           "triples": 56 * edges + 24 * leaves * above * above / 2}[case["kind"]]
    out = {"values": F, "train": 2 * F, "pairs": F * F + F,
           "triples": F * (F - 1) * (F - 2) / 6}[case["kind"]]
    model = 2 * leaves * 32 + (8 * leaves if case["kind"] == "train" else 0)
    return {"bytes": M * F * 4 + M * K * out * size + model, "flops": M * ops}


# ------------------------------------------------- the same results in 64 bits

def _paths(m):
    """Every leaf's path, collapsed to its unique features: feature, interval,
    missing-value rule and cover ratio per slot, slots by feature, and the
    number of slots; on the GPU."""
    leaf = np.flatnonzero(m.left < 0)
    D = int(m.depth[leaf].max()) if leaf.size else 0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    up, is_left, cover = dev(m.up), dev(m.is_left), dev(m.cover)
    feature, thr, dleft = dev(m.feature).long(), dev(m.threshold), dev(m.default_left).bool()
    L = leaf.size
    none = m.n_features
    feat = torch.full((L, D), none, dtype=torch.long, device="cuda")
    lo = torch.full((L, D), -math.inf, device="cuda")
    hi = torch.full((L, D), math.inf, device="cuda")
    ok = torch.ones((L, D), dtype=torch.bool, device="cuda")
    b = torch.ones((L, D), dtype=torch.float64, device="cuda")
    at = dev(leaf)
    for i in range(D):
        p = up[at]
        here = p >= 0
        p0 = p.clamp(min=0)
        f = torch.where(here, feature[p0], none)
        l = is_left[at]
        # the slot that has this feature already, or slot i
        slot = torch.full((L,), i, device="cuda")
        for k in range(i - 1, -1, -1):
            slot = torch.where(here & (feat[:, k] == f), k, slot)
        r = torch.arange(L, device="cuda")[here]
        k = slot[here]
        feat[r, k] = f[here]
        t = thr[p0]
        lo[r, k] = torch.where(l[here], lo[r, k], torch.maximum(lo[r, k], t[here]))
        hi[r, k] = torch.where(l[here], torch.minimum(hi[r, k], t[here]), hi[r, k])
        ok[r, k] &= dleft[p0][here] == l[here]
        b[r, k] *= (cover[at] / cover[p0])[here]
        at = torch.where(here, p, at)
    order = torch.argsort(feat, dim=1, stable=True)
    feat, lo, hi, ok, b = (torch.gather(v, 1, order) for v in (feat, lo, hi, ok, b))
    return SimpleNamespace(feat=feat, lo=lo, hi=hi, ok=ok, b=b, d=(feat < none).sum(1),
                           value=dev(m.value[leaf]), tree=dev(m.tree[leaf]), none=none)


def _blocks(p, X, order, cost):
    """For blocks of paths of alike length and of rows: the paths, the first
    row, and per path P, row S and slot d: follow bits [P, S, d], the weighted
    products at the nodes [P, S, n] (leaf value 1), and the ratios (o - b) / F
    at the nodes of a followed slot [P, d, n] and of another [n]."""
    M = X.shape[0]
    by = torch.argsort(p.d)
    d_of = p.d[by].cpu().numpy()
    i = int(np.searchsorted(d_of, 1))
    while i < by.numel():
        d = int(d_of[min(i + 4095, by.numel() - 1)])
        n = max(1, (d - order + 2) // 2)
        P = int(max(1, min(4096, 1.5e8 / (cost(d, n) * min(M, 64)))))
        d = int(d_of[min(i + P, by.numel()) - 1])
        k = by[i:i + P]
        i += P
        t, w = np.polynomial.legendre.leggauss(n)
        t, w = (torch.from_numpy(v).cuda() for v in ((1 + t) / 2, w / 2))
        feat, b = p.feat[k, :d], p.b[k, :d]
        use = feat < p.none
        f1 = b[:, :, None] + t * (1 - b)[:, :, None]
        r1 = torch.where(use[:, :, None], (1 - b)[:, :, None] / f1, 0.0)
        f0 = b[:, :, None] * (1 - t)
        col = feat.clamp(max=X.shape[1] - 1)
        step = int(max(1, 1.5e8 / (cost(d, n) * k.numel())))
        for s in range(0, M, step):
            x = X[s:s + step].T[col].transpose(1, 2)  # [P, S, d]
            o = (x >= p.lo[k, :d].unsqueeze(1)) & (x < p.hi[k, :d].unsqueeze(1))
            o = torch.where(x.isnan(), p.ok[k, :d].unsqueeze(1), o) | ~use.unsqueeze(1)
            h = w.expand(k.numel(), x.shape[1], n).clone()
            for j in range(d):
                h *= torch.where(o[:, :, j, None], f1[:, None, j], f0[:, None, j])
            yield k, s, feat, use, o, h, r1, -1 / (1 - t)


def _first(o, h, r1, r0):
    """Each slot's share [P, S, d] of a leaf value of 1."""
    e = torch.bmm(h, r1.transpose(1, 2).contiguous())
    return torch.where(o, e, (h * r0).sum(-1, keepdim=True))


def _phi(p, m, X, K):
    F = p.none
    phi = torch.zeros((X.shape[0], K * F), dtype=torch.float64, device="cuda")
    group = p.tree % K
    for k, s, feat, use, o, h, r1, r0 in _blocks(p, X, 1, lambda d, n: 3 * n + 4 * d):
        c = _first(o, h, r1, r0) * p.value[k, None, None] * use[:, None, :]
        c = c.transpose(0, 1).reshape(c.shape[1], -1)
        at = (group[k, None] * F + feat.clamp(max=F - 1)).reshape(-1)
        to = torch.zeros((at.numel(), K * F), dtype=torch.float64, device="cuda")
        to[torch.arange(at.numel(), device="cuda"), at] = 1.0
        phi[s:s + c.shape[0]] += c @ to
    return phi


def exact(case, seed):
    m = _model(case, seed)
    X, target = _rows(case, seed)
    p = _paths(m)
    M, F, K = case["rows"], case["features"], case["outputs"]
    if case["kind"] == "triples":
        out = torch.zeros((M, F * (F - 1) * (F - 2) // 6), dtype=torch.float64, device="cuda")
        for k, s, feat, use, o, h, r1, r0 in _blocks(p, X, 3, lambda d, n: d ** 3 + d * d * n):
            d = feat.shape[1]
            if d < 3:
                continue
            a, b, c = torch.combinations(torch.arange(d, device="cuda"), 3).T
            r = torch.where(o[..., None], r1[:, None], r0)
            t = (h[:, :, None] * r[:, :, a] * r[:, :, b] * r[:, :, c]).sum(-1)
            t *= p.value[k, None, None]
            i, j, l = (feat[:, v] for v in (a, b, c))
            at = l * (l - 1) * (l - 2) // 6 + j * (j - 1) // 2 + i
            at, keep = at.reshape(-1), (l < F).reshape(-1)
            t = t.transpose(0, 1).reshape(t.shape[1], -1)
            out[s:s + t.shape[0]].index_add_(1, at[keep], t[:, keep])
        return out
    phi = _phi(p, m, X, K)
    shape = (M, K, F) if K > 1 else (M, F)
    if case["kind"] == "values":
        return phi.reshape(shape)
    if case["kind"] == "train":
        G = phi - target.double().reshape(M, -1)
        grad = torch.zeros(p.value.numel(), dtype=torch.float64, device="cuda")
        group = p.tree % K
        for k, s, feat, use, o, h, r1, r0 in _blocks(p, X, 1, lambda d, n: 3 * n + 5 * d):
            c = _first(o, h, r1, r0) * use[:, None, :]
            at = group[k, None] * F + feat.clamp(max=F - 1)
            grad[k] += (c * G[s:s + c.shape[1]].T[at].transpose(1, 2)).sum((1, 2))
        return [phi.reshape(shape), grad]
    Phi = torch.zeros((M, F * F), dtype=torch.float64, device="cuda")
    for k, s, feat, use, o, h, r1, r0 in _blocks(p, X, 2, lambda d, n: 3 * d * d + 3 * d * n):
        P, S, d = o.shape
        r = torch.where(o[..., None], r1[:, None], r0)
        g = (r * h[:, :, None] * (p.value[k, None, None, None] / 2)).reshape(P * S, d, -1)
        t = torch.bmm(g, r.reshape(P * S, d, -1).transpose(1, 2).contiguous())
        f = feat.clamp(max=F - 1)
        at = (f[:, :, None] * F + f[:, None, :]).reshape(-1)
        keep = (use[:, :, None] & use[:, None, :] & (f[:, :, None] != f[:, None, :])).reshape(-1)
        t = t.reshape(P, S, d * d).transpose(0, 1).reshape(S, -1)
        Phi[s:s + S].index_add_(1, at[keep], t[:, keep])
    Phi = Phi.reshape(M, F, F)
    Phi.diagonal(dim1=1, dim2=2).copy_(phi - Phi.sum(2))
    return [Phi, phi]
