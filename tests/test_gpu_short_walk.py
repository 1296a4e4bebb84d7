"""The walks of the first-order kernel that sum products over runs of rows,
against the FP64 oracle.  Rows of at most 8 features (8 nodes): at every length of the buckets' longest row (1 to 8:
the number of root-side slots taken per run of rows runs from 0 to 4), on
irregular trees with repeated features, ties and missing values,
at sample counts around the 64-sample tile, on the merged and the plain table
and in the deterministic mode.  Longer rows: irregular deep trees of three
capacities."""
import numpy as np
import pytest

import synth
from tests.parity import check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def q():
    import paper_2605_04497_amd as q
    return q


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("depth", [1, 2, 3, 4, 5, 6, 7, 8])
def test_short_walk_matches_oracle(q, oracle_mod, depth, precision):
    rng = np.random.default_rng(100 + depth)
    for F, n_trees in ((12, 30), (max(1, depth - 1), 5)):
        print("case", depth, precision, F, flush=True)
        ens = synth.random_small_ensemble(rng, n_trees, F, depth, n_train=4000)
        e = q.Ensemble(ens)
        X = rng.normal(size=(130, F)).astype(np.float32)
        X[:, ::2] = np.round(X[:, ::2])
        for missing in (False, True):
            if missing:
                X[rng.random(X.shape) < 0.1] = np.nan
            want = oracle_mod.shap_values(ens, X, n=8)
            Xd = torch.from_numpy(X).cuda()
            for merge in (True, False):
                e.set_sibling_merge(merge)
                for m in (1, 63, 64, 65, 130):
                    got = e.shap_values(Xd[:m], precision).cpu().numpy().astype(np.float64)
                    check(got, want[:m], precision, "M=%d merge=%s" % (m, merge))
            e.set_deterministic(True)
            got = e.shap_values(Xd, precision).cpu().numpy().astype(np.float64)
            e.set_deterministic(False)
            check(got, want, precision, "deterministic")
        e.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("depth,F,leaf", [(12, 16, 0.05), (24, 40, 0.02), (64, 70, 0.0)])
def test_long_walk_matches_oracle(q, oracle_mod, depth, F, leaf, precision):
    print("case", depth, F, precision, flush=True)
    rng = np.random.default_rng(200 + depth)
    ens = synth.random_small_ensemble(rng, 4, F, depth, n_train=400, p_leaf=leaf,
                                      zero_cover=depth == 12)
    e = q.Ensemble(ens)
    assert e.info["max_unique"] > 8
    X = rng.normal(size=(70, F)).astype(np.float32)
    X[:, ::3] = np.round(X[:, ::3])
    for missing in (False, True):
        if missing:
            X[rng.random(X.shape) < 0.1] = np.nan
        want = oracle_mod.shap_values(ens, X, n=8)
        Xd = torch.from_numpy(X).cuda()
        for merge in (True, False):
            e.set_sibling_merge(merge)
            for m in (1, 64, 70):
                got = e.shap_values(Xd[:m], precision).cpu().numpy().astype(np.float64)
                check(got, want[:m], precision, "M=%d merge=%s" % (m, merge))
    e.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("F,K,M", [(20, 1, 1), (20, 3, 12), (20, 1, 13), (300, 1, 5), (300, 2, 64)])
def test_few_samples_match_oracle(q, oracle_mod, F, K, M, precision):
    """A lane per row: one sample to the rule's edges, output groups, wide
    feature spaces (feature-major accumulators), leaf values of the caller's,
    and a table of more than one workgroup's rows."""
    print("case", F, K, M, precision, flush=True)
    over = dict(groups=K) if K > 1 else {}
    wl = synth.make_workload("c2_values", T=12 * K, M=M, n_train=4000, F=F, **over)
    e = q.Ensemble(wl.ensemble)
    X = wl.X.copy()
    X[::2, ::3] = np.nan
    Xd = torch.from_numpy(X).cuda()
    v = np.random.default_rng(3).normal(size=wl.ensemble.n_leaves())
    values = oracle_mod.shap_values_grouped if K > 1 else oracle_mod.shap_values
    for leaf in (None, v):
        ens = wl.ensemble if leaf is None else wl.ensemble.with_leaf_values(leaf)
        want = values(ens, X, n=8).reshape(M, -1)
        lv = None if leaf is None else torch.from_numpy(leaf).cuda()
        got = e.shap_values(Xd, precision, leaf_values=lv).double().cpu().numpy()
        check(got.reshape(M, -1), want, precision, "leaf override %s" % (leaf is not None))
    e.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("T,F,K,M", [
    (3, 9, 1, 70),      # one chunk
    (9, 12, 1, 65),     # chunks of 32 rows
    (60, 190, 1, 130),  # one workgroup per CU
    (61, 9, 7, 1100),   # outputs of unequal row counts in one launch
    (40, 60, 1, 3000),  # several rounds
])
def test_row_chunks_match_oracle(q, oracle_mod, T, F, K, M, precision):
    """Splits of the rows between workgroups, from a single chunk to several
    rounds of them, with a ragged last chunk."""
    print("case", T, F, K, M, precision, flush=True)
    over = dict(groups=K) if K > 1 else {}
    wl = synth.make_workload("c2_values", T=T, M=M, n_train=4000, F=F, **over)
    e = q.Ensemble(wl.ensemble)
    rows = np.unique(np.r_[0:4, M // 2, M - 3:M])
    values = oracle_mod.shap_values_grouped if K > 1 else oracle_mod.shap_values
    want = values(wl.ensemble, wl.X[rows], n=8).reshape(len(rows), -1)
    got = e.shap_values(torch.from_numpy(wl.X).cuda(), precision).double().cpu().numpy()
    check(got.reshape(M, -1)[rows], want, precision, "row chunks")
    e.close()
