"""The adjoint's walks over rows of at most 8 features, against the oracle's
transposed map."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def q():
    import paper_2605_04497_amd as q
    return q


@pytest.mark.parametrize("precision", ["fp64"])
@pytest.mark.parametrize("F,depth", [(12, 3), (12, 6), (12, 8), (300, 6)])
def test_infinite_upstream_gradient(q, oracle_mod, F, depth, precision):
    """An infinite gradient at one sample and feature makes the gradients of
    the leaves whose paths have the feature infinite, by the sign of their
    derivative, and leaves the others as they are."""
    print("case", F, depth, precision, flush=True)
    rng = np.random.default_rng(F + depth)
    ens = synth.random_small_ensemble(rng, 12, F, depth, n_train=4000)
    X = rng.normal(size=(70, F)).astype(np.float32)
    G = rng.normal(size=X.shape)
    used = np.unique(ens.feature[ens.feature >= 0])
    e = q.Ensemble(ens)
    Xd = torch.from_numpy(X).cuda()
    for s, f, v in ((0, used[0], np.inf), (67, used[-1], -np.inf)):
        one = np.zeros_like(G)
        one[s, f] = 1.0
        J = oracle_mod.leaf_grad(ens, X, one)
        rest = G.copy()
        rest[s, f] = 0.0
        want = oracle_mod.leaf_grad(ens, X, rest)
        hit = J != 0
        assert hit.any() and not hit.all()
        Gi = G.copy()
        Gi[s, f] = v
        Gd = torch.from_numpy(Gi).cuda()
        for merge in (True, False):
            e.set_sibling_merge(merge)
            for det in (False, True):
                e.set_deterministic(det)
                got = e.shap_backward(Xd, Gd, precision).cpu().numpy()
                assert np.array_equal(got[hit], v * np.sign(J[hit])), (merge, det)
                assert np.abs(got[~hit] - want[~hit]).max() <= 1e-10 * np.abs(want[~hit]).max()
    e.close()


TOL = {"fp32": 1e-5, "fp64": 1e-10}  # of the largest gradient


def normwise(got, want):
    return float(np.abs(got - want).max() / np.abs(want).max())


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("depth", [1, 2, 3, 4, 5, 6, 7, 8])
def test_longest_rows_of_every_length(q, oracle_mod, depth, precision):
    """The kernel's instance follows the longest row of the table (5 to 8
    features: 1 to 4 root-side slots): irregular trees with repeated features,
    ties and missing values, around the 64-sample block, the merged and the
    plain table."""
    print("case", depth, precision, flush=True)
    rng = np.random.default_rng(300 + depth)
    for F in (12, max(1, depth)):
        ens = synth.random_small_ensemble(rng, 30, F, depth, n_train=4000)
        e = q.Ensemble(ens)
        X = rng.normal(size=(130, F)).astype(np.float32)
        X[:, ::2] = np.round(X[:, ::2])
        X[rng.random(X.shape) < 0.1] = np.nan
        G = rng.normal(size=X.shape).astype(np.float32).astype(np.float64)
        Xd = torch.from_numpy(X).cuda()
        Gd = torch.from_numpy(G).cuda()
        for m in (1, 63, 65, 130):
            want = oracle_mod.leaf_grad(ens, X[:m], G[:m])
            for merge in (True, False):
                e.set_sibling_merge(merge)
                got = e.shap_backward(Xd[:m], Gd[:m], precision).cpu().numpy()
                assert normwise(got, want) <= TOL[precision], (F, m, merge)
        e.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("T,F,M", [(500, 60, 4096), (40, 209, 192)])
def test_leaf_sums_over_sample_blocks(q, oracle_mod, T, F, M, precision):
    """Over 8192 pairs of row chunk and sample block, a workgroup takes several
    blocks and keeps its leaf sums over them (500 trees of depth 8, 64 blocks);
    at 209 features FP64's tiles leave no room for the sums.  The rows repeat
    64 distinct ones, so the oracle takes those with their gradients added."""
    print("case", T, F, M, precision, flush=True)
    wl = synth.make_workload("c2_values", T=T, M=64, n_train=4000, F=F)
    X = np.tile(wl.X, (M // 64, 1))
    G = np.random.default_rng(4).normal(size=X.shape).astype(np.float32).astype(np.float64)
    want = oracle_mod.leaf_grad(wl.ensemble, wl.X, G.reshape(M // 64, 64, F).sum(0))
    e = q.Ensemble(wl.ensemble)
    got = e.shap_backward(torch.from_numpy(X).cuda(), torch.from_numpy(G).cuda(), precision)
    assert normwise(got.cpu().numpy(), want) <= TOL[precision]
    e.close()
