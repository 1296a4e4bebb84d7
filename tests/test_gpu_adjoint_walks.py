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
