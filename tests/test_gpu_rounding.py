"""First order where rounding errors could add up: long sums over rows (every
path's term is added to the FP64 accumulators, so the error stays that of one
path's arithmetic however many paths share a feature), and rows that cancel
exactly (an error that all rows share would be left over)."""
import numpy as np
import pytest

import synth
from tests.parity import row_normwise

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def chain_over_fan(n_top, levels, n_trees):
    """Trees whose first n_top splits form a chain, one feature each (left: a
    leaf of value 0, right: on), above a complete tree of `levels` levels on
    one more feature with leaves of value 1: 2^(levels - 1) pairs of sibling
    leaves that share every slot but the last feature's, and that nearly all
    have the same factors for a sample."""
    n_fan = 2 ** (levels + 1) - 1
    n = 2 * n_top + n_fan
    left = np.full(n, -1, np.int32)
    right = np.full(n, -1, np.int32)
    feature = np.full(n, -1, np.int32)
    threshold = np.zeros(n, np.float32)
    cover = np.zeros(n)
    value = np.zeros(n)
    total = 2.0 ** (levels + n_top)
    for i in range(n_top):  # node i, its leaf n_top + n_fan + i
        left[i], right[i] = n_top + n_fan + i, i + 1
        feature[i] = i
        cover[i] = total / 2 ** i
        cover[n_top + n_fan + i] = cover[i] / 2
    k = np.arange(n_fan)
    level = np.floor(np.log2(k + 1)).astype(int)
    at = n_top + k
    cover[at] = total / 2.0 ** (n_top + level)
    inner = k < 2 ** levels - 1
    left[at[inner]], right[at[inner]] = n_top + 2 * k[inner] + 1, n_top + 2 * k[inner] + 2
    feature[at[inner]] = n_top
    pos = k + 1 - 2 ** level
    threshold[at[inner]] = ((2 * pos + 1) / 2.0 ** (level + 1))[inner]
    value[at[~inner]] = 1.0
    rep = lambda a: np.tile(a, n_trees)  # noqa: E731
    return synth.Ensemble(np.arange(n_trees + 1, dtype=np.int64) * n, rep(left), rep(right),
                          rep(feature), rep(threshold), np.zeros(n * n_trees, np.uint8),
                          rep(cover), rep(value), n_top + 1, 0.0, {})


@pytest.mark.parametrize("n_top", [7, 8, 12])
def test_long_sums_stay_in_fp64(oracle_mod, n_top):
    """At these sizes a wavefront walks about 4000 alike rows one after another
    (deterministic: one wavefront per workgroup).  A path's term is a product
    of up to 9 factors, each within 3 units of 2^-24, 8 node terms summed and
    three roundings more: about 40 roundings, 6 units together if they are
    independent; 2e-6 is 33.  4000 equal terms added in FP32 lose 5e-5."""
    import paper_2605_04497_amd as q
    print("case", n_top, flush=True)
    ens = chain_over_fan(n_top, 13, 16)
    rng = np.random.default_rng(n_top)
    M = 65536
    X = rng.normal(size=(M, n_top + 1)).astype(np.float32)
    X[:, n_top] = rng.random(M)
    rows = np.arange(0, M, M // 8)
    X[rows[:4], :n_top] = np.abs(X[rows[:4], :n_top])  # follow every split of the chain
    want = oracle_mod.shap_values(ens, X[rows], n=8)
    e = q.Ensemble(ens)
    Xd = torch.from_numpy(X).cuda()
    for det in (False, True):
        e.set_deterministic(det)
        got = e.shap_values(Xd, "fp32").double().cpu().numpy()[rows]
        err = row_normwise(got, want)
        print("deterministic %s: %.2e" % (det, err), flush=True)
        assert err <= 2e-6, (det, err)
    if n_top < 8:
        # the same values passed by the caller take the same walk: the same bits
        lv = torch.from_numpy(ens.leaf_values()).cuda()
        own = e.shap_values(Xd[:4096], "fp32")
        assert torch.equal(own, e.shap_values(Xd[:4096], "fp32", leaf_values=lv))
    e.close()


@pytest.mark.parametrize("precision,F,depth,n_trees", [("fp64", 10, 8, 40), ("fp64", 20, 6, 40),
                                                       ("fp32", 12, 12, 6)])
def test_rows_that_cancel(oracle_mod, precision, F, depth, n_trees):
    """Equal leaf values: every feature's value is exactly 0, and what comes out
    is rounding.  It is no more than that of the same sums term by term, in
    which a factor of the row never meets its own quotient: FP64's reference is
    the oracle's own, FP32's the walk that a call with leaf values of its own
    takes.  The walks round about as often; a quarter is for their difference
    (quotients of other nodes than the factors' give about twice)."""
    import paper_2605_04497_amd as q
    print("case", precision, F, depth, flush=True)
    ens = synth.random_small_ensemble(np.random.default_rng(7), n_trees, F, depth, n_train=20000,
                                      p_leaf=0.02)
    ens = ens.with_leaf_values(np.ones(ens.n_leaves()))
    X = np.random.default_rng(8).normal(size=(256, F)).astype(np.float32)
    e = q.Ensemble(ens)
    Xd = torch.from_numpy(X).cuda()
    rms = lambda a: float(np.sqrt(np.mean(np.square(a))))  # noqa: E731
    got = rms(e.shap_values(Xd, precision).double().cpu().numpy())
    if precision == "fp64":
        ref = rms(oracle_mod.shap_values(ens, X, n=8))
    else:
        lv = torch.ones(ens.n_leaves(), dtype=torch.float64, device="cuda")
        ref = rms(e.shap_values(Xd, precision, leaf_values=lv).double().cpu().numpy())
    print("rms %.3e, term by term %.3e" % (got, ref), flush=True)
    assert got <= 1.25 * ref
    e.close()
