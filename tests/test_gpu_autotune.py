"""qts_autotune keeps what an untuned call does where that is the faster: a
tuned ensemble's call at the tuned row count is not slower."""
import statistics

import numpy as np
import pytest

import synth
from tests.parity import check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _us(fn):
    for _ in range(20):
        fn()
    out = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            fn()
        b.record()
        b.synchronize()
        out.append(a.elapsed_time(b) / 20 * 1e3)
    return statistics.median(out)


@pytest.mark.parametrize("kind,T,depth,F,K,M", [
    ("values", 28, 5, 9, 1, 5537),
    ("values", 56, 6, 12, 7, 4100),
    ("backward", 28, 5, 9, 1, 5537),
    ("interactions", 60, 8, 40, 1, 200),
])
def test_tuned_call_is_not_slower(oracle_mod, kind, T, depth, F, K, M):
    """An eighth and 1 us are for the noise of timing calls of 20 to 70 us."""
    import paper_2605_04497_amd as q
    print("case", kind, T, depth, F, K, M, flush=True)
    rng = np.random.default_rng(5)
    ens = synth.random_small_ensemble(rng, T, F, depth, n_train=4000, p_leaf=0.0)
    if K > 1:
        ens = ens.with_groups(np.arange(T) % K, K)
    Xh = rng.normal(size=(M, F)).astype(np.float32)
    X = torch.from_numpy(Xh).cuda()
    plain, tuned = q.Ensemble(ens), q.Ensemble(ens)
    tuned.autotune(M, "fp32")
    G = torch.randn((M, K, F) if K > 1 else (M, F), device="cuda")
    run = {"values": lambda e: e.shap_values(X), "backward": lambda e: e.shap_backward(X, G),
           "interactions": lambda e: e.shap_interactions(X)}[kind]
    t = _us(lambda: run(plain)), _us(lambda: run(tuned))
    print("untuned %.1f us, tuned %.1f us" % t, flush=True)
    assert t[1] <= 1.125 * t[0] + 1
    if kind == "values":
        rows = np.arange(0, M, M // 16)
        values = oracle_mod.shap_values_grouped if K > 1 else oracle_mod.shap_values
        want = values(ens, Xh[rows], n=8).reshape(len(rows), -1)
        got = run(tuned).double().cpu().numpy().reshape(M, -1)[rows]
        check(got, want, "fp32", "tuned")
    plain.close()
    tuned.close()
