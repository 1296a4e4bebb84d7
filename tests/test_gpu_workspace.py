"""The scratch an ensemble keeps between calls on the default stream: calls that
follow each other without waiting, from several threads and on several
streams, of growing and shrinking sizes, each against its own result alone."""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_kept_scratch_is_each_call_s_own(precision):
    import paper_2605_04497_amd as q
    wl = synth.make_workload("c2_values", T=20, M=700, n_train=3000)
    e = q.Ensemble(wl.ensemble)
    X = torch.from_numpy(wl.X).cuda()
    rows = [3, 700, 64, 129, 1, 500]
    e.set_deterministic(True)  # bitwise comparable
    want = [e.shap_values(X[:m], precision).clone() for m in rows]
    torch.cuda.synchronize()
    got = {}

    def work(name, stream):
        out = []
        with torch.cuda.stream(stream):
            for _ in range(8):
                for m in rows:
                    out.append(e.shap_values(X[:m], precision))
        stream.synchronize()
        got[name] = out

    main = torch.cuda.default_stream()
    jobs = [threading.Thread(target=work, args=("a", main)),
            threading.Thread(target=work, args=("b", main)),
            threading.Thread(target=work, args=("c", torch.cuda.Stream()))]
    for j in jobs:
        j.start()
    for j in jobs:
        j.join()
    torch.cuda.synchronize()
    for name in "abc":
        assert len(got[name]) == 8 * len(rows)
        for i, phi in enumerate(got[name]):
            assert np.array_equal(phi.cpu().numpy(), want[i % len(rows)].cpu().numpy()), (name, i)
    e.close()
