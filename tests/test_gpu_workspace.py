"""The device memory an ensemble holds: the scratch kept between calls on the
default stream (calls that follow each other without waiting, from several
threads and on several streams, of growing and shrinking sizes, each against
its own result alone), and the tables that only some settings read."""
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


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_kept_scratch_grows_and_gives_way(precision):
    """Calls queued without waiting whose scratch goes through 1, 2, 4 and 8 MiB
    and past the 64 MiB that are kept, up and down, from two threads on the
    default stream of an ensemble that has none yet; then failing allocations:
    a call that cannot have its scratch returns QTS_E_OOM, and the next one
    works."""
    import paper_2605_04497_amd as q
    from paper_2605_04497_amd import _lib as L
    wl = synth.make_workload("c2_values", T=20, M=700, n_train=3000)
    # bytes of scratch: 64 a row of the table in FP64, and the FP32 call's FP64
    # accumulator of 100 features
    rows = {"fp32": [700, 2000, 1, 4000, 9000, 64, 100000, 3000, 30000, 5000],
            "fp64": [700, 64, 1, 2000]}[precision]
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    X = torch.randn((max(rows), 100), generator=g, device="cuda")
    ref = q.Ensemble(wl.ensemble)
    ref.set_deterministic(True)
    want = [ref.shap_values(X[:m], precision).clone() for m in rows]
    torch.cuda.synchronize()
    e = q.Ensemble(wl.ensemble)
    e.set_deterministic(True)
    got = {"a": [], "b": []}

    def work(name, order):
        with torch.cuda.stream(torch.cuda.default_stream()):
            for _ in range(3):
                for i in order:
                    got[name].append((i, e.shap_values(X[:rows[i]], precision)))

    up = list(range(len(rows)))
    jobs = [threading.Thread(target=work, args=("a", up)),
            threading.Thread(target=work, args=("b", up[::-1]))]
    for j in jobs:
        j.start()
    for j in jobs:
        j.join()
    torch.cuda.synchronize()
    for name in "ab":
        assert len(got[name]) == 3 * len(rows)
        for i, phi in got[name]:
            assert torch.equal(phi, want[i]), (name, rows[i])
    e.close()
    e = q.Ensemble(wl.ensemble)
    e.set_deterministic(True)
    try:
        for i in up:
            out = torch.empty_like(want[i])
            L.check(L.lib().qts_debug_fail_allocations(0))
            try:
                e.shap_values(X[:rows[i]], precision, out=out)
            except L.QtsError as err:
                assert err.code == L.QTS_E_OOM
            L.check(L.lib().qts_debug_fail_allocations(-1))
            e.shap_values(X[:rows[i]], precision, out=out)
            assert torch.equal(out, want[i]), rows[i]
    finally:
        L.lib().qts_debug_fail_allocations(-1)
    e.close()
    ref.close()


def test_kept_scratch_grows_while_another_thread_captures():
    """A call on the default stream whose scratch grows, while this process
    captures a graph on a stream of another thread, is neither refused nor ends
    the capture: it allocates in stream order."""
    import paper_2605_04497_amd as q
    wl = synth.make_workload("c2_values", T=20, M=700, n_train=3000)
    e = q.Ensemble(wl.ensemble)
    e.set_deterministic(True)
    X = torch.randn((9000, 100), device="cuda")
    want = e.shap_values(X, "fp32").clone()
    e.close()
    e = q.Ensemble(wl.ensemble)
    e.set_deterministic(True)
    e.shap_values(X[:700], "fp32")
    out = torch.empty_like(want)
    y = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    errors = []

    def call():
        try:
            with torch.cuda.stream(torch.cuda.default_stream()):
                e.shap_values(X, "fp32", out=out)
        except Exception as err:  # noqa: BLE001
            errors.append(err)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y.add_(1)
        job = threading.Thread(target=call)
        job.start()
        job.join()
        y.add_(1)
    assert not errors, errors
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    graph.replay()
    torch.cuda.synchronize()
    assert float(y.sum()) == 16.0
    e.close()


def test_plain_rows_tables_only_with_merging_off(oracle_mod):
    """The FP64 walk's tables of the unmerged rows (760 bytes a row) are built
    when merging is first turned off, in any thread and during a capture of
    another: two allocations then and none after, and a failing one leaves the
    setting as it was."""
    import paper_2605_04497_amd as q
    from paper_2605_04497_amd import _lib as L
    wl = synth.make_workload("c2_values", T=200, M=70, n_train=3000)
    X = torch.from_numpy(wl.X).cuda()
    want = oracle_mod.shap_values(wl.ensemble, wl.X, n=8)
    e = q.Ensemble(wl.ensemble)
    e.shap_values(X, "fp64")
    y = torch.zeros(8, device="cuda")
    torch.cuda.synchronize()
    errors = []

    def off():
        try:
            e.set_sibling_merge(False)
        except Exception as err:  # noqa: BLE001
            errors.append(err)

    try:
        for k in (0, 1):
            L.check(L.lib().qts_debug_fail_allocations(k))
            with pytest.raises(L.QtsError) as ei:
                e.set_sibling_merge(False)
            assert ei.value.code == L.QTS_E_OOM
        L.check(L.lib().qts_debug_fail_allocations(-1))
        merged = e.shap_values(X, "fp64").cpu().numpy()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            y.add_(1)
            L.check(L.lib().qts_debug_fail_allocations(2))
            job = threading.Thread(target=off)
            job.start()
            job.join()
        assert not errors, errors
        graph.replay()
        L.check(L.lib().qts_debug_fail_allocations(0))
        e.set_sibling_merge(True)
        e.set_sibling_merge(False)
    finally:
        L.lib().qts_debug_fail_allocations(-1)
    assert float(y.sum()) == 8.0
    plain = e.shap_values(X, "fp64").cpu().numpy()
    for got in (merged, plain):
        assert np.abs(got - want).max() <= 1e-10 * np.abs(want).max()
    e.close()
