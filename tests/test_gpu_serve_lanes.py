"""Launch groups of a chunk beside each other (fwi_jobs_advance): more kinds of jobs
than side streams, jobs by rounds among them, and several servers on streams and
threads of their own, give bitwise what one stream gives."""
import threading

import numpy as np
import pytest

from gpu_common import f32
from paper_1912_08063_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _requests():
    from paper_1912_08063_amd import serve
    probs = []
    for i, order in enumerate((8, 2, 4, 16)):
        probs += [("forward", None, wl.small_2d(nz=30 + i, nx=60, nt=50, order=order, seed=i)),
                  ("gradient", None, wl.small_2d(nz=24, nx=70 + i, nt=41, order=order, seed=i)),
                  ("forward", None, wl.small_3d(shape=(14, 13, 60 + i), nt=37, order=order, seed=i)),
                  ("gradient", None, wl.small_3d(shape=(12 + i, 15, 66), nt=29, order=order, seed=i))]
    probs += [("gradient", "revolve:2", wl.small_3d(shape=(12, 15, 66), nt=39, seed=6)),
              ("gradient", "revolve:3", wl.small_2d(nz=28, nx=75, nt=33, seed=4))]
    reqs = [serve.Request(i, kind, 0.0, f32(P), ckpt=ck) for i, (kind, ck, P) in enumerate(probs)]
    serve.attach_observed(reqs)
    return reqs


def _run(reqs):
    from paper_1912_08063_amd import serve
    res, rep = serve.Server(max_active=len(reqs), chunk=9, keep_outputs=True).run(reqs,
                                                                                realtime=False)
    assert rep["failed"] == 0
    return res


def _same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x.traces, y.traces)
        if x.dv is not None:
            assert np.array_equal(x.dv, y.dv) and x.misfit == y.misfit


def test_lanes_equal_one_stream(monkeypatch):
    reqs = _requests()
    monkeypatch.setenv("FWI_LANES", "1")
    ref = _run(reqs)
    assert all(np.any(r.traces) for r in ref)
    monkeypatch.delenv("FWI_LANES")
    for _ in range(2):
        _same(_run(reqs), ref)
    monkeypatch.setenv("FWI_LANES", "2")
    _same(_run(reqs), ref)


def test_lanes_of_several_threads_and_streams(monkeypatch):
    """Ten servers, more than there are sets of side streams on a device."""
    import torch
    reqs = _requests()[:6]
    monkeypatch.setenv("FWI_LANES", "1")
    ref = _run(reqs)
    monkeypatch.delenv("FWI_LANES")
    torch.cuda.synchronize()
    out, errors = {}, []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                out[i] = _run(reqs)
        except Exception as e:   # reported below, in the test's own thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(10)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for i in range(10):
        _same(out[i], ref)
