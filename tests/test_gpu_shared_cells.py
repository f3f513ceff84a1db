"""2-D calls with many receivers on one cell: traces, misfit and gradient bit for
bit those of one step per launch, and a forward that is not held up by them."""
import time

import numpy as np
import pytest

from gpu_common import cfg, f32, gpu_forward, gpu_gradient, inputs
from paper_1912_08063_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _problem(cells, nrec=1000, nt=100, order=8, nshots=1, nz=128, nx=128):
    """nrec receivers over `cells` cells of the model, in turn."""
    P = wl.small_2d(nz=nz, nx=nx, nt=nt, order=order, nshots=nshots, nrec=nrec)
    at = np.arange(nrec) % cells
    P.rec_pos[:] = np.stack([4 + at // 60 * 3, 5 + at % 60], 1)
    P.src_pos[:] = [5, 6]   # beside them: the first steps reach them
    return f32(P)


# 1, 2 and 37 cells of 300 receivers; a call of one launch, and one of several
# segments and of two-step marching launches (FWI_PIPE2D)
@pytest.mark.parametrize("cells,nt", [(1, 3), (2, 50), (37, 51)])
@pytest.mark.parametrize("pipe", ["0", "12"])
def test_traces_and_gradient_equal_single_steps(cells, nt, pipe, monkeypatch):
    P = _problem(cells, nrec=300, nt=nt, nshots=3, nz=70, nx=90)
    P.wavelet = 1e3 * np.random.default_rng(2).standard_normal(P.wavelet.shape)
    P = f32(P)
    obs = 1e-9 * np.random.default_rng(3).standard_normal((P.nshots, P.nt, P.nrec))
    obs = obs.astype(np.float32).astype(np.float64)
    monkeypatch.setenv("FWI_MULTI2D", "0")
    ref = gpu_forward(P), gpu_gradient(P, P.v, obs, "every:17")
    monkeypatch.delenv("FWI_MULTI2D")
    monkeypatch.setenv("FWI_PIPE2D", pipe)
    got = gpu_forward(P), gpu_gradient(P, P.v, obs, "every:17")
    assert np.any(ref[0]) and np.any(ref[1][1])
    assert np.array_equal(got[0], ref[0])
    assert got[1][0] == ref[1][0]
    assert np.array_equal(got[1][1], ref[1][1]) and np.array_equal(got[1][2], ref[1][2])


def test_a_shared_cell_does_not_hold_up_the_forward():
    """1000 receivers on one cell against 1000 on cells of their own: at most three
    times the time (about equal; a walk over the cell's receivers at every step made
    it 25 times)."""
    import torch
    from paper_1912_08063_amd import api

    def best(P):
        v, w, s, r = inputs(P)
        ws, c = api.Workspace(), cfg(P)
        times = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            api.forward(v, w, s, r, c, workspace=ws)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        return min(times)

    apart, shared = best(_problem(1000)), best(_problem(1))
    assert shared <= 3 * apart, (shared, apart)
