"""2-D gradients by several steps per launch (the default for small grids, every-K and
all-levels checkpoints) in the cases that test_gpu_gradient.py holds the one-step
kernels to: the FP64 oracle with receivers on tile edges, the one-cell-per-lane kernel
bit for bit, and a workspace of NaN bytes."""
import numpy as np
import pytest

from gpu_common import cfg, f32, gpu_gradient, inputs, oracle_forward
from paper_1912_08063_amd import _lib, api, workloads as wl
from test_gpu_gradient import _check, _run_on, _setup

pytestmark = pytest.mark.gpu


def _multi(P, ckpt, monkeypatch):
    """Whether the call takes several steps per launch: it holds two more fields."""
    v, _, _, _ = inputs(P)
    prob = api.make_problem(v, P.nt, cfg(P), P.nshots, P.nrec)
    size = lambda: _lib.fwi_workspace_bytes(prob, _lib.MODE_GRADIENT, api.parse_ckpt(ckpt))
    full = size()
    with monkeypatch.context() as m:
        m.setenv("FWI_MULTI2D", "0")
        return full > size()


def test_receivers_on_tile_and_chunk_edges(monkeypatch):
    P = wl.small_2d(nz=40, nx=150, nt=120, nb=6, nshots=2, nrec=156)
    rec = [[4, x] for x in range(150)] + [[3, 53], [3, 54], [13, 117], [14, 118], [39, 149],
                                          [3, 53]]
    P.rec_pos[:] = np.array(rec, dtype=np.int32)
    P.src_pos[:] = [[20, 75], [5, 10]]
    P, obs, v0 = _setup(P)
    assert _multi(P, "every:10", monkeypatch)
    _check(P, obs, v0, "every:10")


@pytest.mark.parametrize("order", [8, 16, 2])
def test_equal_to_the_one_cell_per_lane_kernel(order, monkeypatch):
    P, obs, v0 = _setup(wl.small_2d(nz=45, nx=140, nt=150, order=order, nshots=3, nrec=33))
    P.rec_pos[1, :4] = [[0, 0], [0, 63 - 6], [44, 139], [20, 64 - 6]]
    assert _multi(P, "every:13", monkeypatch)
    got = gpu_gradient(P, v0, obs, "every:13")
    monkeypatch.setenv("FWI_DIRECT2D", "1")
    assert not _multi(P, "every:13", monkeypatch)
    ref = gpu_gradient(P, v0, obs, "every:13")
    assert got[0] == ref[0]
    assert np.array_equal(got[1], ref[1]) and np.array_equal(got[2], ref[2])


@pytest.mark.parametrize("pipe", ["0", "12"])   # tiled; two-step marching forward launches
@pytest.mark.parametrize("ckpt", ["all", "every:7", "every:12"])
def test_results_do_not_depend_on_workspace_contents(ckpt, pipe, monkeypatch):
    monkeypatch.setenv("FWI_PIPE2D", pipe)
    P = f32(wl.small_2d(nz=48, nx=131, nt=90, order=8, nshots=2, nrec=40))
    assert _multi(P, ckpt, monkeypatch)
    obs = np.asarray(oracle_forward(P), dtype=np.float32).astype(np.float64)
    v0 = np.asarray(wl.smooth(P.v, 3.0), dtype=np.float32).astype(np.float64)
    ws = api.Workspace()
    _run_on(0, P, v0, obs, ckpt, ws)          # sizes the workspace
    clean = _run_on(0, P, v0, obs, ckpt, ws)
    dirty = _run_on(255, P, v0, obs, ckpt, ws)
    for a, b in zip(clean, dirty):
        assert np.all(np.isfinite(a))
        assert np.array_equal(a, b)
