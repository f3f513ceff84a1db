"""2-D launches of several time steps (k_step2d_tb, k_step2d_pipe): traces,
misfit and gradient bit for bit those of one step per launch (which the other
tests hold to the FP64 oracle), at the sizes where tiles, aprons, chunks and
receiver lists have their edges."""
import numpy as np
import pytest

from gpu_common import f32, gpu_forward, gpu_gradient
from paper_1912_08063_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _problem(nz, nx, nt, order, nb, nshots=2, dense=False, seed=5):
    """Receivers on the model's corners, on a shared cell and scattered, or
    (dense) one in every cell: more than a block has threads."""
    P = wl.small_2d(nz=nz, nx=nx, nt=nt, order=order, nb=nb, seed=seed, nshots=nshots, nrec=12)
    P.rec_pos[:, :4] = [[0, 0], [0, nx - 1], [nz - 1, 0], [nz - 1, nx - 1]]
    if dense:
        z, x = np.meshgrid(np.arange(nz), np.arange(nx), indexing="ij")
        P.rec_pos = np.broadcast_to(np.stack([z.ravel(), x.ravel()], 1),
                                    (nshots, nz * nx, 2)).astype(np.int32).copy()
    P.src_pos[0] = [nz - 1, nx // 2]
    P.rec_pos[:, 4:7] = P.src_pos[:, None] // 2 * 2   # beside or at the source
    # a source that is strong from the first step, so that the few steps of these
    # runs fill the grid
    P.wavelet = 1e3 * np.random.default_rng(seed).standard_normal(P.wavelet.shape)
    return f32(P)


def _both(P, ckpt, monkeypatch, env):
    obs = np.random.default_rng(3).standard_normal((P.nshots, P.nt, P.nrec)) * 1e-9
    obs = obs.astype(np.float32).astype(np.float64)
    for k in ("FWI_MULTI2D", "FWI_TB2D", "FWI_PIPE2D"):
        monkeypatch.delenv(k, raising=False)
    monkeypatch.setenv("FWI_MULTI2D", "0")
    ref = gpu_forward(P), gpu_gradient(P, P.v, obs, ckpt)
    monkeypatch.delenv("FWI_MULTI2D")
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    got = gpu_forward(P), gpu_gradient(P, P.v, obs, ckpt)
    assert np.any(ref[0]) and np.any(ref[1][1])
    assert np.array_equal(got[0], ref[0])
    assert got[1][0] == ref[1][0]
    assert np.array_equal(got[1][1], ref[1][1])
    assert np.array_equal(got[1][2], ref[1][2])


# (nz, nx, sponge): a grid inside one region; regions that end with the grid,
# its frame and one cell past either; several tiles with ragged tails
SIZES = [(5, 7, 0), (28, 44, 4), (29, 45, 4), (27, 43, 4), (37, 101, 6), (90, 150, 0),
         (71, 219, 21)]


@pytest.mark.parametrize("shape", ["0", "1", "2", "3", "4"])
@pytest.mark.parametrize("order", [2, 4, 8, 16])
def test_tile_launches_equal_single_steps(shape, order, monkeypatch):
    for i, (nz, nx, nb) in enumerate(SIZES):
        P = _problem(nz, nx, 23 + i, order, nb)   # every remainder of 2, 3, 4 and 8 steps
        _both(P, ["every:9", "all", "every:5", "every:3", "every:2"][i % 5], monkeypatch,
              {"FWI_TB2D": shape})


@pytest.mark.parametrize("order", [2, 8, 16])
def test_more_receivers_than_threads(order, monkeypatch):
    _both(_problem(33, 60, 14, order, 3, dense=True), "every:6", monkeypatch, {})


@pytest.mark.parametrize("order", [4, 8])
@pytest.mark.parametrize("rows", ["12", "24", "48"])
def test_two_step_marching_launches_equal_single_steps(order, rows, monkeypatch):
    for i, (nz, nx, nb) in enumerate(SIZES + [(48, 104, 4), (49, 105, 4), (100, 330, 11)]):
        P = _problem(nz, nx, 30 + i, order, nb)
        _both(P, ["every:9", "every:10", "all", "every:13", "every:2"][i % 5], monkeypatch,
              {"FWI_PIPE2D": rows})
    _both(_problem(40, 140, 25, order, 5, dense=True), "every:12", monkeypatch,
          {"FWI_PIPE2D": rows})
