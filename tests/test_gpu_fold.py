"""The transposed edge padding of the gradient (k_fold_x / k_fold_y / k_fold_z) at
the widths where its tasks end (256 columns), at grids of one to three cells across
and at sponges wider than a wave's 64 lanes, against the FP64 oracle at the
repository's bar for gradients (relative L2 1e-3), over all cells and over the
edge cells alone, which sum their part of the sponge."""
import numpy as np
import pytest

from gpu_common import f32, gpu_gradient, oracle_forward, oracle_gradient, rel_l2
from paper_1912_08063_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _check(P):
    P = f32(P)
    obs = np.asarray(0.9 * oracle_forward(P), np.float32).astype(np.float64)
    _, want = oracle_gradient(P, P.v, obs)
    _, got, _ = gpu_gradient(P, P.v, obs, "every:9")
    assert np.any(want) and rel_l2(got, want) <= 1e-3
    for axis in range(want.ndim):
        for i in (0, -1):
            a, b = np.take(got, i, axis), np.take(want, i, axis)
            # (an edge the waves have not reached holds products below the range of
            # fp32, 1e-52 in the oracle: nothing to compare)
            if np.max(np.abs(b)) > 1e-12 * np.max(np.abs(want)):
                assert rel_l2(a, b) <= 1e-3, (axis, i)


@pytest.mark.parametrize("nx", [1, 2, 3, 255, 256, 257, 300])
@pytest.mark.parametrize("nb", [3, 70])
def test_fold_2d(nx, nb):
    P = wl.small_2d(nz=9, nx=max(nx, 2), nt=60, nb=nb, nshots=2, nrec=7)
    P.v, P.src_pos, P.rec_pos = P.v[:, :nx].copy(), P.src_pos % [9, nx], P.rec_pos % [9, nx]
    P.src_pos[0] = [1, nx - 1]
    _check(P)


@pytest.mark.parametrize("shape,nb", [((2, 3, 257), 5), ((3, 1, 70), 6), ((5, 9, 2), 65)])
def test_fold_3d(shape, nb):
    full = tuple(max(n, 2) for n in shape)
    P = wl.small_3d(shape=full, nt=40, nb=nb, nshots=1, nrec=6)
    nz, ny, nx = shape
    P.v = P.v[:nz, :ny, :nx].copy()
    P.src_pos, P.rec_pos = P.src_pos % list(shape), P.rec_pos % list(shape)
    _check(P)
