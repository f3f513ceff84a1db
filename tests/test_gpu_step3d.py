"""3-D step kernels: marching (k_step3d, the large grids' kernel) against the FP64
oracle and, bit for bit, against the kernel without marching (k_step3d_tile,
which small grids take), at grids with ragged tiles in x, y and z, chunks that end
inside and with a queue's unrolled group, and receivers on tile edges, on one
cell and in every cell of a plane."""
import numpy as np
import pytest

from gpu_common import (f32, gpu_forward, gpu_gradient, oracle_forward, oracle_gradient, rel_l2)
from paper_1912_08063_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _problem(shape, order, nt=33, nb=5, nshots=2, seed=8):
    P = wl.small_3d(shape=shape, nt=nt, order=order, nb=nb, seed=seed, nshots=nshots, nrec=12)
    nz, ny, nx = shape
    P.rec_pos[:, :5] = [[0, 0, 0], [nz - 1, ny - 1, nx - 1], [nz // 2, min(ny - 1, 16 - nb), 2],
                        [3, 1, min(nx - 1, 64 - order // 2 - nb)], [3, 1, 0]]
    P.rec_pos[:, 5:7] = P.src_pos[:, None]
    P.wavelet = 1e3 * np.random.default_rng(seed).standard_normal(P.wavelet.shape)
    return f32(P)


def _obs(P):
    o = 1e-9 * np.random.default_rng(4).standard_normal((P.nshots, P.nt, P.nrec))
    return o.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("order", [2, 4, 8, 16])
@pytest.mark.parametrize("shape", [(21, 19, 70), (9, 6, 118), (33, 38, 54), (4, 40, 5)])
def test_marching_equals_no_marching(order, shape, monkeypatch):
    P = _problem(shape, order)
    obs = _obs(P)
    monkeypatch.setenv("FWI_TILE3D", "100000000")
    ref = gpu_forward(P), gpu_gradient(P, P.v, obs, "every:8")
    assert np.any(ref[0]) and np.any(ref[1][1])
    monkeypatch.setenv("FWI_TILE3D", "0")
    for chunk, split in (("0", "0"), ("1", "0"), ("7", "0"), ("10", "0"), ("18", "1"), ("40", "0")):
        monkeypatch.setenv("FWI_SPLIT_ADJ", split)
        if chunk != "0":
            monkeypatch.setenv("FWI_ZCHUNK", chunk)
        got = gpu_forward(P), gpu_gradient(P, P.v, obs, "every:8")
        assert np.array_equal(got[0], ref[0]), chunk
        assert got[1][0] == ref[1][0], chunk
        assert np.array_equal(got[1][1], ref[1][1]), chunk


@pytest.mark.parametrize("kernel", ["0", "100000000"])
@pytest.mark.parametrize("order", [8, 16, 4])
def test_against_the_oracle(order, kernel, monkeypatch):
    """Relative L2 1e-4 on traces and 1e-3 on the gradient, the bars of the
    repository's parity tests."""
    monkeypatch.setenv("FWI_TILE3D", kernel)
    P = f32(wl.small_3d(shape=(24, 21, 75), nt=70, order=order, nshots=2, nrec=25))
    assert rel_l2(gpu_forward(P), oracle_forward(P)) <= 1e-4
    obs = np.asarray(oracle_forward(P), np.float32).astype(np.float64)
    v0 = np.asarray(wl.smooth(P.v, 1.5), np.float32).astype(np.float64)
    mis, dv, _ = gpu_gradient(P, v0, obs, "every:12")
    omis, odv = oracle_gradient(P, v0, obs)
    assert abs(mis - omis) <= 1e-3 * omis
    assert rel_l2(dv, odv) <= 1e-3


@pytest.mark.parametrize("kernel", ["0", "100000000"])
def test_a_receiver_in_every_cell_of_a_plane(kernel, monkeypatch):
    """More receivers in a tile's plane than a block has threads."""
    P = _problem((14, 21, 66), 8, nt=21, nshots=1)
    y, x = np.meshgrid(np.arange(21), np.arange(66), indexing="ij")
    P.rec_pos = np.stack([np.full(y.size, 4), y.ravel(), x.ravel()], 1)[None].astype(np.int32)
    obs = _obs(P)
    monkeypatch.setenv("FWI_TILE3D", kernel)
    mis, dv, tr = gpu_gradient(P, P.v, obs, "all")
    omis, odv = oracle_gradient(P, P.v, obs)
    assert rel_l2(tr, oracle_forward(P)) <= 1e-4
    assert abs(mis - omis) <= 1e-3 * omis and rel_l2(dv, odv) <= 1e-3


@pytest.mark.parametrize("order", [2, 8, 16])
def test_chunk_directions_and_order_bitwise_equal(order, monkeypatch):
    """Odd chunks marching down (the default) or up, the chunks of a column
    consecutive or not, for chunks of one plane to a short last one."""
    P = _problem((21, 19, 70), order)
    obs = _obs(P)
    monkeypatch.setenv("FWI_TILE3D", "0")
    for chunk in ("1", "7", "16", "30"):
        monkeypatch.setenv("FWI_ZCHUNK", chunk)
        runs = []
        for alt, fast in (("1", "0"), ("0", "0"), ("1", "1"), ("0", "1")):
            monkeypatch.setenv("FWI_ZALT", alt)
            monkeypatch.setenv("FWI_ZFAST", fast)
            runs.append((gpu_forward(P), gpu_gradient(P, P.v, obs, "every:8")))
        assert np.any(runs[0][0]) and np.any(runs[0][1][1])
        for tr, (mis, dv, _) in runs[1:]:
            assert np.array_equal(tr, runs[0][0]), chunk
            assert mis == runs[0][1][0] and np.array_equal(dv, runs[0][1][1]), chunk
