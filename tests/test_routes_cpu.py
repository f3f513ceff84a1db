"""Which 2-D calls take several time steps per launch, read from the workspace sizes
(no device): such a call holds two more wavefields (adjoint calls: adjoint fields)
per shot than FWI_MULTI2D=0, which keeps one step per launch."""
import pytest

from paper_1912_08063_amd import _lib


def _prob(nz, nx, order=16, nsponge=0, nshots=1, nt=200, ndim=2):
    p = _lib.FwiProblem()
    p.ndim, p.dx, p.dt, p.nt, p.order, p.nsponge = ndim, 10.0, 1e-3, nt, order, nsponge
    p.shape[0], p.shape[1] = nz, nx
    p.eta_max, p.nshots, p.nrec = -1.0, nshots, 7
    return p


def _field(p):
    """Bytes of one wavefield."""
    M, nb = p.order // 2, p.nsponge
    pitch = (p.shape[1] + 2 * nb + 2 * M + 63) // 64 * 64
    return 4 * pitch * (p.shape[0] + 2 * nb + 2 * M)


EVERY = _lib.FwiCkpt(kind=_lib.CKPT_EVERY, every=50)


def _extra(p, mode, monkeypatch):
    """Wavefields per shot that multi-step launches add."""
    ck = None if mode == _lib.MODE_FORWARD else EVERY
    monkeypatch.delenv("FWI_MULTI2D", raising=False)
    full = _lib.fwi_workspace_bytes(p, mode, ck)
    monkeypatch.setenv("FWI_MULTI2D", "0")
    one = _lib.fwi_workspace_bytes(p, mode, ck)
    monkeypatch.delenv("FWI_MULTI2D")
    n, rest = divmod(full - one, _field(p) * p.nshots)
    assert rest == 0
    return n


# padded grids at 16th order and the 64 x 48 regions they give (32 x 16 cells each);
# forward and gradient by several steps per launch or not
@pytest.mark.parametrize("nz,nx,shots,forward,gradient", [
    (261, 509, 1, True, True),      # 256 regions: one round of the CUs
    (293, 477, 1, True, False),     # 270
    (327, 525, 1, True, False),     # 320
    (389, 477, 1, True, True),      # 360
    (485, 541, 1, True, True),      # 510
    (416, 666, 1, False, False),    # 546: a third round
    (460, 640, 1, False, False),    # 588
    (85, 157, 12, True, True),      # 300 in 12 shots
    (165, 157, 12, False, False),   # 600 (more than 300 k cells as well)
    (303, 555, 4, True, True),      # 128 x 64 regions
])
def test_16th_order_goes_by_rounds_of_regions(nz, nx, shots, forward, gradient, monkeypatch):
    p = _prob(nz, nx, nshots=shots)
    assert _extra(p, _lib.MODE_FORWARD, monkeypatch) == (2 if forward else 0)
    assert _extra(p, _lib.MODE_GRADIENT, monkeypatch) == (2 if gradient else 0)
    # the two halves of a differentiable forward agree on the checkpoint buffer
    assert _extra(p, _lib.MODE_BACKWARD, monkeypatch) == (2 if gradient else 0)
    assert _extra(p, _lib.MODE_CKPT_BUF, monkeypatch) == 0


@pytest.mark.parametrize("nz,nx", [(64, 80), (900, 1200), (1900, 1700)])
def test_jobs_hold_no_fields_of_multi_step_launches(nz, nx, monkeypatch):
    """Serving jobs step one level per launch: two forward fields and two adjoint ones,
    which is the footprint that admits them."""
    p = _prob(nz, nx, order=8, nsponge=20)
    got = (_lib.fwi_job_bytes(p, _lib.JOB_FORWARD, 50), _lib.fwi_job_bytes(p, _lib.JOB_GRADIENT, 50),
           _lib.fwi_job_bytes(p, _lib.JOB_GRADIENT, 50, _lib.FwiCkpt(kind=_lib.CKPT_ALL)))
    monkeypatch.setenv("FWI_MULTI2D", "0")
    ck = _lib.FwiCkpt(kind=_lib.CKPT_ALL)
    assert got == (_lib.fwi_workspace_bytes(p, _lib.MODE_FORWARD),
                   _lib.fwi_workspace_bytes(p, _lib.MODE_GRADIENT, EVERY),
                   _lib.fwi_workspace_bytes(p, _lib.MODE_GRADIENT, ck))


@pytest.mark.parametrize("direct", ["0", "1"])
def test_naming_a_one_step_kernel_keeps_one_step_per_launch(direct, monkeypatch):
    """FWI_DIRECT2D=0/1 forces the marching or the one-cell-per-lane kernel."""
    p = _prob(64, 80, order=8, nsponge=10)
    assert _extra(p, _lib.MODE_GRADIENT, monkeypatch) == 2
    monkeypatch.setenv("FWI_DIRECT2D", direct)
    for mode in (_lib.MODE_FORWARD, _lib.MODE_GRADIENT, _lib.MODE_BACKWARD):
        assert _extra(p, mode, monkeypatch) == 0
