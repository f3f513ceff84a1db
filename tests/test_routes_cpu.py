"""Which 2-D calls take several time steps per launch, read from the workspace sizes
(no device): such a call holds two more wavefields (adjoint calls: adjoint fields)
per shot than FWI_MULTI2D=0, which keeps one step per launch."""
import ctypes

import pytest
import torch

from paper_1912_08063_amd import _lib, api


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


ALL = _lib.FwiCkpt(kind=_lib.CKPT_ALL)


@pytest.mark.parametrize("mode,ck,fields", [
    (_lib.MODE_FORWARD, None, 2), (_lib.MODE_GRADIENT, EVERY, 2), (_lib.MODE_GRADIENT, ALL, 2),
    (_lib.MODE_BACKWARD, EVERY, 2), (_lib.MODE_FORWARD_CKPT, EVERY, 0), (_lib.MODE_CKPT_BUF, EVERY, 0),
    (_lib.MODE_GRADIENT, _lib.FwiCkpt(kind=_lib.CKPT_REVOLVE, slots=3), 0)])
def test_one_step_size(mode, ck, fields, monkeypatch):
    """The flag MODE_ONE_STEP reports what FWI_MULTI2D=0 reports: the fields of
    multi-step launches less."""
    p = _prob(64, 80, order=8, nsponge=10, nshots=3)
    small = _lib.fwi_workspace_bytes(p, mode | _lib.MODE_ONE_STEP, ck)
    assert _lib.fwi_workspace_bytes(p, mode, ck) - small == fields * 3 * _field(p)
    monkeypatch.setenv("FWI_MULTI2D", "0")
    assert _lib.fwi_workspace_bytes(p, mode, ck) == small


def test_unknown_modes_stay_refused():
    p = _prob(64, 80)
    for mode in (-1, 5, 0x200, _lib.MODE_ONE_STEP | 5, 0x201):
        with pytest.raises(_lib.FwiError) as e:
            _lib.fwi_workspace_bytes(p, mode, EVERY)
        assert e.value.status == _lib.FWI_EINVAL


def test_a_workspace_of_exactly_the_one_step_size_is_accepted():
    """It passes the size check (and is refused for its NULL arrays); a byte less or
    more is FWI_ENOMEM, as every size below the full one was."""
    p = _prob(64, 80, order=8, nsponge=10)
    lib = _lib.load()
    small = _lib.fwi_workspace_bytes(p, _lib.MODE_FORWARD | _lib.MODE_ONE_STEP)
    full = _lib.fwi_workspace_bytes(p, _lib.MODE_FORWARD)

    def call(n):
        return lib.fwi_forward(ctypes.byref(p), None, None, None, None, None, 256, n, None)

    assert call(small) == call(full) == _lib.FWI_EINVAL
    for n in (0, small - 1, small + 1, small + 256, full - 1):
        assert call(n) == _lib.FWI_ENOMEM


class _Device:
    """Stands in for a device's memory: refuses allocations above `room` bytes."""

    def __init__(self, room):
        self.room, self.asked = room, []

    def empty(self, n, dtype=None, device=None):
        self.asked.append(n)
        if n > self.room:
            raise torch.cuda.OutOfMemoryError("no room")
        return torch.zeros(n, dtype=dtype)


def test_a_device_without_room_takes_the_smaller_workspace(monkeypatch):
    p = _prob(64, 80, order=8, nsponge=10)
    size = lambda flag: _lib.fwi_workspace_bytes(p, _lib.MODE_GRADIENT | flag, EVERY)
    full, small = size(0), size(_lib.MODE_ONE_STEP)
    cpu = torch.device("cpu")
    get = lambda ws: api.call_workspace(p, _lib.MODE_GRADIENT, EVERY, ws, cpu)
    dev = _Device(full - 1)
    monkeypatch.setattr(api.torch, "empty", dev.empty)
    ws = api.Workspace()
    for _ in range(2):   # and is not asked for the larger one at every call
        buf, n = get(ws)
        assert n == small and buf.numel() == small
    assert dev.asked == [full, small]
    dev.room = full
    buf, n = get(api.Workspace())
    assert n == full and buf.numel() == full
    dev.room = small - 1
    with pytest.raises(torch.cuda.OutOfMemoryError):
        get(api.Workspace())
