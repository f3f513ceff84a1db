"""Performance cases of the FWI hot path: what a user has it compute.

Every case is one call (or one served batch) through the public Python entry
points: ``api.forward``, ``api.gradient``, ``autograd.FWIForward`` and
``serve.Server``.  Grids, wavelets, receiver layouts and checkpoint policies
follow ``workloads.py``, ``bench.py`` and the tests; step counts are shorter than
a production run's, because every step costs the same.

A case is a dict of plain values:

* ``entry``: "forward", "gradient", "autograd" (a training step: loss, backward)
  or "serve" (a batch of one-shot requests);
* ``nz``, ``ny``, ``nx``: the model grid (``ny`` 0: a 2-D model);
* ``order``, ``nsponge``, ``nt``, ``shots``, ``ckpt`` as in ``api.Config``;
* ``model``: "anomaly", "smooth" or "layered"; ``rec``: "surface" (every cell of
  the row or plane at depth 4) or "random" (per shot, some on the same cell).
"""
import math

import numpy as np
import torch

from paper_1912_08063_amd import api, autograd, serve
from paper_1912_08063_amd import workloads as wl

DX = 10.0


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # The smallest call in the workloads: 500 steps of a 128 x 128 model with
        # 128 receivers.  Launches and their latency are all it is.
        dict(name="fwd2d_anomaly_128", entry="forward", nz=128, ny=0, nx=128, order=8, nsponge=20,
             nt=500, shots=1, ckpt="", model="anomaly", rec="surface"),
        # A ragged survey with scattered receivers per shot, at 4th order: the
        # sizes that no tile divides.
        dict(name="fwd2d_ragged_o4", entry="forward", nz=301, ny=0, nx=733, order=4, nsponge=17,
             nt=411, shots=5, ckpt="", model="smooth", rec="random"),
        # Modelling of a whole 2-D survey: 32 shots over 1024 x 320 in one call.
        dict(name="fwd2d_32shots", entry="forward", nz=320, ny=0, nx=1024, order=8, nsponge=20,
             nt=600, shots=32, ckpt="", model="smooth", rec="surface"),
        # The gradient of one shot of that survey: what a user who sends shot
        # after shot calls.
        dict(name="grad2d_1shot", entry="gradient", nz=320, ny=0, nx=1024, order=8, nsponge=20,
             nt=1000, shots=1, ckpt="every:50", model="smooth", rec="surface"),
        # The gradient of the whole survey in one call, with the default
        # checkpoints: an iteration of the inversion loop.
        dict(name="grad2d_32shots", entry="gradient", nz=320, ny=0, nx=1024, order=8, nsponge=20,
             nt=300, shots=32, ckpt="every:50", model="smooth", rec="surface"),
        # A training step at 16th order on an odd grid: forward with
        # checkpoints, loss, backward through the autograd function.
        dict(name="train2d_o16", entry="autograd", nz=257, ny=0, nx=509, order=16, nsponge=23,
             nt=350, shots=4, ckpt="every:25", model="smooth", rec="surface"),
        # A small 3-D crop (64^3 and its sponge), which cannot fill the GPU.
        dict(name="fwd3d_64", entry="forward", nz=64, ny=64, nx=64, order=8, nsponge=24, nt=600,
             shots=1, ckpt="", model="layered", rec="surface"),
        # The headline forward: 256^3 and its sponge, 256 x 256 receivers.
        dict(name="fwd3d_256", entry="forward", nz=256, ny=256, nx=256, order=8, nsponge=24,
             nt=500, shots=1, ckpt="", model="layered", rec="surface"),
        # The same model at 16th order.
        dict(name="fwd3d_256_o16", entry="forward", nz=256, ny=256, nx=256, order=16, nsponge=24,
             nt=200, shots=1, ckpt="", model="layered", rec="surface"),
        # The 3-D gradient on the headline grid with the default checkpoints.
        dict(name="grad3d_256", entry="gradient", nz=256, ny=256, nx=256, order=8, nsponge=24,
             nt=150, shots=1, ckpt="every:50", model="layered", rec="surface"),
        # The largest model, 512 x 512 x 256, under binomial checkpointing.
        dict(name="grad3d_salt_revolve", entry="gradient", nz=256, ny=512, nx=512, order=8,
             nsponge=24, nt=40, shots=1, ckpt="revolve:8", model="layered", rec="surface"),
        # Twelve requests of the serving stream at an eighth of its size (2-D and
        # 3-D, forwards and gradients), all waiting when the server starts: from
        # host arrays to host arrays.
        dict(name="serve_12", entry="serve", requests=12, scale=0.125),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any size between the smallest and the largest listed ones,
    odd ones among them, any order, shots, sponge, receivers and policy."""
    if rng.random() < 0.05:
        return dict(entry="serve", requests=rng.randint(4, 14), scale=rng.uniform(0.06, 0.125))
    entry = rng.choice(["forward", "forward", "gradient", "gradient", "autograd"])
    order = rng.choice([8, 8, 8, 8, 4, 16, 16, 2])
    c = dict(entry=entry, order=order, ckpt="", model=rng.choice(["smooth", "layered", "layered"]),
             rec=rng.choice(["surface", "surface", "random"]))
    if rng.random() < 0.5:
        c.update(nz=_log(rng, 64, 1200), ny=0, nx=_log(rng, 64, 1600),
                 nsponge=rng.randint(0, 40), shots=_log(rng, 1, 32), nt=_log(rng, 40, 800))
    else:
        c.update(nz=_log(rng, 40, 280), ny=_log(rng, 40, 320), nx=_log(rng, 40, 320),
                 nsponge=rng.randint(0, 26), shots=rng.choice([1, 1, 1, 2]),
                 nt=_log(rng, 30, 300))
    if entry != "forward":
        c["ckpt"] = rng.choice(["every:50", "every:50", "every:%d" % rng.randint(7, 60), "all",
                                "revolve:%d" % rng.randint(4, 30)])
    # no more work than the largest listed case, no more levels than fit
    most = 0.8 * max(work(k)["bytes"] for k in listed())
    while work(c)["bytes"] > most and c["nt"] > 8:
        c["nt"] = max(8, int(0.8 * c["nt"]))
    if c["ckpt"] == "all" and 4.0 * _cells(c) * c["shots"] * c["nt"] > 20e9:
        c["ckpt"] = "every:50"
    return c


# ----------------------------------------------------------------- the inputs
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _shape(c):
    return (c["nz"], c["ny"], c["nx"]) if c["ny"] else (c["nz"], c["nx"])


def _cells(c):
    """Cells of the padded grid."""
    return math.prod(n + 2 * c["nsponge"] for n in _shape(c))


def _blur(a, sigma):
    """Gaussian smoothing of a 2-D field along both axes."""
    for axis in range(2):
        n = a.shape[axis]
        i = torch.arange(n, device=a.device, dtype=torch.float32)
        w = torch.exp(-0.5 * ((i[:, None] - i[None, :]) / sigma) ** 2)
        w = w / w.sum(1, keepdim=True)
        a = w @ a if axis == 0 else a @ w.T
    return a


def _inputs(c, seed):
    """Velocity, wavelets, positions and (gradients) observed traces, from the
    seed alone: the value ranges and layouts of workloads.py."""
    dev, shape, S, nt = _device(), _shape(c), c["shots"], c["nt"]
    rng = np.random.default_rng([seed, c["nz"], c["nx"]])
    g = torch.Generator(device=dev)
    g.manual_seed(int(rng.integers(1 << 31)))
    if c["model"] == "smooth" and len(shape) == 2:
        a = _blur(torch.randn(shape, generator=g, device=dev), 10.0)
        v = 1500.0 + 3000.0 * (a - a.min()) / (a.max() - a.min())
    elif c["model"] == "anomaly":
        z = torch.arange(shape[0], device=dev)[:, None] - shape[0] // 2
        x = torch.arange(shape[1], device=dev)[None, :] - shape[1] // 2
        v = 2000.0 + float(rng.uniform(200, 400)) * torch.exp(-(z * z + x * x) / 128.0)
    else:
        prof = torch.as_tensor(wl.layered((shape[0],), rng, noise=0.0), device=dev)
        v = prof.reshape((-1,) + (1,) * (len(shape) - 1)) * (
            1.0 + 0.05 * torch.randn(shape, generator=g, device=dev)).clamp(0.7, 1.3)
    v = v.to(torch.float32).contiguous()
    vmax = float(v.max())
    dt = float(np.float32(wl.dt_from_cfl(vmax, DX, 0.35)))
    t = torch.arange(nt, device=dev, dtype=torch.float64) * dt
    f = float(rng.uniform(9.0, 15.0))
    src = _ricker(f, t - 1.5 / f).to(torch.float32).expand(S, nt).contiguous()
    # shots along the surface; receivers along it, or scattered
    xs = ((np.arange(S) + rng.uniform(0.3, 0.7)) * shape[-1] / S).astype(np.int64)
    src_pos = np.full((S, len(shape)), 4)
    src_pos[:, -1] = np.clip(xs, 0, shape[-1] - 1)
    if len(shape) == 3:
        src_pos[:, 1] = shape[1] // 2
    if c["rec"] == "surface":
        rec_pos = wl.surface_receivers(shape, 4)
    else:
        R = 40 + (7 * c["nz"] + 13 * c["nx"]) % 360
        rec_pos = np.stack([rng.integers(0, n, (S, R)) for n in shape], axis=2)
        rec_pos[:, -1] = rec_pos[:, 0]   # two receivers on one cell
    src_pos = torch.as_tensor(src_pos, dtype=torch.int32, device=dev)
    rec_pos = torch.as_tensor(rec_pos, dtype=torch.int32, device=dev)
    obs = None
    if c["entry"] != "forward":
        # a direct arrival and a later reflection per receiver, in the
        # amplitude range of the modelled traces
        d = (rec_pos if rec_pos.dim() == 3 else rec_pos[None]) - src_pos[:, None]
        r = d.double().pow(2).sum(-1).sqrt() * DX
        vm = float(v.mean())
        amp = 1.0 / (4.0 * math.pi * vm * vm) / (r + 10 * DX)
        if len(shape) == 2:
            amp = amp * torch.sqrt(r + 10 * DX) * math.sqrt(vm / f)
        obs = torch.empty((S, nt, r.shape[1]), device=dev)
        for s in range(S):
            lag = r[s][None] / vm + 1.5 / f
            deep = torch.sqrt(r[s][None] ** 2 + (0.8 * shape[0] * DX) ** 2) / vm + 1.5 / f
            obs[s] = amp[s] * (_ricker(f, t[:, None] - lag) + 0.2 * _ricker(f, t[:, None] - deep))
    return v, obs, src, src_pos, rec_pos, dt


def _ricker(f, t):
    a = (math.pi * f * t) ** 2
    return (1.0 - 2.0 * a) * torch.exp(-a)


def _requests(c, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(c["requests"]):
        # alternate dimension and direction, so that every batch has all four;
        # sizes are the stream's, the velocities the seed's
        force = {"dim": 2 + i % 2, "kind": "gradient" if i % 4 >= 2 else "forward"}
        kind, P = serve.make_request_problem(i, scale=c["scale"], force=force)
        v = wl.layered(P.v.shape, rng)
        P = wl._pack(P.name, v, P.dx, wl.dt_from_cfl(float(v.max()), P.dx, 0.4), P.nt, P.order,
                     P.nb, 10.0, P.src_pos, P.rec_pos)
        r = serve.Request(i, kind, 0.0, P)
        if kind == "gradient":
            lag = rng.uniform(0.0, 0.2, (1, 1, P.nrec)) + 0.15
            t = np.arange(P.nt)[None, :, None] * P.dt - lag
            a = (np.pi * 10.0 * t) ** 2
            r.obs = (1e-10 * (1 - 2 * a) * np.exp(-a)).astype(np.float32)
        out.append(r)
    return out


def prepare(case, seed):
    if case["entry"] == "serve":
        return dict(entry="serve", requests=_requests(case, seed),
                    server=serve.Server(keep_outputs=True))
    v, obs, src, src_pos, rec_pos, dt = _inputs(case, seed)
    cfg = api.Config(dt=dt, dx=DX, order=case["order"], nsponge=case["nsponge"],
                     ckpt=case["ckpt"] or "every:50")
    # the workspace is what an inversion loop keeps between its calls
    return dict(entry=case["entry"], v=v, obs=obs, src=src, src_pos=src_pos, rec_pos=rec_pos,
                cfg=cfg, ws=api.Workspace())


# ------------------------------------------------------------------- one pass
def run(state):
    s = state
    if s["entry"] == "serve":
        results, _ = s["server"].run(s["requests"], realtime=False)
        return [[r.traces] if r.kind == "forward" else [r.traces, r.dv, r.misfit]
                for r in results]
    if s["entry"] == "forward":
        return api.forward(s["v"], s["src"], s["src_pos"], s["rec_pos"], s["cfg"],
                           workspace=s["ws"])
    if s["entry"] == "gradient":
        misfit, dv = api.gradient(s["v"], s["obs"], s["src"], s["src_pos"], s["rec_pos"],
                                  s["cfg"], workspace=s["ws"])
        return {"misfit": misfit, "dv": dv}
    v = s["v"].detach().requires_grad_(True)
    traces = autograd.FWIForward.apply(v, s["src"], s["src_pos"], s["rec_pos"], s["cfg"])
    loss = ((traces - s["obs"]) ** 2).sum()
    loss.backward()
    return {"traces": traces.detach(), "loss": loss.detach(), "grad": v.grad}


# -------------------------------------------------------------------- the work
def _steps(c):
    """(forward steps, adjoint steps) that the call's policy asks for."""
    nt = c["nt"]
    if c["entry"] == "forward":
        return nt, 0
    kind, _, arg = c["ckpt"].partition(":")
    if kind == "every":
        last = (nt - 1) % int(arg) + 1 if int(arg) < nt else nt
        return nt + (nt - last), nt
    if kind == "revolve":   # binomial optimum with the given slots
        s, r = int(arg) + 1, 0
        while math.comb(s + r, s) < nt:
            r += 1
        return nt + max(0, r * nt - math.comb(s + r, s + 1) - nt + 1), nt
    return nt, nt


def work(case):
    """A time step reads two levels and the model and writes one level (an
    adjoint step reads the forward level and updates the gradient as well), each
    cell once; the model is one for all shots of a call.  Arithmetic: the star
    stencil's sums and products, the update, and the imaging condition."""
    c = case
    if c["entry"] == "serve":
        total = {"bytes": 0, "flops": 0}
        for r in _requests(c, 0):
            P = r.problem
            shape = (P.v.shape + (0,))[:3] if P.ndim == 3 else (P.v.shape[0], 0, P.v.shape[1])
            one = work(dict(entry=r.kind, nz=shape[0], ny=shape[1], nx=shape[2], order=P.order,
                            nsponge=P.nb, nt=P.nt, shots=1, ckpt="every:50", rec="", nrec=P.nrec))
            total = {k: total[k] + one[k] for k in total}
        return total
    S, n, D, M = c["shots"], _cells(c), len(_shape(c)), c["order"] // 2
    nrec = c.get("nrec") or (math.prod(_shape(c)[1:]) if c["rec"] == "surface" else 200)
    fwd, adj = _steps(c)
    model = math.prod(_shape(c))
    io = 4 * (model * (2 if adj else 1) + S * c["nt"] * (1 + nrec * (2 if adj else 1)))
    lap = (2 * D + 1) * M + 2
    return {"bytes": fwd * n * (12 * S + 4) + adj * n * (24 * S + 4) + io,
            "flops": S * n * (fwd * (lap + 4) + adj * (2 * lap + 6))}


# ----------------------------------------------------- the same in 64 bits
def _star(p, M):
    """dx^2 times the Laplacian of [S][...] fields with zeros outside."""
    D = p.dim() - 1
    f = math.factorial
    q = torch.nn.functional.pad(p, (M, M) * D)
    n = p.shape[1:]

    def at(axis, m):
        for a in range(D):
            lo = M + (m if a == axis else 0)
            yield lo, lo + n[a]
    out = torch.zeros_like(p)
    for axis in range(D):
        for m in range(1, M + 1):
            w = 2.0 * (-1.0) ** (m + 1) * f(M) ** 2 / (m * m * f(M - m) * f(M + m))
            hi = q[(slice(None),) + tuple(slice(*k) for k in at(axis, m))]
            lo = q[(slice(None),) + tuple(slice(*k) for k in at(axis, -m))]
            out.add_(hi, alpha=w).add_(lo, alpha=w).add_(p, alpha=-2.0 * w)
    return out


def _solve(v, obs, src, src_pos, rec_pos, dt, dx, order, nb, eta_max=None):
    """Traces, and with obs the misfit and the gradient of sum (traces - obs)^2."""
    dev, D, S, M = v.device, v.dim(), src_pos.shape[0], order // 2
    v, src = v.double(), src.double()
    src_pos = src_pos.long()
    rec_pos = rec_pos.long().expand(S, -1, -1) if rec_pos.dim() == 3 else \
        rec_pos.long()[None].expand(S, -1, -1)
    vp, d2 = v, 0.0
    for a, n in enumerate(v.shape):
        i = torch.arange(n + 2 * nb, device=dev)
        vp = vp.index_select(a, (i - nb).clamp(0, n - 1))
        d = torch.clamp(torch.maximum(nb - i, i - (n + nb - 1)), min=0).double()
        d2 = d2 + (d * d).reshape([-1 if b == a else 1 for b in range(D)])
    if eta_max is None:
        eta_max = 3.0 * float(v.max()) * math.log(1000.0) / (2 * nb * dx) if nb else 0.0
    e = (eta_max * dt / (nb * nb) if nb else 0.0) * d2
    alpha, beta = 1.0 / (1.0 + e), (1.0 - e) / (1.0 + e)
    kappa = (vp * dt / dx) ** 2
    shot = torch.arange(S, device=dev)
    sidx = (shot,) + tuple(src_pos[:, a] + nb for a in range(D))
    ridx = (shot[:, None],) + tuple(rec_pos[:, :, a] + nb for a in range(D))
    nt = src.shape[1]
    scale = dt * dt / dx ** D
    p = torch.zeros((S,) + tuple(kappa.shape), dtype=torch.float64, device=dev)
    q = torch.zeros_like(p)
    traces, levels = [], [p]
    for n in range(nt):
        new = 2.0 * p + kappa * _star(p, M)
        new[sidx] += scale * src[:, n]
        new = alpha * new - beta * q
        q, p = p, new
        traces.append(p[ridx])
        if obs is not None:
            levels.append(p)
    traces = torch.stack(traces, dim=1)
    if obs is None:
        return traces, None, None
    res = 2.0 * (traces - obs.double())
    x1, x2 = torch.zeros_like(p), torch.zeros_like(p)
    g = torch.zeros_like(kappa)
    for k in range(nt, 0, -1):
        if k < nt:
            g += (x1 * _star(levels[k], M)).sum(0)
        levels[k] = None
        x = alpha * (2.0 * x1 + kappa * _star(x1, M)) - beta * x2
        x.index_put_(ridx, kappa[ridx[1:]] * res[:, k - 1], accumulate=True)
        x1, x2 = x, x1
    for a, n in enumerate(v.shape):
        i = (torch.arange(n + 2 * nb, device=dev) - nb).clamp(0, n - 1)
        shape = list(g.shape)
        shape[a] = n
        g = torch.zeros(shape, dtype=torch.float64, device=dev).index_add_(a, i, g)
    return traces, float(((traces - obs.double()) ** 2).sum()), 2.0 * g / v


def exact(case, seed):
    with torch.no_grad():
        if case["entry"] == "serve":
            dev, outs = _device(), []
            for r in _requests(case, seed):
                P = r.problem
                f32 = lambda a: torch.as_tensor(np.asarray(a, np.float32), device=dev)
                tr, mis, dv = _solve(
                    f32(P.v), None if r.obs is None else f32(r.obs), f32(P.wavelet),
                    torch.as_tensor(P.src_pos, device=dev), torch.as_tensor(P.rec_pos, device=dev),
                    float(np.float32(P.dt)), float(np.float32(P.dx)), P.order, P.nb,
                    float(np.float32(P.eta_max)))
                tr = tr.cpu().numpy()
                outs.append([tr] if r.kind == "forward" else [tr, dv.cpu().numpy(), mis])
            return outs
        v, obs, src, src_pos, rec_pos, dt = _inputs(case, seed)
        tr, mis, dv = _solve(v, obs, src, src_pos, rec_pos, dt, DX, case["order"],
                             case["nsponge"])
        if case["entry"] == "forward":
            return tr
        if case["entry"] == "gradient":
            return {"misfit": mis, "dv": dv}
        return {"traces": tr, "loss": torch.tensor(mis, dtype=torch.float64), "grad": dv}
