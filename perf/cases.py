"""Workloads whose time this repository watches, from one small shot to the largest grids.

A case is one call sequence of a user's program through the public entry points: a
forward shot (``Solver.run``) or a propagation from a given wavefield
(``Solver.write_field`` and ``Solver.step``), the velocity gradient through
``wave_forward`` and autograd, and a batch of requests through ``ShotServer``.
Grids are (nx, ny, nz) with x fastest.  Every case uses the default create-time
tuning; the solver of a shot is made in ``prepare`` (one model serves many
shots), the gradient and the server make theirs inside the pass, as their
users' programs do.

``exact`` computes the same outputs in float64 from plain torch slices.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2404_04441_amd import Solver
from paper_2404_04441_amd.autograd import Geometry, wave_forward
from paper_2404_04441_amd.serve import GpuBackend, ShotRequest, ShotServer

H = 10.0                       # grid spacing, m
COURANT = 0.22642776165920997  # v_max dt / h: half the stability limit of the 3D scheme
V_LO, V_HI = 1500.0, 4500.0    # m/s
SPONGE_ALPHA = 0.015


def _forward(name, nx, ny, nz, nt, storage="f32", model_bits=32, sponge=0, cpml=0, graph=0, rec="line", start="rest"):
    return dict(name=name, kind="forward", nx=nx, ny=ny, nz=nz, nt=nt, storage=storage, model_bits=model_bits,
                sponge=sponge, cpml=cpml, graph=graph, rec=rec, start=start)


def _gradient(name, nx, ny, nz, nt, sponge, rec):
    return dict(name=name, kind="gradient", nx=nx, ny=ny, nz=nz, nt=nt, sponge=sponge, rec=rec)


def _serve(name, classes, nt):
    return dict(name=name, kind="serve", classes=classes, nt=nt)


def listed():
    return [
        # the small workload, a whole shot: steps of a few microseconds, where latency counts
        _forward("small-64", 64, 64, 64, 200),
        # a request of the smallest serving class, replayed in graphs of 20 steps as the server does
        _forward("shot-128-graph", 128, 128, 128, 200, sponge=20, graph=20),
        # the 256 x 192 x 128 serving class in half storage
        _forward("shot-256x192x128-f16", 256, 192, 128, 200, storage="f16", sponge=20, graph=20),
        # an odd grid with scattered receivers: no row is aligned
        _forward("ragged-301x211x157", 301, 211, 157, 100, sponge=12, rec="list", start="field"),
        # the largest serving class, float32
        _forward("shot-384", 384, 384, 384, 100, sponge=20, start="field"),
        # the benchmark's shot: sponge and a plane of 262144 receivers
        _forward("large-512", 512, 512, 512, 100, sponge=20, rec="plane", start="field"),
        # the same grid inside absorbing layers
        _forward("cpml-512", 512, 512, 512, 100, cpml=20, rec="plane"),
        # the same grid in half storage
        _forward("large-512-f16", 512, 512, 512, 100, storage="f16", sponge=20, rec="plane", start="field"),
        # a grid between the powers of two
        _forward("shot-768", 768, 768, 768, 40, start="field"),
        # the largest grid, in the smallest storage
        _forward("precision-1024-bf16m", 1024, 1024, 1024, 30, storage="bf16", model_bits=16, start="field"),
        # one iteration of an inversion: traces, misfit and velocity gradient through autograd
        _gradient("gradient-256", 256, 256, 256, 100, 0, "plane"),
        # requests of the three smaller serving classes together, both storages
        _serve("serve-mix", "128x128x128 f32, 256x192x128 f16, 256x256x256 f32, 128x128x128 f16, 256x192x128 f32", 500),
    ]


_LARGEST = 3.2e11  # bytes of the largest listed case: no drawn one costs more


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def side(lo, hi):  # half of the grids are laid out in whole vectors, the others as they come
        n = log_int(lo, hi)
        return max(lo, n // 4 * 4) if rng.random() < 0.5 else n

    kind = rng.choice(["forward"] * 6 + ["cpml", "gradient", "gradient", "serve"])
    if kind == "serve":
        classes = []
        for _ in range(rng.randint(2, 4)):
            classes.append("%dx%dx%d %s" % (side(64, 256), log_int(64, 256), log_int(64, 256), rng.choice(["f32", "f16"])))
        return _drop_name(_serve("", ", ".join(classes), rng.randint(200, 500)))
    if kind == "gradient":
        nx, ny, nz = side(48, 256), log_int(48, 256), log_int(48, 256)
        return _drop_name(_gradient("", nx, ny, nz, rng.randint(40, 120), rng.choice([0, 20]), rng.choice(["plane", "list"])))
    hi = 512 if kind == "cpml" else 896
    nx, ny, nz = side(56, hi), log_int(56, hi), log_int(56, hi)
    storage = "f32" if kind == "cpml" else rng.choice(["f32", "f32", "f16", "bf16"])
    nt = max(10, min(200, int(_LARGEST / 2 / (16.0 * nx * ny * nz)) // 10 * 10))
    return _drop_name(_forward(
        "", nx, ny, nz, nt, storage=storage, model_bits=rng.choice([32, 16]) if storage != "f32" else 32,
        sponge=0 if kind == "cpml" else rng.choice([0, 20]), cpml=20 if kind == "cpml" else 0,
        graph=rng.choice([0, 20]) if nt % 20 == 0 else 0, rec=rng.choice(["line", "plane", "list"]),
        start="rest" if kind == "cpml" else ("field" if nt < 60 else rng.choice(["rest", "field"]))))


def _drop_name(case):
    return {k: v for k, v in case.items() if k != "name"}


# ------------------------------------------------------------ inputs


def _waves(shape, gen, device, modes, lo, hi, phase=0.0):
    """Sum of plane waves of lo..hi periods per 512 nodes (float32), largest magnitude near 1."""
    nz, ny, nx = shape
    out = torch.zeros(shape, dtype=torch.float32, device=device)
    amps = gen.uniform(0.5, 1.0, size=modes)
    for a in amps:
        k = gen.uniform(lo, hi, size=3) * gen.choice([-1.0, 1.0], size=3) * (2 * math.pi / 512)
        ph = gen.uniform(0, 2 * math.pi)
        X, Y, Z = (torch.arange(n, dtype=torch.float64, device=device) * float(q) for n, q in zip((nx, ny, nz), k))
        Z = Z + ph + phase * float(np.linalg.norm(k))
        cyx = (torch.cos(Y)[:, None] * torch.cos(X) - torch.sin(Y)[:, None] * torch.sin(X)).float()
        syx = (torch.sin(Y)[:, None] * torch.cos(X) + torch.cos(Y)[:, None] * torch.sin(X)).float()
        w = float(a / amps.sum())
        out.addcmul_(torch.cos(Z).float()[:, None, None], cyx, value=w)
        out.addcmul_(torch.sin(Z).float()[:, None, None], syx, value=-w)
    return out


def _model(shape, gen, device, lo=V_LO, hi=V_HI):
    """A smooth velocity model between lo and hi m/s."""
    return _waves(shape, gen, device, 5, 0.5, 4.0).mul_(0.5 * (hi - lo)).add_(0.5 * (hi + lo)).clamp_(lo, hi)


def _ricker(nt, dt, f0):
    tau = np.arange(nt) * dt - 1.0 / f0
    a = (math.pi * f0 * tau) ** 2
    return (1.0 - 2.0 * a) * np.exp(-a)


def _receivers(kind, nx, ny, nz, gen):
    if kind == "line":
        r = np.zeros((nx, 3), dtype=np.int32)
        r[:, 0], r[:, 1], r[:, 2] = np.arange(nx), ny // 2, min(4, nz - 1)
        return r
    if kind == "plane":
        yy, xx = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
        return np.stack([xx.ravel(), yy.ravel(), np.full(nx * ny, min(4, nz - 1))], axis=1).astype(np.int32)
    far = np.stack([gen.integers(0, n, size=236) for n in (nx, ny, nz)], axis=1)
    near = np.array([nx // 2, ny // 2, min(10, nz // 2)]) + gen.integers(-16, 17, size=(64, 3))  # around the source
    return np.clip(np.concatenate([far, near]), 0, np.array([nx, ny, nz]) - 1).astype(np.int32)


def _sponge_table(n, W, device):
    d = np.minimum(np.arange(n), n - 1 - np.arange(n))
    return torch.tensor(np.where(d < W, np.exp(-(SPONGE_ALPHA * (W - d)) ** 2), 1.0), device=device)


def _sponge(shape, W, device, dtype):
    gz, gy, gx = (_sponge_table(n, W, device).to(dtype) for n in shape)
    return gz[:, None, None] * gy[None, :, None] * gx[None, None, :]


def _inputs(case, seed, device):
    """What both the framework and the float64 computation are given."""
    gen = np.random.default_rng(seed)
    s = SimpleNamespace()
    if case["kind"] == "serve":
        s.requests = []
        for i, text in enumerate(case["classes"].split(", ")):
            grid, storage = text.split(" ")
            nx, ny, nz = (int(v) for v in grid.split("x"))
            layers = int(gen.integers(2, 7))
            depths = np.sort(gen.choice(np.arange(1, nz), size=layers - 1, replace=False))
            vels = np.sort(gen.uniform(V_LO, V_HI, size=layers)).astype(np.float32)
            s.requests.append(ShotRequest(
                id=i, arrival=0.0, shape=(nz, ny, nx), nt=case["nt"], storage=storage, h=H, dt=COURANT * H / V_HI,
                src=(nx // 2, ny // 2, 4), rec=_receivers("line", nx, ny, nz, gen), f0=15.0, t0=1.0 / 15.0,
                velocity=vels[np.searchsorted(depths, np.arange(nz), side="right")]))
        return s
    nx, ny, nz, nt = case["nx"], case["ny"], case["nz"], case["nt"]
    shape = (nz, ny, nx)
    gradient = case["kind"] == "gradient"
    lo, hi = (2000.0, 3000.0) if gradient else (V_LO, V_HI)
    s.dt = COURANT * H / hi
    s.vel = _model(shape, gen, device, lo, hi)
    s.rec = _receivers(case["rec"], nx, ny, nz, gen)
    s.src = (nx // 2, ny // 2, min(10, nz // 2))
    f0 = 25.0 if nt <= 200 else 15.0
    s.wavelet = torch.tensor(_ricker(nt, s.dt, f0) * gen.uniform(0.5, 2.0), dtype=torch.float32, device=device)
    if gradient:  # observed traces: a pulse of the traces' size that arrives later at some receivers
        delay = gen.uniform(0.0, 0.5 * nt, size=len(s.rec))
        tau = torch.arange(nt, device=device, dtype=torch.float64)[:, None] - torch.tensor(delay, device=device)
        s.obs = (2e-11 * torch.exp(-((tau - 0.25 * nt) / 8.0) ** 2)).float()
    elif case["start"] == "field":  # a wavefield that fills the grid and its previous time level
        state = gen.bit_generator.state
        s.cur = _waves(shape, gen, device, 3, 10.0, 50.0)
        gen.bit_generator.state = state
        s.prev = _waves(shape, gen, device, 3, 10.0, 50.0, phase=3000.0 * s.dt / H)
        s.wavelet = s.wavelet * 1e9  # a source of the field's size
    return s


def prepare(case, seed):
    device = torch.device("cuda", torch.cuda.current_device())
    s = _inputs(case, seed, device)
    s.case = case
    if case["kind"] == "serve":
        s.backend = GpuBackend(device=device, graph_steps=20)
        s.backend.pretune(s.requests)
        return s
    if case["kind"] == "gradient":
        s.vel.requires_grad_(True)
        s.geometry = Geometry(h=H, dt=s.dt, nt=case["nt"], src=s.src, rec=s.rec, sponge_width=case["sponge"])
        return s
    s.solver = Solver(s.vel, H, s.dt, src=s.src, rec=s.rec, sponge_width=case["sponge"], storage=case["storage"],
                      model_bits=case["model_bits"], cpml_width=case["cpml"], cpml_f0=15.0 if case["cpml"] else 0.0,
                      graph_steps=case["graph"])
    s.traces = torch.empty((case["nt"], len(s.rec)), dtype=torch.float32, device=device)
    s.field = torch.empty((case["nz"], case["ny"], case["nx"]), dtype=torch.float32, device=device)
    s.vel = None  # the solver has its own copy
    if case["start"] == "field" and case["storage"] != "f32":  # 16-bit storage is given V = A - g A_prev
        s.prev = s.cur - s.prev * _sponge(s.cur.shape, case["sponge"], device, torch.float32)
    return s


def run(s):
    case = s.case
    if case["kind"] == "serve":
        server = ShotServer(s.backend, budget_bytes=32 << 30, max_slots=8, chunk_steps=200)
        results = server.run(s.requests)
        return [results[r.id].traces for r in s.requests]
    if case["kind"] == "gradient":
        s.vel.grad = None
        traces = wave_forward(s.vel, s.wavelet, s.geometry)
        loss = 0.5 * ((traces - s.obs) ** 2).sum()
        loss.backward()
        return {"traces": traces.detach(), "grad": s.vel.grad}
    if case["start"] == "rest":
        s.solver.run(case["nt"], s.wavelet, s.traces)
    else:
        s.solver.reset()
        s.solver.write_field(0, s.cur)
        s.solver.write_field(1 if case["storage"] == "f32" else 2, s.prev)
        s.solver.step(case["nt"], s.wavelet, s.traces)
    return {"traces": s.traces, "field": s.solver.read_field(0, s.field)}


def work(case):
    """One pass: every step reads its fields and its model once and writes the new level once."""
    flops = 45.0  # a node and step: 25 points, leapfrog, sponge
    if case["kind"] == "serve":
        b = f = 0.0
        for text in case["classes"].split(", "):
            grid, storage = text.split(" ")
            n = float(np.prod([int(v) for v in grid.split("x")])) * case["nt"]
            b += n * (16 if storage == "f32" else 12)
            f += n * flops
        return {"bytes": b, "flops": f}
    n = float(case["nx"]) * case["ny"] * case["nz"]
    if case["kind"] == "gradient":
        # a step forward, a step again that keeps its field, a step of the adjoint (which also reads that
        # field and adds to the image)
        return {"bytes": n * case["nt"] * (16 + 16 + 28), "flops": n * case["nt"] * (3 * flops + 40)}
    per = 16 if case["storage"] == "f32" else (10 if case["model_bits"] == 16 else 12)
    b = n * per * case["nt"] + 4 * n + (8 * n if case["start"] == "field" else 0)
    if case["cpml"]:  # on the layers: two memory variables read and written, one of them read again
        cross = float(case["ny"]) * case["nz"] + float(case["nx"]) * case["nz"] + float(case["nx"]) * case["ny"]
        b += 20.0 * 2 * case["cpml"] * cross * case["nt"]
    return {"bytes": b, "flops": n * flops * case["nt"]}


# ------------------------------------------------------------ the same in float64

C2 = (-205.0 / 72.0, 8.0 / 5.0, -1.0 / 5.0, 8.0 / 315.0, -1.0 / 560.0)  # second derivative, 8th order
C1 = (4.0 / 5.0, -1.0 / 5.0, 4.0 / 105.0, -1.0 / 280.0)                 # first derivative, 8th order


def _shifted(u, axis, m):
    """(where, from): slices such that node i of the first is node i + m of the second."""
    n = u.shape[axis]
    a, b = [slice(None)] * 3, [slice(None)] * 3
    a[axis] = slice(max(0, -m), n - max(0, m))
    b[axis] = slice(max(0, m), n + min(0, m))
    return tuple(a), tuple(b)


def _add_d2(out, u, axis):
    out.add_(u, alpha=C2[0] / H ** 2)
    for m in (1, 2, 3, 4):
        for s in (m, -m):
            a, b = _shifted(u, axis, s)
            out[a].add_(u[b], alpha=C2[m] / H ** 2)


def _add_d1(out, u, axis):
    for m in (1, 2, 3, 4):
        for s in (m, -m):
            a, b = _shifted(u, axis, s)
            out[a].add_(u[b], alpha=math.copysign(C1[m - 1] / H, s) if C1[m - 1] > 0 else -math.copysign(-C1[m - 1] / H, s))


def _laplacian(u):
    out = torch.zeros_like(u)
    for axis in range(3):
        _add_d2(out, u, axis)
    return out


def _cpml(case, s, vmax):
    W, axes = case["cpml"], []
    for axis, n in ((2, case["nx"]), (1, case["ny"]), (0, case["nz"])):
        i = np.arange(n)
        xi = np.maximum(np.maximum(W - i, i - (n - 1 - W)), 0) / W
        d = -3.0 * vmax * math.log(1e-3) / (2 * W * H) * xi ** 2
        alpha = math.pi * 15.0 * (1 - xi)
        b = np.exp(-(d + alpha) * s.dt)
        a = np.where(d > 0, d * (b - 1) / np.where(d + alpha > 0, d + alpha, 1.0), 0.0)
        shape = [1, 1, 1]
        shape[axis] = n
        a, b = (torch.tensor(t.reshape(shape), device=s.vel.device) for t in (a, b))
        axes.append((axis, a, b, torch.zeros_like(s.vel, dtype=torch.float64), torch.zeros_like(s.vel, dtype=torch.float64)))
    return axes


def _propagate(case, s, keep=None):
    """Traces and last field in float64; `keep` collects (field, its Laplacian) of every step."""
    nt = case["nt"]
    m = s.vel.double().mul_(s.dt).square_()
    W = case["sponge"]
    tabs = [t.view([-1 if d == k else 1 for d in range(3)])
            for k, t in enumerate(_sponge_table(n, W, s.vel.device) for n in s.vel.shape)] if W else []
    layers = _cpml(case, s, float(s.vel.max())) if case.get("cpml") else []
    cur = s.cur.double() if hasattr(s, "cur") else torch.zeros_like(m)
    prev = s.prev.double() if hasattr(s, "prev") else torch.zeros_like(m)
    rec = [torch.as_tensor(s.rec[:, k].astype(np.int64), device=m.device) for k in range(3)]
    traces = torch.empty((nt, len(s.rec)), dtype=torch.float64, device=m.device)
    q = s.wavelet.double() * (s.dt ** 2 / H ** 3)
    ix, iy, iz = s.src
    for n in range(nt):
        if layers:
            lap = torch.zeros_like(cur)
            for axis, a, b, psi, zeta in layers:
                d = torch.zeros_like(cur)
                _add_d1(d, cur, axis)
                psi.mul_(b).addcmul_(a, d)
                d.zero_()
                _add_d2(d, cur, axis)
                _add_d1(d, psi, axis)
                zeta.mul_(b).addcmul_(a, d)
                lap.add_(d).add_(zeta)
        else:
            lap = _laplacian(cur)
        if keep is not None:
            keep.append((cur, lap.clone()))
        for t in tabs:
            prev = prev * t
        new = lap.mul_(m).add_(cur, alpha=2.0).sub_(prev)
        new[iz, iy, ix] += q[n]
        for t in tabs:
            new.mul_(t)
        traces[n] = new[rec[2], rec[1], rec[0]]
        prev, cur = cur, new
    return traces, cur, m, tabs, rec


def exact(case, seed):
    device = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    s = _inputs(case, seed, device)
    if case["kind"] == "serve":
        out = []
        for r in s.requests:
            one = SimpleNamespace(dt=r.dt, rec=r.rec, src=r.src)
            one.vel = torch.tensor(r.velocity, device=device).view(-1, 1, 1).expand(r.shape)
            one.wavelet = torch.tensor(_ricker(r.nt, r.dt, r.f0), dtype=torch.float32, device=device)
            out.append(_propagate(dict(nt=r.nt, sponge=r.sponge_width), one)[0])
        return out
    if case["kind"] == "forward":
        traces, field = _propagate(case, s)[:2]
        return {"traces": traces, "field": field}
    steps = []
    traces, _, m, tabs, rec = _propagate(case, s, keep=steps)
    resid = traces - s.obs.double()
    bar, bar_next = torch.zeros_like(m), torch.zeros_like(m)  # dJ/dA^{n+1}, and what A^{n+2} gave to A^n
    grad = torch.zeros_like(m)
    for n in range(case["nt"] - 1, -1, -1):
        bar.index_put_((rec[2], rec[1], rec[0]), resid[n], accumulate=True)
        w = bar
        for t in tabs:
            w = w * t
        grad.addcmul_(w, steps[n][1])
        older = w
        for t in tabs:
            older = older * t
        bar, bar_next = bar_next + 2.0 * w + _laplacian(m * w), -older
        steps[n] = None
    v = s.vel.double()
    return {"traces": traces, "grad": grad.mul_(2.0 * s.dt ** 2).mul_(v)}
