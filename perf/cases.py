"""Workloads of the wave solver: what its users run, at the sizes they run it.

A case is a dict of plain values.  `kind` names the entry points it goes through:

  run     a whole simulation: Wave.start (ghost level) and Wave.step from u^0
  steps   nsteps more steps of a running simulation, with a point source and receivers
  tdc     steps with a coefficient that changes in time, one Wave.step_tdc call each
  batch   steps of many simulations at once (Batch, tuned and captured as its users do)
  adjoint differentiable traces and their backward pass (simulate_traces)
  lines   tridiag_solve_batched, contiguous or interleaved systems

`exact` is the same arithmetic in 64-bit torch: the factored scheme of eq. (CN1) with
its line systems solved by parallel cyclic reduction down to couplings below 1e-22.
"""
import math

import torch

import paper_2006_10142_amd as adw

DEV = "cuda"


def listed():
    return [
        # the paper's standing wave (128^2, 200 steps, its FP64): a whole short run, bound by launches
        dict(name="standing_128_f64", kind="run", nx=128, ny=128, dtype="f64", cfl=0.5, hetero=False, nsteps=200),
        # the Gaussian pulse at 2048^2, c = 1, dt = h/2: the ordinary size, in both types
        dict(name="pulse_2048_f32", kind="steps", nx=2048, ny=2048, dtype="f32", cfl=0.5, hetero=False, nsteps=20, nrec=0),
        dict(name="pulse_2048_f64", kind="steps", nx=2048, ny=2048, dtype="f64", cfl=0.5, hetero=False, nsteps=20, nrec=0),
        # the headline workload: 8192^2, per-node speed in [1, 3], Ricker source, a row of receivers
        dict(name="ricker_8192_f32", kind="steps", nx=8192, ny=8192, dtype="f32", cfl=0.4, hetero=True, nsteps=4, nrec=64),
        dict(name="ricker_8192_f64", kind="steps", nx=8192, ny=8192, dtype="f64", cfl=0.4, hetero=True, nsteps=4, nrec=64),
        # a domain whose sides are whatever the model's are: odd and unequal
        dict(name="ragged_1501x997_f32", kind="steps", nx=1501, ny=997, dtype="f32", cfl=0.4, hetero=True, nsteps=20, nrec=64),
        # what an implicit scheme is taken for: a time step at the explicit limit and beyond
        dict(name="long_step_3072_f32", kind="steps", nx=3072, ny=3072, dtype="f32", cfl=1.0, hetero=True, nsteps=10, nrec=64),
        # coefficient changing in time (eq. (CN1) with c^{k-1} and c^{k+1})
        dict(name="moving_1024_f32", kind="tdc", nx=1024, ny=1024, dtype="f32", cfl=0.4, hetero=True, nsteps=8, nrec=64),
        # 256 simulations of 256^2 to 1024^2 side by side
        dict(name="batch_256_f32", kind="batch", count=256, lo=256, hi=1024, by=64, dtype="f32", cfl=0.4, nsteps=4),
        # the inverse problem at 1024^2: traces of 64 receivers, and the gradient by the adjoint
        dict(name="adjoint_1024_f32", kind="adjoint", nx=1024, ny=1024, dtype="f32", cfl=0.4, nsteps=400, every=100, nrec=64),
        # the line solver by itself: 8192 systems of 8192 unknowns, row by row and side by side
        dict(name="lines_8192_f32", kind="lines", n=8192, count=8192, dtype="f32", layout="contiguous"),
        dict(name="lines_across_8192_f32", kind="lines", n=8192, count=8192, dtype="f32", layout="interleaved"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _side(rng, lo, hi):
    n = _log(rng, lo, hi)
    return n if rng.random() < 0.5 else max(8, n // 8 * 8)


def draw(rng):
    kind = rng.choice(["run", "steps", "steps", "steps", "tdc", "batch", "adjoint", "lines", "lines"])
    dtype = rng.choice(["f32", "f32", "f64"])
    if kind == "lines":
        n, count = _log(rng, 64, 8192), _log(rng, 16, 8192)
        return dict(kind=kind, n=n, count=count, dtype=dtype if n * count <= 1 << 25 else "f32",
                    layout=rng.choice(["contiguous", "interleaved"]))
    if kind == "batch":
        return dict(kind=kind, count=_log(rng, 4, 256), lo=_log(rng, 64, 256), hi=_log(rng, 257, 1024),
                    by=rng.choice([1, 64]), dtype=dtype, cfl=0.4, nsteps=4)
    cfl = rng.choice([0.4, 0.4, 0.5, 0.8, 1.0, 2.0])
    if kind == "adjoint":
        return dict(kind=kind, nx=_side(rng, 64, 1024), ny=_side(rng, 64, 1024), dtype=dtype, cfl=rng.choice([0.4, 0.5, 0.8]),
                    nsteps=_log(rng, 40, 200), every=rng.choice([20, 50, 100]), nrec=rng.choice([8, 64]))
    nx, ny = _side(rng, 64, 8192), _side(rng, 64, 8192)
    most = max(1, min(50, (1 << 27) // (nx * ny)))
    if kind == "run":
        nx, ny = min(nx, 2048), min(ny, 2048)
        return dict(kind=kind, nx=nx, ny=ny, dtype=dtype, cfl=cfl, hetero=rng.random() < 0.5, nsteps=_log(rng, 2, 50))
    if kind == "tdc":
        return dict(kind=kind, nx=min(nx, 2048), ny=min(ny, 2048), dtype=dtype, cfl=cfl, hetero=True, nsteps=rng.choice([2, 4, 8]),
                    nrec=rng.choice([0, 64]))
    return dict(kind=kind, nx=nx, ny=ny, dtype=dtype, cfl=cfl, hetero=rng.random() < 0.7, nsteps=_log(rng, 1, most),
                nrec=rng.choice([0, 64]))


# ------------------------------------------------------------------- inputs ----
def _type(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _gen(seed):
    return torch.Generator().manual_seed(seed)


def _axes(nx, ny):
    x = torch.arange(1, nx + 1, dtype=torch.float64, device=DEV) / (nx + 1)
    y = torch.arange(1, ny + 1, dtype=torch.float64, device=DEV) / (ny + 1)
    return x, y


def _bumps(nx, ny, lo, hi, g):
    """A smooth field in [lo, hi]: 16 Gaussian bumps of random place, width and sign."""
    at = torch.rand(16, 2, generator=g, dtype=torch.float64).to(DEV)
    wide = (0.05 + 0.15 * torch.rand(16, 1, generator=g, dtype=torch.float64)).to(DEV)
    high = (2 * torch.rand(16, 1, generator=g, dtype=torch.float64) - 1).to(DEV)
    x, y = _axes(nx, ny)
    gx = torch.exp(-((x - at[:, :1]) ** 2) / (2 * wide * wide))
    gy = high * torch.exp(-((y - at[:, 1:]) ** 2) / (2 * wide * wide))
    f = gy.t().contiguous() @ gx
    low, top = f.min(), f.max()
    return f.sub_(low).mul_((hi - lo) / (top - low)).add_(lo).clamp_(lo, hi)


def _pulse(nx, ny, g, sigma=0.05):
    at = (0.3 + 0.4 * torch.rand(2, generator=g, dtype=torch.float64)).tolist()
    x, y = _axes(nx, ny)
    return torch.outer(torch.exp(-((y - at[1]) ** 2) / (2 * sigma * sigma)),
                       torch.exp(-((x - at[0]) ** 2) / (2 * sigma * sigma)))


def _ricker(nsteps, dt, h, first, f0):
    t = torch.arange(first, first + nsteps, dtype=torch.float64) * dt
    a = (math.pi * f0 * (t - 1.0 / f0)) ** 2
    return (((1 - 2 * a) * torch.exp(-a)) / (h * h)).reshape(nsteps, 1).to(DEV)


def _receivers(nx, ny, nrec):
    row = max(0, min(ny - 1, int(0.1 * (ny + 1) + 0.5) - 1))
    cols = [max(0, min(nx - 1, int((k + 0.5) * (nx + 1) / nrec))) for k in range(nrec)]
    return torch.tensor([row * nx + i for i in cols], dtype=torch.int32, device=DEV)


def _grid(case):
    h = 1.0 / (max(case["nx"], case["ny"]) + 1)
    return h, case["cfl"] * h / (3.0 if case.get("hetero", True) else 1.0)


def _inputs(case, seed):
    """What a program hands to the solver, as tensors of the case's type."""
    g, dt_ = _gen(seed), _type(case)
    kind = case["kind"]
    if kind == "lines":
        n, count = case["n"], case["count"]
        shape = (count, n) if case["layout"] == "contiguous" else (n, count)
        gd = torch.Generator(device=DEV).manual_seed(seed)
        # rows of an implicit diffusion step: off-diagonals -r with r in [0.05, 1], row sum 1
        a = -(0.05 + 0.95 * torch.rand(shape, generator=gd, device=DEV, dtype=dt_))
        c = -(0.05 + 0.95 * torch.rand(shape, generator=gd, device=DEV, dtype=dt_))
        d = torch.randn(shape, generator=gd, device=DEV, dtype=dt_)
        return dict(a=a, b=1 - a - c, c=c, d=d)
    if kind == "batch":
        n = torch.randint(case["lo"], case["hi"] + 1, (case["count"],), generator=_gen(4)).tolist()
        n = [max(8, v // case["by"] * case["by"]) for v in n]
        first, total = [], 0
        for v in n:
            first.append(total)
            total += (v * v + 63) // 64 * 64
        c, up = [], torch.zeros(total, dtype=dt_, device=DEV)
        for v, o in zip(n, first):
            c.append(_bumps(v, v, 1.0, 3.0, g).to(dt_))
            up[o:o + v * v] = _pulse(v, v, g).to(dt_).reshape(-1)
        return dict(n=n, first=first, c=c, up=up, uc=up.clone())
    nx, ny = case["nx"], case["ny"]
    h, dt = _grid(case)
    if kind == "adjoint":
        # source and receivers near one wall, as in a survey; the wavelet falls into the run
        f0 = (2.0 + 2.0 * torch.rand(1, generator=g).item()) / (dt * case["nsteps"])
        return dict(h=h, dt=dt, kappa=_bumps(nx, ny, 1.0, 9.0, g).to(dt_),
                    up=(0.1 * _pulse(nx, ny, g)).to(dt_), amp=_ricker(case["nsteps"], dt, h, 1, f0).to(dt_),
                    src=torch.tensor([min(ny - 1, ny // 10 + 16) * nx + nx // 2], dtype=torch.int32, device=DEV),
                    rec=_receivers(nx, ny, case["nrec"]))
    got = dict(h=h, dt=dt, c=_bumps(nx, ny, 1.0, 3.0, g).to(dt_) if case["hetero"] else 1.0,
               up=_pulse(nx, ny, g).to(dt_))
    if kind == "run":
        return got
    # the run is under way: its wavelet peaks in these steps
    f0 = 5.0 + 10.0 * torch.rand(1, generator=g).item()
    got["amp"] = _ricker(case["nsteps"], dt, h, int(1.0 / f0 / dt), f0).to(dt_)
    got["src"] = torch.tensor([(ny // 2) * nx + nx // 2], dtype=torch.int32, device=DEV)
    got["rec"] = _receivers(nx, ny, case["nrec"]) if case["nrec"] else None
    if kind == "tdc":
        k0, k1 = _bumps(nx, ny, 1.0, 7.0, g), _bumps(nx, ny, 0.0, 2.0, g)
        # kappa at the levels n-1, n, ... of the run: a slow swing around k0
        got["kappa"] = [(k0 + k1 * (1 - math.cos(0.2 * k)) / 2).to(dt_) for k in range(case["nsteps"] + 2)]
    return got


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind, dt_ = case["kind"], _type(case)
    if kind == "lines":
        return s
    if kind == "batch":
        sizes = [(v, v) for v in s["n"]]
        hs = [1.0 / (v + 1) for v in s["n"]]
        s["batch"] = adw.Batch(sizes, hs, [case["cfl"] * h / 3.0 for h in hs], s["c"], dtype=dt_)

        def views(flat):
            return [flat[o:o + v * v].view(v, v) for v, o in zip(s["n"], s["first"])]

        s["batch"].bind(views(s["up"]), views(s["uc"]))
        s["batch"].autotune(trial_steps=5)
        s["batch"].graph(True)
        return s
    if kind == "adjoint":
        s["wave"] = adw.Wave(case["nx"], case["ny"], s["h"], s["dt"], kappa=s["kappa"], dtype=dt_)
        s["kappa"].requires_grad_(True)
        s["amp"].requires_grad_(True)
        s["target"] = torch.zeros(case["nsteps"], case["nrec"], dtype=dt_, device=DEV)
        return s
    if kind == "tdc":
        s["wave"] = adw.Wave(case["nx"], case["ny"], s["h"], s["dt"], kappa=s["kappa"][0], dtype=dt_)
    else:
        s["wave"] = adw.Wave(case["nx"], case["ny"], s["h"], s["dt"], c=s["c"], dtype=dt_)
    if kind != "run":
        s["uc"] = s["up"].clone()
        s["traces"] = torch.zeros(case["nsteps"], case["nrec"], dtype=dt_, device=DEV) if case["nrec"] else None
    return s


# --------------------------------------------------------------------- a pass ----
def run(s):
    case = s["case"]
    kind, n = case["kind"], case.get("nsteps", 0)
    if kind == "run":
        u0 = s["up"].clone()
        return s["wave"].step(u0, s["wave"].start(u0), n)
    if kind == "steps":
        s["up"], s["uc"] = s["wave"].step(s["up"], s["uc"], n, src_idx=s["src"], src_amp=s["amp"],
                                          rec_idx=s["rec"], traces=s["traces"])
        return [s["up"], s["uc"]] + ([s["traces"]] if case["nrec"] else [])
    if kind == "tdc":
        up, uc = s["up"], s["uc"]
        for k in range(n):
            up, uc = s["wave"].step_tdc(up, uc, s["kappa"][k], s["kappa"][k + 2], src_idx=s["src"], src_amp=s["amp"][k],
                                        rec_idx=s["rec"], traces=s["traces"][k] if case["nrec"] else None)
        s["up"], s["uc"] = up, uc
        return [up, uc] + ([s["traces"]] if case["nrec"] else [])
    if kind == "batch":
        s["batch"].step(n)
        return [s["up"], s["uc"]]
    if kind == "adjoint":
        s["kappa"].grad = s["amp"].grad = None
        traces = adw.simulate_traces(s["wave"], s["kappa"], s["up"], s["up"], n, s["src"], s["amp"], s["rec"],
                                     checkpoint_every=case["every"])
        (0.5 * (traces - s["target"]).square().sum()).backward()
        return [traces.detach(), s["kappa"].grad, s["amp"].grad]
    stride = dict(sys_stride=case["n"], elem_stride=1) if case["layout"] == "contiguous" \
        else dict(sys_stride=1, elem_stride=case["count"])
    return adw.tridiag_solve_batched(s["a"], s["b"], s["c"], s["d"], case["n"], case["count"], **stride)


def work(case):
    """Bytes: a step reads u^{n-1}, u^n and the coefficient and writes u^{n+1} (the
    time-dependent one reads a second coefficient); a step of the gradient is a forward
    step, its recomputation, and the reverse step, which reads two adjoint levels, u^n,
    the coefficient and the gradient and writes a level and the gradient; a line system
    is read and its solution written.  Operations: counted from the formulas."""
    e = 4 if case["dtype"] == "f32" else 8
    kind = case["kind"]
    if kind == "lines":
        m = case["n"] * case["count"]
        return {"bytes": 5.0 * e * m, "flops": 8.0 * m}
    if kind == "batch":
        lo, hi = case["lo"], case["hi"]
        m = case["count"] * (lo * lo + lo * hi + hi * hi) / 3.0
    else:
        m = case["nx"] * case["ny"]
    m *= case["nsteps"] + (1 if kind == "run" else 0)
    fields, ops = {"tdc": (5, 45), "adjoint": (15, 120)}.get(kind, (4, 30))
    return {"bytes": float(fields) * e * m, "flops": float(ops) * m}


# ------------------------------------------------------------ the same in 64 bits ----
class _Lines:
    """x_i = (d_i + p_i x_{i-s} + q_i x_{i+s}) along one axis, the distance s doubled
    until the couplings are gone."""

    def __init__(self, p, q, axis):
        self.axis, self.levels, s = axis, [], 1
        while s < p.shape[axis] and max(p.abs().max().item(), q.abs().max().item()) > 1e-22:
            den = torch.ones_like(p)
            self._add(den, -p, q, s, -1)
            self._add(den, -q, p, s, 1)
            self.levels.append((s, p / den, q / den, 1.0 / den))
            p2, q2 = torch.zeros_like(p), torch.zeros_like(q)
            self._add(p2, self.levels[-1][1], p, s, -1)
            self._add(q2, self.levels[-1][2], q, s, 1)
            p, q, s = p2, q2, 2 * s

    def _add(self, out, f, x, s, side):
        """out_i += f_i x_{i + side s}"""
        m = out.shape[self.axis] - s
        here, there = (s, 0) if side < 0 else (0, s)
        o, g, v = (t.narrow(self.axis, k, m) for t, k in ((out, here), (f, here), (x, there)))
        o.addcmul_(g, v)

    def solve(self, d):
        for s, p, q, inv in self.levels:
            e = d * inv
            self._add(e, p, d, s, -1)
            self._add(e, q, d, s, 1)
            d = e
        return d


def _system(r, axis, transposed=False):
    """-r_i x_{i-1} + (1 + 2 r_i) x_i - r_i x_{i+1} = d_i, or its transpose; the diagonal apart."""
    b = 1 + 2 * r
    p = r / b
    q = p.clone()
    if transposed:
        n = r.shape[axis]
        p.narrow(axis, 1, n - 1).copy_(r.narrow(axis, 0, n - 1) / b.narrow(axis, 1, n - 1))
        q.narrow(axis, 0, n - 1).copy_(r.narrow(axis, 1, n - 1) / b.narrow(axis, 0, n - 1))
    p.narrow(axis, 0, 1).zero_()
    q.narrow(axis, r.shape[axis] - 1, 1).zero_()
    lines = _Lines(p, q, axis)
    return lambda d: lines.solve(d / b)


def _second(u, axis):
    out = -2 * u
    n = u.shape[axis]
    out.narrow(axis, 1, n - 1).add_(u.narrow(axis, 0, n - 1))
    out.narrow(axis, 0, n - 1).add_(u.narrow(axis, 1, n - 1))
    return out


def _lap(u):
    return _second(u, 0).add_(_second(u, 1))


def _sizes(kappa, h, dt):
    return kappa * (dt * dt / (2 * h * h))


def _march(r, up, uc, dt, nsteps, src=None, amp=None, rec=None):
    along, across = _system(r, 1), _system(r, 0)
    traces = []
    for k in range(nsteps):
        rho = _lap(uc).mul_(r).mul_(2)
        if src is not None:
            rho.view(-1)[src.long()] += dt * dt * amp[k]
        d = across(along(rho))
        up, uc = uc, 2 * uc - up + d
        if rec is not None:
            traces.append(uc.view(-1)[rec.long()])
    return up, uc, torch.stack(traces) if rec is not None else None


def _gradient(case, s):
    h, dt, n = s["h"], s["dt"], case["nsteps"]
    kappa, amp = s["kappa"].double(), s["amp"].double()
    r, beta = _sizes(kappa, h, dt), dt * dt / 2
    src, rec = s["src"].long(), s["rec"].long()
    along, across = _system(r, 1), _system(r, 0)
    u, ws = [s["up"].double(), s["up"].double()], []
    for k in range(n):
        rho = _lap(u[-1]).mul_(r).mul_(2)
        rho.view(-1)[src] += dt * dt * amp[k]
        ws.append(along(rho))
        u.append(2 * u[-1] - u[-2] + across(ws[-1]))
    traces = torch.stack([v.view(-1)[rec] for v in u[2:]])
    along, across = _system(r, 1, True), _system(r, 0, True)
    grad, gamp = torch.zeros_like(r), torch.zeros_like(amp)
    lam2 = torch.zeros_like(r)
    lam = torch.zeros_like(r)
    lam.view(-1).index_add_(0, rec, traces[n - 1])      # the loss is half the square of the traces
    for k in range(n - 1, -1, -1):
        nu = across(lam)
        mu = along(nu)
        d = u[k + 2] - 2 * u[k + 1] + u[k]
        grad += (2 * beta * mu * _lap(u[k + 1]) + beta * (mu * _second(ws[k], 1) + nu * _second(d, 0))) / (h * h)
        gamp[k] = dt * dt * mu.view(-1)[src]
        back = 2 * lam - lam2 + _lap(kappa * mu) * (dt * dt / (h * h))
        if k > 0:
            back.view(-1).index_add_(0, rec, traces[k - 1])
        lam, lam2 = back, lam
        u.pop()
        ws.pop()
    return [traces, grad, gamp]


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "lines":
        axis = 1 if case["layout"] == "contiguous" else 0
        b = s["b"].double()
        p, q = -s["a"].double() / b, -s["c"].double() / b
        p.narrow(axis, 0, 1).zero_()
        q.narrow(axis, case["n"] - 1, 1).zero_()
        return _Lines(p, q, axis).solve(s["d"].double() / b)
    if kind == "batch":
        up, uc = s["up"].double(), s["uc"].double()
        for v, o, c in zip(s["n"], s["first"], s["c"]):
            h = 1.0 / (v + 1)
            dt = case["cfl"] * h / 3.0
            u, w = (f[o:o + v * v].view(v, v) for f in (up, uc))
            a, b, _ = _march(_sizes(c.double().square(), h, dt), u, w, dt, case["nsteps"])
            up[o:o + v * v], uc[o:o + v * v] = a.reshape(-1), b.reshape(-1)
        return [up, uc]
    if kind == "adjoint":
        return _gradient(case, s)
    h, dt, up = s["h"], s["dt"], s["up"].double()
    if kind == "tdc":
        uc, traces = up.clone(), []
        r = [_sizes(k.double(), h, dt) for k in s["kappa"]]
        for k in range(case["nsteps"]):
            old, new = r[k], r[k + 2]
            rho = 2 * new * _lap(uc) + (old - new) * _lap(up)
            rho.view(-1)[s["src"].long()] += dt * dt * s["amp"][k].double()
            d = _system(new, 0)(_system(new, 1)(rho))
            up, uc = uc, 2 * uc - up + d
            if case["nrec"]:
                traces.append(uc.view(-1)[s["rec"].long()])
        return [up, uc] + ([torch.stack(traces)] if case["nrec"] else [])
    kappa = s["c"].double().square() if case["hetero"] else torch.ones_like(up)
    r = _sizes(kappa, h, dt)
    if kind == "run":
        e = _system(r, 0)(_system(r, 1)(_lap(up) * r))
        return list(_march(r, up, up + e, dt, case["nsteps"])[:2])
    up, uc, traces = _march(r, up, up.clone(), dt, case["nsteps"], s["src"], s["amp"].double(), s["rec"])
    return [up, uc] + ([traces] if case["nrec"] else [])
