"""Cases that time the library through its public entry points: what a program that uses it runs.

  solve    lgf_convolve: one Poisson solve (one component) or a vector potential (three)
  step     vor2vel, then one IF-HERK step: the whole hot path from a vorticity, as bench.py runs it
  batch    herk_step_batched over an ensemble of uneven boxes
  refresh  velocity_refresh: the velocity rebuilt from its vorticity, every few dozen steps of a run
  active   HerkState.run_active: steps on the active box that follows the flow
  if       if_apply: the integrating factor alone, alpha from a small step to strong diffusion
  monitor  flow_diagnostics, block_weights and max_cell_speed: what a run prints and decides on
  layer    one 3x3x3 layer of the surrogate network in training: casts, forward, both gradients

Sizes are the ones of the tests, the workloads and the benchmark (boxes of 32 to 256 cells per axis, the
batch's 48 to 192, the network's layers on grids of 32 to 128), and ragged ones between them.  Flows are
Gaussian vortex rings with a seeded wavy centreline, as in the workloads, sampled on the GPU.  The
reference values (`exact`) are plain 64-bit torch and numpy, independent of the library.
"""
import math
import random

import numpy as np
import torch

import paper_1601_00035_amd as nslgf
from paper_1601_00035_amd import surrogate

DEV = "cuda" if torch.cuda.is_available() else "cpu"
DT = {"f64": torch.float64, "f32": torch.float32}
BATCH = (48, 64, 96, 128, 160, 192)


def listed():
    return [
        # the smallest solve of the tests: five short launches, latency
        dict(name="solve_32_f64", op="solve", nx=32, ny=32, nz=32, ncomp=1, dtype="f64"),
        # the vector potential of the largest box in single precision
        dict(name="solve3_256_f32", op="solve", nx=256, ny=256, nz=256, ncomp=3, dtype="f32"),
        # the benchmark's step: the largest box in double precision
        dict(name="step_256_f64", op="step", nx=256, ny=256, nz=256, dtype="f64", scheme="A", sigma=0.1, n_buf=16),
        # the middle-sized ring in single precision
        dict(name="step_128_f32", op="step", nx=128, ny=128, nz=128, dtype="f32", scheme="A", sigma=0.2, n_buf=16),
        # a small box: dozens of short launches
        dict(name="step_48_f64", op="step", nx=48, ny=48, nz=48, dtype="f64", scheme="C", sigma=0.2, n_buf=4),
        # an ensemble over the batch's sizes
        dict(name="batch_8_f64", op="batch", sizes="48,64,64,96,96,128,160,192", dtype="f64", scheme="A"),
        # a ragged box whose three padded lengths differ (384, 320, 192)
        dict(name="refresh_ragged_f64", op="refresh", nx=171, ny=150, nz=90, dtype="f64", sigma=0.2, n_buf=8),
        # two steps that follow a thin ring on a 192^3 grid
        dict(name="active_192_f64", op="active", nx=192, ny=192, nz=192, dtype="f64", sigma=0.1, block=16, steps=2),
        # strong diffusion (low Reynolds number) on a ragged box with odd rows
        dict(name="if_ragged_f64", op="if", nx=177, ny=144, nz=160, ncomp=3, dtype="f64", alpha=0.5),
        # the integrals and block weights of a running simulation
        dict(name="monitor_192_f64", op="monitor", nx=192, ny=192, nz=192, dtype="f64", sigma=0.1, block=16, n_buf=8),
        # the network's full-resolution layer at its training size, and its coarsest one
        dict(name="layer_128_32_32", op="layer", n=128, cin=32, cout=32),
        dict(name="layer_16_96_128", op="layer", n=16, cin=96, cout=128),
    ]


def _size(rng, lo, hi):
    """Log-uniform in lo..hi, any parity."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    op = rng.choice(("solve", "solve", "step", "step", "batch", "refresh", "active", "if", "if", "monitor", "layer",
                     "layer"))
    dtype = rng.choice(("f64", "f64", "f32"))
    if op == "solve":
        return dict(op=op, nx=_size(rng, 24, 256), ny=_size(rng, 24, 256), nz=_size(rng, 24, 256),
                    ncomp=rng.choice((1, 3)), dtype=dtype)
    if op == "step":
        n = _size(rng, 40, 230)
        nx, ny, nz = (min(256, max(32, int(n * rng.uniform(0.75, 1.1)))) for _ in range(3))
        return dict(op=op, nx=nx, ny=ny, nz=nz, dtype=dtype, scheme=rng.choice("ABC"),
                    sigma=round(rng.uniform(0.1, 0.3), 3), n_buf=max(2, min(nx, ny, nz) // 16))
    if op == "batch":
        sizes = [rng.choice(BATCH) for _ in range(rng.randint(2, 12))]
        while len(sizes) > 1 and sum(s ** 3 for s in sizes) > 1.4e7:
            sizes.remove(max(sizes))
        return dict(op=op, sizes=",".join(str(s) for s in sizes), dtype=dtype, scheme=rng.choice("ABC"))
    if op == "refresh":
        return dict(op=op, nx=_size(rng, 40, 256), ny=_size(rng, 40, 256), nz=_size(rng, 40, 256), dtype=dtype,
                    sigma=round(rng.uniform(0.1, 0.3), 3), n_buf=rng.randint(2, 8))
    if op == "active":
        block = rng.choice((8, 16))
        n = 16 * rng.randint(4, 12)
        return dict(op=op, nx=n, ny=n, nz=n, dtype="f64", sigma=round(rng.uniform(0.1, 0.2), 3), block=block,
                    steps=rng.randint(1, 3))
    if op == "if":
        return dict(op=op, nx=_size(rng, 32, 256), ny=_size(rng, 32, 256), nz=_size(rng, 32, 256),
                    ncomp=rng.choice((1, 3, 6)), dtype=dtype,
                    alpha=round(math.exp(rng.uniform(math.log(0.004), math.log(1.5))), 5))
    if op == "monitor":
        n = _size(rng, 48, 256)
        nx, ny, nz = (min(256, max(32, int(n * rng.uniform(0.75, 1.1)))) for _ in range(3))
        return dict(op=op, nx=nx, ny=ny, nz=nz, dtype=dtype, sigma=round(rng.uniform(0.1, 0.3), 3),
                    block=rng.choice((8, 16)), n_buf=rng.randint(1, 8))
    # a layer of the network on one of its training grids
    cin, cout, level = rng.choice([(a, b, l) for (a, b), l in zip(surrogate.LAYERS, surrogate.LEVEL)])
    return dict(op="layer", n=(16 * rng.randint(2, 8)) >> level, cin=cin, cout=cout)


# ---- inputs -------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _ring_dx(nx, ny, sigma):
    return 2.0 * (1.0 + 5.0 * sigma) / (min(nx, ny) - 16)


def _ring(nx, ny, nz, sigma, dtype, seed):
    """Edge vorticity [3][nz][ny][nx] of a Gaussian ring (radius 1, circulation 1, wavy centreline)."""
    dx = _ring_dx(nx, ny, sigma)
    r = np.random.default_rng(seed)
    amp, phi = r.uniform(-1.0, 1.0, 8), r.uniform(0.0, 2.0 * math.pi, 8)
    shift = r.uniform(-0.3, 0.3)
    w = torch.zeros((3, nz, ny, nx), dtype=torch.float64, device=DEV)
    pos = [(torch.arange(n, dtype=torch.float64, device=DEV) - (n - 1) / 2.0) * dx for n in (nx, ny, nz)]
    for q in range(2):  # (no axial vorticity)
        x, y, z = (p - 0.5 * dx if a == q else p for a, p in enumerate(pos))
        x, y, z = x[None, None, :], y[None, :, None], z[:, None, None]
        rho, th = torch.sqrt(x * x + y * y), torch.atan2(y, x)
        rc = 1.0 + 0.01 * sum(float(amp[m]) * torch.cos((m + 1) * th + float(phi[m])) for m in range(8))
        wt = torch.exp(-((rho - rc) ** 2 + (z - shift * dx) ** 2) / sigma ** 2) / (math.pi * sigma ** 2)
        w[q] = -wt * torch.sin(th) if q == 0 else wt * torch.cos(th)
    return w.to(DT[dtype]).contiguous(), dx


def _dt(dx, sigma):
    """Half a cell per step at the ring's largest speed (about 0.14 / sigma)."""
    return 0.5 * dx * sigma / 0.14


RE = 500.0


def _layer_inputs(c, seed):
    g = _gen(seed)
    n, cin, cout = c["n"], c["cin"], c["cout"]
    nv = n ** 3
    x = torch.relu(torch.randn((nv, cin), generator=g, device=DEV))
    w = torch.randn((27, cout, cin), generator=g, device=DEV) * math.sqrt(2.0 / (27 * cin))
    act = torch.relu(torch.randn((nv, cout), generator=g, device=DEV))
    gy = torch.randn((nv, cout), generator=g, device=DEV) * 1e-3
    return x, w, act, gy


def prepare(case, seed):
    c = dict(case)
    op = c["op"]
    st = {"c": c}
    if op == "layer":
        x, w, act, gy = _layer_inputs(c, seed)
        n, cin, cout = c["n"], c["cin"], c["cout"]
        nv = n ** 3
        wb = surrogate.bf16_empty(w.numel(), DEV)
        surrogate.call("sur_cast_bf16", w, wb, w.numel())
        L = nslgf.lib()
        nbytes = L.sur_bwd_weight_blocked_work_bytes(n, n, n, cin, cout)
        st["blocked"] = nbytes > 0  # (grids whose rows are not whole groups of 8 take the plain form)
        if not nbytes:
            nbytes = L.sur_bwd_weight_work_bytes(n, n, n, cin, cout)
        st.update(x=x, wb=wb, act=act, gy=gy, work=torch.empty(nbytes // 4 + 64, device=DEV),
                  xb=surrogate.bf16_empty(nv * cin, DEV), xk=surrogate.bf16_empty(nv * cin, DEV),
                  gb=surrogate.bf16_empty(nv * cout, DEV), gk=surrogate.bf16_empty(nv * cout, DEV),
                  wt=surrogate.bf16_empty(w.numel(), DEV), y=torch.empty((nv, cout), device=DEV),
                  dw=torch.empty((27, cout, cin), device=DEV), dx=torch.empty((nv, cin), device=DEV))
        return st
    if op == "batch":
        st["sts"], st["u0"] = [], []
        for i, n in enumerate(int(s) for s in c["sizes"].split(",")):
            w, dx = _ring(n, n, n, 0.2, "f64", seed + 1000 * (i + 1))
            u0 = nslgf.vor2vel(w, dx).to(DT[c["dtype"]])
            st["u0"].append(u0)
            st["sts"].append(nslgf.HerkState(u0.clone(), dx, _dt(dx, 0.2), RE, c["scheme"], n_buf=max(2, n // 16)))
        return st
    shape = (c["nz"], c["ny"], c["nx"])
    if op == "if":
        st["src"] = torch.randn((c["ncomp"],) + shape, generator=_gen(seed), device=DEV, dtype=DT[c["dtype"]])
        st["out"] = torch.empty_like(st["src"])
        return st
    if op == "solve":
        st["src"] = _solve_src(c, seed)
        st["out"] = torch.empty_like(st["src"])
        return st
    w, dx = _ring(c["nx"], c["ny"], c["nz"], c["sigma"], c["dtype"], seed)
    st["dx"] = dx
    if op == "step":
        st["w"] = w
        st["st"] = nslgf.HerkState(torch.zeros_like(w), dx, _dt(dx, c["sigma"]), RE, c["scheme"], n_buf=c["n_buf"])
    elif op == "active":
        st["u0"] = nslgf.vor2vel(w, dx)
        st["st"] = nslgf.HerkState(st["u0"].clone(), dx, _dt(dx, c["sigma"]), RE, "A", n_buf=2)
    else:  # refresh, monitor
        st["u0"] = nslgf.vor2vel(w, dx)
        st["u"] = st["u0"].clone()
    return st


def _solve_src(c, seed):
    """Random source on an ellipsoid inside the box, zero mean per component."""
    shape = (c["nz"], c["ny"], c["nx"])
    s = torch.randn((c["ncomp"],) + shape, generator=_gen(seed), device=DEV, dtype=torch.float64)
    r2 = 0.0
    for a, n in enumerate(shape):
        p = (torch.arange(n, device=DEV, dtype=torch.float64) - (n - 1) / 2.0) / (0.375 * n)
        r2 = r2 + p.reshape([n if b == a else 1 for b in range(3)]) ** 2
    m = (r2 <= 1.0).double()
    s = (s - (s * m).sum((1, 2, 3), keepdim=True) / m.sum()) * m
    return s.to(DT[c["dtype"]]).contiguous()


# ---- one pass -----------------------------------------------------------------------------------
def run(st):
    c = st["c"]
    op = c["op"]
    if op == "solve":
        return nslgf.lgf_convolve(st["src"], 1.0, st["out"])
    if op == "if":
        return nslgf.if_apply(st["src"], c["alpha"], st["out"])
    if op == "step":
        h = st["st"]
        nslgf.vor2vel(st["w"], st["dx"], out=h.u)
        h.step()
        return [h.u, h.d]
    if op == "batch":
        for h, u0 in zip(st["sts"], st["u0"]):  # (the members start from given velocities)
            h.u.copy_(u0)
        nslgf.herk_step_batched(st["sts"])
        return [[h.u, h.d] for h in st["sts"]]
    if op == "refresh":
        st["u"].copy_(st["u0"])
        return nslgf.velocity_refresh(st["u"], st["dx"], c["n_buf"])
    if op == "active":
        h = st["st"]
        h.u.copy_(st["u0"])
        got = h.run_active(c["steps"], c["block"], 1e-4, 1e-3, 1)
        return [h.u, h.d, list(got[2]), list(got[3])]
    if op == "monitor":
        dx, o = st["dx"], [-(c[k] - 1) / 2.0 * st["dx"] for k in ("nx", "ny", "nz")]
        r = nslgf.flow_diagnostics(st["u"], dx, o, c["n_buf"])
        mu, nu = nslgf.block_weights(st["u"], dx, c["block"], c["n_buf"])
        # (the components along the ring's axis: the others are near-cancelling sums)
        return [r["I"][2], r["K"], r["E"], mu, nu, nslgf.max_cell_speed(st["u"])]
    call = surrogate.call
    n, cin, cout = c["n"], c["cin"], c["cout"]
    nv = n ** 3
    call("sur_cast_bf16_ex", st["x"], None, st["xb"], st["xk"], nv, cin)
    call("sur_conv3d_fwd", st["xb"], st["wb"], st["y"], n, n, n, cin, cout, 1)
    call("sur_cast_bf16_ex", st["gy"], st["act"], st["gb"], st["gk"], nv, cout)
    if st["blocked"]:
        call("sur_conv3d_bwd_weight_blocked", st["gk"], st["xk"], st["dw"], st["work"], n, n, n, cin, cout)
    else:
        call("sur_conv3d_bwd_weight", st["gb"], st["xb"], st["dw"], st["work"], n, n, n, cin, cout)
    out = [st["y"], st["dw"], st["xb"], st["gb"]]
    if cin % 32 == 0:  # (the first layer's input needs no gradient)
        call("sur_weight_transpose", st["wb"], st["wt"], cin, cout)
        call("sur_conv3d_bwd_data", st["gb"], st["wt"], st["dx"], n, n, n, cin, cout)
        out.append(st["dx"])
    return out


# ---- what a pass cannot do without --------------------------------------------------------------
def _solve_flops(nx, ny, nz):
    """Real operations of a zero-padded FFT convolution of one component (2.5 N log2 N per real pencil)."""
    px, py, pz = 2 * nx, 2 * ny, 2 * nz
    fft = lambda n: 5.0 * n * math.log2(n)  # noqa: E731
    return 2 * (ny * nz * fft(px) / 2 + (nx + 1) * nz * fft(py) + (nx + 1) * py * fft(pz)) + 2.0 * (nx + 1) * py * pz


def _step_work(nx, ny, nz, es, scheme):
    # u and the tables in, u and d out; three pressure solves, five or six vector integrating factors of
    # radius about 7, three nonlinear terms
    m = nx * ny * nz
    return m * es * 7, 3 * _solve_flops(nx, ny, nz) + 15 * 3 * 23.0 * m + 3 * 70.0 * m


def work(case):
    c = case
    if c["op"] == "layer":
        nv, ci, co = c["n"] ** 3, c["cin"], c["cout"]
        grads = 3 if ci % 32 == 0 else 2
        # x, act, gy and the weights in; y, dw, the four 16-bit copies and dx out
        by = nv * (4 * ci + 8 * co) + 27 * ci * co * (2 + 4) + nv * (4 * co + 4 * ci + 4 * co) + (nv * 4 * ci if grads == 3 else 0)
        return {"bytes": by, "flops": grads * 2.0 * 27 * nv * ci * co}
    es = 8 if c["dtype"] == "f64" else 4
    if c["op"] == "batch":
        by = fl = 0.0
        for n in (int(s) for s in c["sizes"].split(",")):
            b, f = _step_work(n, n, n, es, c["scheme"])
            by, fl = by + b, fl + f
        return {"bytes": by, "flops": fl}
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    m = nx * ny * nz
    if c["op"] == "solve":
        return {"bytes": 2.0 * c["ncomp"] * m * es + m * es, "flops": c["ncomp"] * _solve_flops(nx, ny, nz)}
    if c["op"] == "if":
        r = len(_if_weights(c["alpha"])) - 1
        return {"bytes": 2.0 * c["ncomp"] * m * es, "flops": c["ncomp"] * 3.0 * (3 * r + 1) * m}
    if c["op"] == "refresh":
        return {"bytes": 6.0 * m * es + m * es, "flops": 3 * _solve_flops(nx, ny, nz) + 24.0 * m}
    if c["op"] == "monitor":
        return {"bytes": 3.0 * m * es, "flops": 150.0 * m}
    if c["op"] == "active":
        b, f = _step_work(nx, ny, nz, es, "A")  # (a third of the grid, about, holds the flow)
        return {"bytes": m * es * 10, "flops": c["steps"] * f / 3}
    b, f = _step_work(nx, ny, nz, es, c["scheme"])
    return {"bytes": b + 3.0 * m * es, "flops": f + 3 * _solve_flops(nx, ny, nz)}


# ---- reference values in 64 bits ----------------------------------------------------------------
def _if_weights(alpha):
    """e^{-2a} I_k(2a), k = 0 .. until below 1e-19 of the first (power series)."""
    w, lead, k = [], math.exp(-2.0 * alpha), 0
    while True:
        term = s = lead
        for j in range(1, 400):
            term *= alpha * alpha / (j * (j + k))
            s += term
            if term < 1e-20 * s:
                break
        w.append(s)
        if k > 0 and s < 1e-17 * w[0]:
            return w
        k += 1
        lead *= alpha / k


def _heat(f, alpha):
    """The masked integrating factor of [ncomp][nz][ny][nx], one axis after the other."""
    if alpha == 0.0:
        return f
    w = _if_weights(alpha)
    for ax in (1, 2, 3):
        out = w[0] * f
        for d in range(1, min(len(w), f.shape[ax])):
            n = f.shape[ax] - d
            out.narrow(ax, d, n).add_(f.narrow(ax, 0, n), alpha=w[d])
            out.narrow(ax, 0, n).add_(f.narrow(ax, d, n), alpha=w[d])
        f = out
    return f


def _bessel_nodes(nmax):
    """Nodes t, weights and B[q][n] = e^{-2t} I_n(2t) for the trapezoidal rule in log t."""
    h, t1 = 0.18, 4e5
    ts = torch.exp(torch.arange(-42.0, 96.0, h, dtype=torch.float64))
    near, far = ts[ts <= t1], ts[ts > t1]
    rows = []
    for t in near.split(32):
        m = 1 << int(math.ceil(math.log2(4 * nmax + 64 + 20.0 * math.sqrt(2.0 * float(t[-1])))))
        th = torch.arange(m, dtype=torch.float64) * (2.0 * math.pi / m)
        rows.append(torch.fft.rfft(torch.exp(-4.0 * t[:, None] * torch.sin(0.5 * th) ** 2)).real[:, : nmax + 1] / m)
    # large t: e^{-z} I_n(z) by its series in 1 / z, z = 2 t
    n2 = 4.0 * torch.arange(nmax + 1, dtype=torch.float64) ** 2
    term = torch.ones((len(far), nmax + 1), dtype=torch.float64)
    s = term.clone()
    for k in range(1, 12):
        term = -term * (n2[None, :] - (2 * k - 1) ** 2) / (k * 16.0 * far[:, None])
        s += term
    rows.append(s / torch.sqrt(4.0 * math.pi * far)[:, None])
    return ts * h, torch.cat(rows)


_green = {}


def _green_table(nmax):
    """g(i, j, k) = -int_0^inf prod_j e^{-2t} I_j(2t) dt for 0 <= i, j, k <= nmax."""
    if nmax not in _green:
        wt, b = _bessel_nodes(nmax)
        wt, b = wt.to(DEV), b.to(DEV)
        g = torch.empty((nmax + 1,) * 3, dtype=torch.float64, device=DEV)
        for i in range(nmax + 1):
            g[i] = -(b * (wt * b[:, i])[:, None]).T @ b
        _green.clear()
        _green[nmax] = g
    return _green[nmax]


def _solver(nz, ny, nx):
    """src [nz][ny][nx] -> g * src on the box."""
    g = _green_table(max(nz, ny, nx) - 1)
    P = (2 * nz, 2 * ny, 2 * nx)
    k = g[:nz, :ny, :nx]
    for ax, n in enumerate((nz, ny, nx)):  # even periodic extension; the entry at n is never read
        k = torch.cat([k, torch.zeros_like(k.narrow(ax, 0, 1)), k.narrow(ax, 1, n - 1).flip(ax)], ax)
    kh = torch.fft.rfftn(k).real.clone()
    del k

    def solve(s):
        return torch.fft.irfftn(torch.fft.rfftn(s, s=P) * kh, s=P)[:nz, :ny, :nx].contiguous()

    return solve


def _sh(a, ax, d):
    """a shifted so that out[i] = a[i + d] along ax (0: x, 1: y, 2: z), zero outside."""
    dim = a.dim() - 1 - ax
    n = a.shape[dim]
    out = torch.zeros_like(a)
    if d > 0:
        out.narrow(dim, 0, n - d).copy_(a.narrow(dim, d, n - d))
    else:
        out.narrow(dim, -d, n + d).copy_(a.narrow(dim, 0, n + d))
    return out


def _curl(f):
    """Faces to edges: component q is the difference of the two others across the next cell."""
    out = []
    for q in range(3):
        a, b = (q + 1) % 3, (q + 2) % 3
        out.append(f[a] - _sh(f[a], b, 1) + _sh(f[b], a, 1) - f[b])
    return torch.stack(out)


def _curl_bar(e):
    """Edges to faces (the adjoint differences)."""
    out = []
    for q in range(3):
        a, b = (q + 1) % 3, (q + 2) % 3
        out.append(_sh(e[a], b, -1) - e[a] + e[b] - _sh(e[b], a, -1))
    return torch.stack(out)


def _div(f):
    return sum(f[q] - _sh(f[q], q, -1) for q in range(3))


def _nonlinear(f, dx):
    """The discrete omega x u on the faces, from the curl of the zero-extended field (one layer kept)."""
    p = torch.nn.functional.pad(f, (1,) * 6)
    e = _curl(p) / dx
    out = []
    for q in range(3):
        a, b = (q + 1) % 3, (q + 2) % 3
        # averages onto face q: e_a with u_b, one step back along b; e_b with u_a, one step back along a
        hb = e[a] * (p[b] + _sh(p[b], q, 1))
        ha = e[b] * (p[a] + _sh(p[a], q, 1))
        out.append(0.25 * (hb + _sh(hb, b, -1) - ha - _sh(ha, a, -1)))
    return torch.stack(out)[:, 1:-1, 1:-1, 1:-1]


def _vor2vel(w, dx, solve):
    return _curl_bar(torch.stack([-dx * dx * solve(w[q]) for q in range(3)])) / dx


_S3 = math.sqrt(3.0)
_TABLEAU = {  # shifted: a~_ij, c~_i
    "A": ([[0.5], [_S3 / 3, (3 - _S3) / 3], [(3 + _S3) / 6, -_S3 / 3, (3 + _S3) / 6]], [0.0, 0.5, 1.0, 1.0]),
    "B": ([[1 / 3], [-1.0, 2.0], [0.0, 0.75, 0.25]], [0.0, 1 / 3, 1.0, 1.0]),
    "C": ([[8 / 15], [0.25, 5 / 12], [0.25, 0.0, 0.75]], [0.0, 8 / 15, 2 / 3, 1.0]),
}


def _inner(shape, n_buf):
    m = torch.zeros(shape, dtype=torch.float64, device=DEV)
    m[tuple(slice(n_buf, n - n_buf) for n in shape)] = 1.0
    return m


def _step(u, dx, dt, scheme, n_buf, solve):
    at, ct = _TABLEAU[scheme]
    beta = dt / (dx * dx * RE)
    mask = _inner(u.shape[1:], n_buf)
    q, w, prev = u, [], u
    for i in range(3):
        if i > 0:
            a = (ct[i] - ct[i - 1]) * beta
            q = _heat(q, a)
            w = [_heat(x, a) for x in w]
        g = -at[i][i] * dt * mask * _nonlinear(prev, dx)
        r = q + g
        for j in range(i):
            r = r + dt * at[i][j] * w[j]
        d = dx * dx * solve(mask * _div(r) / dx)
        gd = torch.stack([_sh(d, a, 1) - d for a in range(3)]) / dx
        prev = _heat(r - gd, (ct[i + 1] - ct[i]) * beta)
        w.append((g - gd) / (at[i][i] * dt))
    return prev, d / (at[2][2] * dt)


def _conv3(x, w, sign, n):
    """y[v][o] = sum_tap sum_i x[v + sign off(tap)][i] w[tap][o][i]."""
    xp = torch.nn.functional.pad(x.reshape(n, n, n, -1), (0, 0) + (1,) * 6)
    y = 0.0
    for t in range(27):
        o = [1 + sign * (d - 1) for d in (t // 9, t // 3 % 3, t % 3)]
        y = y + xp[o[0]:o[0] + n, o[1]:o[1] + n, o[2]:o[2] + n].reshape(n ** 3, -1) @ w[t].T
    return y


def exact(case, seed):
    c = case
    op = c["op"]
    if op == "layer":
        x, w, act, gy = _layer_inputs(c, seed)
        n = c["n"]
        bf = lambda a: a.to(torch.bfloat16).double()  # noqa: E731
        x, w, g = bf(x), bf(w), bf(torch.where(act > 0, gy, torch.zeros_like(gy)))
        xp = torch.nn.functional.pad(x.reshape(n, n, n, -1), (0, 0) + (1,) * 6)
        dw = torch.stack([g.T @ xp[a:a + n, b:b + n, d:d + n].reshape(n ** 3, -1)
                          for a in range(3) for b in range(3) for d in range(3)])
        out = [torch.relu(_conv3(x, w, 1, n)), dw, None, None]
        if c["cin"] % 32 == 0:
            out.append(_conv3(g, w.transpose(1, 2), -1, n))
        return out
    if op == "active":
        return None
    if op == "batch":
        out = []
        for i, n in enumerate(int(s) for s in c["sizes"].split(",")):
            w, dx = _ring(n, n, n, 0.2, "f64", seed + 1000 * (i + 1))
            solve = _solver(n, n, n)
            u = _vor2vel(w, dx, solve).to(DT[c["dtype"]]).double()
            out.append(list(_step(u, dx, _dt(dx, 0.2), c["scheme"], max(2, n // 16), solve)))
        return out
    if op == "if":
        src = torch.randn((c["ncomp"], c["nz"], c["ny"], c["nx"]), generator=_gen(seed), device=DEV, dtype=DT[c["dtype"]])
        return _heat(src.double(), c["alpha"])
    if op == "solve":
        solve = _solver(c["nz"], c["ny"], c["nx"])
        src = _solve_src(c, seed).double()
        return torch.stack([solve(s) for s in src])
    solve = _solver(c["nz"], c["ny"], c["nx"])
    w, dx = _ring(c["nx"], c["ny"], c["nz"], c["sigma"], c["dtype"], seed)
    u = _vor2vel(w.double(), dx, solve)
    if op == "step":
        return list(_step(u, dx, _dt(dx, c["sigma"]), c["scheme"], c["n_buf"], solve))
    if c["dtype"] == "f32":
        u = u.float().double()
    m = _inner(u.shape[1:], c["n_buf"])
    om = m * _curl(u) / dx
    if op == "refresh":
        return _vor2vel(om, dx, solve)
    # monitor
    pos = [(torch.arange(c[k], dtype=torch.float64, device=DEV) - (c[k] - 1) / 2.0) * dx for k in ("nx", "ny", "nz")]
    at = lambda half: [(p - 0.5 * dx if h else p).reshape([-1 if b == 2 - a else 1 for b in range(3)])  # noqa: E731
                       for a, (p, h) in enumerate(zip(pos, half))]
    e0, e1 = at((1, 0, 0)), at((0, 1, 0))
    Iz = 0.5 * dx ** 3 * (e1[0] * om[1] - e0[1] * om[0]).sum()
    xc = at((1, 1, 1))
    uc = [0.5 * (u[q] + _sh(u[q], q, -1)) for q in range(3)]
    wc = []
    for q in range(3):
        a, b = (q + 1) % 3, (q + 2) % 3
        s = om[q] + _sh(om[q], a, -1)
        wc.append(0.25 * (s + _sh(s, b, -1)))
    K = dx ** 3 * sum(uc[q] * (xc[(q + 1) % 3] * wc[(q + 2) % 3] - xc[(q + 2) % 3] * wc[(q + 1) % 3]) for q in range(3)).sum()
    E = 0.5 * dx ** 3 * (om ** 2).sum()
    nb = c["block"]
    s = m * (_div(_nonlinear(u, dx)) / dx).abs()

    def blocks(f):
        f = torch.nn.functional.pad(f, [v for n in (f.shape[2], f.shape[1], f.shape[0]) for v in (0, -n % nb)])
        z, y, x = f.shape
        return f.reshape(z // nb, nb, y // nb, nb, x // nb, nb).amax((1, 3, 5))

    speed = torch.sqrt(uc[0] ** 2 + uc[1] ** 2 + uc[2] ** 2).max()
    return [float(Iz), float(K), float(E), blocks(om.abs().amax(0)).cpu().numpy(), blocks(s).cpu().numpy(), float(speed)]
