"""Performance cases: the calls that programs built on this package make.

Kinds of case (``kind``):

* ``operator``: one application of the Mindlin and / or Boussinesq operator,
  the inner step of every plasticity iteration and a call of its own;
* ``batch``: the fused operator for several contexts of different grids in
  one call;
* ``return_map``: the J2 radial return of every voxel;
* ``contact``: frictionless contact of a rough surface under a given load;
* ``tangential``: partial slip under a given pressure (Coulomb friction);
* ``solve``: elastoplastic contact, contact and plasticity coupled.

Inputs are made on the GPU from the seed, with the distributions of the
package's benchmark: Gaussian eigenstrain and traction filtered by |k|^-2 in
the plane (the eigenstrain decaying in depth), self-affine rough surfaces and
paraboloids.  E = 1, nu = 0.3, sigma_y0 = 0.01, E_h = 0.1, cell 1 x 1 unless a
case says otherwise.  The contexts, and preallocated outputs of the operators,
are kept between passes, as an iterating program keeps them.
"""
import math

import torch

from paper_1811_11558_amd import Context, EPOptions, operator_apply_batch

E, NU, SY0, EH = 1.0, 0.3, 0.01, 0.1
MU = E / (2.0 * (1.0 + NU))
LAM = E * NU / ((1.0 + NU) * (1.0 - 2.0 * NU))
# the eight grids of the benchmark's batched workload
BATCH = "64x64x32,32x32x16,128x128x64,64x32x16,32x64x32,64x64x16,128x64x32,32x32x8"


def listed():
    return [
        # the smallest solve grid of the benchmark: launches and latency
        _op("op_f64_32x32x16", 32, 32, 16),
        # unequal sides, ragged depth, every output a program can ask for
        _op("op_f64_64x128x33_all", 64, 128, 33, ly=2.0, lz=0.3, want="strain,stress,disp,surf_u3"),
        # the benchmark's operator workload, and the surface load alone on it
        # (what each outer pass of a solve does first)
        _op("op_f64_256x256x64", 256, 256, 64),
        _op("bouss_f64_256x256x64", 256, 256, 64, op="boussinesq"),
        # the largest rough-contact grid
        _op("op_f64_1024x1024x64", 1024, 1024, 64),
        # float32 transforms on the mixed-precision grid
        _op("op_f32_512x512x128", 512, 512, 128, precision="fp32_refined"),
        # several small problems in one call
        {"name": "batch_f64_8_grids", "kind": "batch", "grids": BATCH, "precision": "fp64"},
        # the pointwise part of every plasticity iteration
        {"name": "return_map_256x256x64", "kind": "return_map", "nx": 256, "ny": 256, "nz": 64},
        # elastic contact of a rough surface, the first half of every outer pass
        {"name": "contact_256x256", "kind": "contact", "nx": 256, "ny": 256, "ly": 1.0, "hurst": 0.8, "k_roll": 4,
         "k_cut": 64, "load": 0.01},
        # the friction part of a contact step
        {"name": "tangential_512x512", "kind": "tangential", "nx": 512, "ny": 512, "ly": 1.0, "mu_f": 0.3,
         "q_ratio": 0.5},
        # whole solves: a paraboloid in float64 on a small grid, and a rough
        # surface as the solve server runs it (float32 kernels refined)
        _solve("solve_f64_32x32x16", 32, 16, "paraboloid", "fp64", load=0.004, steps=2),
        _solve("solve_f32_128x128x64", 128, 64, "rough", "fp32_refined", load=0.01, steps=1),
    ]


def draw(rng):
    kind = rng.choice(["operator"] * 5 + ["batch", "return_map", "contact", "contact", "tangential", "solve"])
    if kind == "operator":
        while True:
            nx = 2 ** rng.randint(4, 10)
            ny = min(1024, max(16, (nx >> 2) << rng.randint(0, 4)))
            nz = round(math.exp(rng.uniform(math.log(5), math.log(160))))
            if nx * ny * nz <= 1 << 25:
                break
        op = rng.choice(["fused", "fused", "mindlin", "boussinesq"])
        want = rng.choice(["strain", "strain", "strain,stress", "surf_u3", "strain,stress,disp,surf_u3"])
        if nx * ny * nz > 1 << 23 and want.count(",") > 1:
            want = "strain"
        return {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "ly": rng.choice([1.0, 0.5, 2.0]),
                "lz": round(rng.uniform(0.1, 0.5), 3), "op": op, "want": want,
                "precision": rng.choice(["fp64", "fp64", "fp32_refined"]),
                "graded": rng.choice([0.0, 0.0, 0.0, 2.0])}
    if kind == "batch":
        grids = []
        for _ in range(rng.randint(2, 10)):
            nz = round(math.exp(rng.uniform(math.log(4), math.log(64))))
            grids.append("%dx%dx%d" % (2 ** rng.randint(4, 7), 2 ** rng.randint(4, 7), nz))
        return {"kind": kind, "grids": ",".join(grids), "precision": rng.choice(["fp64", "fp64", "fp32_refined"])}
    if kind == "return_map":
        nx, ny = 2 ** rng.randint(4, 9), 2 ** rng.randint(4, 9)
        return {"kind": kind, "nx": nx, "ny": ny, "nz": round(math.exp(rng.uniform(math.log(5), math.log(128))))}
    if kind == "contact":
        nx = 2 ** rng.randint(4, 10)
        ny = nx if rng.random() < 0.6 else min(1024, max(16, nx * rng.choice([2, 4]) // rng.choice([1, 8])))
        return {"kind": kind, "nx": nx, "ny": ny, "ly": 1.0 if nx == ny else ny / nx, "hurst": round(rng.uniform(0.5, 0.9), 3),
                "k_roll": 4 if nx > 16 else 2, "k_cut": max(3, min(nx, ny) // 4),
                "load": round(math.exp(rng.uniform(math.log(1e-3), math.log(0.05))), 6)}
    if kind == "tangential":
        nx = 2 ** rng.randint(5, 9)
        ny = nx if rng.random() < 0.6 else max(32, nx // 2)
        return {"kind": kind, "nx": nx, "ny": ny, "ly": ny / nx, "mu_f": round(rng.uniform(0.1, 0.6), 3),
                "q_ratio": round(rng.uniform(0.2, 0.8), 3)}
    n = 2 ** rng.randint(4, 7)
    nz = round(math.exp(rng.uniform(math.log(8), math.log(min(n, 64)))))
    return {k: v for k, v in _solve("", n, nz, "paraboloid" if n < 64 else "rough", rng.choice(["fp64", "fp32_refined"]),
                                    load=round(rng.uniform(0.002, 0.02), 5), steps=1).items() if k != "name"}


def _op(name, nx, ny, nz, op="fused", want="strain", precision="fp64", ly=1.0, lz=0.25, graded=0.0):
    return {"name": name, "kind": "operator", "nx": nx, "ny": ny, "nz": nz, "ly": ly, "lz": lz, "op": op,
            "want": want, "precision": precision, "graded": graded}


def _solve(name, n, nz, surface, precision, load, steps):
    return {"name": name, "kind": "solve", "nx": n, "ny": n, "nz": nz, "surface": surface, "precision": precision,
            "load": load, "steps": steps}


# ------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


class _Dft:
    """Discrete Fourier transform of planes [..., ny, nx] to half spectra
    [..., ny, nx / 2 + 1] and back (forward unscaled), as matrix products:
    torch.fft.rfft2 gave wrong values on this device for some batches of
    small planes (7 planes of 64 x 64 among them)."""

    def __init__(self, nx, ny):
        self.nx, self.ny, self.kxh = nx, ny, nx // 2 + 1
        self.fx, self.fy = self._matrix(nx)[:, :self.kxh], self._matrix(ny)
        # weights of the half spectrum in the sum over all modes
        w = torch.full((self.kxh,), 2.0 / (nx * ny), dtype=torch.float64, device="cuda")
        w[0] = w[-1] = 1.0 / (nx * ny)
        self.bx = (self.fx.conj() * w).T.contiguous()

    @staticmethod
    def _matrix(n):
        j = torch.arange(n, device="cuda")
        a = (j[:, None] * j[None, :] % n).double() * (2.0 * math.pi / n)
        return torch.complex(torch.cos(a), -torch.sin(a))

    def _columns(self, s, f):
        t = s.transpose(-1, -2).contiguous().view(-1, self.ny) @ f
        return t.view(s.shape[:-2] + (self.kxh, self.ny)).transpose(-1, -2).contiguous()

    def forward(self, f):
        s = f.reshape(-1, self.nx).to(torch.complex128) @ self.fx
        return self._columns(s.view(f.shape[:-1] + (self.kxh,)), self.fy)

    def back(self, s):
        f = self._columns(s, self.fy.conj()).view(-1, self.kxh)
        f = f.real.contiguous() @ self.bx.real.contiguous() - f.imag.contiguous() @ self.bx.imag.contiguous()
        return f.view(s.shape[:-1] + (self.nx,))


def _wavenumbers(nx, ny):
    ky = torch.arange(ny, device="cuda")
    return torch.arange(nx // 2 + 1, device="cuda").double(), torch.where(2 * ky <= ny, ky, ky - ny).double()


def _plane(k):
    return k[0][None, :], k[1][:, None]


def _filtered(shape, gen, depth_decay=None):
    """Gaussian planes of the given shape filtered by |k|^-2."""
    ny, nx = shape[-2:]
    kx, ky = _plane(_wavenumbers(nx, ny))
    k = torch.hypot(kx, ky)
    amp = torch.where(k > 0, k.clamp(min=1.0) ** -2, torch.zeros_like(k))
    dft = _Dft(nx, ny)
    out = torch.empty(shape, dtype=torch.float64, device="cuda")
    for c in range(shape[0]):
        noise = torch.randn(shape[1:], dtype=torch.float64, device="cuda", generator=gen)
        out[c] = dft.back(dft.forward(noise) * amp)
        if depth_decay is not None:
            out[c] *= depth_decay
    return out


def _eigenstrain(g, gen):
    z = torch.linspace(0.0, g["lz"], g["nz"], dtype=torch.float64, device="cuda")
    f = _filtered((6, g["nz"], g["ny"], g["nx"]), gen, torch.exp(-z / 0.1)[:, None, None])
    return f.mul_(1e-3 / float(torch.linalg.vector_norm(f, float("inf"))))


def _traction(g, gen):
    f = _filtered((3, g["ny"], g["nx"]), gen)
    return f.mul_(1e-2 / float(f.abs().max()))


def _rough(nx, ny, ly, hurst, k_roll, k_cut, gen):
    """Self-affine profile, rms slope 0.1, highest point at 0."""
    kx, ky = _plane(_wavenumbers(nx, ny))
    k = torch.hypot(kx, ky)
    psd = torch.zeros_like(k)
    psd[(k >= 1) & (k < k_roll)] = 1.0
    tail = (k >= k_roll) & (k <= k_cut)
    psd[tail] = (k[tail] / k_roll) ** (-2.0 * (1.0 + hurst))
    phase = 2.0 * math.pi * torch.rand(k.shape, dtype=torch.float64, device="cuda", generator=gen)
    h = _Dft(nx, ny).back(torch.polar(psd.sqrt(), phase))
    # rms slope from the spectrum of the profile
    w = _Dft(nx, ny).forward(h).abs() / (nx * ny)
    w[:, 1:-1] *= math.sqrt(2.0)
    q2 = (2.0 * math.pi) ** 2 * (kx ** 2 + (ky / ly) ** 2)
    h = h * (0.1 / torch.sqrt((q2 * w ** 2).sum()))
    return (h - h.max()).contiguous()


def _spots(nx, ny, ly, gen):
    """Pressure of some twenty Hertzian contact spots."""
    x = torch.arange(nx, device="cuda").double() / nx
    y = torch.arange(ny, device="cuda").double() * (ly / ny)
    r = torch.rand((20, 3), dtype=torch.float64, device="cuda", generator=gen)
    p = torch.zeros((ny, nx), dtype=torch.float64, device="cuda")
    for cx, cy, a in r.tolist():
        dx, dy = x - cx, y - ly * cy
        dx, dy = dx - torch.round(dx), dy - ly * torch.round(dy / ly)
        rad = min(1.0, ly) * (0.02 + 0.06 * a)
        p += 0.5 * rad * torch.sqrt(torch.clamp(1.0 - (dx[None, :] ** 2 + dy[:, None] ** 2) / rad ** 2, min=0.0))
    return p


def _surface(c, gen):
    """Profile of a solve case; the paraboloid's place comes from the seed."""
    nx, ny = c["nx"], c["ny"]
    if c["surface"] == "rough":
        return _rough(nx, ny, 1.0, 0.7, 4, nx // 4, gen)
    s = torch.rand(2, dtype=torch.float64, device="cuda", generator=gen).tolist()
    x, y = torch.arange(nx, device="cuda").double() / nx - s[0], torch.arange(ny, device="cuda").double() / ny - s[1]
    x, y = x - torch.round(x), y - torch.round(y)
    return (-(x[None, :] ** 2 + y[:, None] ** 2)).contiguous()             # R = 0.5


def _grid(nx, ny, nz, ly=1.0, lz=0.25):
    return {"nx": nx, "ny": ny, "nz": nz, "lx": 1.0, "ly": ly, "lz": lz}


def _grids(c):
    return [_grid(*(int(v) for v in t.split("x"))) for t in c["grids"].split(",")]


def _nodes(c):
    """Depth nodes of a graded case (None: uniform)."""
    if not c["graded"]:
        return None
    n = c["nz"] - 1
    z = [c["lz"] * (i / n) ** c["graded"] for i in range(n + 1)]
    z[-1] = c["lz"]
    return z


def _inputs(c, seed):
    gen = _gen(seed)
    kind = c["kind"]
    if kind == "operator":
        g = _grid(c["nx"], c["ny"], c["nz"], c["ly"], c["lz"])
        return {"g": g, "eps": _eigenstrain(g, gen) if c["op"] != "boussinesq" else None,
                "t": _traction(g, gen) if c["op"] != "mindlin" else None}
    if kind == "batch":
        return [{"g": g, "eps": _eigenstrain(g, gen), "t": _traction(g, gen)} for g in _grids(c)]
    if kind == "return_map":
        f = (c["nz"], c["ny"], c["nx"])
        r = lambda s: torch.randn(s, dtype=torch.float64, device="cuda", generator=gen)
        return {"g": _grid(*f[::-1]), "d_eps": r((6,) + f).mul_(0.003), "sigma": r((6,) + f).mul_(0.003),
                "ep": r(f).mul_(0.01).abs_()}
    if kind == "contact":
        return {"g": _grid(c["nx"], c["ny"], 2, c["ly"]),
                "h": _rough(c["nx"], c["ny"], c["ly"], c["hurst"], c["k_roll"], c["k_cut"], gen)}
    if kind == "tangential":
        p = _spots(c["nx"], c["ny"], c["ly"], gen)
        W = float(p.mean()) * c["ly"]
        a = float(torch.rand(1, dtype=torch.float64, device="cuda", generator=gen)) * 2.0 * math.pi
        Q = c["q_ratio"] * c["mu_f"] * W
        return {"g": _grid(c["nx"], c["ny"], 2, c["ly"]), "p": p, "Q": (Q * math.cos(a), Q * math.sin(a))}
    return {"g": _grid(c["nx"], c["ny"], c["nz"]), "h": _surface(c, gen)}


# -------------------------------------------------------------- the measured
def prepare(case, seed):
    s = {"case": case, "in": _inputs(case, seed)}
    kind = case["kind"]
    prec = case.get("precision", "fp64")
    if kind == "batch":
        s["ctx"] = [Context(i["g"], E, NU, precision=prec) for i in s["in"]]
        return s
    s["ctx"] = ctx = Context(s["in"]["g"], E, NU, SY0, EH, precision=prec)
    if kind == "operator":
        if case["graded"]:
            ctx.set_depth_nodes(_nodes(case))
        shapes = {"strain": ctx.tensor_shape, "stress": ctx.tensor_shape, "disp": ctx.vector_shape,
                  "surf_u3": ctx.surface_shape}
        s["out"] = {k: torch.empty(shapes[k], dtype=torch.float64, device="cuda") for k in case["want"].split(",")}
    elif kind == "return_map":
        s["out"] = {"d_eps_p": torch.empty(ctx.tensor_shape, dtype=torch.float64, device="cuda"),
                    "d_ep": torch.empty(ctx.scalar_shape, dtype=torch.float64, device="cuda"),
                    "sigma_np1": torch.empty(ctx.tensor_shape, dtype=torch.float64, device="cuda")}
    elif kind == "solve":
        # tolerances at which a solution is determined to well below 1e-9
        s["opts"] = EPOptions(tol_outer=1e-12, relax=0.3, tol_plastic=1e-12, tol_contact=1e-14, max_outer=400,
                              max_plastic=20000, max_contact=50000, anderson_m=5, warm_start=1, inner_rel=0.1)
    return s


def run(s):
    c, i, ctx = s["case"], s["in"], s["ctx"]
    kind = c["kind"]
    if kind == "operator":
        if c["op"] == "fused":
            return ctx.operator_apply(i["eps"], i["t"], want=(), out=s["out"])
        if c["op"] == "mindlin":
            return ctx.mindlin_apply(i["eps"], want=(), out=s["out"])
        return ctx.boussinesq_apply(i["t"], want=(), out=s["out"])
    if kind == "batch":
        return operator_apply_batch(ctx, [x["eps"] for x in i], [x["t"] for x in i])
    if kind == "return_map":
        return ctx.return_map(i["d_eps"], i["sigma"], i["ep"], **s["out"])
    if kind == "contact":
        p, gap, _ = ctx.contact_solve(i["h"], c["load"] * c["ly"], tol=1e-12, max_iter=50000, want_gap=True)
        return {"p": p, "gap": gap}
    if kind == "tangential":
        return ctx.tangential_solve(i["p"], c["mu_f"], i["Q"], tol=1e-12)[0]
    st = ctx.new_state()
    ctx.elastoplastic_solve(i["h"], [c["load"] * (k + 1) / c["steps"] for k in range(c["steps"])], st, s["opts"])
    return st


def _op_work(nx, ny, nz, pin, pout):
    v, m = nx * ny, (nx // 2 + 1) * ny
    return {"bytes": 8.0 * v * (pin + pout),
            "flops": 2.5 * v * math.log2(v) * (pin + pout) + 300.0 * m * nz}


def work(case):
    kind = case["kind"]
    if kind == "operator":
        nz = case["nz"]
        planes = {"strain": 6 * nz, "stress": 6 * nz, "disp": 3 * nz, "surf_u3": 1}
        pin = (6 * nz if case["op"] != "boussinesq" else 0) + (3 if case["op"] != "mindlin" else 0)
        return _op_work(case["nx"], case["ny"], nz, pin, sum(planes[k] for k in case["want"].split(",")))
    if kind == "batch":
        w = [_op_work(g["nx"], g["ny"], g["nz"], 6 * g["nz"] + 3, 6 * g["nz"]) for g in _grids(case)]
        return {k: sum(x[k] for x in w) for k in ("bytes", "flops")}
    n = case["nx"] * case["ny"]
    if kind == "return_map":
        return {"bytes": 8.0 * 26 * n * case["nz"], "flops": 70.0 * n * case["nz"]}
    # an iterative solve: its inputs and outputs, and one step of its iteration
    if kind == "contact":
        return {"bytes": 8.0 * 3 * n, "flops": 10.0 * n * math.log2(n) + 30.0 * n}
    if kind == "tangential":
        return {"bytes": 8.0 * 3 * n, "flops": 10.0 * n * math.log2(n) + 60.0 * n}
    w = _op_work(case["nx"], case["ny"], case["nz"], 6 * case["nz"] + 3, 6 * case["nz"])
    return {"bytes": case["steps"] * 8.0 * n * (13 * case["nz"] + 5), "flops": case["steps"] * w["flops"]}


# ------------------------------------------------------- 64-bit plain torch
def _element(s):
    """exp(-s) and G0, G0', H0, H0': s times the integrals over 0 < t < 1 of
    (1 - t) e, t e and s^2 times those of t (1 - t) e, t^2 e, e = exp(-s t)."""
    x, small = s.clamp(min=1.0), s < 1.0
    e = torch.exp(-x)
    i0, i1, i2 = 1 - e, 1 - e * (1 + x), 2 - e * (2 + x * (2 + x))
    closed = (i0 - i1 / x, i1 / x, i1 - i2 / x, i2 / x)
    y = torch.where(small, s, torch.zeros_like(s))
    series = [torch.zeros_like(s) for _ in range(4)]
    for k in range(24, -1, -1):
        f = (-1.0) ** k / math.factorial(k)
        for j, d in enumerate(((k + 1) * (k + 2), k + 2, (k + 2) * (k + 3), k + 3)):
            series[j] = series[j] * y + f / d
    series = [series[0] * y, series[1] * y, series[2] * y * y, series[3] * y * y]
    return (torch.exp(-s),) + tuple(torch.where(small, a, b) for a, b in zip(series, closed))


def _modes(q1, q2, z, ep, t, want_disp):
    """Strain [6][nz][M] (and displacement [3][nz][M]) of the modes
    exp(i (q1 x + q2 y)), |q| > 0, of the half-space with the P1 eigenstrain ep
    [6][nz][M] under the traction t [3][M]: the decaying solution in depth by
    exact propagators over each element, growing coordinates upwards from zero
    below the last node, decaying ones downwards from the surface condition."""
    kap = LAM / MU
    q = torch.sqrt(q1 * q1 + q2 * q2)
    n1, n2 = q1 / q, q2 / q
    nz = len(z)
    kp2 = kap + 2
    kk = (kap + 1) / kp2
    tr = kap * (ep[0] + ep[1] + ep[2])
    o0 = tr + 2 * (n1 * n1 * ep[0] + 2 * n1 * n2 * ep[5] + n2 * n2 * ep[1])
    o1 = tr + 2 * ep[2]
    o2 = -2j * (n1 * ep[4] + n2 * ep[3])
    o3 = -2j * ((n1 * n1 - n2 * n2) * ep[5] - n1 * n2 * (ep[0] - ep[1]))
    o4 = 2 * (n1 * ep[3] - n2 * ep[4])
    ec, et = o1 / kp2, o0 - kap / kp2 * o1
    f0 = -kk * ec - et / (2 * kp2)
    f1 = kk * (0.5 * et - ec - o2)
    f3 = kk * (0.5 * et - ec + o2)
    fm, fp = 0.5 * (o4 + o3), 0.5 * (o4 - o3)
    steps = {}

    def elem(e):
        h = z[e + 1] - z[e]
        if h not in steps:
            steps[h] = (q * h,) + _element(q * h)
            if len(steps) > 2:
                steps.pop(next(iter(steps)))
        return steps[h]

    m2, m3, mp = (torch.zeros_like(ep[0]) for _ in range(3))
    for e in range(nz - 2, -1, -1):
        s, r, g0, g0p, h0, h0p = elem(e)
        m3[e] = r * m3[e + 1] - f3[e] * g0 - f3[e + 1] * g0p
        m2[e] = r * (m2[e + 1] - s * m3[e + 1]) + f0[e] * g0 + f0[e + 1] * g0p + f3[e] * h0 + f3[e + 1] * h0p
        mp[e] = r * mp[e + 1] - fp[e] * g0 - fp[e + 1] * g0p
    m0, m1, mm = (torch.zeros_like(ep[0]) for _ in range(3))
    m0[0] = -t[2] - m2[0]
    m1[0] = 1j * (n1 * t[0] + n2 * t[1]) + m0[0] - m2[0] - m3[0]
    mm[0] = mp[0] - (n2 * t[0] - n1 * t[1])
    for e in range(nz - 1):
        s, r, g0, g0p, h0, h0p = elem(e)
        m1[e + 1] = r * m1[e] + f1[e] * g0p + f1[e + 1] * g0
        m0[e + 1] = r * (m0[e] + s * m1[e]) + f0[e] * g0p + f0[e + 1] * g0 + f1[e] * h0p + f1[e + 1] * h0
        mm[e + 1] = r * mm[e] + fm[e] * g0p + fm[e + 1] * g0
    a = 0.5 * (m0 + m2) + (m3 - m1) / (2 * kk)
    v = mp + mm
    exx, exe = -a, 0.5j * v
    ezz = (kap * a + m0 + m2 + o1) / kp2
    exz = 0.5j * (m1 - m0 + m2 + m3 + o2)
    eez = 0.5 * (mp - mm + o4)
    strain = torch.stack([n1 * n1 * exx - 2 * n1 * n2 * exe, n2 * n2 * exx + 2 * n1 * n2 * exe, ezz,
                          n2 * exz + n1 * eez, n1 * exz - n2 * eez, n1 * n2 * exx + (n1 * n1 - n2 * n2) * exe])
    if not want_disp:
        return strain, None
    c = 0.5 * (m2 - m0) - (m1 + m3) / (2 * (kap + 1))
    U, V = 1j * a / q, v / q
    return strain, torch.stack([n1 * U - n2 * V, n2 * U + n1 * V, c / q])


def _operator_exact(g, eps, t, want, z=None):
    nx, ny, nz = g["nx"], g["ny"], g["nz"]
    z = z or [i * g["lz"] / (nz - 1) for i in range(nz)]
    kxh, dft = nx // 2 + 1, _Dft(nx, ny)
    zero = lambda *s: torch.zeros(s, dtype=torch.complex128, device="cuda")
    scale = 1.0 / (nx * ny)
    nm = ny * kxh                         # modes are indexed ky * kxh + kx
    eh = (dft.forward(eps) * scale).view(6, nz, nm) if eps is not None else zero(6, nz, nm)
    th = (dft.forward(t) * (scale / MU)).view(3, nm) if t is not None else zero(3, nm)
    disp = "disp" in want or "surf_u3" in want
    kx, ky = (k.expand(ny, kxh).reshape(nm) for k in _plane(_wavenumbers(nx, ny)))
    q1, q2 = 2 * math.pi * kx, 2 * math.pi / g["ly"] * ky
    sh, dh = zero(6, nz, nm), zero(3, nz, nm) if disp else None

    def put(sel, signs):                  # modes sel <- the mean over the sign replicas
        a, b = q1[sel], q2[sel]
        for s1, s2 in signs:
            st, d = _modes(s1 * a, s2 * b, z, eh[:, :, sel], th[:, sel], disp)
            sh[:, :, sel] += st / len(signs)
            if disp:
                dh[:, :, sel] += d / len(signs)

    nyx, nyy = 2 * kx == nx, 2 * ky == ny
    plain = ~(nyx | nyy)
    plain[0] = False
    for part in plain.nonzero()[:, 0].split(max(1, (1 << 24) // nz)):     # bounds the scratch memory
        put(part, [(1, 1)])
    put((nyx & ~nyy).nonzero()[:, 0], [(1, 1), (-1, 1)])
    put((nyy & ~nyx).nonzero()[:, 0], [(1, 1), (1, -1)])
    put((nyx & nyy).nonzero()[:, 0], [(1, 1), (-1, 1), (1, -1), (-1, -1)])
    # laterally uniform mode: sigma . e3 = -t, no in-plane strain
    e0, t0 = eh[:, :, 0], th[:, 0]
    sh[4, :, 0] = e0[4] - 0.5 * t0[0]
    sh[3, :, 0] = e0[3] - 0.5 * t0[1]
    kap = LAM / MU
    sh[2, :, 0] = (kap * (e0[0] + e0[1] + e0[2]) + 2 * e0[2] - t0[2]) / (kap + 2)
    back = lambda f: dft.back(f.view(f.shape[:-1] + (ny, kxh))) * (nx * ny)
    out = {}
    if "strain" in want or "stress" in want:
        out["strain"] = back(sh)
    if "stress" in want:
        el = out["strain"] - eps if eps is not None else out["strain"]
        out["stress"] = 2 * MU * el
        out["stress"][:3] += LAM * (el[0] + el[1] + el[2])
    if "disp" in want:
        out["disp"] = back(dh)
    if "surf_u3" in want:
        out["surf_u3"] = back(dh[2, 0])
    return {k: out[k] for k in want}


def _return_map_exact(i):
    de, sn, ep = i["d_eps"], i["sigma"], i["ep"]
    s = sn + 2 * MU * de
    s[:3] += LAM * (de[0] + de[1] + de[2])
    d = s.clone()
    d[:3] -= (s[0] + s[1] + s[2]) / 3
    seq = torch.sqrt(1.5 * ((d[:3] ** 2).sum(0) + 2 * (d[3:] ** 2).sum(0)))
    dp = torch.clamp(seq - (SY0 + EH * ep), min=0.0) / (3 * MU + EH)
    dep = torch.where(dp > 0, 1.5 * dp / seq, torch.zeros_like(dp)) * d
    return dep, dp, s - 2 * MU * dep


def _wavevectors(g):
    kx, ky = _plane(_wavenumbers(g["nx"], g["ny"]))
    q1, q2 = 2 * math.pi * kx, 2 * math.pi / g["ly"] * ky
    q = torch.sqrt(q1 ** 2 + q2 ** 2)
    q[0, 0] = 1.0
    return q1, q2, q


def _contact_exact(i, c):
    """Conjugate gradients on the contact set with projection (Polonsky and
    Keer), run until the pressure no longer changes."""
    g, h, W = i["g"], i["h"], c["load"] * c["ly"]
    n, dft = h.numel(), _Dft(g["nx"], g["ny"])
    m = 2 * (1 - NU ** 2) / E / _wavevectors(g)[2]
    m[0, 0] = 0.0
    M = lambda f: dft.back(dft.forward(f) * m)
    dA = g["ly"] / n
    p, t = torch.full_like(h, W / g["ly"]), torch.zeros_like(h)
    G0, delta, err = 1.0, 0.0, 1.0
    for _ in range(4000):
        on = p > 0
        gap = M(p) - h
        gap = gap - gap[on].mean()
        G = float((gap[on] ** 2).sum())
        t = torch.where(on, gap + delta * G / G0 * t, torch.zeros_like(t))
        G0 = G
        r = M(t)
        r = r - r[on].mean()
        den = float((r[on] * t[on]).sum())
        tau = float((gap[on] * t[on]).sum()) / den if den else 0.0
        new = torch.clamp(p - tau * t, min=0.0)
        enter = (new == 0) & (gap < 0)
        new = torch.where(enter, -tau * gap, new)
        delta = 0.0 if bool(enter.any()) else 1.0
        new = new * (W / (dA * float(new.sum())))
        err = dA * float((new - p).abs().sum()) / W
        p = new
        if err < 3e-15:
            break
    gap = M(p) - h
    return {"p": p, "gap": gap - gap[p > 0].mean()}


def _tangential_exact(i, c):
    """Accelerated projected gradient; each step's load constraint by Newton's
    method on the rigid shift."""
    g, rho = i["g"], c["mu_f"] * i["p"]
    n, dft = rho.numel(), _Dft(g["nx"], g["ny"])
    q1, q2, q = _wavevectors(g)
    n1, n2 = (q1 / q).expand_as(q), (q2 / q).expand_as(q)
    cross = -NU * n1 * n2
    cross[:, -1] = 0.0
    cross[g["ny"] // 2] = 0.0
    f = 1.0 / (MU * q)
    f[0, 0] = 0.0

    def C(a):
        s = dft.forward(a)
        return dft.back(f * torch.stack([(1 - NU * n1 ** 2) * s[0] + cross * s[1],
                                         cross * s[0] + (1 - NU * n2 ** 2) * s[1]]))

    S = torch.tensor(i["Q"], dtype=torch.float64, device="cuda") / (g["ly"] / n)
    inv_l = MU * 2 * math.pi * min(1.0, 1.0 / g["ly"])
    lam = torch.zeros(2, dtype=torch.float64, device="cuda")
    W = float(i["p"].sum())
    x = rho * (S / (c["mu_f"] * W))[:, None, None]
    y, tk = x.clone(), 1.0
    eye = torch.eye(2, dtype=torch.float64, device="cuda")
    for it in range(6000):
        v = y - inv_l * C(y)
        for _ in range(3):
            w = v + lam[:, None, None]
            r = torch.sqrt(w[0] ** 2 + w[1] ** 2)
            slip = r > rho
            rs = torch.where(slip, r, torch.ones_like(r))
            s = torch.where(slip, rho / rs, torch.ones_like(r))
            b = torch.where(slip, rho / rs ** 3, torch.zeros_like(r))
            P = s * w
            j12 = -(b * w[0] * w[1]).sum()
            J = torch.stack([torch.stack([(s - b * w[0] ** 2).sum(), j12]), torch.stack([j12, (s - b * w[1] ** 2).sum()])])
            lam = lam - torch.linalg.solve(J + 1e-14 * (J.trace() + 1.0) * eye, P.sum((1, 2)) - S)
        w = v + lam[:, None, None]
        new = w * torch.clamp(rho / torch.sqrt(w[0] ** 2 + w[1] ** 2).clamp(min=1e-300), max=1.0)
        d = new - x
        if it % 8 == 7 and float(d.abs().sum()) < 1e-14 * c["mu_f"] * W:
            return new
        if float(((y - new) * d).sum()) > 0:
            tk, beta = 1.0, 0.0
        else:
            tn = 0.5 * (1 + math.sqrt(1 + 4 * tk * tk))
            beta, tk = (tk - 1) / tn, tn
        x, y = new, new + beta * d
    return x


def exact(case, seed):
    i = _inputs(case, seed)
    kind = case["kind"]
    if kind == "operator":
        return _operator_exact(i["g"], i["eps"], i["t"], case["want"].split(","), _nodes(case))
    if kind == "batch":
        return [_operator_exact(x["g"], x["eps"], x["t"], ["strain"]) for x in i]
    if kind == "return_map":
        return _return_map_exact(i)
    if kind == "contact":
        return _contact_exact(i, case)
    if kind == "tangential":
        return _tangential_exact(i, case)
    return None                            # a coupled solve: minutes in plain torch
