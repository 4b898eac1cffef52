"""The work that users of this solver have it do, as measured cases.

One case is one call (or one batch of requests) through the public entry
points, at sizes of the repository's own configurations or generic ones:
solves of small, ordinary and large grids with each precision,
preconditioner and upper boundary, from device and host arrays; a fixed
number of iterations on a grid that streams from HBM; the operator, the
preconditioner and the field output by themselves; and the batching server.

    listed()           the named cases
    draw(rng)          one more case of the same ranges
    prepare(case, s)   inputs of seed s and the context a program keeps
    run(state)         one pass
    work(case)         bytes and operations a pass cannot do without
    exact(case, s)     what run returns, by plain torch and numpy in FP64

A converged solve returns Phi (and the pole values where the program asks for
them).  The iteration count and the residual at exit are not returned: they
say after which step the tolerance was met, and any change of rounding moves
them by a step.  A solve of a fixed count returns its count too.
"""
import math

import numpy as np
import torch

import paper_1709_01126_amd as pot3d
from paper_1709_01126_amd.pot3d import pot3d_solve_noalloc

R1 = 2.5
TOL = 1e-10
MAXIT = 40_000


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _case(kind, nr, nt, np_, name=None, **more):
    c = {"kind": kind, "nr": nr, "nt": nt, "np": np_}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # the smallest configured grid: a quick look at a low-resolution map, bound by latency
        _case("solve", 32, 64, 128, "solve_32x64x128", theta="uniform"),
        # the most frequent size of the serving trace, one at a time
        _case("solve", 64, 128, 256, "solve_64x128x256"),
        # a ragged grid with the closed upper wall, and the pole values with it
        _case("solve", 45, 91, 179, "closed_45x91x179", closed=True, poles=True),
        # the middle size of the serving trace, from and to host arrays
        _case("solve", 101, 201, 401, "host_101x201x401", host=True),
        # the configured benchmark grid: the headline solve
        _case("solve", 151, 301, 601, "solve_151x301x601"),
        # the same grid with FP32 inner iterations
        _case("solve", 151, 301, 601, "refined_151x301x601", refined=True),
        # the same grid with the phi-line preconditioner
        _case("solve", 151, 301, 601, "line_151x301x601", line=True),
        # the largest configured grid, where every vector streams from HBM: a fixed count of iterations
        # (few: by the fortieth, two runs that differ in the last bit differ by 1e-9)
        _case("solve", 301, 641, 1281, "fixed_301x641x1281", iters=16),
        # the operator by itself (a program's own Krylov method, or a check of a residual)
        _case("apply", 151, 301, 601, "apply_151x301x601"),
        # the phi-line preconditioner by itself
        _case("precondition", 101, 201, 401, "precondition_101x201x401", line=True),
        # the magnetic field of a potential: what most users want in the end
        _case("field", 151, 301, 601, "field_151x301x601"),
        # a burst of requests at the batching server: small ones beside a larger one
        _case("server", 64, 128, 256, "server_burst", small=4, large=1),
    ]


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["fixed", "apply", "precondition", "field"])

    def size(lo, hi):
        np_ = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        nt = max(8, int(round(np_ * rng.uniform(0.4, 0.6))))
        nr = max(6, int(round(np_ * rng.uniform(0.2, 0.3))))
        return nr, nt, np_

    if kind == "solve":
        nr, nt, np_ = size(48, 440)
        c = _case("solve", nr, nt, np_)
        how = rng.choice(["plain", "plain", "refined", "line", "refined_line", "closed", "host", "noalloc"])
        if how == "noalloc":
            nr, nt, np_ = size(48, 240)   # what its fixed scratch takes
            return _case("solve", nr, nt, np_, noalloc=True)
        for opt in how.split("_"):
            if opt != "plain":
                c[opt] = True
        return c
    if kind == "fixed":
        nr, nt, np_ = size(300, 1281)
        return _case("solve", nr, nt, np_, iters=rng.randint(8, 16))
    nr, nt, np_ = size(64, 601)
    c = _case(kind, nr, nt, np_)
    if kind == "precondition":
        c["line"] = rng.random() < 0.5
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _faces(case, nr=None, nt=None, np_=None):
    """Radially stretched, polar cells three times wider at the poles (or uniform), uniform azimuth."""
    nr, nt, np_ = nr or case["nr"], nt or case["nt"], np_ or case["np"]
    b = 151.0 * math.log(1.02)
    rf = 1.0 + (R1 - 1.0) * np.expm1(b * np.arange(nr + 1) / nr) / math.expm1(b)
    rf[0], rf[-1] = 1.0, R1
    s = np.arange(nt + 1) / nt
    tf = math.pi * s
    if case.get("theta") != "uniform":
        tf = tf + 0.25 * np.sin(2.0 * math.pi * s)
    tf[0], tf[-1] = 0.0, math.pi
    pf = 2.0 * math.pi * np.arange(np_ + 1) / np_
    pf[-1] = 2.0 * math.pi
    return rf, tf, pf


def _surface_map(tf, pf, seed, device, bipoles=60):
    """A dipole and Gaussian bipoles (active regions) of power-law flux: the character of an observed map."""
    g = np.random.default_rng(seed)
    tc = torch.from_numpy(0.5 * (tf[:-1] + tf[1:])).to(device)[:, None]
    pc = torch.from_numpy(0.5 * (pf[:-1] + pf[1:])).to(device)[None, :]
    st, ct = torch.sin(tc), torch.cos(tc)
    ex, ey = st * torch.cos(pc), st * torch.sin(pc)
    br = 5.0 * ct * torch.ones_like(pc)
    for _ in range(bipoles):
        z, lon, tilt = g.uniform(-0.95, 0.95), g.uniform(0.0, 2.0 * math.pi), g.uniform(0.0, 2.0 * math.pi)
        sigma = math.radians(g.uniform(2.0, 5.0))
        u = g.uniform()
        flux = (0.01 ** -0.8 - u * (0.01 ** -0.8 - 1.0)) ** (-1.25)
        c = np.array([math.sqrt(1.0 - z * z) * math.cos(lon), math.sqrt(1.0 - z * z) * math.sin(lon), z])
        north = np.array([-z * math.cos(lon), -z * math.sin(lon), math.sqrt(1.0 - z * z)])
        east = np.array([-math.sin(lon), math.cos(lon), 0.0])
        t = math.cos(tilt) * north + math.sin(tilt) * east
        for sign in (1.0, -1.0):
            a = math.cos(2.0 * sigma) * c + sign * math.sin(2.0 * sigma) * t
            cosd = ex * a[0] + ey * a[1] + ct * a[2]
            br += (sign * flux / (2.0 * math.pi * sigma * sigma)) * torch.exp((cosd - 1.0) / (sigma * sigma))
    return br.contiguous()


def _potential(rf, tf, pf, seed, device):
    """A smooth potential that decays with r: low multipoles with seeded amplitudes."""
    g = np.random.default_rng(seed)
    rc, tc, pc = (torch.from_numpy(0.5 * (f[:-1] + f[1:])).to(device) for f in (rf, tf, pf))
    out = torch.zeros((rc.numel(), tc.numel(), pc.numel()), dtype=torch.float64, device=device)
    for m in range(6):
        c = g.normal(size=2)
        ang = (c[0] * torch.sin(tc) ** m * torch.cos(tc))[:, None] * torch.cos(m * pc + c[1])[None, :]
        out += (rc ** -(m + 2.0) - R1 ** (-2.0 * m - 3.0) * rc ** (m + 1.0))[:, None, None] * ang
    return out


def _solver(case, faces):
    s = pot3d.Solver(*faces, upper_bc=pot3d.UPPER_CLOSED_WALL if case.get("closed") else pot3d.UPPER_SOURCE_SURFACE,
                     precision=pot3d.FP32_REFINED if case.get("refined") else pot3d.FP64, device=0)
    if case.get("line"):
        s.set_preconditioner(pot3d.PC_PHI_LINE)
    return s


def _requests(case, seed, device):
    """The server's requests: grids and surface maps, in the order of their submission."""
    sizes = [(case["nr"], case["nt"], case["np"])] * case["small"]
    sizes[1:1] = [(101, 201, 401)] * case["large"]
    out = []
    for q, (nr, nt, np_) in enumerate(sizes):
        faces = _faces(case, nr, nt, np_)
        out.append((faces, _surface_map(faces[1], faces[2], seed * 16 + q, device)))
    return out


def prepare(case, seed):
    dev = torch.device("cuda", 0)
    st = {"case": case}
    if case["kind"] == "server":
        st["requests"] = [(f, br.cpu().numpy()) for f, br in _requests(case, seed, dev)]
        st["server"] = pot3d.Server(max_slots=8, device=0)
        return st
    faces = st["faces"] = _faces(case)
    rf, tf, pf = faces
    shape = (len(rf) - 1, len(tf) - 1, len(pf) - 1)
    if not case.get("noalloc"):
        st["solver"] = _solver(case, faces)
    if case["kind"] in ("apply", "precondition"):
        gen = torch.Generator(device=dev).manual_seed(seed)
        st["x"] = torch.randn(shape, dtype=torch.float64, device=dev, generator=gen)
        st["y"] = torch.empty_like(st["x"])
        return st
    br = _surface_map(tf, pf, seed, dev)
    if case["kind"] == "field":
        # the context of a program that has its potential already (from a file, say)
        phi = _potential(rf, tf, pf, seed, dev)
        torch.cuda.synchronize()   # the solver works on a stream of its own beside torch's default one
        st["solver"].solve_device(br, torch.empty_like(phi), 0.0, 0, phi0=phi)
        return st
    if case.get("host"):
        st["br"] = br.cpu().numpy()
    else:
        st["br"] = br
        st["phi"] = torch.empty(shape, dtype=torch.float64, device=dev)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "server":
        sv = st["server"]
        ids = [sv.submit(*faces, br, TOL, MAXIT) for faces, br in st["requests"]]
        while True:
            active, queued, _ = sv.step()
            if not active and not queued:
                break
        return [sv.take(i)[0] for i in ids]
    if kind == "apply":
        st["solver"].apply(st["x"], st["y"])
        return st["y"]
    if kind == "precondition":
        st["solver"].precondition(st["x"], st["y"])
        return st["y"]
    if kind == "field":
        return st["solver"].field()
    tol, maxit = (0.0, case["iters"]) if case.get("iters") else (TOL, MAXIT)
    if case.get("noalloc"):
        pot3d_solve_noalloc(*st["faces"], pot3d.UPPER_SOURCE_SURFACE, st["br"].data_ptr(), None,
                            st["phi"].data_ptr(), torch.cuda.current_stream().cuda_stream, tol, maxit)
        return st["phi"]
    s = st["solver"]
    if case.get("host"):
        return s.solve(st["br"], tol, maxit)[0]
    _, iters, _ = s.solve_device(st["br"], st["phi"], tol, maxit)
    if case.get("iters"):
        return [st["phi"], iters]
    if case.get("poles"):
        return [st["phi"], *s.pole_values()]
    return st["phi"]


def _iterations(case, np_):
    """About how many PCG iterations a solve to TOL takes: they grow with the azimuthal resolution."""
    return case.get("iters") or (4.0 if case.get("line") else 10.0) * np_


def work(case):
    def solve(nr, nt, np_):
        n = nr * nt * np_
        # per iteration and unknown: the 7-point operator, three vector updates, the preconditioner, three sums
        return 8.0 * (nt * np_ + n), _iterations(case, np_) * n * 27.0

    nr, nt, np_ = case["nr"], case["nt"], case["np"]
    n = float(nr * nt * np_)
    if case["kind"] == "server":
        small, large = solve(nr, nt, np_), solve(101, 201, 401)
        b, f = (case["small"] * small[q] + case["large"] * large[q] for q in (0, 1))
    elif case["kind"] == "apply":
        b, f = 16.0 * n, 13.0 * n
    elif case["kind"] == "precondition":
        b, f = 16.0 * n, 8.0 * n
    elif case["kind"] == "field":
        b, f = 8.0 * (n + nt * np_) + 8.0 * (3.0 * n + nt * np_ + nr * np_), 6.0 * n
    else:
        b, f = solve(nr, nt, np_)
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# the same in FP64 by plain torch and numpy
# ---------------------------------------------------------------------------
class _Scheme:
    """The finite-volume scheme of a grid with uniform azimuthal faces, from its faces alone."""

    def __init__(self, faces, closed, dev):
        rf, tf, pf = faces
        self.nr, self.nt, self.np = len(rf) - 1, len(tf) - 1, len(pf) - 1
        self.dev = dev
        self.h = 2.0 * math.pi / self.np
        rc, tc = 0.5 * (rf[:-1] + rf[1:]), 0.5 * (tf[:-1] + tf[1:])
        self.dr, dt = np.diff(rf), np.diff(tf)
        self.rc, self.sin = rc, np.sin(tc)
        self.face = self.sin * dt                                     # r-face area / (r^2 h)
        self.a = np.zeros(self.nr + 1)                                # radial couplings, on the faces
        self.a[1:-1] = rf[1:-1] ** 2 / np.diff(rc)
        if not closed:
            self.a[-1] = rf[-1] ** 2 / (rf[-1] - rc[-1])
        self.c = np.zeros(self.nt + 1)                                # polar couplings, on the faces
        self.c[1:-1] = np.sin(tf[1:-1]) / np.diff(tc)
        self.q = dt / self.sin                                        # azimuthal coupling * h / dr
        self.rf, self.tf, self.tc, self.closed = rf, tf, tc, closed

    def t(self, a):
        return torch.as_tensor(a, dtype=torch.float64, device=self.dev)

    def diag(self):
        s = self.t(self.a[:-1] + self.a[1:])[:, None] * self.t(self.face) + self.t(self.dr)[:, None] * self.t(self.c[:-1] + self.c[1:])
        return (self.h * s + self.t(self.dr)[:, None] * self.t(self.q) * (2.0 / self.h))[:, :, None]

    def weights(self):
        """Diagonal without the azimuthal part, and the azimuthal weight, of every (r, theta) row."""
        w = self.t(self.dr)[:, None] * self.t(self.q) / self.h
        return self.diag()[:, :, 0] - 2.0 * w, w

    def apply(self, x):
        y = self.diag() * x
        y[1:] -= (self.h * self.t(self.a[1:-1]))[:, None, None] * self.t(self.face)[:, None] * x[:-1]
        y[:-1] -= (self.h * self.t(self.a[1:-1]))[:, None, None] * self.t(self.face)[:, None] * x[1:]
        k = (self.h * self.t(self.dr))[:, None, None] * self.t(self.c[1:-1])[:, None]
        y[:, 1:] -= k * x[:, :-1]
        y[:, :-1] -= k * x[:, 1:]
        w = self.weights()[1][:, :, None]
        y -= w * torch.roll(x, 1, 2)
        y -= w * torch.roll(x, -1, 2)
        return y

    def rhs(self, br):
        area = self.h * self.rf[0] ** 2 * self.t(self.face)[:, None]
        if self.closed:
            br = br - (area * br).sum() / (area.sum() * self.np)
        return area * br

    def solve(self, br):
        """A Phi = b exactly: Fourier modes in azimuth, eigenvectors in radius, elimination in the polar angle."""
        R = np.diag(self.a[:-1] + self.a[1:]) - np.diag(self.a[1:-1], 1) - np.diag(self.a[1:-1], -1)
        sq = 1.0 / np.sqrt(self.dr)
        mu, v = np.linalg.eigh(sq[:, None] * R * sq[None, :])
        V = self.t(sq[:, None] * v)
        if self.closed:
            mu[0] = 0.0
        bh = torch.fft.rfft(self.rhs(br) / self.h, dim=1)             # nt x modes, on the first layer
        modes = torch.arange(bh.shape[1], device=self.dev, dtype=torch.float64)
        lam = 4.0 * torch.sin(math.pi * modes / self.np) ** 2 / self.h ** 2
        mu_t, v0 = self.t(mu)[:, None], V[0][:, None]
        fac, c, q = self.face, self.c, self.q
        d = []
        y = torch.empty((self.nt, self.nr, bh.shape[1]), dtype=torch.complex128, device=self.dev)
        for j in range(self.nt):
            dj = fac[j] * mu_t + (c[j] + c[j + 1]) + q[j] * lam
            rj = v0 * bh[j]
            if j == 0 and self.closed:
                dj[0, 0] += 1.0      # the constant, fixed below by the mean
            if j:
                f = c[j] / d[-1]
                dj = dj - f * c[j]
                rj = rj + f * y[j - 1]
            d.append(dj)
            y[j] = rj
        y[-1] /= d[-1]
        for j in range(self.nt - 2, -1, -1):
            y[j] = (y[j] + c[j + 1] * y[j + 1]) / d[j]
        phi = torch.empty((self.nr, self.nt, self.np), dtype=torch.float64, device=self.dev)
        for j in range(self.nt):
            phi[:, j] = V @ torch.fft.irfft(y[j], n=self.np, dim=1)
        if self.closed:
            vol = self.t(self.rc ** 2 * self.dr)[:, None] * self.t(self.face)
            phi -= (vol[:, :, None] * phi).sum() / (vol.sum() * self.np)
        return phi

    def pcg(self, br, iters):
        """Textbook point-Jacobi PCG from zero, a fixed count."""
        x = torch.zeros((self.nr, self.nt, self.np), dtype=torch.float64, device=self.dev)
        r = torch.zeros_like(x)
        r[0] = self.rhs(br)
        inv = 1.0 / self.diag()
        dot = lambda a, b: torch.dot(a.reshape(-1), b.reshape(-1))  # noqa: E731
        p = r * inv
        rho = dot(r, p)
        for _ in range(iters):
            w = self.apply(p)
            alpha = rho / dot(p, w)
            x.add_(alpha * p)
            r.sub_(w.mul_(alpha))
            z = w.copy_(r).mul_(inv)
            new = dot(r, z)
            p.mul_(new / rho).add_(z)
            rho = new
        return x

    def field(self, phi, br):
        h = self.h
        bfr = torch.empty((self.nr + 1, self.nt, self.np), dtype=torch.float64, device=self.dev)
        bfr[0] = self.rhs(br) / (h * self.rf[0] ** 2 * self.t(self.face)[:, None])
        bfr[1:-1] = -(phi[1:] - phi[:-1]) / self.t(np.diff(self.rc))[:, None, None]
        bfr[-1] = 0.0 if self.closed else phi[-1] / (self.rf[-1] - self.rc[-1])
        bft = torch.zeros((self.nr, self.nt + 1, self.np), dtype=torch.float64, device=self.dev)
        bft[:, 1:-1] = -(phi[:, 1:] - phi[:, :-1]) / (self.t(np.diff(self.tc))[:, None] * self.t(self.rc)[:, None, None])
        bfp = -(torch.roll(phi, -1, 2) - phi) / (h * self.t(self.rc)[:, None, None] * self.t(self.sin)[:, None])
        return bfr, bft, bfp


def exact(case, seed):
    dev = torch.device("cuda", 0)
    if case["kind"] == "server":
        return [_Scheme(f, False, dev).solve(br) for f, br in _requests(case, seed, dev)]
    faces = _faces(case)
    rf, tf, pf = faces
    g = _Scheme(faces, bool(case.get("closed")), dev)
    shape = (g.nr, g.nt, g.np)
    if case["kind"] in ("apply", "precondition"):
        gen = torch.Generator(device=dev).manual_seed(seed)
        x = torch.randn(shape, dtype=torch.float64, device=dev, generator=gen)
        if case["kind"] == "apply":
            return g.apply(x)
        if not case.get("line"):
            return x / g.diag()
        s, w = g.weights()
        lam = 4.0 * torch.sin(math.pi * torch.arange(g.np // 2 + 1, device=dev, dtype=torch.float64) / g.np) ** 2
        return torch.fft.irfft(torch.fft.rfft(x, dim=2) / (s[:, :, None] + w[:, :, None] * lam), n=g.np, dim=2)
    br = _surface_map(tf, pf, seed, dev)
    if case["kind"] == "field":
        return g.field(_potential(rf, tf, pf, seed, dev), br)
    if case.get("iters"):
        return [g.pcg(br, case["iters"]), None]
    phi = g.solve(br)
    if case.get("poles"):
        return [phi, phi[:, 0].mean(1), phi[:, -1].mean(1)]
    return phi
