"""The work that a user of this framework has it do, as cases that can be timed.

Each case is one pass through the public entry points (`AlgMortar.pcg`,
`AlgMortar.apply`, set-up, `set_smoother`, `DarcyModel` / `AlgMortarSolve`) on
a two-point-flux Darcy system.  Grids, permeability fields, boundary
conditions, partitions and tolerances are those of the synthetic workloads
that the tests and the benchmark use, made here on the GPU.

A case's values:
  op      solve (PCG on a handle), apply (one preconditioner application),
          setup (a new matrix: set-up, one solve, release), gradient (forward
          and adjoint solve for one permeability, handle reused), smooth (PCG
          with block-Jacobi smoothing, one step before and after)
  nx, ny, nz   grid;  geom: cart (unit cells) or hex (displaced vertices)
  bx, by, bz   subdomain block, or 0: recursive bisection into 200..800 cells
  field   grf (ln K Gaussian), layered (log10 K in [-3, 3] by z-plane plus
          noise), cross (1e6 channels);  sigma, ell: of the Gaussian field
  nrhs, prec (precision of the local factors), tol
"""
import math

import numpy as np
import torch

import paper_2607_22905_amd as am

DEV = "cuda:0"


def _case(name, op, dims, block, field="grf", sigma=1.0, ell=8.0, geom="cart", nrhs=1,
          prec="fp64", tol=1e-8):
    c = dict(op=op, nx=dims[0], ny=dims[1], nz=dims[2], bx=block[0], by=block[1], bz=block[2],
             field=field, sigma=sigma, ell=ell, geom=geom, nrhs=nrhs, prec=prec, tol=tol)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest solve in use: a 2-D slice, 16 subdomains, latency bound
        _case("solve_2d_64", "solve", (64, 64, 1), (16, 16, 1), tol=1e-10),
        # one small preconditioner application, as another Krylov method calls it
        _case("apply_32", "apply", (32, 32, 32), (8, 8, 8), field="layered", sigma=1.5, ell=16.0),
        # a high-contrast reservoir model of ordinary size, many iterations
        _case("solve_layered_64", "solve", (64, 64, 64), (8, 8, 8), field="layered", sigma=1.5,
              ell=16.0),
        # the benchmark's system: the largest single right-hand side
        _case("solve_128", "solve", (128, 128, 128), (8, 8, 8)),
        # the same system with FP32 local factors (the mixed-precision form)
        _case("solve_128_fp32", "solve", (128, 128, 128), (8, 8, 8), prec="fp32"),
        # BF16 local factors to a tight tolerance
        _case("solve_64_bf16", "solve", (64, 64, 64), (8, 8, 8), prec="bf16", tol=1e-10),
        # one application on the largest system
        _case("apply_128", "apply", (128, 128, 128), (8, 8, 8)),
        # an irregular grid, uneven subdomains, a batch of well pairs
        _case("solve_hex_16rhs", "solve", (128, 128, 64), (0, 0, 0), sigma=2.0, geom="hex", nrhs=16),
        # a ragged irregular grid, four vectors at once
        _case("apply_hex_4rhs", "apply", (50, 45, 30), (0, 0, 0), sigma=2.0, geom="hex", nrhs=4),
        # parameter estimation: one gradient of a misfit, handle reused
        _case("gradient_96", "gradient", (96, 96, 96), (8, 8, 8), sigma=2.0, ell=12.0, tol=1e-10),
        # a new matrix solved once, on a ragged grid of 240-cell subdomains
        _case("setup_ragged", "setup", (50, 42, 36), (10, 6, 4), tol=1e-10),
        # the smoothed preconditioner (Sec. 5.4) on the high-contrast model
        _case("smooth_layered_64", "smooth", (64, 64, 64), (8, 8, 8), field="layered", sigma=1.5,
              ell=16.0),
    ]


def draw(rng):
    op = rng.choice(["solve", "solve", "solve", "apply", "apply", "setup", "gradient", "smooth"])
    most = {"solve": 128 ** 3, "apply": 128 ** 3, "setup": 160000, "gradient": 96 ** 3,
            "smooth": 64 ** 3}[op]
    field, sigma, ell, tol, prec, nrhs, geom = "grf", rng.choice([1.0, 2.0]), 8.0, 1e-8, "fp64", 1, "cart"
    if op in ("solve", "smooth") and rng.random() < 0.3:
        field, sigma, ell, most = rng.choice(["layered", "cross"]), 1.5, 16.0, min(most, 64 ** 3)
    if op == "solve" and field == "grf":
        prec = rng.choice(["fp64", "fp64", "fp64", "fp32", "bf16"])
        tol = 1e-10 if prec == "bf16" else rng.choice([1e-8, 1e-8, 1e-10])
    if op in ("gradient", "setup"):
        tol = 1e-10
    if op in ("solve", "apply") and prec == "fp64" and field != "cross" and rng.random() < 0.4:
        nrhs = rng.choice([2, 3, 4, 6, 8, 16])
        most = min(most, 128 * 128 * 64 * 16 // nrhs // (2 if nrhs < 16 else 1))
    n = math.exp(rng.uniform(math.log(4096), math.log(most)))
    if op in ("solve", "apply") and field == "grf" and rng.random() < 0.35:
        n = min(n, 128 * 128 * 64)
        a = [max(6, round(n ** (1 / 3) * rng.uniform(0.8, 1.25))) for _ in range(2)]
        dims, block, geom = (a[0], a[1], max(6, int(n / a[0] / a[1]))), (0, 0, 0), "hex"
    else:
        block = rng.choice([(8, 8, 8), (8, 8, 8), (6, 5, 4), (10, 6, 4), (7, 8, 8), (10, 9, 5)])
        cells = block[0] * block[1] * block[2]
        parts = max(8.0, min(n / cells, 4096.0))
        cx = max(2, round(parts ** (1 / 3) * rng.uniform(0.7, 1.3)))
        cy = max(2, round(math.sqrt(parts / cx) * rng.uniform(0.8, 1.2)))
        cz = max(2, int(min(parts, most / cells) / cx / cy))
        cz += cz % 2 if op == "smooth" and cz < 3 else -(cz % 2) if op == "smooth" else 0
        dims = (cx * block[0], cy * block[1], cz * block[2])
    return _case(None, op, dims, block, field, sigma, ell, geom, nrhs, prec, tol)


# ---------------------------------------------------------------------------
# inputs


class _Csr:
    """Host CSR matrix, both triangles, columns ascending (what the set-up takes)."""

    def __init__(self, n, row_ptr, col, val):
        self.n, self.row_ptr, self.col, self.val = n, row_ptr, col, val


class _Faces:
    pass


def _gen(seed, k):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * int(seed) + k)
    return g


def _grf(shape, ell, sigma, gen):
    """Gaussian random field with covariance exp(-r^2 / 2 ell^2): white noise
    on a padded grid, smoothed along each axis, standardised."""
    pad = [int(math.ceil(3 * e)) for e in ell]
    g = torch.randn([s + 2 * p for s, p in zip(shape, pad)], generator=gen, device=DEV,
                    dtype=torch.float64)
    for ax in range(3):
        if shape[ax] == 1:
            g = g.narrow(ax, 0, 1)
            continue
        i = torch.arange(shape[ax] + 2 * pad[ax], device=DEV, dtype=torch.float64)
        j = torch.arange(shape[ax], device=DEV, dtype=torch.float64) + pad[ax]
        w = torch.exp(-((i[:, None] - j[None, :]) / ell[ax]) ** 2)
        g = torch.matmul(g.transpose(ax, 2), w).transpose(ax, 2)
    g = g - g.mean()
    return (g / g.std() * sigma).contiguous()


def _log_k(c, seed):
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    gen = _gen(seed, 1)
    if c["field"] == "cross":
        band = [((torch.arange(m, device=DEV) % 8 >= 3) & (torch.arange(m, device=DEV) % 8 <= 4)).int()
                for m in (nz, ny, nx)]
        cnt = band[0][:, None, None] + band[1][None, :, None] + band[2][None, None, :]
        lk = torch.where(cnt >= 2, math.log(1e6), 0.0).to(torch.float64)
        return lk + 0.1 * torch.randn(lk.shape, generator=gen, device=DEV, dtype=torch.float64)
    if c["field"] == "layered":
        g = _grf((nz, ny, nx), (c["ell"] / 8, c["ell"], c["ell"]), c["sigma"], gen)
        u = torch.rand(nz, generator=gen, device=DEV, dtype=torch.float64) * 6 - 3
        return torch.clamp(u[:, None, None] + g / math.log(10.0), -3, 3) * math.log(10.0)
    return _grf((nz, ny, nx), (c["ell"],) * 3, c["sigma"], gen)


def _factors(c, seed):
    """Geometric factors (low cell, high cell) of the interior faces along x,
    y and z, and those of the boundary faces at x = 0 and x = nx."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    if c["geom"] == "cart":
        return [(2.0, 2.0)] * 3, (2.0, 2.0)
    ax = [torch.arange(m + 1, device=DEV, dtype=torch.float64) for m in (nz, ny, nx)]
    z, y, x = torch.meshgrid(*ax, indexing="ij")
    v = torch.stack([x, y, z], dim=-1)
    v = v + (torch.rand(v.shape, generator=_gen(seed, 2), device=DEV, dtype=torch.float64) * 0.6 - 0.3)
    lo, hi, al = slice(None, -1), slice(1, None), slice(None)
    cc = sum(v[a, b, d] for a in (lo, hi) for b in (lo, hi) for d in (lo, hi)) / 8

    def quad(a, b, d, e):
        return (a + b + d + e) / 4, 0.5 * torch.linalg.cross(d - a, e - b)

    fx = quad(v[lo, lo, al], v[lo, hi, al], v[hi, hi, al], v[hi, lo, al])
    fy = quad(v[lo, al, lo], v[hi, al, lo], v[hi, al, hi], v[lo, al, hi])
    fz = quad(v[al, lo, lo], v[al, lo, hi], v[al, hi, hi], v[al, hi, lo])

    def factor(centre, f, sign, cut):
        d = f[0][cut] - centre
        return sign * (d * f[1][cut]).sum(-1) / (d * d).sum(-1)

    s3 = [(al, al, slice(1, -1)), (al, slice(1, -1), al), (slice(1, -1), al, al)]
    c_lo = [cc[:, :, :-1], cc[:, :-1], cc[:-1]]
    c_hi = [cc[:, :, 1:], cc[:, 1:], cc[1:]]
    inner = [(factor(c_lo[k], f, 1.0, s3[k]), factor(c_hi[k], f, -1.0, s3[k]))
             for k, f in enumerate((fx, fy, fz))]
    return inner, (factor(cc[:, :, 0], fx, -1.0, (al, al, 0)), factor(cc[:, :, -1], fx, 1.0, (al, al, -1)))


class _System:
    """TPFA system as a seven-point stencil: face transmissibilities t[axis],
    Dirichlet diagonal and right-hand side, all [z, y, x] float64 tensors."""

    def __init__(self, c, log_k, geometry):
        k = torch.exp(log_k)
        inner, edge = geometry
        low = [k[:, :, :-1], k[:, :-1], k[:-1]]
        high = [k[:, :, 1:], k[:, 1:], k[1:]]
        self.t = []
        for a in range(3):
            tl, th = low[a] * inner[a][0], high[a] * inner[a][1]
            self.t.append(tl * th / (tl + th))
        self.d = torch.zeros_like(k)
        self.f = torch.zeros_like(k)
        if c["field"] == "cross":  # p = 0 on y = 0, p = 1 on y = ny
            self.d[:, 0] += 2.0 * k[:, 0]
            self.d[:, -1] += 2.0 * k[:, -1]
            self.f[:, -1] += 2.0 * k[:, -1]
        elif c["field"] == "layered" or c["op"] == "gradient":  # p = 1 on x = 0, 0 on x = nx
            self.d[:, :, 0] += edge[0] * k[:, :, 0]
            self.f[:, :, 0] += edge[0] * k[:, :, 0]
            self.d[:, :, -1] += edge[1] * k[:, :, -1]
        else:  # p = 0 on x = 0, wells in the right-hand side
            self.d[:, :, 0] += edge[0] * k[:, :, 0]
        self.diag = self.d.clone()
        for a in range(3):
            lo, hi = self.cuts(a)
            self.diag[lo] += self.t[a]
            self.diag[hi] += self.t[a]

    @staticmethod
    def cuts(a):
        al = slice(None)
        lo, hi = [al] * 3, [al] * 3
        lo[2 - a], hi[2 - a] = slice(None, -1), slice(1, None)
        return tuple(lo), tuple(hi)

    def mul(self, x):
        """A x for x of shape [..., z, y, x]."""
        y = self.diag * x
        for a in range(3):
            lo, hi = (((Ellipsis,) + s) for s in self.cuts(a))
            y[lo] -= self.t[a] * x[hi]
            y[hi] -= self.t[a] * x[lo]
        return y

    def csr(self):
        nz, ny, nx = self.diag.shape
        n = nx * ny * nz
        val = torch.zeros(nz, ny, nx, 7, dtype=torch.float64, device=DEV)
        for a in range(3):
            lo, hi = self.cuts(a)
            val[hi + (2 - a,)] = -self.t[a]
            val[lo + (4 + a,)] = -self.t[a]
        val[..., 3] = self.diag
        off = torch.tensor([-nx * ny, -nx, -1, 0, 1, nx, nx * ny], device=DEV)
        col = torch.arange(n, device=DEV)[:, None] + off
        val = val.reshape(n, 7)
        keep = val != 0
        rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        rp[1:] = torch.cumsum(keep.sum(1), 0)
        return _Csr(n, rp.cpu().numpy(), col[keep].to(torch.int32).cpu().numpy(), val[keep].cpu().numpy())


_parts = {}  # bisection partitions depend on the grid alone: a program keeps its grid's


def _partition(c, A):
    if c["bx"]:
        return am.partition_blocks((c["nx"], c["ny"], c["nz"]), (c["bx"], c["by"], c["bz"]))
    key = (c["nx"], c["ny"], c["nz"])
    if key not in _parts:
        _parts[key] = am.partition_bisect(A, 200, 800, 3)
    return _parts[key]


def _rhs(c, S, seed):
    """[nrhs, n]: the boundary's right-hand side or well pairs for a solve, a
    residual-like random vector for an application."""
    n = c["nx"] * c["ny"] * c["nz"]
    gen = _gen(seed, 3)
    if c["op"] == "apply":
        return torch.randn(c["nrhs"], n, generator=gen, device=DEV, dtype=torch.float64)
    b = S.f.reshape(1, n).repeat(c["nrhs"], 1)
    if c["field"] == "grf" and c["op"] != "gradient":
        wells = torch.randperm(n, generator=gen, device=DEV)[:2 * c["nrhs"]].reshape(2, c["nrhs"])
        row = torch.arange(c["nrhs"], device=DEV)
        b[row, wells[0]] += 1.0
        b[row, wells[1]] -= 1.0
    elif c["nrhs"] > 1:  # several boundary states of one model
        b = b * (1.0 + torch.arange(c["nrhs"], device=DEV, dtype=torch.float64))[:, None]
        b = b + 1e-3 * b.abs().max() * torch.randn(b.shape, generator=gen, device=DEV, dtype=torch.float64)
    return b


def _observed(c, seed):
    """1000 observed cells and pressures: the mean gradient with local noise."""
    n = c["nx"] * c["ny"] * c["nz"]
    gen = _gen(seed, 4)
    cells = torch.randperm(n, generator=gen, device=DEV)[:1000].sort().values
    x = (cells % c["nx"]).double()
    return cells, 1.0 - (x + 0.5) / c["nx"] + 0.05 * torch.randn(cells.numel(), generator=gen, device=DEV,
                                                                dtype=torch.float64)


def _face_list(c):
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    ids = np.arange(nx * ny * nz, dtype=np.int64).reshape(nz, ny, nx)
    west, east = ids[:, :, 0].ravel(), ids[:, :, -1].ravel()
    F = _Faces()
    F.k = np.concatenate([ids[:, :, :-1].ravel(), ids[:, :-1].ravel(), ids[:-1].ravel(), west, east])
    lo = np.concatenate([ids[:, :, 1:].ravel(), ids[:, 1:].ravel(), ids[1:].ravel()])
    bnd = west.size + east.size
    F.l = np.concatenate([lo, np.full(bnd, -1, np.int64)])
    F.gk = np.full(F.k.size, 2.0)
    F.gl = np.concatenate([np.full(lo.size, 2.0), np.zeros(bnd)])
    F.pD = np.concatenate([np.zeros(lo.size), np.ones(west.size), np.zeros(east.size)])
    return F


class _State:
    def __init__(self, case):
        self.case, self.handle, self.model = case, None, None

    def __del__(self):
        for held in (self.handle, self.model):
            if held is not None:
                held.close()


def prepare(case, seed):
    s = _State(case)
    log_k = _log_k(case, seed)
    if case["op"] == "gradient":
        dims = (case["nx"], case["ny"], case["nz"])
        part, m = am.partition_blocks(dims, (case["bx"], case["by"], case["bz"]))
        s.model = am.DarcyModel(_face_list(case), log_k.numel(), part, m, tol=case["tol"],
                                adjoint_tol=1e-12, reuse_handle=True)
        s.log_k = log_k.reshape(-1)
        s.cells, s.seen = _observed(case, seed)
        s.model.forward_solve(0.9 * s.log_k)  # the estimate before this one: the handle exists
        return s
    S = _System(case, log_k, _factors(case, seed))
    s.A = S.csr()
    s.part, s.nparts = _partition(case, s.A)
    b = _rhs(case, S, seed)
    s.b = b[0].contiguous() if case["nrhs"] == 1 else b.contiguous()
    if case["op"] != "setup":
        s.handle = am.AlgMortar(s.A, s.part, s.nparts, prec=case["prec"], max_nrhs=case["nrhs"])
    if case["op"] == "smooth":
        blocks, nblocks = am.partition_blocks((case["nx"], case["ny"], case["nz"]),
                                              (case["bx"], case["by"], 2 * case["bz"]))
        s.handle.set_smoother(blocks, nblocks, 1)
    return s


def run(s):
    op = s.case["op"]
    if op == "apply":
        return s.handle.apply(s.b)
    if op == "setup":
        h = am.AlgMortar(s.A, s.part, s.nparts)
        x, _, _ = h.pcg(s.b, s.case["tol"])
        h.close()
        return x
    if op == "gradient":
        theta = s.log_k.detach().requires_grad_(True)
        p = am.AlgMortarSolve.apply(theta, s.model)
        misfit = 0.5 * ((p[s.cells] - s.seen) ** 2).sum()
        misfit.backward()
        return {"p": p.detach(), "grad": theta.grad, "misfit": misfit.detach()}
    x, _, _ = s.handle.pcg(s.b, s.case["tol"])
    return x


def work(case):
    """Per application: the vectors, the matrix once, about 20 factor values
    per cell (what a fill-reducing order leaves of a 512-cell box).  Solves:
    that times the usual iteration count of the field; a gradient is two
    solves, a smoothed iteration three times the local solves."""
    n, nr = case["nx"] * case["ny"] * case["nz"], case["nrhs"]
    size = {"fp64": 8, "fp32": 4, "bf16": 2}[case["prec"]]
    local_b, local_f = 20.0 * n * size, 80.0 * n * nr
    if case["op"] == "apply":
        return {"bytes": local_b + 16.0 * n * nr, "flops": local_f}
    its = {"grf": 30.0, "cross": 8.0, "layered": 100.0}[case["field"]]
    rep = {"gradient": 2.0, "smooth": 0.5}.get(case["op"], 1.0)
    loc = 3.0 if case["op"] == "smooth" else 1.0
    return {"bytes": rep * its * (loc * local_b + 84.0 * n + 80.0 * n * nr),
            "flops": rep * its * (loc * local_f + 24.0 * n * nr)}


# ---------------------------------------------------------------------------
# the same results in plain 64-bit torch


def _cg(S, b):
    """A x = b by Jacobi-preconditioned CG with restarts on the true residual."""
    x = torch.zeros_like(b)

    def dot(u, v):
        return (u * v).sum((-3, -2, -1), keepdim=True)

    norm = dot(b, b)
    for _ in range(4):
        r = b - S.mul(x)
        z = r / S.diag
        p, rz, stop = z, dot(r, z), dot(r, r) * 1e-22 + norm * 1e-32
        for it in range(1, 20000):
            q = S.mul(p)
            pq = dot(p, q)
            a = torch.where(pq > 0, rz / pq, torch.zeros_like(pq))
            x = x + a * p
            r = r - a * q
            z = r / S.diag
            new = dot(r, z)
            p = z + torch.where(rz > 0, new / rz, torch.zeros_like(rz)) * p
            rz = new
            if it % 25 == 0 and bool((dot(r, r) <= stop).all()):
                break
    return x


def _exact_apply(case, A, part, nparts, r):
    """Algorithm 2 with dense local operators and a dense interface matrix."""
    n, f64 = A.n, torch.float64
    rp = torch.as_tensor(A.row_ptr, device=DEV)
    col = torch.as_tensor(A.col, device=DEV).long()
    val = torch.as_tensor(A.val, device=DEV)
    row = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
    part = torch.as_tensor(part, device=DEV).long()
    size = torch.bincount(part, minlength=nparts)
    top = int(size.max())
    order = torch.argsort(part, stable=True)
    start = torch.cumsum(size, 0) - size
    loc = torch.empty(n, dtype=torch.int64, device=DEV)
    loc[order] = torch.arange(n, device=DEV) - start[part[order]]
    cross = part[row] != part[col]
    # interfaces: one basis function per pair of touching subdomains
    lo, hi = torch.minimum(part[row], part[col])[cross], torch.maximum(part[row], part[col])[cross]
    pairs, which = torch.unique(lo * nparts + hi, return_inverse=True)
    nl = pairs.numel()
    near = torch.unique(part[row][cross] * nl + which)  # (subdomain, basis function)
    sub, fun = near // nl, near % nl
    count = torch.bincount(sub, minlength=nparts)
    slot = torch.arange(near.numel(), device=DEV) - (torch.cumsum(count, 0) - count)[sub]
    most = int(count.max())
    at = torch.searchsorted(near, part[row][cross] * nl + which)
    funs = torch.full((nparts, most), nl, dtype=torch.int64, device=DEV)
    funs[sub, slot] = fun
    z = torch.zeros(n, r.shape[0], dtype=f64, device=DEV)
    mat = torch.zeros(nl + 1, nl + 1, dtype=f64, device=DEV)
    mat.view(-1).index_add_(0, which * (nl + 2), -0.5 * val[cross])
    rhs = torch.zeros(nl + 1, r.shape[0], dtype=f64, device=DEV)
    kept, chunk = [], max(1, int(2e9 / 8 / top / top))
    for s0 in range(0, nparts, chunk):
        m = min(chunk, nparts - s0)
        here = (part[row] >= s0) & (part[row] < s0 + m)
        local = torch.zeros(m, top, top, dtype=f64, device=DEV)
        e = here & ~cross
        local[part[row[e]] - s0, loc[row[e]], loc[col[e]]] = val[e]
        diag = torch.diagonal(local, dim1=1, dim2=2)
        diag += (torch.arange(top, device=DEV)[None, :] >= size[s0:s0 + m, None]).to(f64)
        e = here & cross
        local.view(-1).index_add_(0, ((part[row[e]] - s0) * top + loc[row[e]]) * top + loc[row[e]], -val[e])
        g = torch.zeros(m, top, most, dtype=f64, device=DEV)  # half the couplings to each interface
        mine = here[cross]
        g.view(-1).index_add_(0, ((part[row[e]] - s0) * top + loc[row[e]]) * most + slot[at[mine]], -0.5 * val[e])
        cells = order[start[s0]:start[s0] + int(size[s0:s0 + m].sum())]
        v = torch.zeros(m, top, r.shape[0], dtype=f64, device=DEV)
        v[part[cells] - s0, loc[cells]] = r[:, cells].T
        both = torch.cholesky_solve(torch.cat([v, 4.0 * g], 2), torch.linalg.cholesky(local))
        pbar, phat = both[:, :, :r.shape[0]], both[:, :, r.shape[0]:]
        gt = g.transpose(1, 2).contiguous()
        ids = funs[s0:s0 + m]
        rhs.index_add_(0, ids.reshape(-1), torch.matmul(gt, pbar).reshape(-1, r.shape[0]))
        mat.view(-1).index_add_(0, (ids[:, :, None] * (nl + 1) + ids[:, None, :]).reshape(-1),
                                -torch.matmul(gt, phat).reshape(-1))
        kept.append((s0, m, cells, pbar, phat))
    sm = mat[:nl, :nl]
    sm = 0.5 * (sm + sm.T)
    eta = torch.zeros(nl + 1, r.shape[0], dtype=f64, device=DEV)
    eta[:nl] = torch.cholesky_solve(rhs[:nl], torch.linalg.cholesky(sm))
    for s0, m, cells, pbar, phat in kept:
        both = pbar + torch.matmul(phat, eta[funs[s0:s0 + m]])
        z[cells] = both[part[cells] - s0, loc[cells]]
    return z.T.contiguous()


def exact(case, seed):
    log_k = _log_k(case, seed)
    S = _System(case, log_k, _factors(case, seed))
    shape = S.diag.shape
    if case["op"] == "gradient":
        p = _cg(S, S.f)
        cells, seen = _observed(case, seed)
        off = p.reshape(-1)[cells] - seen
        src = torch.zeros(p.numel(), dtype=torch.float64, device=DEV)
        src[cells] = off
        lam = _cg(S, src.reshape(shape))
        k = torch.exp(log_k)
        grad = torch.zeros_like(p)
        for a in range(3):
            lo, hi = S.cuts(a)
            flux = S.t[a] * (lam[lo] - lam[hi]) * (p[lo] - p[hi])
            share = k[hi] / (k[lo] + k[hi])
            grad[lo] -= share * flux
            grad[hi] -= (1.0 - share) * flux
        grad[:, :, 0] -= 2.0 * k[:, :, 0] * lam[:, :, 0] * (p[:, :, 0] - 1.0)
        grad[:, :, -1] -= 2.0 * k[:, :, -1] * lam[:, :, -1] * p[:, :, -1]
        return {"p": p.reshape(-1), "grad": grad.reshape(-1), "misfit": 0.5 * (off * off).sum()}
    b = _rhs(case, S, seed)
    if case["op"] == "apply":
        A = S.csr()
        x = _exact_apply(case, A, *_partition(case, A), b)
    else:
        x = _cg(S, b.reshape((-1,) + tuple(shape))).reshape(b.shape)
    return x[0].contiguous() if case["nrhs"] == 1 else x
