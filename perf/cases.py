"""The work a program has this library do, as timed cases.

Every case goes through the Python entry points (`lapfoam.Mesh`, `Problem`, `Batch`, `Group`) the way a program
calls them: the initial field is set, the steps are taken and the field is read back on the device; or a gradient is
asked for; or a set of requests is run in the batched or in the grouped form.  Boxes, boundary conditions, diffusivities
and time steps are those of the repository's configurations (the 32^3, 256^3 and 192^3 boxes, the request stream), of
its benchmark (the skewed boxes' gradient and corrected step) and of the evaluation boxes of the paper (uniform cubes,
dt = 0.2 s).

Meshes are built here with torch, so that `exact` can form the same systems without the library: it assembles them
face by face in 64 bits and solves each step far below the tolerance of the timed solves.
"""
import math
from types import SimpleNamespace

import torch

from paper_2507_18268_amd import lapfoam as L

TOL = 1e-9
T_LO, T_HI = 273.0, 573.0                # fixed values at x = 0 and x = 1, and the range of the initial field
SKEW = ((1.0, 0.30, 0.10), (0.20, 1.0, 0.25), (-0.10, 0.15, 1.0))
PRECOND = {"diagonal": L.LF_PC_DIAGONAL, "dic": L.LF_PC_DIC, "amg": L.LF_PC_AMG}

# (DT, dt) of the configurations: the plain and the graded boxes, the randomly numbered box, the paper's boxes
PLAIN, GRADED, PERMUTED, PAPER = (1e-3, 5e-3), (1e-3, 1e-3), (5e-4, 1e-3), (1e-4, 0.2)


def _step(name, shape, physics, steps, z_ratio=1.0, numbering="natural", precond="diagonal", precision="fp64",
          skew=False):
    return dict(name=name, kind="step", nx=shape[0], ny=shape[1], nz=shape[2], z_ratio=z_ratio, numbering=numbering,
                skew=skew, precond=precond, precision=precision, DT=physics[0], dt=physics[1], steps=steps)


def _grad(name, shape, numbering):
    return dict(name=name, kind="grad", nx=shape[0], ny=shape[1], nz=shape[2], z_ratio=4.0, numbering=numbering,
                skew=True)


def _cube(n):
    return (n, n, n)


def listed():
    return [
        # the smallest configuration, 20 steps: what a step costs in launches and waits
        _step("plain_32", _cube(32), PLAIN, 20),
        # the smallest box of the paper's evaluation (10 of its 500 steps): one million cells, all in the caches
        _step("paper_100", _cube(100), PAPER, 10),
        # the flagship: the graded box of 16.8 M cells in FP64, bound by memory
        _step("graded_256", _cube(256), GRADED, 5, z_ratio=10.0),
        # the same box in the precision form (FP32 inner solves, FP64 residual and update)
        _step("mixed_256", _cube(256), GRADED, 5, z_ratio=10.0, precision="mixed"),
        # the same box numbered red cells first, with the DIC preconditioner
        _step("dic_256", _cube(256), GRADED, 5, z_ratio=10.0, numbering="red_black", precond="dic"),
        # a mesh without structure in its numbering (the row layout), as unstructured meshes come
        _step("permuted_160", _cube(160), PERMUTED, 5, z_ratio=10.0, numbering="random"),
        # the paper's second box with the multigrid preconditioner
        _step("paper_200_amg", _cube(200), PAPER, 5, precond="amg"),
        # skewed cells: gradient, non-orthogonal correction, assembly and solve in every step
        _step("skewed_128", _cube(128), GRADED, 5, z_ratio=10.0, skew=True),
        # one Gauss gradient of a field on a skewed box, structured and random numbering
        _grad("grad_skewed_192", _cube(192), "natural"),
        _grad("grad_permuted_128", _cube(128), "random"),
        # the small requests of a serving stream: one workgroup per problem, 10 steps each, snapshots kept
        dict(name="batch_64", kind="batch", count=64, lo=16, hi=32, steps=10, threads=512),
        # the whole range of the stream's requests in one group: 24 problems of sides 16 to 96, 10 steps each
        dict(name="group_24", kind="group", count=24, lo=16, hi=96, steps=10),
    ]


def _shape(rng, lo, hi, most):
    """A box near a cube whose side is log-uniform in [lo, hi]; the sides differ and are odd as often as not."""
    side = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    n = [max(4, round(side * rng.uniform(0.85, 1.18))) for _ in range(3)]
    while n[0] * n[1] * n[2] > most:
        n = [k - 1 for k in n]
    return tuple(n)


def draw(rng):
    kind = rng.choice(["fp64", "fp64", "paper", "mixed", "dic", "permuted", "amg", "skewed", "grad", "grad_permuted",
                       "batch", "group"])
    z = rng.choice([1.0, 10.0])
    if kind == "fp64":
        s = _shape(rng, 20, 256, 256 ** 3)
        c = _step("", s, rng.choice([PLAIN, GRADED]), rng.randint(4, 6) if s[0] > 80 else rng.randint(10, 20), z)
    elif kind == "paper":
        c = _step("", _shape(rng, 50, 200, 200 ** 3), PAPER, rng.randint(4, 8))
    elif kind == "mixed":
        c = _step("", _shape(rng, 16, 256, 256 ** 3), GRADED, rng.randint(3, 5), z, precision="mixed")
    elif kind == "dic":
        c = _step("", _shape(rng, 32, 224, 224 ** 3), GRADED, rng.randint(3, 5), z, numbering="red_black",
                  precond="dic")
    elif kind == "permuted":
        c = _step("", _shape(rng, 24, 160, 160 ** 3), PERMUTED, rng.randint(3, 5), z, numbering="random")
    elif kind == "amg":
        c = _step("", _shape(rng, 48, 200, 200 ** 3), PAPER, rng.randint(3, 5), precond="amg")
    elif kind == "skewed":
        c = _step("", _shape(rng, 32, 128, 128 ** 3), GRADED, rng.randint(3, 5), z, skew=True)
    elif kind == "grad":
        c = _grad("", _shape(rng, 32, 192, 192 ** 3), "natural")
    elif kind == "grad_permuted":
        c = _grad("", _shape(rng, 32, 128, 128 ** 3), "random")
    elif kind == "batch":
        c = dict(kind="batch", count=rng.randint(16, 96), lo=16, hi=rng.randint(24, 36), steps=rng.randint(5, 10),
                 threads=rng.choice([512, 1024]))
    else:
        c = dict(kind="group", count=rng.randint(4, 24), lo=rng.randint(16, 32), hi=rng.randint(48, 96),
                 steps=rng.randint(5, 10))
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------------------------------------------
# meshes
# ---------------------------------------------------------------------------------------------------------------
def _nodes(n, ratio):
    """Nodes of n cells on [0, 1], widths growing geometrically so that last / first = ratio."""
    if ratio == 1.0 or n == 1:
        x = torch.arange(n + 1, dtype=torch.float64) / n
    else:
        g = ratio ** (1.0 / (n - 1))
        x = torch.cat([torch.zeros(1, dtype=torch.float64), torch.cumsum(g ** torch.arange(n, dtype=torch.float64), 0)])
        x = x / x[-1]
    return x.cuda()


def _mesh(case):
    """A box in face addressing as device tensors: internal faces sorted by (owner, neighbour), six boundary patches
    (xmin, xmax, ymin, ymax, zmin, zmax); `old` is each label's cell in the natural numbering."""
    n = (case["nx"], case["ny"], case["nz"])
    x = [_nodes(n[0], 1.0), _nodes(n[1], 1.0), _nodes(n[2], case["z_ratio"])]
    h = [v[1:] - v[:-1] for v in x]
    mid = [0.5 * (v[1:] + v[:-1]) for v in x]
    N = n[0] * n[1] * n[2]
    lab = torch.arange(N, device="cuda")
    ijk = [lab % n[0], lab // n[0] % n[1], lab // (n[0] * n[1])]
    C = torch.stack([mid[a][ijk[a]] for a in range(3)], 1)
    w = torch.stack([h[a][ijk[a]] for a in range(3)], 1)
    V = w.prod(1)
    inner = torch.stack([ijk[a] < n[a] - 1 for a in range(3)], 1).reshape(-1)
    f = torch.nonzero(inner).reshape(-1)
    own, ax = f // 3, f % 3
    del f, inner
    nei = own + torch.tensor([1, n[0], n[0] * n[1]], device="cuda")[ax]
    Sf = torch.zeros((own.numel(), 3), dtype=torch.float64, device="cuda")
    Sf.scatter_(1, ax[:, None], (V[own] / w[own].gather(1, ax[:, None]).reshape(-1))[:, None])
    Cf = C[own]
    Cf.scatter_add_(1, ax[:, None], 0.5 * w[own].gather(1, ax[:, None]))
    bcell, bS, bC, start = [], [], [], [0]
    for p in range(6):
        a, hi = p // 2, p % 2
        cells = lab[ijk[a] == (n[a] - 1 if hi else 0)]
        S, c = torch.zeros((cells.numel(), 3), dtype=torch.float64, device="cuda"), C[cells].clone()
        S[:, a] = (1.0 if hi else -1.0) * V[cells] / w[cells, a]
        c[:, a] = 1.0 if hi else 0.0
        bcell.append(cells)
        bS.append(S)
        bC.append(c)
        start.append(start[-1] + cells.numel())
    bcell, bS, bC = torch.cat(bcell), torch.cat(bS), torch.cat(bC)
    old = None
    if case["numbering"] != "natural":
        if case["numbering"] == "random":
            g = torch.Generator(device="cuda")
            g.manual_seed(1)
            old = torch.randperm(N, generator=g, device="cuda")
        else:
            par = (ijk[0] + ijk[1] + ijk[2]) % 2
            old = torch.cat([lab[par == 0], lab[par == 1]])
        new = torch.empty_like(old)
        new[old] = lab
        a, b = new[own], new[nei]
        swap = a > b
        own, nei = torch.minimum(a, b), torch.maximum(a, b)
        Sf = torch.where(swap[:, None], -Sf, Sf)
        order = torch.sort(own * N + nei)[1]
        own, nei, Sf, Cf = own[order], nei[order], Sf[order], Cf[order]
        V, C, bcell = V[old], C[old], new[bcell]
    if case["skew"]:
        A = torch.tensor(SKEW, dtype=torch.float64, device="cuda")
        det = torch.linalg.det(A)
        cof = det * torch.linalg.inv(A)
        V, C, Cf, bC, Sf, bS = det * V, C @ A.T, Cf @ A.T, bC @ A.T, Sf @ cof, bS @ cof
    return SimpleNamespace(N=N, own=own, nei=nei, V=V, C=C, Sf=Sf, Cf=Cf, start=start, bcell=bcell, bS=bS, bC=bC,
                           old=old)


def _device_mesh(m, gradient, skew):
    """The library's mesh of these arrays, which cross its interface on the host."""
    i32 = lambda t: t.to(torch.int32).cpu().numpy()          # noqa: E731
    f64 = lambda t: t.cpu().numpy()                          # noqa: E731
    h = SimpleNamespace(n_cells=m.N, n_faces=int(m.own.numel()), owner=i32(m.own), neighbour=i32(m.nei),
                        cell_volume=f64(m.V), cell_centre=f64(m.C), face_area=f64(m.Sf),
                        face_centre=f64(m.Cf) if gradient else None, patch_start=i32(torch.tensor(m.start)),
                        bface_cell=i32(m.bcell), bface_area=f64(m.bS), bface_centre=f64(m.bC))
    return L.Mesh(h, gradient=gradient, non_orthogonal=skew)


def _field(n, seed, salt, lo, hi):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1009 + salt)
    return lo + (hi - lo) * torch.rand(n, generator=g, device="cuda", dtype=torch.float64)


def _initial(m, seed, salt=0):
    """Uniform in [273, 573), drawn in the natural numbering."""
    t = _field(m.N, seed, salt, T_LO, T_HI)
    return t if m.old is None else t[m.old]


BCS = [(L.LF_BC_FIXED_VALUE, T_LO), (L.LF_BC_FIXED_VALUE, T_HI)] + [(L.LF_BC_ZERO_GRADIENT, 0.0)] * 4


def _requests(case):
    """The cubes of a batch or group: sides log-spaced in [lo, hi], diffusivities log-spaced in [1e-4, 1e-2]."""
    out = []
    for i in range(case["count"]):
        u, v = (i + 0.5) / case["count"], ((7 * i + 3) % case["count"] + 0.5) / case["count"]
        side = round(case["lo"] * (case["hi"] / case["lo"]) ** u)
        out.append(dict(nx=side, ny=side, nz=side, z_ratio=1.0, numbering="natural", skew=False, DT=1e-4 * 100.0 ** v,
                        dt=1e-3))
    return out


# ---------------------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    s = SimpleNamespace(case=case)
    if case["kind"] == "step":
        m = _mesh(case)
        s.T0 = _initial(m, seed)
        s.mesh = _device_mesh(m, case["skew"], case["skew"])
        del m
        torch.cuda.empty_cache()
        opts = L.make_opts(tol=TOL, precond=PRECOND[case["precond"]],
                           precision=L.LF_PREC_MIXED if case["precision"] == "mixed" else L.LF_PREC_FP64)
        s.problem = L.Problem(s.mesh, BCS, case["DT"], case["dt"], opts)
        s.T = torch.empty_like(s.T0)
    elif case["kind"] == "grad":
        m = _mesh(case)
        s.T = _initial(m, seed)
        s.Tb, s.snb = _boundary(m, seed)
        s.mesh = _device_mesh(m, True, True)
    else:
        opts = L.make_opts(tol=TOL, precision=L.LF_PREC_MIXED)
        meshes, s.problems, s.T0, s.snaps, at = {}, [], [], [], 0
        requests = _requests(case)
        # every request's snapshots one after another in one buffer
        s.out = torch.empty(case["steps"] * sum(q["nx"] ** 3 for q in requests), dtype=torch.float64, device="cuda")
        for i, q in enumerate(requests):
            m = _mesh(q)
            if q["nx"] not in meshes:
                meshes[q["nx"]] = _device_mesh(m, False, False)
            s.T0.append(_initial(m, seed, i))
            s.problems.append(L.Problem(meshes[q["nx"]], BCS, q["DT"], q["dt"], opts))
            s.snaps.append(s.out[at:at + case["steps"] * m.N])
            at += case["steps"] * m.N
        s.engine = (L.Batch(case["count"], case["steps"]) if case["kind"] == "batch" else L.Group(case["count"]))
    return s


def _boundary(m, seed):
    """Boundary values and normal gradients of the gradient's field."""
    B = m.bcell.numel()
    return _field(B, seed, 1, T_LO, T_HI), _field(B, seed, 2, -200.0, 200.0)


def run(state):
    case = state.case
    if case["kind"] == "step":
        state.problem.set_T(state.T0)
        state.problem.step(case["steps"])
        return state.problem.get_T(state.T)
    if case["kind"] == "grad":
        return state.mesh.grad(state.T, state.Tb, state.snb)
    if case["kind"] == "batch":
        for P, T0 in zip(state.problems, state.T0):
            P.set_T(T0)
        state.engine.launch(state.problems, case["steps"], block_threads=case["threads"], snapshots=state.snaps)
        state.engine.wait()
    else:
        for P, T0, snap in zip(state.problems, state.T0, state.snaps):
            state.engine.add(P, case["steps"], snap, T0=T0)
        left = case["count"]
        while left:
            left -= len(state.engine.poll())
    return state.out


# ---------------------------------------------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------------------------------------------
def _iterations(c):
    """About the iterations a diagonally preconditioned CG needs to fall by 1e-9 (from the condition number of the
    scaled matrix 1 + 4 DT dt sum 1/h^2), so that a solve's passes can be counted."""
    zr, nz = c["z_ratio"], c["nz"]
    hz = 1.0 / nz if zr == 1.0 or nz == 1 else (zr ** (1.0 / (nz - 1)) - 1.0) / (zr ** (nz / (nz - 1.0)) - 1.0)
    kappa = 1.0 + 4.0 * c["DT"] * c["dt"] * (c["nx"] ** 2 + c["ny"] ** 2 + hz ** -2)
    return max(2.0, 0.65 * 0.5 * math.log(2e9) * math.sqrt(kappa))


def _step_work(c, word):
    """Per step: the face factors, V and T once, and per iteration the two passes of a CG (the product with its
    direction: r, p, x, the coefficients read, p, q, x written; the update: q, r read, r written)."""
    cells = c["nx"] * c["ny"] * c["nz"]
    its = _iterations(c)
    if c.get("precond") in ("dic", "amg"):
        its *= 0.5          # each iteration then applies the preconditioner: coefficients, r and w once more
    extra = 5 if c.get("precond") in ("dic", "amg") else 0
    return cells * (72.0 + its * word * (12 + extra)), cells * (60.0 + its * (30 + 5 * extra))


def work(case):
    if case["kind"] == "grad":
        cells = case["nx"] * case["ny"] * case["nz"]
        faces = 3.0 * cells
        index = 8.0 * faces if case["numbering"] != "natural" else 0.0
        return dict(bytes=cells * (8 + 8 + 24) + faces * 32 + index, flops=faces * 20)
    if case["kind"] == "step":
        b, f = _step_work(case, 4 if case["precision"] == "mixed" else 8)
        return dict(bytes=case["steps"] * b, flops=case["steps"] * f)
    b = f = 0.0
    for q in _requests(case):
        qb, qf = _step_work(q, 4)
        b, f = b + case["steps"] * (qb + 8 * q["nx"] ** 3), f + case["steps"] * qf
    return dict(bytes=b, flops=f)


# ---------------------------------------------------------------------------------------------------------------
# the same results in 64 bits, face by face
# ---------------------------------------------------------------------------------------------------------------
def _sum_faces(m, owned, lower):
    """Per cell: the sum of `owned` over the faces it owns plus the sum of `lower` over those it is neighbour of."""
    out = torch.zeros((m.N,) + tuple(owned.shape[1:]), dtype=torch.float64, device="cuda")
    out.index_add_(0, m.own, owned)
    out.index_add_(0, m.nei, lower)
    return out


def _gradient(m, T, Tb):
    """The Gauss gradient with linear interpolation."""
    a = (m.Sf * (m.Cf - m.C[m.own])).sum(1).abs()
    b = (m.Sf * (m.C[m.nei] - m.Cf)).sum(1).abs()
    w = b / (a + b)
    s = m.Sf * (w * (T[m.own] - T[m.nei]) + T[m.nei])[:, None]
    g = _sum_faces(m, s, -s)
    g.index_add_(0, m.bcell, m.bS * Tb[:, None])
    return g / m.V[:, None], w


def _exact_steps(m, case, T, steps, keep):
    DT, dt = case["DT"], case["dt"]
    d = m.C[m.nei] - m.C[m.own]
    mag = m.Sf.norm(dim=1)
    nd = (m.Sf * d).sum(1) / mag
    delta = 1.0 / torch.maximum(nd, 0.05 * d.norm(dim=1))
    k = m.Sf / mag[:, None] - delta[:, None] * d if case["skew"] else None
    del d, nd
    up = delta * DT * mag
    diag = m.V / dt + _sum_faces(m, up, up)
    nb = m.bS.norm(dim=1)
    fixed = slice(0, m.start[2])                                   # xmin and xmax
    vb = torch.full_like(nb[fixed], T_LO)
    vb[m.start[1]:] = T_HI
    gb = DT * nb[fixed] ** 2 / (m.bS[fixed] * (m.bC[fixed] - m.C[m.bcell[fixed]])).sum(1)
    diag.index_add_(0, m.bcell[fixed], gb)
    src = torch.zeros_like(diag).index_add_(0, m.bcell[fixed], gb * vb)

    def product(x):
        return diag * x - _sum_faces(m, up * x[m.nei], up * x[m.own])

    out = []
    for _ in range(steps):
        b = m.V / dt * T + src
        if k is not None:
            Tb = T[m.bcell]
            Tb[fixed] = vb
            g, w = _gradient(m, T, Tb)
            flux = DT * mag * (k * (w[:, None] * (g[m.own] - g[m.nei]) + g[m.nei])).sum(1)
            b = b + _sum_faces(m, flux, -flux)
        x = T.clone()
        r = b - product(x)
        z = r / diag
        p, rz, top = z.clone(), torch.dot(r, z), None
        for _ in range(400):
            q = product(p)
            alpha = rz / torch.dot(p, q)
            x += alpha * p
            r -= alpha * q
            z = r / diag
            new = torch.dot(r, z)
            p = z + (new / rz) * p
            rz = new
            top = new.item() if top is None else max(top, new.item())
            if new.item() <= 1e-30 * max(top, 1e-300) or new.item() <= 1e-32 * torch.dot(b, b / diag).item():
                break
        T = x
        if keep:
            out.append(T)
    return torch.cat(out) if keep else T


def exact(case, seed):
    if case["kind"] == "grad":
        m = _mesh(case)
        Tb, snb = _boundary(m, seed)
        g, _ = _gradient(m, _initial(m, seed), Tb)
        n = m.bS / m.bS.norm(dim=1)[:, None]
        gc = g[m.bcell]
        return g, gc + n * (snb - (n * gc).sum(1))[:, None]
    if case["kind"] == "step":
        m = _mesh(case)
        return _exact_steps(m, case, _initial(m, seed), case["steps"], False)
    out = []
    for i, q in enumerate(_requests(case)):
        m = _mesh(q)
        out.append(_exact_steps(m, q, _initial(m, seed, i), case["steps"], True))
    return torch.cat(out)
