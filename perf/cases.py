"""The work this solver is used for, as measurable cases.

Each case is one call through the public binding (``paper_1506_05996_amd.sem``) on a perturbed
box mesh of hexahedra: the operator (``Mesh.apply_A``), the two-scale preconditioner
(``Mesh.precond``), PCG to a true residual of 1e-10 in FP64 and in the FP32-refined form
(``Mesh.solve``), a backward Euler step of the heat equation (``Mesh.heat_step``) and a batched
solve (``Batch.solve``).  ``listed()`` names the sizes, ``draw(rng)`` gives others of the same
ranges, ``prepare`` builds the mesh handle and the input vectors from a seed, ``run`` is the call,
``work`` is what the call cannot do without and ``exact`` evaluates it in plain FP64 torch.
"""
import math

import numpy as np
import torch

from paper_1506_05996_amd import sem

DEV = "cuda:0"
RTOL = 1e-10
KAPPA, DT = 1e-2, 0.04  # the heat rod's diffusivity and time step


# --- cases -----------------------------------------------------------------------------------

def _case(name, op, k, order, dtype="f64", lz=1.0, perturb=0.1, permute=False, coef="none", mode="fp64", count=0):
    """kx, ky, kz: hexahedra per direction; lz: the box is 1 x 1 x lz; coef: constants kappa = 1,
    c = 0 ("none"), one kappa and c per element ("element") or per node ("node")."""
    c = dict(op=op, kx=k[0], ky=k[1], kz=k[2], order=order, dtype=dtype, lz=lz, perturb=perturb, permute=permute,
             coef=coef, mode=mode, count=count)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest problem of the tests and the benchmark (4,913 nodes): launches and latency
        _case("apply_4c_n4", "apply", (4, 4, 4), 4),
        # the headline workload: 56^3 hexahedra with shuffled ids at order 7, 60.7 M nodes
        _case("apply_56c_n7", "apply", (56, 56, 56), 7, perturb=0.15, permute=True),
        # odd extents at a middling order in FP32, as the refined form's inner iterations apply it
        _case("apply_37x41x43_n5_f32", "apply", (37, 41, 43), 5, dtype="f32", permute=True),
        # the high-order end: hexahedra stretched 8:1 at order 15
        _case("apply_16c_n15", "apply", (16, 16, 16), 15, lz=8.0),
        # low order with one kappa and one c per element (a layered medium with reaction)
        _case("apply_33c_n3_element", "apply", (33, 33, 33), 3, coef="element"),
        # the preconditioner alone, FP64, at the headline's order
        _case("precond_40c_n7", "precond", (40, 40, 40), 7, perturb=0.15, permute=True),
        # and in FP32 on a small ragged mesh
        _case("precond_23x29x31_n4_f32", "precond", (23, 29, 31), 4, dtype="f32"),
        # a whole solve at the smallest size: a serving loop of small problems
        _case("solve_4c_n4", "solve", (4, 4, 4), 4),
        # a whole FP64 solve, 4.8 M nodes
        _case("solve_24c_n7", "solve", (24, 24, 24), 7, perturb=0.15, permute=True),
        # a whole FP32-refined solve, 22 M nodes
        _case("solve_refined_40c_n7", "solve", (40, 40, 40), 7, perturb=0.15, permute=True, mode="refined"),
        # one time step of the heat equation on a bar, started from the step before
        _case("heat_10x10x125_n7", "heat", (10, 10, 125), 7, lz=12.5, permute=True),
        # 16 independent problems of orders 3..8 and 2..20 hexahedra per side, solved together
        _case("batch16_n3to8", "batch", (2, 20, 0), 3, count=16),
    ]


def draw(rng):
    op = rng.choice(["apply"] * 4 + ["precond"] * 3 + ["solve"] * 3 + ["heat", "batch"])
    if op == "batch":
        return _case("", "batch", (2, rng.randint(8, 18), 0), 3, count=rng.randint(3, 16),
                     mode=rng.choice(["fp64", "fp64", "refined"]))
    order = rng.randint(2, 15) if op in ("apply", "precond") else rng.randint(2, 10)
    most = 2.5e7 if op in ("apply", "precond") else 6e6
    local = math.exp(rng.uniform(math.log(2e4), math.log(most)))
    e = max(8.0, local / (order + 1) ** 3)
    k = [max(2, round(e ** (1 / 3) * math.exp(rng.uniform(-0.25, 0.25)))) for _ in range(2)]
    k.append(max(2, round(e / (k[0] * k[1]))))
    solve = op in ("solve", "heat")
    return _case("", op, tuple(k), order, dtype="f64" if solve else rng.choice(["f64", "f64", "f32"]),
                 lz=round(k[2] / k[0] * rng.uniform(0.7, 1.5), 3), perturb=rng.choice([0.0, 0.1, 0.15]),
                 permute=rng.random() < 0.5,
                 coef="none" if solve else rng.choice(["none", "none", "none", "element", "node"]),
                 mode=rng.choice(["fp64", "refined"]) if solve else "fp64")


# --- inputs ----------------------------------------------------------------------------------

def _box(kx, ky, kz, lz, perturb, permute, rng):
    """Vertices [V, 3] and hexahedra [E, 8] of the box 1 x 1 x lz (vertex ids and corners x fastest),
    interior vertices moved by up to perturb h, and the lattice position [E, 3] of each element."""
    n = (kx + 1, ky + 1, kz + 1)
    h = np.array([1.0 / kx, 1.0 / ky, lz / kz])
    c, b, a = (g.ravel() for g in np.meshgrid(*(np.arange(v) for v in n[::-1]), indexing="ij"))
    vtx = np.stack([a, b, c], axis=1) * h
    inner = (a > 0) & (a < kx) & (b > 0) & (b < ky) & (c > 0) & (c < kz)
    vtx[inner] += rng.uniform(-perturb, perturb, (int(inner.sum()), 3)) * h
    ez, ey, ex = (g.ravel() for g in np.meshgrid(np.arange(kz), np.arange(ky), np.arange(kx), indexing="ij"))
    pos = np.stack([ex, ey, ez], axis=1)
    if permute:
        pos = pos[rng.permutation(len(pos))]
    corner = np.array([[p & 1, p >> 1 & 1, p >> 2] for p in range(8)])
    at = pos[:, None, :] + corner[None]
    return vtx, at[..., 0] + n[0] * (at[..., 1] + n[1] * at[..., 2]), pos


def _meshes(case, seed):
    """(vtx, hex, pos, order, (kx, ky, kz)) of the case's mesh, or of each of its instances."""
    rng = np.random.default_rng([1506, seed])
    if case["op"] != "batch":
        k = case["kx"], case["ky"], case["kz"]
        return [(*_box(*k, case["lz"], case["perturb"], case["permute"], rng), case["order"], k)], rng
    # the sizes belong to the case, the perturbations and right-hand sides to the seed
    size, out = np.random.default_rng(1506 + case["count"]), []
    for _ in range(case["count"]):
        order, k = int(size.integers(3, 9)), int(size.integers(case["kx"], case["ky"] + 1))
        out.append((*_box(k, k, k, 1.0, 0.1, False, rng), order, (k, k, k)))
    return out, rng


def _coefficients(case, n_elem, order, rng):
    """kappa and c of the case (None: 1 and 0): kappa log-uniform over a decade, c over (0, 10)."""
    shape = {"none": None, "element": (n_elem,), "node": (n_elem, (order + 1) ** 3)}[case["coef"]]
    if shape is None:
        return None, None
    return 10.0 ** rng.uniform(-0.5, 0.5, shape), rng.uniform(0.0, 10.0, shape)


def _noise(n, seed, dtype=torch.float64):
    g = torch.Generator(device=DEV).manual_seed(seed * 7919 + 11)
    return (torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * 2 - 1).to(dtype)


def _modes(xyz, lz, seed):
    """A smooth source: eight products of sines with random wave numbers 1..4 and amplitudes."""
    rng = np.random.default_rng([6005, seed])
    s = torch.zeros(xyz.shape[0], dtype=torch.float64, device=DEV)
    for w, amp in zip(rng.integers(1, 5, (8, 3)) * math.pi, rng.normal(size=8)):
        s += amp * (torch.sin(w[0] * xyz[:, 0]) * torch.sin(w[1] * xyz[:, 1]) * torch.sin(w[2] / lz * xyz[:, 2]))
    return s


def _rod(xyz, lz, seed):
    """A bar warmed by a spot that has come to a random place: the temperature and the source."""
    z = lz * (0.2 + 0.6 * np.random.default_rng([61, seed]).uniform())
    d2 = (xyz[:, 0] - 0.5) ** 2 + (xyz[:, 1] - 0.5) ** 2
    inside = torch.sin(math.pi * xyz[:, 0]) * torch.sin(math.pi * xyz[:, 1]) * torch.sin(math.pi / lz * xyz[:, 2])
    spot = lambda at: torch.exp(-(d2 + (xyz[:, 2] - at) ** 2) / 0.08)  # noqa: E731
    return 0.05 * inside * (spot(z - 0.3) + spot(z)), 0.18 * spot(z)


def prepare(case, seed):
    meshes, rng = _meshes(case, seed)
    if case["op"] == "batch":
        batch = sem.Batch([(v, h, n) for v, h, _, n, _ in meshes])
        b = [_noise(n, seed * 64 + i) for i, n in enumerate(batch.n_global)]
        return dict(case=case, batch=batch, b=b, x=[torch.zeros_like(v) for v in b])
    vtx, hexes, _, order, _ = meshes[0]
    mesh = sem.Mesh(vtx, hexes, order)
    kappa, c = _coefficients(case, mesh.n_elem, order, rng)
    if case["coef"] == "element":
        mesh.set_element_coefficients(kappa, c)
    elif case["coef"] == "node":
        mesh.set_node_coefficients(kappa, c)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.float64
    state = dict(case=case, mesh=mesh)
    if case["op"] == "apply":
        state["u"] = _noise(mesh.n_global, seed, dtype)
        state["y"] = torch.empty_like(state["u"])
    elif case["op"] == "precond":  # a residual: zero on the Dirichlet set
        free = torch.from_numpy(mesh.boundary_mask() == 0).to(DEV)
        state["u"] = _noise(mesh.n_global, seed, dtype) * free
        state["y"] = torch.empty_like(state["u"])
    else:
        xyz = torch.from_numpy(mesh.node_coords()).to(DEV)
        if case["op"] == "solve":
            state["u"] = torch.from_numpy(mesh.lumped_mass()).to(DEV) * _modes(xyz, case["lz"], seed)
        else:
            mesh.set_coefficients(KAPPA, 1.0 / DT)
            state["u"], state["q"] = _rod(xyz, case["lz"], seed)
        state["y"] = torch.zeros_like(state["u"])
    return state


def run(state):
    case = state["case"]
    mode = sem.SOLVE_FP32_REFINED if case["mode"] == "refined" else sem.SOLVE_FP64
    if case["op"] == "apply":
        return state["mesh"].apply_A(state["u"], state["y"])
    if case["op"] == "precond":
        return state["mesh"].precond(state["u"], state["y"])
    if case["op"] == "solve":
        return state["mesh"].solve(state["u"], state["y"], mode=mode, rtol=RTOL, inner_rtol=3e-3)[0]
    if case["op"] == "heat":
        return state["mesh"].heat_step(state["u"], DT, KAPPA, q=state["q"], u_next=state["y"], mode=mode, rtol=RTOL)[0]
    return state["batch"].solve(state["b"], state["x"], mode=mode, rtol=RTOL)[0]


def work(case):
    """Bytes: every vector that a step takes or gives once, the vertices and the coefficients; flops:
    the contractions and the factors rebuilt at each node (the operator), the six contractions by
    even and odd parts (the patch solves).  Solves: a typical number of iterations (the tolerance
    and the preconditioner fix it, 35 to 65 here), each an operator, a preconditioner and the
    updates of three vectors."""
    size = 4 if case["dtype"] == "f32" else 8

    def parts(k, n):
        elems, nodes = k[0] * k[1] * k[2], (k[0] * n + 1) * (k[1] * n + 1) * (k[2] * n + 1)
        local = elems * (n + 1) ** 3
        coef = {"none": 0, "element": 2 * elems, "node": 2 * local}[case["coef"]] * size
        return (size * (2 * nodes + 24 * elems) + coef, local * (12.0 * (n + 1) + 122), size * 2 * nodes,
                6.0 * elems * (n + 3) ** 4, nodes)

    if case["op"] == "batch":
        sizes = [(m[4], m[3]) for m in _meshes(case, 0)[0]]
    else:
        sizes = [((case["kx"], case["ky"], case["kz"]), case["order"])]
    total = {"bytes": 0.0, "flops": 0.0}
    for k, n in sizes:
        ab, af, pb, pf, nodes = parts(k, n)
        if case["op"] == "apply":
            b, f = ab, af
        elif case["op"] == "precond":
            b, f = pb, pf
        else:
            its = 12 if case["op"] == "heat" else 45
            if case["mode"] == "refined":  # FP32 vectors in the inner iterations
                ab, pb = ab / 2, pb / 2
            b = its * (ab + pb + (4 if case["mode"] == "refined" else 8) * 8 * nodes)
            f = its * (af + pf + 12.0 * nodes)
        total["bytes"] += b
        total["flops"] += f
    return total


# --- the same in plain FP64 ------------------------------------------------------------------

def _gll(n):
    """Gauss-Lobatto-Legendre points, weights and D[i, j] = phi_j'(t_i)."""
    leg = np.polynomial.legendre.Legendre.basis(n)
    t = np.concatenate([[-1.0], np.sort(leg.deriv().roots().real), [1.0]])
    p, dp = leg(t), leg.deriv()
    for _ in range(3):  # polish the inner roots of P_n'
        t[1:-1] -= dp(t[1:-1]) / dp.deriv()(t[1:-1])
    p = leg(t)
    with np.errstate(divide="ignore", invalid="ignore"):
        d = p[:, None] / (p[None, :] * (t[:, None] - t[None, :]))
    np.fill_diagonal(d, 0.0)
    d[0, 0], d[-1, -1] = -n * (n + 1) / 4.0, n * (n + 1) / 4.0
    return t, 2.0 / (n * (n + 1) * p ** 2), d


class _Plain:
    """The operator c m - div(kappa grad) and its two-scale preconditioner on a box mesh."""

    def __init__(self, mesh, kappa=None, c=None):
        vtx, hexes, pos, n, k = mesh
        self.n, self.k, self.n1, self.elems = n, k, n + 1, len(hexes)
        t, rho, d = _gll(n)
        self.t, self.rho, self.d = (torch.from_numpy(v).to(DEV) for v in (t, rho, d))
        self.mesh, self.pos = mesh, torch.from_numpy(pos).to(DEV)
        self.x8 = torch.from_numpy(vtx).to(DEV)[torch.from_numpy(hexes).to(DEV)]
        self.lat = self._lattice(hexes)
        self.nodes = self.lat.numel()
        ar = torch.arange(self.n1, device=DEV)
        axis = [self.pos[:, q, None] * n + ar for q in range(3)]
        self.l2g = self.lat[axis[2][:, :, None, None], axis[1][:, None, :, None], axis[0][:, None, None, :]]
        shape = (self.elems, self.n1, self.n1, self.n1)

        def per_node(v, default):
            if v is None:
                return torch.full((1, 1, 1, 1), float(default), dtype=torch.float64, device=DEV).expand(shape)
            v = torch.as_tensor(v, dtype=torch.float64, device=DEV)
            return v.reshape(shape) if v.numel() > self.elems else v.reshape(-1, 1, 1, 1).expand(shape)

        self.kappa, self.c = per_node(kappa, 1.0), per_node(c, 0.0)
        self.free = torch.zeros(self.nodes, dtype=torch.float64, device=DEV)
        self.free[self.lat[1:-1, 1:-1, 1:-1].reshape(-1)] = 1.0
        self.kept = None

    def _lattice(self, hexes):
        """Global id of each node of the (k n + 1)^3 lattice: vertices, then edges, faces (each by its
        smallest vertex, then xy, xz, yz) and element interiors."""
        n, (kx, ky, kz), m = self.n, self.k, self.n - 1
        v = torch.arange((kx + 1) * (ky + 1) * (kz + 1), device=DEV).reshape(kz + 1, ky + 1, kx + 1)
        lat = torch.empty((kz * n + 1, ky * n + 1, kx * n + 1), dtype=torch.int64, device=DEV)
        lat[::n, ::n, ::n] = v
        if m == 0:
            return lat
        room = [v % (kx + 1) < kx, torch.div(v, kx + 1, rounding_mode="floor") % (ky + 1) < ky,
                torch.div(v, (kx + 1) * (ky + 1), rounding_mode="floor") < kz]
        ar = torch.arange(m, device=DEV)
        inner = lambda q: [slice(1 + r, None, n) for r in range(m)] if q else [slice(0, None, n)]  # noqa: E731
        base = v.numel()
        # an entity spans a set of axes from its smallest vertex; entities of one kind are ranked together
        for kind in ([(0,), (1,), (2,)], [(0, 1), (0, 2), (1, 2)]):
            here = torch.stack([torch.stack([room[a] for a in axes]).all(0).reshape(-1) for axes in kind], dim=1)
            rank = (torch.cumsum(here.reshape(-1).to(torch.int64), 0) - 1).reshape(here.shape)
            size = m ** len(kind[0])
            for q, axes in enumerate(kind):
                ids = base + rank[:, q].reshape(v.shape) * size
                ids = ids[tuple(slice(0, v.shape[2 - a] - 1) if a in axes else slice(None) for a in (2, 1, 0))]
                for x, sx in enumerate(inner(0 in axes)):
                    for y, sy in enumerate(inner(1 in axes)):
                        for z, sz in enumerate(inner(2 in axes)):
                            o = [w for w, a in zip((x, y, z), (0, 1, 2)) if a in axes]
                            lat[sz, sy, sx] = ids + sum(w * m ** i for i, w in enumerate(o))
            base += int(here.sum()) * size
        at = [self.pos[:, q, None] * n + 1 + ar for q in range(3)]
        lat[at[2][:, :, None, None], at[1][:, None, :, None], at[0][:, None, None, :]] = (
            base + torch.arange(self.elems, device=DEV)[:, None, None, None] * m ** 3
            + (ar[:, None, None] * m + ar[None, :, None]) * m + ar[None, None, :])
        return lat

    def _shape(self):
        """phi[corner, k, j, i] of the trilinear map and its three derivatives."""
        p = torch.stack([(1 - self.t) / 2, (1 + self.t) / 2])
        g = torch.tensor([[-0.5], [0.5]], dtype=torch.float64, device=DEV).expand(2, self.n1)
        pick = lambda f, s: f[[q >> s & 1 for q in range(8)]]  # noqa: E731
        out = []
        for which in (None, 0, 1, 2):
            fx, fy, fz = (pick(g if which == a else p, a) for a in range(3))
            out.append(fz[:, :, None, None] * fy[:, None, :, None] * fx[:, None, None, :])
        return out

    def coords(self):
        x = torch.tensordot(self.x8.transpose(1, 2), self._shape()[0], dims=([2], [0]))  # [E, 3, k, j, i]
        out = torch.empty((self.nodes, 3), dtype=torch.float64, device=DEV)
        for q in range(3):
            out[self.l2g.reshape(-1), q] = x[:, q].reshape(-1)
        return out

    def _factors(self, e0, e1):
        """Weighted inverse metric (times kappa) and mass of elements e0..e1."""
        x = self.x8[e0:e1].transpose(1, 2)
        j = [torch.tensordot(x, s, dims=([2], [0])) for s in self._shape()[1:]]  # dx/dxi_a: [e, 3, k, j, i]
        cof = [torch.linalg.cross(j[1], j[2], dim=1), torch.linalg.cross(j[2], j[0], dim=1),
               torch.linalg.cross(j[0], j[1], dim=1)]
        det = (j[0] * cof[0]).sum(1)
        w = self.rho[:, None, None] * self.rho[None, :, None] * self.rho[None, None, :]
        s = self.kappa[e0:e1] * w / det
        return [[s * (cof[a] * cof[b]).sum(1) if a <= b else None for b in range(3)] for a in range(3)], w * det

    def _chunks(self):
        step = max(1, 4_000_000 // self.n1 ** 3)
        return [(e, min(self.elems, e + step)) for e in range(0, self.elems, step)]

    def mass(self):
        out = torch.zeros(self.nodes, dtype=torch.float64, device=DEV)
        for e0, e1 in self._chunks():
            out.index_add_(0, self.l2g[e0:e1].reshape(-1), self._factors(e0, e1)[1].reshape(-1))
        return out

    def apply(self, u):
        if self.kept is None:
            self.kept = [self._factors(*c) for c in self._chunks()] if self.l2g.numel() <= 9_000_000 else []
        y, n1 = torch.zeros_like(u), self.n1
        for q, (e0, e1) in enumerate(self._chunks()):
            g, m = self.kept[q] if self.kept else self._factors(e0, e1)
            v = u[self.l2g[e0:e1]]
            du = [v @ self.d.T.contiguous(), self.d @ v, (self.d @ v.reshape(-1, n1, n1 * n1)).reshape(v.shape)]
            f = [sum(g[min(a, b)][max(a, b)] * du[b] for b in range(3)) for a in range(3)]
            dt = self.d.T.contiguous()
            out = f[0] @ self.d + dt @ f[1] + (dt @ f[2].reshape(-1, n1, n1 * n1)).reshape(v.shape)
            out += self.c[e0:e1] * m * v
            y.index_add_(0, self.l2g[e0:e1].reshape(-1), out.reshape(-1))
        return y * self.free

    def diagonal(self):
        """The operator's diagonal without its mixed terms: a Jacobi preconditioner."""
        out = torch.zeros(self.nodes, dtype=torch.float64, device=DEV)
        d2 = self.d.T.contiguous() ** 2
        for e0, e1 in self._chunks():
            g, m = self._factors(e0, e1)
            v = g[0][0] @ d2.T.contiguous() + d2 @ g[1][1]
            v += (d2 @ g[2][2].reshape(-1, self.n1, self.n1 ** 2)).reshape(v.shape) + self.c[e0:e1] * m
            out.index_add_(0, self.l2g[e0:e1].reshape(-1), v.reshape(-1))
        return out

    def solve(self, b, tol=1e-14, most=6000):
        b = b * self.free
        inv = self.free / self.diagonal()
        x, r = torch.zeros_like(b), b.clone()
        z = inv * r
        p, rz, stop = z.clone(), torch.dot(r, z), tol * float(torch.linalg.norm(b))
        for it in range(most):
            w = self.apply(p)
            alpha = rz / torch.dot(p, w)
            x += alpha * p
            r -= alpha * w
            if it % 20 == 19 and float(torch.linalg.norm(r)) <= stop:
                break
            z = inv * r
            rz, old = torch.dot(r, z), rz
            p = z + (rz / old) * p
        r = b - self.apply(x)
        return x if float(torch.linalg.norm(r)) <= 1e-11 * float(torch.linalg.norm(b)) else None

    def element_means(self):
        w = self.rho[:, None, None] * self.rho[None, :, None] * self.rho[None, None, :] / 8
        return (self.kappa * w).sum((1, 2, 3)), (self.c * w).sum((1, 2, 3))

    def precond(self, r):
        n, m = self.n, self.n + 3
        kap, c = self.element_means()
        # the 1D pencil of an element and one node of each neighbour, K S = M S diag(lam), S^T M S = I
        d, rho = self.d.cpu().numpy(), self.rho.cpu().numpy()
        st = d.T @ np.diag(rho) @ d
        kk, mm = np.zeros((m, m)), np.zeros(m)
        for at, keep in ((slice(1, n + 2), slice(0, n + 1)), (slice(0, 2), slice(n - 1, n + 1)),
                         (slice(n + 1, m), slice(0, 2))):
            kk[at, at] += st[keep, keep]
            mm[at] += rho[keep]
        lam, q = np.linalg.eigh(kk / np.sqrt(mm[:, None] * mm[None, :]))
        s = torch.from_numpy(q / np.sqrt(mm)[:, None]).to(DEV)
        lam, sT = torch.from_numpy(lam).to(DEV), s.T.contiguous()
        edge = lambda a: torch.stack([torch.linalg.norm(self.x8[:, p | 1 << a] - self.x8[:, p], dim=1)  # noqa: E731
                                      for p in range(8) if not p >> a & 1]).mean(0)
        h = [edge(a) for a in range(3)]
        pad = torch.zeros([v + 2 for v in self.lat.shape], dtype=torch.float64, device=DEV)
        pad[1:-1, 1:-1, 1:-1] = r[self.lat]
        z = torch.zeros_like(pad).reshape(-1)
        idx = torch.arange(pad.numel(), device=DEV).reshape(pad.shape)
        ar = torch.arange(m, device=DEV)
        step = max(1, 4_000_000 // m ** 3)
        cube = lambda v, x: ((x @ v.T.contiguous()).transpose(2, 3) @ v.T.contiguous()).transpose(2, 3)  # noqa: E731
        line = lambda v, x: (v @ x.reshape(-1, m, m * m)).reshape(x.shape)  # noqa: E731
        for e0 in range(0, self.elems, step):
            e = slice(e0, min(self.elems, e0 + step))
            at = [self.pos[e, a, None] * n + ar for a in range(3)]
            node = idx[at[2][:, :, None, None], at[1][:, None, :, None], at[0][:, None, None, :]]
            v = pad.reshape(-1)[node]
            v = line(sT, cube(sT, v))
            shift = [lam[None, :] / h[a][e, None] ** 2 for a in range(3)]
            v = v / (4 * kap[e, None, None, None] * (shift[0][:, None, None, :] + shift[1][:, None, :, None]
                                                     + shift[2][:, :, None, None]) + c[e, None, None, None])
            v = line(s, cube(s, v)) * (8 / (h[0] * h[1] * h[2]))[e, None, None, None]
            z.index_add_(0, node.reshape(-1), v.reshape(-1))
        out = torch.zeros_like(r)
        out[self.lat.reshape(-1)] = z.reshape(pad.shape)[1:-1, 1:-1, 1:-1].reshape(-1)
        # the order-1 correction: interpolate, solve on the vertices, interpolate back
        vtx, hexes, pos, _, k = self.mesh
        coarse = _Plain((vtx, hexes, pos, 1, k), kap, c)
        phi = self._shape()[0].reshape(8, -1)
        first = torch.full((self.nodes,), self.l2g.numel(), dtype=torch.int64, device=DEV)
        flat = self.l2g.reshape(-1)
        first.scatter_reduce_(0, flat, torch.arange(flat.numel(), device=DEV), "amin")
        own = first[flat] == torch.arange(flat.numel(), device=DEV)
        rl = (r[flat] * own).reshape(self.elems, -1)
        rc = torch.zeros(coarse.nodes, dtype=torch.float64, device=DEV)
        rc.index_add_(0, coarse.l2g.reshape(-1), (rl @ phi.T.contiguous()).reshape(-1))
        if float(coarse.free.sum()) > 0:
            zc = coarse.solve(rc)
            if zc is None:
                return None
            zl = (zc[coarse.l2g.reshape(self.elems, 8)] @ phi).reshape(-1)
            corr = torch.empty_like(out)
            corr[flat] = zl  # the same at every copy of a node
            out += corr
        return out * self.free


def exact(case, seed):
    meshes, rng = _meshes(case, seed)
    if case["op"] == "batch":
        out = []
        for i, mesh in enumerate(meshes):
            if len(mesh[1]) * (mesh[3] + 1) ** 3 > 250_000:
                out.append(None)
                continue
            plain = _Plain(mesh)
            out.append(plain.solve(_noise(plain.nodes, seed * 64 + i)))
        return out
    local = len(meshes[0][1]) * (case["order"] + 1) ** 3
    if case["op"] in ("solve", "heat") and local > 7_500_000:
        return None
    kappa, c = _coefficients(case, len(meshes[0][1]), case["order"], rng)
    if case["op"] == "heat":
        kappa, c = np.full(len(meshes[0][1]), KAPPA), np.full(len(meshes[0][1]), 1.0 / DT)
    plain = _Plain(meshes[0], kappa, c)
    dtype = torch.float32 if case["dtype"] == "f32" else torch.float64
    if case["op"] == "apply":
        return plain.apply(_noise(plain.nodes, seed, dtype).double())
    if case["op"] == "precond":
        return plain.precond(_noise(plain.nodes, seed, dtype).double() * plain.free)
    if case["op"] == "solve":
        return plain.solve(plain.mass() * _modes(plain.coords(), case["lz"], seed))
    u, q = _rod(plain.coords(), case["lz"], seed)
    return plain.solve(plain.mass() * (u / DT + q))
