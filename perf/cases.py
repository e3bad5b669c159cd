"""Measured work of this framework, through its public entry points.

A case is one call (or the short chain of calls) that a laminate analysis makes, on a part
of this repository's own kinds: the flat laminate and the curved, wrinkled L-section of
``workloads``, resin interfaces between the plies, at sizes from the 8 x 8 x 12 coupon to
the 3M-DOF plate.  ``op`` names the call:

* ``spmv``      y = K x, what a program's own Krylov or time-stepping loop calls;
* ``assemble``  K and f of a mesh, and K u0 for a starting guess (warm starts need it);
* ``setup``     decomposition, GenEO coarse space and factors, and one application of P;
* ``pcg``       one solve with a preconditioner that is there (many load cases, one part);
* ``solve``     the whole step: mesh, assembly, set-up and solve;
* ``sweep``     the same for several wrinkle samples at once (``Batch``, lockstep PCG);
* ``adjoint``   J and its gradient for a displacement (the backward direction);
* ``stress``    delamination criterion at every Gauss point and J (after each solve);
* ``band``      the batched band Cholesky and its solves on their own.

The seed draws the wrinkle, the ply moduli (5% scatter), the load and the vectors.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1707_04228_amd as gx
import workloads

ANGLES = (0, 45, 90, -45)
RADIUS, PLY_T, RESIN_T = 5.0, 0.25, 0.05
S33, S13 = 61.0, 97.0
PRECISION = {"fp64": gx.GX_FP64, "mixed": gx.GX_MIXED}


# ---- cases ---------------------------------------------------------------------------------
def part(op, geometry, nx, ny, plies, ply_nel, px=1, py=1, overlap=2, precision="fp64",
         limb=10.0, **more):
    return dict(op=op, geometry=geometry, nx=nx, ny=ny, plies=plies, ply_nel=ply_nel, px=px,
                py=py, overlap=overlap, precision=precision, limb=limb, **more)


def listed():
    return [
        # the smallest product: one coupon, bound by the call itself
        dict(name="spmv_coupon", **part("spmv", "flat", 8, 8, 4, 2)),
        # the 3M-DOF plate's product: the largest matrix, bound by memory
        dict(name="spmv_plate", **part("spmv", "flat", 64, 64, 12, 4)),
        # a 490k-DOF corner strip (the sensitivity mesh), assembled again for each wrinkle
        dict(name="assemble_strip", **part("assemble", "lsection", 240, 4, 12, 2, limb=40.0)),
        # set-up of a 750k-DOF plate in 16 subdomains: factorisations and eigensolves
        dict(name="setup_plate", **part("setup", "flat", 32, 32, 12, 4, 4, 4)),
        # one load case on the 3M-DOF plate, FP32 factors: the largest solve
        dict(name="pcg_plate_mixed", **part("pcg", "flat", 64, 64, 12, 4, 8, 8,
                                            precision="mixed")),
        # one load case on the corner strip: few subdomains, a long chain of small solves
        dict(name="pcg_strip", **part("pcg", "lsection", 240, 4, 12, 2, 16, 1, limb=40.0)),
        # the smallest whole step: launches and latency
        dict(name="solve_coupon", **part("solve", "flat", 8, 8, 4, 2, 2, 2, overlap=1)),
        # one wrinkle sample of ordinary size, whole step, mixed precision
        dict(name="solve_sample_mixed", **part("solve", "lsection", 64, 9, 8, 2, 5, 1,
                                               precision="mixed")),
        # four small samples of the wrinkle sweep together, different in layup
        dict(name="sweep_four_mixed", **part("sweep", "lsection", 40, 4, 6, 2, 2, 1,
                                             precision="mixed", samples=4)),
        # gradient of the unfolding functional on a corner, one optimisation step
        dict(name="adjoint_corner", **part("adjoint", "lsection", 48, 6, 6, 2, 6, 1)),
        # strength assessment of the corner strip after its solve
        dict(name="stress_strip", **part("stress", "lsection", 240, 4, 12, 2, limb=40.0)),
        # local problems of ragged sizes with a block of right-hand sides
        dict(name="band_ragged", op="band", n_mat=12, n=2500, bw=420, nrhs=16),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["spmv", "assemble", "setup", "pcg", "solve", "sweep", "adjoint", "stress",
                     "band"])
    if op == "band":
        return dict(op=op, n_mat=rng.randint(1, 24), n=log(60, 3000), bw=log(3, 600),
                    nrhs=rng.choice([1, 8, 16, 32, 40]))
    geometry = rng.choice(["flat", "lsection"])
    plies, ply_nel = rng.randint(2, 12), rng.choice([1, 2, 3, 4])
    if op in ("spmv", "assemble", "stress"):          # no decomposition: any size
        nx = log(12, 100) if geometry == "lsection" else log(3, 64)
        return part(op, geometry, nx, log(2, 40), plies, ply_nel, limb=rng.choice([10.0, 40.0]))
    px = rng.randint(2, 4) if op in ("sweep", "adjoint") else rng.randint(2, 8)
    nx = px * rng.randint(6, 9) + rng.randint(0, 3)
    nx = max(nx, 24) if geometry == "lsection" else nx
    ny = rng.randint(3, 12)
    if op in ("sweep", "adjoint"):
        plies, ny = rng.randint(2, 6), rng.randint(2, 6)
    case = part(op, geometry, nx, ny, plies, min(ply_nel, 2), px, 2 if ny >= 10 else 1,
                rng.choice([1, 2]), rng.choice(["fp64", "mixed"]) if op in
                ("pcg", "solve", "sweep") else "fp64")
    if op == "sweep":
        case["samples"] = rng.randint(2, 4)
    return case


def descriptor(case, seed):
    """The laminate descriptor of a case: layup and mesh from the case, the rest drawn."""
    rng = np.random.default_rng(seed)
    layers = workloads.ply_layers([ANGLES[k % 4] for k in range(case["plies"])], PLY_T,
                                  case["ply_nel"], RESIN_T, 1)
    for L in layers:
        key, mean = (("E1", workloads.PLY["E1"]) if L["mat"] == "ply" else
                     ("E", workloads.RESIN["E"]))
        L[key] = float(mean * rng.uniform(0.95, 1.05))
    cfg = dict(name="case", geometry=case["geometry"], nx=case["nx"], ny=case["ny"],
               layers=layers, wrinkle=(float(rng.uniform(0.02, 0.3)), float(rng.uniform(3, 8))),
               solver=dict(px=case["px"], py=case["py"], overlap=case["overlap"], nev=0,
                           tau=0.1, nev_max=32, rtol=1e-8))
    if case["geometry"] == "flat":
        cfg.update(length=0.8 * case["nx"], width=0.8 * case["ny"],
                   load={"kind": "traction",
                         "t0": (1.0, float(rng.normal(0, 0.1)), float(rng.normal(0, 0.01)))})
    else:
        thick = sum(L["t"] for L in layers)
        arc = 0.5 * math.pi * (RADIUS + 0.5 * thick)
        cfg.update(radius=RADIUS, limb=case["limb"], width=10.0,
                   nx_limb=int(round(case["nx"] * case["limb"] / (2 * case["limb"] + arc))),
                   load={"kind": "moment",
                         "M": float(workloads.PAPER_MOMENT * rng.uniform(0.5, 1.5))})
    return cfg


def samples_of(case, seed):
    """The laminates of a sweep: further plies from sample to sample."""
    return [descriptor(dict(case, plies=case["plies"] + k % 3), 1000 * seed + k)
            for k in range(case["samples"])]


def vector(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n, dtype=torch.float64, device="cuda", generator=g)


def bands(case, seed):
    """Band matrices of ragged orders and widths: decaying off-diagonals, dominant diagonal
    (as the equilibrated local stiffness has), row-major band storage; and right-hand sides."""
    rng = np.random.default_rng(case["n"] + case["bw"])      # the sizes belong to the case
    n = np.maximum(1, (case["n"] * rng.uniform(0.5, 1.0, case["n_mat"])).astype(np.int64))
    bw = np.minimum(np.maximum(1, (case["bw"] * rng.uniform(0.6, 1.0, case["n_mat"]))
                               .astype(np.int64)), n - 1)
    g = torch.Generator(device="cuda").manual_seed(seed)
    mats = []
    for nj, bj in zip(n.tolist(), bw.tolist()):
        d = torch.arange(bj, -1, -1, dtype=torch.float64, device="cuda")    # column distance
        a = torch.randn(nj, bj + 1, dtype=torch.float64, device="cuda", generator=g)
        a = a * torch.exp(-4.0 * d / (bj + 1)) / math.sqrt(bj + 1)
        a[:, bj] = 4.0 + a[:, bj].abs()
        r = torch.arange(nj, device="cuda")[:, None]
        a[r - d.long()[None, :] < 0] = 0.0                                  # left of column 0
        mats.append(a)
    x = torch.randn(int(n.sum()) * case["nrhs"], dtype=torch.float64, device="cuda", generator=g)
    return n, bw, mats, x


# ---- one pass --------------------------------------------------------------------------------
def prepare(case, seed):
    op = case["op"]
    st = {"op": op, "case": case}
    if op == "band":
        n, bw, mats, x = bands(case, seed)
        st.update(solver=gx.Solver(stream=torch.cuda.Stream()), n=n, bw=bw,
                  band=torch.cat([m.reshape(-1) for m in mats]), b=x)
    elif op == "sweep":
        st["cfgs"] = samples_of(case, seed)
    else:
        s = st["solver"] = gx.Solver(stream=torch.cuda.Stream())
        cfg = st["cfg"] = descriptor(case, seed)
        if op != "solve":
            st["mesh"] = s.laminate(cfg)
        if op in ("spmv", "assemble"):
            st["x"] = vector(3 * st["mesh"]["n_nodes"], seed)
        if op in ("spmv", "setup", "pcg", "adjoint", "stress"):
            st["f"] = s.assemble()
        if op in ("setup", "pcg", "adjoint"):
            st["part"] = s.partition(cfg, case["px"], case["py"])
        if op in ("pcg", "adjoint"):
            set_up(s, case, st["part"])
        if op == "adjoint":
            st["u"] = s.pcg(st["f"], rtol=1e-12, maxit=5000)["x"]
        if op == "stress":
            st["u"] = displacement(st["mesh"]["xyz"].view(-1, 3), seed).reshape(-1).contiguous()
    torch.cuda.synchronize()
    return st


def set_up(s, case, elem_part):
    return s.geneo_setup(elem_part, case["px"] * case["py"], overlap=case["overlap"], tau=0.1,
                         nev_max=32, precision=PRECISION[case["precision"]])


def displacement(xyz, seed):
    """A smooth bending-and-stretching field of the size a loaded part has (mm)."""
    rng = np.random.default_rng(seed + 1)
    k = torch.tensor(rng.uniform(0.05, 0.25, (3, 3)), dtype=torch.float64, device=xyz.device)
    a = torch.tensor(rng.uniform(0.01, 0.05, 3), dtype=torch.float64, device=xyz.device)
    ph = torch.tensor(rng.uniform(0, 6, 3), dtype=torch.float64, device=xyz.device)
    return a * torch.sin(xyz @ k.T + ph)


def run(st):
    op, case = st["op"], st["case"]
    if op == "sweep":
        batch = gx.Batch(st["cfgs"], precision=PRECISION[case["precision"]])
        batch.setup()
        xs, _, _, status = batch.solve(rtol=1e-8, maxit=3000)
        batch.close()
        if np.any(status):
            raise RuntimeError(f"sweep did not converge: {status}")
        return xs
    s = st["solver"]
    if op == "spmv":
        return s.spmv(st["x"])
    if op == "assemble":
        f = s.assemble(st["cfg"], st["mesh"])
        return {"f": f, "Ku": s.spmv(st["x"])}
    if op == "setup":
        nev, n0 = set_up(s, case, st["part"])
        return {"nev": nev, "n0": n0, "z": s.precond(st["f"]),
                "lambda": np.concatenate([s.eigenvalues(j) for j in range(len(nev))])}
    if op == "pcg":
        return s.pcg(st["f"], rtol=1e-8, maxit=3000)["x"]
    if op == "solve":
        cfg = st["cfg"]
        s.laminate(cfg)
        f = s.assemble()
        set_up(s, case, s.partition(cfg, case["px"], case["py"]))
        return {"f": f, "x": s.pcg(f, rtol=1e-8, maxit=3000)["x"]}
    if op == "adjoint":
        J, g, _ = s.adjoint(st["u"], st["cfg"], region=1, rtol=1e-12, maxit=5000)
        return {"J": np.array([J]), "dJdp": g}
    if op == "stress":
        r = s.failure(st["u"], per_gauss=True)
        return {"J": np.array([s.objective(st["u"], st["cfg"], region=1)]),
                "F_max": np.array([r["F_max"]]), "elem": r["elem"], "gauss": r["gauss"],
                "stress": r["stresses"], "F_elem": r["F_elem"], "F_gauss": r["F_gauss"]}
    return s.band_factor_solve(st["n"], st["bw"], st["band"], st["b"].clone())


# ---- what a pass cannot do without --------------------------------------------------------
def work(case):
    if case["op"] == "band":
        n, b = 0.75 * case["n"], min(0.8 * case["bw"], 0.75 * case["n"])
        e = case["n_mat"] * n * b                     # stored entries, on average
        return {"bytes": 8 * (2 * e + 2 * case["n_mat"] * n * case["nrhs"]),
                "flops": e * b + 4 * e * case["nrhs"]}
    if case["op"] == "sweep":
        one = [work(dict(case, op="solve", plies=case["plies"] + k % 3))
               for k in range(case["samples"])]
        return {k: sum(w[k] for w in one) for k in one[0]}
    nx, ny = case["nx"], case["ny"]
    nz = case["plies"] * (case["ply_nel"] + 1) - 1
    ne = nx * ny * nz
    nodes = (nx + 1) * (ny + 1) * (nz + 1) + nx * (ny + 1) * (nz + 1) \
        + ny * (nx + 1) * (nz + 1) + nz * (nx + 1) * (ny + 1)
    # couplings: vertices see 81 nodes and mid-edge nodes 51 inside the mesh
    blocks = 81 * (nx + 1) * (ny + 1) * (nz + 1) + 51 * (nodes - (nx + 1) * (ny + 1) * (nz + 1))
    k_bytes, vec, mesh = 76 * blocks, 24 * nodes, 80 * ne + 24 * nodes
    # element matrices: 27 points, the upper half of B^T C B
    k_flops = 27 * 2.0 * (60 * 6 * 6 + 60 * 61 / 2 * 6) * ne
    if case["op"] == "spmv":
        return {"bytes": k_bytes + 2 * vec, "flops": 18 * blocks}
    if case["op"] == "assemble":
        return {"bytes": mesh + 2 * k_bytes + 3 * vec, "flops": k_flops + 18 * blocks}
    if case["op"] == "stress":
        return {"bytes": 2 * (mesh + vec) + 8 * 28 * ne, "flops": 27 * 3000.0 * ne}
    # subdomains: boxes grown by the overlap, thickness-major order, so the half-bandwidth is
    # one element layer's share of DOFs
    bx = min(nx, nx / case["px"] + 2 * case["overlap"] * (case["px"] > 1))
    by = min(ny, ny / case["py"] + 2 * case["overlap"] * (case["py"] > 1))
    bw = 3 * 4 * bx * by
    entries = case["px"] * case["py"] * bw * nz * bw * 0.86
    w = 8 if case["precision"] == "fp64" else 4
    setup = {"bytes": w * 4 * entries + 2 * 10 * w * entries, "flops": 2 * entries * bw}
    solve = {"bytes": 60 * (2 * w * entries + k_bytes + 10 * vec), "flops": 60 * 4 * entries}
    if case["op"] == "setup":
        return setup
    if case["op"] == "pcg":
        return solve
    if case["op"] == "adjoint":
        return {"bytes": 2 * solve["bytes"], "flops": 2 * solve["flops"] + 27 * 2e4 * ne}
    return {"bytes": mesh + k_bytes + setup["bytes"] + solve["bytes"],
            "flops": k_flops + setup["flops"] + solve["flops"]}


# ---- exact values -----------------------------------------------------------------------------
# The discrete problem once more in plain torch, 64 bits: mesh, serendipity shape functions,
# 3 x 3 x 3 Gauss points, strains turned into the ply's axes, all matrix-free.
_F8 = dict(dtype=torch.float64, device="cuda" if torch.cuda.is_available() else "cpu")
_VERT = [(i, j, k) for k in (-1, 1) for j in (-1, 1) for i in (-1, 1)]
_EDGE = [(0, j, k) for k in (-1, 1) for j in (-1, 1)] + \
    [(i, 0, k) for k in (-1, 1) for i in (-1, 1)] + [(i, j, 0) for j in (-1, 1) for i in (-1, 1)]
_REF = _VERT + _EDGE
_G = math.sqrt(0.6)
_GAUSS = [(-_G, 5 / 9), (0.0, 8 / 9), (_G, 5 / 9)]


def _shape(p):
    """Shape functions [P, 20] and their reference gradients [P, 20, 3] at points p [P, 3]."""
    p = p.clone().requires_grad_(True)
    N = []
    for r in _REF:
        f = [1 + p[:, i] * r[i] if r[i] else 1 - p[:, i] ** 2 for i in range(3)]
        v = f[0] * f[1] * f[2]
        N.append(0.125 * v * (sum(p[:, i] * r[i] for i in range(3)) - 2) if all(r) else 0.25 * v)
    g = [torch.autograd.grad(v.sum(), p, retain_graph=True)[0] for v in N]
    return torch.stack(N, 1).detach(), torch.stack(g, 1)


class _Part:
    def __init__(self, cfg):
        self.cfg = cfg
        nx, ny, layers = cfg["nx"], cfg["ny"], cfg["layers"]
        nz = sum(L["nel"] for L in layers)
        z, lay, z0 = [0.0], [], 0.0
        for i, L in enumerate(layers):
            z += [z0 + L["t"] * (k + 1) / L["nel"] for k in range(L["nel"])]
            lay += [i] * L["nel"]
            z0 += L["t"]
        self.T = z0
        flat = cfg["geometry"] == "flat"
        if flat:
            s = np.linspace(0, cfg["length"], nx + 1)
        else:
            rm, nl = RADIUS + 0.5 * self.T, cfg["nx_limb"]
            h = 0.25 * math.pi * rm
            s = np.concatenate([np.linspace(-h - cfg["limb"], -h, nl + 1)[:-1],
                                np.linspace(-h, h, nx - 2 * nl + 1),
                                np.linspace(h, h + cfg["limb"], nl + 1)[1:]])

        def lattice(b):
            out = np.empty(2 * len(b) - 1)
            out[0::2], out[1::2] = b, 0.5 * (np.asarray(b)[1:] + np.asarray(b)[:-1])
            return torch.tensor(out, **_F8)

        dev = _F8["device"]
        k2, j2, i2 = torch.meshgrid(torch.arange(2 * nz + 1, device=dev),
                                    torch.arange(2 * ny + 1, device=dev),
                                    torch.arange(2 * nx + 1, device=dev), indexing="ij")
        node = (k2 % 2 + j2 % 2 + i2 % 2) <= 1
        number = torch.cumsum(node.reshape(-1).long(), 0).reshape(node.shape) - 1
        S, Y, Z = (lattice(b)[i[node]] for b, i in
                   ((s, i2), (np.linspace(0, cfg["width"], ny + 1), j2), (z, k2)))
        amp, wl = cfg["wrinkle"]
        d = S - 0.5 * cfg["length"] if flat else S
        Z = Z + amp * torch.exp(-(d / wl) ** 2) * torch.cos(2 * math.pi * d / wl)
        if flat:
            X = S
        else:
            rho, th = RADIUS + Z, (S + h) / rm
            X = torch.where(S < -h, cfg["limb"] + S + h,
                            torch.where(S > h, cfg["limb"] + rho, cfg["limb"] + rho * torch.sin(th)))
            Z = torch.where(S < -h, rho, torch.where(S > h, h - S, rho * torch.cos(th)))
        self.xyz = torch.stack([X, Y, Z], 1)
        ez, ey, ex = (t.reshape(-1) for t in torch.meshgrid(
            torch.arange(nz, device=dev), torch.arange(ny, device=dev),
            torch.arange(nx, device=dev), indexing="ij"))
        self.conn = torch.stack([number[2 * ez + 1 + r[2], 2 * ey + 1 + r[1], 2 * ex + 1 + r[0]]
                                 for r in _REF], 1)
        self.ex, self.layer = ex, torch.tensor(lay, device=dev)[ez]
        self.clamped = number[:, :, 0][node[:, :, 0]]
        self.n = 3 * self.xyz.shape[0]
        self.arc = torch.ones_like(ex, dtype=torch.bool) if flat else \
            (ex >= cfg["nx_limb"]) & (ex < nx - cfg["nx_limb"])
        pts = [(x, y, w, a * b * c) for w, c in _GAUSS for y, b in _GAUSS for x, a in _GAUSS]
        self.w = torch.tensor([p[3] for p in pts], **_F8)
        _, self.dN = _shape(torch.tensor([p[:3] for p in pts], **_F8))
        self.C = torch.stack([self._stiffness(L) for L in layers])
        self.angle = torch.tensor([math.radians(L["angle"]) for L in layers], **_F8)

    @staticmethod
    def _stiffness(L):
        S = torch.zeros(6, 6, **_F8)
        if L["mat"] == "ply":
            p = dict(workloads.PLY, E1=L["E1"])
        else:
            e, nu = L["E"], workloads.RESIN["nu"]
            p = dict(E1=e, E2=e, E3=e, nu12=nu, nu13=nu, nu23=nu,
                     **{k: e / (2 * (1 + nu)) for k in ("G12", "G13", "G23")})
        S[0, 0], S[1, 1], S[2, 2] = 1 / p["E1"], 1 / p["E2"], 1 / p["E3"]
        S[0, 1] = S[1, 0] = -p["nu12"] / p["E1"]
        S[0, 2] = S[2, 0] = -p["nu13"] / p["E1"]
        S[1, 2] = S[2, 1] = -p["nu23"] / p["E2"]
        S[3, 3], S[4, 4], S[5, 5] = 1 / p["G23"], 1 / p["G13"], 1 / p["G12"]
        return torch.linalg.inv(S.cpu()).to(S.device)

    def chunks(self, size=16384):
        return torch.arange(self.conn.shape[0], device=self.conn.device).split(size)

    def points(self, e):
        """Physical gradients [E, 27, 20, 3], det J w [E, 27] and local frames [E, 27, 3, 3]."""
        J = torch.einsum("eai,qaj->eqij", self.xyz[self.conn[e]], self.dN)
        c0, c1, c2 = J.unbind(-1)
        n12 = torch.linalg.cross(c1, c2)
        det = (c0 * n12).sum(-1)
        inv = torch.stack([n12, torch.linalg.cross(c2, c0), torch.linalg.cross(c0, c1)], -2) \
            / det[..., None, None]
        e1 = c0 / c0.norm(dim=-1, keepdim=True)
        e2 = c1 - (c1 * e1).sum(-1, keepdim=True) * e1
        e2 = e2 / e2.norm(dim=-1, keepdim=True)
        frame = torch.stack([e1, e2, torch.linalg.cross(e1, e2)], -2)
        return torch.einsum("qaj,eqji->eqai", self.dN, inv), det * self.w, frame

    def axes(self, e, E):
        """The plies' axes: the frames turned by the ply angles about their normals."""
        a = self.angle[self.layer[e]][:, None, None]
        return torch.stack([torch.cos(a) * E[..., 0, :] + torch.sin(a) * E[..., 1, :],
                            torch.cos(a) * E[..., 1, :] - torch.sin(a) * E[..., 0, :],
                            E[..., 2, :]], -2)

    def local_stress(self, e, u):
        """Stress tensors in the plies' axes, the axes Q, the frames, gradients and weights."""
        G, wd, E = self.points(e)
        Q = self.axes(e, E)
        H = torch.einsum("eai,eqaj->eqij", u.view(-1, 3)[self.conn[e]], G)
        t = Q @ (0.5 * (H + H.transpose(-1, -2))) @ Q.transpose(-1, -2)
        v = torch.stack([t[..., 0, 0], t[..., 1, 1], t[..., 2, 2], 2 * t[..., 1, 2],
                         2 * t[..., 0, 2], 2 * t[..., 0, 1]], -1)
        s = torch.einsum("eij,eqj->eqi", self.C[self.layer[e]], v)
        S = s[..., [0, 5, 4, 5, 1, 3, 4, 3, 2]].reshape(*s.shape[:-1], 3, 3)
        return S, Q, E, G, wd

    def apply(self, x):
        """K x, clamped degrees of freedom as identity rows and columns."""
        fixed = (3 * self.clamped[:, None] + torch.arange(3, device=x.device)).reshape(-1)
        u = x.clone()
        u[fixed] = 0.0
        y = torch.zeros(self.n // 3, 3, **_F8)
        for e in self.chunks():
            S, Q, _, G, wd = self.local_stress(e, u)
            S = Q.transpose(-1, -2) @ S @ Q * wd[..., None, None]
            y.index_add_(0, self.conn[e].reshape(-1),
                         torch.einsum("eqij,eqaj->eai", S, G).reshape(-1, 3))
        y = y.reshape(-1)
        y[fixed] = x[fixed]
        return y

    def dense(self):
        """K as a dense matrix (small parts)."""
        fixed = (3 * self.clamped[:, None] + torch.arange(3, device=self.ex.device)).reshape(-1)
        K = torch.zeros(self.n * self.n, **_F8)
        for e in self.chunks(64):
            G, wd, E = self.points(e)
            Q = self.axes(e, E)
            Qg = torch.einsum("eqli,eqai->eqal", Q, G)
            t = torch.einsum("eqki,eqal->eqaikl", Q, Qg)
            t = 0.5 * (t + t.transpose(-1, -2)).reshape(*wd.shape, 60, 9)
            B = torch.stack([t[..., 0], t[..., 4], t[..., 8], 2 * t[..., 5], 2 * t[..., 2],
                             2 * t[..., 1]], -1)
            Ke = torch.einsum("eqxi,eij,eqyj,eq->exy", B, self.C[self.layer[e]], B, wd)
            dof = (3 * self.conn[e][..., None] + torch.arange(3, device=e.device)).reshape(-1, 60)
            K.index_add_(0, (dof[:, :, None] * self.n + dof[:, None, :]).reshape(-1),
                         Ke.reshape(-1))
        K = K.view(self.n, self.n)
        K[fixed] = 0.0
        K[:, fixed] = 0.0
        K[fixed, fixed] = 1.0
        return K

    def load(self):
        """Consistent end loads of the s = s_max face."""
        e = torch.nonzero(self.ex == self.cfg["nx"] - 1).reshape(-1)
        pts = [(1.0, y, z, a * b) for z, b in _GAUSS for y, a in _GAUSS]
        N, dN = _shape(torch.tensor([p[:3] for p in pts], **_F8))
        X = self.xyz[self.conn[e]]
        x = torch.einsum("eai,qa->eqi", X, N)
        J = torch.einsum("eai,qaj->eqij", X, dN)
        n = torch.linalg.cross(J[..., 1], J[..., 2])
        dA = n.norm(dim=-1, keepdim=True)
        ld = self.cfg["load"]
        if ld["kind"] == "traction":
            t = torch.tensor(ld["t0"], **_F8) * dA
        else:
            amp, wl = self.cfg["wrinkle"]
            end = 0.25 * math.pi * (RADIUS + 0.5 * self.T) + self.cfg["limb"]
            mid = self.cfg["limb"] + RADIUS + 0.5 * self.T \
                + amp * math.exp(-(end / wl) ** 2) * math.cos(2 * math.pi * end / wl)
            t = -12 * ld["M"] / self.T ** 3 * (x[..., :1] - mid) * n
        w = torch.tensor([p[3] for p in pts], **_F8)
        f = torch.zeros(self.n // 3, 3, **_F8)
        f.index_add_(0, self.conn[e].reshape(-1),
                     torch.einsum("q,qa,eqi->eai", w, N, t).reshape(-1, 3))
        f[self.clamped] = 0.0
        return f.reshape(-1)

    def strength(self, u):
        """F at the Gauss points, the largest one with its stresses, and J of the arc."""
        resin = torch.tensor([L["mat"] == "resin" for L in self.cfg["layers"]],
                             device=u.device)[self.layer]
        F = torch.zeros(self.conn.shape[0], 27, **_F8)
        J, best, stress = 0.0, -1.0, None
        for e in self.chunks():
            S, Q, E, _, wd = self.local_stress(e, u)
            J += float((S[..., 2, 2] ** 2 * wd)[self.arc[e]].sum())
            R = E @ Q.transpose(-1, -2)
            S = R @ S @ R.transpose(-1, -2)
            f = torch.sqrt((S[..., 2, 2].clamp_min(0) / S33) ** 2 + (S[..., 0, 2] / S13) ** 2
                           + (S[..., 1, 2] / S13) ** 2) * resin[e][:, None]
            F[e] = f
            if float(f.max()) > best:
                best = float(f.max())
                s = S.reshape(-1, 3, 3)[int(f.argmax())]
                stress = torch.stack([s[0, 0], s[1, 1], s[2, 2], s[1, 2], s[0, 2], s[0, 1]])
        return {"J": np.array([J]), "F_max": np.array([best]), "elem": None, "gauss": None,
                "stress": stress.cpu().numpy(), "F_elem": F.max(1).values, "F_gauss": F.reshape(-1)}


def exact(case, seed):
    op = case["op"]
    if op == "band":
        n, _, mats, x = bands(case, seed)
        out, at = [], 0
        for a, nj in zip(mats, n.tolist()):
            b = a.shape[1] - 1
            full = torch.zeros(nj, nj, **_F8)
            for d in range(b + 1):
                full.diagonal(-d).copy_(a[d:, b - d])
            full = full + full.tril(-1).T
            m = nj * case["nrhs"]
            out.append(torch.linalg.solve(full.cpu(), x[at:at + m].view(nj, -1).cpu()).reshape(-1))
            at += m
        return torch.cat(out).cuda()
    if op in ("setup", "pcg", "sweep", "adjoint"):
        return None
    p = _Part(descriptor(case, seed))
    if op == "spmv":
        return p.apply(vector(p.n, seed))
    if op == "assemble":
        return {"f": p.load(), "Ku": p.apply(vector(p.n, seed))}
    if op == "stress":
        return p.strength(displacement(p.xyz, seed).reshape(-1))
    f = p.load()
    if p.n > 12000:                    # a dense solution would take too long
        return {"f": f, "x": None}
    return {"f": f, "x": torch.linalg.solve(p.dense().cpu(), f.cpu()).cuda()}
