"""Timed cases of the library: what a FETI program has it do, call by call.

A program plans a batch of subdomains once (`Plan`), gives it the values of
the regularised stiffness matrices (`factor`, or `preprocess` with the
assembly in one go), assembles the dual operators F_i on the GPU
(`assemble`), and then applies them to dual vectors, alone (`apply`,
`apply_implicit`) or inside the projected CG (`pcpg`).  F_i stays in the plan
and is read through those calls; a program that wants the matrices themselves
takes them out with `get_F_device`.  The operations of a case:

  assemble    assemble the batch, then q = F p
  export      assemble the batch, then every F_i as a dense device matrix
  pcpg        assemble the batch, then `iters` projected CG iterations
  apply       q = F p with F assembled before
  implicit    q = F p with the factors, nothing assembled
  preprocess  host factorisation and assembly from new stiffness values, q = F p

Subdomains come from the repository's generator: boxes of Q1 / hex8 elements
(heat, elasticity) and the P1 triangle / tetrahedron meshes.  A seed draws the
gluing signs, one material coefficient (a power of two) per subdomain and the
dual vectors; sizes belong to the case.

A mixed-precision plan stores F in 32 bits; what such a program hands on, the
matrices and their products, is returned in that type.  The projected CG runs
on FP64 plans and for its first iterations, each of which costs the same: a
relative perturbation of F is multiplied by about 50 in ten iterations and by
up to 1e9 in 25 (F is huge along the projected-out rigid modes).
"""
import random
from functools import lru_cache

import numpy as np
import torch

import scgen
from paper_2509_21037_amd import scasm

# kind: mesh and physics; ex, ey, ez: elements per axis; spread: every axis of
# every subdomain is drawn from [e - spread, e + spread] (stream `shapes`);
# count: subdomains in the batch; gluing: "unique" (each surface DOF once) or
# "per_face" (edge and corner DOFs once per face); split, panel: factor blocks
# (0 = the library's width).
_DEFAULTS = dict(ey=0, ez=0, spread=0, shapes=1, gluing="unique", precision="fp64", split="etree", panel=0, iters=0)


def _case(name, op, kind, ex, ey, ez, count, **kw):
    return dict(_DEFAULTS, name=name, op=op, kind=kind, ex=ex, ey=ey, ez=ez, count=count, **kw)


def listed():
    return [
        # one small 2D subdomain, the smallest call: launches and latency
        _case("heat2d_single", "assemble", "heat", 16, 16, 0, 1, split="uniform"),
        # many small equal 3D subdomains, the usual cut of a heat problem, in
        # both precisions
        _case("heat3d_fp64", "assemble", "heat", 12, 12, 12, 512, panel=48),
        _case("heat3d_mixed", "assemble", "heat", 12, 12, 12, 512, panel=48, precision="mixed"),
        # an uneven decomposition of an elastic body (6..16 elements an axis):
        # ragged sizes side by side in one batch, library defaults
        _case("elast_uneven_fp64", "assemble", "elasticity", 11, 11, 11, 64, spread=5, split="uniform"),
        # the same kind of batch taken to a solution
        _case("elast_uneven_pcpg", "pcpg", "elasticity", 11, 11, 11, 64, spread=5, iters=10),
        # large elastic subdomains glued face by face, in both precisions
        _case("elast_large_fp64", "assemble", "elasticity", 20, 20, 20, 16, gluing="per_face"),
        _case("elast_large_mixed", "assemble", "elasticity", 20, 20, 20, 16, gluing="per_face", precision="mixed"),
        # 2D triangles: large sparse factors, few multipliers
        _case("tri2d_fp64", "assemble", "tri", 128, 0, 0, 128),
        # tetrahedra, the dense F_i handed over to the program
        _case("tet3d_export", "export", "tet", 13, 0, 0, 32),
        # the iteration phase on large subdomains: F read, or the factors read
        _case("elast_large_apply", "apply", "elasticity", 20, 20, 20, 16, gluing="per_face"),
        _case("elast_large_implicit", "implicit", "elasticity", 20, 20, 20, 16, gluing="per_face"),
        # a time step with new coefficients: host factorisation and assembly
        _case("elast_uneven_preprocess", "preprocess", "elasticity", 11, 11, 11, 64, spread=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng: random.Random):
    """One more case: any operation on any mesh, sizes over the listed range.
    A batch holds at most about the unknowns of the large listed ones."""
    op = rng.choice(["assemble", "assemble", "assemble", "export", "pcpg", "apply", "implicit", "preprocess"])
    kind = rng.choice(["heat", "elasticity"] if op == "pcpg" else ["heat", "heat", "elasticity", "elasticity", "tri", "tet"])
    c = dict(_DEFAULTS, op=op, kind=kind, precision=rng.choice(["fp64", "mixed"]),
             split=rng.choice(["etree", "etree", "uniform"]), panel=rng.choice([0, 0, 32, 48]),
             gluing=rng.choice(["unique", "unique", "per_face"]), shapes=rng.randrange(1, 1 << 20),
             iters=rng.randrange(4, 11) if op == "pcpg" else 0)
    if kind == "tri":
        c["ex"], dofs, cap = _log_int(rng, 16, 128), 1, 1_200_000
        nodes = (c["ex"] + 1) ** 2
    elif kind == "tet":
        c["ex"], dofs, cap = _log_int(rng, 4, 20), 1, 280_000
        nodes = (c["ex"] + 1) ** 3
    else:
        dofs, top, cap = (1, 14, 800_000) if kind == "heat" else (3, 16, 240_000)
        if kind == "heat" and op != "pcpg" and rng.random() < 0.25:
            c["ex"], c["ey"] = _log_int(rng, 6, 64), _log_int(rng, 6, 64)
            nodes = (c["ex"] + 1) * (c["ey"] + 1)
        else:
            c["ex"], c["ey"], c["ez"] = (rng.randrange(5, top + 1) for _ in range(3))
            c["spread"] = rng.choice([0, 0, 1, 2])
            nodes = (c["ex"] + 1) * (c["ey"] + 1) * (c["ez"] + 1)
    most = max(1, min(512, cap // (nodes * dofs)))
    if op == "pcpg":         # repeated DOFs make F singular: no solution for any d
        c["gluing"] = "unique"
    if op in ("pcpg", "implicit"):    # FP64 vectors, and factors read in FP64
        c["precision"] = "fp64"
    if op == "export":       # dense matrices: bounded by their elements
        m = max(_mesh(c, sh, 1).dof.shape[0] for sh in _shapes(dict(c, count=8)))
        most = max(1, min(most, 48, 30_000_000 // (m * m)))
    c["count"] = _log_int(rng, 1, most)
    return c


# ------------------------------------------------------------------ inputs
def _shapes(case):
    """Elements per axis of every subdomain."""
    e = [case[k] for k in ("ex", "ey", "ez") if case[k] > 0]
    if not case["spread"]:
        return [tuple(e)] * case["count"]
    s = case["spread"]
    rng = np.random.default_rng(case["shapes"])
    return [tuple(int(v) + int(rng.integers(-s, s + 1)) for v in e) for _ in range(case["count"])]


def _mesh(case, shape, seed):
    if case["kind"] in ("tri", "tet"):
        return scgen.simplex_subdomain(2 if case["kind"] == "tri" else 3, shape[0], seed)
    return scgen.box_subdomain(case["kind"], shape, 1.0 / max(shape), seed, gluing=case["gluing"])


class _Sub:
    """One subdomain: the mesh's pattern, its values times a coefficient."""

    def __init__(self, mesh, exponent):
        for k in ("n", "rowptr", "col", "dof", "sign", "coords", "dofs_per_node", "R"):
            setattr(self, k, getattr(mesh, k))
        self.unit_val, self.exponent = mesh.val, exponent
        self.val = np.ldexp(mesh.val, exponent)


def _inputs(case, seed):
    """(subdomains, dual vector in [-1, 1))."""
    rng = np.random.default_rng(seed)
    base = int(rng.integers(1, 1 << 62))
    exps = rng.integers(-3, 4, size=case["count"])
    subs = [_Sub(_mesh(case, sh, base + i), int(exps[i])) for i, sh in enumerate(_shapes(case))]
    return subs, rng.uniform(-1.0, 1.0, size=sum(s.dof.shape[0] for s in subs))


def prepare(case, seed):
    subs, p = _inputs(case, seed)
    plan = scasm.Plan(subs, precision=case["precision"], block_split=case["split"], panel_width=case["panel"])
    st = {"op": case["op"], "mixed": case["precision"] == "mixed", "plan": plan, "iters": case["iters"]}
    st["p"] = torch.from_numpy(p).cuda()
    st["q"] = torch.zeros_like(st["p"])
    if case["op"] == "preprocess":
        st["kvals"] = [s.val for s in subs]
    else:
        plan.factor()
    if case["op"] == "apply":
        plan.assemble()
    if case["op"] == "export":
        st["F"] = [torch.zeros(s.dof.shape[0] ** 2, dtype=torch.float64, device="cuda") for s in subs]
    return st


def run(state):
    plan, p, q, op, mixed = state["plan"], state["p"], state["q"], state["op"], state["mixed"]
    if op == "implicit":
        return plan.apply_implicit(p, q)
    if op == "preprocess":
        plan.preprocess(state["kvals"])
    elif op != "apply":
        plan.assemble()
    if op == "export":
        F = [plan.get_F_device(i, out=f) for i, f in enumerate(state["F"])]
        return [f.float() for f in F] if mixed else F
    if op == "pcpg":
        plan.pcpg(p, q, state["iters"])
        return q
    plan.apply(p, q)
    return q.float() if mixed else q


# -------------------------------------------------------------------- work
@lru_cache(maxsize=None)
def _counts(kind, shape, gluing, split, panel):
    """(n, m, factor nonzeros, assembly flops on nonzero rows, factor flops)
    of one subdomain; the flops of the paper's count, restricted to the rows
    of L^{-1} B^T that can be nonzero."""
    mesh = _mesh(dict(kind=kind, gluing=gluing), shape, 1)
    a = scasm.host_analyze(mesh, values=False, block_split=split, panel_width=panel)
    return int(mesh.n), int(mesh.dof.shape[0]), int(a["nnzL"]), a["trsm_reach"] + a["syrk_reach"], a["factor_flops"]


def work(case):
    elem = 8 if case["precision"] == "fp64" else 4        # stored F
    by = fl = 0.0
    for sh in _shapes(case):
        n, m, nnz, asm, fac = _counts(case["kind"], sh, case["gluing"], case["split"], case["panel"])
        sym = m * (m + 1) / 2                              # F is symmetric
        op = case["op"]
        if op == "apply":
            by += elem * sym + 16 * m
            fl += 2.0 * m * m
        elif op == "implicit":
            by += 8 * nnz + 16 * m
            fl += 4.0 * nnz
        else:
            by += 8 * nnz + elem * sym                     # factor read, F written
            fl += asm
            if op == "preprocess":
                fl += fac
            if op == "export":
                by += 8.0 * m * m
            else:
                times = case["iters"] if op == "pcpg" else 1
                by += times * elem * sym + 16 * m
                fl += times * 2.0 * m * m
    return {"bytes": by, "flops": fl}


# ------------------------------------------------------------------- exact
class _Dense:
    """K^{-1} of one mesh by a dense Cholesky factorisation in torch, with
    residuals in extended precision."""

    def __init__(self, sub):
        self.n, self.rowptr, self.col, self.val = sub.n, sub.rowptr, sub.col, sub.unit_val
        self.rows = np.repeat(np.arange(self.n), np.diff(self.rowptr))
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        K = torch.zeros(self.n, self.n, dtype=torch.float64, device=dev)
        K[torch.from_numpy(self.rows).to(dev), torch.from_numpy(self.col.astype(np.int64)).to(dev)] = \
            torch.from_numpy(np.array(self.val)).to(dev)
        self.L = torch.linalg.cholesky(K)

    def raw(self, b):
        """n x k torch tensor -> K^{-1} b in 64 bits."""
        return torch.cholesky_solve(b, self.L)

    def solve(self, b, steps):
        x = self.raw(torch.from_numpy(b).to(self.L.device)).cpu().numpy().astype(np.longdouble)
        v = self.val.astype(np.longdouble)
        for _ in range(steps):
            r = np.empty_like(b)
            for k in range(b.shape[1]):
                r[:, k] = (b[:, k] - np.add.reduceat(v * x[self.col, k], self.rowptr[:-1])).astype(np.float64)
            x += self.raw(torch.from_numpy(r).to(self.L.device)).cpu().numpy()
        return x


def _pcpg(apply_F, G, d, iters):
    def project(r):
        return r - G @ torch.linalg.solve(G.T @ G, G.T @ r) if G.shape[1] else r
    lam, r = torch.zeros_like(d), d.clone()
    w = project(r)
    p, ww = w.clone(), w @ w
    for _ in range(iters):
        q = apply_F(p)
        pq = p @ q
        if not (pq > 0 and ww > 0):
            break
        lam += (ww / pq) * p
        r -= (ww / pq) * q
        w = project(r)
        new = w @ w
        p, ww = w + (new / ww) * p, new
    return lam


def exact(case, seed):
    subs, p = _inputs(case, seed)
    off = np.concatenate([[0], np.cumsum([s.dof.shape[0] for s in subs])])
    same = {}
    for i, sh in enumerate(_shapes(case)):
        same.setdefault(sh, []).append(i)
    out = np.zeros(off[-1])
    mats = [None] * len(subs)
    for idx in same.values():
        s0 = subs[idx[0]]
        D = _Dense(s0)
        m = s0.dof.shape[0]
        if case["op"] == "export":
            E = np.zeros((s0.n, m))
            E[s0.dof, np.arange(m)] = 1.0
            F = D.solve(E, 1)[s0.dof, :].astype(np.float64)
            for i in idx:
                g = subs[i].sign.astype(np.float64)
                mats[i] = torch.from_numpy(np.ldexp(g[:, None] * F * g[None, :], -subs[i].exponent))
        elif case["op"] == "pcpg":
            dev = D.L.device
            dof = torch.from_numpy(s0.dof.astype(np.int64)).to(dev)
            E = torch.zeros(s0.n, m, dtype=torch.float64, device=dev)
            E[dof, torch.arange(m, device=dev)] = 1.0
            F = D.raw(E)[dof]
            for i in idx:
                g = torch.from_numpy(subs[i].sign.astype(np.float64)).to(dev)

                def apply_F(v):
                    return g * (F @ (g * v)) * 2.0 ** -subs[i].exponent

                G = g[:, None] * torch.from_numpy(np.array(s0.R)).to(dev)[dof]
                out[off[i]:off[i + 1]] = _pcpg(apply_F, G, torch.from_numpy(p[off[i]:off[i + 1]]).to(dev),
                                               case["iters"]).cpu().numpy()
        else:
            b = np.zeros((s0.n, len(idx)))
            for k, i in enumerate(idx):
                np.add.at(b[:, k], s0.dof, subs[i].sign * p[off[i]:off[i + 1]])
            x = D.solve(b, 2)
            for k, i in enumerate(idx):
                out[off[i]:off[i + 1]] = np.ldexp((subs[i].sign * x[s0.dof, k]).astype(np.float64), -subs[i].exponent)
    return mats if case["op"] == "export" else torch.from_numpy(out)
