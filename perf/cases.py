"""Performance cases: the calls a program makes into the library, over the sizes it makes them at.

A case is one call (or one fixed sequence of calls) through the entry points of
`paper_0809_4802_amd.binding` on one of the repository's synthetic workload families:

  family  mesh and physics                                          size parameters
  cavity  lid-driven unit cube, steady, one pinned pressure         n cells per side
  es      jittered cube, Ethier-Steinman flow, backward Euler       n cells per side
  bfs     backward-facing step, open outlet, backward Euler         cells per unit length
  jet     jet from an orifice in a wall, backward Euler             cells per unit length

Meshes and boundary conditions are shared between the seeds of a case; the state (velocity,
pressure, fine scales, previous velocity, body force), the Reynolds number and the vectors come
from the seed.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_0809_4802_amd import binding as B
import workloads as W

DEV = "cuda:0"


# ------------------------------------------------------------------------------- meshes, states
@functools.lru_cache(maxsize=12)
def _mesh(family, a, b, c):
    """(mesh, Dirichlet data at t = 0, number of 4x4 blocks) of a family at one size."""
    if family == "cavity":
        m = W.cavity_mesh(a)
        bc = W.cavity_bc(m)
    elif family == "es":
        m = W.jittered_cube(a, seed=0)
        bc = W.ethier_steinman_bc(m, 0.0, 0.002)
    elif family == "bfs":
        m = W.backward_facing_step(a, b, c)
        bc = W.bfs_bc(m)
    else:
        m = W.jet_box(a)
        bc = W.jet_bc(m)
    return m, bc, m.n_nodes + 2 * W.count_edges(m.tets, m.n_nodes)


def _mesh_of(case):
    return _mesh(case["family"], case["a"], case.get("b", 0), case.get("c", 0))


def _smooth(x, rng, comps, amp):
    """A smooth random field: a few Fourier modes per component."""
    out = np.zeros((x.shape[0], comps))
    for k in range(comps):
        for _ in range(4):
            f = rng.uniform(0.5, 3.0, 3)
            out[:, k] += rng.normal() * np.sin(math.pi * (x @ f) + rng.uniform(0, 2 * math.pi))
    return 0.5 * amp * out


def _state(case, seed):
    """Host inputs of a case: the state a Newton step of the workload starts from."""
    m, bc, _ = _mesh_of(case)
    rng = np.random.default_rng(seed)
    x = m.xyz / max(1.0, float(np.ptp(m.xyz[:, 1])))
    s = {"dt": 0.0, "u_prev": None, "body": None}
    if case["family"] == "es":
        # a later time step: the exact field at t, the boundary at t + dt
        s["Re"], s["dt"] = float(rng.uniform(800.0, 1200.0)), 0.01
        t, nu_l = float(rng.uniform(0.0, 0.1)), 2.0 / s["Re"]
        field = lambda at: np.concatenate([np.stack(W.es_velocity(*m.xyz.T, at, nu_l), axis=1),  # noqa: E731
                                           W.es_pressure(*m.xyz.T, at, nu_l)[:, None]], axis=1)
        prev = field(t)
        u = prev.copy()
        u.reshape(-1)[bc.dofs] = field(t + s["dt"]).reshape(-1)[bc.dofs]
    else:
        s["Re"] = float(rng.uniform(75.0, 125.0) if case["family"] == "cavity" else rng.uniform(600.0, 1000.0))
        u = np.concatenate([_smooth(x, rng, 3, 0.3), _smooth(x, rng, 1, 0.1)], axis=1)
        W.apply_dirichlet(u, bc)
        prev = u + np.concatenate([_smooth(x, rng, 3, 0.02), np.zeros((m.n_nodes, 1))], axis=1)
        if case["family"] != "cavity":
            s["dt"] = 0.05 if case["family"] == "bfs" else 0.01
    if case.get("Re"):
        s["Re"] = float(case["Re"])
    s["u"] = u
    s["beta"] = 1e-3 * rng.standard_normal((m.n_elems, 3))
    if s["dt"] > 0:
        s["u_prev"] = prev
    if case.get("body"):
        s["body"] = _smooth(x, rng, 3, 1.0)
    s["rng"] = rng
    return m, bc, s


def _dev(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


# ---------------------------------------------------------------------------------------- cases
def listed():
    return [
        # one Newton step of the smallest configuration, solved to the paper's linear tolerance:
        # a call whose time is launches and waits
        {"name": "newton_cavity4_fp64", "kind": "newton", "family": "cavity", "a": 4, "prec": "fp64", "Re": 1.0,
         "rtol": 1e-12, "deflate": 0, "det": False},
        # one Newton step of a transient in mixed precision on a reproducible context: assembly,
        # preconditioner, GMRES, recovery and the new residual in one call
        {"name": "newton_es24_mixed", "kind": "newton", "family": "es", "a": 24, "prec": "mixed", "rtol": 1e-4,
         "deflate": 10, "det": True},
        # the benchmark's assembly: condensed tangent and residual of the 32^3 cavity
        {"name": "assemble_cavity32_mixed", "kind": "assemble", "family": "cavity", "a": 32, "prec": "mixed",
         "det": False},
        # the largest cube, transient, FP64: 1.57 million tets
        {"name": "assemble_es64_fp64", "kind": "assemble", "family": "es", "a": 64, "prec": "fp64", "det": False},
        # the residual alone, with a body force, on a channel of uneven sizes (a line search or a
        # convergence check)
        {"name": "residual_bfs_fp64", "kind": "residual", "family": "bfs", "a": 4, "b": 7, "c": 5, "prec": "fp64",
         "body": True, "det": False},
        # raw element residuals and tangents, for a caller that assembles or checks them itself
        {"name": "tangents_es19_fp64", "kind": "tangents", "family": "es", "a": 19, "prec": "fp64", "det": False},
        # the block matrix times a vector, for a caller's own Krylov method
        {"name": "spmv_bfs_fp64", "kind": "spmv", "family": "bfs", "a": 5, "b": 9, "c": 7, "prec": "fp64",
         "det": False},
        # the linear solves: the 32^3 cavity in mixed precision with deflated restarts (the first
        # four cycles of such a solve), ...
        {"name": "gmres_cavity32_mixed", "kind": "gmres", "family": "cavity", "a": 32, "prec": "mixed", "deflate": 10,
         "steps": 170, "det": False},
        # ... the largest cube in mixed precision with plain restarts, ...
        {"name": "gmres_es64_mixed", "kind": "gmres", "family": "es", "a": 64, "prec": "mixed", "deflate": 0,
         "steps": 150, "det": False},
        # ... and a channel without a pressure pin in FP64 with deflated restarts
        {"name": "gmres_bfs_fp64", "kind": "gmres", "family": "bfs", "a": 4, "b": 5, "c": 5, "prec": "fp64",
         "deflate": 10, "steps": 170, "det": False},
        # one training step of the learned preconditioner correction (batch of 8 residuals)
        {"name": "train_cavity32_mixed", "kind": "train", "family": "cavity", "a": 32, "prec": "mixed", "batch": 8,
         "det": False},
        # the uncondensed system that Newton-Raphson assembles
        {"name": "full_cavity20_mixed", "kind": "full", "family": "cavity", "a": 20, "prec": "mixed", "det": False},
    ]


def _size(rng, family, lo, hi):
    """A family's size parameters with about n^3 cells, n log-uniform in [lo, hi]."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if family in ("cavity", "es"):
        return {"a": max(lo, min(hi, round(n)))}
    if family == "jet":
        return {"a": max(1, round(n / 4))}
    # about 260 cx cy cz cells, in uneven proportions
    k = (n ** 3 / 260.0) ** (1.0 / 3.0)
    return {"a": max(1, round(k * rng.uniform(0.7, 1.2))), "b": max(1, round(k * rng.uniform(0.8, 1.4))),
            "c": max(1, round(k * rng.uniform(0.8, 1.4)))}


def draw(rng):
    kind = rng.choice(["newton", "assemble", "assemble", "residual", "tangents", "spmv", "gmres", "gmres", "train",
                       "full"])
    prec = rng.choice(["fp64", "mixed"])
    family = rng.choice(["cavity", "es", "bfs", "jet"])
    case = {"kind": kind, "family": family, "prec": prec, "det": False}
    if kind == "newton":
        # transient steps; steady ones on small cavities in FP64 only
        if family == "cavity":
            case.update(a=rng.randint(3, 6), prec="fp64", Re=1.0, rtol=1e-12, deflate=0)
        else:
            case.update(family="es", a=_size(rng, "es", 8, 24)["a"], rtol=1e-4, deflate=rng.choice([0, 10]))
        case["det"] = rng.choice([False, True])
    elif kind in ("assemble", "residual", "spmv"):
        case.update(_size(rng, family, 5, 56))
        case["det"] = rng.choice([False, False, True])
        if kind != "spmv":
            case["body"] = rng.choice([False, False, True])
    elif kind in ("tangents", "full"):
        case.update(_size(rng, family, 5, 24))
    elif kind == "gmres":
        case.update(_size(rng, family, 5, 48))
        case["deflate"] = rng.choice([0, 10])
        case["steps"] = 170 if case["deflate"] else 150
    else:
        case.update(_size(rng, family, 5, 32))
        case["batch"] = rng.randint(1, 8)
    return case


# -------------------------------------------------------------------------------- prepare and run
def prepare(case, seed):
    m, bc, h = _state(case, seed)
    rng = h.pop("rng")
    kind = case["kind"]
    s = {"kind": kind, "case": case, "Re": h["Re"], "dt": h["dt"]}
    s["ctx"] = ctx = B.Context(_dev(m.xyz), _dev(m.tets), _dev(bc.dofs),
                               precision=B.VMS_FP64 if case["prec"] == "fp64" else B.VMS_MIXED,
                               full_system=kind == "full", deterministic=bool(case["det"]))
    for k in ("u", "beta", "u_prev", "body"):
        s[k] = _dev(h[k])
    if kind == "newton":
        s["u0"], s["beta0"] = s["u"].clone(), s["beta"].clone()
        s["lin"] = B.solve_opts(restart=50, rtol=case["rtol"], max_iters=20000, deflate=case["deflate"])
    elif kind in ("assemble", "full"):
        s["A"] = ctx.new_bsr() if kind == "assemble" else ctx.new_full_bsr()
        s["rhs"] = ctx.new_vec() if kind == "assemble" else ctx.new_full_vec()
        s["rn"] = torch.zeros(1, dtype=torch.float64, device=DEV)
    elif kind == "residual":
        s["r"], s["rn"] = ctx.new_vec(), torch.zeros(1, dtype=torch.float64, device=DEV)
    elif kind == "tangents":
        s["K"] = torch.empty((ctx.n_elems, 19, 19), dtype=torch.float64, device=DEV)
        s["R"] = torch.empty((ctx.n_elems, 19), dtype=torch.float64, device=DEV)
    else:
        s["A"], s["rhs"], _ = B.vms_condense_assemble(ctx, s["u"], s["beta"], h["Re"], h["dt"], s["u_prev"],
                                                      s["body"])
        if kind == "spmv":
            s["x"] = _dev(rng.standard_normal((m.n_nodes, 4))).to(ctx.dtype)
            s["y"] = torch.empty_like(s["x"])
        elif kind == "gmres":
            s["x"] = ctx.new_vec()
            s["lin"] = B.solve_opts(restart=50, rtol=1e-13, max_iters=case["steps"], deflate=case["deflate"])
        else:
            # residual samples, and weights some way into a training (the output layer is no
            # longer zero)
            s["r"] = _dev(rng.standard_normal((case["batch"], m.n_nodes, 4)).astype(np.float32) *
                          np.exp(_smooth(m.xyz, rng, 1, 1.0)).astype(np.float32)[None])
            lim = math.sqrt(6.0 / (B.PC_NIN + B.PC_NHID))
            w = 0.02 * rng.standard_normal(B.PC_NWEIGHTS)
            w[:B.PC_NHID * B.PC_NIN] = rng.uniform(-lim, lim, B.PC_NHID * B.PC_NIN)
            s["w"] = _dev(w.astype(np.float32))
            s["adam"] = torch.zeros((2, B.PC_NWEIGHTS), dtype=torch.float32, device=DEV)
            s["grad"] = torch.zeros(B.PC_NWEIGHTS, dtype=torch.float32, device=DEV)
            s["loss"] = torch.zeros(1, dtype=torch.float32, device=DEV)
            s["step"] = 0
    return s


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "newton":
        s["u"].copy_(s["u0"])
        s["beta"].copy_(s["beta0"])
        info = B.vms_newton_step(ctx, s["u"], s["beta"], s["Re"], s["dt"], s["u_prev"], s["body"], s["lin"])
        return {"u": s["u"], "beta": s["beta"], "rnorm_before": info.rnorm_before}
    if kind == "assemble":
        B.vms_condense_assemble(ctx, s["u"], s["beta"], s["Re"], s["dt"], s["u_prev"], s["body"], s["A"], s["rhs"],
                                s["rn"])
        return {"A": s["A"], "rhs": s["rhs"], "rnorm": s["rn"]}
    if kind == "full":
        B.vms_full_assemble(ctx, s["u"], s["beta"], s["Re"], s["dt"], s["u_prev"], s["body"], s["A"], s["rhs"],
                            s["rn"])
        return {"A": s["A"], "rhs": s["rhs"], "rnorm": s["rn"]}
    if kind == "residual":
        B.vms_residual(ctx, s["u"], s["beta"], s["Re"], s["dt"], s["u_prev"], s["body"], s["r"], s["rn"])
        return {"r": s["r"], "rnorm": s["rn"]}
    if kind == "tangents":
        B.vms_element_tangents(ctx, s["u"], s["beta"], s["Re"], s["dt"], s["u_prev"], s["body"], s["K"], s["R"])
        return {"K": s["K"], "R": s["R"]}
    if kind == "spmv":
        return B.vms_bsr_spmv(ctx, s["A"], s["x"], s["y"])
    if kind == "gmres":
        s["x"].zero_()
        B.vms_gmres_solve(ctx, s["A"], s["rhs"], s["x"], s["lin"], allow_noconv=True)
        return s["x"]
    s["step"] += 1
    B.vms_pc_train_step(ctx, s["A"], s["r"], s["w"], s["adam"], s["step"], 3e-4, s["grad"], s["loss"])
    return {"weights": s["w"], "adam": s["adam"], "grad": s["grad"], "loss": s["loss"]}


# ------------------------------------------------------------------------------------------ work
# operations of one element's condensed tangent and residual, shared terms once: about 1500 in
# FP64 (geometry, fields, residuals, K_ff^-1, K_cf K_ff^-1) and 2400 in the blocks
_ELEM_FLOPS, _RES_FLOPS = 3950.0, 800.0


def work(case):
    m, _, nb = _mesh_of(case)
    nn, ne, es = float(m.n_nodes), float(m.n_elems), 8.0 if case["prec"] == "fp64" else 4.0
    dt, body = case["family"] != "cavity", bool(case.get("body"))
    state = ne * 40.0 + nn * (56.0 + (24.0 if dt else 0.0) + (24.0 if body else 0.0))
    vec = 4.0 * nn * es
    spmv = nb * (16.0 * es + 4.0) + 4.0 * nn + 2.0 * vec
    assemble = {"bytes": state + nb * 16.0 * es + 32.0 * nn, "flops": _ELEM_FLOPS * ne}

    def krylov(steps, m_=50.0):
        # per step: the matrix, the basis so far and the new vector; the second pass of a vector
        # and the next one share a reading of the basis
        return {"bytes": steps * (spmv + (0.5 * m_ + 2.0) * vec), "flops": steps * (32.0 * nb + 8.0 * 0.5 * m_ * 4.0 * nn)}

    kind = case["kind"]
    if kind == "assemble":
        return assemble
    if kind == "residual":
        return {"bytes": state + 32.0 * nn, "flops": _RES_FLOPS * ne}
    if kind == "tangents":
        return {"bytes": state + ne * 380.0 * 8.0, "flops": _ELEM_FLOPS * ne}
    if kind == "spmv":
        return {"bytes": spmv, "flops": 32.0 * nb}
    if kind == "gmres":
        return krylov(case["steps"])
    if kind == "newton":
        k = krylov(250.0 if case["family"] == "cavity" else 60.0)
        return {"bytes": assemble["bytes"] + 2.0 * state + k["bytes"],
                "flops": assemble["flops"] + 2.0 * _RES_FLOPS * ne + k["flops"]}
    if kind == "train":
        # the matrix once for A P r and once for A^T e over the whole batch, the samples, the
        # network forward and backward per node
        b = float(case["batch"])
        return {"bytes": 2.0 * nb * (16.0 * es + 4.0) + b * nn * 16.0 + nn * 64.0,
                "flops": b * 64.0 * nb + nn * 3.0 * 2.0 * 2624.0}
    nbf, nr = nb + 9.0 * ne, nn + ne
    return {"bytes": state + nbf * 16.0 * es + 32.0 * nr, "flops": _ELEM_FLOPS * ne}


# ----------------------------------------------------------------------------- results in 64 bits
def _elements(m, s, dev):
    """Element residual [ne, 19] and tangent [ne, 19, 19] from the weak form integrated in closed
    form (linear tets, bubble 256 l0 l1 l2 l3, viscous coefficient 2 nu, backward Euler)."""
    T = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    tets = T(m.tets).long()
    nu, idt = 1.0 / s["Re"], (1.0 / s["dt"] if s["dt"] > 0 else 0.0)
    X, u = T(m.xyz)[tets], T(s["u"])[tets]
    J = (X[:, 1:] - X[:, :1]).transpose(1, 2)
    g3 = torch.linalg.inv(J)
    g = torch.cat([-g3.sum(1, keepdim=True), g3], 1)                    # [ne, 4, 3]
    vol = torch.linalg.det(J) / 6.0
    v, p, be = u[..., :3], u[..., 3], T(s["beta"])
    f = T(s["body"])[tets] if s["body"] is not None else torch.zeros_like(v)
    dv = v - T(s["u_prev"])[tets][..., :3] if s["dt"] > 0 else torch.zeros_like(v)
    c = lambda x: x[:, None]  # noqa: E731
    B1, Bb, C = 8 / 105 * vol, 32 / 105 * vol, 8192 / 51975 * vol
    Kb = 4096 / 945 * vol * (g * g).sum((1, 2))
    eye3, eye4 = torch.eye(3, dtype=X.dtype, device=dev), torch.eye(4, dtype=X.dtype, device=dev)
    M = vol[:, None, None] / 20 * (1 + eye4)                             # [ne, 4, 4]
    G = v.transpose(1, 2) @ g                                            # grad v: [ne, 3, 3]
    th = G.diagonal(dim1=1, dim2=2).sum(1)
    Wv = c(B1) * v.sum(1)
    V = M @ v
    gW, gb = (g * Wv[:, None]).sum(2), (g * be[:, None]).sum(2)          # [ne, 4]
    Gb = (G * be[:, None]).sum(2)
    Rc = V @ G.transpose(1, 2) + c(c(B1) * Gb) - (gW + c(th * B1) + 0.5 * c(C) * gb)[..., None] * c(be)
    Rc = Rc + 2 * nu * vol[:, None, None] * (g @ G.transpose(1, 2)) - (0.25 * vol * p.sum(1))[:, None, None] * g
    Rc = Rc - M @ f + idt * (M @ dv)
    Rp = -c(th * vol * 0.25) + c(Bb) * gb
    Rf = (G * Wv[:, None]).sum(2) + c(C) * (Gb - 0.5 * c(th) * be) + 2 * nu * c(Kb) * be
    Rf = Rf + c(Bb) * (p[..., None] * g).sum(1) - c(B1) * f.sum(1) + idt * c(B1) * dv.sum(1)
    R = torch.cat([torch.cat([Rc, Rp[..., None]], 2).reshape(-1, 16), Rf], 1)
    gT = g.transpose(1, 2)
    diag = V @ gT + idt * M + 2 * nu * vol[:, None, None] * (g @ gT) + (c(B1) * gb)[:, None, :]
    Kvv = diag[..., None, None] * eye3 + M[..., None, None] * G[:, None, None]
    Kvv = Kvv - B1[:, None, None, None, None] * be[:, None, None, :, None] * (g[:, :, None, None, :] + g[:, None, :, None, :])
    ne = X.shape[0]
    K = torch.zeros((ne, 19, 19), dtype=X.dtype, device=dev)
    Kc = torch.zeros((ne, 4, 4, 4, 4), dtype=X.dtype, device=dev)        # (a, r, b, c)
    Kc[:, :, :3, :, :3] = Kvv.permute(0, 1, 3, 2, 4)
    q = -0.25 * vol[:, None, None] * g
    Kc[:, :, :3, :, 3] = q[..., None]
    Kc[:, :, 3, :, :3] = q[:, None]
    K[:, :16, :16] = Kc.reshape(ne, 16, 16)
    Kcf = torch.zeros((ne, 4, 4, 3), dtype=X.dtype, device=dev)
    Kcf[:, :, :3] = (-(gW + c(th * B1)) - 0.5 * c(C) * gb)[..., None, None] * eye3 + (B1[:, None, None] * G)[:, None] \
        - 0.5 * C[:, None, None, None] * be[:, None, :, None] * g[:, :, None, :]
    Kcf[:, :, 3] = Bb[:, None, None] * g
    Kfc = torch.zeros((ne, 3, 4, 4), dtype=X.dtype, device=dev)
    dfc = gW + c(C) * gb + c(B1 * idt)
    Kfc[..., :3] = (dfc[..., None, None] * eye3 + (B1[:, None, None] * G)[:, None]
                    - 0.5 * C[:, None, None, None] * be[:, None, :, None] * g[:, :, None, :]).permute(0, 2, 1, 3)
    Kfc[..., 3] = Bb[:, None, None] * gT
    K[:, :16, 16:] = Kcf.reshape(ne, 16, 3)
    K[:, 16:, :16] = Kfc.reshape(ne, 3, 16)
    K[:, 16:, 16:] = C[:, None, None] * (G - 0.5 * th[:, None, None] * eye3) + (2 * nu * Kb)[:, None, None] * eye3
    return R, K


def _condensed(R, K):
    Wm = torch.linalg.solve(K[:, 16:, 16:], torch.cat([K[:, 16:, :16], R[:, 16:, None]], 2))
    S = torch.cat([K[:, :16, :16], R[:, :16, None]], 2) - K[:, :16, 16:] @ Wm
    return S[..., :16], S[..., 16]


def _free(m, bc, n_rows, dev):
    free = torch.ones((n_rows, 4), dtype=torch.float64, device=dev)
    free.view(-1)[torch.from_numpy(bc.dofs.astype(np.int64)).to(dev)] = 0.0
    free[m.n_nodes:, 3] = 0.0
    return free


def _blocks(keys, vals, free, n_rows):
    """Blocks (keys = row n_rows + column) summed and sorted, fixed dofs made the identity."""
    uniq, inv = torch.unique(keys, return_inverse=True)
    A = torch.zeros((uniq.numel(), 4, 4), dtype=torch.float64, device=vals.device).index_add_(0, inv, vals)
    i, j = uniq // n_rows, uniq % n_rows
    A = A * free[i][:, :, None] * free[j][:, None, :]
    d = torch.nonzero(i == j)[:, 0]
    A[d] += torch.diag_embed(1.0 - free[i[d]])
    return A.reshape(-1, 16), i, j


def _assembled(m, bc, s, dev):
    """Condensed block matrix, rhs and residual norm."""
    R, K = _elements(m, s, dev)
    tets, nn = torch.from_numpy(m.tets).to(dev).long(), m.n_nodes
    free = _free(m, bc, nn, dev)
    rg = torch.zeros((nn, 4), dtype=torch.float64, device=dev).index_add_(0, tets.reshape(-1), R[:, :16].reshape(-1, 4))
    rnorm = torch.sqrt((rg * free).square().sum() + R[:, 16:].square().sum())
    S, r = _condensed(R, K)
    del K
    rhs = -torch.zeros((nn, 4), dtype=torch.float64, device=dev).index_add_(0, tets.reshape(-1), r.reshape(-1, 4)) * free
    keys = (tets[:, :, None] * nn + tets[:, None, :]).reshape(-1)
    S = S.reshape(-1, 4, 4, 4, 4).permute(0, 1, 3, 2, 4).reshape(-1, 4, 4)
    A, i, j = _blocks(keys, S, free, nn)
    return A, i, j, rhs, rnorm, free


def _exact_train(s, A, i, j, free, w0):
    """One step of the preconditioner's training from zero Adam state, by autograd."""
    n = free.shape[0]
    r = s["r"].double()
    A4 = A.reshape(-1, 4, 4)
    dg = torch.nonzero(i == j)[:, 0]
    D = A4[dg]
    off = torch.zeros((n, 4), dtype=torch.float64, device=A.device).index_add_(0, i, A4.abs().sum(2)) - D.abs().sum(2)
    fro = D.square().sum((1, 2)).sqrt()
    x = torch.cat([(D / fro[:, None, None]).reshape(n, 16), fro.log()[:, None],
                   torch.log1p(off / D.diagonal(dim1=1, dim2=2).abs()), 1.0 - free], 1)
    w = w0.double().requires_grad_(True)
    nh, ni, no = B.PC_NHID, B.PC_NIN, B.PC_NOUT
    W1, b1, W2, b2 = torch.split(w, [nh * ni, nh, no * nh, no])
    y = torch.tanh(x @ W1.reshape(nh, ni).T + b1) @ W2.reshape(no, nh).T + b2
    Mi = torch.eye(4, dtype=torch.float64, device=A.device) + y.reshape(n, 4, 4) * free[:, :, None] * free[:, None, :]
    P = torch.linalg.inv(D) @ Mi
    loss = 0.0
    for b in range(r.shape[0]):
        t = (P @ r[b][:, :, None])[..., 0]
        e = r[b] - torch.zeros_like(t).index_add(0, i, (A4 @ t[j][:, :, None])[..., 0])
        loss = loss + e.square().sum() / r[b].square().sum() / r.shape[0]
    grad, = torch.autograd.grad(loss, w)
    mom, var = 0.1 * grad, 0.001 * grad.square()
    wn = w.detach() - 3e-4 * (mom / 0.1) / ((var / 0.001).sqrt() + 1e-8)
    return {"weights": wn, "adam": torch.stack([mom, var]), "grad": grad, "loss": loss.detach().reshape(1)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "gmres" or (kind == "newton" and case["a"] > 8):
        return None          # iterates of a solve that is stopped early, or too large to factor
    dev = DEV if torch.cuda.is_available() else "cpu"
    m, bc, s = _state(case, seed)
    if m.n_elems > 700000:
        return None          # the element matrices alone are gigabytes
    if kind == "tangents":
        R, K = _elements(m, s, dev)
        return {"K": K, "R": R}
    if kind == "residual":
        R, _ = _elements(m, s, dev)
        free = _free(m, bc, m.n_nodes, dev)
        tets = torch.from_numpy(m.tets).to(dev).long()
        r = free * torch.zeros_like(free).index_add_(0, tets.reshape(-1), R[:, :16].reshape(-1, 4))
        return {"r": r, "rnorm": torch.sqrt(r.square().sum() + R[:, 16:].square().sum()).reshape(1)}
    if kind == "full":
        R, K = _elements(m, s, dev)
        tets, nn, ne = torch.from_numpy(m.tets).to(dev).long(), m.n_nodes, m.n_elems
        nr = nn + ne
        free = _free(m, bc, nr, dev)
        el = torch.cat([tets, torch.arange(nn, nr, device=dev)[:, None]], 1)
        Kp = torch.zeros((ne, 20, 20), dtype=torch.float64, device=dev)
        Kp[:, :19, :19] = K
        Rp = torch.zeros((ne, 20), dtype=torch.float64, device=dev)
        Rp[:, :19] = R
        rg = free * torch.zeros_like(free).index_add_(0, el.reshape(-1), Rp.reshape(-1, 4))
        keys = (el[:, :, None] * nr + el[:, None, :]).reshape(-1)
        A, _, _ = _blocks(keys, Kp.reshape(-1, 5, 4, 5, 4).permute(0, 1, 3, 2, 4).reshape(-1, 4, 4), free, nr)
        return {"A": A, "rhs": -rg, "rnorm": rg.norm().reshape(1)}
    A, i, j, rhs, rnorm, free = _assembled(m, bc, s, dev)
    if kind == "assemble":
        return {"A": A, "rhs": rhs, "rnorm": rnorm.reshape(1)}
    if kind == "newton":
        n = m.n_nodes
        D = torch.zeros((n, n, 4, 4), dtype=torch.float64, device=dev)
        D[i, j] = A.reshape(-1, 4, 4)
        du = torch.linalg.solve(D.permute(0, 2, 1, 3).reshape(4 * n, 4 * n).cpu(), rhs.reshape(-1).cpu())
        du = du.reshape(n, 4).to(dev)
        R, K = _elements(m, s, dev)
        de = du[torch.from_numpy(m.tets).to(dev).long()].reshape(-1, 16, 1)
        db = torch.linalg.solve(K[:, 16:, 16:], -R[:, 16:, None] - K[:, 16:, :16] @ de)[..., 0]
        return {"u": torch.from_numpy(s["u"]).to(dev) + du, "beta": torch.from_numpy(s["beta"]).to(dev) + db,
                "rnorm_before": float(rnorm)}
    # the remaining kinds multiply by the matrix as it is stored
    if case["prec"] == "mixed":
        A = A.float().double()
    if kind == "spmv":
        x = torch.from_numpy(s["rng"].standard_normal((m.n_nodes, 4))).to(dev)
        if case["prec"] == "mixed":
            x = x.float().double()
        return torch.zeros_like(x).index_add_(0, i, (A.reshape(-1, 4, 4) @ x[j][:, :, None])[..., 0])
    t = prepare(case, seed)
    return _exact_train(t, A, i, j, free, t["w"])
