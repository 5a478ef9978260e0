"""Set-up of a linear solve: preconditioner blocks, A P, A z and the coarse pressure mode (gpu).

Random systems on the block patterns of boxes and of fans (every tetrahedron shares one edge, whose two
nodes couple to all the others: rows of 7, 17, 42 and 202 blocks, around and beyond the blocks a
launch takes at a time), with pressures pinned on some nodes.  The iterate after a few steps against
the oracle's GMRES on A P, P = block-Jacobi + z z^T / (z^T A z), z = 1 on the free pressures (FP64
rounding, and FP32 vectors on a well-conditioned system); the network's features and the block
inverses of blocks that need pivoting, and of singular ones, against numpy's.
"""
import numpy as np
import pytest
import torch

from oracle import learned_pc as LP
from oracle import vms as O
from workloads import kuhn_box
from tests.gpu_common import DEV, bsr_to_csr, make_context, rel_fro, to_dev

pytestmark = pytest.mark.gpu


def _fan(k):
    class M:
        pass
    t = 2.0 * np.pi * np.arange(k) / k
    ring = np.stack([np.cos(t), np.sin(t), np.zeros(k)], 1)
    m = M()
    m.xyz = np.concatenate([[[0.0, 0.0, -1.0], [0.0, 0.0, 1.0]], ring])
    i = np.arange(k)
    m.tets = np.stack([np.zeros(k), np.ones(k), 2 + i, 2 + (i + 1) % k], 1).astype(np.int32)
    d = m.xyz[m.tets]
    if np.linalg.det(d[0, 1:] - d[0, 0]) < 0:
        m.tets = m.tets[:, [1, 0, 2, 3]]
    m.n_nodes, m.n_elems = k + 2, k
    return m


def _system(B, mesh, precision):
    m = _fan(mesh) if isinstance(mesh, int) else kuhn_box(mesh, (0, 0, 0), (1, 1, 1))
    pins = np.arange(1, m.n_nodes, 5)
    ctx = make_context(B, m, np.sort(4 * pins + 3), precision)
    _, _, diagpos = ctx.bsr_pattern()
    rng = np.random.default_rng(m.n_nodes)
    rowptr = ctx.bsr_pattern()[0]
    row = np.repeat(np.diff(rowptr), np.diff(rowptr))
    vals = rng.standard_normal((ctx.nb, 4, 4)) / np.sqrt(row)[:, None, None]
    vals[diagpos] = 4.0 * np.eye(4) + 0.3 * rng.standard_normal((m.n_nodes, 4, 4))
    A = torch.from_numpy(vals.reshape(ctx.nb, 16)).to(DEV).to(ctx.dtype).contiguous()
    return m, pins, ctx, diagpos, A, rng


@pytest.mark.parametrize("precision,tol", [(0, 1e-10), (1, 1e-4)])
@pytest.mark.parametrize("mesh", [5, 15, 40, 200, (1, 1, 1), (3, 4, 5), (6, 7, 8)])
def test_coarse_pressure_mode(vms_lib, mesh, precision, tol):
    B = vms_lib
    m, pins, ctx, diagpos, A, rng = _system(B, mesh, precision)
    b = rng.standard_normal((m.n_nodes, 4))
    Am = bsr_to_csr(ctx, A).toarray()
    z = np.zeros((m.n_nodes, 4))
    z[:, 3] = 1.0
    z[pins, 3] = 0.0
    z = z.ravel()
    P = np.outer(z, z) / (z @ Am @ z)
    for i, D in enumerate(np.linalg.inv(A.double().cpu().numpy().reshape(-1, 4, 4)[diagpos])):
        P[4 * i:4 * i + 4, 4 * i:4 * i + 4] += D
    for steps in (1, 3, 6):
        x = ctx.new_vec()
        B.vms_gmres_solve(ctx, A, to_dev(b), x, B.solve_opts(restart=30, rtol=1e-14, max_iters=steps),
                          allow_noconv=True)
        ref = P @ O.gmres(Am @ P, b.ravel(), restart=30, max_iters=steps, rtol=1e-14).x
        err = np.linalg.norm(x.cpu().numpy().ravel() - ref) / np.linalg.norm(ref)
        print(f"set-up: {mesh}, precision {precision}, {steps} steps: error {err:.2e}", flush=True)
        assert err <= tol


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("mesh", [5, 40, (1, 1, 1), (3, 4, 5)])
def test_blocks_that_need_pivoting(vms_lib, mesh, precision):
    B = vms_lib
    m, pins, ctx, diagpos, A, rng = _system(B, mesh, precision)
    D = rng.standard_normal((m.n_nodes, 4, 4))
    D[::2, 0, 0] = 1e-3                             # a small first pivot
    D[::3] = np.eye(4)[[3, 0, 1, 2]] + 0.05 * D[::3]
    A.view(-1, 4, 4)[torch.from_numpy(diagpos).long().to(DEV)] = torch.from_numpy(D).to(DEV).to(A.dtype)
    Ds = A.double().cpu().numpy().reshape(-1, 4, 4)[diagpos]
    P = B.vms_pc_blocks(ctx, A, None).cpu().numpy().reshape(-1, 4, 4)
    inv = np.linalg.inv(Ds)
    # backward stable elimination, result stored in FP32
    bound = 1e-6 + 1e-14 * np.linalg.cond(Ds)
    err = np.linalg.norm(P - inv, axis=(1, 2)) / np.linalg.norm(inv, axis=(1, 2))
    assert (err <= bound).all()
    x_o, _ = LP.features(bsr_to_csr(ctx, A), m.n_nodes, 4 * pins + 3)
    assert rel_fro(B.vms_pc_features(ctx, A).cpu().numpy(), x_o) <= 1e-5
    A.view(-1, 4, 4)[int(diagpos[0])] = 0.0         # singular: the identity instead
    P = B.vms_pc_blocks(ctx, A, None).cpu().numpy().reshape(-1, 4, 4)
    assert np.array_equal(P[0], np.eye(4)) and np.isfinite(P).all()
