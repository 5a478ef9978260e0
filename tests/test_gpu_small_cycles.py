"""Whole GMRES cycles of small systems in one launch.

Systems of at most 128 nodes run cycles of at most 58 columns in one workgroup; larger systems,
longer cycles and cycles whose launches are timed one by one take three launches a step.  Both form
every sum in the same order, so a solve with the timers on (every cycle by steps) and one with them
off give the same bits: iterates, steps, cycles and residuals, plain and deflated, in FP64 and mixed
precision, for solves that end at every place of a cycle.  Box meshes whose node counts lie at the
edges of the 64-node parts of a dot product, of the 88 rows of an SpMV pass and of the 128-node
limit, restart lengths around the 58-column limit.  The cavity's solves agree with scipy's direct
solve (bound of tests/test_gpu_deflate.py).
"""
import numpy as np
import pytest
import scipy.sparse.linalg as spla
import torch

from workloads import kuhn_box, jitter_interior, boundary_nodes, cavity_bc, cavity_mesh, apply_dirichlet
from tests.gpu_common import bsr_to_csr, make_context, random_state, to_dev

pytestmark = pytest.mark.gpu


def _box(B, cells, precision, max_restart):
    m = jitter_interior(kuhn_box(cells, (0, 0, 0), (1.0, 1.2, 1.4)), 0.2, 4)
    bnd = np.nonzero(boundary_nodes(m.tets, m.n_nodes))[0][::2]
    dofs = np.unique(np.concatenate([(4 * bnd[:, None] + np.arange(3)).ravel(), [3]]))
    u, _, beta, _ = random_state(m, 1)
    ctx = make_context(B, m, dofs, precision, max_restart=max_restart)
    A, rhs, _ = B.vms_condense_assemble(ctx, to_dev(u), to_dev(beta), 40.0)
    return ctx, A, rhs


def _solve(B, ctx, A, rhs, restart, k, steps, timed):
    x = ctx.new_vec()
    if timed:
        B.vms_profile(ctx, True)
    _, info = B.vms_gmres_solve(ctx, A, rhs, x, B.solve_opts(restart=restart, rtol=1e-12, max_iters=steps, deflate=k),
                                allow_noconv=True)
    if timed:
        B.vms_profile(ctx, False)
    return x, (info.iters, info.restarts, info.true_rel_res)


def _same(B, system, restart, k, steps):
    a, ia = _solve(B, *system, restart, k, steps, False)
    b, ib = _solve(B, *system, restart, k, steps, True)
    assert torch.isfinite(a).all() and torch.equal(a, b) and ia == ib, (restart, k, steps, ia, ib)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("cells", [(1, 1, 1), (2, 2, 6), (3, 3, 3), (1, 2, 10), (1, 6, 6), (1, 3, 10), (2, 4, 5), (3, 4, 5), (1, 10, 10),
                                   (4, 4, 4), (1, 7, 7), (3, 3, 7), (2, 2, 14), (2, 6, 6)])
def test_node_counts(vms_lib, cells, precision):
    system = _box(vms_lib, cells, precision, 50)
    for steps in (1, 2, 3, 9, 30, 31, 200):
        _same(vms_lib, system, 30, 0, steps)
    _same(vms_lib, system, 20, 6, 200)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("restart,k", [(1, 0), (2, 0), (15, 1), (57, 0), (58, 0), (59, 0), (58, 32), (59, 32), (34, 32),
                                       (64, 10)])
def test_cycle_lengths(vms_lib, restart, k, precision):
    system = _box(vms_lib, (4, 4, 4), precision, 64)
    for steps in (1, restart, restart + 1, 2 * restart + 5, 300):
        _same(vms_lib, system, restart, k, steps)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("k", [0, 8])
@pytest.mark.parametrize("n", [2, 4])
def test_against_a_direct_solve(vms_lib, n, k, precision):
    m = cavity_mesh(n)
    bc = cavity_bc(m)
    u = np.zeros((m.n_nodes, 4))
    apply_dirichlet(u, bc)
    ctx = make_context(vms_lib, m, bc.dofs, precision)
    A, rhs, _ = vms_lib.vms_condense_assemble(ctx, to_dev(u), to_dev(np.zeros((m.n_elems, 3))), 400.0)
    x = ctx.new_vec()
    rc, info = vms_lib.vms_gmres_solve(ctx, A, rhs, x, vms_lib.solve_opts(restart=25, rtol=1e-10, max_iters=20000,
                                                                          deflate=k))
    assert rc == vms_lib.VMS_OK and info.true_rel_res <= 1e-10
    xd = spla.spsolve(bsr_to_csr(ctx, A).tocsc(), rhs.cpu().numpy().ravel())
    assert np.linalg.norm(x.cpu().numpy().ravel() - xd) <= 1e-6 * np.linalg.norm(xd)
