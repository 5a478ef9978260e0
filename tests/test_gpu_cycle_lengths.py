"""Deflated cycles of every back-substitution form (gpu): one wave to 64 columns, staged beyond.

The backward-facing step's system of tests/test_gpu_deflate.py (plain block-Jacobi, FP64), restart
lengths on both sides of 64 and the longest, few and as many kept vectors as the library takes: steps and
cycles of the oracle's GMRES-DR within the bounds of that file (the larger of 3 steps and 1%, one
cycle), its iterate to 1e-7; without deflation the textbook GMRES's.
"""
import numpy as np
import pytest

from oracle import vms as O
from oracle.gmres_dr import gmres_dr

from workloads import backward_facing_step, bfs_bc, apply_dirichlet
from tests.gpu_common import bsr_to_csr, make_context, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def system(vms_lib):
    B = vms_lib
    m = backward_facing_step(1, 2, 1)
    bc = bfs_bc(m)
    u = np.zeros((m.n_nodes, 4))
    apply_dirichlet(u, bc)
    ctx = make_context(B, m, bc.dofs, B.VMS_FP64, max_restart=128)
    A, rhs, _ = B.vms_condense_assemble(ctx, to_dev(u), to_dev(np.zeros((m.n_elems, 3))), 50.0)
    Am = bsr_to_csr(ctx, A)
    return ctx, A, rhs, Am, O.block_jacobi_inverse(Am, m.n_nodes)


@pytest.mark.parametrize("restart,k", [(63, 0), (64, 0), (65, 0), (128, 0), (64, 1), (64, 32), (65, 1), (65, 32),
                                       (128, 32)])
def test_steps_and_iterate(vms_lib, system, restart, k):
    B = vms_lib
    ctx, A, rhs, Am, Minv = system
    b = rhs.cpu().numpy().ravel()
    x = ctx.new_vec()
    _, info = B.vms_gmres_solve(ctx, A, rhs, x, B.solve_opts(restart=restart, rtol=1e-10, max_iters=20000, deflate=k))
    solve = gmres_dr if k else O.gmres
    ref = solve(Am, b, restart=restart, max_iters=20000, rtol=1e-10, Minv_blocks=Minv, **({"k": k} if k else {}))
    err = np.linalg.norm(x.cpu().numpy().ravel() - ref.x) / np.linalg.norm(ref.x)
    print(f"cycle lengths: restart {restart}, k {k}: steps {info.iters} / {ref.iters}, cycles {info.restarts} / "
          f"{ref.restarts}, error {err:.1e}", flush=True)
    assert abs(info.iters - ref.iters) <= max(3, 0.01 * ref.iters)
    assert abs(info.restarts - ref.restarts) <= 1
    assert err <= 1e-7
