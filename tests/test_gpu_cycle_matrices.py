"""Recorded cycles and the caller's matrix: a mixed context with an FP64 basis multiplies by the matrix
that each solve is given.  Two matrices in buffers of their own, solved in turn on one context by full
restart cycles, plain and deflated, give what a context of each one's own gives, bit for bit (the solve
adds in a fixed order), and a residual within rtol of the FP32-stored matrix, formed on the host."""
import numpy as np
import pytest
import torch

from workloads import cavity_mesh, cavity_bc, apply_dirichlet
from tests.gpu_common import bsr_to_csr, make_context, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("restart,k", [(20, 0), (20, 5), (50, 10)])
def test_matrices_in_turn(vms_lib, restart, k):
    B = vms_lib
    m = cavity_mesh(6)
    bc = cavity_bc(m)
    u = np.zeros((m.n_nodes, 4))
    apply_dirichlet(u, bc)
    beta = to_dev(np.zeros((m.n_elems, 3)))
    rtol = 1e-10

    def context():
        return make_context(B, m, bc.dofs, B.VMS_MIXED, basis_fp64=True)

    def solve(ctx, A, rhs):
        x = ctx.new_vec()
        rc, info = B.vms_gmres_solve(ctx, A, rhs, x, B.solve_opts(restart=restart, rtol=rtol, max_iters=20000, deflate=k,
                                                                  basis_fp64=1))
        assert rc == B.VMS_OK and info.restarts > 2          # full cycles among them
        return x, info.iters

    ctx = context()
    systems = [B.vms_condense_assemble(ctx, to_dev(scale * u), beta, Re)[:2] for Re, scale in ((100.0, 1.0), (10.0, 0.5))]
    alone = [solve(context(), A, rhs) for A, rhs in systems]
    for i in (0, 1, 0, 1, 1, 0):
        A, rhs = systems[i]
        x, iters = solve(ctx, A, rhs)
        b = rhs.cpu().numpy().ravel()
        rel = np.linalg.norm(b - bsr_to_csr(ctx, A) @ x.cpu().numpy().ravel()) / np.linalg.norm(b)
        print(f"matrix {i}, restart {restart}, kept {k}: {iters} steps, residual {rel:.2e}", flush=True)
        assert rel <= 1.01 * rtol
        assert iters == alone[i][1] and torch.equal(x, alone[i][0])
