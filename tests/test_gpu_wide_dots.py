"""The Gram-Schmidt dots of large meshes (131,072 nodes and more), which take two finished vectors a
workgroup and add their 64 partials per slot in a launch of its own (gpu).

A random system on a box's block pattern (no Dirichlet dofs, so plain block-Jacobi), at the smallest
box on the large side of the line and one just below it: the iterate after 1, 2, 3 and 8 steps (none,
an odd and an even number of finished vectors in the last step, more than one pair) against the
oracle's GMRES on the same stored matrix.  The system is well conditioned, so a step's rounding is
all that differs: FP64 sums over half a million entries, or FP32 vectors and preconditioner (6e-8 an
entry, a few steps).
"""
import numpy as np
import pytest
import torch

from oracle import vms as O
from workloads.mesh import kuhn_box
from tests.gpu_common import DEV, bsr_to_csr, make_context, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [(0, 1e-11), (1, 1e-5)])
@pytest.mark.parametrize("dims", [(50, 50, 49), (50, 50, 50)])
def test_iterates_after_a_few_steps(vms_lib, dims, precision, tol):
    B = vms_lib
    m = kuhn_box(dims, (0, 0, 0), (1, 1, 1), name="box")
    ctx = make_context(B, m, np.zeros(0, np.int32), precision)
    _, _, diagpos = ctx.bsr_pattern()
    rng = np.random.default_rng(precision)
    vals = 1.5 * rng.standard_normal((ctx.nb, 4, 4)) / np.sqrt(15.0)
    vals[diagpos] = 4.0 * np.eye(4) + 0.3 * rng.standard_normal((m.n_nodes, 4, 4))
    A = torch.from_numpy(vals.reshape(ctx.nb, 16)).to(DEV).to(ctx.dtype).contiguous()
    rhs = to_dev(rng.standard_normal((m.n_nodes, 4)))
    Am, b = bsr_to_csr(ctx, A), rhs.cpu().numpy().ravel()
    Minv = np.linalg.inv(A.double().cpu().numpy().reshape(-1, 4, 4)[diagpos])
    for steps in (1, 2, 3, 8):
        x = ctx.new_vec()
        _, info = B.vms_gmres_solve(ctx, A, rhs, x, B.solve_opts(restart=30, rtol=1e-14, max_iters=steps),
                                    allow_noconv=True)
        ref = O.gmres(Am, b, restart=30, max_iters=steps, rtol=1e-14, Minv_blocks=Minv)
        err = np.linalg.norm(x.cpu().numpy().ravel() - ref.x) / np.linalg.norm(ref.x)
        print(f"wide dots: {dims}, precision {precision}, {steps} steps: error {err:.2e}", flush=True)
        assert info.iters == steps and err <= tol
