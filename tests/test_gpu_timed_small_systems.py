"""Phase timers on small systems: a cycle that ends before the restart length is launched step by step
while the timers are on, and every every-th launch of a phase is timed, whatever the system's size
(27 nodes, where a cycle is one launch otherwise; 343 nodes, where it never is).  Full cycles are
sampled whole.  The launches that vms_profile_read counts, for solves that end on their step count."""
import numpy as np
import pytest

from workloads import cavity_mesh, cavity_bc, apply_dirichlet
from tests.gpu_common import make_context, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 6])
@pytest.mark.parametrize("precision", [0, 1])
def test_sampled_launches(vms_lib, n, precision):
    B = vms_lib
    m = cavity_mesh(n)
    bc = cavity_bc(m)
    u = np.zeros((m.n_nodes, 4))
    apply_dirichlet(u, bc)
    ctx = make_context(B, m, bc.dofs, precision)
    A, rhs, _ = B.vms_condense_assemble(ctx, to_dev(u), to_dev(np.zeros((m.n_elems, 3))), 400.0)

    def launches(every, restart, steps, solves):
        B.vms_profile(ctx, True, ["spmv", "dots", "update"], every)
        for _ in range(solves):
            _, info = B.vms_gmres_solve(ctx, A, rhs, ctx.new_vec(),
                                        B.solve_opts(restart=restart, rtol=1e-14, max_iters=steps), allow_noconv=True)
            assert info.iters == steps
        got = B.vms_profile_read(ctx)
        B.vms_profile(ctx, False)
        return [got[p][1] for p in ("spmv", "dots", "update")]

    assert launches(1, 20, 3, 4) == [12] * 3
    assert launches(2, 20, 3, 4) == [6] * 3          # partial cycles: every second launch
    assert launches(3, 20, 3, 4) == [4] * 3
    assert launches(2, 3, 3, 4) == [6] * 3           # full cycles: every second cycle, all of it
