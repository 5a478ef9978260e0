"""A node with more elements than a tile's records number (65,535): copies of one element, as many as
vms_create has always taken.  Residual rows and norms, from the residual alone and from the assembly, against the FP64 oracle.
The rows are sums of as many terms as there are copies, on both sides: the bound is the worst rounding of two
such sums, 2 n 2^-53 of the terms' magnitudes, and 1e-12 of them for the elements' own rounding."""
import numpy as np
import pytest

from oracle import vms as O
from tests.gpu_common import random_state, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copies", [65534, 65535, 65536, 67600])
def test_residual(vms_lib, copies):
    class M:
        pass
    m = M()
    m.xyz = np.array([[0, 0, 0], [1, 0, 0.1], [0.2, 1, 0], [0.1, 0.2, 0.9]], dtype=np.float64)
    m.tets = np.tile(np.array([[0, 1, 2, 3]], dtype=np.int32), (copies, 1))
    m.n_nodes, m.n_elems = 4, copies
    dofs = np.array([3], dtype=np.int32)
    u, up, beta, body = random_state(m, 3)
    Re, dt = 40.0, 0.05
    ctx = vms_lib.Context(to_dev(m.xyz), to_dev(m.tets), to_dev(dofs))
    args = (to_dev(u), to_dev(beta), Re, dt, to_dev(up), to_dev(body))
    R, _ = O.Problem(m.xyz, m.tets, dofs, nu=1.0 / Re, dt=dt, u_prev=up, body=body).element(u, beta)
    ref = O.assemble_vector(m.tets, m.n_nodes, R[:, :16]).ravel()
    size = O.assemble_vector(m.tets, m.n_nodes, np.abs(R[:, :16])).ravel()
    ref[dofs] = size[dofs] = 0.0
    tol = 1e-12 + 2 * copies * 2.0 ** -53
    rn_ref = O.residual_norm(m.tets, m.n_nodes, R, dofs)
    r, rn = vms_lib.vms_residual(ctx, *args)
    assert np.linalg.norm(r.cpu().numpy().ravel() - ref) <= tol * np.linalg.norm(size)
    _, rhs, rn_a = vms_lib.vms_condense_assemble(ctx, *args)
    scale = np.linalg.norm(size) + rn_ref
    assert abs(rn.item() - rn_ref) <= tol * scale and abs(rn_a.item() - rn_ref) <= tol * scale
    assert np.isfinite(rhs.cpu().numpy()).all()
