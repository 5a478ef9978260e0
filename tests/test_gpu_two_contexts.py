"""Contexts of different tile sizes in turn: the largest dynamic LDS a kernel may be launched with belongs
to the kernel, not to a context.  A context whose residual tile takes more than 64 KB (a node with more
elements than a tile stages rows of) works after a context with small tiles was made, and the
other way round; the residual against the FP64 oracle, norm-wise 1e-12 (the bound of the residual
tiles' own tests)."""
import numpy as np
import pytest

from oracle import vms as O
from workloads import kuhn_box
from tests.gpu_common import random_state, to_dev

pytestmark = pytest.mark.gpu


def _mesh(copies):
    if not copies:
        return kuhn_box((1, 1, 1), (0, 0, 0), (1, 1, 1))

    class M:
        pass
    m = M()
    m.xyz = np.array([[0, 0, 0], [1, 0, 0.1], [0.2, 1, 0], [0.1, 0.2, 0.9]], dtype=np.float64)
    m.tets = np.tile(np.array([[0, 1, 2, 3]], dtype=np.int32), (copies, 1))
    m.n_nodes, m.n_elems = 4, copies
    return m


@pytest.mark.parametrize("copies", [(2100, 0), (0, 2100, 0), (2100, 0, 3000, 0)])
def test_in_turn(vms_lib, copies):
    dofs = np.array([3], dtype=np.int32)
    meshes = [_mesh(c) for c in copies]
    contexts = [vms_lib.Context(to_dev(m.xyz), to_dev(m.tets.astype(np.int32)), to_dev(dofs)) for m in meshes]
    for m, ctx in list(zip(meshes, contexts)) * 2:
        u, up, beta, body = random_state(m, 1)
        r, _ = vms_lib.vms_residual(ctx, to_dev(u), to_dev(beta), 40.0, 0.05, to_dev(up), to_dev(body))
        R, _ = O.Problem(m.xyz, m.tets, dofs, nu=1.0 / 40.0, dt=0.05, u_prev=up, body=body).element(u, beta)
        ref = O.assemble_vector(m.tets, m.n_nodes, R[:, :16]).ravel()
        ref[dofs] = 0.0
        assert np.linalg.norm(r.cpu().numpy().ravel() - ref) <= 1e-12 * np.linalg.norm(ref)
