"""The residual alone, whose tiles are its own: meshes around a tile's nodes (32) and threads, every
combination of previous velocity and body force, contexts of both precisions and kinds, and nodes
with more elements than a tile stages rows of (copies of one element).  Against the FP64 oracle and
the residual rows' norm, norm-wise 1e-12 (the oracle sums in another order); two calls agree bit for
bit."""
import numpy as np
import pytest
import torch

from oracle import vms as O
from workloads import kuhn_box, jitter_interior, boundary_nodes
from tests.gpu_common import DEV, to_dev, random_state

pytestmark = pytest.mark.gpu


def _check(B, m, dofs, transient, body_on, precision=0, det=False, seed=1):
    u, up, beta, body = random_state(m, seed)
    Re, dt = 40.0, (0.05 if transient else 0.0)
    up = up if transient else None
    body = body if body_on else None
    ctx = B.Context(to_dev(m.xyz), to_dev(m.tets.astype(np.int32)), to_dev(dofs), precision=precision,
                    deterministic=det)
    d = [None if x is None else to_dev(x) for x in (u, beta, up, body)]
    r, rn = torch.full((m.n_nodes, 4), 7.0, dtype=torch.float64, device=DEV), torch.zeros(1, dtype=torch.float64,
                                                                                          device=DEV)
    B.vms_residual(ctx, d[0], d[1], Re, dt, d[2], d[3], r, rn)
    prob = O.Problem(m.xyz, m.tets, dofs, nu=1.0 / Re, dt=dt, u_prev=up, body=body)
    R, _ = prob.element(u, beta)
    r_o = O.assemble_vector(m.tets, m.n_nodes, R[:, :16]).ravel()
    r_o[dofs] = 0.0
    got = r.cpu().numpy().ravel()
    assert np.linalg.norm(got - r_o) <= 1e-12 * np.linalg.norm(r_o)
    rn_o = O.residual_norm(m.tets, m.n_nodes, R, dofs)
    assert abs(rn.item() - rn_o) <= 1e-12 * rn_o
    r2, rn2 = torch.zeros_like(r), torch.zeros_like(rn)
    B.vms_residual(ctx, d[0], d[1], Re, dt, d[2], d[3], r2, rn2)
    assert torch.equal(r, r2) and torch.equal(rn, rn2)


def _box(cells):
    m = jitter_interior(kuhn_box(cells, (0, 0, 0), (1.0, 1.2, 1.4)), 0.2, 4)
    bnd = np.nonzero(boundary_nodes(m.tets, m.n_nodes))[0]
    return m, np.unique(np.concatenate([(4 * bnd[:, None] + np.arange(3)).ravel(), [3]])).astype(np.int32)


@pytest.mark.parametrize("transient", [False, True])
@pytest.mark.parametrize("body_on", [False, True])
@pytest.mark.parametrize("cells", [(1, 1, 1), (1, 3, 3), (2, 2, 3), (1, 1, 15), (1, 2, 10), (5, 6, 7)])
def test_residual(vms_lib, cells, transient, body_on):
    m, dofs = _box(cells)
    _check(vms_lib, m, dofs, transient, body_on)


@pytest.mark.parametrize("precision,det", [(0, True), (1, False), (1, True)])
def test_other_contexts(vms_lib, precision, det):
    m, dofs = _box((4, 3, 6))
    _check(vms_lib, m, dofs, True, True, precision, det)


@pytest.mark.parametrize("copies", [2047, 2048, 2049, 4200])
def test_more_elements_at_a_node_than_staged_rows(vms_lib, copies):
    class M:
        pass
    m = M()
    m.xyz = np.array([[0, 0, 0], [1, 0, 0.1], [0.2, 1, 0], [0.1, 0.2, 0.9]], dtype=np.float64)
    m.tets = np.tile(np.array([[0, 1, 2, 3]], dtype=np.int32), (copies, 1))
    m.n_nodes, m.n_elems = 4, copies
    _check(vms_lib, m, np.array([3], dtype=np.int32), True, True)
