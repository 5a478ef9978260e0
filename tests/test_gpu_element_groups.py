"""Element-wise kernels at counts around their workgroups (16 elements share a wave): raw element
residuals and tangents, each output alone and both, with nothing written past the last element.
Tolerances as for the larger meshes (FP64 1e-12, tangents of a mixed context 1e-5)."""
import ctypes

import numpy as np
import pytest
import torch

from oracle.element import element_residual_tangent
from workloads import kuhn_box, jitter_interior
from tests.gpu_common import DEV, to_dev, make_context, random_state

pytestmark = pytest.mark.gpu


class _Cut:
    """The first n_elems elements of a jittered box, on the nodes they touch."""

    def __init__(self, n_elems):
        m = jitter_interior(kuhn_box((2, 3, 3), (0, 0, 0), (1.0, 1.1, 0.9)), 0.2, 5)
        used, loc = np.unique(m.tets[:n_elems], return_inverse=True)
        self.xyz = np.ascontiguousarray(m.xyz[used])
        self.tets = np.ascontiguousarray(loc.reshape(-1, 4).astype(np.int32))
        self.n_nodes, self.n_elems = len(used), n_elems


@pytest.mark.parametrize("precision,tol", [(0, 1e-12), (1, 1e-5)])
@pytest.mark.parametrize("n_elems", [1, 15, 16, 17, 31, 33, 64, 107])
def test_raw_outputs(vms_lib, n_elems, precision, tol):
    B = vms_lib
    m = _Cut(n_elems)
    ctx = make_context(B, m, np.array([3], dtype=np.int32), precision)
    u, up, beta, body = random_state(m, n_elems)
    R_o, K_o = element_residual_tangent(m.xyz, m.tets, u, beta, 1 / 40.0, 0.05, up, body)
    args = [to_dev(x) for x in (u, up, beta, body)]
    guard = 7.0
    for want_k, want_r in ((True, True), (True, False), (False, True)):
        K = torch.full((n_elems + 1, 19, 19), guard, dtype=torch.float64, device=DEV)
        R = torch.full((n_elems + 1, 19), guard, dtype=torch.float64, device=DEV)
        p = [ctypes.c_void_p(t.data_ptr()) for t in args]
        rc = B._lib.vms_element_tangents(ctx.handle, p[0], p[1], p[2], 40.0, 0.05, p[3],
                                         ctypes.c_void_p(K.data_ptr()) if want_k else None,
                                         ctypes.c_void_p(R.data_ptr()) if want_r else None, None)
        torch.cuda.synchronize()
        assert rc == 0
        assert bool((K[-1] == guard).all()) and bool((R[-1] == guard).all())
        if want_k:
            ek = np.linalg.norm(K[:-1].cpu().numpy() - K_o, axis=(1, 2)) / np.linalg.norm(K_o, axis=(1, 2))
            assert ek.max() <= tol
        else:
            assert bool((K == guard).all())
        if want_r:
            er = np.linalg.norm(R[:-1].cpu().numpy() - R_o, axis=1) / np.linalg.norm(R_o, axis=1)
            assert er.max() <= 1e-12
        else:
            assert bool((R == guard).all())
