"""Training step of the learned correction over batch sizes and node counts: groups of one to
eight samples (several groups, a last smaller one, groups shortened by a small Krylov basis),
node counts off the 16-node tiles, and a mesh that takes every kernel of the step past its
largest grid.  Loss and gradient against the FP64 oracle, which is fed the GPU's own matrix;
tolerances as for the single training step (FP32 kernels: loss 1e-4, gradient 1e-3)."""
import numpy as np
import pytest
import torch

from oracle import learned_pc as LP
from workloads import cavity_mesh, cavity_bc, apply_dirichlet
from tests.gpu_common import DEV, to_dev, make_context, bsr_to_csr, rel_fro

pytestmark = pytest.mark.gpu


def _check(B, n, precision, batch, max_restart):
    m = cavity_mesh(n)
    bc = cavity_bc(m)
    u = np.zeros((m.n_nodes, 4))
    apply_dirichlet(u, bc)
    ctx = make_context(B, m, bc.dofs, precision, max_restart=max_restart)
    A_g, _, _ = B.vms_condense_assemble(ctx, to_dev(u), to_dev(np.zeros((m.n_elems, 3))), 50.0)
    rng = np.random.default_rng(100 * n + batch)
    rs = rng.standard_normal((batch, m.n_nodes, 4)).astype(np.float32)
    rs *= np.exp(rng.standard_normal((batch, 1, 1))).astype(np.float32)
    w = LP.init_weights(1)
    n_out = LP.N_OUT * LP.N_HID + LP.N_OUT
    w[-n_out:] = 0.05 * rng.standard_normal(n_out)
    w = w.astype(np.float32)
    grad = torch.zeros(B.PC_NWEIGHTS, dtype=torch.float32, device=DEV)
    loss = torch.zeros(1, dtype=torch.float32, device=DEV)
    B.vms_pc_train_step(ctx, A_g, to_dev(rs), to_dev(w), None, 0, 0.0, grad, loss)
    A = bsr_to_csr(ctx, A_g)
    x_o, D = LP.features(A, m.n_nodes, bc.dofs)
    L_o, g_o = LP.loss_and_grad(w.astype(np.float64), A, x_o, D, LP.dirichlet_mask(m.n_nodes, bc.dofs),
                                [r.ravel().astype(np.float64) for r in rs])
    assert abs(loss.item() - L_o) <= 1e-4 * L_o
    assert rel_fro(grad.cpu().numpy(), g_o) <= 1e-3
    # the same call again gives the same bits (fixed summation orders)
    grad2, loss2 = torch.zeros_like(grad), torch.zeros_like(loss)
    B.vms_pc_train_step(ctx, A_g, to_dev(rs), to_dev(w), None, 0, 0.0, grad2, loss2)
    assert torch.equal(grad, grad2) and torch.equal(loss, loss2)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("batch", [1, 2, 3, 8, 9, 21])
def test_batch_sizes(vms_lib, precision, batch):
    _check(vms_lib, 4, precision, batch, 50)


@pytest.mark.parametrize("precision,max_restart", [(0, 1), (0, 3), (1, 2), (1, 4), (1, 8)])
def test_groups_that_a_short_basis_holds(vms_lib, precision, max_restart):
    _check(vms_lib, 3, precision, 7, max_restart)


@pytest.mark.parametrize("precision", [0, 1])
def test_several_passes_of_every_kernel(vms_lib, precision):
    _check(vms_lib, 40, precision, 3, 50)
