"""Arrays aligned to their entries and no further: views that start one entry into a buffer give the same
bits as arrays of their own, in every call that reads or writes a caller's array in wide pieces (matrix,
state, increments, preconditioner blocks, element tangents)."""
import numpy as np
import pytest
import torch

from workloads import cavity_mesh, cavity_bc
from tests.gpu_common import DEV, random_state, to_dev

pytestmark = pytest.mark.gpu


def _offset(t):
    """t's values in a view that starts one entry into its buffer."""
    v = torch.empty(t.numel() + 1, dtype=t.dtype, device=DEV)[1:].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 == t.element_size() and v.is_contiguous()
    return v


def _as_is(t):
    return t.clone()


def _calls(B, ctx, m, precision, place):
    u, up, beta, body = random_state(m, 2)
    state = [place(to_dev(x)) for x in (u, beta, up, body)]
    args = (state[0], state[1], 40.0, 0.05, state[2], state[3])
    out = []
    A, rhs, rn = B.vms_condense_assemble(ctx, *args, place(ctx.new_bsr()), place(ctx.new_vec()))
    out += [A, rhs, rn]
    out += B.vms_residual(ctx, *args, place(ctx.new_vec()))
    Ke, Re = B.vms_element_tangents(ctx, *args, place(torch.zeros((m.n_elems, 19, 19), dtype=torch.float64, device=DEV)),
                                    place(torch.zeros((m.n_elems, 19), dtype=torch.float64, device=DEV)))
    out += [Ke, Re]
    out += B.vms_full_assemble(ctx, *args, place(ctx.new_full_bsr()), place(ctx.new_full_vec()))
    rng = np.random.default_rng(5)
    x = place(to_dev(rng.standard_normal((m.n_nodes, 4)), ctx.dtype))
    out.append(B.vms_bsr_spmv(ctx, A, x, place(torch.zeros_like(x))))
    w = place(to_dev(0.1 * rng.standard_normal(B.PC_NWEIGHTS), torch.float32))
    out.append(B.vms_pc_features(ctx, A, place(torch.zeros((m.n_nodes, B.PC_NIN), dtype=torch.float32, device=DEV))))
    for weights in (None, w):
        out.append(B.vms_pc_blocks(ctx, A, weights, place(torch.zeros((m.n_nodes, 16), dtype=torch.float32, device=DEV))))
    for b64 in ((0, 1) if precision else (0,)):
        for k in (0, 5):
            y = place(ctx.new_vec())
            _, info = B.vms_gmres_solve(ctx, A, rhs, y, B.solve_opts(restart=20, rtol=1e-9, max_iters=50, deflate=k,
                                                                     basis_fp64=b64), allow_noconv=True)
            out += [y, torch.tensor([info.iters])]
    u2, beta2 = place(to_dev(u)), place(to_dev(beta))
    B.vms_recover_update(ctx, u2, beta2, y, 40.0, 0.05, state[2], state[3])
    out += [u2, beta2]
    r = place(to_dev(rng.standard_normal((3, m.n_nodes, 4)), torch.float32))
    adam, grad = (place(torch.zeros(n, dtype=torch.float32, device=DEV)) for n in (2 * B.PC_NWEIGHTS, B.PC_NWEIGHTS))
    B.vms_pc_train_step(ctx, A, r, w, adam, 1, 1e-3, grad)
    return out + [w, adam, grad]


@pytest.mark.parametrize("precision", [0, 1])
def test_same_bits(vms_lib, precision):
    B = vms_lib
    m = cavity_mesh(6)
    ctx = B.Context(to_dev(m.xyz), to_dev(m.tets.astype(np.int32)), to_dev(cavity_bc(m).dofs), precision=precision,
                    full_system=True, deterministic=True, basis_fp64=precision == 1)
    a = _calls(B, ctx, m, precision, _as_is)
    b = _calls(B, ctx, m, precision, _offset)
    for i, (x, y) in enumerate(zip(a, b)):
        assert torch.isfinite(x.double()).all() and torch.equal(x, y), i
