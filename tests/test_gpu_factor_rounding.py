"""The voxel blocks' Cholesky factors and inverses divide with one rounding.

Blocks whose pivots are whole numbers make every other step exact, so an entry
of the factor is b / p and one of the inverse (1 / p) (b / p), each operation
rounded once: compared bitwise with NumPy's.  A product with the rounded
reciprocal misses many of them.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g(built_library):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_1606_00980_amd import gmrf
    return gmrf


@pytest.mark.parametrize("K", [2, 6, 15, 16, 17])
@pytest.mark.parametrize("p", [3.0, 5.0, 7.0, 11.0])
def test_factors_and_inverses(g, K, p):
    import torch
    N = 300
    mask = np.zeros((1, 1, 2 * N - 1), dtype=np.uint8)
    mask[0, 0, ::2] = 1   # isolated voxels of the first colour: the solve is the inverse
    ctx = g.gp_ctx_create(0, torch.cuda.current_stream().cuda_stream, 0)
    op = g.gp_op_create(ctx, mask, 4, K)
    b10 = np.arange(1, N + 1) * 0.5
    x = torch.zeros((1, K, N), dtype=torch.float64, device="cuda")
    out = torch.zeros_like(x)
    x[0, 0] = 1.0
    zero = torch.zeros((K, N), dtype=torch.float64, device="cuda")
    z1 = torch.zeros((1, K, 2, N), dtype=torch.float64, device="cuda")

    def blocks(b00, off, b11):
        B = np.repeat(np.eye(K)[None], N, 0)
        B[:, 0, 0], B[:, 0, 1], B[:, 1, 0], B[:, 1, 1] = b00, off, off, b11
        g.gp_op_set_blocks(op, torch.from_numpy(B).cuda())
        g.gp_op_set_alpha(op, np.zeros(K))

    # L_10 = b_10 / p, below the pivot p
    blocks(p * p, b10, b10 * b10 + 1.0)
    g.gp_perturb_rhs(op, 1, zero, z1, x, out)
    assert np.array_equal(out[0, 1].cpu().numpy(), b10 / p)
    # (L^{-1})_10 = -b_10 / p, in the row of the pivot p; the inverse's entry is that times 1 / p
    blocks(1.0, b10, b10 * b10 + p * p)
    o = g.gp_opts_default(tol=1e-12, precision=g.GP_PREC_FP64, precond=g.GP_PRECOND_RB_IC0, zero_guess=1)
    g.gp_solve(op, 1, x, out, o)
    assert np.array_equal(out[0, 1].cpu().numpy(), (1.0 / p) * -(b10 / p))
    g.gp_op_destroy(op)
    g.gp_ctx_destroy(ctx)
