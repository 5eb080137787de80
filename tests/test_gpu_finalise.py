"""Steps finalised by the update launch (few partials to read again) and by a
launch of their own (many): the same bits for a right-hand side in a batch that
takes the one and in a batch that takes the other."""
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


@pytest.mark.parametrize("precond,precision", [("BLOCK_JACOBI", "FP32_REFINE64"), ("JACOBI", "FP64"),
                                               ("RB_IC0", "FP32_REFINE64"), ("RB_IC0", "FP64")])
def test_many_right_hand_sides_and_few(g, precond, precision):
    import torch
    # 516 tiles (red-black: 258 a colour): 13 right-hand sides read 3.5e6 (8.7e5) partials per value, two 5e5 (1.3e5)
    nx, ny, R = 400, 330, 13
    r = np.random.default_rng(2)
    N = nx * ny
    ctx = g.gp_ctx_create(0, torch.cuda.current_stream().cuda_stream, 0)
    op = g.gp_op_create(ctx, np.ones((1, ny, nx), dtype=np.uint8), 4, 1)
    g.gp_op_set_blocks(op, torch.from_numpy(r.uniform(0.5, 4.0, (N, 1, 1))).cuda())
    g.gp_op_set_alpha(op, np.ones(1))
    b = torch.from_numpy(r.standard_normal((R, 1, N))).cuda()
    o = g.gp_opts_default(tol=1e-9, zero_guess=1, precond=getattr(g, "GP_PRECOND_" + precond),
                          precision=getattr(g, "GP_PREC_" + precision))
    x = torch.zeros_like(b)
    _, st = g.gp_solve(op, R, b, x, o)
    for r0 in (0, 11):
        few = torch.zeros_like(b[:2])
        _, sf = g.gp_solve(op, 2, b[r0:r0 + 2], few, o)
        assert torch.equal(few, x[r0:r0 + 2])
        for i in range(2):
            assert sf[i]["relres"] == st[r0 + i]["relres"] <= 1e-9
            assert sf[i]["inner_iters"] == st[r0 + i]["inner_iters"]
    y = torch.zeros_like(b)
    g.gp_apply(op, R, x, y)
    assert ((y - b).flatten(1).norm(dim=1) <= 1.01e-9 * b.flatten(1).norm(dim=1)).all()
    g.gp_op_destroy(op)
    g.gp_ctx_destroy(ctx)
