"""Block-Jacobi solves whose preconditioner blocks do not stay in registers
(FP64 from K = 9, FP32 from K = 13): entries streamed in groups, K on both sides
of the limit and with every kind of remainder, against the oracle."""
import numpy as np
import pytest

from oracle import gmrf_oracle as orc
from paper_1606_00980_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g(built_library):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_1606_00980_amd import gmrf
    return gmrf


@pytest.mark.parametrize("precision,K", [("FP64", k) for k in (8, 9, 10, 11, 12, 15, 16, 24)] +
                         [("FP32_REFINE64", k) for k in (12, 13, 14, 15, 16, 20, 24)])
def test_streamed_blocks(g, precision, K):
    import torch
    w = synth.tiny((9, 8, 7), 6, K, seed=K)
    R, tol = 3, 1e-10
    ctx = g.gp_ctx_create(0, torch.cuda.current_stream().cuda_stream, 0)
    op = g.gp_op_create(ctx, w.mask, w.conn, w.K)
    B = torch.from_numpy(w.B).cuda()
    g.gp_op_set_blocks(op, B)
    g.gp_op_set_alpha(op, w.alpha)
    b = np.random.default_rng(K).standard_normal((R, w.K, w.N))
    bd, x = torch.from_numpy(b).cuda(), torch.zeros((R, w.K, w.N), dtype=torch.float64, device="cuda")
    o = g.gp_opts_default(tol=tol, precision=getattr(g, "GP_PREC_" + precision), rhs_tile=2)
    _, st = g.gp_solve(op, R, bd, x, o)
    Q = orc.precision(orc.grid(w.mask, w.conn), w.alpha, w.B)
    xs = x.cpu().numpy()
    assert all(s["status"] == g.GP_OK for s in st) and np.all(orc.relres(Q, xs, b) <= 1.01 * tol)
    ref = orc.solve_direct(Q, b)
    assert np.linalg.norm(xs - ref) <= 1e-6 * np.linalg.norm(ref)
    g.gp_op_destroy(op)
    g.gp_ctx_destroy(ctx)
