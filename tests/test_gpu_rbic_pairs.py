"""The red-black solver's FP64 outer step on two right-hand sides together (K
from 9 to 12, enough work items), at both ends of that range of K and beside
it: an odd number of right-hand sides, zero ones between the others, a random
start value for some.  Every right-hand side must reach its FP64 relative
residual (the outer iteration stops on it), by the operator on the device and,
for two of them, by the same product in NumPy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


@pytest.fixture(scope="module")
def g(built_library, torch_cuda):
    from paper_1606_00980_amd import gmrf
    return gmrf


@pytest.fixture(scope="module")
def ctx(g, torch_cuda):
    h = g.gp_ctx_create(0, torch_cuda.cuda.current_stream().cuda_stream, 0)
    yield h
    torch_cuda.cuda.synchronize()
    g.gp_ctx_destroy(h)


def q_times(B, alpha, x, dims):
    """(B + blkdiag_k alpha_k G'G) x on a full box."""
    v = x.reshape((len(alpha),) + dims[::-1])
    lap = np.zeros_like(v)
    for ax in (1, 2, 3):
        d = np.diff(v, axis=ax)
        pad = [(0, 0)] * 4
        pad[ax] = (1, 0)
        lap += np.pad(d, pad)
        pad[ax] = (0, 1)
        lap -= np.pad(d, pad)
    return np.einsum("nkl,ln->kn", B, x) + alpha[:, None] * lap.reshape(x.shape)


@pytest.mark.parametrize("K,R,dims", [(8, 15, (48, 46, 37)), (9, 15, (48, 46, 37)), (10, 15, (48, 46, 37)),
                                      (12, 15, (48, 46, 37)), (13, 15, (48, 46, 37)), (9, 1, (13, 11, 7)),
                                      (12, 3, (13, 11, 7))])
def test_outer_step_in_pairs(g, ctx, torch_cuda, K, R, dims):
    N = dims[0] * dims[1] * dims[2]
    r = np.random.default_rng(K + R)
    mask = np.ones(dims[::-1], dtype=np.uint8)
    A = r.standard_normal((N, K, K + 2))
    B = np.matmul(A, A.transpose(0, 2, 1)) / (K + 2)
    alpha = r.uniform(0.5, 3.0, K)
    op = g.gp_op_create(ctx, mask, 6, K)
    try:
        g.gp_op_set_blocks(op, torch_cuda.from_numpy(B).cuda())
        g.gp_op_set_alpha(op, alpha)
        b = r.standard_normal((R, K, N)) * np.linspace(0.1, 10.0, R)[:, None, None]
        x0 = np.zeros_like(b)
        if R > 4:
            b[3] = b[R - 1] = 0.0
            x0[::4] = r.standard_normal(x0[::4].shape)
        bd, x = torch_cuda.from_numpy(b).cuda(), torch_cuda.from_numpy(x0).cuda()
        tol = 1e-9
        g.gp_solve(op, R, bd, x, g.gp_opts_default(tol=tol, precond=g.GP_PRECOND_RB_IC0))
        y = torch_cuda.empty_like(x)
        g.gp_apply(op, R, x, y)
        res = (bd - y).flatten(1).norm(dim=1).cpu().numpy()
        nb = bd.flatten(1).norm(dim=1).cpu().numpy()
        assert (res <= 1.01 * tol * nb).all(), res / np.maximum(nb, 1e-300)
        xs = x.cpu().numpy()
        if R > 4:
            assert not xs[3].any() and not xs[R - 1].any()
        for i in {0, R // 2}:
            assert np.linalg.norm(b[i] - q_times(B, alpha, xs[i], dims)) <= 1.01 * tol * np.linalg.norm(b[i])
    finally:
        torch_cuda.cuda.synchronize()
        g.gp_op_destroy(op)


@pytest.mark.parametrize("K,R,dims", [(1, 1, (3, 1, 1)), (6, 3, (13, 11, 7)), (9, 5, (48, 46, 37)), (9, 7, (48, 46, 37)),
                                      (10, 7, (48, 46, 37)), (24, 2, (9, 8, 4))])
def test_product_of_several_right_hand_sides(g, ctx, torch_cuda, K, R, dims):
    """One, two and four right-hand sides to a workgroup, the last ones fewer."""
    N = dims[0] * dims[1] * dims[2]
    r = np.random.default_rng(3 * K + R)
    A = r.standard_normal((N, K, K + 2))
    B = np.matmul(A, A.transpose(0, 2, 1)) / (K + 2)
    alpha = r.uniform(0.5, 3.0, K)
    x = r.standard_normal((R, K, N))
    op = g.gp_op_create(ctx, np.ones(dims[::-1], dtype=np.uint8), 6, K)
    try:
        g.gp_op_set_blocks(op, torch_cuda.from_numpy(B).cuda())
        g.gp_op_set_alpha(op, alpha)
        y = torch_cuda.empty((R, K, N), dtype=torch_cuda.float64, device="cuda")
        g.gp_apply(op, R, torch_cuda.from_numpy(x).cuda(), y)
        ys = y.cpu().numpy()
        for i in range(R):
            # sums of K + 6 products in another order
            scale = np.einsum("nkl,ln->kn", np.abs(B), np.abs(x[i])) + 12 * alpha[:, None] * np.abs(x).max()
            assert (np.abs(ys[i] - q_times(B, alpha, x[i], dims)) <= 1e-15 * 2 * (K + 6) * scale).all()
    finally:
        torch_cuda.cuda.synchronize()
        g.gp_op_destroy(op)
