"""FP64 solves of small operators (one workgroup per right-hand side) against
the oracle and the grouped kernels, at the edges of their voxel tilings."""
import numpy as np
import pytest

from oracle import gmrf_oracle as orc
from paper_1606_00980_amd import synth

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


def operator(nx, ny, K, seed):
    """A box slice with random SPD blocks and alpha."""
    r = np.random.default_rng(seed)
    N = nx * ny
    X = r.standard_normal((N, K + 3, K))
    B = np.einsum("ntk,ntl->nkl", X, X) + 0.2 * np.eye(K)
    return np.ones((1, ny, nx), dtype=np.uint8), B, r.gamma(2.0, 1.0, K), r.standard_normal((3, K, N))


# (nx, ny): one voxel, around 512 voxels per workgroup sweep, several per lane
@pytest.mark.parametrize("pc", ["JACOBI", "BLOCK_JACOBI"])
@pytest.mark.parametrize("nx,ny,K", [(1, 1, 1), (7, 73, 2), (16, 32, 8), (27, 19, 7), (41, 25, 6), (37, 41, 5),
                                     (43, 47, 4), (45, 57, 3), (61, 67, 2), (79, 77, 1)])
def test_small_solves(g, ctx, torch_cuda, pc, nx, ny, K):
    torch = torch_cuda
    mask, B, alpha, b = operator(nx, ny, K, nx + ny + K)
    op = g.gp_op_create(ctx, mask, 4, K)
    Bd = torch.from_numpy(B).cuda()
    g.gp_op_set_blocks(op, Bd)
    g.gp_op_set_alpha(op, alpha)
    Q = orc.precision(orc.grid(mask, 4), alpha, B)
    ref = np.stack([orc.solve(Q, b[i:i + 1])[0] for i in range(3)])
    bd = torch.from_numpy(b).cuda()
    kw = dict(tol=1e-10, precision=g.GP_PREC_FP64, precond=getattr(g, "GP_PRECOND_" + pc))
    x = torch.full_like(bd, float("nan"))
    _, st = g.gp_solve(op, 3, bd, x, g.gp_opts_default(zero_guess=1, **kw))
    grouped = torch.zeros_like(bd)
    _, sg = g.gp_solve(op, 3, bd, grouped, g.gp_opts_default(rhs_tile=4, **kw))
    for i in range(3):
        scale = np.linalg.norm(ref[i])
        assert st[i]["relres"] <= 1e-10
        assert np.linalg.norm(x[i].cpu().numpy() - ref[i]) <= 1e-8 * scale
        # the same iterates in exact arithmetic
        assert abs(st[i]["inner_iters"] - sg[i]["inner_iters"]) <= 1
        assert np.linalg.norm((x[i] - grouped[i]).cpu().numpy()) <= 1e-8 * scale
    # alone and in a batch with another operator: the same bits
    one = torch.zeros_like(bd[:1])
    g.gp_solve(op, 1, bd[1:2], one, g.gp_opts_default(zero_guess=1, **kw))
    assert torch.equal(one[0], x[1])
    w = synth.tiny((13, 11, 7), 6, 3, seed=3)
    other = g.gp_op_create(ctx, w.mask, w.conn, w.K)
    wB, wb = torch.from_numpy(w.B).cuda(), torch.from_numpy(w.bw[None].copy()).cuda()
    g.gp_op_set_blocks(other, wB)
    g.gp_op_set_alpha(other, w.alpha)
    x2, xo = torch.zeros_like(bd), torch.zeros_like(wb)
    _, sb = g.gp_solve_batch(ctx, [(op, 3, bd, x2), (other, 1, wb, xo)], g.gp_opts_default(zero_guess=1, **kw))
    assert torch.equal(x2, x) and all(s["status"] == g.GP_OK for s in sb)
    # a warm start at the solution, b = 0, an iteration cap and a NaN
    _, sw = g.gp_solve(op, 3, bd, x2, g.gp_opts_default(**kw))
    assert all(s["inner_iters"] <= 1 for s in sw)
    bd2 = bd.clone()
    bd2[0] = 0.0
    bd2[2, 0, 0] = float("nan")
    x3 = torch.full_like(bd, float("nan"))
    st3, s3 = g.gp_solve(op, 3, bd2, x3, g.gp_opts_default(zero_guess=1, **kw), check=False)
    assert s3[0]["status"] == g.GP_OK and s3[0]["inner_iters"] == 0 and not x3[0].any()
    assert s3[1]["status"] == g.GP_OK and torch.equal(x3[1], x[1])
    assert s3[2]["status"] == g.GP_ERR_BREAKDOWN
    if st[0]["inner_iters"] > 2:
        _, sc = g.gp_solve(op, 3, bd, x3, g.gp_opts_default(zero_guess=1, max_iter=2, **kw), check=False)
        assert sc[0]["status"] == g.GP_ERR_NOT_CONVERGED and sc[0]["inner_iters"] == 2
    g.gp_op_destroy(other)
    g.gp_op_destroy(op)


@pytest.mark.parametrize("pc,prec", [("BLOCK_JACOBI", "FP32_REFINE64"), ("JACOBI", "FP64"), ("RB_IC0", "FP32_REFINE64"),
                                     ("RB_IC0", "FP64")])
def test_both_finalisations_in_one_batch(g, ctx, torch_cuda, pc, prec):
    """A K = 1 operator of more tiles than the update launch finalises itself
    (its steps take the finalising launch) grouped with one of a few tiles:
    each right-hand side converges and equals its solve alone, bitwise."""
    torch = torch_cuda
    kw = dict(tol=1e-8, precond=getattr(g, "GP_PRECOND_" + pc), precision=getattr(g, "GP_PREC_" + prec), rhs_tile=2,
              zero_guess=1)
    items, keep = [], []
    for nx, ny, seed in ((170, 151, 1), (40, 31, 2)):   # 101 and 5 tiles (red-black: 51 and 3 a colour)
        mask, B, alpha, b = operator(nx, ny, 1, seed)
        op = g.gp_op_create(ctx, mask, 4, 1)
        Bd, bd = torch.from_numpy(B).cuda(), torch.from_numpy(b).cuda()
        g.gp_op_set_blocks(op, Bd)
        g.gp_op_set_alpha(op, alpha)
        items.append((op, 3, bd, torch.zeros_like(bd)))
        keep.append((Bd, orc.precision(orc.grid(mask, 4), alpha, B), b))
    _, st = g.gp_solve_batch(ctx, items, g.gp_opts_default(**kw))
    at = 0
    for (op, R, bd, x), (_, Q, b) in zip(items, keep):
        alone = torch.zeros_like(bd)
        _, sa = g.gp_solve(op, R, bd, alone, g.gp_opts_default(**kw))
        assert torch.equal(alone, x)
        for r in range(R):
            res = np.linalg.norm(b[r].ravel() - Q @ x[r].cpu().numpy().ravel()) / np.linalg.norm(b[r])
            assert res <= 1.01e-8 and st[at + r]["inner_iters"] == sa[r]["inner_iters"]
        at += R
        g.gp_op_destroy(op)


@pytest.mark.parametrize("K,N", [(10, 512), (11, 512), (11, 513), (12, 1), (12, 512), (13, 512)])
def test_jacobi_around_the_largest_k(g, ctx, torch_cuda, K, N):
    """Jacobi solves in FP64 on either side of the largest K that the
    one-workgroup kernel exists for, alone and in one batch with an operator
    that it takes."""
    torch = torch_cuda
    kw = dict(tol=1e-10, precision=g.GP_PREC_FP64, precond=g.GP_PRECOND_JACOBI, zero_guess=1)
    items, refs, keep = [], [], []
    for nx, k in ((N, K), (70, 2)):
        mask, B, alpha, b = operator(nx, 1, k, nx + k)
        op = g.gp_op_create(ctx, mask, 4, k)
        Bd, bd = torch.from_numpy(B).cuda(), torch.from_numpy(b).cuda()
        g.gp_op_set_blocks(op, Bd)
        g.gp_op_set_alpha(op, alpha)
        Q = orc.precision(orc.grid(mask, 4), alpha, B)
        refs.append(np.stack([orc.solve(Q, b[i:i + 1])[0] for i in range(3)]))
        items.append((op, 3, bd, torch.full_like(bd, float("nan"))))
        keep.append(Bd)
    _, st = g.gp_solve_batch(ctx, items, g.gp_opts_default(**kw))
    assert all(s["status"] == g.GP_OK and s["relres"] <= 1e-10 for s in st)
    for (op, R, bd, x), ref in zip(items, refs):
        assert np.linalg.norm(x.cpu().numpy() - ref) <= 1e-8 * np.linalg.norm(ref)
        alone = torch.zeros_like(bd)
        g.gp_solve(op, R, bd, alone, g.gp_opts_default(**kw))
        assert torch.equal(alone, x)
        g.gp_op_destroy(op)


def test_autotune_knows_the_one_workgroup_solve(g, ctx, torch_cuda, tmp_path):
    """On an operator that automatic options solve in one workgroup, the tuner
    returns them (they are several times faster than any grouped configuration)
    and still keeps a grouped entry in its table; on a larger one it returns a
    grouped configuration as ever."""
    torch = torch_cuda
    for nx, ny, small in ((61, 40, True), (120, 110, False)):
        mask, B, alpha, b = operator(nx, ny, 2, nx)
        op = g.gp_op_create(ctx, mask, 4, 2)
        Bd, bd = torch.from_numpy(B).cuda(), torch.from_numpy(b).cuda()
        g.gp_op_set_blocks(op, Bd)
        g.gp_op_set_alpha(op, alpha)
        o = g.gp_opts_default(tol=1e-10, precision=g.GP_PREC_FP64, zero_guess=1)
        best = g.gp_autotune(op, 3, o)
        assert (best.rhs_tile == 0) == small and (best.matvec == g.GP_MATVEC_AUTO) == small
        x, y = torch.zeros_like(bd), torch.zeros_like(bd)
        g.gp_solve(op, 3, bd, x, best)
        g.gp_solve(op, 3, bd, y, o)
        if small:
            assert torch.equal(x, y)
        path = str(tmp_path / f"tune{nx}.json")
        g.gp_tune_save(ctx, path)
        g.gp_tune_load(ctx, path)
        g.gp_op_destroy(op)
