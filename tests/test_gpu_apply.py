"""The operator product over the work splits that its launch chooses between:
one right-hand side per workgroup on a plain and on a mapped grid, two and four
with the blocks held, ragged last tile and last chunk.  Each right-hand side has
the bits of its product alone, and that is Q x (NumPy)."""
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


# 66 tiles of 256 voxels: up to 4 right-hand sides plain, from 5 mapped, from 19 pairs, from 37 fours (K <= 16)
@pytest.mark.parametrize("K,Rs", [(1, (1, 4, 5, 19, 41)), (4, (5, 20, 37)), (5, (4, 5, 21, 38)), (10, (5, 19)),
                                  (16, (4, 5, 19)), (17, (4, 5, 19)), (24, (1, 5))])
def test_every_split_gives_the_same_bits(g, K, Rs):
    import torch
    nx, ny = 131, 128   # 16,768 voxels
    N = nx * ny
    r = np.random.default_rng(K)
    ctx = g.gp_ctx_create(0, torch.cuda.current_stream().cuda_stream, 0)
    op = g.gp_op_create(ctx, np.ones((1, ny, nx), dtype=np.uint8), 4, K)
    A = r.standard_normal((N, K, K + 1))
    B = np.matmul(A, A.transpose(0, 2, 1)) + np.eye(K)
    alpha = r.uniform(0.5, 3.0, K)
    g.gp_op_set_blocks(op, torch.from_numpy(B).cuda())
    g.gp_op_set_alpha(op, alpha)
    x = torch.from_numpy(r.standard_normal((max(Rs), K, N))).cuda()
    alone = torch.full_like(x, float("nan"))
    for i in range(max(Rs)):
        g.gp_apply(op, 1, x[i:i + 1], alone[i:i + 1])
    for R in Rs:
        y = torch.full_like(x[:R], float("nan"))
        g.gp_apply(op, R, x[:R], y)
        assert torch.equal(y, alone[:R]), R
    for i in (0, max(Rs) - 1):
        v = x[i].cpu().numpy().reshape(K, ny, nx)
        lap = np.zeros_like(v)
        d = np.diff(v, axis=1)
        lap[:, 1:] += d
        lap[:, :-1] -= d
        d = np.diff(v, axis=2)
        lap[:, :, 1:] += d
        lap[:, :, :-1] -= d
        ref = np.einsum("nkl,ln->kn", B, v.reshape(K, N)) + alpha[:, None] * lap.reshape(K, N)
        # K + 6 rounded terms an entry, of the size of the row's products
        scale = np.einsum("nkl,ln->kn", np.abs(B), np.abs(v.reshape(K, N))) + 24.0 * alpha[:, None]
        assert (np.abs(alone[i].cpu().numpy() - ref) <= (K + 6) * 2.3e-16 * scale).all()
    g.gp_op_destroy(op)
    g.gp_ctx_destroy(ctx)
