"""Random signs and the prior's quadratic forms at the edges of their tilings:
lengths around a lane's and a counter block's signs, outputs at odd addresses,
K around the regressors that a workgroup takes."""
import numpy as np
import pytest

from oracle import gmrf_oracle as orc, philox

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


@pytest.mark.parametrize("n", [1, 15, 16, 17, 127, 128, 129, 4095, 4096, 4097, 70001])
@pytest.mark.parametrize("shift", [0, 1, 4, 15])
def test_signs_of_any_length_at_any_address(g, ctx, torch_cuda, n, shift):
    buf = torch_cuda.zeros(shift + n + 16, dtype=torch_cuda.int8, device="cuda")
    g.gp_rng_rademacher(ctx, 9, 4, n, buf[shift:shift + n])
    got = buf.cpu().numpy()
    assert np.array_equal(got[shift:shift + n], philox.rademacher(9, 4, n))
    assert not got[:shift].any() and not got[shift + n:].any()


@pytest.mark.parametrize("K", [1, 3, 4, 5, 8, 9, 17])
@pytest.mark.parametrize("dims,conn", [((9, 8, 5), 6), ((17, 16, 1), 4), ((3, 1, 1), 4)])
def test_quadratic_forms(g, ctx, torch_cuda, K, dims, conn):
    r = np.random.default_rng(K)
    mask = (r.random(dims[::-1]) < 0.8).astype(np.uint8)
    mask[0, 0, :2] = 1
    grid = orc.grid(mask, conn)
    N = int(mask.sum())
    W = r.standard_normal((3, K, N))
    op = g.gp_op_create(ctx, mask, conn, K)
    try:
        qf, _, _ = g.gp_alpha_posterior(op, 3, torch_cuda.from_numpy(W).cuda(), 10.0, 0.1, K)
    finally:
        g.gp_op_destroy(op)
    # a sum of at most 3 N squared differences in another order
    assert np.allclose(qf, orc.quadform(grid, W), rtol=1e-14 * (3 * N + 8), atol=0)


def test_signs_beyond_one_launchs_lanes(g, ctx, torch_cuda):
    """2^36 + 100 signs (64 GiB): more than lanes of 16 signs fit a launch."""
    n = (1 << 36) + 100
    free = torch_cuda.cuda.mem_get_info()[0]
    if free < n + (8 << 30):
        pytest.skip("needs 72 GiB of device memory")
    out = torch_cuda.empty(n, dtype=torch_cuda.int8, device="cuda")
    for at in (0, (1 << 35) - 128, 1 << 35, (1 << 36) - 128):
        out[at:at + 228] = 0
    g.gp_rng_rademacher(ctx, 9, 4, n, out)
    for at in (0, (1 << 35) - 128, 1 << 35, (1 << 36) - 128):
        e = np.arange(at, min(at + 228, n), dtype=np.uint64)
        w = philox.philox4x32_10(np.arange(at // 128, int(e[-1]) // 128 + 1, dtype=np.uint64), 9, 4)
        bits = (w[(e // 128 - at // 128).astype(int), (e % 128 // 32).astype(int)] >> (e % 32).astype(np.uint32)) & 1
        assert np.array_equal(out[at:at + len(e)].cpu().numpy(), np.where(bits == 1, 1, -1))
    del out
    torch_cuda.cuda.empty_cache()
