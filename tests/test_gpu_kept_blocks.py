"""Device blocks that a context keeps for reuse: inside the budget, not
counted as used, and never in the way of an allocation that fits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g(built_library):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1606_00980_amd import gmrf
    return gmrf


@pytest.mark.parametrize("slack", [0, 1 << 20])
def test_datasets_come_and_go_within_the_budget(g, slack):
    """Datasets of changing shapes in a context whose budget holds one of them at a time."""
    import torch
    nx, K, T = 5000, 4, 40
    r = np.random.default_rng(3)
    mask = np.ones((1, 1, nx), dtype=np.uint8)
    Y = torch.from_numpy(r.standard_normal((T, nx))).cuda()
    lam = torch.ones(nx, dtype=torch.float64, device="cuda")
    bw = torch.empty((K, nx), dtype=torch.float64, device="cuda")
    X = r.standard_normal((T, K))
    stream = torch.cuda.current_stream().cuda_stream
    free = g.gp_ctx_create(0, stream, 0)   # what the largest dataset takes
    op = g.gp_op_create(free, mask, 4, K)
    base = g.gp_ctx_memory(free)[0]
    d = g.gp_data_create(op, T, 4, X, Y)
    most = g.gp_ctx_memory(free)[0]
    g.gp_data_destroy(d)
    assert g.gp_ctx_memory(free)[0] == base
    g.gp_op_destroy(op)
    assert g.gp_ctx_memory(free)[0] == 0
    g.gp_ctx_destroy(free)
    ctx = g.gp_ctx_create(0, stream, most + slack)
    op = g.gp_op_create(ctx, mask, 4, K)
    A = torch.zeros((1, 4, nx), dtype=torch.float64, device="cuda")
    first = None
    for P in (4, 1, 4, 0, 3, 4, 4):
        d = g.gp_data_create(op, T, P, X, Y)
        assert g.gp_ctx_memory(ctx)[0] <= most + slack
        g.gp_data_assemble(d, lam, 1, A if P else None, bw)
        g.gp_data_destroy(d)
        assert g.gp_ctx_memory(ctx)[0] == base
        if P == 4:   # the same bits from a new and a reused block
            first = bw.clone() if first is None else first
            assert torch.equal(bw, first)
    g.gp_op_destroy(op)
    assert g.gp_ctx_memory(ctx)[0] == 0
    g.gp_ctx_destroy(ctx)


@pytest.mark.parametrize("how", ["left stream", "graph"])
def test_an_operator_given_back_while_its_product_is_queued(g, how):
    """A product queued behind other work on a stream that the context has left
    (or replayed from a caller's graph there), its operator destroyed and
    another of the same sizes made with other blocks: the product is the first
    operator's, bitwise, in every replay."""
    import torch
    dims, K, R = (40, 36, 24), 6, 4
    N = dims[0] * dims[1] * dims[2]
    r = np.random.default_rng(5)
    mask = np.ones(dims[::-1], dtype=np.uint8)
    x = torch.from_numpy(r.standard_normal((R, K, N))).cuda()
    eye = torch.eye(K, dtype=torch.float64, device="cuda")
    busy = torch.randn((4096, 4096), device="cuda")
    first, other = torch.cuda.Stream(), torch.cuda.Stream()
    ctx = g.gp_ctx_create(0, first.cuda_stream, 0)

    def operator(scale):
        op = g.gp_op_create(ctx, mask, 6, K)
        blocks = (scale * eye)[None].repeat(N, 1, 1).contiguous()
        torch.cuda.synchronize()
        g.gp_op_set_blocks(op, blocks)
        g.gp_op_set_alpha(op, np.full(K, scale))
        return op

    op = operator(1.0)
    want, y = torch.empty_like(x), torch.zeros_like(x)
    torch.cuda.synchronize()
    g.gp_apply(op, R, x, want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    if how == "graph":
        with torch.cuda.graph(graph, stream=other):
            g.gp_ctx_set_stream(ctx, torch.cuda.current_stream().cuda_stream)
            g.gp_apply(op, R, x, y)
        y.zero_()
        torch.cuda.synchronize()
        for _ in range(3):
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, want)
            y.zero_()
        torch.cuda.synchronize()
    with torch.cuda.stream(first):
        for _ in range(20):
            busy = busy @ busy * 1e-4
        if how == "graph":
            graph.replay()
        else:
            g.gp_apply(op, R, x, y)
    g.gp_ctx_set_stream(ctx, other.cuda_stream)
    g.gp_op_destroy(op)
    op = operator(7.0)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    g.gp_op_destroy(op)
    g.gp_ctx_destroy(ctx)


def test_an_allocation_that_fails_takes_every_contexts_kept_blocks(g):
    """A context asked for more than the device has fails with GP_ERR_OOM, after
    the blocks that another context keeps have gone back to the device."""
    import torch
    dims, K, R = (64, 64, 32), 6, 65535
    mask = np.ones(dims[::-1], dtype=np.uint8)
    N = mask.size
    stream = torch.cuda.current_stream().cuda_stream
    keeper, other = g.gp_ctx_create(0, stream, 0), g.gp_ctx_create(0, stream, 0)
    blocks = torch.eye(K, dtype=torch.float64, device="cuda")[None].repeat(N, 1, 1).contiguous()
    op = g.gp_op_create(other, mask, 6, K)
    g.gp_op_set_blocks(op, blocks)
    g.gp_op_set_alpha(op, np.ones(K))
    bw = torch.zeros((K, N), dtype=torch.float64, device="cuda")
    w = torch.zeros(1, dtype=torch.float64, device="cuda")   # not reached
    g.gp_op_destroy(g.gp_op_create(keeper, mask, 6, K))
    kept = 8 * N * K * (K + 1) // 2 * 4   # its blocks, factors and preconditioner, FP64 and FP32
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    assert R * K * N * 8 > torch.cuda.mem_get_info()[1]
    st = g.lib.gp_sample(op, R, bw.data_ptr(), None, None, w.data_ptr(), None, None)
    assert st == g.GP_ERR_OOM
    assert torch.cuda.mem_get_info()[0] >= before + kept
    assert g.gp_ctx_memory(keeper)[0] == 0
    g.gp_op_destroy(op)
    g.gp_ctx_destroy(keeper)
    g.gp_ctx_destroy(other)
