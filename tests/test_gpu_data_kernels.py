"""GPU parity of the data-term kernels at the edges of their tilings, against
the explicit whitening of every scan (Appendix A.2) in NumPy: few scans (the
lag windows of the two ends overlap), voxel counts around a wavefront, every
AR order, K on both sides of the regressor chunk."""
import ctypes

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


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def whitened(Z, A, P):
    """Z[t] - sum_p A[p] Z[t - 1 - p] over the scans t = P .. T - 1 (Z: (T, ...), A: (P, N))."""
    out = Z[P:].copy()
    for p in range(P):
        out -= A[p] * Z[P - 1 - p:Z.shape[0] - 1 - p]
    return out


def problem(nx, K, T, P, Ns, seed):
    r = np.random.default_rng(seed)
    X = r.standard_normal((T, K))
    Y = r.standard_normal((T, nx))
    A = r.uniform(-0.4, 0.4, (Ns, P, nx))
    lam = r.uniform(0.5, 2.0, nx)
    return X, Y, A, lam


CASES = [(P, T, nx, K) for P in range(5) for T, nx, K in
         ((P + 1, 1, 1), (P + 2, 63, 2), (2 * P + 1, 64, 3), (2 * P + 2, 65, 5), (3 * P + 3, 130, 4), (41, 257, 9))]


@pytest.mark.parametrize("P,T,nx,K", CASES)
def test_tensors_at_the_edges(g, ctx, torch_cuda, P, T, nx, K):
    """b_w and, where they are positive definite, the blocks from the tensors."""
    X, Y, A, lam = problem(nx, K, T, P, 1, 100 * P + T + nx)
    op = g.gp_op_create(ctx, np.ones((1, 1, nx), dtype=np.uint8), 4, K)
    g.gp_op_set_alpha(op, np.zeros(K))
    d = g.gp_data_create(op, T, P, X, dev(torch_cuda, Y))
    bw = torch_cuda.zeros((K, nx), dtype=torch_cuda.float64, device="cuda")
    # per voxel whitened design and data
    Xw = whitened(np.repeat(X[:, :, None], nx, 2), A[0][:, None, :] if P else A[0], P)   # (T-P, K, N)
    Yw = whitened(Y, A[0], P)
    ref = lam * np.einsum("tkn,tn->kn", Xw, Yw)
    B = lam[:, None, None] * np.einsum("tkn,tln->nkl", Xw, Xw)
    spd = np.linalg.eigvalsh(B).min() > 1e-3
    scale = lam * np.einsum("tkn,tn->kn", np.abs(Xw), np.abs(Yw)) + 1.0
    try:
        g.gp_data_assemble(d, dev(torch_cuda, lam), 1, dev(torch_cuda, A) if P else None, bw)
        done = True
    except g.GmrfError as e:
        assert e.status == g.GP_ERR_NOT_SPD and not spd
        done = False
    # sums of at most 41 scans of order-one terms, expanded over (P + 1)^2 lag pairs
    assert (np.abs(bw.cpu().numpy() - ref) / scale).max() < 1e-12
    if done:
        x = np.random.default_rng(1).standard_normal((1, K, nx))
        y = torch_cuda.empty((1, K, nx), dtype=torch_cuda.float64, device="cuda")
        g.gp_apply(op, 1, dev(torch_cuda, x), y)
        want = np.einsum("nkl,ln->kn", B, x[0])
        assert np.abs(y.cpu().numpy()[0] - want).max() < 1e-12 * max(1.0, np.abs(B).max() * K * 10)
    g.gp_data_destroy(d)
    g.gp_op_destroy(op)


@pytest.mark.parametrize("P,Ns,nx,K", [(0, 1, 1, 1), (1, 2, 63, 2), (2, 3, 64, 3), (3, 1, 65, 4), (3, 5, 129, 15),
                                       (4, 2, 200, 6), (4, 1, 70, 24), (1, 4, 130, 17)])
def test_blocks_and_residual_sums_over_draws(g, ctx, torch_cuda, P, Ns, nx, K):
    """Blocks, b_w and residual sums of squares as means over draws of the whitened products."""
    T = 60
    X, Y, A, lam = problem(nx, K, T, P, Ns, 7 * P + Ns + nx + K)
    W = np.random.default_rng(K).standard_normal((Ns, K, nx))
    op = g.gp_op_create(ctx, np.ones((1, 1, nx), dtype=np.uint8), 4, K)
    g.gp_op_set_alpha(op, np.zeros(K))
    d = g.gp_data_create(op, T, P, X, dev(torch_cuda, Y))
    Ad = dev(torch_cuda, A) if P else None
    bw = torch_cuda.zeros((K, nx), dtype=torch_cuda.float64, device="cuda")
    g.gp_data_assemble(d, dev(torch_cuda, lam), Ns, Ad, bw)
    B, b, rss = np.zeros((nx, K, K)), np.zeros((K, nx)), np.zeros(nx)
    for j in range(Ns):
        Xw = whitened(np.repeat(X[:, :, None], nx, 2), A[j][:, None, :] if P else A[j], P)
        Yw = whitened(Y, A[j], P)
        B += lam[:, None, None] * np.einsum("tkn,tln->nkl", Xw, Xw) / Ns
        b += lam * np.einsum("tkn,tn->kn", Xw, Yw) / Ns
        rss += ((Yw - np.einsum("tkn,kn->tn", Xw, W[j])) ** 2).sum(0) / Ns
    assert np.abs(bw.cpu().numpy() - b).max() < 1e-12 * np.abs(b).max() * 10
    x = np.random.default_rng(1).standard_normal((1, K, nx))
    y = torch_cuda.empty((1, K, nx), dtype=torch_cuda.float64, device="cuda")
    g.gp_apply(op, 1, dev(torch_cuda, x), y)
    want = np.einsum("nkl,ln->kn", B, x[0])
    assert np.abs(y.cpu().numpy()[0] - want).max() < 1e-12 * np.abs(want).max() * 10
    out = [torch_cuda.empty(nx, dtype=torch_cuda.float64, device="cuda") for _ in range(3)]
    g.gp_data_lambda(d, Ns, dev(torch_cuda, W), Ad, 10.0, 0.1, *out)
    # the quadratic form cancels terms of up to about T K^2 against rss
    assert (np.abs(out[0].cpu().numpy() - rss) / rss).max() < 1e-14 * T * K * K
    u1t = 1.0 / (0.5 * out[0].cpu().numpy() + 0.1)
    assert np.allclose(out[1].cpu().numpy(), u1t, rtol=1e-14, atol=0)
    assert np.allclose(out[2].cpu().numpy(), u1t * (0.5 * (T - P) + 0.1), rtol=1e-14, atol=0)
    g.gp_data_destroy(d)
    g.gp_op_destroy(op)


@pytest.mark.parametrize("K,P,T", [(6, 3, 45), (15, 3, 31), (3, 4, 40), (5, 1, 140), (4, 2, 19), (2, 0, 23)])
def test_sums_over_scans_are_one_chain_each(g, ctx, torch_cuda, K, P, T):
    """Every sum over scans is one chain of fused multiply-adds, and B_n and b_w
    add their terms in the order of their definition: the bits of the same
    operations done here with libm's fma, at voxel counts of each split of the
    regressors (few, more and many wavefronts)."""
    torch = torch_cuda
    libm = ctypes.CDLL("libm.so.6")
    libm.fma.restype, libm.fma.argtypes = ctypes.c_double, [ctypes.c_double] * 3
    ufma = np.frompyfunc(libm.fma, 3, 1)

    def fma(x, y, z):
        return ufma(x, y, z).astype(np.float64)

    few, sizes = 20, (20, 64 * (400 // K) + 65, 64 * 801 + 7)
    X, Y, A, lam = problem(sizes[-1], K, T, P, 1, K + P)
    y, a, lm = Y[:, :few], A[0, :, :few], lam[:few]
    XX, YX = np.zeros((K, K)), np.zeros((K, few))
    R, S = np.zeros((K, K, P)), np.zeros((P, K, K, P))
    Bt, Dt = np.zeros((P, K, few)), np.zeros((P, K, P, few))
    for t in range(P, T):
        x, lx, ly = X[t], X[t - P:t][::-1], y[t - P:t][::-1]   # row p: t - 1 - p
        XX = fma(x[:, None], x, XX)
        YX = fma(y[t], x[:, None], YX)
        if P:
            R = fma(x[:, None, None], lx.T, R)
            S = fma(lx[:, :, None, None], lx.T, S)
            Bt = Bt + fma(y[t], lx[:, :, None], ly[:, None] * x[:, None])
            Dt = fma(ly[:, None, None], lx.T[:, :, None], Dt)
    B, b = np.zeros((few, K, K)), np.zeros((K, few))
    for p in range(P):
        b = fma(Bt[p], a[p], b)
        B = fma((R[..., p] + R[..., p].T), a[p][:, None, None], B)
        for q in range(P):
            b = fma(-Dt[p, :, q], a[p] * a[q], b)
            B = fma(-S[p, ..., q], (a[p] * a[q])[:, None, None], B)
    b = lm * (YX - b)
    B = lm[:, None, None] * (XX - B)
    B = 0.5 * (B + B.transpose(0, 2, 1))
    for nx in sizes:
        op = g.gp_op_create(ctx, np.ones((1, 1, nx), dtype=np.uint8), 4, K)
        g.gp_op_set_alpha(op, np.zeros(K))
        d = g.gp_data_create(op, T, P, X, dev(torch, Y[:, :nx]))
        bw = torch.zeros((K, nx), dtype=torch.float64, device="cuda")
        g.gp_data_assemble(d, dev(torch, lam[:nx]), 1, dev(torch, A[:, :, :nx]) if P else None, bw)
        unit = torch.eye(K, dtype=torch.float64, device="cuda")[:, :, None].expand(K, K, nx).contiguous()
        cols = torch.empty_like(unit)
        g.gp_apply(op, K, unit, cols)
        g.gp_data_destroy(d)
        g.gp_op_destroy(op)
        assert np.array_equal(bw[:, :few].cpu().numpy(), b), nx
        assert np.array_equal(cols[:, :, :few].cpu().numpy(), B.transpose(1, 2, 0)), nx


@pytest.mark.parametrize("K", [10, 13, 14, 15, 24])
def test_assembly_of_few_and_many_voxels(g, ctx, torch_cuda, K):
    """b_w and the blocks of a voxel do not depend on whether b_w is formed by
    the assembly's launch (few workgroups) or by its own (many, from K = 14)."""
    torch = torch_cuda
    nx, few, T, P = 13121, 500, 45, 2
    X, Y, A, lam = problem(nx, K, T, P, 2, K)
    got = []
    for n in (nx, few):
        op = g.gp_op_create(ctx, np.ones((1, 1, n), dtype=np.uint8), 4, K)
        d = g.gp_data_create(op, T, P, X, dev(torch, Y[:, :n]))
        bw = torch.full((K, n), float("nan"), dtype=torch.float64, device="cuda")
        g.gp_data_assemble(d, dev(torch, lam[:n]), 2, dev(torch, A[:, :, :n]), bw)
        g.gp_op_set_alpha(op, np.zeros(K))
        x, y = torch.ones((1, K, n), dtype=torch.float64, device="cuda"), torch.zeros((1, K, n), dtype=torch.float64,
                                                                                     device="cuda")
        g.gp_apply(op, 1, x, y)
        got.append((bw[:, :few].clone(), y[:, :, :few].clone()))
        g.gp_data_destroy(d)
        g.gp_op_destroy(op)
    assert torch.isfinite(got[0][0]).all()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
