"""GPU parity of the data-term kernels at the edges of their tilings, against
the explicit whitening of every scan (Appendix A.2) in NumPy: few scans (the
lag windows of the two ends overlap), voxel counts around a wavefront, every
AR order, K on both sides of the regressor chunk."""
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


@pytest.mark.parametrize("K,P,T,Ns", [(6, 3, 200, 1), (15, 3, 200, 5), (4, 1, 160, 2), (5, 0, 160, 1)])
def test_sums_over_scans_round_less_than_one_chain(g, ctx, torch_cuda, K, P, T, Ns):
    """b_w and the residual sums of data with a large mean, against 80-bit
    arithmetic, beside the same tensors summed scan by scan in one chain and
    combined in FP64 (NumPy).  A chain of n additions of like terms is off by
    about sqrt(n / 3) roundings of the whole, parts of 28 scans by about
    sqrt(28 / 3 / (n / 28) + n / 28 / 3): 0.25 of the chain at n = 200, with
    the few roundings of the combination on both sides under 0.6; b_w is held
    to 0.7 of the chain's error and the residual sums too."""
    torch = torch_cuda
    nx, q = 1000, np.longdouble
    r = np.random.default_rng(K + T)
    X = r.standard_normal((T, K))
    X[:, 0] = 1.0
    W = r.standard_normal((Ns, K, nx))
    W[:, 0] += 100.0
    Y = X @ W[0] + r.standard_normal((T, nx))
    A = r.uniform(-0.4, 0.4, (Ns, P, nx))
    lam = r.uniform(0.5, 2.0, nx)
    # sums over scans of y[t - a] X[t - b] and of y[t - a] y[t - b], one chain each
    C, D = np.zeros((P + 1, P + 1, K, nx)), np.zeros((P + 1, P + 1, nx))
    for t in range(P, T):
        for a in range(P + 1):
            for b in range(P + 1):
                C[a, b] += X[t - b][:, None] * Y[t - a]
                D[a, b] += Y[t - a] * Y[t - b]
    G = np.array([[X[P - a:T - a].T @ X[P - b:T - b] for b in range(P + 1)] for a in range(P + 1)])
    c = np.concatenate([np.ones((Ns, 1, nx)), -A], 1)
    cq, Xq, Yq = c.astype(q), X.astype(q), Y.astype(q)
    bw, bwq = np.zeros((K, nx)), np.zeros((K, nx), q)
    rss, rssq = np.zeros(nx), np.zeros(nx, q)
    for a in range(P, -1, -1):   # the small terms first
        for b in range(P, -1, -1):
            bw += (c[:, a] * c[:, b]).mean(0) * C[a, b]
            bwq += (cq[:, a] * cq[:, b]).mean(0) * (Xq[P - b:T - b].T @ Yq[P - a:T - a])
            for j in range(Ns):
                quad = (W[j] * (G[a, b] @ W[j])).sum(0)
                rss += c[j, a] * c[j, b] * (D[a, b] - 2.0 * (C[a, b] * W[j]).sum(0) + quad)
    bw, bwq, rss = lam * bw, lam.astype(q) * bwq, rss / Ns
    for j in range(Ns):
        e = Yq - Xq @ W[j].astype(q)
        f = sum(cq[j, a] * e[P - a:T - a] for a in range(P + 1))
        rssq += (f * f).sum(0) / Ns
    op = g.gp_op_create(ctx, np.ones((1, 1, nx), dtype=np.uint8), 4, K)
    g.gp_op_set_alpha(op, np.zeros(K))
    d = g.gp_data_create(op, T, P, X, dev(torch, Y))
    out = torch.zeros((K, nx), dtype=torch.float64, device="cuda")
    res = torch.zeros(nx, dtype=torch.float64, device="cuda")
    Ad = dev(torch, A) if P else None
    g.gp_data_assemble(d, dev(torch, lam), Ns, Ad, out)
    g.gp_data_lambda(d, Ns, dev(torch, W), Ad, 10.0, 0.1, res, None, None)
    g.gp_data_destroy(d)
    g.gp_op_destroy(op)

    def off(v, ref):
        return float(np.sqrt(((v - ref) ** 2).sum() / (ref ** 2).sum()))

    assert off(out.cpu().numpy(), bwq) <= 0.7 * off(bw, bwq)
    assert off(res.cpu().numpy(), rssq) <= 0.7 * off(rss, rssq)


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
