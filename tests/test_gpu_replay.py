"""Rounds that replay an operator's previous solves, of the Jacobi and
block-Jacobi solver: one shape per operator whatever items a batch has, idle
iterations bounded where the start values change, no iteration past the cap,
and the same answer whatever was replayed.  Iterations enqueued are the matvec
launches of a profiled solve, refinements the refine launches."""
import numpy as np
import pytest

from paper_1606_00980_amd import synth

pytestmark = pytest.mark.gpu

CHUNK = 6        # iterations of a planned FP64 round
REPLAYED = 16    # iterations replayed between looks at the states, from a start value


@pytest.fixture(scope="module")
def g(built_library):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    from paper_1606_00980_amd import gmrf
    return gmrf


@pytest.fixture()
def bench(g):
    """An operator, a right-hand side, its solution and the function that solves from given start values."""
    import torch
    w = synth.tiny((23, 19, 9), 6, 3, seed=17)
    ctx = g.gp_ctx_create(0, torch.cuda.current_stream().cuda_stream, 0)
    op = g.gp_op_create(ctx, w.mask, w.conn, w.K)
    B = torch.from_numpy(w.B).cuda()
    g.gp_op_set_blocks(op, B)
    g.gp_op_set_alpha(op, w.alpha)
    b = torch.from_numpy(np.random.default_rng(3).standard_normal((2, w.K, w.N))).cuda()

    def solve(starts, **kw):
        """One batch, an item per start value; (x, stats, iterations and refinements enqueued)."""
        o = g.gp_opts_default(**{"tol": 1e-10, "precision": g.GP_PREC_FP64, "rhs_tile": 4, **kw})
        xs = [s.clone() for s in starts]
        g.gp_ctx_profile(ctx, True)
        _, st = g.gp_solve_batch(ctx, [(op, 2, b, x) for x in xs], o, check=False)
        prof = g.gp_ctx_profile_read(ctx)
        g.gp_ctx_profile(ctx, False)
        return xs, st, prof["matvec"]["launches"], prof["refine"]["launches"]

    far = torch.zeros_like(b)
    near = solve([far], tol=1e-12, zero_guess=1)[0][0]
    yield solve, far, near
    torch.cuda.synchronize()
    g.gp_op_destroy(op)
    g.gp_ctx_destroy(ctx)


@pytest.mark.parametrize("order", [("far", "near"), ("near", "far")])
def test_items_of_one_operator_share_one_shape(g, bench, order):
    import torch
    solve, far, near = bench
    starts = [{"far": far, "near": near}[k] for k in order]
    first = solve(starts)
    again = solve(starts)
    most = max(s["inner_iters"] for s in again[1])
    assert most > CHUNK and min(s["inner_iters"] for s in again[1]) < most
    # exactly the iterations and refinements that the items need together
    assert again[2] == most
    assert again[3] == len({s["inner_iters"] for s in again[1]} | {0})
    for x, y in zip(first[0], again[0]):
        assert torch.equal(x, y)


def test_idle_iterations_after_other_start_values(g, bench):
    import torch
    solve, far, near = bench
    want, idle, seen = {}, {}, []
    for k in ("far", "far", "near", "near", "far", "near", "far", "near"):
        x, st, its, _ = solve([{"far": far, "near": near}[k]])
        want.setdefault(k, x[0])
        assert torch.equal(x[0], want[k])
        idle = its - max(s["inner_iters"] for s in st)
        assert idle <= REPLAYED
        if "near" in seen[-2:]:   # one of the last two solves was short
            assert idle < CHUNK
        seen.append(k)
    # from a zero start value, after solves from a given one
    x, st, its, _ = solve([far], zero_guess=1)
    x2, st2, its2, refines = solve([far], zero_guess=1)
    assert torch.equal(x[0], x2[0]) and its2 == max(s["inner_iters"] for s in st2)
    assert refines == len({s["inner_iters"] for s in st2} | {0})


@pytest.mark.parametrize("zero", [0, 1])
@pytest.mark.parametrize("cap", [1, 3, 7])
def test_a_cap_below_the_replayed_solve(g, bench, zero, cap):
    import torch
    solve, far, near = bench
    ref, sr, _, _ = solve([far], zero_guess=zero, max_iter=cap, chunk=4)   # a given chunk replays nothing
    solve([far], zero_guess=zero)
    x, st, its, _ = solve([far], zero_guess=zero, max_iter=cap)
    assert its == cap and all(s["status"] == g.GP_ERR_NOT_CONVERGED and s["inner_iters"] == cap for s in st)
    assert torch.equal(x[0], ref[0])
