"""What is timed: the calls that programs make of this library, over their real range of sizes.

A case names one public call (or the short sequence of calls that makes one
iteration of a user's program) on one synthetic fMRI operator.  The operators
are those of the repository's own workloads -- the 64 x 64 slice (K = 2), the
52,740-voxel whole brain (K = 6; K = 15 as the paper's real data), the uneven
operators up to N = 289,592 and K = 10 -- and generic ones of odd sizes drawn
between them.  Inputs are made on the GPU from the seed: design matrix, AR(P)
noise, data Y, blocks B_n and b_w as the model has them.
"""
import math

import numpy as np
import torch

from paper_1606_00980_amd import gmrf as g
from paper_1606_00980_amd import synth

PRECOND = {"jacobi": g.GP_PRECOND_JACOBI, "block": g.GP_PRECOND_BLOCK_JACOBI, "rb": g.GP_PRECOND_RB_IC0}
PRECISION = {"fp64": g.GP_PREC_FP64, "fp32": g.GP_PREC_FP32_REFINE64}
GOLDEN = 0x9E3779B97F4A7C15
M64 = (1 << 64) - 1

BRAIN = {"nx": 64, "ny": 64, "nz": 33, "ax": 28.0, "ay": 30.0, "az": 15.0}
LARGEST = {"nx": 96, "ny": 96, "nz": 60, "ax": 48.0, "ay": 48.0, "az": 30.0}


def _axes(nx, ny, nz, fill):
    """Semi-axes of an ellipsoid that fills the given part of its box."""
    c = (6.0 * fill / math.pi) ** (1.0 / 3.0)
    return {"nx": nx, "ny": ny, "nz": nz, "ax": min(0.5 * nx * c, 0.5 * nx), "ay": min(0.5 * ny * c, 0.5 * ny),
            "az": min(0.5 * nz * c, 0.5 * nz)}


def listed():
    return [
        # one 2D slice (the slice-wise analysis): a mean and a sample in FP64 to 1e-10; the smallest solves, where
        # latency and launches count
        {"name": "slice_mean_sample_fp64", "kind": "mean_sample", "nx": 64, "ny": 64, "nz": 1, "ax": 28.0, "ay": 28.0,
         "az": 1.0, "K": 2, "P": 1, "T": 160, "R": 1, "precond": "jacobi", "precision": "fp64", "tol": 1e-10},
        # the posterior mean of one whole brain in plain FP64: one right-hand side, the library's block Jacobi
        {"name": "brain_mean_fp64", "kind": "solve", **BRAIN, "K": 6, "P": 3, "T": 200, "R": 1, "precond": "block",
         "precision": "fp64", "tol": 1e-8},
        # an operator applied to a few vectors (residual checks, a caller's own iteration)
        {"name": "apply_r8", "kind": "apply", **BRAIN, "K": 6, "P": 3, "T": 200, "R": 8},
        # Algorithm 2 with the library's default options and random vectors drawn on the device
        {"name": "brain_sample_r16_default", "kind": "sample", **BRAIN, "K": 6, "P": 3, "T": 200, "R": 16,
         "precond": "block", "precision": "fp32", "tol": 1e-8},
        # one iteration of the Gibbs chain on the whole brain: one draw of W from the previous one, alpha, lambda
        {"name": "gibbs_brain", "kind": "gibbs", **BRAIN, "K": 6, "P": 3, "T": 200, "R": 1, "precond": "rb",
         "precision": "fp32", "tol": 1e-8},
        # one spatial VB iteration at the paper's real-data K = 15 with few Monte Carlo samples (its first iterations)
        {"name": "svb_brain_k15", "kind": "svb", **BRAIN, "K": 15, "P": 3, "T": 200, "R": 5, "precond": "rb",
         "precision": "fp32", "tol": 1e-8},
        # a new dataset: its time-summed tensors and the first data term from them
        {"name": "dataset_brain_k15", "kind": "dataset", **BRAIN, "K": 15, "P": 3, "T": 200, "R": 1},
        # the batched VB step of the benchmark: data term, 32 samples and 32 probes in one solve, the trace
        {"name": "brain_step_r64", "kind": "step", **BRAIN, "K": 6, "P": 3, "T": 200, "R": 64, "precond": "rb",
         "precision": "fp32", "tol": 1e-8},
        # a trace estimate in FP64 on a middling operator of odd sizes
        {"name": "trace_fp64_odd", "kind": "trace", **_axes(45, 47, 29, 0.47), "K": 5, "P": 3, "T": 200, "R": 16,
         "precond": "rb", "precision": "fp64", "tol": 1e-8},
        # sixteen subjects of different sizes and K = 2..10 in one grouped solve, samples, probes and traces
        {"name": "uneven16", "kind": "uneven", "ops": 16, "R": 8, "precond": "rb", "precision": "fp32", "tol": 1e-8,
         "P": 3, "T": 200, "smin": 1.0, "smax": 3.0},
        # the largest operator with many right-hand sides: a working set of gigabytes
        {"name": "largest_k10_r64", "kind": "solve", **LARGEST, "K": 10, "P": 3, "T": 200, "R": 64, "precond": "rb",
         "precision": "fp32", "tol": 1e-8},
        # a burst of mixed requests (solve, sample, trace) to the serving loop over six resident operators
        {"name": "serve_burst", "kind": "serve", "ops": 6, "requests": 30, "R": 8, "precond": "rb",
         "precision": "fp32", "tol": 1e-8, "P": 3, "T": 200, "smin": 1.0, "smax": 2.0},
    ]


def draw(rng):
    def log_int(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    kind = rng.choice(["mean_sample", "solve", "solve", "apply", "sample", "gibbs", "svb", "dataset", "step", "trace",
                       "uneven", "serve"])
    tol = {"fp64": rng.choice([1e-8, 1e-10]), "fp32": 1e-8}
    if kind in ("uneven", "serve"):
        lo = rng.uniform(0.6, 1.2)
        c = {"kind": kind, "ops": rng.randint(3, 16 if kind == "uneven" else 6), "R": rng.choice([2, 4, 6, 8]),
             "precond": rng.choice(["rb", "rb", "block"]), "precision": "fp32", "tol": 1e-8, "P": 3, "T": 200,
             "smin": lo, "smax": lo + rng.uniform(0.3, 1.2)}
        if kind == "serve":
            c["requests"] = rng.randint(6, 30)
        return c
    if kind == "mean_sample":   # a slice
        n = rng.randint(24, 96)
        r = round(n * rng.uniform(0.38, 0.49), 2)
        precision = rng.choice(["fp64", "fp64", "fp32"])
        return {"kind": kind, "nx": n, "ny": n, "nz": 1, "ax": r, "ay": r, "az": 1.0, "K": rng.randint(1, 6), "P": 1,
                "T": 160, "R": rng.choice([1, 1, 2, 5]), "precond": rng.choice(["jacobi", "block", "rb"]),
                "precision": precision, "tol": tol[precision]}
    s = math.exp(rng.uniform(math.log(0.5), math.log(2.6)))
    dims = [max(5, int(round(s * d)) + rng.randint(-3, 3)) for d in (32, 32, 20)]
    box = _axes(*dims, rng.uniform(0.4, 0.6))
    cells = 0.5 * dims[0] * dims[1] * dims[2]
    K = rng.randint(2, 10)
    if kind in ("svb", "dataset"):
        K = rng.randint(2, 16)
        K = max(2, min(K, int(1.6e6 / cells)))
    c = {"kind": kind, **box, "K": K, "P": rng.choice([1, 3, 3]), "T": rng.choice([160, 200])}
    most = {"solve": 64, "apply": 32, "sample": 32, "gibbs": 1, "svb": 10, "dataset": 1, "step": 64, "trace": 32}[kind]
    R = min(log_int(1, most), max(1, int(4.0e7 / (cells * K))))
    if kind == "gibbs":
        R = 1
    if kind == "step":
        R = max(2, R // 2 * 2)
    c["R"] = R
    if kind not in ("apply", "dataset"):
        precision = rng.choice(["fp32", "fp32", "fp64"])
        c.update(precond=rng.choice(["rb", "rb", "block"]), precision=precision, tol=tol[precision])
    return c


# ------------------------------------------------------------------ inputs
def _dims(case):
    """One (dims, axes, K) per operator of the case."""
    if case["kind"] not in ("uneven", "serve"):
        return [(case, case["K"])]
    r = np.random.default_rng([7, case["ops"], int(1000 * case["smin"]), int(1000 * case["smax"])])
    out = []
    for _ in range(case["ops"]):
        s = r.uniform(case["smin"], case["smax"])
        out.append((_axes(*(int(round(s * d)) for d in (32, 32, 20)), r.uniform(0.4, 0.6)), int(r.integers(2, 11))))
    return out


def _mask(box):
    return synth.ellipsoid_mask((box["nx"], box["ny"], box["nz"]), (box["ax"], box["ay"], box["az"]))


class Model:
    """The data of one operator: mask, design, AR coefficients, noise variances, Y, blocks and b_w."""

    def __init__(self, case, box, K, seed, data=False):
        self.mask = _mask(box)
        self.K, self.P, self.T = K, case["P"], case["T"]
        self.conn = 4 if box["nz"] == 1 else 6
        N = self.N = int(self.mask.sum())
        self.dirs = 2 if self.conn == 4 else 3
        r = np.random.default_rng([11, seed % (1 << 31)])
        t = self.torch = torch.Generator(device="cuda")
        t.manual_seed(seed)
        dev = {"device": "cuda", "dtype": torch.float64}
        if K >= 2:
            self.X, roles = synth.design_matrix(K, self.T, "uneven")
        else:
            self.X, roles = np.ones((self.T, 1)), ["const"]
        X = torch.from_numpy(np.ascontiguousarray(self.X)).cuda()
        self.alpha = r.gamma(2.0, 1.0, size=K)
        if self.P == 1:
            self.ar = 0.2 + 0.3 * torch.rand((1, N), generator=t, **dev)
        else:
            self.ar = torch.from_numpy(synth.pacf_to_ar(r.uniform(-0.5, 0.5, size=(self.P, N)))).cuda()
        self.lam = 1.0 / (0.5 + 1.5 * torch.rand(N, generator=t, **dev))
        W = torch.zeros((K, N), **dev)
        lin = np.flatnonzero(self.mask.ravel())
        for k, role in enumerate(roles):
            if role == "task":
                W[k] = torch.from_numpy(synth._blob(self.mask, int(lin[r.integers(0, N)]), 4.0, 2.0)).cuda()
            elif role == "const":
                W[k] = 100.0 + 14.4 * torch.randn(N, generator=t, **dev)
        Y = X @ W
        sd, past = self.lam.rsqrt(), [torch.zeros(N, **dev) for _ in range(self.P)]
        for i in range(-20, self.T):
            e = torch.randn(N, generator=t, **dev) * sd
            for p in range(self.P):
                e += self.ar[p] * past[p]
            past = [e] + past[:-1]
            if i >= 0:
                Y[i] += e
        self.Xd = X
        self.B, self.bw = _data_term(X, Y, self.ar[None], self.lam)
        self.Y = Y if data else None

    def normal(self, *shape):
        return torch.randn(shape, generator=self.torch, device="cuda", dtype=torch.float64)

    def signs(self, *shape):
        return (2 * torch.randint(0, 2, shape, generator=self.torch, device="cuda", dtype=torch.int8) - 1)


def _data_term(X, Y, A, lam):
    """B_n and b_n by whitening with (1, -a_1, .., -a_P), mean over the draws A [Ns][P][N]."""
    P, T = A.shape[1], X.shape[0]
    c = torch.cat([torch.ones_like(A[:, :1]), -A], 1)
    K, N = X.shape[1], Y.shape[1]
    B = torch.zeros((N, K, K), device=X.device, dtype=X.dtype)
    bw = torch.zeros((K, N), device=X.device, dtype=X.dtype)
    for p in range(P + 1):
        for q in range(P + 1):
            cc = (c[:, p] * c[:, q]).mean(0) * lam
            B += cc[:, None, None] * (X[P - p:T - p].T @ X[P - q:T - q])[None]
            bw += cc[None] * (X[P - p:T - p].T @ Y[P - q:T - q])
    return 0.5 * (B + B.transpose(1, 2).contiguous()), bw


class State(dict):
    """What a program holds: handles and buffers, given back together."""

    def __del__(self):
        torch.cuda.synchronize()
        if "srv" in self:
            g.gp_server_destroy(self["srv"])
        if "data" in self:
            g.gp_data_destroy(self["data"])
        for op in self.get("ops", []):
            g.gp_op_destroy(op)
        if "ctx" in self:
            g.gp_ctx_destroy(self["ctx"])


def _opts(case, **more):
    return g.gp_opts_default(tol=case["tol"], precond=PRECOND[case["precond"]], precision=PRECISION[case["precision"]],
                             **more)


def _models(case, seed, data=False):
    return [Model(case, box, K, 1000 * seed + i, data) for i, (box, K) in enumerate(_dims(case))]


def _inputs(case, seed):
    """The models and the random vectors of the call, from the seed alone."""
    kind, R = case["kind"], case["R"]
    ms = _models(case, seed, kind in ("gibbs", "svb", "dataset", "step"))
    v = {}
    m = ms[0]
    if kind in ("mean_sample", "solve"):
        v["b"] = m.bw + m.normal(R, m.K, m.N)
    if kind in ("mean_sample", "svb"):
        v["z1"], v["z2"] = m.normal(R, m.K, m.dirs, m.N), m.normal(R, m.K, m.N)
    if kind == "step":
        v["z1"], v["z2"] = m.normal(R // 2, m.K, m.dirs, m.N), m.normal(R // 2, m.K, m.N)
        v["probes"] = m.signs(R // 2, m.K, m.N)
    if kind == "trace":
        v["probes"] = m.signs(R, m.K, m.N)
    if kind in ("apply", "dataset"):
        v["x"] = m.normal(R, m.K, m.N)
    if kind == "svb":
        v["A"] = m.ar[None] + 0.03 * m.normal(R, m.P, m.N)
    if kind in ("gibbs", "svb"):
        # the state of a running chain: W near its mean, alpha and lambda off theirs
        v["W"] = m.bw[None] / m.B.diagonal(dim1=1, dim2=2).T[None] * (1 + 0.1 * m.normal(R, m.K, m.N))
        v["alpha"] = m.alpha.copy()
        v["lam"] = m.lam * (1 + 0.1 * torch.rand(m.N, generator=m.torch, device="cuda", dtype=torch.float64))
    if kind == "uneven":
        v["z"] = [(m.normal(R // 2, m.K, m.dirs, m.N), m.normal(R // 2, m.K, m.N)) for m in ms]
        v["pr"] = [m.signs(R - R // 2, m.K, m.N) for m in ms]
    if kind == "serve":
        v["req"] = [(i % 3, (i * 5 + i // 3) % len(ms), 977 * seed + i) for i in range(case["requests"])]
    v["seed"] = 77 + seed
    return ms, v


def prepare(case, seed):
    ms, v = _inputs(case, seed)
    kind, R = case["kind"], case["R"]
    s = State(case=case, kind=kind, R=R, keep=[m.bw for m in ms], **v)
    s["ctx"] = g.gp_ctx_create(0, torch.cuda.current_stream().cuda_stream, 0)
    s["ops"] = []
    for m in ms:
        op = g.gp_op_create(s["ctx"], m.mask, m.conn, m.K)
        s["ops"].append(op)
        g.gp_op_set_blocks(op, m.B)
        g.gp_op_set_alpha(op, m.alpha)
    m, op = ms[0], s["ops"][0]
    s.update(op=op, K=m.K, N=m.N, P=m.P, T=m.T, bw=m.bw)
    new = lambda *shape: torch.zeros(shape, device="cuda", dtype=torch.float64)  # noqa: E731
    if "tol" in case:
        s["opts"] = _opts(case, zero_guess=0 if kind in ("gibbs", "svb", "sample") else 1, seed=v["seed"])
    if kind in ("solve", "mean_sample", "sample", "trace", "step"):
        s["out"] = new(R, m.K, m.N)
    if kind == "mean_sample":
        s["w"] = new(R, m.K, m.N)
    if kind in ("apply", "dataset"):
        s["out"] = new(R, m.K, m.N)
    if kind in ("gibbs", "svb", "dataset", "step"):
        s.update(X=m.X, Y=m.Y, ar=m.ar[None].contiguous(), lam0=v.get("lam", m.lam), bww=new(m.K, m.N), alpha=m.alpha)
    if kind in ("gibbs", "svb", "step"):
        s["data"] = g.gp_data_create(op, m.T, m.P, m.X, m.Y)
    if kind in ("gibbs", "svb"):
        s.update(Ww=torch.empty_like(v["W"]), lamw=torch.empty_like(v["lam"]))
    if kind == "step":
        s["rhs"] = new(R, m.K, m.N)
    if kind == "uneven":
        s["models"] = [(m.K, m.alpha) for m in ms]
        s["B"] = [m.B for m in ms]
        s["rhs"] = [new(R, m.K, m.N) for m in ms]
        s["xs"] = [new(R, m.K, m.N) for m in ms]
    if kind == "serve":
        s["outs"] = [new(*((R,) if k == g.GP_REQ_TRACE else (1,)), ms[i].K, ms[i].N) for k, i, _ in v["req"]]
        s["Ks"] = [m.K for m in ms]
        s["srv"] = g.gp_server_create(s["ctx"], s["ops"], [m.bw for m in ms],
                                      g.gp_server_cfg_default(probes=R, opts=_opts(case)))
    return s


# --------------------------------------------------------------------- run
def run(s):
    return globals()["_run_" + s["kind"]](s)


def _run_solve(s):
    g.gp_solve(s["op"], s["R"], s["b"], s["out"], s["opts"])
    return s["out"]


def _run_mean_sample(s):
    g.gp_solve(s["op"], s["R"], s["b"], s["out"], s["opts"])
    g.gp_sample(s["op"], s["R"], s["bw"], s["z1"], s["z2"], s["w"], s["opts"])
    return s["out"], s["w"]


def _run_sample(s):
    s["out"].zero_()
    g.gp_sample(s["op"], s["R"], s["bw"], None, None, s["out"], s["opts"])
    return s["out"]


def _run_apply(s):
    g.gp_apply(s["op"], s["R"], s["x"], s["out"])
    return s["out"]


def _run_trace(s):
    t, tk, gk, _ = g.gp_trace(s["op"], s["R"], s["probes"], s["out"], s["K"], s["opts"])
    return s["out"], t, tk, gk


def _run_gibbs(s):
    # one iteration from the same state of the chain
    s["Ww"].copy_(s["W"])
    s["lamw"].copy_(s["lam"])
    a = s["alpha"].copy()
    g.gp_gibbs_step(s["data"], s["ar"][0], None, None, s["Ww"], s["lamw"], a, s["bww"], s["seed"], 5, None, s["opts"])
    return s["Ww"], s["lamw"], a


def _run_svb(s):
    s["Ww"].copy_(s["W"])
    s["lamw"].copy_(s["lam"])
    a = s["alpha"].copy()
    g.gp_svb_step(s["data"], s["R"], s["A"], s["z1"], s["z2"], s["Ww"], s["lamw"], a, s["bww"], None, s["opts"])
    return s["Ww"], s["lamw"], a


def _run_dataset(s):
    d = g.gp_data_create(s["op"], s["T"], s["P"], s["X"], s["Y"])
    g.gp_data_assemble(d, s["lam0"], 1, s["ar"], s["bww"])
    g.gp_data_destroy(d)
    g.gp_apply(s["op"], s["R"], s["x"], s["out"])
    return s["bww"], s["out"]


def _run_step(s):
    h, K, N = s["R"] // 2, s["K"], s["N"]
    g.gp_data_assemble(s["data"], s["lam0"], 1, s["ar"], s["bww"])
    g.gp_op_set_alpha(s["op"], s["alpha"])
    g.gp_perturb_rhs(s["op"], h, s["bww"], s["z1"], s["z2"], s["rhs"][:h])
    g.gp_probe_rhs(s["op"], h, s["probes"], s["rhs"][h:])
    g.gp_solve_batch(s["ctx"], [(s["op"], h, s["rhs"][:h], s["out"][:h]), (s["op"], h, s["rhs"][h:], s["out"][h:])],
                     s["opts"])
    t, tk, gk = g.gp_trace_reduce(s["op"], h, s["probes"], s["out"][h:], K)
    return s["out"], t, tk, gk


def _run_uneven(s):
    h = s["R"] // 2
    items = []
    for i, op in enumerate(s["ops"]):
        g.gp_op_set_blocks(op, s["B"][i])
        g.gp_op_set_alpha(op, s["models"][i][1])
        g.gp_perturb_rhs(op, h, s["keep"][i], *s["z"][i], s["rhs"][i][:h])
        g.gp_probe_rhs(op, s["R"] - h, s["pr"][i], s["rhs"][i][h:])
        items += [(op, h, s["rhs"][i][:h], s["xs"][i][:h]), (op, s["R"] - h, s["rhs"][i][h:], s["xs"][i][h:])]
    g.gp_solve_batch(s["ctx"], items, s["opts"])
    tr = []
    for i, op in enumerate(s["ops"]):
        t, tk, gk = g.gp_trace_reduce(op, s["R"] - h, s["pr"][i], s["xs"][i][h:], s["models"][i][0])
        tr.append(np.concatenate([[t], tk, gk]))
    return s["xs"], tr


def _run_serve(s):
    at = {}
    for j, (kind, i, seed) in enumerate(s["req"]):
        at[g.gp_server_submit(s["srv"], kind, i, seed, s["outs"][j])] = j
    g.gp_server_drain(s["srv"])
    tr = [None] * len(s["req"])
    for r in g.gp_server_poll(s["srv"]):
        if r["status"] != g.GP_OK:
            raise RuntimeError("request failed with status %d" % r["status"])
        K = s["Ks"][r["op_index"]]
        if r["kind"] == g.GP_REQ_TRACE:
            tr[at[r["ticket"]]] = np.concatenate([[r["trace_total"]], r["trace_kk"][:K], r["trace_Gkk"][:K]])
    return s["outs"], np.concatenate([t for t in tr if t is not None])


# -------------------------------------------------------------------- work
def work(case):
    """Bytes: each input read once, each output written once.  Flops: the operator and preconditioner products of a
    usual number of iterations (7 with the red-black factor, 13 with block Jacobi, 60 with Jacobi)."""
    kind, R = case["kind"], case["R"]
    by = fl = 0.0
    for box, K in _dims(case):
        N = int(_mask(box).sum())
        NB, dirs = K * (K + 1) // 2, 2 if box["nz"] == 1 else 3
        v = 8.0 * K * N
        P, T = case["P"], case["T"]
        tens = 8.0 * N * (K + P * K + P * K * P + 1 + P + P * P)
        per = N * (14.0 * K + 6.0 * K * K)
        its = {"rb": 7, "block": 13, "jacobi": 60}.get(case.get("precond"), 1)
        by += 8.0 * NB * N
        if kind in ("solve", "trace"):
            by += R * 2 * v if kind == "solve" else R * (v + v / 8)
            fl += its * R * per
        elif kind == "mean_sample":
            by += R * v * (3 + dirs + 1) + v
            fl += 2 * its * R * per
        elif kind == "sample":
            by += R * v + v
            fl += R * (its * per + 200.0 * K * N * (dirs + 1))
        elif kind == "apply":
            by += R * 2 * v
            fl += R * N * (14.0 * K + 2.0 * K * K)
        elif kind == "gibbs":
            by += tens + 2 * v + 8.0 * N * (P + 2)
            fl += its * per + N * (2.0 * P * P * K * K)
        elif kind == "svb":
            by += tens + R * v * (2 + dirs + 1) + 8.0 * N * (R * P + 2)
            fl += R * (its * per + N * 2.0 * (P + 1) * K * K) + N * (2.0 * P * P * K * K)
        elif kind == "dataset":
            by += 8.0 * T * N + tens + v * (1 + 2 * R) + 8.0 * N * (P + 1)
            fl += 2.0 * T * N * K * (2 * P + 1) + N * (2.0 * P * P * K * K)
        elif kind == "step":
            by += tens + (R // 2) * v * (dirs + 1 + 1.0 / 8) + R * v
            fl += its * R * per
        elif kind == "uneven":
            by += 8.0 * N * (K * K - NB) + (R // 2) * v * (dirs + 1 + 1.0 / 8) + R * v + v
            fl += its * R * per
        elif kind == "serve":
            n = case["requests"] / case["ops"]
            by += n * v * (2 + R) / 3 + v
            fl += n * its * per * (2 + R) / 3
    return {"bytes": by, "flops": fl}


# ------------------------------------------------------------------- exact
class Exact:
    """The operator of one model in plain torch, FP64."""

    def __init__(self, m, B, alpha):
        self.K, self.N, self.dirs, self.B = m.K, m.N, m.dirs, B
        self.alpha = torch.as_tensor(alpha, device="cuda", dtype=torch.float64)
        idx = torch.full(m.mask.shape, -1, dtype=torch.int64)
        idx[torch.from_numpy(m.mask != 0)] = torch.arange(m.N)
        pad = torch.full([d + 2 for d in m.mask.shape], -1, dtype=torch.int64)
        pad[1:-1, 1:-1, 1:-1] = idx
        own = torch.from_numpy(m.mask != 0)
        nb = []
        for d in range(m.dirs):
            ax = 2 - d
            for step in (-1, 1):
                nb.append(torch.roll(pad, -step, ax)[1:-1, 1:-1, 1:-1][own])
        self.nb = [n.cuda() for n in nb]   # -x, +x, -y, +y, (-z, +z); -1 outside
        self.has = [n >= 0 for n in self.nb]
        self.deg = sum(h.double() for h in self.has)
        M = B.clone()
        M.diagonal(dim1=1, dim2=2).add_(self.deg[:, None] * self.alpha[None])
        self.Minv = self.inverse(M)

    @staticmethod
    def cholesky(B):
        """L of every block, column by column."""
        K = B.shape[1]
        L = torch.zeros_like(B)
        for j in range(K):
            L[:, j, j] = (B[:, j, j] - (L[:, j, :j] ** 2).sum(1)).sqrt()
            for i in range(j + 1, K):
                L[:, i, j] = (B[:, i, j] - (L[:, i, :j] * L[:, j, :j]).sum(1)) / L[:, j, j]
        return L

    @classmethod
    def inverse(cls, M):
        """Inverse of every SPD block through its Cholesky factor."""
        L, K = cls.cholesky(M), M.shape[1]
        Li = torch.zeros_like(L)
        for c in range(K):
            for i in range(c, K):
                Li[:, i, c] = ((1.0 if i == c else 0.0) - (L[:, i, c:i] * Li[:, c:i, c]).sum(1)) / L[:, i, i]
        out = torch.empty_like(M)
        for i in range(K):
            for j in range(K):
                out[:, i, j] = (Li[:, :, i] * Li[:, :, j]).sum(1)
        return out

    def blocks(self, S, v):
        y = torch.empty_like(v)
        for k in range(self.K):
            y[:, k] = S[:, k, 0] * v[:, 0]
            for j in range(1, self.K):
                y[:, k].addcmul_(S[:, k, j], v[:, j])
        return y

    def laplace(self, v):
        y = self.deg * v
        for n, h in zip(self.nb, self.has):
            y -= torch.where(h, v[..., n.clamp(min=0)], 0.0)
        return y

    def apply(self, v):
        return self.blocks(self.B, v).addcmul_(self.alpha[None, :, None].expand_as(v), self.laplace(v))

    def solve(self, b):
        """Block-Jacobi PCG, restarted from the true residual until it no longer falls."""
        out = torch.empty_like(b)
        per = max(1, int(4e7 / (self.K * self.N)))
        for r0 in range(0, b.shape[0], per):
            out[r0:r0 + per] = self._solve(b[r0:r0 + per])
        return out

    def _solve(self, b):
        dot = lambda u, v: (u * v).sum((1, 2), keepdim=True)  # noqa: E731
        x = torch.zeros_like(b)
        for _ in range(3):
            r = b - self.apply(x)
            z = self.blocks(self.Minv, r)
            p, rz = z.clone(), dot(r, z)
            stop = 1e-9 * dot(r, r).sqrt()
            for it in range(600):
                q = self.apply(p)
                a = rz / dot(p, q).clamp(min=1e-300)
                x += a * p
                r -= a * q
                if it % 4 == 3 and bool((dot(r, r).sqrt() <= stop).all()):
                    break
                z = self.blocks(self.Minv, r)
                new = dot(r, z)
                p = z + new / rz.clamp(min=1e-300) * p
                rz = new
        return x

    def perturbed(self, bw, z1, z2):
        """Algorithm 2, step 4."""
        L = self.cholesky(self.B)
        b = bw[None] + self.blocks(L, z2)
        for d in range(self.dirs):
            lo, up = self.nb[2 * d], self.nb[2 * d + 1]
            e = torch.where(up >= 0, z1[:, :, d], 0.0) - torch.where(lo >= 0, z1[:, :, d][..., lo.clamp(min=0)], 0.0)
            b += self.alpha.sqrt()[None, :, None] * e
        return b

    def quad(self, W):
        return (W * self.laplace(W)).sum(2)

    def traces(self, v, u):
        v = v.double()
        kk, gg = (v * u).sum(2).mean(0), (self.laplace(v) * u).sum(2).mean(0)
        return kk.sum().item(), kk.cpu().numpy(), gg.cpu().numpy()


def _words(seed, stream, q):
    """Philox4x32-10 words of the blocks q (int64 tensor), as int64 values below 2^32."""
    m = 0xFFFFFFFF
    c = [q & m, q >> 32, torch.full_like(q, stream & m), torch.full_like(q, (stream >> 32) & m)]
    k0, k1 = seed & m, (seed >> 32) & m
    for i in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & m) ^ c[1] ^ k0, p1 & m, ((p0 >> 32) & m) ^ c[3] ^ k1, p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c


def _uniform(lo, hi):
    return ((((hi << 32) | lo) >> 11 & ((1 << 53) - 1)).double() + 0.5) * 2.0 ** -53


def _normals(seed, stream, *shape):
    n = math.prod(shape)
    w = _words(seed, stream, torch.arange((n + 1) // 2, device="cuda"))
    rad, ang = (-2.0 * torch.log(_uniform(w[0], w[1]))).sqrt(), 2.0 * math.pi * _uniform(w[2], w[3])
    return torch.stack([rad * torch.cos(ang), rad * torch.sin(ang)], 1).reshape(-1)[:n].reshape(shape)


def _signs(seed, stream, *shape):
    n = math.prod(shape)
    w = torch.stack(_words(seed, stream, torch.arange((n + 127) // 128, device="cuda")), 1)
    bits = (w[:, :, None] >> torch.arange(32, device="cuda")) & 1
    return (2 * bits.reshape(-1)[:n] - 1).to(torch.int8).reshape(shape)


def _gamma(seed, stream, shape, scale):
    """Marsaglia and Tsang's draws (shape > 1)."""
    n, d = scale.numel(), shape - 1.0 / 3.0
    c = 1.0 / math.sqrt(9.0 * d)
    out, todo = torch.full((n,), d, device="cuda", dtype=torch.float64), torch.arange(n, device="cuda")
    for t in range(64):
        w = _words(seed, stream, 128 * todo + 2 * t)
        x = (-2.0 * torch.log(_uniform(w[0], w[1]))).sqrt() * torch.cos(2.0 * math.pi * _uniform(w[2], w[3]))
        w = _words(seed, stream, 128 * todo + 2 * t + 1)
        u, v = _uniform(w[0], w[1]), (1.0 + c * x) ** 3
        ok = (v > 0) & ((u < 1.0 - 0.0331 * x ** 4) |
                        (torch.log(u) < 0.5 * x * x + d * (1.0 - v + torch.log(v.clamp(min=1e-300)))))
        out[todo[ok]] = d * v[ok]
        todo = todo[~ok]
        if not todo.numel():
            break
    return out * scale


def _residual_ss(m, W, A):
    """Whitened residual sum of squares of every pair, mean over the pairs."""
    tot = torch.zeros(m.N, device="cuda", dtype=torch.float64)
    for j in range(W.shape[0]):
        e = m.Y - m.Xd @ W[j]
        f = e[m.P:].clone()
        for p in range(m.P):
            f -= A[j, p] * e[m.P - 1 - p:m.T - 1 - p]
        tot += (f * f).sum(0)
    return tot / W.shape[0]


def exact(case, seed):
    ms, v = _inputs(case, seed)
    kind, R, m = case["kind"], case["R"], ms[0]
    if kind == "uneven":
        xs, tr = [], []
        for i, m in enumerate(ms):
            E, h = Exact(m, m.B, m.alpha), R // 2
            xs.append(E.solve(torch.cat([E.perturbed(m.bw, *v["z"][i]), v["pr"][i].double()])))
            t, tk, gk = E.traces(v["pr"][i], xs[-1][h:])
            tr.append(np.concatenate([[t], tk, gk]))
        return xs, tr
    if kind == "serve":
        Es, outs, tr = [Exact(m, m.B, m.alpha) for m in ms], [], []
        for k, i, sd in v["req"]:
            m, E = ms[i], Es[i]
            if k == g.GP_REQ_SOLVE:
                outs.append(E.solve(m.bw[None] + _normals(sd, 4, 1, m.K, m.N)))
            elif k == g.GP_REQ_SAMPLE:
                outs.append(E.solve(E.perturbed(m.bw, _normals(sd, 1, 1, m.K, m.dirs, m.N),
                                                _normals(sd, 2, 1, m.K, m.N))))
            else:
                pr = _signs(sd, 3, R, m.K, m.N)
                outs.append(E.solve(pr.double()))
                t, tk, gk = E.traces(pr, outs[-1])
                tr.append(np.concatenate([[t], tk, gk]))
        return outs, np.concatenate(tr)
    if kind in ("gibbs", "svb", "dataset", "step"):
        A = v["A"] if kind == "svb" else m.ar[None]
        B, bw = _data_term(m.Xd, m.Y, A, v["lam"] if "lam" in v else m.lam)
    else:
        B, bw = m.B, m.bw
    E = Exact(m, B, m.alpha)
    if kind == "solve":
        return E.solve(v["b"])
    if kind == "mean_sample":
        return E.solve(v["b"]), E.solve(E.perturbed(bw, v["z1"], v["z2"]))
    if kind == "sample":
        sd = v["seed"]
        return E.solve(E.perturbed(bw, _normals(sd, 1, R, m.K, m.dirs, m.N), _normals(sd, 2, R, m.K, m.N)))
    if kind == "apply":
        return E.apply(v["x"])
    if kind == "dataset":
        return bw, E.apply(v["x"])
    if kind == "trace":
        u = E.solve(v["probes"].double())
        return (u, *E.traces(v["probes"], u))
    if kind == "step":
        x = E.solve(torch.cat([E.perturbed(bw, v["z1"], v["z2"]), v["probes"].double()]))
        return (x, *E.traces(v["probes"], x[R // 2:]))
    if kind == "svb":
        W = E.solve(E.perturbed(bw, v["z1"], v["z2"]))
        alpha = (0.5 * m.N + 0.1) / (0.5 * E.quad(W).mean(0) + 0.1)
        lam = (0.5 * (m.T - m.P) + 0.1) / (0.5 * _residual_ss(m, W, A) + 0.1)
        return W, lam, alpha.cpu().numpy()
    sd = v["seed"]   # gibbs
    wd = (sd ^ (5 * GOLDEN)) & M64
    W = E.solve(E.perturbed(bw, _normals(wd, 1, 1, m.K, m.dirs, m.N), _normals(wd, 2, 1, m.K, m.N)))
    alpha = _gamma(sd, 16 + 2 * 5, 0.5 * m.N + 0.1, 1.0 / (0.5 * E.quad(W)[0] + 0.1))
    lam = _gamma(sd, 17 + 2 * 5, 0.5 * (m.T - m.P) + 0.1, 1.0 / (0.5 * _residual_ss(m, W, A) + 0.1))
    return W, lam, alpha.cpu().numpy()
