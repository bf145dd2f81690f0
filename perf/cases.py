"""The work that a program built on this framework has it do, as timed cases.

`listed()` holds the cases, `draw()` more of the same ranges.  A case names a public call, the structure of the data
and the sizes; `prepare()` makes the inputs on the GPU from a seed and the handle that a training or scoring program
keeps; `run()` is one pass through the entry points of `paper_2004_13940_amd.binding`.

Data structures (the five synthetic workloads of `paper_2004_13940_amd/workloads.py` and the small tables there):
  table    every feature stored in every row, standard normal values
  uniform  a fixed number of distinct uniform columns per row, values U(0,1)
  text     row lengths ~ Poisson, Zipf(1.0) columns over a random permutation, rows L2-normalised
  click    13 always-present numeric columns and one column in each of 26 one-hot fields, Zipf(1.1) inside a field
  hashed   row lengths U[50,150], Zipf(1.05) over a large hashed space, values 1; K is large, V does not fit a cache
A token that a row draws twice is stored once, as a counting or hashing vectoriser does.  The parameters are those of
a model in training (no zeros), the labels are drawn at the rate of the workload.
"""
import math

import numpy as np
import torch

from paper_2004_13940_amd import binding as B

CLICK_DENSE, CLICK_FIELDS = 13, 26


def listed():
    return [
        # A small regression table: one full-gradient step with its objective, the loop a user watches converge.
        # The smallest call there is: launches and host latency.
        dict(name="epoch_small", call="epoch", data="table", N=513, D=8, K=4, loss="squared", objective=True),
        # Validation metrics of a classification table after an epoch.
        dict(name="evaluate_table", call="evaluate", data="table", N=49_990, D=22, K=4, loss="logistic"),
        # The tiny sparse workload, doubly-separable epoch with its objective.
        dict(name="stratified_tiny", call="stratified", data="uniform", N=2_000, D=1_000, row=10, K=8, P=4,
             loss="logistic", objective=True),
        # Scoring rows that arrive from outside: host CSR to predictions, a handle per batch of requests.
        dict(name="score_requests", call="score", data="text", N=5_003, D=20_000, row=50, K=16, loss="logistic"),
        # Text-like classification: full-gradient epoch and stratified epoch.
        dict(name="epoch_text", call="epoch", data="text", N=50_000, D=20_000, row=50, K=16, loss="logistic"),
        dict(name="stratified_text", call="stratified", data="text", N=50_000, D=20_000, row=50, K=16, P=32,
             loss="logistic"),
        # A tall regression table that stores every feature.
        dict(name="epoch_table", call="epoch", data="table", N=1_000_000, D=64, K=32, loss="squared"),
        # Click logs: mini-batch pass, doubly-separable epoch, opening a data set from host memory and taking the
        # first stratified epoch on it, and the headline full-gradient epoch at its full size.
        dict(name="minibatch_click", call="minibatch", data="click", N=2_500_000, D=1_000_000, K=16, B=16,
             loss="logistic"),
        dict(name="stratified_click", call="stratified", data="click", N=10_000_000, D=1_000_000, K=16, P=64,
             loss="logistic"),
        dict(name="load_click", call="load", data="click", N=1_250_003, D=1_000_000, K=16, P=16, loss="logistic"),
        dict(name="epoch_click", call="epoch", data="click", N=10_000_000, D=1_000_000, K=16, loss="logistic"),
        # A caller with an optimiser of its own: forward (aggregates and multipliers out), then the gradient, on the
        # hashed workload with its large latent size.
        dict(name="gradient_hashed", call="gradient", data="hashed", N=400_001, D=4_000_000, K=64, loss="logistic"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    data = rng.choice(["table", "uniform", "text", "text", "click", "click", "hashed"])
    call = rng.choice(["epoch", "epoch", "stratified", "minibatch", "gradient", "evaluate", "score", "load"])
    K = rng.choice([4, 8, 8, 10, 16, 16, 16, 20, 32, 64])
    c = dict(call=call, data=data, loss=rng.choice(["logistic", "squared"]))
    if data == "table":
        c.update(N=_log_int(rng, 300, 1_000_000), D=rng.choice([32, 64, rng.randint(5, 64)]))
        P = rng.randint(2, 16)
    elif data == "uniform":
        c.update(N=_log_int(rng, 500, 20_000), D=_log_int(rng, 200, 5_000), row=rng.randint(5, 20))
        P = rng.randint(2, 8)
    elif data == "text":
        c.update(N=_log_int(rng, 3_000, 200_000), D=_log_int(rng, 5_000, 100_000), row=rng.randint(20, 100))
        P = rng.choice([8, 16, 32])
    elif data == "click":
        top = {"epoch": 5_000_000, "gradient": 2_500_000, "evaluate": 2_500_000, "score": 500_000, "load": 1_000_000}
        c.update(N=_log_int(rng, 50_000, top.get(call, 2_000_000)), D=_log_int(rng, 100_000, 1_000_000))
        K = min(K, 32)
        P = rng.choice([16, 32, 64])
    else:
        N = _log_int(rng, 20_000, 400_000)
        c.update(N=N, D=10 * N + rng.randint(0, 999))
        K = rng.choice([32, 64])
        P = rng.choice([16, 32, 64])
    c["K"] = K
    if call in ("stratified", "load"):
        c["P"] = P
    elif call == "minibatch":
        c["B"] = rng.randint(4, 32)
    if call in ("epoch", "stratified", "minibatch"):
        c["objective"] = rng.random() < 0.3
    if call in ("epoch", "minibatch", "gradient", "evaluate") and K % 4 == 0 and rng.random() < 0.2:
        c["half"] = True  # rows of V gathered from a half-precision copy
    return c


# ---------------------------------------------------------------- inputs ----

def _zipf(u, n, s):
    """Ranks 0..n-1 of a Zipf law with exponent s by the inverse of its continuous distribution function."""
    if abs(s - 1.0) < 1e-9:
        x = torch.exp(u * math.log(n + 1))
    else:
        x = (1 + u * ((n + 1) ** (1 - s) - 1)) ** (1 / (1 - s))
    return (x.long() - 1).clamp_(0, n - 1)


def _distinct(rows, cols, N, D):
    """Sorted distinct (row, column) pairs as a row pointer array and columns."""
    key = torch.unique(rows * D + cols)
    r = key // D
    rowptr = torch.zeros(N + 1, dtype=torch.int64, device=key.device)
    rowptr[1:] = torch.cumsum(torch.bincount(r, minlength=N), 0)
    return rowptr, (key - r * D).int(), r


def _matrix(case, gen):
    """(rowptr int64, col int32, val float32) on the GPU."""
    N, D, data, dev = case["N"], case["D"], case["data"], "cuda"
    if data == "table":
        rowptr = torch.arange(N + 1, device=dev) * D
        return rowptr, torch.arange(D, dtype=torch.int32, device=dev).repeat(N), torch.randn(N * D, generator=gen, device=dev)
    if data == "click":
        nz, span = CLICK_DENSE + CLICK_FIELDS, D - CLICK_DENSE
        col = torch.empty(N, nz, dtype=torch.int32, device=dev)
        val = torch.ones(N, nz, device=dev)
        col[:, :CLICK_DENSE] = torch.arange(CLICK_DENSE, dtype=torch.int32, device=dev)
        val[:, :CLICK_DENSE] = torch.log1p(torch.poisson(torch.full((N, CLICK_DENSE), 3.0, device=dev), generator=gen))
        for f in range(CLICK_FIELDS):
            lo, hi = f * span // CLICK_FIELDS, (f + 1) * span // CLICK_FIELDS
            u = torch.rand(N, generator=gen, device=dev, dtype=torch.float64)
            col[:, CLICK_DENSE + f] = CLICK_DENSE + lo + _zipf(u, hi - lo, 1.1)
        return torch.arange(N + 1, device=dev) * nz, col.reshape(-1), val.reshape(-1)
    if data == "uniform":
        lengths = torch.full((N,), case["row"], device=dev)
    elif data == "text":
        lengths = torch.poisson(torch.full((N,), float(case["row"]), device=dev), generator=gen).long().clamp_(1, D)
    else:
        lengths = torch.randint(50, 151, (N,), generator=gen, device=dev)
    rows = torch.repeat_interleave(torch.arange(N, device=dev), lengths)
    u = torch.rand(len(rows), generator=gen, device=dev, dtype=torch.float64)
    if data == "uniform":
        cols = (u * D).long().clamp_(0, D - 1)
    elif data == "text":
        cols = torch.randperm(D, generator=gen, device=dev)[_zipf(u, D, 1.0)]
    else:
        cols = _zipf(u, D, 1.05)
    rowptr, col, r = _distinct(rows, cols, N, D)
    if data == "uniform":
        val = torch.rand(len(col), generator=gen, device=dev)
    elif data == "text":
        val = torch.exp(torch.randn(len(col), generator=gen, device=dev))
        val /= torch.segment_reduce(val * val, "sum", lengths=rowptr[1:] - rowptr[:-1]).sqrt_()[r]
    else:
        val = torch.ones(len(col), device=dev)
    return rowptr, col, val


# eta, lambda of the workloads; the loss is averaged over the rows
_STEP = {"table": (0.05, 1e-5), "uniform": (1.0, 1e-4), "text": (4.0, 1e-4), "click": (0.02, 1e-6), "hashed": (0.05, 1e-6)}


class State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    N, D, K, call = case["N"], case["D"], case["K"], case["call"]
    st = State()
    st.case = case
    rowptr, col, val = (t.cpu().numpy() for t in _matrix(case, gen))
    if case["loss"] == "squared":
        st.y = torch.randn(N, generator=gen, device="cuda")
    else:
        rate = 0.03 if case["data"] == "click" else 0.5
        st.y = torch.where(torch.rand(N, generator=gen, device="cuda") < rate, 1.0, -1.0)
    st.w0 = torch.full((1,), 0.25, device="cuda")
    st.w = torch.randn(D, generator=gen, device="cuda") * 0.05
    st.V = torch.randn(D * K, generator=gen, device="cuda") * 0.05
    eta, lam = _STEP[case["data"]]
    st.p = B.make_params(K, B.FM_LOSS_SQUARED if case["loss"] == "squared" else B.FM_LOSS_LOGISTIC, lam, lam, eta,
                         1.0 / N, half_gather=int(case.get("half", False)))
    if call in ("load", "score"):  # the data set stays on the host: opening it is part of the pass
        st.host = (rowptr, col, val)
        st.yhat = torch.empty(N, device="cuda")
        return st
    st.m = B.Matrix(N, D, rowptr, col, val)
    if call != "evaluate":
        st.m.fm_build_csc()
    if call == "stratified":
        st.m.fm_partition(case["P"])
    elif call == "minibatch":
        st.m.fm_partition_batches(case["B"])
    elif call == "gradient":
        st.yhat, st.r = torch.empty(N, device="cuda"), torch.empty(N, device="cuda")
        st.G = torch.empty(N * K, device="cuda")
        st.g0, st.gw, st.gV = torch.empty(1, device="cuda"), torch.empty(D, device="cuda"), torch.empty(D * K, device="cuda")
    return st


# ------------------------------------------------------------------ pass ----

def run(st):
    c, p = st.case, st.p
    call = c["call"]
    if call == "evaluate":
        return st.m.fm_evaluate(p, st.y, st.w0, st.w, st.V)
    if call == "score":
        m = B.Matrix(c["N"], c["D"], *st.host)
        m.fm_forward(p, None, st.w0, st.w, st.V, yhat=st.yhat)
        m.close()
        return st.yhat
    if call == "gradient":
        st.m.fm_forward(p, st.y, st.w0, st.w, st.V, yhat=st.yhat, G=st.G, r=st.r)
        st.m.fm_gradient(p, st.r, st.G, st.w, st.V, grad_w0=st.g0, grad_w=st.gw, grad_V=st.gV)
        return st.yhat, st.r, st.G, st.g0, st.gw, st.gV
    objective = None
    if call == "load":
        m = B.Matrix(c["N"], c["D"], *st.host)
        m.fm_build_csc()
        m.fm_partition(c["P"])
        m.fm_stratified_epoch(p, st.y, st.w0, st.w, st.V)
        m.close()
    else:
        step = {"epoch": st.m.fm_sgd_epoch, "stratified": st.m.fm_stratified_epoch, "minibatch": st.m.fm_minibatch_epoch}[call]
        objective = step(p, st.y, st.w0, st.w, st.V, want_objective=c.get("objective", False))
    return st.w0, st.w, st.V, objective


# ----------------------------------------------------------- cost, limits ----

def work(case):
    """The matrix, the labels and the parameters read once, what comes out written once; products and sums of the
    scores (4 per stored entry and latent dimension), of the gradient (4) and of the refresh of the aggregates (2)."""
    N, D, K, call = case["N"], case["D"], case["K"], case["call"]
    row = {"table": D, "click": CLICK_DENSE + CLICK_FIELDS, "hashed": 80}.get(case["data"]) or case["row"]
    nnz, params = N * row, D * (K + 1) + 1
    x = 8 * nnz + 8 * (N + 1) + 4 * N
    if call == "evaluate":
        return {"bytes": x + 4 * params, "flops": 4 * nnz * K}
    if call == "score":
        return {"bytes": x + 4 * params, "flops": 4 * nnz * K}
    if call == "gradient":
        return {"bytes": x + 8 * params + 4 * N * (K + 2), "flops": 8 * nnz * K}
    return {"bytes": x + 8 * params, "flops": (10 if call in ("stratified", "load") else 8) * nnz * K}


def tolerance(case):
    """32-bit sums.  The accuracy that fm_evaluate counts moves by whole rows."""
    return {"rel": 1e-4 if case["call"] == "evaluate" else 1e-5}
