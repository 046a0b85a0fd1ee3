"""The work a program that uses this library has it do, as timed cases.

Every case goes through the public entry points of ``paper_2607_24518_amd``.
``kind`` names the entry point, the other fields its sizes and options:

* ``solve``      - ``steps`` solver iterations on a stored S (ten are one check
                   interval of the stop rule), then the iterate, the gradient and
                   the statistics of the last step, as a solve loop reads them.
* ``build``      - S from a returns panel, |corr| or TPDM.
* ``objective``  - f(H) and E(H), by which kept iterates are compared.
* ``warm``       - the learned warm start: sketch, coordinates, network, scale.
* ``train``      - one training step of the warm start's network.
* ``kmeans``     - Lloyd iterations of spherical K-means from given seed rows.
"""
import math

import torch

import paper_2607_24518_amd as sym

KMEANS_ITERS = 3
DTYPE = {"fp32": sym.S_FP32, "bf16": sym.S_BF16, "fp8": sym.S_FP8}
METHOD = {"admm": sym.ADMM, "mu": sym.MU, "adagrad": sym.ADAGRAD, "row_svrg": sym.ROW_SVRG,
          "block_svrg": sym.BLOCK_SVRG}
HIDDEN, WIDTH = 256, 64

_context = None


def context():
    """One context for the whole program, as its documentation asks of a host thread."""
    global _context
    if _context is None:
        _context = sym.symnmf_create(0)
    return _context


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the 512-instrument instance with 8 groups: a small portfolio, where a
        # step is a handful of short kernels
        {"name": "solve_n512_k16", "kind": "solve", "steps": 10, "n": 512, "rows": 512, "row0": 0, "k": 16,
         "T": 2000, "groups": 8, "dtype": "fp32", "method": "admm"},
        # an index-sized universe with a rank chosen by the data, not by the kernels
        {"name": "solve_n4100_k20", "kind": "solve", "steps": 10, "n": 4100, "rows": 4100, "row0": 0, "k": 20,
         "T": 1500, "groups": 20, "dtype": "fp32", "method": "mu"},
        # the benchmark's workload, n = 100000, k = 32, with the solver that
        # reaches the lowest objective on it; FP32 storage, then the FP8 storage
        # that the precision ladder starts on
        {"name": "solve_n100000_k32_fp32", "kind": "solve", "steps": 2, "n": 100000, "rows": 100000, "row0": 0, "k": 32,
         "T": 2500, "groups": 32, "dtype": "fp32", "method": "admm"},
        {"name": "solve_n100000_k32_fp8", "kind": "solve", "steps": 2, "n": 100000, "rows": 100000, "row0": 0, "k": 32,
         "T": 2500, "groups": 32, "dtype": "fp8", "method": "admm"},
        # one GPU's share of a row-sharded n = 10^6 problem
        {"name": "solve_panel_n1000000_k64", "kind": "solve", "steps": 2, "n": 1000000, "rows": 12500, "row0": 0, "k": 64,
         "T": 1000, "groups": 64, "dtype": "bf16", "method": "admm"},
        # the sampled solver: a snapshot step and nine sampled ones
        {"name": "block_svrg_n20000_k32", "kind": "solve", "steps": 10, "n": 20000, "rows": 20000, "row0": 0, "k": 32,
         "T": 2500, "groups": 32, "dtype": "fp32", "method": "block_svrg"},
        # S of a 20000-instrument universe, rebuilt whenever the returns window moves
        {"name": "build_corr_n20000", "kind": "build", "s": "corr", "n": 20000, "T": 2500, "groups": 32,
         "dtype": "fp32", "q": 0.05, "raw": 0},
        # the 4096-instrument tail dependence matrix
        {"name": "build_tpdm_n4096", "kind": "build", "s": "tpdm", "n": 4096, "T": 20000, "groups": 16,
         "dtype": "fp32", "q": 0.05, "raw": 0},
        # judging a kept iterate of a k = 64 solve
        {"name": "objective_n20000_k64", "kind": "objective", "n": 20000, "k": 64, "T": 1000, "groups": 64,
         "dtype": "fp32"},
        # starting a solve on a new matrix
        {"name": "warm_n20000_k32", "kind": "warm", "n": 20000, "k": 32, "T": 2500, "groups": 32, "dtype": "fp32"},
        # training the warm start on solved instances of n = 20000
        {"name": "train_m20000_k64", "kind": "train", "m": 20000, "k": 64, "residual": 1},
        # clustering the rows of S with about sqrt(n) clusters
        {"name": "kmeans_n20000_K141", "kind": "kmeans", "n": 20000, "K": 141, "T": 1000, "groups": 64,
         "dtype": "fp32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 4 + ["panel", "svrg", "build", "build", "objective", "warm", "train", "kmeans"])
    dtype = rng.choice(["fp32", "fp32", "bf16", "fp8"])
    if kind == "solve":
        n = _log(rng, 300, 40000)
        return {"kind": "solve", "steps": 10 if n < 6000 else 2, "n": n, "rows": n, "row0": 0,
                "k": rng.choice([16, 32, 64, rng.randint(2, 64), rng.randint(2, 64), rng.randint(2, 40)]),
                "T": rng.randint(200, 3000), "groups": rng.randint(4, 40), "dtype": dtype,
                "method": rng.choice(["admm", "admm", "mu"])}
    if kind == "panel":
        n = _log(rng, 20000, 300000)
        rows = _log(rng, 600, 12500)
        return {"kind": "solve", "steps": 2, "n": n, "rows": rows, "row0": rng.randint(0, n - rows),
                "k": rng.choice([32, 64, 64, 40]), "T": rng.randint(200, 1000), "groups": 64, "dtype": rng.choice(["fp32", "bf16"]),
                "method": "admm"}
    if kind == "svrg":
        n = _log(rng, 3000, 40000)
        return {"kind": "solve", "steps": 10, "n": n, "rows": n, "row0": 0, "k": rng.choice([16, 32, 32, 64]),
                "T": rng.randint(500, 2500), "groups": rng.randint(8, 40), "dtype": rng.choice(["fp32", "bf16"]),
                "method": rng.choice(["block_svrg", "row_svrg"])}
    if kind == "build":
        if rng.random() < 0.5:
            return {"kind": "build", "s": "corr", "n": _log(rng, 300, 30000), "T": _log(rng, 250, 5000),
                    "groups": rng.randint(4, 40), "dtype": rng.choice(["fp32", "bf16"]), "q": 0.05, "raw": 0}
        raw = rng.choice([0, 0, 1])
        return {"kind": "build", "s": "tpdm", "n": _log(rng, 200, 8000), "T": _log(rng, 1000, 30000),
                "groups": rng.randint(4, 40), "dtype": rng.choice(["fp32", "bf16"]), "q": rng.choice([0.01, 0.05, 0.1]),
                "raw": raw}
    if kind == "objective":
        return {"kind": "objective", "n": _log(rng, 500, 40000), "k": rng.choice([16, 32, 64, rng.randint(2, 64)]),
                "T": rng.randint(200, 2500), "groups": rng.randint(4, 64), "dtype": dtype}
    if kind == "warm":
        k = rng.choice([8, 16, 32])
        return {"kind": "warm", "n": _log(rng, 2000, 40000), "k": k, "T": rng.randint(1000, 2500), "groups": k,
                "dtype": rng.choice(["fp32", "bf16"])}
    if kind == "train":
        return {"kind": "train", "m": _log(rng, 500, 40000), "k": rng.choice([16, 32, 64, rng.randint(4, 64)]),
                "residual": rng.randint(0, 1)}
    n = _log(rng, 1000, 20000)
    return {"kind": "kmeans", "n": n, "K": rng.choice([math.isqrt(n), rng.randint(4, 64), rng.randint(4, 200)]),
            "T": rng.randint(500, 1500), "groups": rng.randint(16, 64), "dtype": dtype}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator("cuda").manual_seed(seed)


def _loadings(g, n, groups):
    """Market loading 0.4, a primary group with loading U[0.3, 0.9], and for a
    quarter of the instruments a second group: the overlapping-group recipe."""
    A = torch.zeros(n, groups + 1, device="cuda")
    A[:, 0] = 0.4
    rows = torch.arange(n, device="cuda")
    first = torch.randint(0, groups, (n,), generator=g, device="cuda")
    A[rows, first + 1] = 0.3 + 0.6 * torch.rand(n, generator=g, device="cuda")
    second = torch.randint(0, groups, (n,), generator=g, device="cuda")
    load = 0.3 + 0.6 * torch.rand(n, generator=g, device="cuda")
    take = (torch.rand(n, generator=g, device="cuda") < 0.25) & (second != first)
    A[rows[take], second[take] + 1] = load[take]
    return A


def _returns(seed, T, n, groups):
    """Gaussian factor-model returns, T x n float32."""
    g = _gen(seed)
    A = _loadings(g, n, groups)
    X = (0.5 * torch.randn(T, groups + 1, generator=g, device="cuda")) @ A.T
    for lo in range(0, T, 250):
        X[lo:lo + 250] += 0.5 * torch.randn(min(250, T - lo), n, generator=g, device="cuda")
    return X.contiguous()


def _student(g, shape):
    """Student-t draws with 3 degrees of freedom."""
    z = torch.randn(shape, generator=g, device="cuda")
    chi = sum(torch.randn(shape, generator=g, device="cuda").square() for _ in range(3))
    return z / (chi / 3.0).sqrt()


def _tail_returns(seed, T, n, groups, raw):
    """Heavy-tailed factor-model returns: Student-t(3) factors and noise, or
    (raw) the positive Pareto(2) draws that need no rank transform."""
    g = _gen(seed)
    A = _loadings(g, n, groups)

    def sample(shape):
        if not raw:
            return _student(g, shape)
        return (1.0 - torch.rand(shape, generator=g, device="cuda")).clamp_min(1e-7).rsqrt()

    X = sample((T, groups + 1)) @ A.T
    for lo in range(0, T, 1000):
        X[lo:lo + 1000] += 0.3 * sample((min(1000, T - lo), n))
    return X.contiguous()


def _case_returns(case, seed):
    if case.get("s") == "tpdm":
        return _tail_returns(seed, case["T"], case["n"], case["groups"], case["raw"])
    return _returns(seed, case["T"], case["n"], case["groups"])


def _factor(seed, n, k, groups):
    """A factor as a solve in progress has it: column j follows the loadings of
    group j (mod groups), with entries dropped and noise added."""
    A, g = _loadings(_gen(seed), n, groups), _gen(seed + 77)
    H = A[:, 1 + torch.arange(k, device="cuda") % groups] * (torch.rand(n, k, generator=g, device="cuda") < 0.8)
    return (0.8 * H + 0.15 * torch.rand(n, k, generator=g, device="cuda")).contiguous()


def _params(case):
    return sym.symnmf_params_default(method=METHOD[case["method"]], eta=math.sqrt(0.1 / case["k"]),
                                     eps=2.0 ** -23 if case["method"] == "mu" else 1e-10)


def _train_data(case, seed):
    """Canonical coordinates (mixtures of a few anchors, zero-padded to the
    network's width) and a solved factor near them."""
    g, m, k = _gen(seed), case["m"], case["k"]
    C = torch.rand(m, k, generator=g, device="cuda")
    C *= torch.rand(m, k, generator=g, device="cuda") < 3.0 / k
    C += 0.02 * torch.randn(m, k, generator=g, device="cuda")
    X = torch.zeros(m, WIDTH, device="cuda")
    X[:, :k] = C
    B = (C + 0.1 * torch.randn(m, k, generator=g, device="cuda")).clamp_min(0.0)
    return X.contiguous(), B.contiguous()


def _network(seed, k):
    """A network with all layers in use (a trained one's last layer is small)."""
    P = sym.symnmf_mlp_init(context(), WIDTH, HIDDEN, k, seed, torch.empty(sym.symnmf_mlp_param_count(WIDTH, HIDDEN, k),
                                                                          device="cuda"))
    w3 = HIDDEN * WIDTH + HIDDEN * HIDDEN
    P[w3:w3 + k * HIDDEN] *= 0.1
    return P


def prepare(case, seed):
    ctx, kind = context(), case["kind"]
    if kind == "build":
        return {"case": case, "X": _case_returns(case, seed)}
    if kind == "train":
        X, B = _train_data(case, seed)
        net = sym.symnmf_mlp_create(ctx, WIDTH, HIDDEN, case["k"], _network(seed, case["k"]))
        sym.symnmf_mlp_set_output(ctx, net, bool(case["residual"]))
        sym.symnmf_mlp_reserve(ctx, net, case["m"], training=True)
        return {"case": case, "X": X, "B": B, "net": net, "grad": torch.empty(net.count, device="cuda")}
    X = _returns(seed, case["T"], case["n"], case["groups"])
    n = case["n"]
    rows, row0 = case.get("rows", n), case.get("row0", 0)
    S = sym.symnmf_build_S(ctx, X, dtype=DTYPE[case["dtype"]], row0=row0, rows=rows)
    del X
    state = {"case": case, "S": S}
    if kind == "solve":
        k = case["k"]
        state["st"] = sym.symnmf_state_create(ctx, S, k, _params(case), _factor(seed, n, k, case["groups"]))
        state["H"] = torch.empty(n, k, device="cuda")
        state["G"] = torch.empty(rows, k, device="cuda")
    elif kind == "objective":
        state["H"] = _factor(seed, n, case["k"], case["groups"])
    elif kind == "warm":
        net = sym.symnmf_mlp_create(ctx, WIDTH, HIDDEN, case["k"], _network(seed, case["k"]))
        sym.symnmf_mlp_set_output(ctx, net, True)
        sym.symnmf_mlp_reserve(ctx, net, n)
        state.update(net=net, H=torch.empty(n, case["k"], device="cuda"), omega=seed)
    elif kind == "kmeans":
        pick = torch.randperm(n, generator=_gen(seed + 5), device="cuda")[:case["K"]]
        state.update(rows=pick.tolist(), labels=torch.empty(n, dtype=torch.int32, device="cuda"),
                     C=torch.empty(n, case["K"], device="cuda"))
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    ctx, case = context(), state["case"]
    kind = case["kind"]
    if kind == "solve":
        S, st = state["S"], state["st"]
        for _ in range(case["steps"]):
            sym.symnmf_step(ctx, S, st, want_stats=False)
        sym.symnmf_state_read(ctx, st, 0, state["H"])
        sym.symnmf_state_read(ctx, st, 6, state["G"])
        stats = sym.symnmf_state_stats(ctx, st)
        got = {"H": state["H"], "G": state["G"]}
        return dict(got, kkt=stats.kkt) if stats.full else got   # a sampled step has no residual of the whole
    if kind == "build":
        S = sym.symnmf_build_S(ctx, state["X"], kind=sym.TPDM if case["s"] == "tpdm" else sym.ABS_CORR,
                               dtype=DTYPE[case["dtype"]], q=case["q"], lower_tail=0 if case["raw"] else 1,
                               raw_marginals=case["raw"])
        return {"S": S.buf.view(torch.float32 if case["dtype"] == "fp32" else torch.bfloat16), "fro2": S.fro2,
                "mean": S.mean}
    if kind == "objective":
        f, E = sym.symnmf_objective(ctx, state["S"], state["H"], case["k"])
        return {"f": f, "E": E}
    if kind == "warm":
        return sym.symnmf_warm_start(ctx, state["S"], state["net"], WIDTH, case["k"], state["omega"], state["H"])
    if kind == "train":
        loss = sym.symnmf_mlp_train_step(ctx, state["net"], state["X"], state["B"], lr=1e-4, loss_kind=1)
        return {"loss": loss, "grad": sym.symnmf_mlp_read(ctx, state["net"], "grad", state["grad"])}
    got = sym.symnmf_kmeans(ctx, state["S"], case["K"], state["labels"], init_rows=state["rows"], tol=0.0,
                            max_iter=KMEANS_ITERS, C=state["C"], allow_notconv=True)
    return {"C": state["C"], "labels": state["labels"], "J": got["J"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind == "train":
        m, k = case["m"], case["k"]
        macs = WIDTH * HIDDEN + HIDDEN * HIDDEN + HIDDEN * k
        params = macs + 2 * HIDDEN + k
        return {"bytes": 4 * (m * (WIDTH + k) + 8 * params), "flops": m * (6 * macs - 2 * WIDTH * HIDDEN + 14 * k * k)}
    n = case["n"]
    size = {"fp32": 4, "bf16": 2, "fp8": 1}[case["dtype"]]
    if kind == "build":
        # the input once, S once; the products on and above the diagonal
        K = case["T"] if case["s"] == "corr" else int(case["q"] * case["T"])
        return {"bytes": 4 * case["T"] * n + size * n * n, "flops": n * (n + 1) * K}
    if kind == "solve":
        rows, k, steps = case["rows"], case["k"], case["steps"]
        share = 1.0
        if case["method"] in ("row_svrg", "block_svrg"):
            blocks = -(-n // 1024)
            if case["method"] == "row_svrg":
                part = math.ceil(0.5 * blocks) / blocks
            else:   # S_IJ and its mirror, the common part once
                p = math.ceil(math.sqrt(0.75) * blocks) / blocks
                part = 2 * p * p - p ** 4
            share = (1 + (steps - 1) * part) / steps
        # S, H of every column, and the rows of the iterate, the gradient and the
        # method's other buffer
        step = share * size * rows * n + 4 * k * (n + 4 * rows)
        return {"bytes": steps * step, "flops": steps * (share * 2 * rows * n * k + 6 * rows * k * k)}
    if kind == "objective":
        k = case["k"]
        return {"bytes": size * n * n + 4 * n * k, "flops": 2 * n * n * k + 2 * n * k * k}
    if kind == "warm":
        k = case["k"]
        # S times the sketch, then (its scale) S times the factor that came of it
        macs = WIDTH * HIDDEN + HIDDEN * HIDDEN + HIDDEN * k
        return {"bytes": 2 * size * n * n + 4 * n * (WIDTH + k),
                "flops": 2 * n * n * (WIDTH + k) + 2 * n * (macs + WIDTH * WIDTH + 2 * WIDTH * k + 2 * k * k)}
    K = case["K"]
    # row lengths and seeds, then a product for the assignment of the seeds and
    # two per iteration
    passes = 1 + 2 * KMEANS_ITERS
    return {"bytes": (1 + passes) * size * n * n + 4 * n * K * (2 * passes), "flops": 2 * passes * n * n * K}


# ---------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------
def _exact_corr(X, row0, rows):
    """|Pearson correlation| rows [row0, row0 + rows) in FP64, unit diagonal."""
    Z = X.double()
    Z -= Z.mean(0)
    Z /= Z.square().sum(0).sqrt()
    n = Z.shape[1]
    S = torch.empty(rows, n, dtype=torch.float64, device="cuda")
    for lo in range(0, rows, 4096):
        hi = min(lo + 4096, rows)
        torch.mm(Z[:, row0 + lo:row0 + hi].T.contiguous(), Z, out=S[lo:hi])
        S[lo:hi].abs_()
        i = torch.arange(lo, hi, device="cuda")
        S[i, row0 + i] = 1.0
    return S


def _rounded(S, dtype, row0):
    """The storage rounding of S, in place (256-row scale panels for FP8, whose
    diagonal is kept exactly)."""
    for lo in range(0, S.shape[0], 256):
        P = S[lo:lo + 256]
        if dtype == "fp32":
            P.copy_(P.float())
        elif dtype == "bf16":
            P.copy_(P.to(torch.bfloat16))
        else:
            i = torch.arange(P.shape[0], device="cuda")
            P[i, row0 + lo + i] = 0.0
            scale = (448.0 / P.max().float()).double()
            P.copy_((P * scale).float().to(torch.float8_e4m3fn).double() / scale)
            P[i, row0 + lo + i] = 1.0
    return S


def _exact_tpdm(X, case):
    T, n = X.shape
    if case["raw"]:
        x = X.double()
    else:
        # ranks of -X (lower tail), ties to the lower sample
        x = torch.empty(T, n, dtype=torch.float64, device="cuda")
        rank = torch.arange(1, T + 1, dtype=torch.float64, device="cuda")[:, None]
        for lo in range(0, n, 512):
            order = torch.sort(-X[:, lo:lo + 512], dim=0, stable=True).indices
            x[:, lo:lo + 512].scatter_(0, order, (1.0 - rank / (T + 1)).rsqrt().expand(T, order.shape[1]))
    norm = x.square().sum(1).sqrt()
    keep = torch.sort(norm, descending=True, stable=True).indices[:int(math.floor(case["q"] * T))]
    Om = x[keep] / norm[keep][:, None]
    Om /= Om.square().sum(0).sqrt()
    S = (Om.T.contiguous() @ Om).abs()
    S.fill_diagonal_(1.0)
    return S


def _stored_order(S, lanes):
    """A dense square S in the order of its storage: 256 x 256 tiles, a tile as
    [wave][sub-step][row group][lane = (column group, row)][consecutive columns]."""
    n = S.shape[0]
    pad = -(-n // 256) * 256
    P = torch.zeros(pad, pad, dtype=S.dtype, device=S.device)
    P[:n, :n] = S
    t = pad // 256
    P = P.view(t, 4, 4, 16, t, 256 // (4 * lanes), 4, lanes)   # R wave group row | C step lane-group column
    return P.permute(0, 4, 1, 5, 2, 6, 3, 7).reshape(-1)


def _exact_solve(case, seed):
    n, rows, row0, k = case["n"], case["rows"], case["row0"], case["k"]
    S = _rounded(_exact_corr(_returns(seed, case["T"], n, case["groups"]), row0, rows), case["dtype"], row0)
    W = _factor(seed, n, k, case["groups"]).double()
    own = slice(row0, row0 + rows)
    U = torch.zeros(rows, k, dtype=torch.float64, device="cuda")
    eye = torch.eye(k, dtype=torch.float64, device="cuda")
    for _ in range(case["steps"]):
        gram, SW, w = W.T.contiguous() @ W, S @ W, W[own].clone()
        HG = w @ gram
        G = 4.0 * (HG - SW)
        kkt = torch.where(w > 0, G, G.clamp_max(0.0)).norm().item() / (rows * k)
        if case["method"] == "admm":
            H = (2.0 * SW + 500.0 * (w - U)) @ torch.linalg.inv(2.0 * gram + 500.0 * eye)
            new = (H + U).clamp_min(0.0)
            U = U + H - new
        else:
            new = 0.5 * w * (1.0 + SW / (HG + 2.0 ** -23))
        W[own] = new
    return {"H": W, "G": G, "kkt": torch.tensor(kkt, dtype=torch.float64)}


def _exact_train(case, seed):
    X, B = (t.double() for t in _train_data(case, seed))
    P = _network(seed, case["k"]).double().requires_grad_()
    k, at, parts = case["k"], 0, []
    for shape in ((HIDDEN, WIDTH), (HIDDEN, HIDDEN), (k, HIDDEN), (HIDDEN,), (HIDDEN,), (k,)):
        size = math.prod(shape)
        parts.append(P[at:at + size].view(shape))
        at += size
    W1, W2, W3, b1, b2, b3 = parts
    gelu = torch.nn.functional.gelu
    z = gelu(gelu(X @ W1.T + b1) @ W2.T + b2) @ W3.T + b3
    A = (X[:, :k] + z).clamp_min(0.0) if case["residual"] else torch.nn.functional.softplus(z)
    naa, nab, nbb = ((p.T @ q).square().sum() for p, q in ((A, A), (A, B), (B, B)))
    loss = 1.0 - nab.square() / (naa * nbb)
    loss.backward()
    return {"loss": loss.detach(), "grad": P.grad}


def _exact_kmeans(case, seed):
    n, K = case["n"], case["K"]
    S = _rounded(_exact_corr(_returns(seed, case["T"], n, case["groups"]), 0, n), case["dtype"], 0)
    rows = torch.randperm(n, generator=_gen(seed + 5), device="cuda")[:K]
    norm = S.square().sum(1).sqrt()
    weight = torch.zeros(n, K, dtype=torch.float64, device="cuda")
    weight[rows, torch.arange(K, device="cuda")] = 1.0 / norm[rows]
    C = None
    for _ in range(KMEANS_ITERS + 1):
        M = S @ weight
        length = M.square().sum(0).sqrt()
        C = torch.where(length > 0, M / length.clamp_min(1e-300), C if C is not None else M)
        best, label = (S @ C).max(1)
        J = (1.0 - best / norm).sum()
        weight = torch.zeros_like(weight)
        weight[torch.arange(n, device="cuda"), label] = 1.0 / norm
    return {"C": C, "labels": None, "J": J}


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        # the sampled solvers' index sets come from the library's own generator
        return None if case["method"] in ("row_svrg", "block_svrg") else _exact_solve(case, seed)
    if kind == "build":
        X = _case_returns(case, seed)
        S = _exact_tpdm(X, case) if case["s"] == "tpdm" else _exact_corr(X, 0, case["n"])
        return {"S": _stored_order(S, 4 if case["dtype"] == "fp32" else 8), "fro2": S.square().sum(), "mean": S.mean()}
    if kind == "objective":
        S = _rounded(_exact_corr(_returns(seed, case["T"], case["n"], case["groups"]), 0, case["n"]), case["dtype"], 0)
        H = _factor(seed, case["n"], case["k"], case["groups"]).double()
        f = S.square().sum() - 2.0 * (H * (S @ H)).sum() + (H.T.contiguous() @ H).square().sum()
        return {"f": f, "E": f / S.square().sum()}
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "kmeans":
        return _exact_kmeans(case, seed)
    return None   # the sketch comes from the library's own generator
