"""The calls this library is used for, as timed cases.

Six kinds of call, each through a public entry point of ``paper_1302_5010_amd``:

* ``solve``      a batch of sparse-recovery problems (``Solver.solve``): one signal to thousands, Gaussian
                 dictionaries and the face-like class-subspace one, float32 product and bfloat16 screen, host
                 loop, captured segments and one captured graph per solve, cold and from a proposal;
* ``correlate``  one batched correlation G = A^T R (``Solver.correlate``), a few residuals up to a thousand;
* ``classify``   class-residual labels of solved codes (``Solver.classify``);
* ``train``      one training step of the support proposal (``ProposalNet.loss_grad``, ``adam_step``);
* ``scores``     the proposal in use: scores of a batch (``ProposalNet.forward``) and their top k (``topk``);
* ``setup``      a new dictionary (``Solver(...)`` with its float64 Gram table).

Sizes come from the input recipes of ``bmpl_inputs`` and the tests (128 x 512 with 16 signals, 2048 x 16384 with
1024, the face-like 1024 x 20000, rho = 2 and 10) or are generic ones between them.  The e4m3 ranking and the
Q-route are left out: both are slower than the bfloat16 screen and the dense product on every workload.
"""
import math

import torch

import paper_1302_5010_amd as pk


def listed():
    return [
        # the smallest batch of the recipes with every option at its default: launches and host time
        dict(name="solve_small_16", kind="solve", dict="gauss", n=128, m=512, p=16, k_lo=10, k_hi=10, c=0.05, rho=2,
             screen="fp32", graph=False, max_outer=0, warm_k=0, omega=1, tune=False),
        # a single signal of an odd length, default options: the latency of one call
        dict(name="solve_one_signal", kind="solve", dict="gauss", n=1000, m=5001, p=1, k_lo=40, k_hi=40, c=0.02,
             rho=10, screen="fp32", graph=False, max_outer=0, warm_k=0, omega=1, tune=False),
        # the compressive-sensing batch of the benchmark, in the precision of its headline
        dict(name="solve_cs_fp32", kind="solve", dict="gauss", n=2048, m=16384, p=1024, k_lo=100, k_hi=100, c=0.02,
             rho=10, screen="fp32", graph=True, max_outer=16, warm_k=0, omega=1, tune=True),
        # the same batch under the certified bfloat16 screen
        dict(name="solve_cs_bf16", kind="solve", dict="gauss", n=2048, m=16384, p=1024, k_lo=100, k_hi=100, c=0.02,
             rho=10, screen="bf16", graph=True, max_outer=16, warm_k=0, omega=1, tune=True),
        # supports of very different sizes in one batch, no iteration cap: captured segments, factors that
        # outgrow the LDS
        dict(name="solve_ragged", kind="solve", dict="gauss", n=512, m=4096, p=300, k_lo=10, k_hi=160, c=0.03,
             rho=10, screen="fp32", graph=True, max_outer=0, warm_k=0, omega=1, tune=False),
        # a large recognition batch: thousands of small supports on a correlated dictionary
        dict(name="solve_face_bf16", kind="solve", dict="face", n=1024, m=20000, classes=200, p=8192, k_lo=8, k_hi=8,
             c=0.01, rho=10, screen="bf16", graph=True, max_outer=8, warm_k=0, omega=1, tune=True),
        # labels of such a batch's codes
        dict(name="classify_face", kind="classify", n=1024, m=20000, classes=200, p=8192),
        # a few residuals against a large dictionary: the dictionary's bytes bound it
        dict(name="correlate_fp32_few", kind="correlate", n=2048, m=16384, p=8, screen="fp32"),
        # a ragged batch of residuals, reduced precision
        dict(name="correlate_bf16_batch", kind="correlate", n=1024, m=20000, p=1000, screen="bf16"),
        # one step of the proposal's training at the benchmark's batch
        dict(name="train_step", kind="train", n=1024, m=20000, classes=200, d=2048, h=2048, p=1024),
        # the trained network in use on a batch of signals
        dict(name="scores_topk", kind="scores", n=1024, m=20000, classes=200, d=2048, h=2048, p=4096, k=64),
        # a dictionary taken into use (and its Gram table read back)
        dict(name="setup_gram", kind="setup", n=1000, m=6000, screen="fp32"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["solve", "correlate", "classify", "train", "scores", "setup"], [9, 4, 2, 2, 2, 2])[0]
    if kind == "solve":
        face = rng.random() < 0.3
        graph = rng.random() < 0.6
        c = dict(kind=kind, dict="face" if face else "gauss", screen=rng.choice(["fp32", "bf16"]), graph=graph,
                 tune=rng.random() < 0.4, omega=1)
        if face:
            classes = rng.randint(20, 200)
            c.update(n=rng.randint(256, 1024), classes=classes, m=classes * rng.randint(20, 100),
                     p=_log(rng, 16, 8192), k_lo=8, k_hi=8, c=0.01, rho=rng.choice([5, 10]),
                     max_outer=8 if graph and rng.random() < 0.7 else 0, warm_k=rng.choice([0, 0, 32, 64]))
        else:
            n = _log(rng, 64, 2048)
            k = max(2, int(n * rng.uniform(0.03, 0.06)))
            rho = rng.choice([2, 5, 10]) if k < 40 else 10
            c.update(n=n, m=min(16384, int(n * rng.uniform(4, 12))), p=_log(rng, 1, 1024), k_hi=k,
                     k_lo=rng.choice([k, max(1, k // 4)]), c=rng.choice([0.02, 0.03, 0.05]), rho=rho,
                     max_outer=rng.choice([0, 40]) if graph else 0, warm_k=rng.choice([0, 0, 0, 32]))
            if c["screen"] == "fp32" and rng.random() < 0.15:
                c["omega"] = 3
        return c
    if kind == "correlate":
        return dict(kind=kind, n=_log(rng, 64, 2048), m=_log(rng, 500, 20000), p=_log(rng, 1, 1024),
                    screen=rng.choice(["fp32", "bf16"]))
    classes = rng.randint(20, 200)
    m = classes * rng.randint(20, 100)
    n = rng.randint(256, 1024)
    if kind == "classify":
        return dict(kind=kind, n=n, m=m, classes=classes, p=_log(rng, 16, 8192))
    if kind == "setup":
        return dict(kind=kind, n=_log(rng, 64, 1024), m=_log(rng, 500, 6000), screen=rng.choice(["fp32", "bf16"]))
    c = dict(kind=kind, n=n, m=m, classes=classes, d=64 * rng.randint(4, 32), h=64 * rng.randint(4, 32),
             p=_log(rng, 32, 1024 if kind == "train" else 4096))
    if kind == "scores":
        c["k"] = rng.choice([32, 64, 256])
    return c


# ------------------------------------------------------------------------------------------------------------
# Inputs, from the seed alone (torch generators on the GPU, sums in a fixed order)
# ------------------------------------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _unit_rows(a):
    return a / a.double().square().sum(1, keepdim=True).sqrt().float()


def _gauss(case, g):
    """Gaussian unit-norm atoms, k-sparse signals with amplitudes +-U[1, 2] and a little noise."""
    n, m, p = case["n"], case["m"], case.get("p", 1)
    At = _unit_rows(_randn(g, m, n))
    if "k_hi" not in case:
        return At, 0.05 * _randn(g, p, n), None
    kk = torch.randint(case["k_lo"], case["k_hi"] + 1, (p,), generator=g, device="cuda")
    idx = torch.rand(p, m, generator=g, device="cuda").topk(case["k_hi"], dim=1).indices
    amp = 1.0 + torch.rand(p, case["k_hi"], generator=g, device="cuda")
    amp = torch.where(torch.rand(p, case["k_hi"], generator=g, device="cuda") < 0.5, -amp, amp)
    amp = amp * (torch.arange(case["k_hi"], device="cuda")[None, :] < kk[:, None])
    Bt = 0.005 * _randn(g, p, n)
    for j in range(case["k_hi"]):
        Bt += amp[:, j, None] * At[idx[:, j]]
    return At, Bt, idx


def _face(case, g):
    """Classes of atoms near random rank-8 subspaces; a signal lies near one class's subspace, 5 % noise."""
    n, classes, p, rank = case["n"], case["classes"], case["p"], 8
    per = case["m"] // classes
    W, V = _randn(g, classes, rank, n), _randn(g, classes, rank, per)
    At = 0.05 * _randn(g, classes, per, n)
    for r in range(rank):
        At += V[:, r, :, None] * W[:, r, None, :]
    At = _unit_rows(At.reshape(classes * per, n)).contiguous()
    cls = torch.randint(0, classes, (p,), generator=g, device="cuda")
    w = _randn(g, p, rank)
    s = torch.zeros(p, n, device="cuda")
    for r in range(rank):
        s += w[:, r, None] * W[cls, r]
    Bt = (_unit_rows(s) + 0.05 * _unit_rows(_randn(g, p, n))).contiguous()
    supp = cls[:, None] * per + torch.rand(p, per, generator=g, device="cuda").topk(rank, dim=1).indices
    return At, Bt, supp


def _data(case, seed):
    g = _gen(seed)
    return (_face if "classes" in case else _gauss)(case, g) + (g,)


def _net(case, At, g):
    """The projection and the flat parameters of a network early in its training, and the proposal's net."""
    d, h, m = case["d"], case["h"], case["m"]
    P = _randn(g, m, d) / math.sqrt(d)
    parts = [_randn(g, h, d) / math.sqrt(d), torch.zeros(h, device="cuda"), _randn(g, h, h) / math.sqrt(h),
             torch.zeros(h, device="cuda"), _randn(g, m, h) / math.sqrt(h),
             torch.full((m,), math.log(10.0 / m), device="cuda")]
    return P, torch.cat([q.reshape(-1) for q in parts])


def prepare(case, seed):
    At, Bt, supp, g = _data(case, seed)
    kind = case["kind"]
    if kind == "setup":
        return dict(case=case, At=At)
    if kind == "correlate":
        return dict(case=case, R=Bt, solver=pk.Solver(At, 0.1, screen=case["screen"]))
    if kind in ("train", "scores"):
        P, params = _net(case, At, g)
        net = pk.ProposalNet(At, P, case["h"], max_batch=case["p"])
        net.set_params(params)
        lens = torch.full((case["p"],), supp.shape[1], dtype=torch.int32, device="cuda")
        return dict(case=case, net=net, B=Bt, supp=supp.int().contiguous(), lens=lens)
    if kind == "classify":
        solver = pk.Solver(At, 0.01, mode="rel", screen="bf16", graph=True, max_outer=8)
        per = case["m"] // case["classes"]
        return dict(case=case, B=Bt, solver=solver, code=solver.solve(Bt),
                    cls=(torch.arange(case["m"], device="cuda") // per).int())
    solver = pk.Solver(At, case["c"], mode="rel", rho=case["rho"], screen=case["screen"], graph=case["graph"],
                       max_outer=case["max_outer"], omega=case["omega"])
    if case["tune"]:
        solver.autotune(case["p"])
    warm = None
    if case["warm_k"]:   # a proposal that holds most of the support and other atoms
        good = supp[:, : case["warm_k"] * 3 // 4]
        rest = torch.randint(0, case["m"], (case["p"], case["warm_k"] - good.shape[1]), generator=g, device="cuda")
        warm = torch.cat([good, rest], 1).int().sort(1).values.contiguous()
    return dict(case=case, solver=solver, B=Bt, warm=warm)


def run(state):
    kind = state["case"]["kind"]
    if kind == "solve":
        out = state["solver"].solve(state["B"], warm=state["warm"])
        # kkt is left out: at a natural stop it is the rounding of the certificate itself (about 1e-13)
        return {k: out[k] for k in ("x_val", "x_idx", "supp_len", "iters", "lambda", "objective", "status")}
    if kind == "correlate":
        return state["solver"].correlate(state["R"])
    if kind == "classify":
        return state["solver"].classify(state["B"], state["code"], state["cls"])
    if kind == "train":
        net = state["net"]
        loss, grad = net.loss_grad(state["B"], state["supp"], state["lens"], 20.0)
        net.adam_step(1e-3, grad=grad)
        return loss, grad
    if kind == "scores":
        scores = state["net"].forward(state["B"])
        return scores, pk.topk(scores, state["case"]["k"])
    solver = pk.Solver(state["At"], 0.02, mode="rel", screen=state["case"]["screen"])
    gram = solver.gram_table()
    solver.close()
    return gram


def work(case):
    """Each input read once, each output written once, and the arithmetic the path cannot avoid."""
    kind, n, m, p = case["kind"], case["n"], case["m"], case.get("p", 0)
    if kind == "solve":
        # a pass over the dictionary for every rho atoms of the support, one more for the stop; the master
        # problem's residuals; results of min(2n, m, n) slots per signal
        k = 0.5 * (case["k_lo"] + case["k_hi"])
        its = (0 if case["warm_k"] else math.ceil(k / case["rho"])) + 1
        return {"bytes": (4 if case["screen"] == "fp32" else 2) * m * n + 4.0 * n * p + 8.0 * min(m, n) * p,
                "flops": 2.0 * m * n * p * its + 2.0 * n * k * p * its}
    if kind == "correlate":
        e = 4 if case["screen"] == "fp32" else 2
        return {"bytes": e * m * n + 4.0 * n * p + 4.0 * m * p, "flops": 2.0 * m * n * p}
    if kind == "classify":
        return {"bytes": 4.0 * (m * n + n * p) + 100.0 * p, "flops": 2.0 * 10 * n * p}
    if kind == "setup":
        return {"bytes": 4.0 * m * n + 2 * 8.0 * m * m, "flops": 1.0 * m * m * n}
    d, h = case["d"], case["h"]
    weights = h * d + h * h + m * h
    fwd = 2.0 * p * (n * d + weights)
    if kind == "scores":
        return {"bytes": 2.0 * (n * d + weights) + 4.0 * p * (n + m + case["k"]), "flops": fwd}
    # a step: forward, both backward products, the float32 weights and moments read and written
    return {"bytes": 4.0 * n * p + 2.0 * weights + (4 * 4 + 4 * 3 + 2) * weights, "flops": 3 * fwd}


# ------------------------------------------------------------------------------------------------------------
# The same results in 64 bits, in plain torch
# ------------------------------------------------------------------------------------------------------------
def _lasso64(A, B, lam):
    """min 1/2 ||b - A^T x||^2 + lam ||x||_1 for every row b of B (rows of A: atoms), by a sign-fixed active set;
    dense (p, m), or None where the optimality conditions do not come out."""
    p, m = B.shape[0], A.shape[0]
    X = torch.zeros(p, m, dtype=torch.float64, device=A.device)
    beta, S = B @ A.T, torch.zeros(p, m, dtype=torch.bool, device=A.device)
    sign = torch.zeros_like(X)
    for _ in range(150):
        g = (B - X @ A) @ A.T
        viol = (g.abs() > lam[:, None] * (1 + 1e-10)) & ~S
        if not viol.any():
            break
        score = torch.where(viol, g.abs(), torch.zeros_like(g))
        top = score.topk(min(8, m), dim=1)
        for j in range(top.indices.shape[1]):
            rows = (top.values[:, j] > 0).nonzero()[:, 0]
            S[rows, top.indices[rows, j]] = True
            sign[rows, top.indices[rows, j]] = g[rows, top.indices[rows, j]].sign()
        for _ in range(50):
            K = int(S.sum(1).max())
            idx = S.to(torch.int8).topk(K, dim=1).indices
            live = torch.gather(S, 1, idx)
            x = torch.zeros(p, K, dtype=torch.float64, device=A.device)
            for r0 in range(0, p, 64):
                sl = slice(r0, r0 + 64)
                a = A[idx[sl]] * live[sl, :, None]
                gram = torch.bmm(a, a.transpose(1, 2).contiguous()) + torch.diag_embed((~live[sl]).double())
                rhs = (torch.gather(beta[sl], 1, idx[sl]) - lam[sl, None] * torch.gather(sign[sl], 1, idx[sl])) * live[sl]
                x[sl] = torch.cholesky_solve(rhs[:, :, None], torch.linalg.cholesky(gram))[:, :, 0]
            bad = live & (x * torch.gather(sign, 1, idx) <= 0)
            if not bad.any():
                break
            S.scatter_(1, idx, live & ~bad)
        X = torch.zeros_like(X).scatter_(1, idx, x * live)
    g = (B - X @ A) @ A.T
    on, off = ((g - lam[:, None] * sign).abs() * S).amax(1), (g.abs() * ~S).amax(1)
    return X if bool(((on <= 1e-8 * lam) & (off <= lam * (1 + 1e-8))).all()) else None


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        k = case["k_hi"]
        if case["dict"] != "gauss" or case["p"] * k * k * case["n"] > 3e10:
            return None
        At, Bt, _, _ = _data(case, seed)
        A, B = At.double(), Bt.double()
        lam = case["c"] * (B @ A.T).abs().amax(1)
        X = _lasso64(A, B, lam)
        if X is None:
            return None
        ld = min(case["m"], case["n"])
        order = (X == 0).to(torch.int8).sort(dim=1, stable=True).indices[:, :ld]
        obj = 0.5 * (B - X @ A).square().sum(1) + lam * X.abs().sum(1)
        return {"x_val": torch.gather(X, 1, order), "x_idx": None, "supp_len": None, "iters": None, "lambda": lam,
                "objective": obj, "status": None}
    At, Bt, supp, g = _data(case, seed)
    if kind == "correlate":
        return Bt.double() @ At.double().T
    if kind == "setup":
        return At.double() @ At.double().T
    if kind == "classify":
        return None
    P, params = _net(case, At, g)
    d, h, m, p = case["d"], case["h"], case["m"], case["p"]
    z = Bt.double() @ (P.double().T @ At.double()).T
    z = z * math.sqrt(d) / z.square().sum(1, keepdim=True).sqrt()
    flat = params.double().requires_grad_(kind == "train")
    w1, b1, w2, b2, w3, b3 = torch.split(flat, [h * d, h, h * h, h, m * h, m])
    gelu = torch.nn.functional.gelu
    u = gelu(z @ w1.view(h, d).T + b1)
    u = gelu(u @ w2.view(h, h).T + b2)
    s = u @ w3.view(m, h).T + b3
    if kind == "scores":
        return s, None
    y = torch.zeros(p, m, dtype=torch.float64, device="cuda").scatter_(1, supp, 1.0)
    w = torch.tensor(20.0, dtype=torch.float64, device="cuda")
    loss = torch.nn.functional.binary_cross_entropy_with_logits(s, y, pos_weight=w, reduction="sum") / p
    loss.backward()
    return loss.detach().reshape(1), flat.grad
