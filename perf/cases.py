"""Timed cases of the library's public entry points over the range its users meet.

A case is one rating matrix (shape, number of ratings, law of the degrees), a factor width
and what is done with it: a sweep of plain, weighted or tensor ALS, a Gibbs iteration of
BPMF or BPTF, the RMSE over the training and validation ratings, or predictions. Inputs are
synthetic and made on the GPU from the seed: degrees and ratings follow the laws of the
data the method was published on (lognormal users and Zipf items on 1.0M x 625k x 263M;
ratings 0..100, 30 % of them zero), factors start from N(0, 0.1).

``exact`` repeats a pass in 64 bits with plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1108_2580_amd import ALS

DEV = "cuda:0"

# Hyperpriors of the Gibbs cases: those of the repository's benchmark.
BETA0, ALPHA, ALPHA_W0, ALPHA_NU0 = 2.0, 0.01, 1.0, 2.0


def listed():
    return [
        # the smallest training sweep anyone runs: a 50 000-rating set; launches and latency
        dict(name="als_tiny_d10", task="als", users=2_000, items=1_000, ratings=50_000,
             law="uniform", width=10, lam=0.05),
        # an ordinary training sweep: 10M ratings with Zipf users and items
        dict(name="als_mid_d20", task="als", users=100_000, items=50_000, ratings=10_000_000,
             law="zipf", width=20, lam=0.065),
        # the published data set's shape, the sweep that the library's headline is quoted on
        dict(name="als_full_d20", task="als", users=1_000_990, items=624_961,
             ratings=262_810_175, law="lognormal", width=20, lam=0.065),
        # the wide model on a quarter of that data set (a user sample, or one GPU's share)
        dict(name="als_quarter_d100", task="als", users=250_248, items=156_240,
             ratings=65_702_544, law="lognormal", width=100, lam=0.065),
        # the widest model on data with items rated by every user
        dict(name="als_hub_d128", task="als", users=100_000, items=40_000, ratings=10_000_000,
             law="hub", width=128, lam=0.05),
        # a small set at an odd width, with the RMSE of the new state after each sweep
        # (the monitored training loop)
        dict(name="als_small_rmse_d33", task="als_rmse", users=20_011, items=9_973,
             ratings=1_000_003, law="lognormal", width=33, lam=0.065),
        # weighted ALS (confidence per rating) at an ordinary size
        dict(name="weighted_mid_d50", task="weighted", users=60_000, items=30_000,
             ratings=5_000_000, law="zipf", width=50, lam=0.065),
        # one BPMF Gibbs iteration: both hyperparameter draws and both sides' row draws
        dict(name="bpmf_mid_d100", task="bpmf", users=100_000, items=50_000,
             ratings=10_000_000, law="lognormal", width=100),
        # a tensor ALS sweep (items, users, time bins) on a small time-stamped set
        dict(name="tensor_small_d10", task="tensor", users=20_000, items=10_000,
             ratings=1_000_000, law="lognormal", width=10, bins=500, lam=0.05),
        # one BPTF iteration with the published data set's 6649 time bins
        dict(name="bptf_mid_d20", task="bptf", users=100_000, items=50_000,
             ratings=10_000_000, law="zipf", width=20, bins=6_649),
        # model selection: training RMSE and the RMSE of 200 000 held-out ratings
        dict(name="validate_mid_d50", task="validate", users=100_000, items=50_000,
             ratings=10_000_000, law="zipf", width=50, pairs=200_000),
        # scoring a list of 4M (user, item) pairs, grouped by user, with tables of full size
        dict(name="predict_full_d20", task="predict", users=1_000_990, items=624_961,
             ratings=4_000_000, law="lognormal", width=20, pairs=4_106_408),
    ]


def draw(rng):
    def log_int(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    task = rng.choice(["als", "als", "als_rmse", "weighted", "bpmf", "tensor", "bptf",
                       "validate", "predict"])
    width = rng.randint(*rng.choice([(1, 20), (10, 20), (21, 64), (65, 128)]))
    ratings = log_int(50_000, 30_000_000)
    mean = math.exp(rng.uniform(math.log(20), math.log(250)))
    users = int(max(ratings / mean, math.sqrt(60.0 * ratings)))  # at most 6 % of the positions
    items = int(users * rng.uniform(0.3, 1.0))
    case = dict(task=task, users=users, items=items, ratings=ratings, width=width,
                law=rng.choice(["uniform", "zipf", "lognormal", "hub"]))
    if task in ("als", "als_rmse", "weighted", "tensor"):
        case["lam"] = round(rng.uniform(0.03, 0.1), 4)
    if task in ("tensor", "bptf"):
        case["ratings"] = min(ratings, 10_000_000)
        case["bins"] = log_int(50, 6_649)
    if task in ("validate", "predict"):
        case["pairs"] = log_int(1_000, 4_000_000)
    return case


# ---- inputs --------------------------------------------------------------------------------

def _clamped(raw, lo, hi, total):
    """raw scaled so that its values, clamped to [lo, hi], add up to total."""
    a, b = 0.0, total / max(float(raw.min()), 1e-12)
    for _ in range(100):
        m = 0.5 * (a + b)
        if float((raw * m).clamp(lo, hi).sum()) < total:
            a = m
        else:
            b = m
    return (raw * b).clamp(lo, hi)


def _keys(n_rows, n_cols, deg, weights, gen):
    """row * n_cols + column of about deg[r] draws in each row r, columns by weight; a row
    that asks for more than an eighth of the columns takes each with equal probability."""
    dense = torch.nonzero(deg > n_cols / 8).flatten()
    parts = []
    for r in dense.split(max(1, 100_000_000 // n_cols)):
        hit = torch.rand((r.numel(), n_cols), generator=gen, device=DEV) < (deg[r] / n_cols)[:, None]
        at = torch.nonzero(hit)
        parts.append(r[at[:, 0]] * n_cols + at[:, 1])
    light = deg.clone()
    light[dense] = 0.0
    count = torch.floor(light * 1.12 + torch.rand(n_rows, generator=gen, device=DEV,
                                                  dtype=torch.float64)).long()
    rows = torch.repeat_interleave(torch.arange(n_rows, device=DEV), count)
    cum = torch.cumsum(weights, 0)
    at = torch.rand(rows.numel(), generator=gen, device=DEV, dtype=torch.float64) * cum[-1]
    parts.append(rows * n_cols + torch.searchsorted(cum, at).clamp_(max=n_cols - 1))
    return torch.cat(parts)


def _matrix(case, seed):
    """(row_ptr, rows, col, val) on the GPU: the ratings in user order."""
    M, N, nnz, law = case["users"], case["items"], case["ratings"], case["law"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    f64 = dict(device=DEV, dtype=torch.float64)

    def ranks(n):
        return 1.0 + torch.randperm(n, generator=gen, device=DEV).double()

    if law == "hub":  # item degrees ~ r^-1.5, the top ones rated by every user; users r^-0.6
        deg = _clamped(ranks(N) ** -1.5, 1.0, float(M), nnz)
        key = _keys(N, M, deg, ranks(M) ** -0.6, gen)
        key = (key % M) * N + torch.div(key, M, rounding_mode="floor")
    else:
        if law == "uniform":
            deg, weights = torch.full((M,), nnz / M, **f64), torch.ones(N, **f64)
        elif law == "zipf":
            deg = _clamped(1.0 / ranks(M), min(5.0, nnz / M), N / 2.0, nnz)
            weights = torch.clamp(1.0 / ranks(N), min=0.25 / N ** 0.5)
        else:  # lognormal users around a median of half the mean, Zipf-Mandelbrot items
            sigma = math.sqrt(2.0 * math.log(2.0))
            raw = torch.exp(sigma * torch.randn(M, generator=gen, **f64))
            deg = _clamped(raw, min(10.0, nnz / M), N / 10.0, nnz)
            weights = (ranks(N) + 32.0) ** -1.1
        key = _keys(M, N, deg, weights, gen)
    key = torch.sort(key).values
    key = key[torch.cat([torch.ones(1, dtype=torch.bool, device=DEV), key[1:] != key[:-1]])]
    if key.numel() > nnz:  # thinned evenly to the number asked for
        key = key[torch.div(torch.arange(nnz, device=DEV) * key.numel(), nnz,
                            rounding_mode="floor")]
    rows = torch.div(key, N, rounding_mode="floor")
    col = (key - rows * N).int()
    ptr = torch.zeros(M + 1, dtype=torch.int64, device=DEV)
    ptr[1:] = torch.cumsum(torch.bincount(rows, minlength=M), 0)
    a = torch.rand(col.numel(), generator=gen, device=DEV)
    b = torch.rand(col.numel(), generator=gen, device=DEV)
    val = torch.where(a < 0.3, torch.zeros_like(b),
                      torch.where(a < 0.5, 90 + torch.floor(b * 11), 1 + torch.floor(b * 89)))
    return ptr, rows, col, val.clamp_(max=100).byte()


def _inputs(case, seed):
    """Everything a pass reads, on the GPU (host arrays where the library takes those)."""
    M, N, D, task = case["users"], case["items"], case["width"], case["task"]
    ptr, rows, col, val = _matrix(case, seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed + 1)
    rng = np.random.default_rng(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device=DEV)

    s = dict(ptr=ptr, rows=rows, col=col, val=val, U=0.1 * normal(M, D), V=0.1 * normal(N, D))
    nnz = col.numel()
    if task == "weighted":  # confidences, log-uniform on [0.25, 4)
        s["w"] = torch.exp2(4.0 * torch.rand(nnz, generator=gen, device=DEV) - 2.0)
    if task in ("tensor", "bptf"):  # every user starts at some bin and stays for a while
        K = case["bins"]
        start = torch.randint(0, K, (M,), generator=gen, device=DEV)
        spread = -torch.log(1.0 - torch.rand(nnz, generator=gen, device=DEV)) * (0.045 * K)
        s["bins"] = (start[rows] + spread.long()).clamp_(max=K - 1).int()
        s["T"] = 1.0 + 0.1 * normal(K, D)
    if task in ("bpmf", "bptf"):
        sides = dict(items=N, users=M)
        if task == "bptf":
            sides["time"] = case["bins"]
            s["chi2_alpha"] = float(rng.chisquare(ALPHA_NU0 + nnz))
        for side, n in sides.items():
            s["z_" + side] = normal(n, D)
            s["var_" + side] = tuple(torch.from_numpy(np.atleast_1d(a)).to(DEV) for a in (
                rng.chisquare(D + n - np.arange(D)), rng.normal(size=D * (D - 1) // 2),
                rng.normal(size=D)))
    if task in ("validate", "predict"):
        # held-out pairs with the degree distributions of both sides, grouped by user
        at = torch.randint(0, nnz, (case["pairs"],), generator=gen, device=DEV)
        at = torch.sort(at).values
        s["pu"] = rows[at].int()
        s["pi"] = col[torch.randint(0, nnz, (case["pairs"],), generator=gen, device=DEV)]
        s["pr"] = torch.randint(0, 101, (case["pairs"],), generator=gen, device=DEV).byte()
        # a trained model's predictions spread around the ratings' mean
        s["U"] = s["U"] + 6.0 / D ** 0.5
        s["V"] = s["V"] + 6.0 / D ** 0.5
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    D, task = case["width"], case["task"]
    als = ALS(case["users"], case["items"], s["ptr"].cpu().numpy(), s["col"].cpu().numpy(),
              s["val"].cpu().numpy(), D)
    state = dict(als=als, task=task, U=s["U"], V=s["V"])
    if "lam" in case:
        state["lam"] = case["lam"]
    if task == "weighted":
        als.set_weights(s["w"].cpu().numpy())
    if task in ("tensor", "bptf"):
        als.set_time_bins(case["bins"], s["bins"].cpu().numpy())
        state["T"] = s["T"]
    if task in ("bpmf", "bptf"):
        for side in ("items", "users") + (("time",) if task == "bptf" else ()):
            als.set_nw_prior(side, np.full(D, float(side == "time")), BETA0, np.eye(D), float(D))
            state["z_" + side], state["var_" + side] = s["z_" + side], s["var_" + side]
            state["mu_" + side] = torch.empty(D, dtype=torch.float64, device=DEV)
            state["Lambda_" + side] = torch.empty((D, D), dtype=torch.float64, device=DEV)
        state["chi2_alpha"] = s.get("chi2_alpha")
    if task == "validate":
        als.set_holdout(s["pu"].cpu().numpy(), s["pi"].cpu().numpy(), s["pr"].cpu().numpy())
    if task == "predict":
        state["pu"], state["pi"] = s["pu"], s["pi"]
    return state


# ---- one pass ------------------------------------------------------------------------------

def run(state):
    als, task, U, V = state["als"], state["task"], state["U"], state["V"]
    if task in ("als", "weighted"):
        als.half_sweep("items", U, state["lam"], V)
        als.half_sweep("users", V, state["lam"], U)
        return dict(U=U, V=V, rmse=als.rmse_in())
    if task == "als_rmse":
        als.half_sweep("items", U, state["lam"], V)
        rmse = als.half_sweep("users", V, state["lam"], U, rmse=True)
        return dict(U=U, V=V, rmse=rmse)
    if task == "tensor":
        T = state["T"]
        for mode in ("items", "users", "bins"):
            als.tensor_half_sweep(mode, U, V, T, state["lam"])
        return dict(U=U, V=V, T=T, rmse=als.rmse_in())
    if task == "bpmf":
        for side, fixed, out in (("items", U, V), ("users", V, U)):
            mu, Lam = state["mu_" + side], state["Lambda_" + side]
            als.sample_hyper(side, out, *state["var_" + side], mu, Lam)
            als.gibbs_half_sweep(side, fixed, ALPHA, Lam, mu, state["z_" + side], out)
        return dict(U=U, V=V, rmse=als.rmse_in(),
                    mu=[state["mu_items"], state["mu_users"]],
                    Lambda=[state["Lambda_items"], state["Lambda_users"]])
    if task == "bptf":
        T = state["T"]
        alpha = als.tensor_sample_alpha(U, V, T, ALPHA_W0, state["chi2_alpha"])
        for side, X in (("items", V), ("users", U), ("time", T)):
            als.sample_hyper(side, X, *state["var_" + side], state["mu_" + side],
                             state["Lambda_" + side])
        for mode, side in (("items", "items"), ("users", "users"), ("bins", "time")):
            als.tensor_gibbs_half_sweep(mode, U, V, T, alpha, state["Lambda_" + side],
                                        state["mu_" + side], state["z_" + side])
        return dict(U=U, V=V, T=T, rmse=als.rmse_in(), alpha=alpha,
                    mu=[state["mu_" + k] for k in ("items", "users", "time")],
                    Lambda=[state["Lambda_" + k] for k in ("items", "users", "time")])
    if task == "validate":
        return dict(train=als.rmse(U, V), held_out=als.holdout_rmse(U, V))
    return als.predict(U, V, state["pu"], state["pi"])


def work(case):
    """Per pass: every index, rating, weight and bin once per half-sweep that walks them,
    every factor table once per read and write; normal equations as D (D + 1) flops per
    rating (symmetric), right-hand side and residual 2 D each, D^3 / 3 + 2 D^2 per row."""
    M, N, nnz, D, task = (case[k] for k in ("users", "items", "ratings", "width", "task"))
    K = case.get("bins", 0)
    row = D ** 3 / 3 + 2 * D * D
    gram = nnz * (D * (D + 1.0) + 4 * D)
    if task in ("als", "als_rmse", "weighted"):
        per = 9 if task == "weighted" else 5
        more = 1 if task == "als_rmse" else 0  # the new state's residuals
        return {"bytes": (2 + more) * per * nnz + 4 * D * (M + N) * (3 + more),
                "flops": 2 * gram + (M + N) * row + more * 2 * D * nnz}
    if task == "bpmf":
        return {"bytes": 2 * 5 * nnz + 4 * D * (M + N) * 5,
                "flops": 2 * gram + (M + N) * (row + D * D)}
    if task == "tensor":
        return {"bytes": 3 * 9 * nnz + 4 * D * (M + N + K) * 4,
                "flops": 3 * (gram + nnz * D) + (M + N + K) * row}
    if task == "bptf":
        return {"bytes": 4 * 9 * nnz + 4 * D * (M + N + K) * 6,
                "flops": 3 * (gram + nnz * D) + 3 * nnz * D + (M + N + K) * (row + D * D)}
    if task == "validate":
        return {"bytes": 5 * nnz + 9 * case["pairs"] + 2 * 4 * D * (M + N),
                "flops": 2.0 * D * (nnz + case["pairs"])}
    pairs = case["pairs"]
    return {"bytes": 12 * pairs + 4 * D * (min(M, pairs) + min(N, pairs)),
            "flops": 2.0 * D * pairs}


def tolerance(case):
    """About four times what was measured against ``exact`` and between schedules that sum in
    another order, over the listed and some 40 drawn cases, after one pass and after two.
    ALS's second half-sweep solves from the first one's rows, and the second pass from
    those: the systems' conditioning (up to 1e4 where light rows meet wide factors) travels
    through, while the first half-sweep's rows stay at 1e-7..1e-6. The Gibbs conditionals
    carry the prior's precision and stay near the data type's own error."""
    task = case["task"]
    if task in ("bpmf", "bptf"):  # seen: 2e-6 / 4e-5
        return {"rel": 1e-5, "max": 2e-4}
    if task == "validate":  # 1e-8
        return {"rel": 1e-7}
    if task == "predict":  # 1e-7 / 6e-7
        return {"rel": 5e-7, "max": 3e-6}
    if case["law"] == "uniform" or case["ratings"] >= 50 * case["users"]:  # 3e-4 / 1e-2
        return {"rel": 1.2e-3, "max": 0.05}
    return {"rel": 0.01, "max": 0.4}  # light rows: 3e-3 / 0.1


# ---- the same pass in 64 bits --------------------------------------------------------------

def _sse64(rows, idx, val, X, F, idx2=None, F2=None):
    total = 0.0
    step = max(1, 60_000_000 // X.shape[1])
    for a in range(0, idx.numel(), step):
        f = F[idx[a:a + step].long()]
        if idx2 is not None:
            f = f * F2[idx2[a:a + step].long()]
        e = val[a:a + step].double() - (X[rows[a:a + step]] * f).sum(1)
        total += float((e * e).sum())
    return total


def _cholesky(A):
    """Lower factors of a batch of symmetric positive definite matrices, in place."""
    D = A.shape[-1]
    for k in range(D):
        A[:, k:, k] /= A[:, k, k].sqrt()[:, None]
        A[:, k, k + 1:] = 0.0
        if k + 1 < D:
            c = A[:, k + 1:, k]
            A[:, k + 1:, k + 1:] -= c[:, :, None] * c[:, None, :]
    return A


def _rows64(ptr, idx, val, F, X, lam=None, w=None, idx2=None, F2=None, alpha=1.0, P0=None,
            h0=None, z=None, only=None, scale=None):
    """Every row's solution (ALS with lam; a Gibbs draw with P0, h0 and z), into X."""
    D = F.shape[1]
    deg = (ptr[1:] - ptr[:-1]).cpu()
    order = torch.argsort(deg, descending=True, stable=True)
    if only is not None:
        order = order[(order % 2) == only]
    if lam is not None:
        order = order[deg[order] > 0]
    sizes = deg[order].tolist()
    at = 0
    while at < len(sizes):
        L = max(1, sizes[at])
        B = int(max(1, min(len(sizes) - at, 40_000_000 // (max(L, D) * D), 30_000)))
        r = order[at:at + B].to(DEV)
        n = deg[order[at:at + B]].to(DEV)
        at += B
        on = torch.arange(L, device=DEV)[None, :] < n[:, None]
        pos = (ptr[r][:, None] + torch.arange(L, device=DEV)[None, :]).clamp_(max=max(0, idx.numel() - 1))
        f = F[idx[pos].long()]
        if idx2 is not None:
            f = f * F2[idx2[pos].long()]
        f = torch.where(on[:, :, None], f, torch.zeros((), dtype=torch.float64, device=DEV))
        g = f if w is None else f * w[pos][:, :, None].double()
        ft = g.transpose(1, 2).contiguous()
        A = torch.bmm(ft, f) * alpha
        b = torch.bmm(ft, val[pos][:, :, None].double())[:, :, 0] * alpha
        if lam is not None:
            A += (lam * n.double())[:, None, None] * torch.eye(D, device=DEV, dtype=torch.float64)
        else:
            A += P0 if scale is None else P0 * scale[r][:, None, None]
            b += h0 if h0.dim() == 1 else h0[r]
        Lc = _cholesky(A)
        for k in range(D):  # forward, then the variates, then backward
            b[:, k] = (b[:, k] - (Lc[:, k, :k] * b[:, :k]).sum(1)) / Lc[:, k, k]
        if z is not None:
            b = b + z[r].double()
        for k in range(D - 1, -1, -1):
            b[:, k] = (b[:, k] - (Lc[:, k + 1:, k] * b[:, k + 1:]).sum(1)) / Lc[:, k, k]
        X[r] = b


def _hyper64(mu0, mean, count, scatter, var, D):
    """(mu, Lambda) by Bartlett's construction; scatter: what W0^-1 = I grows by before the
    shrinkage term, count: the draws around mu, mean: theirs."""
    chi2, off, zmu = (t.cpu() for t in var)
    beta = BETA0 + count
    d = (mu0 - mean)[:, None]
    Winv = torch.eye(D, dtype=torch.float64) + scatter + BETA0 * count / beta * (d @ d.T)
    W = torch.linalg.inv(Winv)
    Fc = torch.linalg.cholesky(0.5 * (W + W.T))
    B = torch.zeros((D, D), dtype=torch.float64)
    i, j = torch.tril_indices(D, D, -1)
    B[i, j] = off
    B += torch.diag(chi2.sqrt())
    E = Fc @ B
    Lam = E @ E.T
    R = torch.linalg.cholesky(beta * Lam)
    mu = (BETA0 * mu0 + count * mean) / beta + torch.linalg.solve_triangular(
        R.T, zmu[:, None], upper=True)[:, 0]
    return mu.to(DEV), Lam.to(DEV)


def _side64(X, var, D):
    mean = X.mean(0)
    c = X - mean
    return _hyper64(torch.zeros(D, dtype=torch.float64), mean.cpu(), X.shape[0],
                    (c.T.contiguous() @ c).cpu(), var, D)


def exact(case, seed):
    s = _inputs(case, seed)
    M, N, D, task = case["users"], case["items"], case["width"], case["task"]
    U, V, nnz = s["U"].double(), s["V"].double(), s["col"].numel()
    ptr, rows, col, val = s["ptr"], s["rows"], s["col"], s["val"]
    lam = float(np.float32(case["lam"])) if "lam" in case else None
    if task == "predict":
        return (U[s["pu"].long()] * V[s["pi"].long()]).sum(1)
    if task == "validate":
        return dict(train=math.sqrt(_sse64(rows, col, val, U, V) / nnz),
                    held_out=math.sqrt(_sse64(s["pu"].long(), s["pi"], s["pr"], U, V) / case["pairs"]))

    def grouped(key, n):
        perm = torch.sort(key.long(), stable=True).indices
        p = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        p[1:] = torch.cumsum(torch.bincount(key.long(), minlength=n), 0)
        return p, perm

    iptr, perm = grouped(col, N)
    irow, ival = rows[perm].int(), val[perm]
    if task in ("als", "als_rmse", "weighted"):
        w = s.get("w")
        _rows64(iptr, irow, ival, U, V, lam, None if w is None else w[perm])
        rmse = math.sqrt(_sse64(rows, col, val, U, V) / nnz)
        _rows64(ptr, col, val, V, U, lam, w)
        if task == "als_rmse":
            rmse = math.sqrt(_sse64(rows, col, val, U, V) / nnz)
        return dict(U=U, V=V, rmse=rmse)
    if task == "bpmf":
        a = float(np.float32(ALPHA))
        mi, Li = _side64(V, s["var_items"], D)
        _rows64(iptr, irow, ival, U, V, alpha=a, P0=Li, h0=Li @ mi, z=s["z_items"])
        rmse = math.sqrt(_sse64(rows, col, val, U, V) / nnz)
        mu, Lu = _side64(U, s["var_users"], D)
        _rows64(ptr, col, val, V, U, alpha=a, P0=Lu, h0=Lu @ mu, z=s["z_users"])
        return dict(U=U, V=V, rmse=rmse, mu=[mi, mu], Lambda=[Li, Lu])
    T, K, bins = s["T"].double(), case["bins"], s["bins"]
    tptr, tperm = grouped(bins, K)
    tu, ti, tv = rows[tperm].int(), col[tperm], val[tperm]
    if task == "tensor":
        _rows64(iptr, irow, ival, U, V, lam, idx2=bins[perm], F2=T)
        _rows64(ptr, col, val, V, U, lam, idx2=bins, F2=T)
        rmse = math.sqrt(_sse64(rows, col, val, U, V, bins, T) / nnz)
        _rows64(tptr, tu, tv, U, T, lam, idx2=ti, F2=V)
        return dict(U=U, V=V, T=T, rmse=rmse)
    alpha = s["chi2_alpha"] / (1.0 / ALPHA_W0 + _sse64(rows, col, val, U, V, bins, T))
    a = float(np.float32(alpha))
    mi, Li = _side64(V, s["var_items"], D)
    mu, Lu = _side64(U, s["var_users"], D)
    step = T[1:] - T[:-1]
    mt, Lt = _hyper64(torch.ones(D, dtype=torch.float64), T[0].cpu(), 1,
                      (step.T.contiguous() @ step).cpu(), s["var_time"], D)
    _rows64(iptr, irow, ival, U, V, alpha=a, P0=Li, h0=Li @ mi, z=s["z_items"], idx2=bins[perm], F2=T)
    _rows64(ptr, col, val, V, U, alpha=a, P0=Lu, h0=Lu @ mu, z=s["z_users"], idx2=bins, F2=T)
    rmse = math.sqrt(_sse64(rows, col, val, U, V, bins, T) / nnz)
    scale = torch.full((K,), 2.0, device=DEV, dtype=torch.float64)
    scale[-1] = 1.0
    for parity in (0, 1):
        around = torch.cat([mt[None, :], T[:-1]])
        around[:-1] += T[1:]
        _rows64(tptr, tu, tv, U, T, alpha=a, P0=Lt, h0=around @ Lt, z=s["z_time"], idx2=ti, F2=V,
                only=parity, scale=scale)
    return dict(U=U, V=V, T=T, rmse=rmse, alpha=alpha, mu=[mi, mu, mt], Lambda=[Li, Lu, Lt])
