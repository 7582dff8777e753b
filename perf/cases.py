"""Performance cases of the SpAMM library: what its users run, through the
public Python binding, over the sizes, leaves and precisions it supports.

Kinds of work:
  product    one `multiply` call per product, result buffers allocated by the call
  staged     `prepare(schedule=True)` + `execute_scheduled` with kept buffers
  precision  `multiply_precision` (bf16 or f16x3) with a kept split buffer
  batch      `Batch.run` over products of arbitrary sizes
  ratio      norm pyramids of A and B and the valid-ratio threshold search
  tau_error  norm pyramids and the threshold search for an error target
  train      one gradient and Adam step of the threshold network

Matrices: `exp` is exp(-alpha |i-j|) (0.5 + 0.5 u), `alg` is +-1 / (1 + |i-j|)^2
and `paper` the symmetric Toeplitz matrix 0.1 / (|i-j|^0.1 + 1).
"""

import math

import numpy as np
import torch

from paper_2103_13042_amd import binding as sp
from paper_2103_13042_amd import inputs

DEV = "cuda"

# thresholds of the paper matrix at leaf 32: (n, kept share in per cent) -> tau
PAPER_TAU = {
    (1024, 30): 1.434815, (1024, 15): 1.521774, (1024, 5): 1.695691,
    (2048, 30): 1.310666, (2048, 15): 1.40003, (2048, 5): 1.548969,
    (4096, 30): 1.195803, (4096, 15): 1.277335, (4096, 5): 1.413222,
    (8192, 30): 1.093354, (8192, 15): 1.171746, (8192, 5): 1.28727,
}


def listed():
    return [
        # the smallest everyday call: one small banded product, where launches
        # and latency are all there is
        {"name": "exp300_leaf32", "kind": "product", "matrix": "exp", "alpha": 0.05, "n": 300, "leaf": 32, "tau": 1e-3},
        # a small product in a loop over many of them
        {"name": "exp1024_leaf32", "kind": "product", "matrix": "exp", "alpha": 0.05, "n": 1024, "leaf": 32,
         "tau": 1e-6},
        # the method's own evaluation matrix at 15 % kept pairs
        {"name": "paper4096_leaf32", "kind": "product", "matrix": "paper", "n": 4096, "leaf": 32, "tau": 1.277335},
        # the benchmark's workload, as a program that keeps its buffers runs it
        {"name": "alg8192_leaf64_staged", "kind": "staged", "matrix": "alg", "n": 8192, "leaf": 64, "tau": 1e-6},
        # a matrix size taken as it comes: odd, no multiple of any tile
        {"name": "alg5003_leaf64", "kind": "product", "matrix": "alg", "n": 5003, "leaf": 64, "tau": 1e-6},
        # the finest pruning (leaf 16)
        {"name": "exp2048_leaf16", "kind": "product", "matrix": "exp", "alpha": 0.05, "n": 2048, "leaf": 16,
         "tau": 1e-6},
        # slow decay with the coarsest leaf, ragged at the edge
        {"name": "exp6000_leaf128", "kind": "product", "matrix": "exp", "alpha": 0.01, "n": 6000, "leaf": 128,
         "tau": 1e-6},
        # the largest single product, in the accurate half-precision form
        {"name": "exp16384_f16x3", "kind": "precision", "precision": "f16x3", "matrix": "exp", "alpha": 0.01,
         "n": 16384, "leaf": 64, "tau": 1e-6},
        # many independent products of arbitrary sizes bound once, run per step
        {"name": "batch48", "kind": "batch", "count": 48, "specs": 13, "n_lo": 256, "n_hi": 4096, "leaf": 64,
         "tau": 1e-6},
        # picking tau for a wanted share of kept pairs on a new pair of matrices
        {"name": "ratio8192_leaf32", "kind": "ratio", "matrix": "paper", "n": 8192, "leaf": 32, "target": 0.15,
         "tol": 0.01},
        # picking tau for a wanted error (labels of the threshold network)
        {"name": "tau_error2048", "kind": "tau_error", "alpha": 0.05, "alpha_b": 0.2, "n": 2048, "leaf": 64,
         "target": 1e-4},
        # one step of training the threshold network
        {"name": "train256", "kind": "train", "batch": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["product", "staged", "precision", "batch", "ratio", "tau_error", "train"],
                       [9, 2, 3, 2, 1, 2, 1])[0]
    if kind == "product":
        matrix = rng.choice(["exp", "exp", "alg", "paper"])
        if matrix == "paper":
            n, share = rng.choice(sorted(PAPER_TAU))
            return {"kind": kind, "matrix": matrix, "n": n, "leaf": 32, "tau": PAPER_TAU[n, share]}
        leaf = rng.choice([16, 32, 32, 64, 64, 64, 128])
        n = _log_int(rng, 100, {16: 4000, 32: 6500, 64: 8300, 128: 8300}[leaf])
        if rng.random() < 0.4:  # a padded size, as much as one taken as it comes
            n = max(128, n // 128 * 128)
        case = {"kind": kind, "matrix": matrix, "n": n, "leaf": leaf, "tau": 10.0 ** rng.uniform(-7.5, -3.5)}
        if matrix == "exp":
            case["alpha"] = round(10.0 ** rng.uniform(-2.0, -0.4), 4)
        return case
    if kind == "staged":
        n = 128 * _log_int(rng, 8, 64)
        return {"kind": kind, "matrix": "alg", "n": n, "leaf": rng.choice([32, 64, 64, 128]),
                "tau": 10.0 ** rng.uniform(-6.5, -4.0)}
    if kind == "precision":
        return {"kind": kind, "precision": rng.choice(["bf16", "f16x3"]), "matrix": "exp",
                "alpha": round(10.0 ** rng.uniform(-1.9, -1.0), 4), "n": 128 * _log_int(rng, 8, 100), "leaf": 64,
                "tau": 10.0 ** rng.uniform(-6.0, -4.0)}
    if kind == "batch":
        lo = _log_int(rng, 64, 512)
        return {"kind": kind, "count": rng.randint(4, 48), "specs": rng.randint(14, 10000), "n_lo": lo,
                "n_hi": lo * rng.randint(1, 6), "leaf": rng.choice([32, 64, 64, 128]), "tau": 1e-6}
    if kind == "ratio":
        matrix = rng.choice(["paper", "exp"])
        case = {"kind": kind, "matrix": matrix, "n": _log_int(rng, 1000, 8300), "leaf": rng.choice([32, 64]),
                "target": round(rng.uniform(0.05, 0.3), 3), "tol": 0.01}
        if matrix == "exp":
            case["alpha"] = round(10.0 ** rng.uniform(-2.0, -1.0), 4)
        return case
    if kind == "tau_error":
        return {"kind": kind, "alpha": round(rng.uniform(0.01, 0.5), 4), "alpha_b": round(rng.uniform(0.01, 0.5), 4),
                "n": _log_int(rng, 700, 3000), "leaf": 64, "target": 10.0 ** rng.uniform(-5.5, -2.5)}
    return {"kind": kind, "batch": _log_int(rng, 16, 1024)}


# -- inputs -------------------------------------------------------------------


def _matrix(kind, n, alpha, seed):
    if kind == "exp":
        return inputs.exp_decay_torch(n, alpha, seed, torch.device(DEV))
    if kind == "paper":
        # the Toeplitz matrix has no seed of its own: its entries are scaled by
        # 1 +- 1e-4, which moves no threshold of interest and makes every pair new
        gen = torch.Generator(device=DEV).manual_seed(seed)
        u = torch.rand((n, n), generator=gen, device=DEV)
        return inputs.paper_algebraic_torch(n, torch.device(DEV)) * (1.0 + 1e-4 * (2.0 * u - 1.0))
    gen = torch.Generator(device=DEV).manual_seed(seed)
    d = torch.arange(n, dtype=torch.float32, device=DEV)
    out = torch.rand((n, n), generator=gen, device=DEV)
    out = torch.where(out < 0.5, -1.0, 1.0)
    return out.div_((1.0 + (d[:, None] - d[None, :]).abs_()).square_())


def _pair(case, seed):
    kind = case.get("matrix", "exp")
    a = _matrix(kind, case["n"], case.get("alpha", 0.0), 2 * seed)
    b = _matrix(kind, case["n"], case.get("alpha_b", case.get("alpha", 0.0)), 2 * seed + 1)
    return a, b


def _batch_specs(case):
    return inputs.batch_specs(case["count"], case["specs"], case["n_lo"], case["n_hi"])


def _batch_pairs(case, seed):
    dev = torch.device(DEV)
    out = []
    for q, (n, alpha_a, alpha_b, _, _) in enumerate(_batch_specs(case)):
        s = 1000 * seed + 2 * q
        out.append((inputs.exp_decay_torch(n, alpha_a, s, dev), inputs.exp_decay_torch(n, alpha_b, s + 1, dev)))
    return out


def _train_inputs(case, seed):
    """Network, optimiser state in the middle of training, and one minibatch:
    histogram features (most bins empty, the others up to the cap of 4) with
    the log10 of the error target, and log10 thresholds."""
    gen = torch.Generator(device="cpu").manual_seed(seed)
    rows, p = case["batch"], sp.mlp_param_count()
    hist = torch.rand((rows, 128), generator=gen) * 4.0
    hist = hist * (torch.rand((rows, 128), generator=gen) < 0.3)
    x = torch.cat([hist, -6.0 + 4.0 * torch.rand((rows, 1), generator=gen)], dim=1)
    t = -8.0 + 7.0 * torch.rand(rows, generator=gen)
    m = 1e-2 * torch.randn(p, generator=gen)
    v = 1e-3 * (0.1 + torch.rand(p, generator=gen))
    params = torch.from_numpy(inputs.mlp_init(seed))
    return [q.to(torch.float32).contiguous() for q in (params, x, t, m, v)]


def prepare(case, seed):
    kind, dev = case["kind"], torch.device(DEV)
    if kind == "train":
        params, x, t, m, v = (q.to(dev) for q in _train_inputs(case, seed))
        return {"case": case, "params": params, "x": x, "t": t, "m": m, "v": v, "acts": sp.mlp_acts(case["batch"], dev),
                "grad": torch.empty_like(params), "loss": torch.empty(1, device=dev)}
    if kind == "batch":
        pairs = _batch_pairs(case, seed)
        k = len(pairs)
        return {"case": case, "batch": sp.Batch([a for a, _ in pairs], [b for _, b in pairs], [case["leaf"]] * k,
                                                [case["tau"]] * k)}
    a, b = _pair(case, seed)
    state = {"case": case, "a": a, "b": b}
    n, leaf = case["n"], case["leaf"]
    if kind == "staged":
        state["bufs"] = sp.plan_buffers(n, leaf, dev)
        state["ws"] = torch.empty(sp.workspace_bytes(n, leaf), dtype=torch.uint8, device=dev)
        state["c"] = torch.empty_like(a)
    elif kind == "precision":
        state["split"] = sp.split_buffer(n, case["precision"], dev)
        state["c"] = torch.empty_like(a)
    elif kind == "tau_error":
        state["e"] = torch.empty_like(a)
        sp.multiply(a, b, 0.0, leaf, c=state["e"], sync=False)
        state["ab_sumsq"] = float(sp.sumsq(state["e"]).item())
    return state


# -- one pass -----------------------------------------------------------------


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "product":
        return sp.multiply(state["a"], state["b"], case["tau"], case["leaf"], sync=False)
    if kind == "staged":
        offsets, klist, pairs = sp.prepare(state["a"], state["b"], case["tau"], case["leaf"], bufs=state["bufs"],
                                           ws=state["ws"], schedule=True)
        c = sp.execute_scheduled(state["a"], state["b"], case["leaf"], offsets, klist, c=state["c"], ws=state["ws"])
        return c, pairs
    if kind == "precision":
        return sp.multiply_precision(state["a"], state["b"], case["tau"], case["leaf"], case["precision"],
                                     c=state["c"], split_buf=state["split"], sync=False)
    if kind == "batch":
        return state["batch"].run(), state["batch"].pairs
    if kind == "train":
        loss, grad = sp.mlp_loss_grad(state["params"], state["x"], state["t"], acts=state["acts"],
                                      grad=state["grad"], loss=state["loss"])
        sp.mlp_adam(state["params"], grad, state["m"], state["v"], 100, 1e-3)
        return loss, grad, state["params"], state["m"], state["v"]
    a, b, n, leaf = state["a"], state["b"], case["n"], case["leaf"]
    pa, pb = sp.pyramid(a, leaf), sp.pyramid(b, leaf)
    if kind == "ratio":
        return pa, pb, sp.search_valid_ratio(pa, pb, n, leaf, case["target"], case["tol"])
    return pa, pb, sp.search_tau_for_error(a, b, leaf, case["target"], pa, pb, state["ab_sumsq"], e=state["e"])


# -- the same in 64 bits, in plain torch --------------------------------------


def _leaf_norms(x, leaf):
    n = x.shape[0]
    b = -(-n // leaf)
    p = torch.zeros((b * leaf, b * leaf), dtype=torch.float64, device=x.device)
    p[:n, :n] = x
    return p.square_().view(b, leaf, b, leaf).sum(dim=(1, 3)).sqrt()


def _pyramid(norms):
    """Flat norm pyramid over the leaf norms, root first, zero padded to a power of two."""
    b, side = norms.shape[0], 1
    while side < b:
        side *= 2
    level = torch.zeros((side, side), dtype=torch.float64, device=norms.device)
    level[:b, :b] = norms.square()
    levels = [level.flatten().sqrt()]
    while side > 1:
        side //= 2
        level = level.view(side, 2, side, 2).sum(dim=(1, 3))
        levels.append(level.flatten().sqrt())
    return torch.cat(levels[::-1])


def _masked_product(a, b, leaf, keep_of):
    """C and the kept pairs of the leaf products that keep_of(norm products of one k) selects."""
    n = a.shape[0]
    na, nb = _leaf_norms(a, leaf), _leaf_norms(b, leaf)
    c = torch.zeros((n, n), dtype=torch.float64, device=a.device)
    count = torch.zeros(1, dtype=torch.int64, device=a.device)
    for k in range(na.shape[0]):
        keep = keep_of(na[:, k, None] * nb[None, k, :])
        count += keep.sum()
        rows = torch.nonzero(keep.any(dim=1)).flatten().tolist()
        cols = torch.nonzero(keep.any(dim=0)).flatten().tolist()
        if not rows:
            continue
        i0, i1, j0, j1 = rows[0], rows[-1] + 1, cols[0], cols[-1] + 1
        r0, r1, c0, c1 = i0 * leaf, min(n, i1 * leaf), j0 * leaf, min(n, j1 * leaf)
        ks = slice(k * leaf, min(n, (k + 1) * leaf))
        part = a[r0:r1, ks].double() @ b[ks, c0:c1].double()
        box = keep[i0:i1, j0:j1]
        if not bool(box.all()):
            part *= box.repeat_interleave(leaf, 0)[: r1 - r0].repeat_interleave(leaf, 1)[:, : c1 - c0]
        c[r0:r1, c0:c1] += part
    return c, count


def _exact_train(case, seed):
    params, x, t, m, v = (q.double() for q in _train_inputs(case, seed))
    params.requires_grad_(True)
    at, parts = 0, []
    for shape in inputs.MLP_SHAPES:
        k = int(np.prod(shape))
        parts.append(params[at:at + k].view(shape))
        at += k
    h = torch.nn.functional.gelu(x @ parts[0].t() + parts[1])
    h = torch.nn.functional.gelu(h @ parts[2].t() + parts[3])
    loss = ((h @ parts[4] + parts[5]) - t).square().mean()
    (grad,) = torch.autograd.grad(loss, params)
    b1, b2, eps, lr, step = 0.9, 0.999, 1e-8, 1e-3, 100
    m = b1 * m + (1 - b1) * grad
    v = b2 * v + (1 - b2) * grad.square()
    p = params.detach() - lr * (m / (1 - b1 ** step)) / ((v / (1 - b2 ** step)).sqrt() + eps)
    return loss.detach().reshape(1), grad, p, m, v


def _exact_ratio(case, seed):
    a, b = _pair(case, seed)
    na, nb = _leaf_norms(a, case["leaf"]), _leaf_norms(b, case["leaf"])
    total = float(na.shape[0]) ** 3

    def ratio(tau):
        return sum(int((na[:, k, None] * nb[None, k, :] >= tau).sum()) for k in range(na.shape[0])) / total

    ave = float((na.sum(dim=0) * nb.sum(dim=1)).sum()) / total
    target, tol, tau, k = case["target"], case["tol"], ave, 1
    r = ratio(tau)
    while r > target + tol and k < 1024:
        k += 1
        tau = k * ave
        r = ratio(tau)
    lo, hi = 0.0, k * ave
    for _ in range(20):
        if abs(r - target) <= tol:
            break
        tau = 0.5 * (lo + hi)
        r = ratio(tau)
        if r > target:
            lo = tau
        else:
            hi = tau
    return _pyramid(na), _pyramid(nb), (tau, None, None)


def _exact_tau_error(case, seed):
    """The largest norm product whose dropped leaf products stay within the target."""
    a, b = _pair(case, seed)
    leaf = case["leaf"]
    na, nb = _leaf_norms(a, leaf), _leaf_norms(b, leaf)
    whole = float((a.double() @ b.double()).norm())
    products = torch.unique((na[:, :, None] * nb[None, :, :]).flatten())
    products = products[products > 0].cpu().numpy()

    def error(tau):
        dropped, _ = _masked_product(a, b, leaf, lambda p: p < tau)
        return float(dropped.norm()) / whole

    lo, hi, err = 0, len(products), 0.0
    while hi - lo > 1:
        mid = (lo + hi) // 2
        e = error(float(products[mid]))
        if e <= case["target"]:
            lo, err = mid, e
        else:
            hi = mid
    return _pyramid(na), _pyramid(nb), (float(products[lo]), err, None, None)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "ratio":
        return _exact_ratio(case, seed)
    if kind == "tau_error":
        return _exact_tau_error(case, seed)
    if kind == "batch":
        both = [_masked_product(a, b, case["leaf"], lambda p: p >= case["tau"]) for a, b in _batch_pairs(case, seed)]
        return [c for c, _ in both], torch.cat([k for _, k in both])
    a, b = _pair(case, seed)
    return _masked_product(a, b, case["leaf"], lambda p: p >= case["tau"])


# -- what one pass cannot do without ------------------------------------------


def _tile_norm_by_distance(case, n, leaf, alpha):
    """Expected Frobenius norm of a leaf tile by its distance from the diagonal, 0 .. bdim-1."""
    b = -(-n // leaf)
    d = np.abs(np.arange(-(leaf - 1), b * leaf, dtype=np.float64))
    kind = case.get("matrix", "exp")
    if kind == "exp":
        sq = np.exp(-2.0 * alpha * d) * (7.0 / 12.0)
    elif kind == "alg":
        sq = (1.0 + d) ** -4.0
    else:
        sq = (0.1 / (d ** 0.1 + 1.0)) ** 2
    w = leaf - np.abs(np.arange(-(leaf - 1), leaf))
    return np.sqrt(np.array([np.dot(sq[t * leaf:t * leaf + 2 * leaf - 1], w) for t in range(b)]))


def _kept(case, n, leaf, tau, alpha=0.0, alpha_b=None):
    """Kept tile products (i, k, j), from the expected tile norms."""
    fa = _tile_norm_by_distance(case, n, leaf, alpha)
    fb = _tile_norm_by_distance(case, n, leaf, alpha if alpha_b is None else alpha_b)
    b = len(fa)
    # for a distance p = |i - k| the largest distance q = |k - j| that is kept
    reach = np.searchsorted(-fb, -(tau / np.maximum(fa, 1e-300)), side="right") - 1
    total = 0
    for p in range(b):
        q = int(reach[p])
        if q < 0:
            continue
        k = np.arange(b)
        cols = np.minimum(k, q) + np.minimum(b - 1 - k, q) + 1
        rows = (k >= p).astype(int) + ((k + p) < b).astype(int) if p else np.ones(b, dtype=int)
        total += int(np.dot(rows, cols))
    return total


def work(case):
    kind = case["kind"]
    if kind == "train":
        rows, p = case["batch"], 129 * 128 + 128 + 128 * 128 + 128 + 128 + 1
        return {"bytes": 4.0 * (rows * 130 + 7 * p + 1), "flops": 2.0 * rows * (2 * 129 * 128 + 3 * 128 * 128 + 3 * 128)}
    if kind == "batch":
        flops = bytes_ = 0.0
        for n, alpha_a, alpha_b, _, _ in _batch_specs(case):
            leaf = case["leaf"]
            kept = _kept(case, n, leaf, case["tau"], alpha_a, alpha_b)
            flops += 2.0 * kept * leaf * leaf * min(leaf, n)
            bytes_ += 12.0 * n * n
        return {"bytes": bytes_, "flops": flops}
    n, leaf = case["n"], case["leaf"]
    b = -(-n // leaf)
    if kind == "ratio":
        return {"bytes": 8.0 * n * n, "flops": 2.0 * 2.0 * n * n + 2.0 * float(b) ** 2}
    if kind == "tau_error":
        # the norms, and at least the error of the threshold it returns
        return {"bytes": 8.0 * n * n, "flops": 2.0 * n ** 3}
    kept = _kept(case, n, leaf, case["tau"], case.get("alpha", 0.0))
    per = 3.0 if case.get("precision") == "f16x3" else 1.0
    return {"bytes": 12.0 * n * n, "flops": 2.0 * per * kept * float(leaf) ** 3}
