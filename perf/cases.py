"""Performance cases: what a program that compresses, queries and restores tensors asks of this framework.

A case is a dict of plain values with a ``kind``:

* ``compress``: `sthosvd` (or `sthosvd_ranks`) of a tensor in HBM and a reconstruction from the handle, the whole
  life of a compressed tensor;
* ``batch``: `Batch` over many small tensors, one run, every tensor's core and factors taken out;
* ``gram``, ``eig``, ``ttm``: the single steps, for programs that drive the mode loop themselves;
* ``reconstruct``: restoring a stored model (`from_model`), whole or a sub-range;
* ``preprocess``: hyperslice statistics and the rescaling of one mode, before a compression.

Inputs follow the synthetic recipe of the tests and the benchmark: a random core with decaying slices times
orthonormal factors, plus Gaussian noise below the requested error, so that the ranks are those of the planted core.
Sizes are those of the benchmark's workloads (64^3, 200^3 x 16, 256^3 x 11 x 50, 672 x 672 x 33 x T, batches of modes
16..128) and odd ones between them.  Sizes, orders and modes are in the paper's order (mode 0 fastest).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1901_06043_amd as tk

DEV = "cuda"
DTYPES = {"f32": torch.float32, "f64": torch.float64}


def _text(vals):
    return "x".join(str(int(v)) for v in vals)


def _ints(text):
    return [int(v) for v in str(text).split("x")]


def listed():
    return [
        # one small tensor: a single field or a patch of one, where launches and read-backs are what is waited for
        {"name": "compress_64", "kind": "compress", "dims": "64x64x64", "ranks": "8x8x8", "order": "0x1x2",
         "dtype": "f64", "prec": "fp64", "eps": 1e-4, "noise": 1e-6, "decay": 1.0, "given": False, "part": 1.0},
        # the synthetic tensor of the benchmark: modes of 200, a 50 x 50 x 50 window read back
        {"name": "compress_200", "kind": "compress", "dims": "200x200x200x16", "ranks": "20x20x20x8",
         "order": "0x1x2x3", "dtype": "f64", "prec": "fp64", "eps": 1e-4, "noise": 1e-5, "decay": 0.8,
         "given": False, "part": 0.25},
        # a simulation's share of one GPU (2 space, 33 variables, time), little compressible, restored whole
        {"name": "compress_672", "kind": "compress", "dims": "672x672x33x313", "ranks": "447x336x33x235",
         "order": "3x2x0x1", "dtype": "f32", "prec": "fp64", "eps": 2e-4, "noise": 1e-4, "decay": 0.99,
         "given": False, "part": 1.0},
        # a combustion-shaped field (3 space, variables, time) in the FP32 form, restored whole
        {"name": "compress_256_fp32", "kind": "compress", "dims": "256x256x256x11x50", "ranks": "27x27x27x11x12",
         "order": "0x1x2x3x4", "dtype": "f32", "prec": "fp32", "eps": 1e-3, "noise": 1e-4, "decay": 0.9,
         "given": False, "part": 1.0},
        # the same kind of field on an odd grid in the BF16x6 form, a window read back
        {"name": "compress_161_bf16x6", "kind": "compress", "dims": "161x161x160x11x25", "ranks": "23x22x21x11x9",
         "order": "0x1x2x3x4", "dtype": "f32", "prec": "bf16x6", "eps": 1e-3, "noise": 1e-4, "decay": 0.9,
         "given": False, "part": 0.5},
        # many small tensors at once, every result taken out of the plan
        {"name": "batch_96", "kind": "batch", "count": 96, "lo": 16, "hi": 128, "dtype": "f32", "prec": "fp64",
         "eps": 1e-3, "noise": 1e-4},
        # single steps: a small odd Gram (latency), a large one of double data with unit stride
        {"name": "gram_61", "kind": "gram", "dims": "57x61x43", "mode": 1, "dtype": "f64"},
        {"name": "gram_672", "kind": "gram", "dims": "672x448x33x64", "mode": 0, "dtype": "f64"},
        # the eigensolve of a large mode, three quarters of it kept
        {"name": "eig_626", "kind": "eig", "J": 626, "R": 469},
        # the first product of a compression: float data, last mode, odd rank
        {"name": "ttm_626", "kind": "ttm", "dims": "672x224x8x626", "mode": 3, "K": 469, "dtype": "f32"},
        # a stored model restored whole in single precision: small core, large output
        {"name": "reconstruct_256", "kind": "reconstruct", "dims": "256x256x256x11x50", "ranks": "27x27x27x11x12",
         "out": "f32", "part": 1.0},
        # standardising the 33 variables of a simulation before its compression
        {"name": "preprocess_33", "kind": "preprocess", "dims": "672x672x33x64", "mode": 2, "method": "standardize",
         "dtype": "f32"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_dims(rng, lo, hi, n_lo=3, n_hi=5, largest=672):
    """3 to 5 sizes with a product near a target drawn over its logarithm."""
    N = rng.randint(n_lo, n_hi)
    target = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    side = target ** (1.0 / N)
    dims = [max(8, min(largest, int(round(side * math.exp(rng.uniform(-0.6, 0.6)))))) for _ in range(N)]
    k = rng.randrange(N)
    rest = math.prod(dims) // dims[k]
    dims[k] = max(8, min(largest, int(target / rest)))
    return dims


def _draw_ranks(rng, dims):
    """Ranks of a tenth to a half of the sizes, each at most half the product of the others."""
    ranks = [max(2, int(d * rng.uniform(0.1, 0.5))) for d in dims]
    for _ in range(len(dims)):
        for n in range(len(dims)):
            rest = math.prod(ranks) // ranks[n]
            ranks[n] = max(2, min(ranks[n], rest // 2))
    return ranks


def draw(rng):
    kind = rng.choice(["compress", "compress", "compress", "compress", "batch", "gram", "gram", "eig", "ttm",
                       "reconstruct", "preprocess"])
    if kind == "compress":
        dims = _draw_dims(rng, 2e4, 6e8)
        ranks = _draw_ranks(rng, dims)
        order = list(range(len(dims)))
        rng.shuffle(order)
        prec = rng.choice(["fp64", "fp64", "fp64", "fp32", "bf16x6", "bf16x3"])
        dtype = rng.choice(["f32", "f64"]) if prec == "fp64" else "f32"
        given = prec == "fp64" and rng.random() < 0.25
        return {"kind": kind, "dims": _text(dims), "ranks": _text(ranks), "order": _text(order), "dtype": dtype,
                "prec": prec, "eps": 1e-2 if prec == "bf16x3" else 1e-3, "noise": 1e-4,
                "decay": round(0.1 ** (1.0 / max(ranks)), 4), "given": given, "part": rng.choice([1.0, 0.5, 0.2])}
    if kind == "batch":
        lo = rng.randint(4, 48)
        return {"kind": kind, "count": _log_int(rng, 8, 384), "lo": lo, "hi": rng.randint(lo + 16, 128),
                "dtype": rng.choice(["f32", "f64"]), "prec": "fp64", "eps": 1e-3, "noise": 1e-4}
    if kind in ("gram", "ttm"):
        dims = _draw_dims(rng, 2e4, 6e8, 2, 5)
        mode = rng.randrange(len(dims))
        case = {"kind": kind, "dims": _text(dims), "mode": mode, "dtype": rng.choice(["f32", "f64"])}
        if kind == "ttm":
            case["K"] = max(1, int(dims[mode] * rng.uniform(0.05, 0.9)))
        return case
    if kind == "eig":
        J = _log_int(rng, 8, 900)
        return {"kind": kind, "J": J, "R": max(1, int(J * rng.uniform(0.1, 0.8)))}
    if kind == "reconstruct":
        dims = _draw_dims(rng, 2e4, 1e9)
        return {"kind": kind, "dims": _text(dims), "ranks": _text(_draw_ranks(rng, dims)),
                "out": rng.choice(["f32", "f64"]), "part": rng.choice([1.0, 0.5, 0.2])}
    dims = _draw_dims(rng, 2e4, 9e8)
    return {"kind": kind, "dims": _text(dims), "mode": rng.randrange(len(dims)),
            "method": rng.choice(["standardize", "max"]), "dtype": rng.choice(["f32", "f64"])}


# ---------------------------------------------------------------- inputs

def _factor(rng, I, R):
    """I x R with orthonormal columns, on the GPU."""
    Q, _ = np.linalg.qr(rng.standard_normal((I, R)))
    return torch.from_numpy(np.ascontiguousarray(Q)).to(DEV)


def _mode_product(T, n, M):
    """T x_n M of a tensor of shape dims[::-1] (mode n is axis N - 1 - n), in T's type."""
    N = T.dim()
    ax = N - 1 - n
    pre, J, post = math.prod(T.shape[:ax]), T.shape[ax], math.prod(T.shape[ax + 1:])
    M = M.to(T.dtype)
    shape = list(T.shape)
    shape[ax] = M.shape[0]
    out = torch.empty(shape, dtype=T.dtype, device=T.device)
    src, dst = T.reshape(pre, J, post), out.view(pre, M.shape[0], post)
    if post == 1:
        Mt = M.t().contiguous()
        for a in range(0, pre, 1 << 22):
            torch.mm(src[a:a + (1 << 22), :, 0], Mt, out=dst[a:a + (1 << 22), :, 0])
    elif pre <= 4096:
        for a in range(pre):
            torch.mm(M, src[a], out=dst[a])
    else:
        step = max(1, (1 << 28) // (J * post))
        for a in range(0, pre, step):
            b = src[a:a + step].transpose(0, 1).reshape(J, -1)
            dst[a:a + step] = torch.mm(M, b).view(M.shape[0], -1, post).transpose(0, 1)
    return out


def _planted(dims, ranks, decay, noise, dtype, seed):
    """A core with slices scaled by decay^r along every mode, times orthonormal factors, plus relative noise."""
    rng = np.random.default_rng(seed)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    work = dtype if math.prod(dims) > (1 << 26) else torch.float64
    X = torch.randn(ranks[::-1], generator=g, device=DEV, dtype=work)
    N = len(dims)
    for n in range(N):
        shape = [1] * N
        shape[N - 1 - n] = ranks[n]
        X *= (decay ** torch.arange(ranks[n], device=DEV, dtype=torch.float64)).to(work).view(shape)
    for n in sorted(range(N), key=lambda k: dims[k] / ranks[k]):
        X = _mode_product(X, n, _factor(rng, dims[n], ranks[n]))
    flat = X.view(-1)
    scale = noise * float(torch.linalg.vector_norm(flat)) / math.sqrt(flat.numel())
    for a in range(0, flat.numel(), 1 << 28):
        part = flat[a:a + (1 << 28)]
        part += scale * torch.randn(part.shape, generator=g, device=DEV, dtype=work)
    return X.to(dtype)


def _batch_dims(case, seed):
    """Sizes and ranks of a batch's tensors: the same for every seed, as a program's shapes are."""
    rng = np.random.default_rng(4000 + int(case["count"]))
    out = []
    for _ in range(int(case["count"])):
        dims = [int(v) for v in rng.integers(case["lo"], case["hi"] + 1, size=3)]
        ranks = [int(rng.integers(2, max(2, d // 4) + 1)) for d in dims]
        for n in range(3):
            ranks[n] = max(2, min(ranks[n], math.prod(ranks) // ranks[n] // 2))
        out.append((dims, ranks))
    return out


def _window(dims, part):
    """A window of about ``part`` of every mode of at least 16, the whole of the others."""
    b, e = [], []
    for d in dims:
        w = max(1, int(round(d * part))) if d > 16 else d
        b.append((d - w) // 2)
        e.append((d - w) // 2 + w)
    return b, e


def _spectrum(J, R):
    """R eigenvalues over three decades, above a floor of 1e-9."""
    lam = np.full(J, 1e-9)
    lam[:R] = np.exp(-6.9 * np.arange(R) / R)
    return lam


def prepare(case, seed):
    kind = case["kind"]
    state = dict(case)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    if kind == "compress":
        dims = _ints(case["dims"])
        state["x"] = _planted(dims, _ints(case["ranks"]), case["decay"], case["noise"], DTYPES[case["dtype"]], seed)
        state["ranks"], state["order"] = _ints(case["ranks"]), _ints(case["order"])
        state["begin"], state["end"] = _window(dims, case["part"])
    elif kind == "batch":
        shapes = _batch_dims(case, seed)
        xs = [_planted(d, r, 1.0, case["noise"], DTYPES[case["dtype"]], seed * 1009 + i)
              for i, (d, r) in enumerate(shapes)]
        state["plan"] = tk.Batch(xs, case["eps"], prec=case["prec"])
    elif kind in ("gram", "ttm"):
        dims = _ints(case["dims"])
        state["y"] = torch.randn(dims[::-1], generator=g, device=DEV, dtype=DTYPES[case["dtype"]])
        if kind == "ttm":
            # U_n^T of a factor, as the mode loop passes it: its rows are the contiguous columns of U_n
            U = _factor(np.random.default_rng(seed), dims[case["mode"]], int(case["K"]))
            state["m"] = U.t().contiguous()
    elif kind == "eig":
        J, R = int(case["J"]), int(case["R"])
        Q = _factor(np.random.default_rng(seed), J, J).cpu()
        lam = _spectrum(J, R)
        S = (Q * torch.from_numpy(lam)) @ Q.t().contiguous()
        state["s"] = (0.5 * (S + S.t())).contiguous().to(DEV)
        state["thr"] = float(lam[R:].sum()) + 0.5 * float(lam[R - 1])
    elif kind == "reconstruct":
        dims, ranks = _ints(case["dims"]), _ints(case["ranks"])
        rng = np.random.default_rng(seed)
        core = torch.randn(ranks[::-1], generator=g, device=DEV, dtype=torch.float64)
        factors = [_factor(rng, i, r) for i, r in zip(dims, ranks)]
        state["model"], state["core"], state["factors"] = tk.from_model(core, factors), core, factors
        state["begin"], state["end"] = _window(dims, case["part"])
    else:
        dims = _ints(case["dims"])
        x = torch.randn(dims[::-1], generator=g, device=DEV, dtype=DTYPES[case["dtype"]])
        # variables of different magnitudes and offsets
        J, N = dims[case["mode"]], len(dims)
        shape = [1] * N
        shape[N - 1 - case["mode"]] = J
        mul = torch.logspace(-3, 3, J, device=DEV, dtype=torch.float64).to(x.dtype).view(shape)
        state["x"] = x.mul_(mul).add_(0.5 * mul)
    return state


# ---------------------------------------------------------------- the passes

def run(state):
    kind = state["kind"]
    if kind == "compress":
        if state["given"]:
            t = tk.sthosvd_ranks(state["x"], state["ranks"], mode_order=state["order"], prec=state["prec"])
        else:
            t = tk.sthosvd(state["x"], state["eps"], mode_order=state["order"], prec=state["prec"])
        xh = t.reconstruct(state["begin"], state["end"])
        if state["prec"] != "fp64":
            # a model of the reduced forms is kept in single precision
            return {"ranks": t.ranks, "core": t.core, "factors": [u.float() for u in t.factors], "xhat": xh}
        return {"ranks": t.ranks, "core": t.core, "factors": t.factors,
                "eigenvalues": [t.eigenvalues(n) for n in range(t.N)], "xhat": xh}
    if kind == "batch":
        plan = state["plan"]
        plan.run()
        items = [plan.item(i) for i in range(plan.count)]
        return {"ranks": torch.tensor([t.ranks for t in items]),
                "cores": torch.cat([t.core.reshape(-1) for t in items]),
                "factors": torch.cat([t.factor(n).t().reshape(-1) for t in items for n in range(3)])}
    if kind == "gram":
        return tk.gram(state["y"], state["mode"])
    if kind == "ttm":
        return tk.ttm(state["y"], state["mode"], state["m"])
    if kind == "eig":
        lam, U, r, disc = tk.eig_truncate(state["s"], state["thr"])
        return {"lam": lam, "U": U, "R": r, "disc": disc}
    if kind == "reconstruct":
        return state["model"].reconstruct(state["begin"], state["end"], out_dtype=DTYPES[state["out"]])
    return tk.preprocess(state["x"], state["mode"], state["method"])


# ---------------------------------------------------------------- what a pass cannot do without

def _steps(dims, ranks, order):
    """Flops of the mode loop: the upper triangle of each Gram (J^2 K) and each product (2 R J K)."""
    cur, flops = list(dims), 0.0
    for n in order:
        K = math.prod(cur) // cur[n]
        flops += float(cur[n]) ** 2 * K + 2.0 * ranks[n] * cur[n] * K + 4.0 / 3.0 * cur[n] ** 3
        cur[n] = ranks[n]
    return flops


def _restore(ranks, sizes):
    """Flops of the product chain in the order of least growth."""
    cur, flops = list(ranks), 0.0
    for n in sorted(range(len(cur)), key=lambda k: sizes[k] / ranks[k]):
        flops += 2.0 * sizes[n] * math.prod(cur)
        cur[n] = sizes[n]
    return flops


def work(case):
    kind = case["kind"]
    es = 8 if case.get("dtype", "f64") == "f64" else 4
    if kind == "batch":
        total = {"bytes": 0.0, "flops": 0.0}
        for dims, ranks in _batch_dims(case, 0):
            model = math.prod(ranks) + sum(i * r for i, r in zip(dims, ranks))
            total["bytes"] += es * math.prod(dims) + 8 * model
            total["flops"] += _steps(dims, ranks, [0, 1, 2])
        return total
    if kind == "eig":
        J, R = case["J"], case["R"]
        return {"bytes": 8.0 * (J * J + J * R + J), "flops": 4.0 / 3.0 * J ** 3 + 2.0 * J * J * R}
    dims = _ints(case["dims"])
    size = float(math.prod(dims))
    if kind == "compress":
        ranks = _ints(case["ranks"])
        b, e = _window(dims, case["part"])
        sizes = [y - x for x, y in zip(b, e)]
        ws = 8 if case["prec"] == "fp64" else 4
        model = math.prod(ranks) + sum(i * r for i, r in zip(dims, ranks))
        return {"bytes": es * size + ws * math.prod(sizes) + 8.0 * model,
                "flops": _steps(dims, ranks, _ints(case["order"])) + _restore(ranks, sizes)}
    if kind == "reconstruct":
        ranks = _ints(case["ranks"])
        b, e = _window(dims, case["part"])
        sizes = [y - x for x, y in zip(b, e)]
        return {"bytes": (4.0 if case["out"] == "f32" else 8.0) * math.prod(sizes) + 8.0 * math.prod(ranks),
                "flops": _restore(ranks, sizes)}
    if kind == "preprocess":
        return {"bytes": 2.0 * es * size, "flops": 5.0 * size}
    J = dims[case["mode"]]
    if kind == "gram":
        return {"bytes": es * size + 8.0 * J * J, "flops": J * size}
    return {"bytes": es * (size + size / J * case["K"]) + 8.0 * J * case["K"], "flops": 2.0 * case["K"] * size}


# ---------------------------------------------------------------- the same in 64 bits

def _columns(X, n, step):
    """The mode-n unfolding of X in float64, `step` values at a time (columns in any order)."""
    ax = X.dim() - 1 - n
    pre, J, post = math.prod(X.shape[:ax]), X.shape[ax], math.prod(X.shape[ax + 1:])
    Y = X.reshape(pre, J, post)
    rows = max(1, step // (J * post))
    cols = post if rows > 1 else max(1, step // J)
    for a in range(0, pre, rows):
        for c in range(0, post, cols):
            yield Y[a:a + rows, :, c:c + cols].double().transpose(0, 1).reshape(J, -1)


def _gram(X, n):
    J = X.shape[X.dim() - 1 - n]
    S = torch.zeros((J, J), dtype=torch.float64, device=X.device)
    for A in _columns(X, n, 1 << 28):
        S += torch.mm(A, A.t().contiguous())
    return S


def _eig(S):
    """Eigenvalues descending, eigenvectors with the entry of largest magnitude positive."""
    lam, V = torch.linalg.eigh(S.cpu())
    lam, V = lam.flip(0), V.flip(1)
    top = V.gather(0, V.abs().argmax(0, keepdim=True))
    return lam.to(DEV), (V * torch.where(top < 0, -1.0, 1.0)).to(DEV)


def _kept(lam, thr):
    tail = torch.cumsum(lam.clamp(min=0).flip(0), 0)
    return max(1, lam.numel() - int((tail <= thr).sum()))


def _hosvd(X, order, eps, given):
    N = X.dim()
    norm2 = sum(float(p.double().square().sum()) for p in X.reshape(-1).split(1 << 28))
    factors, eigenvalues, ranks = [None] * N, [None] * N, [0] * N
    Y = X
    for n in order:
        lam, V = _eig(_gram(Y, n))
        ranks[n] = min(given[n], lam.numel()) if given else _kept(lam, eps * eps * norm2 / N)
        factors[n], eigenvalues[n] = V[:, :ranks[n]].contiguous(), lam
        ax = N - 1 - n
        shape = list(Y.shape)
        shape[ax] = ranks[n]
        Z = torch.empty(shape, dtype=torch.float64, device=DEV)
        pre, post = math.prod(Y.shape[:ax]), math.prod(Y.shape[ax + 1:])
        src, dst = Y.reshape(pre, -1, post), Z.view(pre, ranks[n], post)
        Ut = factors[n].t().contiguous()
        rows = max(1, (1 << 28) // (src.shape[1] * post))
        for a in range(0, pre, rows):
            A = src[a:a + rows].double().transpose(0, 1).reshape(src.shape[1], -1)
            dst[a:a + rows] = torch.mm(Ut, A).view(ranks[n], -1, post).transpose(0, 1)
        Y = Z
    return Y, factors, eigenvalues, ranks


def _restored(core, factors, begin, end):
    N = core.dim()
    sizes = [e - b for b, e in zip(begin, end)]
    for n in sorted(range(N), key=lambda k: sizes[k] / core.shape[N - 1 - k]):
        core = _mode_product(core, n, factors[n][begin[n]:end[n]])
    return core


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        out = {"ranks": [], "cores": [], "factors": []}
        for i, (d, r) in enumerate(_batch_dims(case, seed)):
            x = _planted(d, r, 1.0, case["noise"], DTYPES[case["dtype"]], seed * 1009 + i)
            core, factors, _, ranks = _hosvd(x, [0, 1, 2], case["eps"], None)
            out["ranks"].append(ranks)
            out["cores"].append(core.reshape(-1))
            out["factors"] += [u.t().reshape(-1) for u in factors]
        return {"ranks": torch.tensor(out["ranks"]), "cores": torch.cat(out["cores"]),
                "factors": torch.cat(out["factors"])}
    if kind == "reconstruct":
        s = prepare(case, seed)
        return _restored(s["core"], s["factors"], s["begin"], s["end"])
    s = prepare(case, seed)
    if kind == "compress":
        core, factors, eigenvalues, ranks = _hosvd(s["x"], s["order"], s["eps"], s["ranks"] if s["given"] else None)
        out = {"ranks": ranks, "core": core, "factors": factors}
        if s["prec"] == "fp64":
            out["eigenvalues"] = eigenvalues
        del s["x"]
        out["xhat"] = _restored(core, factors, s["begin"], s["end"])
        return out
    if kind == "gram":
        return _gram(s["y"], s["mode"])
    if kind == "ttm":
        y = s["y"].double()
        return _mode_product(y, s["mode"], s["m"])
    if kind == "eig":
        lam, V = _eig(s["s"])
        r = _kept(lam, s["thr"])
        return {"lam": lam, "U": V[:, :r], "R": r, "disc": float(lam.clamp(min=0)[r:].sum())}
    x, n = s["x"].double(), s["mode"]
    axes = [a for a in range(x.dim()) if a != x.dim() - 1 - n]
    if s["method"] == "standardize":
        shift = x.mean(axes)
        scale = (x - shift.view([-1 if a not in axes else 1 for a in range(x.dim())])).square().mean(axes).sqrt()
    else:
        shift, scale = torch.zeros(x.shape[x.dim() - 1 - n], dtype=x.dtype, device=DEV), x.abs().amax(axes)
    view = [-1 if a not in axes else 1 for a in range(x.dim())]
    return (x - shift.view(view)) / scale.view(view), shift, scale
