"""What a user of the lazy arrays has them do, as cases with a size: the programs of the paper and of this
repository's workloads, through the public entry points, from one small vector to arrays that fill the caches many
times over.

A case is a dict of plain values: `kind` names the program, the rest its sizes and options.  `prepare` makes the
input tensors and whatever else the program holds before the call, `run` is one pass, `exact` the same values in
binary64 by plain torch."""
import math

import torch

from paper_1901_03771_amd import lazy as gr
from paper_1901_03771_amd import workloads as wl

SWEEPS = 10  # of a Jacobi pass


def listed():
    return [
        # a small pointwise chain, recorded once and replayed on new data: the shortest call there is
        dict(name="chain_replayed", kind="chain", n=100_003, replay=True),
        # the same program on a megaelement, recorded on every pass as a plain NumPy-style program does
        dict(name="chain_recorded", kind="chain", n=1 << 20, replay=False),
        # option prices: a long chain with log, exp, sqrt and erf
        dict(name="blackscholes", kind="blackscholes", n=1 << 24),
        # broadcast normalisation of a large matrix, the headline workload
        dict(name="normalize", kind="normalize", rows=8192, cols=8192),
        # feature standardisation of a tall table: column means and deviations, then the broadcast map
        dict(name="standardize", kind="standardize", rows=100_003, cols=257, axis=0),
        # row softmax
        dict(name="softmax", kind="softmax", rows=16384, cols=4096),
        # two-level image stencil over shifted slices
        dict(name="stencil", kind="stencil", rows=8192, cols=8192),
        # ten Jacobi sweeps, each a slice assignment into a grid that lives in the caller's own tensor
        dict(name="jacobi", kind="jacobi", rows=4096, cols=4096, storage="wrapped"),
        # one logistic-regression step: matrix-vector product, epilogue, transposed product, update
        dict(name="logreg", kind="logreg", rows=262144, cols=512),
        # a dense layer in training: product with bias and tanh, then the three gradients (plain and transposed operands)
        dict(name="dense_step", kind="dense", m=4096, k=784, n=512),
        # squared distances of points to centres and the nearest one's: the inner step of k-means
        dict(name="distances", kind="distances", n=1 << 18, c=32, d=16),
        # running sums down the columns of a matrix
        dict(name="cumsum_columns", kind="cumsum", rows=8192, cols=8192, axis=0, dtype="f32"),
    ]


def _size(rng, lo, hi):
    """Log-uniform; a third of the draws in multiples of 64, as sizes often come, the others as they fall."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if v >= 128 and rng.random() < 1 / 3:
        v = v // 64 * 64
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["chain", "blackscholes", "normalize", "standardize", "softmax", "stencil", "jacobi", "logreg", "dense",
                       "distances", "cumsum"])
    if kind == "chain":
        return dict(kind=kind, n=_size(rng, 1 << 10, 1 << 26), replay=rng.random() < 0.5)
    if kind == "blackscholes":
        return dict(kind=kind, n=_size(rng, 1 << 10, 1 << 26))
    if kind == "dense":
        m, k, n = _size(rng, 64, 16384), _size(rng, 16, 4096), _size(rng, 10, 4096)
        while 3 * m * k * n > 1 << 34:
            m, k, n = max(64, m // 2), max(16, k - k // 4), max(10, n - n // 4)
        return dict(kind=kind, m=m, k=k, n=n)
    if kind == "distances":
        c, d = _size(rng, 4, 64), _size(rng, 2, 64)
        return dict(kind=kind, n=_size(rng, 1 << 10, min(1 << 20, (1 << 28) // (c * d))), c=c, d=d)
    # a matrix of 2^14 to 2^26 elements, flat, square or tall (2^24 for the ten sweeps over a grid)
    cols = {"logreg": (16, 4096), "softmax": (32, 65536), "standardize": (16, 8192)}.get(kind, (64, 16384))
    cols = _size(rng, *cols)
    rows = _size(rng, max(64, (1 << 14) // cols), max(64, (1 << (24 if kind == "jacobi" else 26)) // cols))
    case = dict(kind=kind, rows=rows, cols=cols)
    if kind == "standardize":
        case["axis"] = rng.choice([0, 1])
    if kind == "jacobi":
        case["storage"] = rng.choice(["wrapped", "lent", "owned"])
    if kind == "cumsum":
        case["axis"] = rng.choice([0, 1])
        case["dtype"] = rng.choice(["f32", "f32", "i32"])
    return case


def standardize(xp, X, axis):
    """Zero mean and unit deviation along one axis (each feature of a table, each row of a layer)."""
    return (X - xp.mean(X, axis, True)) / xp.sqrt(xp.var(X, axis, True) + 1e-5)


_PROGRAM = {"chain": wl.chain, "blackscholes": wl.blackscholes, "normalize": wl.normalize, "softmax": wl.softmax, "stencil": wl.stencil,
            "logreg": wl.logreg}
_ctx = None
_seen = set()


def _context():
    global _ctx
    if _ctx is None:
        _ctx = gr.Context()
    return _ctx


def _inputs(case, seed):
    """The input tensors in the order of the program's arguments, values in the ranges of the repository's workloads."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def uniform(lo, hi, *shape):
        return torch.rand(shape, generator=g, device="cuda").mul_(hi - lo).add_(lo)

    def normal(sigma, *shape):
        return torch.randn(shape, generator=g, device="cuda").mul_(sigma)

    kind = case["kind"]
    if kind == "chain":
        return [uniform(-1, 1, case["n"]), uniform(-1, 1, case["n"])]
    if kind == "blackscholes":
        n = case["n"]
        return [uniform(5, 30, n), uniform(1, 100, n), uniform(0.25, 10, n)]
    if kind == "dense":
        m, k, n = case["m"], case["k"], case["n"]
        return [normal(1.0, m, k), normal(1.0 / math.sqrt(k), k, n), normal(0.1, n), normal(1.0, m, n)]
    if kind == "distances":
        return [normal(1.0, case["n"], case["d"]), normal(1.0, case["c"], case["d"])]
    r, c = case["rows"], case["cols"]
    if kind == "normalize":
        return [normal(1.0, r, c), uniform(-0.5, 0.5, 1, c), uniform(0.5, 2, 1, c), uniform(0.5, 1.5, c), uniform(0.5, 1.5, c)]
    if kind == "standardize":
        return [normal(2.0, r, c).add_(0.5)]
    if kind == "softmax":
        return [normal(2.0, r, c)]
    if kind in ("stencil", "jacobi"):
        return [uniform(0, 255, r, c)]
    if kind == "logreg":
        return [normal(1.0, r, c), normal(math.sqrt(0.05), c), (torch.rand(r, generator=g, device="cuda") < 0.5).float()]
    if kind == "cumsum":
        if case["dtype"] == "i32":
            return [torch.randint(-1000, 1000, (r, c), generator=g, device="cuda", dtype=torch.int32)]
        return [uniform(0, 1, r, c)]
    raise KeyError(kind)


def _outputs(case):
    kind = case["kind"]
    if kind == "dense":
        m, k, n = case["m"], case["k"], case["n"]
        shapes = dict(y=(m, n), dW=(k, n), db=(n,), dX=(m, k))
        return {name: torch.empty(s, device="cuda") for name, s in shapes.items()}
    if kind == "distances":
        return [torch.empty(case["n"], case["c"], device="cuda"), torch.empty(case["n"], device="cuda")]
    if kind == "jacobi":
        return None
    if "n" in case:
        return torch.empty(case["n"], device="cuda")
    r, c = case["rows"], case["cols"]
    shape = (r - 4, c - 4) if kind == "stencil" else (c,) if kind == "logreg" else (r, c)
    return torch.empty(shape, device="cuda", dtype=torch.int64 if case.get("dtype") == "i32" else torch.float32)


def _state(case, seed):
    ctx = _context()
    x = _inputs(case, seed)
    s = dict(case=case, ctx=ctx, x=x, out=_outputs(case))
    if case.get("replay"):
        leaves = [ctx.array(t) for t in x]
        s["program"] = ctx.program(_PROGRAM[case["kind"]](gr, *leaves), leaves)
    if case["kind"] == "distances":
        s["broadcast"] = (x[0][:, None, :], x[1][None, :, :])
    if case["kind"] == "jacobi":
        if case["storage"] == "lent":
            s["second"] = torch.empty_like(x[0])
            s["grid"] = ctx.array(x[0], second=s["second"])
        else:
            s["grid"] = ctx.array(x[0])
            if case["storage"] == "owned":
                s["grid"] = s["grid"].copy()
    return s


def prepare(case, seed):
    case = {k: v for k, v in case.items() if k != "name"}
    key = tuple(sorted(case.items()))
    if key not in _seen:
        # once per program: have its kernels compiled and loaded, as a program does that waits for them at its start
        run(_state(case, 0))
        _context().compile_wait()
        torch.cuda.synchronize()
        _seen.add(key)
    return _state(case, seed)


def run(s):
    case, ctx, x, out = s["case"], s["ctx"], s["x"], s["out"]
    kind = case["kind"]
    if kind == "jacobi":
        grid = wl.jacobi(gr, s["grid"], SWEEPS)
        if case["storage"] == "wrapped":
            return x[0]
        if case["storage"] == "lent":
            return grid.current(x[0], s["second"])
        return grid.torch(copy=False)
    if "program" in s:
        s["program"].run(x, out)
        return out
    if kind == "dense":
        X, W, b, dY = (ctx.array(t) for t in x)
        y = gr.tanh(X @ W + b)
        y.materialize_into(out["y"])
        G = dY * (1.0 - y * y)
        (X.T @ G).materialize_into(out["dW"])
        gr.sum(G, 0).materialize_into(out["db"])
        (G @ W.T).materialize_into(out["dX"])
        return out
    if kind == "distances":
        points, centres = (ctx.array(t) for t in s["broadcast"])
        diff = points - centres
        D = gr.sum(diff * diff, axis=2)
        D.materialize_into(out[0])
        gr.min(D, axis=1).materialize_into(out[1])
        return out
    leaves = [ctx.array(t) for t in x]
    if kind == "cumsum":
        gr.cumsum(leaves[0], case["axis"]).materialize_into(out)
    elif kind == "standardize":
        standardize(gr, leaves[0], case["axis"]).materialize_into(out)
    else:
        _PROGRAM[kind](gr, *leaves).materialize_into(out)
    return out


def work(case):
    kind = case["kind"]
    if kind == "dense":
        m, k, n = case["m"], case["k"], case["n"]
        return {"bytes": 4 * (2 * m * k + 2 * k * n + 2 * m * n + 2 * n), "flops": 6 * m * k * n + 10 * m * n}
    if kind == "distances":
        n, c, d = case["n"], case["c"], case["d"]
        return {"bytes": 4 * (n * d + c * d + n * c + n), "flops": 3 * n * c * d + n * c}
    if kind == "chain":
        return {"bytes": 12 * case["n"], "flops": 12 * case["n"]}
    if kind == "blackscholes":
        return {"bytes": 16 * case["n"], "flops": 30 * case["n"]}
    r, c = case["rows"], case["cols"]
    if kind == "normalize":
        return {"bytes": 8 * r * c + 16 * c, "flops": 5 * r * c}
    if kind == "standardize":
        return {"bytes": 8 * r * c, "flops": 6 * r * c}
    if kind == "softmax":
        return {"bytes": 8 * r * c, "flops": 5 * r * c}
    if kind == "stencil":
        return {"bytes": 4 * r * c + 4 * (r - 4) * (c - 4), "flops": 16 * r * c}
    if kind == "jacobi":
        return {"bytes": SWEEPS * (4 * r * c + 4 * (r - 2) * (c - 2)), "flops": SWEEPS * 5 * r * c}
    if kind == "logreg":
        return {"bytes": 4 * (r * c + r + 2 * c), "flops": 4 * r * c}
    if kind == "cumsum":
        return {"bytes": (12 if case["dtype"] == "i32" else 8) * r * c, "flops": r * c}
    raise KeyError(kind)


def tolerance(case):
    """About four times what this path and plain torch in float32 measure against binary64 over the ranges above,
    whichever is more; `max` is of single elements, in root mean squares or of the value."""
    kind = case["kind"]
    if case.get("dtype") == "i32":
        return "exact"
    if kind == "cumsum":  # long running sums of positive values in another association: 7e-7, single elements 3.4e-6
        return {"rel": 3e-6, "max": 1.5e-5}
    if kind == "dense":  # sums of signed products that cancel: 2.1e-6, single elements 1.5e-5
        return {"rel": 8e-6, "max": 6e-5}
    if kind == "jacobi":  # a rounding per operation and sweep: 2.2e-7, single elements 5.8e-7
        return {"rel": 9e-7, "max": 2.5e-6}
    return {"rel": 5e-7, "max": 4e-6}  # 1.5e-7 at most, single elements 9.3e-7


def exact(case, seed):
    kind = case["kind"]
    x = [t.double() if t.is_floating_point() else t.long() for t in _inputs(case, seed)]
    if kind == "chain":
        a, b = x
        return ((a + b) * (a - b) + 2.5 * a) / (b.abs() + 1) - torch.exp(-a * a)
    if kind == "blackscholes":
        S, K, T = x
        r, sigma = 0.02, 0.30
        root = T.sqrt()
        d1 = (torch.log(S / K) + (r + 0.5 * sigma * sigma) * T) / (sigma * root)
        d2 = d1 - sigma * root
        cdf1, cdf2 = (0.5 * (1 + torch.erf(d / math.sqrt(2))) for d in (d1, d2))
        return S * cdf1 - K * torch.exp(-r * T) * cdf2
    if kind == "normalize":
        X, mu, sigma, gamma, beta = x
        return torch.clamp_min((X - mu) / sigma * gamma + beta, 0)
    if kind == "standardize":
        X, axis = x[0], case["axis"]
        d = X - X.mean(axis, keepdim=True)
        return d / torch.sqrt((d * d).mean(axis, keepdim=True) + 1e-5)
    if kind == "softmax":
        return torch.softmax(x[0], 1)
    if kind == "stencil":
        I = x[0]
        B = 0.2 * (I[1:-1, 1:-1] + I[:-2, 1:-1] + I[2:, 1:-1] + I[1:-1, :-2] + I[1:-1, 2:])
        return torch.sqrt((B[1:-1, 2:] - B[1:-1, :-2]) ** 2 + (B[2:, 1:-1] - B[:-2, 1:-1]) ** 2)
    if kind == "jacobi":
        u = x[0]
        for _ in range(SWEEPS):
            v = u.clone()
            v[1:-1, 1:-1] = 0.2 * (u[1:-1, 1:-1] + u[:-2, 1:-1] + u[1:-1, 2:] + u[1:-1, :-2] + u[2:, 1:-1])
            u = v
        return u
    if kind == "logreg":
        X, w, y = x
        resid = torch.sigmoid(X @ w) - y
        return w - 0.1 * ((X.T @ resid) / X.shape[0] + 1e-4 * w)
    if kind == "dense":
        X, W, b, dY = x
        y = torch.tanh(X @ W + b)
        G = dY * (1 - y * y)
        return {"y": y, "dW": X.T @ G, "db": G.sum(0), "dX": G @ W.T}
    if kind == "distances":
        P, C = x
        D = torch.stack([((P - c) ** 2).sum(1) for c in C], 1)
        return [D, D.min(1).values]
    if kind == "cumsum":
        return torch.cumsum(x[0], case["axis"])
    raise KeyError(kind)
