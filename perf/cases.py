"""The work that a user of the library has it do, as cases that can be timed and compared.

A case is a dict of plain values; `kind` says which entry point it goes through:

  solve     an LP on a kept handle (lp.Problem): a solve from the cold start of a fixed number of accepted steps
            (every kernel of the loop, the check and the restart at the end of a check window among them), then
            the point
  product   the two products with the scaled matrix on device buffers (spmv_noalloc), K x then K'y
  batch     many LPs of their own on one handle (lp.Batch), then every member's point
  shared    many LPs of one family on one handle (lp.Shared: one K, each its own c, q, l, u), then every
            member's point
  forward   the warm-start network's prediction for a batch of sketches
  gradient  its loss on the minibatches of a training set and the last one's gradient
  gemm      the network's matrix product by itself

LPs are synthetic, feasible and bounded by construction, as in paper_2312_14832_amd.gen (whose recipes these
are, drawn on the GPU so that large ones are made quickly).  The step counts are fixed, and stop while the
method's own sensitivity to rounding (it multiplies an error of a step by about a thousand per check window) is
far below what its precision can tell: a run to a tolerance ends at another step after any change of rounding.
"""
import math

import numpy as np
import torch

from paper_2312_14832_amd import gen, lp, warmstart

DEVICE = "cuda" if torch.cuda.is_available() else "cpu"
F64 = torch.float64


def listed():
    return [
        # one small LP, the time of a step with nothing to hide it behind: what a program that solves small LPs one
        # after another pays (the library's tiny workload)
        dict(name="solve small", kind="solve", family="uniform", columns=1000, rows=500, per_column=5,
             precision="fp64", pointers="host", steps=96),
        # an LP of ordinary size, odd: too large for one workgroup, too small to fill the GPU
        dict(name="solve medium", kind="solve", family="uniform", columns=23457, rows=11003, per_column=6,
             precision="fp64", pointers="host", steps=96),
        # the headline workload: power-law columns, row scales over six decades, 2e6 columns, about 2e7 nonzeros
        dict(name="solve large", kind="solve", family="powerlaw", columns=2000000, rows=1000000, per_column=10,
             precision="fp64", pointers="device", steps=96),
        # the same family in mixed precision
        dict(name="solve large mixed", kind="solve", family="powerlaw", columns=1000000, rows=500000, per_column=10,
             precision="mixed", pointers="device", steps=16),
        # the PageRank LP: one dense row, very short others
        dict(name="solve pagerank", kind="solve", family="pagerank", columns=1000000, rows=1000001, per_column=8,
             precision="fp64", pointers="device", steps=96),
        # products by themselves, for code that builds its own iteration on them (captured loops, serving)
        dict(name="products", kind="product", family="uniform", columns=150001, rows=75007, per_column=8,
             precision="fp64"),
        # a queue of LPs of uneven sizes on one handle
        dict(name="batch uneven", kind="batch", members=32, columns=2000, columns_most=200000, per_column=8,
             precision="fp64", steps=64),
        # a queue of small ones
        dict(name="batch small", kind="batch", members=256, columns=300, columns_most=1000, per_column=5,
             precision="fp64", steps=64),
        # a parametric family: labels for the warm-start network, scenarios of one model
        dict(name="shared family", kind="shared", members=64, columns=100000, rows=50000, per_column=10,
             precision="fp64", steps=64),
        # the network's prediction for the family of 2e5 columns and 1e5 rows (and one output for the weight)
        dict(name="predict", kind="forward", batch=256, outputs=300001, precision="bf16"),
        # its training, on the family of 2e4 columns: loss and gradient of eight minibatches
        dict(name="train", kind="gradient", batch=256, minibatches=8, outputs=30001, precision="bf16"),
        # the matrix product at the size the library quotes it at
        dict(name="gemm", kind="gemm", m=4096, n=4096, k=4096, trans_a=False, trans_b=False, precision="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _steps(rng, precision):
    return 16 if precision == "mixed" else rng.choice([48, 64])


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "product", "batch", "shared", "forward", "gradient", "gemm"])
    if kind in ("solve", "product"):
        precision = rng.choice(["fp64", "fp64", "mixed"])
        family = rng.choice(["uniform", "uniform", "powerlaw", "pagerank"] if precision == "fp64" else ["uniform", "powerlaw"])
        columns = _log(rng, 200 if (family, precision) != ("powerlaw", "mixed") else 100000, 1000000)
        rows = columns + 1 if family == "pagerank" else max(20, int(columns * rng.uniform(0.3, 0.8)))
        c = dict(kind=kind, family=family, columns=columns, rows=rows,
                 per_column={"uniform": rng.randint(3, 10), "powerlaw": 10, "pagerank": 8}[family],
                 precision=precision)
        if kind == "solve":
            c["pointers"] = rng.choice(["host", "device"])
            c["steps"] = _steps(rng, precision)
        return c
    if kind == "batch":
        small = rng.random() < 0.5
        precision = rng.choice(["fp64", "fp64", "mixed"])
        return dict(kind=kind, members=_log(rng, 16, 192) if small else _log(rng, 4, 24),
                    columns=200 if small else 2000, columns_most=rng.randint(500, 1000) if small else _log(rng, 20000, 200000),
                    per_column=rng.randint(4, 8), precision=precision,
                    steps=_steps(rng, precision))
    if kind == "shared":
        precision = rng.choice(["fp64", "fp64", "mixed"])
        members = rng.randint(3, 80)
        columns = min(_log(rng, 1000, 200000), 6400000 // (1 << (members - 1).bit_length()))
        return dict(kind=kind, members=members, columns=columns, rows=columns // 2, per_column=rng.randint(5, 10),
                    precision=precision, steps=_steps(rng, precision))
    if kind == "forward":
        return dict(kind=kind, batch=rng.randint(1, 256), outputs=_log(rng, 1000, 300000), precision="bf16")
    if kind == "gradient":
        return dict(kind=kind, batch=rng.randint(16, 256), minibatches=rng.randint(1, 8),
                    outputs=_log(rng, 1000, 30000), precision="bf16")
    return dict(kind=kind, m=_log(rng, 64, 4096), n=_log(rng, 64, 4096), k=_log(rng, 64, 4096),
                trans_a=rng.random() < 0.5, trans_b=rng.random() < 0.5,
                precision=rng.choice(["bf16", "bf16", "fp32"]))


# --------------------------------------------------------------------------------------------------------------
# data
# --------------------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _rand(g, *size):
    return torch.rand(*size, generator=g, device=DEVICE, dtype=F64)


def _randn(g, *size):
    return torch.randn(*size, generator=g, device=DEVICE, dtype=F64)


class _Matrix:
    """A CSR matrix that multiplies dense columns, its long rows by themselves (torch's product takes such a row in
    one thread)."""

    def __init__(self, row_ptr, col, val, m, n):
        row_ptr, col = row_ptr.long(), col.long()
        self.long = [(r, col[a:b], val[a:b]) for r, a, b in
                     ((r, int(row_ptr[r]), int(row_ptr[r + 1])) for r in (row_ptr.diff() > 4096).nonzero()[:, 0].tolist())]
        if self.long:
            keep = torch.ones_like(col, dtype=torch.bool)
            for r, c, _ in self.long:
                keep[row_ptr[r]:row_ptr[r + 1]] = False
            count = row_ptr.diff()
            count[[r for r, _, _ in self.long]] = 0
            row_ptr = torch.cat([row_ptr[:1], torch.cumsum(count, 0)])
            col, val = col[keep], val[keep]
        self.rows = torch.sparse_csr_tensor(row_ptr, col, val, (m, n))

    def __matmul__(self, x):
        out = self.rows @ x
        for r, c, v in self.long:
            out[r] = (v * x[c] if x.dim() == 1 else v[:, None] * x[c]).sum(0)
        return out


def _sparse(row_ptr, col, val, m, n):
    return _Matrix(row_ptr, col, val, m, n)


def _transposed(row_ptr, col, val, m, n):
    """CSR of the transpose."""
    row = torch.repeat_interleave(torch.arange(m, device=val.device), row_ptr.long().diff())
    order = torch.argsort(col.long() * m + row)
    tp = torch.zeros(n + 1, dtype=torch.int64, device=val.device)
    tp[1:] = torch.cumsum(torch.bincount(col.long(), minlength=n), 0)
    return tp, row[order], val[order]


def _pattern(key, m, n):
    """CSR row pointers and columns of the distinct keys row * n + col."""
    key = torch.unique(key)
    row, col = key // n, key % n
    rp = torch.zeros(m + 1, dtype=torch.int64, device=DEVICE)
    rp[1:] = torch.cumsum(torch.bincount(row, minlength=m), 0)
    return rp.int(), col.int(), row


def _certificate(g, m, n, m1, rp, col, val, box_hi=10.0):
    """c, q, l, u with a primal-dual certificate (gen.certificate_lp's recipe); and the certificate."""
    K, KT = _sparse(rp, col, val, m, n), _sparse(*_transposed(rp, col, val, m, n), n, m)
    perm = torch.randperm(n, generator=g, device=DEVICE)
    kind = torch.full((n,), 2, device=DEVICE)
    kind[perm[:n // 2]] = 0
    kind[perm[n // 2:n // 2 + n // 4]] = 1
    inf = torch.full((n,), math.inf, device=DEVICE, dtype=F64)
    l = torch.where(kind == 2, -inf, torch.zeros_like(inf))
    u = torch.where(kind == 0, torch.full_like(inf, box_hi), inf)
    x0 = 5.0 * _rand(g, n)
    s = _rand(g, m - m1)
    y0 = torch.cat([_randn(g, m1), _rand(g, m - m1)])
    r = _randn(g, n)
    lam0 = torch.where(kind == 0, r, torch.where(kind == 1, r.abs(), torch.zeros_like(r)))
    q = K @ x0
    q[m1:] -= s
    c = KT @ y0 + lam0
    return c, q, l, u, (x0, s, y0, lam0)


def _lp(g, family, n, m, per_column):
    """One LP as device tensors: (m, n, m1, row_ptr, col, val, c, q, l, u)."""
    if family == "pagerank":
        draws = (1 + torch.poisson(torch.full((n,), per_column - 3.0, device=DEVICE), generator=g).long()).clamp(max=n - 1)
        src = torch.repeat_interleave(torch.arange(n, device=DEVICE), draws)
        dst = torch.randint(0, n - 1, (src.numel(),), generator=g, device=DEVICE)
        dst = dst + (dst >= src)
        link = torch.unique(src * n + dst)
        src, dst = link // n, link % n
        weight = -0.85 / torch.bincount(src, minlength=n).double()
        j = torch.arange(n, device=DEVICE)
        key = torch.cat([j, (1 + j) * n + j, (1 + dst) * n + src])
        vals = torch.cat([torch.ones(2 * n, device=DEVICE, dtype=F64), weight[src]])
        order = torch.argsort(key)
        rp, col, _ = _pattern(key, n + 1, n)
        q = torch.full((n + 1,), 0.15 / n, device=DEVICE, dtype=F64)
        q[0] = 1.0
        zero = torch.zeros(n, device=DEVICE, dtype=F64)
        return n + 1, n, 1, rp, col, vals[order], zero, q, zero.clone(), torch.full_like(zero, math.inf)
    if family == "powerlaw":
        k = torch.arange(1, 201, device=DEVICE, dtype=F64)
        p = k ** -1.534
        counts = 1 + torch.bucketize(_rand(g, n), torch.cumsum(p / p.sum(), 0)[:-1])
        counts = counts.clamp(max=max(1, m // 2))
    else:
        counts = torch.full((n,), min(per_column, m), device=DEVICE, dtype=torch.int64)
    cols = torch.repeat_interleave(torch.arange(n, device=DEVICE), counts)
    rows = torch.randint(0, m, (cols.numel(),), generator=g, device=DEVICE)
    rp, col, row = _pattern(rows * n + cols, m, n)
    val = _randn(g, col.numel())
    if family == "powerlaw":
        val = val * 10.0 ** (6.0 * _rand(g, m) - 3.0)[row]
    m1 = m // 2 if family == "powerlaw" else 2 * m // 5
    c, q, l, u, _ = _certificate(g, m, n, m1, rp, col, val)
    return m, n, m1, rp, col, val, c, q, l, u


def _data(parts, pointers="host"):
    """gen.LPData of an LP's parts; on the host unless device pointers are asked for."""
    m, n, m1, *arrays = parts
    if pointers == "host":
        arrays = [a.cpu().numpy() for a in arrays]
    return gen.LPData(m, n, m1, *arrays)


def _sizes(case):
    """The members' columns: even on a logarithmic scale, large and small ones mixed."""
    lo, hi, B = math.log(case["columns"]), math.log(case["columns_most"]), case["members"]
    return [int(round(math.exp(lo + (hi - lo) * ((i * 0.6180339887498949) % 1.0)))) for i in range(B)]


def _members(case, g):
    """The members of a batch, with half as many rows as columns."""
    return [_lp(g, "uniform", n, max(n // 2, 2), case["per_column"]) for n in _sizes(case)]


def _family(case, g):
    """The members of a parametric family: the base certificate perturbed by 10% (gen.parametric_instance's
    recipe), as (m, n, m1, row_ptr, col, val, C, Q, l, u) with C, Q one column per member."""
    n, m, B = case["columns"], case["rows"], case["members"]
    rows = torch.randint(0, m, (n * case["per_column"],), generator=g, device=DEVICE)
    cols = torch.repeat_interleave(torch.arange(n, device=DEVICE), case["per_column"])
    rp, col, _ = _pattern(rows * n + cols, m, n)
    val, m1 = _randn(g, col.numel()), m // 2
    c, q, l, u, (x0, s, y0, lam0) = _certificate(g, m, n, m1, rp, col, val)
    L, U = l[:, None], u[:, None]
    X = (x0[:, None] * (1 + 0.1 * _randn(g, n, B))).clamp(min=L, max=U)
    S = (s[:, None] * (1 + 0.1 * _randn(g, m - m1, B))).clamp(min=0.0)
    Y = y0[:, None] + 0.1 * y0.abs()[:, None] * _randn(g, m, B)
    Y[m1:].clamp_(min=0.0)
    lam = lam0[:, None] + 0.1 * lam0.abs()[:, None] * _randn(g, n, B)
    fl, fu = torch.isfinite(L), torch.isfinite(U)
    lam = torch.where(fl & fu, lam, torch.where(fl, lam.clamp(min=0.0), torch.zeros_like(lam)))
    Q = _sparse(rp, col, val, m, n) @ X
    Q[m1:] -= S
    C = _sparse(*_transposed(rp, col, val, m, n), n, m) @ Y + lam
    return m, n, m1, rp, col, val, C, Q, l, u


def _net_inputs(case, seed):
    """Parameters, input normalization, sketches and targets of a network (He-uniform ReLU layers, a small output
    factor whose bias is the base solution; targets around that)."""
    g = _gen(seed)
    dims = [256, 1024, 1024, 1024, 64, case["outputs"]]
    parts = []
    for i, (a, b) in enumerate(zip(dims[:-1], dims[1:])):
        lim = math.sqrt(6.0 / a) if i < 3 else 0.1 * math.sqrt(1.0 / a)
        parts.append((lim * (2 * _rand(g, a * b) - 1)).float())
        parts.append((2.0 * _randn(g, b)).float() if i == 4 else (0.01 * _randn(g, b)).float())
    rows = case["batch"] * case.get("minibatches", 1)
    mu, sigma = _randn(g, 256).float(), (0.5 + _rand(g, 256)).float()
    X = mu + sigma * torch.randn(rows, 256, generator=g, device=DEVICE)
    Z = None
    if case["kind"] == "gradient":
        Z = parts[-1] + 0.2 * torch.randn(rows, case["outputs"], generator=g, device=DEVICE)
    return dims, parts, mu, sigma, X, Z


def _operands(case, seed):
    g = _gen(seed)
    m, n, k = case["m"], case["n"], case["k"]
    A = torch.randn((k, m) if case["trans_a"] else (m, k), generator=g, device=DEVICE)
    B = torch.randn((n, k) if case["trans_b"] else (k, n), generator=g, device=DEVICE)
    return (A.bfloat16(), B.bfloat16()) if case["precision"] == "bf16" else (A, B)


# --------------------------------------------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("solve", "product"):
        g = _gen(seed)
        parts = _lp(g, case["family"], case["columns"], case["rows"], case["per_column"])
        if kind == "solve":
            torch.cuda.synchronize()
            return dict(case=case, handle=lp.Problem(_data(parts, case["pointers"]), precision=case["precision"],
                                                     ptr_kind=case["pointers"]))
        x, y = _randn(g, parts[1]), _randn(g, parts[0])
        stream = torch.cuda.Stream()   # the products are only enqueued: the program's other work goes to the same stream
        stream.wait_stream(torch.cuda.current_stream())
        return dict(case=case, x=x, y=y, Kx=torch.empty_like(y), KTy=torch.empty_like(x), stream=stream,
                    handle=lp.Problem(_data(parts), precision=case["precision"], stream=stream))
    if kind == "batch":
        return dict(case=case, handle=lp.Batch([_data(p) for p in _members(case, _gen(seed))], precision=case["precision"]))
    if kind == "shared":
        m, n, m1, rp, col, val, C, Q, l, u = _family(case, _gen(seed))
        rp, col, val, C, Q, l, u = (a.cpu().numpy() for a in (rp, col, val, C.T.contiguous(), Q.T.contiguous(), l, u))
        members = [gen.LPData(m, n, m1, rp, col, val, C[b], Q[b], l, u) for b in range(case["members"])]
        return dict(case=case, handle=lp.Shared(members, precision=case["precision"]))
    if kind in ("forward", "gradient"):
        dims, parts, mu, sigma, X, Z = _net_inputs(case, seed)
        net = warmstart.Net(case["outputs"], max_batch=case["batch"], precision=case["precision"])
        net.set_params(torch.cat(parts).cpu().numpy())
        net.set_norm(mu.cpu().numpy(), sigma.cpu().numpy())
        return dict(case=case, net=net, X=X, Z=Z)
    A, B = _operands(case, seed)
    return dict(case=case, A=A, B=B)


def _point(case, x, y, lam):
    """A point as a program keeps it: a mixed-precision one carries 24 bits."""
    if case["precision"] == "mixed":
        x, y, lam = (a.float() if isinstance(a, torch.Tensor) else a.astype(np.float32) for a in (x, y, lam))
    return x, y, lam


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        p = state["handle"]
        p.solve(0.0, case["steps"])
        x, y, lam, info = p.result()
        x, y, lam = _point(case, x, y, lam)
        out = dict(x=x, y=y, steps=info["iterations"], objective=info["pobj"])
        if case["family"] != "pagerank":   # whose multipliers are all zero, up to rounding
            out["lam"] = lam
        return out
    if kind == "product":
        p = state["handle"]
        p.spmv_noalloc(state["x"], state["Kx"])
        p.spmv_noalloc(state["y"], state["KTy"], transpose=True)
        if case["precision"] == "mixed":
            with torch.cuda.stream(state["stream"]):
                return dict(Kx=state["Kx"].float(), KTy=state["KTy"].float())
        return dict(Kx=state["Kx"], KTy=state["KTy"])
    if kind in ("batch", "shared"):
        h = state["handle"]
        h.solve(0.0, case["steps"])
        points, steps = [], []
        for i in range(case["members"]):
            x, y, lam, info = h.result(i)
            points.append(_point(case, x, y, lam))
            steps.append(info["iterations"])
        x, y, lam = (np.concatenate(v) for v in zip(*points))
        return dict(x=x, y=y, lam=lam, steps=np.array(steps))
    if kind == "forward":
        return state["net"].forward(state["X"])
    if kind == "gradient":
        net, b = state["net"], case["batch"]
        losses = [net.loss_grad(state["X"][i * b:(i + 1) * b], state["Z"][i * b:(i + 1) * b])
                  for i in range(case["minibatches"])]
        return dict(losses=np.array(losses), gradient=net.grads())
    return warmstart.gemm(state["A"], state["B"], case["trans_a"], case["trans_b"], case["precision"])


def work(case):
    """One pass.  A step of the method reads the matrix and its transpose (values and 32-bit columns), and reads or
    writes each vector of the iteration once: 11 of a column's and 12 of a row's values, the gathered ones among
    them; 4 operations per nonzero and about 20 per column and row."""
    kind = case["kind"]
    s = 4 if case.get("precision") == "mixed" else 8
    if kind in ("solve", "batch", "shared"):
        n, m = (sum(_sizes(case)), sum(_sizes(case)) // 2) if kind == "batch" else (case["columns"], case["rows"])
        nnz, B = n * case["per_column"], case["members"] if kind == "shared" else 1
        return {"bytes": case["steps"] * (2 * nnz * (s + 4) + 4 * (m + n) + B * s * (11 * n + 12 * m)),
                "flops": case["steps"] * B * (4.0 * nnz + 20 * (n + m))}
    if kind == "product":
        n, m, nnz = case["columns"], case["rows"], case["columns"] * case["per_column"]
        return {"bytes": 2 * nnz * (s + 4) + 4 * (m + n) + 16 * (m + n), "flops": 4.0 * nnz}
    if kind in ("forward", "gradient"):
        B, D = case["batch"], case["outputs"]
        weights = 256 * 1024 + 2 * 1024 * 1024 + 1024 * 64 + 64 * D
        w = 2 if case["precision"] == "bf16" else 4
        if kind == "forward":
            return {"bytes": w * weights + 4 * D + 4 * B * (256 + D), "flops": 2.0 * B * weights}
        k = case["minibatches"]
        return {"bytes": k * ((w + 4) * weights + 8 * D + 4 * B * (256 + D)) + 4 * weights, "flops": k * 6.0 * B * weights}
    m, n, k = case["m"], case["n"], case["k"]
    return {"bytes": (2 if case["precision"] == "bf16" else 4) * (m * k + k * n) + 4 * m * n, "flops": 2.0 * m * n * k}


# --------------------------------------------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# --------------------------------------------------------------------------------------------------------------

def _scaled(rp, col, val, m, n):
    """Ten Ruiz rounds and one Pock-Chambolle round (exponent 1): (scaled values, Dr, Dc)."""
    count = rp.long().diff()
    row = torch.repeat_interleave(torch.arange(m, device=val.device), count)
    col = col.long()
    short = (count <= 4096)[row]   # a long row by itself: torch's scatter takes its entries one after another
    wide = [(r, int(rp[r]), int(rp[r + 1])) for r in (count > 4096).nonzero()[:, 0].tolist()]
    Dr, Dc = torch.ones(m, device=val.device, dtype=F64), torch.ones(n, device=val.device, dtype=F64)
    v = val.clone()
    for it in range(11):
        how = "amax" if it < 10 else "sum"
        r = torch.zeros_like(Dr).scatter_reduce_(0, row[short], v.abs()[short], how)
        for i, a, b in wide:
            r[i] = v[a:b].abs().amax() if it < 10 else v[a:b].abs().sum()
        s = torch.zeros_like(Dc).scatter_reduce_(0, col, v.abs(), how)
        r, s = (torch.where(t > 0, t.sqrt(), torch.ones_like(t)) for t in (r, s))
        v = v / (r[row] * s[col])
        Dr, Dc = Dr * r, Dc * s
    return v, Dr, Dc


def _cone(g, lf, uf):
    """The projection of c - K'y onto the bounds' multipliers."""
    zero = torch.zeros_like(g)
    return torch.where(lf & uf, g, torch.where(lf, g.clamp(min=0), torch.where(uf, g.clamp(max=0), zero)))


def _rpdhg(m, n, m1, rp, col, val, C, Q, l, u, steps, every=64):
    """`steps` accepted steps of restarted PDHG from the cold start, for every column of C [n x B], Q [m x B]:
    x, y, lam [. x B] of the better of the last and the averaged point, and their objectives."""
    v, Dr, Dc = _scaled(rp, col, val, m, n)
    K, KT = _sparse(rp, col, v, m, n), _sparse(*_transposed(rp, col, v, m, n), n, m)
    Dr, Dc, l, u = Dr[:, None], Dc[:, None], l[:, None], u[:, None]
    lf, uf = torch.isfinite(l), torch.isfinite(u)
    c, q, lo, hi = C / Dc, Q / Dr, l * Dc, u * Dc
    nc, nq = c.norm(dim=0), q.norm(dim=0)
    Nc, Nq = C.norm(dim=0), Q.norm(dim=0)
    B = C.shape[1]
    omega = torch.where((nc > 1e-10) & (nq > 1e-10), nc / nq, torch.ones_like(nc))
    eta = torch.full_like(omega, 1.0 / float(v.abs().max()))
    x = torch.zeros_like(c).clamp(min=lo, max=hi)
    y = torch.zeros_like(q)
    kx, kt = K @ x, KT @ y
    xa, ya, kxa, kta, x0, y0 = x, y, kx, kt, x, y
    W = torch.zeros_like(omega)
    k = torch.zeros(B, dtype=torch.int64, device=C.device)
    t = torch.zeros_like(k)
    g_rows = (torch.arange(m, device=C.device) >= m1)[:, None]
    zero, one = torch.zeros_like(omega), torch.ones_like(omega)

    def quantities(x, y, kx, kt, omega):
        r = torch.where(g_rows, (q - kx).clamp(min=0), kx - q)
        lam = _cone(c - kt, lf, uf)
        d = c - kt - lam
        bound = torch.where(lf & (lam > 0), lo * lam, zero) + torch.where(uf & (lam < 0), hi * lam, zero)
        bound = torch.nan_to_num(bound, nan=0.0, posinf=0.0, neginf=0.0)
        p, dual = (c * x).sum(0), (q * y).sum(0) + bound.sum(0)
        gap = dual - p
        rel = torch.stack([(r * Dr).norm(dim=0) / (1 + Nq), (d * Dc).norm(dim=0) / (1 + Nc),
                           gap.abs() / (1 + dual.abs() + p.abs())]).amax(0)
        kkt = lambda w: (w ** 2 * (r * r).sum(0) + (d * d).sum(0) / w ** 2 + gap * gap).sqrt()  # noqa: E731
        return rel, kkt, p

    kkt0 = quantities(x, y, kx, kt, omega)[1](omega)
    kkt_prev = torch.full_like(kkt0, math.inf)
    out = None
    for _ in range(50 * steps):
        live = k < steps
        if not bool(live.any()):
            break
        xn = (x - eta / omega * (c - kt)).clamp(min=lo, max=hi)
        kxn = K @ xn
        yn = y + eta * omega * (q - 2 * kxn + kx)
        yn = torch.where(g_rows, yn.clamp(min=0), yn)
        dx2, dy2, inter = ((xn - x) ** 2).sum(0), ((yn - y) ** 2).sum(0), ((yn - y) * (kxn - kx)).sum(0)
        top, below = omega * dx2 + dy2 / omega, 2 * inter.abs()
        eta_bar = torch.where(below > 0, top / below, torch.full_like(top, math.inf))
        ok = live & (eta <= eta_bar)
        kk = k.double() + 2
        new = torch.minimum((1 - kk ** -0.3) * eta_bar, (1 + kk ** -0.6) * eta)
        W = torch.where(ok, W + eta, W)
        w = torch.where(ok, eta / torch.where(W > 0, W, one), zero)
        eta = torch.where(live, new, eta)
        x, y, kx = torch.where(ok, xn, x), torch.where(ok, yn, y), torch.where(ok, kxn, kx)
        kt = torch.where(ok, KT @ y, kt)
        xa, ya, kxa, kta = xa + w * (x - xa), ya + w * (y - ya), kxa + w * (kx - kxa), kta + w * (kt - kta)
        k, t = k + ok, t + ok
        check = ok & ((k % every == 0) | (k >= steps))
        if not bool(check.any()):
            continue
        rel, kkt, p = quantities(x, y, kx, kt, omega)
        rela, kkta, pa = quantities(xa, ya, kxa, kta, omega)
        avg = check & (rela < rel)
        if out is None:
            out = [x, y, kt, p]
        last = check & (k >= steps)
        new = [torch.where(avg, a, b) for a, b in ((xa, x), (ya, y), (kta, kt), (pa, p))]
        out = [torch.where(last, a, b) for a, b in zip(new, out)]
        z, za = kkt(omega), kkta(omega)
        cur = z < za
        best = torch.where(cur, z, za)
        full = check & (k % every == 0)
        restart = full & ((best <= 0.2 * kkt0) | ((best <= 0.8 * kkt0) & (best > kkt_prev)) | (t.double() >= 0.36 * k.double()))
        kkt_prev = torch.where(full, best, kkt_prev)
        to = [torch.where(cur, a, b) for a, b in ((x, xa), (y, ya), (kx, kxa), (kt, kta))]
        dx, dy = (to[0] - x0).norm(dim=0), (to[1] - y0).norm(dim=0)
        omega_new = torch.where((dx > 1e-10) & (dy > 1e-10), (0.5 * (dy / dx).log() + 0.5 * omega.log()).exp(), omega)
        omega_new = torch.where(restart, omega_new, omega)
        kkt0 = torch.where(restart, torch.where(cur, kkt(omega_new), kkta(omega_new)), kkt0)
        omega = omega_new
        kkt_prev = torch.where(restart, torch.full_like(kkt_prev, math.inf), kkt_prev)
        W, t = torch.where(restart, zero, W), torch.where(restart, torch.zeros_like(t), t)
        x, y, kx, kt = (torch.where(restart, a, b) for a, b in zip(to, (x, y, kx, kt)))
        xa, ya, kxa, kta = (torch.where(restart, a, b) for a, b in zip(to, (xa, ya, kxa, kta)))
        x0, y0 = torch.where(restart, to[0], x0), torch.where(restart, to[1], y0)
    xo, yo, kto, p = out
    return xo / Dc, yo / Dr, _cone((c - kto) * Dc, lf, uf), p


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        m, n, m1, rp, col, val, c, q, l, u = _lp(_gen(seed), case["family"], case["columns"], case["rows"], case["per_column"])
        x, y, lam, p = _rpdhg(m, n, m1, rp, col, val, c[:, None], q[:, None], l, u, case["steps"])
        out = dict(x=x[:, 0], y=y[:, 0], steps=None, objective=float(p[0]))
        return out if case["family"] == "pagerank" else dict(out, lam=lam[:, 0])
    if kind == "product":
        g = _gen(seed)
        m, n, m1, rp, col, val, *_ = _lp(g, case["family"], case["columns"], case["rows"], case["per_column"])
        x, y = _randn(g, n), _randn(g, m)
        v, _, _ = _scaled(rp, col, val, m, n)
        return dict(Kx=_sparse(rp, col, v, m, n) @ x, KTy=_sparse(*_transposed(rp, col, v, m, n), n, m) @ y)
    if kind == "batch":
        got = []
        for m, n, m1, rp, col, val, c, q, l, u in _members(case, _gen(seed)):
            got.append([v[:, 0] for v in _rpdhg(m, n, m1, rp, col, val, c[:, None], q[:, None], l, u, case["steps"])[:3]])
        x, y, lam = (torch.cat(v) for v in zip(*got))
        return dict(x=x, y=y, lam=lam, steps=None)
    if kind == "shared":
        m, n, m1, rp, col, val, C, Q, l, u = _family(case, _gen(seed))
        x, y, lam, _ = _rpdhg(m, n, m1, rp, col, val, C, Q, l, u, case["steps"])
        return dict(x=x.T.reshape(-1), y=y.T.reshape(-1), lam=lam.T.reshape(-1), steps=None)
    if kind == "gemm":
        A, B = (t.double() for t in _operands(case, seed))
        return (A.T.contiguous() if case["trans_a"] else A) @ (B.T.contiguous() if case["trans_b"] else B)
    dims, parts, mu, sigma, X, Z = _net_inputs(case, seed)
    weights = [w.double().reshape(a, b) for w, a, b in zip(parts[0::2], dims[:-1], dims[1:])]
    biases = [b.double() for b in parts[1::2]]

    def layers(X):
        acts = [(X.double() - mu.double()) / sigma.double()]
        for i, (w, b) in enumerate(zip(weights, biases)):
            z = acts[-1] @ w + b
            acts.append(z.clamp(min=0) if i < 3 else z)
        return acts

    if kind == "forward":
        return layers(X)[-1]
    losses, size = [], case["batch"]
    for i in range(case["minibatches"]):
        acts = layers(X[i * size:(i + 1) * size])
        d = acts[-1] - Z[i * size:(i + 1) * size].double()
        losses.append(float((d * d).mean()))
    d, grads = 2 * d / d.numel(), []
    for i in reversed(range(5)):
        if i < 3:
            d = torch.where(acts[i + 1] > 0, d, torch.zeros_like(d))
        grads = [(acts[i].T.contiguous() @ d).reshape(-1), d.sum(0)] + grads
        d = d @ weights[i].T.contiguous()
    return dict(losses=np.array(losses), gradient=torch.cat(grads))
