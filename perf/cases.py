"""Timed cases of the library's public entry points.

Each case is one call (or one batched launch) as a program makes it that keeps
its inputs, its outputs and its workspace on the device.  The sizes are those
of the benchmark, of the tests and of the serving stream: tall-skinny A, a
CountSketch of k = 2 n^2 buckets, a Gaussian stage of k2 = 2 n rows.

listed()        the cases
draw(rng)       one more case of the same ranges
prepare(c, s)   the inputs, workspace and outputs of a case, from a seed
run(state)      one pass; returns the outputs
work(c)         bytes and flops one pass cannot do without
exact(c, s)     the outputs in 64 bits, by plain torch
"""
import math

import torch

import paper_2508_14209_amd as ms
import synth

_DT = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # The smallest sketch of the benchmark: launches and latency count.
        dict(name="sketch small f64", op="countsketch", d=65536, n=32, k=2048, dtype="f64"),
        # A ragged data matrix: odd row count (columns not 16-byte aligned),
        # odd column and bucket counts, single precision.
        dict(name="sketch ragged f32", op="countsketch", d=3000017, n=37, k=3001, dtype="f32"),
        # The widest single-precision sketch: more buckets than one compute
        # unit's LDS holds.
        dict(name="sketch large f32", op="countsketch", d=16777216, n=129, k=32768, dtype="f32"),
        # A reproducible sketch of the double-precision least-squares problem
        # (the bit-exact ascending-row fold).
        dict(name="sketch deterministic f64", op="sorted", d=4194304, n=65, k=8192, dtype="f64"),
        # Grouping the rows of one sketch by bucket, for callers that walk the
        # buckets themselves.
        dict(name="bucket plan", op="plan", d=4194304, k=8192),
        # The smallest request of the serving stream, alone.
        dict(name="solve small f64", op="lstsq", d=16384, n=8, nrhs=2, k=128, k2=16, dtype="f64",
             g="f64", refine=0),
        # The benchmark's solve.
        dict(name="solve f64", op="lstsq", d=4194304, n=64, nrhs=1, k=8192, k2=128, dtype="f64",
             g="f64", refine=0),
        # The paper's widest comparison problem.
        dict(name="solve wide f64", op="lstsq", d=4194304, n=256, nrhs=1, k=131072, k2=512,
             dtype="f64", g="f64", refine=0),
        # Mixed precision with FP64-residual refinement: single-precision data,
        # a 16-bit Gaussian stage, several right-hand sides.
        dict(name="solve mixed refined", op="lstsq", d=8388608, n=256, nrhs=4, k=131072, k2=512,
             dtype="f32", g="bf16", refine=3),
        # One batch of the serving loop: 64 requests of the stream together.
        dict(name="batch of 64 requests", op="batch", count=64, d_lo=16384, d_hi=1048576,
             n_lo=8, n_hi=128, refine=2),
        # The least-squares optimum itself, preconditioned by the sketch.
        dict(name="optimum by cholqr f64", op="cholqr", d=4194304, n=64, nrhs=1, k=8192, k2=128,
             dtype="f64", g="f64"),
        # The direct solver on the paper's widest comparison problem.
        dict(name="normal equations wide f64", op="normal", d=4194304, n=256, nrhs=1,
             dtype="f64"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _rows(rng, lo, hi, row_bytes, most):
    """A row count spread over [lo, hi] with at most `most` bytes of data;
    a third of them powers of two or round, the others as they come."""
    hi = max(lo, min(hi, most // row_bytes))
    d = _log(rng, lo, hi)
    if rng.random() < 0.34:
        d = max(lo, min(hi, d // 4096 * 4096))
    return d


def draw(rng):
    op = rng.choice(["countsketch", "countsketch", "sorted", "plan", "lstsq", "lstsq", "mixed",
                     "batch", "cholqr", "normal"])
    if op == "countsketch":
        dtype = rng.choice(["f64", "f32"])
        n = _log(rng, 1, 129)
        d = _rows(rng, 1 << 14, 1 << 24, n * (8 if dtype == "f64" else 4), 8 << 30)
        return dict(op=op, d=d, n=n, k=_log(rng, 128, 32768), dtype=dtype)
    if op == "sorted":
        dtype = rng.choice(["f64", "f64", "f32"])
        n = _log(rng, 8, 65)
        return dict(op=op, d=_rows(rng, 1 << 14, 1 << 22, n * 8, 2 << 30), n=n,
                    k=_log(rng, 128, 16384), dtype=dtype)
    if op == "plan":
        return dict(op=op, d=_log(rng, 1 << 14, 1 << 23), k=_log(rng, 128, 16384))
    if op == "batch":
        return dict(op=op, count=_log(rng, 4, 64), d_lo=1 << 14, d_hi=1 << rng.randint(16, 20),
                    n_lo=8, n_hi=rng.choice([32, 64, 128]), refine=rng.randint(0, 2) or 2)
    if op == "normal":
        n, nrhs = _log(rng, 8, 256), rng.randint(1, 8)
        dtype = rng.choice(["f64", "f64", "f32"])
        return dict(op=op, d=_rows(rng, 1 << 14, 1 << 22, n * 8, 4 << 30), n=n, nrhs=nrhs,
                    dtype=dtype)
    if op == "cholqr":
        n = _log(rng, 8, 64)
        return dict(op=op, d=_rows(rng, 1 << 14, 1 << 22, n * 8, 2 << 30), n=n,
                    nrhs=rng.randint(1, 8), k=2 * n * n, k2=2 * n, dtype="f64", g="f64")
    if op == "mixed":
        n = _log(rng, 8, 256)
        return dict(op="lstsq", d=_rows(rng, 1 << 15, 1 << 23, n * 4, 4 << 30), n=n,
                    nrhs=rng.randint(1, 8), k=2 * n * n, k2=2 * n, dtype="f32", g="bf16",
                    refine=rng.randint(2, 3))
    n = _log(rng, 8, 256)
    return dict(op="lstsq", d=_rows(rng, 1 << 14, 1 << 22, n * 8, 4 << 30), n=n,
                nrhs=rng.randint(1, 8), k=2 * n * n, k2=2 * n, dtype="f64", g="f64", refine=0)


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _sketch(d, k, g):
    h = torch.randint(0, k, (d,), generator=g, dtype=torch.int32, device="cuda")
    s = torch.randint(0, 2, (d,), generator=g, dtype=torch.int8, device="cuda").mul_(2).sub_(1)
    return h, s


def _normal(rows, cols, dtype, g):
    """rows x cols, column-major, N(0, 1)."""
    return torch.empty((cols, rows), dtype=dtype, device="cuda").normal_(generator=g).t()


def _system(c, g):
    """[A | B] in one allocation: A = Z diag(D), B = A x + 1e-6 noise.  Double
    precision: D = 1.  Single precision: D = logspace(0, -4), the mixed-
    precision workload."""
    d, n, nrhs, dt = c["d"], c["n"], c["nrhs"], _DT[c["dtype"]]
    w = torch.empty((n + nrhs, d), dtype=dt, device="cuda")
    w[:n].normal_(generator=g)
    if c["dtype"] == "f32" and c["op"] == "lstsq":
        w[:n].mul_(torch.logspace(0, -4, n, dtype=dt, device="cuda")[:, None])
    x = torch.empty((nrhs, n), dtype=dt, device="cuda").normal_(generator=g)
    w[n:].normal_(generator=g).mul_(1e-6)
    w[n:].addmm_(x, w[:n])
    return w[:n].t(), w[n:].t()


def _gauss(c, g):
    k2, k = c["k2"], c["k"]
    G = torch.empty((k, k2), dtype=torch.float64, device="cuda").normal_(generator=g)
    return G.div_(math.sqrt(k2)).to(torch.float32).to(_DT[c["g"]]).t()


def _requests(c, seed):
    """Descriptors of the stream's next `count` requests: the sizes belong to
    the case, the values to the seed."""
    ns = tuple(n for n in (8, 16, 32, 64, 128) if c["n_lo"] <= n <= c["n_hi"])
    reqs = synth.serving_requests(c["count"], 14209, c["d_lo"], c["d_hi"], ns)
    for r in reqs:
        r["seed"] = seed * 1000003 + r["id"]
    return reqs


def _request_inputs(r):
    return ms.gen_lstsq_request(r["seed"], r["d"], r["n"], r["nrhs"], r["kappa"], r["k"], r["k2"],
                                g_dtype=ms.MS_BF16, want=("A", "B", "h", "s", "G"))


def prepare(c, seed):
    op, st = c["op"], {"c": c}
    if op == "batch":
        reqs = _requests(c, seed)
        # one buffer for every request's X, each a column-major view of it
        st["X"] = torch.zeros(sum(r["n"] * r["nrhs"] for r in reqs), dtype=torch.float64,
                              device="cuda")
        probs, at = [], 0
        for r in reqs:
            p = _request_inputs(r)
            m = r["n"] * r["nrhs"]
            p.update(k=r["k"], X=st["X"][at:at + m].view(r["nrhs"], r["n"]).t())
            probs.append(p)
            at += m
        st["runner"] = ms.BatchRunner(probs, refine_steps=c["refine"])
        return st
    g = _generator(seed)
    if op == "plan":
        st["h"], _ = _sketch(c["d"], c["k"], g)
        st["ws"] = ms.workspace(ms.workspace_size("bucket_plan", d=c["d"], k=c["k"]))
        return st
    dt = _DT[c["dtype"]]
    a_dt = ms.MS_F64 if c["dtype"] == "f64" else ms.MS_F32
    if op in ("countsketch", "sorted"):
        st["A"] = _normal(c["d"], c["n"], dt, g)
        st["h"], st["s"] = _sketch(c["d"], c["k"], g)
        st["Y"] = ms.empty_colmajor(c["k"], c["n"], dt)
        st["ws"] = ms.workspace(ms.workspace_size(
            "countsketch", d=c["d"], n=c["n"], k=c["k"], a_dtype=a_dt,
            mode="sorted" if op == "sorted" else "auto"))
        return st
    st["A"], st["B"] = _system(c, g)
    st["X"] = ms.empty_colmajor(c["n"], c["nrhs"], torch.float64)
    if op == "normal":
        st["ws"] = ms.workspace(ms.workspace_size("normal_equations", d=c["d"], n=c["n"],
                                                  nrhs=c["nrhs"], a_dtype=a_dt))
        return st
    st["h"], st["s"] = _sketch(c["d"], c["k"], g)
    st["G"] = _gauss(c, g)
    g_dt = {"f64": ms.MS_F64, "f32": ms.MS_F32, "bf16": ms.MS_BF16}[c["g"]]
    st["ws"] = ms.workspace(ms.workspace_size(
        "rand_cholqr" if op == "cholqr" else "lstsq", d=c["d"], n=c["n"], nrhs=c["nrhs"],
        k=c["k"], k2=c["k2"], a_dtype=a_dt, g_dtype=g_dt, refine_steps=c.get("refine", 0)))
    return st


def run(st):
    c = st["c"]
    op = c["op"]
    if op == "batch":
        st["runner"].launch()
        return st["X"]
    if op == "plan":
        cnt, off, perm, _ = ms.bucket_plan(st["h"], c["k"], ws=st["ws"])
        return cnt, off, perm
    if op in ("countsketch", "sorted"):
        Y, _ = ms.countsketch_apply(st["A"], st["h"], st["s"], c["k"], Y=st["Y"], ws=st["ws"],
                                    mode="sorted" if op == "sorted" else "auto")
        return Y
    if op == "normal":
        X, _, _ = ms.normal_equations_lstsq(st["A"], st["B"], X=st["X"], ws=st["ws"])
        return X
    if op == "cholqr":
        X, _, _ = ms.rand_cholqr_lstsq(st["A"], st["B"], st["h"], st["s"], st["G"], c["k"],
                                       X=st["X"], ws=st["ws"])
        return X
    X, _ = ms.sketch_lstsq(st["A"], st["B"], st["h"], st["s"], st["G"], c["k"],
                           refine_steps=c["refine"], X=st["X"], ws=st["ws"])
    return X


# --------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------

def _lstsq_work(d, n, nrhs, k, k2, w, wg, refine):
    nc = n + nrhs
    nbytes = d * (nc * w + 5) + k2 * k * wg + n * nrhs * 8
    flops = d * nc + 2 * k2 * k * nc + 2 * k2 * n * n - 2 * n ** 3 // 3 + 2 * k2 * n * nrhs
    flops += refine * nrhs * (2 * d * n + d + 2 * k2 * k + 2 * k2 * n + n * n)
    # the residual needs the X of the pass before it: one more read of A and B a step
    return nbytes + refine * d * nc * w, flops


def work(c):
    op = c["op"]
    if op == "batch":
        nbytes = flops = 0
        for r in _requests(c, 0):
            b, f = _lstsq_work(r["d"], r["n"], r["nrhs"], r["k"], r["k2"], 4, 2, c["refine"])
            nbytes, flops = nbytes + b, flops + f
        return dict(bytes=nbytes, flops=flops)
    d = c["d"]
    if op == "plan":
        return dict(bytes=8 * d + 8 * c["k"] + 4, flops=0)
    n, w = c["n"], 8 if c["dtype"] == "f64" else 4
    if op in ("countsketch", "sorted"):
        return dict(bytes=d * (n * w + 5) + c["k"] * n * w, flops=d * n)
    nrhs = c["nrhs"]
    gram = d * n * (n + 1) + 2 * d * n * nrhs + n ** 3 // 3 + 2 * n * n * nrhs
    if op == "normal":
        return dict(bytes=d * (n + nrhs) * w + n * nrhs * 8, flops=gram)
    wg = {"f64": 8, "f32": 4, "bf16": 2}[c["g"]]
    if op == "cholqr":
        # two reads of A: the second needs the R0 of the first's sketch
        b, f = _lstsq_work(d, n, 0, c["k"], c["k2"], w, wg, 0)
        return dict(bytes=b + d * (n + nrhs) * w + n * nrhs * 8,
                    flops=f + d * n * (n + 1) + gram)
    b, f = _lstsq_work(d, n, nrhs, c["k"], c["k2"], w, wg, c["refine"])
    return dict(bytes=b, flops=f)


# --------------------------------------------------------------------------
# The same in 64 bits, by plain torch
# --------------------------------------------------------------------------

def _countsketch64(A, h, s, k):
    """S A in FP64 (k x n), a few columns at a time."""
    d, n = A.shape
    out = torch.zeros((k, n), dtype=torch.float64, device=A.device)
    hl, sd = h.long(), s.double()[:, None]
    step = max(1, (1 << 27) // d)
    for j in range(0, n, step):
        part = (A[:, j:j + step].double() * sd).contiguous()
        y = torch.zeros((k, part.shape[1]), dtype=torch.float64, device=A.device)
        y.index_add_(0, hl, part)
        out[:, j:j + step] = y
    return out


def _solve64(A, B, h, s, G, k):
    n = A.shape[1]
    Z = G.double() @ torch.cat([_countsketch64(A, h, s, k), _countsketch64(B, h, s, k)], 1)
    Q, R = torch.linalg.qr(Z[:, :n])
    return torch.linalg.solve_triangular(R, Q.t() @ Z[:, n:], upper=True)


def _optimum64(A, B):
    """argmin ||B - A X|| in FP64: the Gram matrix's Cholesky factor, then
    corrections from FP64 residuals."""
    d, n = A.shape
    step = max(1, (1 << 27) // n)
    M = torch.zeros((n, n), dtype=torch.float64, device=A.device)
    for i in range(0, d, step):
        a = A[i:i + step].double()
        M += a.t() @ a
    L = torch.linalg.cholesky(M)
    X = torch.zeros((n, B.shape[1]), dtype=torch.float64, device=A.device)
    for _ in range(3):
        v = torch.zeros_like(X)
        for i in range(0, d, step):
            a = A[i:i + step].double()
            v += a.t() @ (B[i:i + step].double() - a @ X)
        X += torch.cholesky_solve(v, L)
    return X


def exact(c, seed):
    op = c["op"]
    if op == "batch":
        X = []
        for r in _requests(c, seed):
            p = _request_inputs(r)
            X.append(_solve64(p["A"], p["B"], p["h"], p["s"], p["G"], r["k"]).t().reshape(-1))
        return torch.cat(X)
    g = _generator(seed)
    if op == "plan":
        h, _ = _sketch(c["d"], c["k"], g)
        cnt = torch.bincount(h.long(), minlength=c["k"]).int()
        off = torch.cat([cnt.new_zeros(1), cnt.cumsum(0).int()])
        return cnt, off, torch.sort(h, stable=True).indices.int()
    if op in ("countsketch", "sorted"):
        A = _normal(c["d"], c["n"], _DT[c["dtype"]], g)
        h, s = _sketch(c["d"], c["k"], g)
        return _countsketch64(A, h, s, c["k"])
    A, B = _system(c, g)
    if op in ("normal", "cholqr"):
        return _optimum64(A, B)
    h, s = _sketch(c["d"], c["k"], g)
    return _solve64(A, B, h, s, _gauss(c, g), c["k"])
