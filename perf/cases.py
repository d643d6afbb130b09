"""Performance cases: the calls that users of this library make, over the
sizes they make them at.

The listed cases follow the library's own workloads (the 2^20 x 1000 FP64
solve, the FP32 refinement form, the batched, served and sparse forms, and the
steps of Alg. 1 called by themselves); draw() gives further cases of the same
ranges, odd and ragged sizes among them.  prepare() builds on the GPU what a
caller holds before the call, run() is one call through the public Python
entry points, exact() the same result from plain torch in FP64.
"""
import math
import random  # noqa: F401  (draw() takes a random.Random)

import torch

import paper_2506_03070_amd as sap

DEV = "cuda"
MODES = {"fp64": sap.SAP_MODE_FP64, "fp32": sap.SAP_MODE_MIXED_FP32, "refine": sap.SAP_MODE_MIXED_FP32_REFINE}
DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}


def listed():
    return [
        # Step S1-S3 by itself: the sketch of the 2^20-row workload.
        dict(name="generate", kind="generate", m=1 << 20, d=4000, zeta=8),
        # Step S4 by itself at the FP64 workload's width and embedding dimension.
        dict(name="apply_f64", kind="apply", m=1 << 19, n=1000, d=4000, zeta=8, a="f64", y="f64"),
        # The same call with an FP32 A and the binding's default FP32 sketch, ragged sizes.
        dict(name="apply_f32", kind="apply", m=300007, n=513, d=2052, zeta=8, a="f32", y="f32"),
        # The sketch of a wide FP32 A, accumulated in FP64 as the mixed solves take it.
        dict(name="apply_mixed", kind="apply", m=1 << 18, n=2048, d=8192, zeta=8, a="f32", y="f64"),
        # Step S5 by itself: the FP64 workload's sketch, and a small ragged one.
        dict(name="qr", kind="qr", rows=4000, cols=1001),
        dict(name="qr_small", kind="qr", rows=1026, cols=257),
        # The smallest whole call (latency and launches): the 20000 x 100 solve.
        dict(name="solve_small", kind="solve", m=20000, n=100, d=400, zeta=8, mode="fp64", method="lsqr"),
        # The headline workload: 2^20 x 1000 in FP64.
        dict(name="solve", kind="solve", m=1 << 20, n=1000, d=4000, zeta=8, mode="fp64", method="lsqr"),
        # The refinement form on FP32 A, wider than one wave's columns.
        dict(name="solve_refine", kind="solve", m=1 << 18, n=2048, d=4096, zeta=8, mode="refine", method="lsqr"),
        # Many independent problems at once.
        dict(name="batch", kind="batch", count=48, mode="refine", shapes=1),
        # A burst of requests to the scheduler, all waited for.
        dict(name="serve", kind="serve", count=24, mode="refine", shapes=1),
        # Sparse A at Table 1's sparse size.
        dict(name="csr", kind="csr", m=500000, n=500, per_row=5.0, d=2000, zeta=8, values="sign"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["generate", "apply", "apply", "qr", "qr", "solve", "solve", "solve", "batch", "serve", "csr"])
    zeta = rng.choice([8, 8, 8, 8, 4, 12, 16])
    if kind == "generate":
        return dict(kind=kind, m=_log_int(rng, 1 << 14, 1 << 21), d=_log_int(rng, 128, 16384), zeta=zeta)
    if kind == "apply":
        n = _log_int(rng, 32, 2048)
        d = min(16384, n * rng.choice([2, 3, 4, 4, 8]) + rng.choice([0, 1, 2]))
        m = _log_int(rng, 1 << 14, min(1 << 20, (1 << 29) // n))
        a, y = rng.choice([("f64", "f64"), ("f64", "f64"), ("f32", "f64"), ("f32", "f32"), ("bf16", "f64")])
        return dict(kind=kind, m=m, n=n, d=d, zeta=zeta, a=a, y=y)
    if kind == "qr":
        n = _log_int(rng, 32, 1300)
        rows = min(8192, n * rng.choice([2, 3, 4, 4, 6, 8]))
        return dict(kind=kind, rows=rows, cols=n + 1)
    if kind == "solve":
        n = _log_int(rng, 32, 1400)
        m = _log_int(rng, max(1 << 13, 16 * n), min(1 << 20, (1 << 29) // n))
        d = min(8192, n * rng.choice([3, 4, 4, 6, 8]))
        mode = rng.choice(["fp64", "fp64", "fp32", "refine"])
        method = "lsqr" if mode == "refine" else rng.choice(["lsqr", "lsqr", "lsqr", "hbm"])
        return dict(kind=kind, m=m, n=n, d=d, zeta=8, mode=mode, method=method)
    if kind == "batch":
        return dict(kind=kind, count=_log_int(rng, 4, 48), mode=rng.choice(["refine", "fp32"]), shapes=rng.randrange(2, 1 << 20))
    if kind == "serve":
        return dict(kind=kind, count=_log_int(rng, 2, 24), mode=rng.choice(["refine", "fp32"]), shapes=rng.randrange(2, 1 << 20))
    n = _log_int(rng, 100, 1500)
    m = _log_int(rng, 1 << 15, 1 << 19)
    return dict(kind="csr", m=m, n=n, per_row=round(rng.uniform(2.0, min(16.0, 0.2 * n)), 2), d=min(8192, 4 * n), zeta=8,
                values=rng.choice(["sign", "gauss"]))


# ---------------------------------------------------------------- inputs ----
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _colscale(m, n, cond, g, dtype):
    """Row-major A_ij = g_ij cond^(-j/(n-1)) and b = A x + 1e-8 (||A x|| / sqrt(m)) N(0, 1)."""
    scale = torch.logspace(0.0, -math.log10(cond), n, device=DEV, dtype=torch.float32)
    A = torch.empty(m, n, device=DEV, dtype=dtype)
    x = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    b = torch.empty(m, device=DEV, dtype=torch.float64)
    rows = max(1, (1 << 27) // n)
    for r in range(0, m, rows):
        blk = (torch.randn(min(rows, m - r), n, generator=g, device=DEV) * scale).to(dtype)
        A[r:r + rows] = blk
        b[r:r + rows] = blk.double() @ x
    b += 1e-8 * (torch.linalg.vector_norm(b) / math.sqrt(m)) * torch.randn(m, generator=g, device=DEV, dtype=torch.float64)
    return A, b


def _shapes(case):
    """The problems of a batch (m ~ U[5000, 200000], n ~ U{32..256}) or of a
    burst (m lognormal around 1e5, n of {64, 128, 256, 512}); d = 4 n."""
    r = random.Random(1000003 * case["shapes"] + case["count"])
    out = []
    for _ in range(case["count"]):
        if case["kind"] == "batch":
            n = r.randint(32, 256)
            m = r.randint(5000, 200000)
        else:
            n = r.choice([64, 128, 256, 512])
            m = min(400000, max(8 * n, int(1e5 * math.exp(r.gauss(0.0, 1.0)))))
        out.append((m, n, 4 * n, 10.0 ** r.uniform(2.0, 6.0)))
    return out


def _csr(case, g):
    m, n = case["m"], case["n"]
    p = case["per_row"] / n
    rows = max(1, (1 << 27) // n)
    counts, cols = [], []
    for r in range(0, m, rows):
        mask = torch.rand(min(rows, m - r), n, generator=g, device=DEV) < p
        counts.append(mask.sum(1))
        cols.append(mask.nonzero()[:, 1].to(torch.int32))
    indptr = torch.zeros(m + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.cat(counts), 0, out=indptr[1:])
    indices = torch.cat(cols)
    if case["values"] == "sign":
        values = torch.randint(0, 2, indices.shape, generator=g, device=DEV).double() * 2 - 1
    else:
        values = torch.randn(indices.shape, generator=g, device=DEV, dtype=torch.float64)
    x = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    row = torch.repeat_interleave(torch.arange(m, device=DEV), indptr[1:] - indptr[:-1])
    b = torch.zeros(m, dtype=torch.float64, device=DEV).index_add_(0, row, values * x[indices.long()])
    b += 1e-6 * torch.randn(m, generator=g, device=DEV, dtype=torch.float64)
    return indptr, indices, values, b, row


def _a_dtype(case):
    return torch.float64 if case["mode"] == "fp64" else torch.float32


def _tol(case):
    return 1e-8 if case["mode"] == "refine" else 1e-12


_serve_ctx = None


def _serving():
    """The context that a serving program keeps."""
    global _serve_ctx
    if _serve_ctx is None:
        _serve_ctx = sap.Context(0)
        sap.sap_serve_start(16 << 30, 1024, ctx=_serve_ctx)
    return _serve_ctx


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = dict(case=case, seed=seed)
    if kind == "generate":
        s["idx"] = torch.empty((case["m"], case["zeta"]), dtype=torch.int32, device=DEV)
        s["sign"] = torch.empty((case["m"],), dtype=torch.int64, device=DEV)
    elif kind == "apply":
        s["A"], s["b"] = _colscale(case["m"], case["n"], 1e4, g, DTYPES[case["a"]])
        s["idx"], s["sign"] = sap.sps_generate(case["m"], case["d"], case["zeta"], seed)
        s["Y"] = torch.empty((case["n"] + 1, case["d"]), dtype=DTYPES[case["y"]], device=DEV)
    elif kind == "qr":
        # a sketch of column-scaled data: Gaussian columns of falling norm (rows of Y0 are its columns)
        scale = torch.logspace(0.0, -4.0, case["cols"], device=DEV, dtype=torch.float64)
        s["Y0"] = torch.randn(case["cols"], case["rows"], generator=g, device=DEV, dtype=torch.float64) * scale[:, None]
        s["Y"] = torch.empty_like(s["Y0"])
    elif kind == "solve":
        s["A"], s["b"] = _colscale(case["m"], case["n"], 1e6, g, _a_dtype(case))
        s["x"] = torch.empty(case["n"], dtype=torch.float64, device=DEV)
    elif kind in ("batch", "serve"):
        shapes = _shapes(case)
        s["d"] = [d for _, _, d, _ in shapes]
        s["A"], s["b"] = zip(*[_colscale(m, n, cond, g, torch.float32) for m, n, _, cond in shapes])
        s["flat"] = torch.empty(sum(n for _, n, _, _ in shapes), dtype=torch.float64, device=DEV)
        s["x"] = list(torch.split(s["flat"], [n for _, n, _, _ in shapes]))
        if kind == "serve":
            s["ctx"] = _serving()
    else:
        s["indptr"], s["indices"], s["values"], s["b"], s["row"] = _csr(case, g)
        s["x"] = torch.empty(case["n"], dtype=torch.float64, device=DEV)
    return s


def run(s):
    case, seed = s["case"], s["seed"]
    kind = case["kind"]
    if kind == "generate":
        return sap.sps_generate(case["m"], case["d"], case["zeta"], seed, idx=s["idx"], sign=s["sign"])
    if kind == "apply":
        return sap.sps_apply(s["idx"], s["sign"], case["d"], case["zeta"], s["A"], s["b"], y_dtype=s["Y"].dtype, Y=s["Y"])
    if kind == "qr":
        s["Y"].copy_(s["Y0"])  # the factorisation is in place
        return s["Y"], sap.sap_qr(s["Y"])
    if kind == "solve":
        if case["method"] == "hbm":
            return sap.sap_solve_hbm(s["A"], s["b"], case["d"], case["zeta"], seed, tol=1e-10, mode=MODES[case["mode"]], x=s["x"]).x
        return sap.sap_solve(s["A"], s["b"], case["d"], case["zeta"], seed, tol=_tol(case), mode=MODES[case["mode"]], x=s["x"]).x
    if kind == "batch":
        sap.sap_solve_batch(s["A"], s["b"], s["d"], 8, seed, tol=_tol(case), xs=s["x"], mode=MODES[case["mode"]])
        return s["flat"]
    if kind == "serve":
        tickets = [sap.sap_submit(A, b, d, 8, seed, tol=_tol(case), ctx=s["ctx"], x=x, mode=MODES[case["mode"]])
                   for A, b, d, x in zip(s["A"], s["b"], s["d"], s["x"])]
        for t in tickets:
            sap.sap_poll(t, wait=True, ctx=s["ctx"])
        return s["flat"]
    return sap.sap_solve_csr(s["indptr"], s["indices"], s["values"], (case["m"], case["n"]), s["b"], case["d"], case["zeta"], seed,
                             x=s["x"]).x


# ------------------------------------------------------------------ work ----
def _solve_work(m, n, nnz, e, d, zeta, iters):
    """One pass over A per iteration and one for the sketch; the sketch's QR; M^T q and M v per iteration."""
    bytes_ = (iters + 2) * (nnz * e + 16 * m) + m * (4 * zeta + 8) + 8 * d * (n + 1)
    flops = 4.0 * nnz * (iters + 1) + 2.0 * zeta * nnz + 2.0 * d * n * n - 2.0 * n ** 3 / 3 + 2.0 * n * n * iters
    return bytes_, flops


def _iters(case, n, d):
    """Iterations the rate sqrt(n/d) of eq. (4.1) needs for the tolerance (two inner solves of 1e-6 in the refinement form)."""
    eps = 1e-12 if case.get("mode") != "refine" else 1e-11
    return math.ceil(2 * math.log(eps) / math.log(n / d))


def work(case):
    kind = case["kind"]
    if kind == "generate":
        return {"bytes": case["m"] * (4 * case["zeta"] + 8), "flops": 0}
    if kind == "apply":
        m, n, d, z = case["m"], case["n"], case["d"], case["zeta"]
        ea, ey = {"f64": 8, "f32": 4, "bf16": 2}[case["a"]], {"f64": 8, "f32": 4}[case["y"]]
        return {"bytes": m * n * ea + 8 * m + m * (4 * z + 8) + d * (n + 1) * ey, "flops": m * z * (n + 1)}
    if kind == "qr":
        r, c = case["rows"], case["cols"]
        return {"bytes": 16 * r * c, "flops": int(2.0 * r * c * c - 2.0 * c ** 3 / 3)}
    if kind == "solve":
        m, n, d = case["m"], case["n"], case["d"]
        b, f = _solve_work(m, n, m * n, 8 if case["mode"] == "fp64" else 4, d, case["zeta"], _iters(case, n, d))
        return {"bytes": int(b), "flops": int(f)}
    if kind in ("batch", "serve"):
        t = [_solve_work(m, n, m * n, 4, d, 8, _iters(case, n, d)) for m, n, d, _ in _shapes(case)]
        return {"bytes": int(sum(b for b, _ in t)), "flops": int(sum(f for _, f in t))}
    m, n, d = case["m"], case["n"], case["d"]
    b, f = _solve_work(m, n, int(m * case["per_row"]), 12, d, case["zeta"], _iters(case, n, d))
    return {"bytes": int(b), "flops": int(f)}


# ----------------------------------------------------------------- exact ----
def _lstsq(rows_of, m, n, b):
    """min ||b - A x|| in FP64: normal equations of the column-equilibrated A
    (the condition of these inputs is column scaling) with residual
    refinement.  rows_of(r0, r1): rows r0..r1-1 of A in FP64."""
    step = max(1, (1 << 27) // n)
    blocks = [(r, min(m, r + step)) for r in range(0, m, step)]
    sq = torch.zeros(n, dtype=torch.float64, device=DEV)
    for r0, r1 in blocks:
        sq += rows_of(r0, r1).square().sum(0)
    s = sq.sqrt()
    G = torch.zeros(n, n, dtype=torch.float64, device=DEV)
    for r0, r1 in blocks:
        B = rows_of(r0, r1) / s
        G += B.T.contiguous() @ B
    L = torch.linalg.cholesky(G)
    x = torch.zeros(n, dtype=torch.float64, device=DEV)
    for _ in range(5):
        g = torch.zeros(n, dtype=torch.float64, device=DEV)
        for r0, r1 in blocks:
            B = rows_of(r0, r1)
            g += B.T @ (b[r0:r1] - B @ x)
        x += torch.cholesky_solve((g / s)[:, None], L)[:, 0] / s
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "generate":
        return None
    s = prepare(case, seed)
    if kind == "apply":
        m, n, d = case["m"], case["n"], case["d"]
        Y = torch.zeros(d, n + 1, dtype=torch.float64, device=DEV)
        step = max(1, (1 << 26) // (n + 1))
        for r in range(0, m, step):
            blk = torch.cat([s["A"][r:r + step].double(), s["b"][r:r + step, None]], 1)
            for k in range(case["zeta"]):
                sg = ((s["sign"][r:r + step] >> k) & 1).double() * 2 - 1
                Y.index_add_(0, s["idx"][r:r + step, k].long(), blk * sg[:, None])
        return (Y / math.sqrt(case["zeta"])).T.contiguous()
    if kind == "qr":
        a, tau = torch.geqrf(s["Y0"].cpu().T.contiguous())
        return a.T.contiguous(), tau
    if kind == "solve":
        return _lstsq(lambda r0, r1: s["A"][r0:r1].double(), case["m"], case["n"], s["b"])
    if kind in ("batch", "serve"):
        return torch.cat([_lstsq(lambda r0, r1, A=A: A[r0:r1].double(), A.shape[0], A.shape[1], b) for A, b in zip(s["A"], s["b"])])

    def rows_of(r0, r1):
        e0, e1 = int(s["indptr"][r0]), int(s["indptr"][r1])
        B = torch.zeros(r1 - r0, case["n"], dtype=torch.float64, device=DEV)
        B[s["row"][e0:e1] - r0, s["indices"][e0:e1].long()] = s["values"][e0:e1]
        return B
    return _lstsq(rows_of, case["m"], case["n"], s["b"])
