"""The calls that a user of the library has it do, as timed and checked cases.

Every case is one call of a public entry point (paper_2312_13170_amd.li, the
names of include/li.h) on device buffers that the caller owns.  Sizes are
those of the benchmark and the tests (256^3 GEMM, 2mm at 2048, 4096 x 2048
statistics, 8192^3 products in three precisions, the batch of uneven
problems, atax at 4096, bicg at 16384) and generic ragged ones.  The values
follow the benchmark's recipes: U[-1, 1) for the polybench operands, feature
columns mu + sigma z with mu ~ U[-10, 10) and sigma ~ U[0.1, 5) for the
statistics, and U[-1, 1) with one entry in a hundred times 1000 for the
16-bit products.  Calls that update their output in place use beta = 0.5, so
the values stay in range however often a state is run.
"""
import math
import random

import torch

from paper_2312_13170_amd import li

ALPHA, BETA = 1.5, 0.5
EPS = 0.1  # the standard deviations at or below it count as constant columns


def listed():
    return [
        # the smallest product of the benchmark: launch and latency
        {"name": "gemm_256", "op": "gemm", "M": 256, "N": 256, "K": 256},
        # a product whose rows are not 16-byte aligned and whose tiles are ragged
        {"name": "gemm_1531x1027x777", "op": "gemm", "M": 1531, "N": 1027, "K": 777},
        # the headline: two chained products
        {"name": "mm2_2048", "op": "mm2", "NI": 2048, "NJ": 2048, "NK": 2048, "NL": 2048},
        # the largest FP32 product of the benchmark
        {"name": "gemm_8192", "op": "gemm", "M": 8192, "N": 8192, "K": 8192},
        # covariance of 2048 features from 4096 samples
        {"name": "covariance_2048x4096", "op": "covariance", "M": 2048, "N": 4096},
        # tall, ragged data through the fused correlation
        {"name": "correlation_fused_501x20011", "op": "correlation_fused", "M": 501, "N": 20011},
        # the rank-2k update at the polybench size
        {"name": "syr2k_1024", "op": "syr2k", "N": 1024, "K": 1024},
        # the 16-bit product of the benchmark
        {"name": "gemm_bf16_8192", "op": "gemm_lp", "precision": "bf16", "M": 8192, "N": 8192, "K": 8192},
        # the compensated 16-bit product at an ordinary size
        {"name": "gemm_bf16x3_4096", "op": "gemm_lp", "precision": "bf16x3", "M": 4096, "N": 4096,
         "K": 4096},
        # the polybench matrix-vector kernels at their sizes: one that fits
        # the last-level cache and one that streams 1 GiB
        {"name": "atax_4096", "op": "atax", "M": 4096, "N": 4096},
        {"name": "bicg_16384", "op": "bicg", "M": 16384, "N": 16384},
        # hundreds of uneven products and covariances in one plan
        {"name": "grouped_512", "op": "grouped", "count": 512, "lo": 32, "hi": 1024, "sizes": 5},
    ]


def _size(rng, lo, hi):
    """A size of [lo, hi], even over its logarithm; half of them multiples of 64."""
    v = round(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    if rng.random() < 0.5:
        v = (v + 32) // 64 * 64
    return max(lo, min(hi, v))


def draw(rng):
    op = rng.choice(["gemm", "gemm", "gemm_ws", "mm2", "mm3", "syrk", "syr2k", "covariance",
                     "correlation", "covariance_fused", "correlation_fused", "gemm_lp", "gemm_lp",
                     "atax", "bicg", "mvt", "gesummv", "grouped"])
    if op in ("gemm", "gemm_ws", "gemm_lp"):
        c = {"op": op, "M": _size(rng, 64, 8192), "N": _size(rng, 64, 8192), "K": _size(rng, 64, 8192)}
        if op == "gemm_lp":
            c["precision"] = rng.choice(["bf16", "fp16", "bf16x3"])
        return c
    if op in ("mm2", "mm3"):
        return dict({"op": op}, **{d: _size(rng, 64, 4096)
                                   for d in ("NI", "NJ", "NK", "NL") + (("NM",) if op == "mm3" else ())})
    if op in ("syrk", "syr2k"):
        return {"op": op, "N": _size(rng, 128, 4096), "K": _size(rng, 64, 8192)}
    if op in ("atax", "bicg", "mvt", "gesummv"):
        return {"op": op, "M": _size(rng, 256, 16384), "N": _size(rng, 256, 16384)}
    if op == "grouped":
        return {"op": op, "count": rng.randint(32, 512), "lo": 32, "hi": rng.choice([128, 256, 512, 1024]),
                "sizes": rng.randrange(1 << 30)}
    return {"op": op, "M": _size(rng, 32, 4096), "N": _size(rng, 64, 32768)}


# ---------------------------------------------------------------- inputs
class _Gen:
    """Seeded device tensors."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def u(self, *shape):
        return torch.rand(*shape, device="cuda", generator=self.g).mul_(2.0).sub_(1.0)

    def features(self, n, m):
        mu = self.u(m) * 10.0
        sd = 0.1 + 4.9 * torch.rand(m, device="cuda", generator=self.g)
        return torch.randn(n, m, device="cuda", generator=self.g).mul_(sd).add_(mu)

    def outliers(self, r, c):
        x = self.u(r, c)
        pick = torch.rand(r, c, device="cuda", generator=self.g) < 0.01
        return torch.where(pick, x * 1000.0, x)


def _shapes(case):
    """The (M, N, K) of a batch's products and the (M, N) of its covariances."""
    r = random.Random(case["sizes"])

    def s():
        return round(math.exp(r.uniform(math.log(case["lo"]), math.log(case["hi"]))))

    n = case["count"]
    return [(s(), s(), s()) for _ in range(n)], [(s(), s()) for _ in range(n)]


def _inputs(case, seed):
    g = _Gen(seed)
    op = case["op"]
    if op in ("gemm", "gemm_ws"):
        M, N, K = case["M"], case["N"], case["K"]
        return {"A": g.u(M, K), "B": g.u(K, N), "C": g.u(M, N)}
    if op == "gemm_lp":
        M, N, K = case["M"], case["N"], case["K"]
        return {"A": g.outliers(M, K), "B": g.outliers(K, N)}
    if op == "mm2":
        ni, nj, nk, nl = case["NI"], case["NJ"], case["NK"], case["NL"]
        return {"A": g.u(ni, nk), "B": g.u(nk, nj), "C": g.u(nj, nl), "D": g.u(ni, nl)}
    if op == "mm3":
        ni, nj, nk, nl, nm = case["NI"], case["NJ"], case["NK"], case["NL"], case["NM"]
        return {"A": g.u(ni, nk), "B": g.u(nk, nj), "C": g.u(nj, nm), "D": g.u(nm, nl)}
    if op in ("syrk", "syr2k"):
        n, k = case["N"], case["K"]
        d = {"A": g.u(n, k), "C": g.u(n, n)}
        if op == "syr2k":
            d["B"] = g.u(n, k)
        return d
    if op in ("atax", "bicg", "mvt", "gesummv"):
        m, n = case["M"], case["N"]
        d = {"A": g.u(m, n), "x": g.u(n)}
        if op in ("bicg", "mvt"):
            d["w"] = g.u(m)
        if op == "mvt":
            d["x1"], d["x2"] = g.u(m), g.u(n)
        if op == "gesummv":
            d["B"] = g.u(m, n)
        return d
    if op == "grouped":
        prods, covs = _shapes(case)
        return {"prods": [(g.u(m, k), g.u(k, n), g.u(m, n)) for m, n, k in prods],
                "covs": [g.u(n, m) for m, n in covs]}
    return {"X": g.features(case["N"], case["M"])}


def _bytes(n):
    """A device workspace of n bytes."""
    return torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")


def _empty(*shape, dtype=torch.float32):
    return torch.empty(*shape, dtype=dtype, device="cuda")


class _Pool:
    """One buffer that holds many results, each at a multiple of 64 elements."""

    def __init__(self, shapes, dtype=torch.float32):
        self.shapes, self.at, n = shapes, [], 0
        for sh in shapes:
            self.at.append(n)
            n += (math.prod(sh) + 63) // 64 * 64
        self.buf = torch.zeros(n, dtype=dtype, device="cuda")

    def __getitem__(self, i):
        return self.buf[self.at[i]:self.at[i] + math.prod(self.shapes[i])].view(self.shapes[i])


def _pools(case, wide):
    """A batch's results: products, centred data, means, covariances."""
    prods, covs = _shapes(case)
    f = torch.float64 if wide else torch.float32
    return (_Pool([(m, n) for m, n, _ in prods], f), _Pool([(n, m) for m, n in covs], f),
            _Pool([(m,) for m, _ in covs], torch.float64), _Pool([(m, m) for m, _ in covs], f))


def prepare(case, seed):
    op = case["op"]
    s = dict(_inputs(case, seed), case=case)
    if op == "gemm_ws":
        s["ws"] = _bytes(li.li_gemm_ex_workspace_bytes(case["M"], case["N"], case["K"], "fp32"))
    elif op == "gemm_lp":
        s["C"] = _empty(case["M"], case["N"])
        s["ws"] = _bytes(li.li_gemm_ex_workspace_bytes(case["M"], case["N"], case["K"], case["precision"]))
    elif op == "mm2":
        s["tmp"] = _empty(case["NI"], case["NJ"])
    elif op == "mm3":
        s["E"], s["F"] = _empty(case["NI"], case["NJ"]), _empty(case["NJ"], case["NL"])
        s["G"] = _empty(case["NI"], case["NL"])
    elif op in ("syrk", "syr2k"):
        s["ws"] = _bytes(li.li_syrk_workspace_bytes(case["N"], case["K"]))
    elif op in ("atax", "bicg", "mvt", "gesummv"):
        m, n = case["M"], case["N"]
        s["ws"] = _bytes(li.li_matvec_workspace_bytes(m, n))
        if op != "mvt":
            s["o1"], s["o2"] = _empty(m), _empty(m if op == "gesummv" else n)
    elif op == "grouped":
        problems = []
        C, Y, mean, cov = pools = _pools(case, False)
        for i, (A, B, C0) in enumerate(s["prods"]):
            C[i].copy_(C0)
            problems.append(li.make_problem(li.LI_PROBLEM_GEMM, A.shape[0], B.shape[1], A.shape[1],
                                            ALPHA, BETA, A=A, B=B, C=C[i]))
        for i, X in enumerate(s["covs"]):
            n, m = X.shape
            problems.append(li.make_problem(li.LI_PROBLEM_COVARIANCE, m, n, A=X, C=cov[i],
                                            data_out=Y[i], mean=mean[i]))
        s["plan"], s["outs"] = li.li_group_plan_create(problems), [p.buf for p in pools]
    else:
        m, n = case["M"], case["N"]
        s["ws"] = _bytes(li.li_stats_workspace_bytes(m, n))
        s["mean"], s["out"] = _empty(m, dtype=torch.float64), _empty(m, m)
        if "correlation" in op:
            s["sd"] = _empty(m, dtype=torch.float64)
        if "fused" not in op:
            s["Y"] = _empty(n, m)
    return s


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "gemm":
        li.li_gemm(c["M"], c["N"], c["K"], ALPHA, s["A"], s["B"], BETA, s["C"])
        return [s["C"]]
    if op == "gemm_ws":
        li.li_gemm_ex(c["M"], c["N"], c["K"], ALPHA, s["A"], s["B"], BETA, s["C"], "fp32", s["ws"])
        return [s["C"]]
    if op == "gemm_lp":
        li.li_gemm_ex(c["M"], c["N"], c["K"], 1.0, s["A"], s["B"], 0.0, s["C"], c["precision"], s["ws"])
        return [s["C"]]
    if op == "mm2":
        li.li_mm2(c["NI"], c["NJ"], c["NK"], c["NL"], ALPHA, BETA, s["A"], s["B"], s["tmp"], s["C"], s["D"])
        return [s["tmp"], s["D"]]
    if op == "mm3":
        li.li_mm3(c["NI"], c["NJ"], c["NK"], c["NL"], c["NM"], s["A"], s["B"], s["C"], s["D"], s["E"],
                  s["F"], s["G"])
        return [s["E"], s["F"], s["G"]]
    if op == "syrk":
        li.li_syrk(c["N"], c["K"], ALPHA, s["A"], BETA, s["C"], s["ws"])
        return [s["C"]]
    if op == "syr2k":
        li.li_syr2k(c["N"], c["K"], ALPHA, s["A"], s["B"], BETA, s["C"], s["ws"])
        return [s["C"]]
    if op == "atax":
        li.li_atax(c["M"], c["N"], s["A"], s["x"], s["o1"], s["o2"], s["ws"])
        return [s["o1"], s["o2"]]
    if op == "bicg":
        li.li_bicg(c["M"], c["N"], s["A"], s["x"], s["w"], s["o1"], s["o2"], s["ws"])
        return [s["o1"], s["o2"]]
    if op == "mvt":
        li.li_mvt(c["M"], c["N"], s["A"], s["x"], s["w"], s["x1"], s["x2"], s["ws"])
        return [s["x1"], s["x2"]]
    if op == "gesummv":
        li.li_gesummv(c["M"], c["N"], ALPHA, BETA, s["A"], s["B"], s["x"], s["o1"], s["o2"], s["ws"])
        return [s["o1"], s["o2"]]
    if op == "grouped":
        s["plan"].launch()
        return s["outs"]
    M, N = c["M"], c["N"]
    if op == "covariance":
        li.li_covariance(M, N, s["X"], s["Y"], s["mean"], s["out"], s["ws"])
        return [s["Y"], s["mean"], s["out"]]
    if op == "correlation":
        li.li_correlation(M, N, EPS, s["X"], s["Y"], s["mean"], s["sd"], s["out"], s["ws"])
        return [s["Y"], s["mean"], s["sd"], s["out"]]
    if op == "covariance_fused":
        li.li_covariance_fused(M, N, s["X"], s["mean"], s["out"], s["ws"])
        return [s["mean"], s["out"]]
    li.li_correlation_fused(M, N, EPS, s["X"], s["mean"], s["sd"], s["out"], s["ws"])
    return [s["mean"], s["sd"], s["out"]]


# ---------------------------------------------------------------- work
def _gemm_work(m, n, k, reads_c):
    return 4 * (m * k + k * n + m * n * (2 if reads_c else 1)), 2 * m * n * k


def _stats_work(m, n, centred):
    return 4 * n * m * (2 if centred else 1) + 8 * m + 4 * m * m, n * m * (m + 1)


def work(case):
    """Bytes and operations that one pass cannot do without."""
    op = case["op"]
    if op in ("gemm", "gemm_ws", "gemm_lp"):
        b, f = _gemm_work(case["M"], case["N"], case["K"], op != "gemm_lp")
    elif op in ("mm2", "mm3"):
        ni, nj, nk, nl = case["NI"], case["NJ"], case["NK"], case["NL"]
        b, f = _gemm_work(ni, nj, nk, False)
        if op == "mm2":
            f += 2 * ni * nj * nl
            b += 4 * (nj * nl + 2 * ni * nl)
        else:
            b2, f2 = _gemm_work(nj, nl, case["NM"], False)
            b += b2 + 4 * ni * nl
            f += f2 + 2 * ni * nj * nl
    elif op in ("syrk", "syr2k"):
        n, k = case["N"], case["K"]
        r = 2 if op == "syr2k" else 1
        b, f = 4 * (r * n * k + 2 * n * n), r * k * n * (n + 1)
    elif op in ("atax", "bicg", "mvt", "gesummv"):
        m, n = case["M"], case["N"]
        b, f = 4 * m * n * (2 if op == "gesummv" else 1) + 8 * (m + n), 4 * m * n
    elif op == "grouped":
        prods, covs = _shapes(case)
        w = [_gemm_work(m, n, k, True) for m, n, k in prods] + [_stats_work(m, n, True) for m, n in covs]
        b, f = sum(x[0] for x in w), sum(x[1] for x in w)
    else:
        b, f = _stats_work(case["M"], case["N"], "fused" not in op)
        if "correlation" in op:
            b += 8 * case["M"]
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- exact
def _exact_stats(X, corr, centred):
    x = X.double()
    n = x.shape[0]
    mean = x.mean(0)
    y = x - mean
    if not corr:
        cov = y.t().contiguous().matmul(y) / (n - 1)
        return [y, mean, cov] if centred else [mean, cov]
    sd = y.square().mean(0).sqrt()
    sd = torch.where(sd <= EPS, torch.ones_like(sd), sd)
    y = y / (math.sqrt(n) * sd)
    r = y.t().contiguous().matmul(y)
    r.fill_diagonal_(1.0)
    return [y, mean, sd, r] if centred else [mean, sd, r]


def exact(case, seed):
    """The first run's outputs from the definitions in 64 bits."""
    d = _inputs(case, seed)
    op = case["op"]
    if op == "grouped":
        C, Y, mean, cov = pools = _pools(case, True)
        for i, (A, B, C0) in enumerate(d["prods"]):
            C[i].copy_(ALPHA * A.double().matmul(B.double()) + BETA * C0.double())
        for i, X in enumerate(d["covs"]):
            y, mu, cv = _exact_stats(X, False, True)
            Y[i].copy_(y)
            mean[i].copy_(mu)
            cov[i].copy_(cv)
        return [p.buf for p in pools]
    if "X" in d:
        return _exact_stats(d["X"], "correlation" in op, "fused" not in op)
    if op == "gemm_lp":
        # the operands as the precision holds them, then the exact products
        A, B = d["A"], d["B"]
        t = torch.float16 if case["precision"] == "fp16" else torch.bfloat16
        Ah, Bh = A.to(t).double(), B.to(t).double()
        C = Ah.matmul(Bh)
        if case["precision"] == "bf16x3":
            Al = (A - A.to(t).float()).to(t).double()
            Bl = (B - B.to(t).float()).to(t).double()
            C += Ah.matmul(Bl)
            C += Al.matmul(Bh)
        return [C]
    d = {k: v.double() for k, v in d.items()}
    if op in ("gemm", "gemm_ws"):
        return [ALPHA * d["A"].matmul(d["B"]) + BETA * d["C"]]
    if op == "mm2":
        tmp = ALPHA * d["A"].matmul(d["B"])
        return [tmp, tmp.matmul(d["C"]) + BETA * d["D"]]
    if op == "mm3":
        E, F = d["A"].matmul(d["B"]), d["C"].matmul(d["D"])
        return [E, F, E.matmul(F)]
    if op in ("syrk", "syr2k"):
        A = d["A"]
        if op == "syrk":
            return [ALPHA * A.matmul(A.t().contiguous()) + BETA * d["C"]]
        P = A.matmul(d["B"].t().contiguous())
        return [ALPHA * (P + P.t()) + BETA * d["C"]]
    A, x = d["A"], d["x"]
    At = A.t().contiguous()
    if op == "atax":
        t = A.mv(x)
        return [t, At.mv(t)]
    if op == "bicg":
        return [A.mv(x), At.mv(d["w"])]
    if op == "mvt":
        return [d["x1"] + A.mv(x), d["x2"] + At.mv(d["w"])]
    t = A.mv(x)
    return [t, ALPHA * t + BETA * d["B"].mv(x)]
