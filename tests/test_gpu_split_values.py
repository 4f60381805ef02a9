"""The split tiles (three bf16 parts per FP32 operand, split_tile.h) on values
at and beyond the ends of their range, in every form of contraction: what is
infinite or NaN is so as on the FP32 matrix cores, and finite results stay
within FP32's rounding of the FP64 reference.  NaN and small values among
ordinary ones take no second product."""
import numpy as np
import pytest
import torch

from paper_2312_13170_amd import synth
from gpu_util import dev, empty, host, say

pytestmark = pytest.mark.gpu

BIG = np.finfo(np.float32).max


@pytest.fixture(scope="module")
def li():
    from paper_2312_13170_amd import li as mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    mod.li_init()
    return mod


def modes(li, family, split):
    """Candidates of a family: the split tiles, or one of the FP32 cores."""
    n = li.li_tune_num_candidates(family)
    found = [i for i in range(n) if (li.li_tune_candidate(family, i)["prefetch"] >= 9) == split]
    return found if split else found[:1]


class Forced:
    def __init__(self, li, family, cfg):
        self.args = li, family, cfg

    def __enter__(self):
        li, family, cfg = self.args
        li.li_tune_force(family, cfg)

    def __exit__(self, *exc):
        li, family, _ = self.args
        li.li_tune_force(family, -1)


def put(A, B, what):
    """Sets the values of a test in A (M x K) and B (K x N)."""
    M, K = A.shape
    if what == "inf":
        A[3, 7], A[3, 9], A[60, 0], B[11, 1] = np.inf, -np.inf, -np.inf, np.inf
        B[0, ::3] = 0            # NaN beside the infinities of row 60
        B[0, 1::9] = 1e-45       # the smallest value is no zero
        B[0, 2::9] = -1e-38
    elif what == "nan":
        A[M - 1, K - 1], A[0, 1] = np.nan, np.nan
        B[K // 2, 5] = np.nan
    elif what == "huge":         # infinite as bf16, the result is finite
        A[5, 0] = BIG
        B[0, :] *= 0.25
    elif what == "large_sums":   # finite as the FP32 cores sum them
        A[20, :], B[:, 20] = 2.0 ** 55, 2.0 ** 56
    elif what == "sum_overflow":
        A[20, :], B[:, 20] = 2.0 ** 63, 2.0 ** 62
    elif what == "huge_and_inf":
        A[5, 0], A[9, 2], B[3, 4] = BIG, np.inf, np.nan
        B[0, :] *= 0.25
    elif what == "window":       # third parts that are subnormal bf16 values
        A[:] = np.sign(A) * (1 + np.abs(A)) * np.float32(2.0 ** -106)
    elif what == "subnormal":
        A *= np.float32(2.0 ** -130)
    elif what == "mixed":        # a hundredth far below the rest
        A.reshape(-1)[::97] *= np.float32(1e-36)
        B.reshape(-1)[::89] *= np.float32(1e-41)
    elif what == "both_small":   # part products at the end of the FP32 range
        A *= np.float32(2.0 ** -54)
        B *= np.float32(2.0 ** -54)


VALUES = ["inf", "nan", "huge", "large_sums", "sum_overflow", "huge_and_inf", "window", "subnormal", "mixed",
          "both_small"]


# finite values that the split tiles take themselves: no less accurate than the FP32 cores
HELD = ["window", "mixed", "both_small"]


def agree(out, want, ref, mags, K, what):
    assert np.array_equal(np.isnan(out), np.isnan(want)), what
    assert np.array_equal(np.isinf(out), np.isinf(want)), what
    assert np.array_equal(np.signbit(out[np.isinf(out)]), np.signbit(want[np.isinf(want)])), what
    ok = np.isfinite(want)
    # one rounding per product and sum, and FP32's smallest step in each
    assert np.all(np.abs(out[ok] - ref[ok]) <= 2.0 ** -24 * (K + 40) * mags[ok] + (K + 2) * 2.0 ** -149), what
    if what[0] in HELD:
        assert np.mean((out - ref) ** 2) <= np.mean((want - ref) ** 2), what


def wide(A, B):
    with np.errstate(all="ignore"):
        a, b = A.astype(np.float64), B.astype(np.float64)
        return a @ b, np.abs(a) @ np.abs(b)


@pytest.mark.parametrize("what", VALUES)
def test_products(li, what):
    M, N = 140, 150
    for K in (300, 1100):
        A, B = synth.uniform_pm1(201, "A", (M, K)), synth.uniform_pm1(201, "B", (K, N))
        put(A, B, what)
        ref, mags = wide(A, B)
        dA, dB = dev(A), dev(B)

        def single(cfg):
            C = empty((M, N), fill=float("nan"))
            with Forced(li, li.LI_KERNEL_GEMM_F32, cfg):
                li.li_gemm(M, N, K, 1.0, dA, dB, 0.0, C)
            return host(C)

        def batch(cls):
            C = empty((M, N), fill=float("nan"))
            with Forced(li, li.LI_KERNEL_GROUPED_GEMM, cls):
                plan = li.li_group_plan_create([li.make_problem(li.LI_PROBLEM_GEMM, M, N, K, 1.0, 0.0, dA, dB, C)])
            plan.launch()
            out = host(C)
            plan.close()
            return out

        want = single(modes(li, li.LI_KERNEL_GEMM_F32, False)[0])
        for cfg in modes(li, li.LI_KERNEL_GEMM_F32, True):
            say("gemm", what, K, "candidate", cfg)
            agree(single(cfg), want, ref, mags, K, (what, "gemm", cfg))
        for cls in modes(li, li.LI_KERNEL_GROUPED_GEMM, True):
            say("batch", what, K, "class", cls)
            agree(batch(cls), want, ref, mags, K, (what, "batch", cls))
        need = li.li_gemm_ex_workspace_bytes(M, N, K, "fp32")
        assert (need > 0) == (K == 1100)
        if need:  # tiles cut along K
            say("gemm with a workspace", what)
            C = empty((M, N), fill=float("nan"))
            li.li_gemm_ex(M, N, K, 1.0, dA, dB, 0.0, C, "fp32", empty((need // 4 + 1,), fill=float("nan")))
            agree(host(C), want, ref, mags, K, (what, "workspace"))


@pytest.mark.parametrize("what", VALUES)
def test_rank_updates(li, what):
    n, k = 150, 1100
    A, B = synth.uniform_pm1(202, "A", (n, k)), synth.uniform_pm1(202, "B", (k, n))
    put(A, B, what)
    B = np.ascontiguousarray(B.T)
    p, mags = wide(A, B.T)
    dA, dB = dev(A), dev(B)
    ws = torch.empty(li.li_syrk_workspace_bytes(n, k), dtype=torch.uint8, device="cuda")

    def run(cfg):
        C = empty((n, n), fill=float("nan"))
        with Forced(li, li.LI_KERNEL_SYRK_ROWS, cfg):
            li.li_syr2k(n, k, 1.0, dA, dB, 0.0, C, ws)
        return host(C)

    want = run(modes(li, li.LI_KERNEL_SYRK_ROWS, False)[0])
    with np.errstate(all="ignore"):
        ref = p + p.T
    for cfg in modes(li, li.LI_KERNEL_SYRK_ROWS, True):
        say("syr2k", what, "candidate", cfg)
        agree(run(cfg), want, ref, mags + mags.T, 2 * k, (what, cfg))


# feature columns: an infinity or NaN takes its column with it; values whose
# products leave the FP32 range, or lie at its end
@pytest.mark.parametrize("what", ["inf", "nan", "huge", "large", "window", "subnormal", "mixed"])
@pytest.mark.parametrize("fused", [False, True])
def test_statistics(li, what, fused):
    n, k = 150, 1100
    X = synth.uniform_pm1(203, "X", (k, n)) + np.float32(0.75)
    if what in ("inf", "nan"):
        X[700, 40] = np.inf if what == "inf" else np.nan
    elif what == "huge":      # its products are beyond the FP32 range
        X[:, 40] *= np.float32(2.0 ** 115)
    elif what == "large":     # results of 2^120
        X[:, 40] *= np.float32(2.0 ** 60)
    elif what == "window":
        X[:, 40:] *= np.float32(2.0 ** -50)
    elif what == "subnormal":
        X[:, 40] *= np.float32(2.0 ** -135)
    elif what == "mixed":
        X[::3, 40] *= np.float32(1e-38)
    dX = dev(X)
    mean, sd = (torch.empty(n, dtype=torch.float64, device="cuda") for _ in range(2))
    ws = torch.empty(li.li_stats_workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    x = X.astype(np.float64)
    with np.errstate(all="ignore"):
        x = x - x.mean(0)
        if not fused and what != "inf":
            x = x.astype(np.float32).astype(np.float64)  # as the centred data are stored
        ref, mags = x.T @ x / (k - 1), np.abs(x).T @ np.abs(x) / (k - 1)

    def cov(cfg):
        out = empty((n, n), fill=float("nan"))
        with Forced(li, li.LI_KERNEL_SYRK_F32, cfg):
            if fused:
                li.li_covariance_fused(n, k, dX, mean, out, ws)
            else:
                li.li_covariance(n, k, dX, empty((k, n)), mean, out, ws)
        return host(out)

    def corr(cfg):
        out = empty((n, n), fill=float("nan"))
        with Forced(li, li.LI_KERNEL_SYRK_F32, cfg):
            if fused:
                li.li_correlation_fused(n, k, 0.0, dX, mean, sd, out, ws)
            else:
                li.li_correlation(n, k, 0.0, dX, empty((k, n)), mean, sd, out, ws)
        return host(out)

    plain = modes(li, li.LI_KERNEL_SYRK_F32, False)[0]
    want, wantc = cov(plain), corr(plain)
    for cfg in modes(li, li.LI_KERNEL_SYRK_F32, True):
        say("covariance", what, fused, "candidate", cfg)
        # (centred values are rounded once more than the products and sums)
        agree(cov(cfg), want, ref, mags, k + 4, ("statistics", cfg))
        out = corr(cfg)
        assert np.array_equal(np.isnan(out), np.isnan(wantc)), cfg
        ok = np.isfinite(wantc)
        # correlations are at most 1
        assert np.all(np.abs(out[ok] - wantc[ok]) <= 2 * 2.0 ** -24 * (k + 44)), cfg


def test_time_does_not_depend_on_values(li):
    # one NaN in every row of A, and a hundredth of it far below the rest:
    # every block tile has some, and reads its operands once more; a second
    # product on the FP32 cores would take 1.7 times the first's time
    n = 2048
    A, B = torch.from_numpy(synth.uniform_pm1(204, "A", (n, n))).cuda(), torch.from_numpy(synth.uniform_pm1(204, "B", (n, n))).cuda()
    C = torch.empty((n, n), device="cuda")
    nan, tiny = A.clone(), A.clone()
    nan[:, 77] = float("nan")
    tiny.view(-1)[::97] *= 1e-36

    def best(X):
        times = []
        for _ in range(12):
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s.record()
            for _ in range(8):
                li.li_gemm(n, n, n, 1.0, X, B, 0.0, C)
            e.record()
            torch.cuda.synchronize()
            times.append(s.elapsed_time(e))
        return min(times)

    say("times of ordinary, NaN and tiny values")
    best(A)
    t = [best(X) for X in (A, nan, tiny)]
    say("us per call", [round(x / 8 * 1e3, 1) for x in t])
    assert max(t) < 2 * t[0]
