"""The split tiles (three bf16 parts per FP32 operand, split_tile.h): edges of
tiles and K-tiles against the FP64 oracle, errors no larger than the FP32
matrix cores', and values that three bf16 parts cannot hold."""
import numpy as np
import pytest
import torch

from paper_2312_13170_amd import synth
from gpu_util import dev, empty, host, say

pytestmark = pytest.mark.gpu

FP32_CORES = 18  # a candidate of the FP32 matrix cores that takes every shape


@pytest.fixture(scope="module")
def li():
    from paper_2312_13170_amd import li as mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    mod.li_init()
    return mod


def split_candidates(li):
    F = li.LI_KERNEL_GEMM_F32
    return [i for i in range(li.li_tune_num_candidates(F)) if li.li_tune_candidate(F, i)["prefetch"] >= 9]


def gemm(li, cfg, A, B, C0=None, alpha=1.0, beta=0.0):
    M, K = A.shape
    N = B.shape[1]
    C = dev(C0) if C0 is not None else empty((M, N), fill=float("nan"))
    try:
        li.li_tune_force(li.LI_KERNEL_GEMM_F32, cfg)
        li.li_gemm(M, N, K, alpha, dev(A), dev(B), beta, C)
    finally:
        li.li_tune_force(li.LI_KERNEL_GEMM_F32, -1)
    return host(C)


# one tile and a remainder of one in M and N; K from below one K-tile to past
# the four (eight) K-tiles where the branch-free loop starts, with remainders
# that are no multiple of a piece of 4 or 8 k
@pytest.mark.parametrize("K", [1, 31, 33, 64, 97, 128, 161, 256, 263, 321, 517])
def test_edges(li, orc, K):
    for M, N in ((1, 1), (129, 65), (64, 131), (33, 34)):
        A = synth.uniform_pm1(141, "A%d" % M, (M, K))
        B = synth.uniform_pm1(141, "B%d" % N, (K, N))
        C0 = synth.uniform_pm1(141, "C%d" % M, (M, N))
        ref = orc.gemm(A, B, C0, alpha=1.5, beta=1.2)
        # the omitted part products are below 3 * 2^-25 of |a b|, and at most
        # one rounding per product, part sum and final operation follows,
        # each below 2^-24 of the sum of magnitudes
        mags = 1.5 * np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64)) + 1.2 * np.abs(C0)
        bound = 2.0 ** -24 * (K + 12) * mags
        for cfg in split_candidates(li):
            say("split", (M, N, K), "candidate", cfg)
            out = gemm(li, cfg, A, B, C0, 1.5, 1.2)
            assert np.all(np.abs(out - ref) <= bound), (M, N, cfg)


# U[-1, 1), all positive, entries a thousand times larger in one of a hundred
@pytest.mark.parametrize("dist", ["uniform", "positive", "outliers"])
@pytest.mark.parametrize("K", [200, 1024, 4000])
def test_error_no_larger_than_fp32_cores(li, orc, K, dist):
    n = 192
    A = synth.uniform_pm1(142, "A", (n, K))
    B = synth.uniform_pm1(142, "B", (K, n))
    if dist == "positive":
        A, B = np.abs(A), np.abs(B)
    if dist == "outliers":
        A[::7, ::13] *= 1000
        B[::11, ::9] *= 1000
    ref = orc.gemm(A, B)

    def rms(x):
        return np.sqrt(np.mean((x - ref) ** 2))

    worst = rms(gemm(li, FP32_CORES, A, B))
    for cfg in split_candidates(li):
        say("split error", K, dist, "candidate", cfg)
        assert rms(gemm(li, cfg, A, B)) <= worst, cfg


# values a bf16 part cannot hold: the block tile is reduced on the FP32 cores
@pytest.mark.parametrize("what", ["inf", "nan", "max", "tiny", "subnormal", "sum_overflow"])
def test_values_outside_the_split(li, what):
    M, N, K = 140, 150, 300
    A = synth.uniform_pm1(143, "A", (M, K))
    B = synth.uniform_pm1(143, "B", (K, N))
    if what == "inf":
        A[3, 7], B[11, 130] = np.inf, -np.inf
    elif what == "nan":
        A[137, 299] = np.nan
    elif what == "max":
        A[5, 0] = np.finfo(np.float32).max
        B[0, :] *= 0.5
    elif what == "tiny":
        A[:, :] *= np.float32(2.0 ** -116)
    elif what == "subnormal":
        A[9, :] *= np.float32(2.0 ** -130)
    elif what == "sum_overflow":
        A[20, :], B[:, 20] = 2.0 ** 63, 2.0 ** 62
    with np.errstate(all="ignore"):
        ref = A.astype(np.float64) @ B.astype(np.float64)
        mags = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64))
    want = gemm(li, FP32_CORES, A, B)
    for cfg in split_candidates(li):
        say("split", what, "candidate", cfg)
        out = gemm(li, cfg, A, B)
        assert np.array_equal(np.isnan(out), np.isnan(want)), cfg
        assert np.array_equal(np.isinf(out), np.isinf(want)), cfg
        assert np.array_equal(np.signbit(out[np.isinf(out)]), np.signbit(want[np.isinf(want)])), cfg
        ok = np.isfinite(want)
        # FP32's rounding of every product and sum, and its smallest step
        assert np.all(np.abs(out[ok] - ref[ok]) <= 2.0 ** -24 * (K + 12) * mags[ok] + K * 2.0 ** -149), cfg
