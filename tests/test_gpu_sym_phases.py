"""The symmetric contractions on the split tiles (three bf16 parts per FP32
operand) in phases of whole and cut tiles: edges of tiles, K-tiles and chunks
against the FP64 oracle, the fused centring, values that three bf16 parts
cannot hold, and results that repeat bit for bit."""
import numpy as np
import pytest
import torch

from paper_2312_13170_amd import synth
from gpu_util import dev, empty, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def li():
    from paper_2312_13170_amd import li as mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    mod.li_init()
    return mod


def split_candidates(li, family):
    return [i for i in range(li.li_tune_num_candidates(family)) if li.li_tune_candidate(family, i)["prefetch"] >= 9]


def rank_update(li, cfg, A, B, C0, alpha, beta):
    n, k = A.shape
    C = dev(C0)
    ws = torch.empty(li.li_syrk_workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    try:
        li.li_tune_force(li.LI_KERNEL_SYRK_ROWS, cfg)
        if B is None:
            li.li_syrk(n, k, alpha, dev(A), beta, C, ws)
        else:
            li.li_syr2k(n, k, alpha, dev(A), dev(B), beta, C, ws)
    finally:
        li.li_tune_force(li.LI_KERNEL_SYRK_ROWS, -1)
    return host(C)


def covariance(li, cfg, X, fused):
    k, n = X.shape
    out, mean = empty((n, n)), torch.empty(n, dtype=torch.float64, device="cuda")
    ws = torch.empty(li.li_stats_workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    try:
        li.li_tune_force(li.LI_KERNEL_SYRK_F32, cfg)
        if fused:
            li.li_covariance_fused(n, k, dev(X), mean, out, ws)
        else:
            li.li_covariance(n, k, dev(X), empty((k, n)), mean, out, ws)
    finally:
        li.li_tune_force(li.LI_KERNEL_SYRK_F32, -1)
    return host(out)


# orders around one, two and many tiles of 32, 64 and 128 (17 tiles of 128:
# 153 upper tiles, one whole phase on 256 compute units or three cut ones);
# reductions of one K-tile, of no multiple of a chunk and of many chunks
SIZES = [(1, 1), (31, 40), (65, 1023), (130, 4099), (257, 300), (2113, 530)]


@pytest.mark.parametrize("n,k", SIZES)
def test_rank_updates(li, n, k):
    A, B = synth.uniform_pm1(151, "A", (n, k)), synth.uniform_pm1(151, "B", (n, k))
    C0 = synth.uniform_pm1(151, "C", (n, n))
    C0 = (C0 + C0.T) / 2
    a, b = torch.from_numpy(A).double(), torch.from_numpy(B).double()
    for two in (False, True):
        p = (a @ b.T if two else a @ a.T).numpy()
        mags = (a.abs() @ (b if two else a).abs().T).numpy()
        ref = 1.5 * (p + p.T if two else p) + 0.5 * C0
        # one rounding per product and sum, each below 2^-24 of the magnitudes
        bound = 2.0 ** -24 * ((2 if two else 1) * k + 40) * (1.5 * (mags + mags.T if two else mags) + 0.5 * np.abs(C0))
        for cfg in split_candidates(li, li.LI_KERNEL_SYRK_ROWS):
            say("rank update", (n, k, two), "candidate", cfg)
            out = rank_update(li, cfg, A, B if two else None, C0, 1.5, 0.5)
            assert np.all(np.abs(out - ref) <= bound), (two, cfg)
            assert np.array_equal(out, out.T), (two, cfg)
            again = rank_update(li, cfg, A, B if two else None, C0, 1.5, 0.5)
            assert out.tobytes() == again.tobytes(), (two, cfg)


@pytest.mark.parametrize("n,k", [(n, k) for n, k in SIZES if k > 1])
def test_covariance(li, n, k):
    X = synth.uniform_pm1(152, "X", (k, n)) + np.float32(0.75)
    x = torch.from_numpy(X).double()
    x = x - x.mean(0)
    ref = (x.T @ x / (k - 1)).numpy()
    mags = (x.abs().T @ x.abs() / (k - 1)).numpy()
    # centred values rounded once more than the products and sums
    bound = 2.0 ** -24 * (k + 44) * mags + 1e-30
    for cfg in split_candidates(li, li.LI_KERNEL_SYRK_F32):
        for fused in (False, True):
            say("covariance", (n, k, fused), "candidate", cfg)
            out = covariance(li, cfg, X, fused)
            assert np.all(np.abs(out - ref) <= bound), (fused, cfg)
            assert np.array_equal(out, out.T), (fused, cfg)


# a tile with an infinity, a NaN, or values below the parts' range is reduced
# on the FP32 cores, the others are not touched by it
@pytest.mark.parametrize("value", [np.inf, np.nan, 1e-37])
def test_values_outside_the_split(li, value):
    n, k = 300, 700
    A = synth.uniform_pm1(153, "A", (n, k))
    A[140, 600] = value
    if value == np.float32(1e-37):
        A[140] = value
    C0 = np.zeros((n, n), np.float32)
    a = torch.from_numpy(A).double()
    ref = (a @ a.T).numpy()
    mags = (a.abs() @ a.abs().T).numpy()
    for cfg in split_candidates(li, li.LI_KERNEL_SYRK_ROWS):
        say("special", value, "candidate", cfg)
        out = rank_update(li, cfg, A, None, C0, 1.0, 0.0)
        ok = np.isfinite(ref)
        # (products of two such small values lie below the FP32 range)
        assert np.all(np.abs(out[ok] - ref[ok]) <= 2.0 ** -24 * (k + 40) * mags[ok] + k * 2.0 ** -149), cfg
        assert np.array_equal(np.isnan(out), np.isnan(ref)) and np.array_equal(np.isinf(out), np.isinf(ref)), cfg
