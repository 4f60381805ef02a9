"""The split tiles (three bf16 parts per FP32 operand, split_tile.h): the error
of single products, whose omitted part products no sum averages out, and the
error of sums against the FP32 matrix cores' in every form of contraction."""
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


class Forced:
    def __init__(self, li, family, cfg):
        self.args = li, family, cfg

    def __enter__(self):
        li, family, cfg = self.args
        li.li_tune_force(family, cfg)

    def __exit__(self, *exc):
        li, family, _ = self.args
        li.li_tune_force(family, -1)


def gemm(li, cfg, A, B):
    M, K = A.shape
    C = empty((M, B.shape[1]), fill=float("nan"))
    with Forced(li, li.LI_KERNEL_GEMM_F32, cfg):
        li.li_gemm(M, B.shape[1], K, 1.0, dev(A), dev(B), 0.0, C)
    return host(C)


def rank_update(li, cfg, A, B=None):
    n, k = A.shape
    C = empty((n, n), fill=float("nan"))
    ws = torch.empty(li.li_syrk_workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    with Forced(li, li.LI_KERNEL_SYRK_ROWS, cfg):
        if B is None:
            li.li_syrk(n, k, 1.0, dev(A), 0.0, C, ws)
        else:
            li.li_syr2k(n, k, 1.0, dev(A), dev(B), 0.0, C, ws)
    return host(C)


def grouped(li, cfg, A, B):
    M, K = A.shape
    dA, dB, C = dev(A), dev(B), empty((M, B.shape[1]), fill=float("nan"))
    with Forced(li, li.LI_KERNEL_GROUPED_GEMM, cfg):
        plan = li.li_group_plan_create([li.make_problem(li.LI_PROBLEM_GEMM, M, B.shape[1], K, 1.0, 0.0, dA, dB, C)])
    plan.launch()
    out = host(C)
    plan.close()
    return out


def operands(values, shape, tag):
    if values == "worst":
        # the largest omission of parts whose first one is cut, not rounded
        return np.full(shape, 1 + 2.0 ** -7 - 2.0 ** -16 - 2.0 ** -23, np.float32)
    x = synth.uniform_pm1(191, tag, shape)
    return np.sign(x) * (1 + np.abs(x))


# One product per result.  Of the nine part products three are left out, below
# (2 + 2^-8) 2^-25 of the product; the two sums meet in one rounding, 2^-24 of
# it, and the roundings of the smaller sum are five of 2^-24 of 2^-7 of it.
BOUND = (2 + 2.0 ** -8) * 2.0 ** -25 + 2.0 ** -24 + 5 * 2.0 ** -31


@pytest.mark.parametrize("values", ["worst", "uniform"])
def test_single_products(li, values):
    n = 130
    a, b = operands(values, (n,), "a"), operands(values, (n, n), "b")
    A = np.diag(a)
    ref = a.astype(np.float64)[:, None] * b.astype(np.float64)
    for cfg in split_candidates(li, li.LI_KERNEL_GEMM_F32):
        say("single products", values, "gemm candidate", cfg)
        assert np.all(np.abs(gemm(li, cfg, A, b) - ref) <= BOUND * np.abs(ref)), cfg
    for cfg in split_candidates(li, li.LI_KERNEL_GROUPED_GEMM):
        say("single products", values, "class", cfg)
        assert np.all(np.abs(grouped(li, cfg, A, b) - ref) <= BOUND * np.abs(ref)), cfg
    # rank 1: all products of one vector, then of two (the second's products
    # of the row and of the column operand are summed: one more rounding)
    c = operands(values, (n, 1), "c")
    p = a.astype(np.float64)[:, None] * c.astype(np.float64).T
    q = a.astype(np.float64)[:, None] * a.astype(np.float64)
    for cfg in split_candidates(li, li.LI_KERNEL_SYRK_ROWS):
        say("single products", values, "rank update candidate", cfg)
        out = rank_update(li, cfg, a[:, None])
        assert np.all(np.abs(out - q) <= BOUND * np.abs(q)), cfg
        out = rank_update(li, cfg, a[:, None], c)
        assert np.all(np.abs(out - (p + p.T)) <= (BOUND + 2.0 ** -24) * (np.abs(p) + np.abs(p.T))), cfg
