"""Calls without a reduction (alpha 0): C = beta C, exactly, on the tile of a
product of no products, and never reading the operands."""
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


@pytest.mark.parametrize("n", [1, 129, 700])
def test_alpha_zero(li, n):
    k = 500
    C0 = synth.uniform_pm1(211, "C", (n, n))
    A = empty((n, k), fill=float("nan"))
    ws = torch.empty(li.li_syrk_workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    say("alpha 0", n)
    want = np.float32(0.5) * C0
    C = dev(C0)
    li.li_gemm(n, n, k, 0.0, A, A, 0.5, C)
    assert np.array_equal(host(C), want)
    C = dev(C0)
    li.li_syrk(n, k, 0.0, A, 0.5, C, ws)
    assert np.array_equal(host(C), want)
    C = dev(C0)
    li.li_syr2k(n, k, 0.0, A, A, 0.5, C, ws)
    assert np.array_equal(host(C), want)
    C = dev(C0)
    plan = li.li_group_plan_create([li.make_problem(li.LI_PROBLEM_GEMM, n, n, k, 0.0, 0.5, A, A, C)])
    plan.launch()
    assert np.array_equal(host(C), want)
    plan.close()


def test_no_slower_than_on_the_fp32_cores(li):
    # C = beta C of 3000 x 3000 against the FP32 cores' tile, forced
    n = 3000
    C = torch.ones((n, n), device="cuda")

    def best():
        times = []
        for _ in range(12):
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s.record()
            for _ in range(20):
                li.li_gemm(n, n, n, 0.0, None, None, 1.0, C)
            e.record()
            torch.cuda.synchronize()
            times.append(s.elapsed_time(e))
        return min(times)

    say("times without a reduction")
    best()
    free = best()
    try:
        li.li_tune_force(li.LI_KERNEL_GEMM_F32, 2)
        fp32 = best()
    finally:
        li.li_tune_force(li.LI_KERNEL_GEMM_F32, -1)
    say("us per call", round(free / 20 * 1e3, 1), round(fp32 / 20 * 1e3, 1))
    assert free < 1.3 * fp32
