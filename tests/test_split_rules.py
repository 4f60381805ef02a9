"""Rules that keep calls off the split tiles (three bf16 parts per FP32
operand, main-loop modes 9 to 11).  No GPU."""
import pytest


@pytest.fixture(scope="module")
def li():
    from paper_2312_13170_amd import li as mod
    return mod


def split(li, family, M, N, K):
    return li.li_tune_candidate(family, li.li_tune_pick(family, M, N, K))["prefetch"] >= 9


def test_sums_of_few_products(li):
    # results of fewer than four products keep the FP32 cores' rounding
    for family in (li.LI_KERNEL_GEMM_F32, li.LI_KERNEL_SYRK_F32, li.LI_KERNEL_SYRK_ROWS,
                   li.LI_KERNEL_GROUPED_GEMM, li.LI_KERNEL_GROUPED_COV):
        for M in (1, 33, 64, 500, 1500, 9000):
            for K in (1, 2, 3):
                assert not split(li, family, M, M, K), (family, M, K)
    assert split(li, li.LI_KERNEL_SYRK_ROWS, 64, 64, 4)
    assert split(li, li.LI_KERNEL_GROUPED_GEMM, 64, 64, 4)
