"""Which calls the tuning rules send to the split tiles (three bf16 parts per
FP32 operand, main-loop modes 9 to 11) and which to the FP32 cores.  No GPU."""
import pytest


@pytest.fixture(scope="module")
def li():
    from paper_2312_13170_amd import li as mod
    return mod


LONG = 2 ** 21  # elements of the longest row that the split tiles take


def split(li, family, M, N, K):
    return li.li_tune_candidate(family, li.li_tune_pick(family, M, N, K))["prefetch"] >= 9


def test_products(li):
    F = li.LI_KERNEL_GEMM_F32
    for M, N in ((1, 1), (64, 5000), (2048, 2048), (8192, 8192)):
        assert not split(li, F, M, N, 119)
        assert split(li, F, M, N, 120)
        assert split(li, F, M, N, LONG)
        assert not split(li, F, M, N, LONG + 1)
    # rows of B and C
    assert split(li, F, 3, LONG, 200) and not split(li, F, 3, LONG + 1, 200)


def test_symmetric_contractions(li):
    S, R = li.LI_KERNEL_SYRK_F32, li.LI_KERNEL_SYRK_ROWS
    assert not split(li, S, 500, 500, 200) and split(li, S, 500, 500, 201)
    assert not split(li, S, 705, 705, 256) and split(li, S, 705, 705, 257)
    assert split(li, R, 64, 64, 64) and split(li, R, 2048, 2048, 160)
    assert not split(li, R, 2048, 2048, 159)


def test_every_pick_is_a_candidate(li):
    for family in (li.LI_KERNEL_GEMM_F32, li.LI_KERNEL_SYRK_F32, li.LI_KERNEL_SYRK_ROWS,
                   li.LI_KERNEL_GROUPED_GEMM, li.LI_KERNEL_GROUPED_COV):
        n = li.li_tune_num_candidates(family)
        for M in (1, 33, 700, 1153, 9000):
            for K in (1, 150, 650, 999, 20000, LONG + 5):
                assert 0 <= li.li_tune_pick(family, M, M, K) < n
