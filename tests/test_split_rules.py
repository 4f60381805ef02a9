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


def test_long_ranks(li):
    # rows too long for the split tiles: FP32 stream-K in 64 x 64 tiles where
    # they leave padding out; what is forced stands
    R, K = li.LI_KERNEL_SYRK_ROWS, 2 ** 21 + 1
    for n, tile in ((1, 64), (64, 64), (96, 64), (200, 128), (300, 64), (600, 128), (5000, 128)):
        c = li.li_tune_candidate(R, li.li_tune_pick(R, n, n, K))
        assert (c["bm"], c["split_k"]) == (tile, 0) and c["prefetch"] < 9, n
    try:
        li.li_tune_force(R, 7)
        assert li.li_tune_pick(R, 300, 300, K) == 7
    finally:
        li.li_tune_force(R, -1)


def test_small_orders_are_cut(li):
    # rank updates of small orders: split in four from rank 200 on, as the
    # FP32 cores' tile before them
    R = li.LI_KERNEL_SYRK_ROWS
    for n in (1, 33, 64, 65, 96):
        assert li.li_tune_candidate(R, li.li_tune_pick(R, n, n, 199))["split_k"] == 1
        for k in (200, 379, 999):
            assert li.li_tune_candidate(R, li.li_tune_pick(R, n, n, k))["split_k"] == 4, (n, k)
    assert li.li_tune_candidate(R, li.li_tune_pick(R, 97, 97, 399))["split_k"] == 1


def test_short_ranks(li):
    # ranks that fill no pipeline of K-tiles stay on the FP32 cores; a large
    # result of a middling rank is not taken by whole 128 x 128 tiles
    R = li.LI_KERNEL_SYRK_ROWS
    for n, k in ((600, 39), (1000, 16), (1300, 63), (2047, 20), (2048, 100), (8192, 159)):
        assert not split(li, R, n, n, k), (n, k)
    for n, k in ((512, 16), (1000, 40), (1300, 64), (2048, 160)):
        assert split(li, R, n, n, k), (n, k)
    for n, k in ((8192, 200), (10000, 161), (10000, 639)):
        assert li.li_tune_candidate(R, li.li_tune_pick(R, n, n, k))["split_k"] == 0, (n, k)
