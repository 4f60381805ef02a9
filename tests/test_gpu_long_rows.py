"""Rows around the longest that the split tiles' 32-bit offsets span, on the
paths that only such rows reach: the FP32 stream-K schedules of products and
rank updates, forced split candidates that have to give way, and the split
tiles at the last length.  Whole numbers, so every result is exact."""
import pytest
import torch

from gpu_util import empty, say

pytestmark = pytest.mark.gpu

LONG = 2 ** 21  # elements of the longest row that the split tiles take


@pytest.fixture(scope="module")
def li():
    from paper_2312_13170_amd import li as mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    mod.li_init()
    return mod


class Forced:
    def __init__(self, li, family, cfg):
        self.args = li, family, cfg

    def __enter__(self):
        li, family, cfg = self.args
        li.li_tune_force(family, cfg)

    def __exit__(self, *exc):
        li, family, _ = self.args
        li.li_tune_force(family, -1)


def sparse(rows, cols, seed):
    """Whole numbers, non-zero in one column of 64: sums stay below 2^24."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.zeros((rows, cols), device="cuda")
    at = torch.arange(seed % 7, cols, 64, device="cuda")
    x[:, at] = torch.randint(-2, 4, (rows, len(at)), device="cuda", generator=g).float()
    x[:, -1] = 3
    return x


def exact(A, B):
    # (sums of whole numbers, in chunks: FP64 copies of the operands are large)
    p = torch.zeros((A.shape[0], B.shape[1]), dtype=torch.float64, device="cuda")
    for k in range(0, A.shape[1], 1 << 18):
        p += A[:, k:k + (1 << 18)].double().contiguous() @ B[k:k + (1 << 18)].double().contiguous()
    return p


def of_mode(li, family, split):
    n = li.li_tune_num_candidates(family)
    return [i for i in range(n) if (li.li_tune_candidate(family, i)["prefetch"] >= 9) == split]


@pytest.mark.parametrize("shape", [(3, 5, LONG + 5), (130, 72, LONG + 4), (2, LONG + 3, 1030)],
                         ids=lambda s: "%dx%dx%d" % s)
def test_products_with_a_workspace(li, shape):
    M, N, K = shape
    need = li.li_gemm_ex_workspace_bytes(M, N, K, "fp32")
    A, B = sparse(M, K, 1), sparse(N, K, 2).T.contiguous()
    ref = 2 * exact(A, B)
    C = empty((M, N), fill=float("nan"))
    say("long rows with a workspace", shape, need)
    li.li_gemm_ex(M, N, K, 2.0, A, B, 0.0, C, "fp32", empty((need // 4 + 4,), fill=float("nan")))
    assert torch.equal(C.double(), ref)


def test_forced_split_products_give_way(li):
    M, N, K = 3, 5, LONG + 5
    A, B = sparse(M, K, 1), sparse(N, K, 2).T.contiguous()
    ref = exact(A, B)
    for cfg in of_mode(li, li.LI_KERNEL_GEMM_F32, True):
        say("long rows, candidate", cfg)
        C = empty((M, N), fill=float("nan"))
        with Forced(li, li.LI_KERNEL_GEMM_F32, cfg):
            li.li_gemm(M, N, K, 1.0, A, B, 0.0, C)
        assert torch.equal(C.double(), ref), cfg


@pytest.mark.parametrize("n", [3, 70, 300])
def test_rank_updates(li, n):
    k = LONG + 5
    A, B = sparse(n, k, 1), sparse(n, k, 2)
    p, q = exact(A, A.T), exact(A, B.T)
    ws = torch.empty(li.li_syrk_workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    # the rule's choice, a split tile that gives way and one of the FP32 cores
    for cfg in (-1, of_mode(li, li.LI_KERNEL_SYRK_ROWS, True)[0], 7):
        say("long rank", n, "candidate", cfg)
        with Forced(li, li.LI_KERNEL_SYRK_ROWS, cfg):
            C = empty((n, n), fill=float("nan"))
            li.li_syrk(n, k, 1.0, A, 0.0, C, ws)
            assert torch.equal(C.double(), p), cfg
            C = empty((n, n), fill=float("nan"))
            li.li_syr2k(n, k, 1.0, A, B, 0.0, C, ws)
            assert torch.equal(C.double(), q + q.T), cfg


def test_last_length_of_the_split_tiles(li):
    # 130 rows of the last length: the largest offsets inside a block tile
    M, N, K = 130, 33, LONG
    A, B = sparse(M, K, 1), sparse(N, K, 2).T.contiguous()
    ref, square = exact(A, B), exact(A, A.T)
    for cfg in of_mode(li, li.LI_KERNEL_GEMM_F32, True):
        say("last length, candidate", cfg)
        C = empty((M, N), fill=float("nan"))
        with Forced(li, li.LI_KERNEL_GEMM_F32, cfg):
            li.li_gemm(M, N, K, 1.0, A, B, 0.0, C)
        assert torch.equal(C.double(), ref), cfg
    need = li.li_gemm_ex_workspace_bytes(M, N, K, "fp32")
    C = empty((M, N), fill=float("nan"))
    say("last length with a workspace")
    li.li_gemm_ex(M, N, K, 1.0, A, B, 0.0, C, "fp32", empty((need // 4 + 4,), fill=float("nan")))
    assert torch.equal(C.double(), ref)
    ws = torch.empty(li.li_syrk_workspace_bytes(M, K), dtype=torch.uint8, device="cuda")
    for cfg in of_mode(li, li.LI_KERNEL_SYRK_ROWS, True):
        say("last length, rank update candidate", cfg)
        C = empty((M, M), fill=float("nan"))
        with Forced(li, li.LI_KERNEL_SYRK_ROWS, cfg):
            li.li_syrk(M, K, 1.0, A, 0.0, C, ws)
        assert torch.equal(C.double(), square), cfg
    # and k-major rows: B and C of the last length
    A, B = sparse(M, 64, 1), sparse(64, LONG, 2)
    ref = exact(A, B)
    for cfg in of_mode(li, li.LI_KERNEL_GEMM_F32, True):
        say("last length of B, candidate", cfg)
        C = empty((M, LONG), fill=float("nan"))
        with Forced(li, li.LI_KERNEL_GEMM_F32, cfg):
            li.li_gemm(M, LONG, 64, 1.0, A, B, 0.0, C)
        assert torch.equal(C.double(), ref), cfg
