"""Batches whose problems take different shape classes: rows longer than the
split tiles' offsets span, one problem that outweighs all others, and fewer
tiles than there are XCDs.  Whole-number inputs, so every result is exact."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def li():
    from paper_2312_13170_amd import li as mod
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    mod.li_init()
    return mod


LONG = 2 ** 21  # elements of the longest row that the split tiles take


@pytest.mark.parametrize("shapes", [
    [(3, 5, LONG + 5), (65, 33, 40)],                       # long rows of A
    [(2, LONG + 3, 4), (1, 1, 1)],                          # long rows of B and C
    [(1100, 900, 300)] + [(7, 9, 31 + i) for i in range(5)],  # both split classes, one heavy problem
    [(40, 40, 33)],
])
def test_products_are_exact(li, shapes):
    rng = np.random.default_rng(171)
    problems, refs, outs, held = [], [], [], []
    for m, n, k in shapes:
        A = rng.integers(0, 2, (m, k)).astype(np.float32)
        B = rng.integers(0, 3, (k, n)).astype(np.float32)
        C = rng.integers(-4, 5, (m, n)).astype(np.float32)
        refs.append(2.0 * (A.astype(np.float64) @ B) + C)
        a, b, c = dev(A), dev(B), dev(C)
        outs.append(c)
        held += [a, b]  # a problem holds pointers only
        problems.append(li.make_problem(li.LI_PROBLEM_GEMM, m, n, k, 2.0, 1.0, A=a, B=b, C=c))
    say("grouped classes", shapes[0])
    start = [c.clone() for c in outs]
    plan = li.li_group_plan_create(problems)
    for launch in (plan.launch, plan.launch_loop):
        for c, c0 in zip(outs, start):
            c.copy_(c0)
        launch()
        torch.cuda.synchronize()
        for c, r in zip(outs, refs):
            assert np.array_equal(host(c), r)
    plan.close()
