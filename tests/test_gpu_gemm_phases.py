"""Products with a workspace on the split tiles in phases (tiles cut along the
reduction, their pieces added by a second kernel): edges of tiles, K-tiles and
chunks against the FP64 oracle, and results that repeat bit for bit."""
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


# one tile and remainders of one; fewer columns than a 16-byte load; chunks
# that end in a partial K-tile; one tile row of many cut tiles; whole tiles
# followed by cut ones (18 x 18 tiles of 128)
@pytest.mark.parametrize("shape", [(1, 1, 1024), (64, 3, 4099), (129, 65, 2051), (33, 1300, 1025),
                                   (1024, 1024, 4100), (2200, 2300, 1030)],
                         ids=lambda s: "%dx%dx%d" % s)
def test_phases(li, orc, shape):
    M, N, K = shape
    say("gemm phases", shape)
    need = li.li_gemm_ex_workspace_bytes(M, N, K, "fp32")
    assert need > 0
    A, B = synth.uniform_pm1(181, "A", (M, K)), synth.uniform_pm1(181, "B", (K, N))
    C0 = synth.uniform_pm1(181, "C", (M, N))
    a, b = torch.from_numpy(A).cuda().double(), torch.from_numpy(B).cuda().double()
    p, mags = (a @ b).cpu().numpy(), (a.abs() @ b.abs()).cpu().numpy()
    dA, dB = dev(A), dev(B)
    for alpha, beta in ((1.5, 1.2), (1.0, 0.0)):
        outs = []
        for _ in range(2):
            dC = dev(C0) if beta else empty((M, N), fill=float("nan"))
            ws = empty((need // 4 + 1,), fill=float("nan"))
            li.li_gemm_ex(M, N, K, alpha, dA, dB, beta, dC, "fp32", ws)
            outs.append(host(dC))
        # one rounding per product, sum and final operation, each below 2^-24
        # of the sum of magnitudes
        bound = 2.0 ** -24 * (K + 40) * (alpha * mags + beta * np.abs(C0))
        assert np.all(np.abs(outs[0] - (alpha * p + beta * C0)) <= bound), (alpha, beta)
        assert outs[0].tobytes() == outs[1].tobytes(), (alpha, beta)
