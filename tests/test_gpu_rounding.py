"""round_kernel (Algorithm 2 for M >= 16 by deferred acceptance) against the oracle's sequential selection and swaps."""
import numpy as np
import pytest

import oracle
from paper_2505_23949_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [16, 32, 64])
@pytest.mark.parametrize("share", ["one", "half", "all but one"])
def test_rounding_of_whole_blocks(M, share):
    # N from the smallest to the largest that is solved; numbers of blocks that fill, overfill and leave idle parts of a
    # wave (64 / M blocks); T = 0 on weights of four distinct values (the order is decided by the tie rule nearly
    # everywhere, and is exact on both sides) and T = 30 on continuous ones, both projection orders.
    import torch

    from paper_2505_23949_amd import binding as b

    N = {"one": 1, "half": M // 2, "all but one": M - 1}[share]
    dev = torch.device("cuda:0")
    rng = np.random.Generator(np.random.Philox(900 + M + N))
    per_wave = 64 // M
    for blocks in ((1, 1), (1, 2 * per_wave + 1), (3, per_wave)):
        shape = (blocks[0] * M, blocks[1] * M)
        tied = rng.integers(1, 5, shape).astype(np.float32)
        smooth = rng.standard_normal(shape, dtype=np.float32)
        for W, T, flags in ((tied, 0, 0), (smooth, 30, 0), (smooth, 30, b.TSENOR_FLAG_COLS_FIRST),
                            (smooth, 30, b.TSENOR_FLAG_STRICT_PAPER)):
            print(f"[case] rounding {N}:{M} blocks={blocks} T={T} flags={flags}", flush=True)
            res = b.solve(torch.from_numpy(W).to(dev), N, M, 0.05, T, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, want_stats=True,
                          flags=flags | b.TSENOR_FLAG_TILES_LARGE)
            torch.cuda.synchronize()
            ref = oracle.mask(W, N, M, 0.05, T, tau_mode=synth.TAU_REL_MATRIX_MAX,
                              cols_first=flags == b.TSENOR_FLAG_COLS_FIRST, strict_paper=flags == b.TSENOR_FLAG_STRICT_PAPER)
            assert np.array_equal(res["mask"].cpu().numpy(), ref["mask"])
            assert np.array_equal(res["stats"].cpu().numpy(), ref["stats"])
