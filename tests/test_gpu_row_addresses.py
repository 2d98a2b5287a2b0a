"""The rounding kernels address the rows of a wave's blocks from the first lane's: blocks of one wave in several block rows, and leading
dimensions on both sides of the one beyond which every entry has its own 64-bit offset."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [8, 16, 32, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("ld", [0, (1 << 21) - 24, 1 << 21, (1 << 21) + 40])
@pytest.mark.parametrize("T", [0, 30])
def test_rows_of_a_wave(M, dtype, ld, T):
    import torch

    from paper_2505_23949_amd import binding as b

    rng = np.random.Generator(np.random.Philox(50 + M))
    rows = 128
    # one, two and three block columns: the 64 / M blocks of a wave lie in one to 64 / M block rows, the last wave is not full
    for bc in (1, 2, 3):
        cols = bc * M
        w = rng.standard_normal((rows, cols), dtype=np.float32)
        W = torch.zeros((rows, ld or cols), device="cuda:0", dtype=torch.bfloat16 if dtype == "bf16" else torch.float32)
        at = W.shape[1] - cols  # the last columns: the largest offsets
        W[:, at:] = torch.from_numpy(w).to(W.dtype)
        add = 0.1 * W if T else None
        x = W[:, at:].float().cpu().numpy()
        kw = {}
        if add is not None:
            kw = {"add": add[:, at:], "add_scale": 0.5}
            x = x + np.float32(0.5) * add[:, at:].float().cpu().numpy()
        print(f"[case] rows of a wave M={M} {dtype} ld={ld} bc={bc} T={T}", flush=True)
        res = b.solve(W[:, at:], M // 2, M, 0.05, T, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, flags=b.TSENOR_FLAG_TILES_LARGE, want_stats=True, **kw)
        torch.cuda.synchronize()
        ref = oracle.mask(x, M // 2, M, 0.05, T, tau_mode=oracle.TAU_REL_MATRIX_MAX)
        assert np.array_equal(res["mask"].cpu().numpy(), ref["mask"])
