"""Iterations whose state repeats itself are not run: bit for bit the result of running them all.

The early-exit kernels do not look for repetitions: with the smallest tolerance they run a block, with the same arithmetic,
until T or until a check meets an iteration whose factors are all exactly 1.  (A block stopped by the latter no longer takes
part when the fp32 tile of its wave is formed anew, which rounds it differently: such blocks are left out in fp32.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _weights(M, dist, blocks):
    rng = np.random.Generator(np.random.Philox(40 + M))
    if dist == "normal":  # far from convergence after T iterations
        return rng.standard_normal((blocks[0] * M, blocks[1] * M), dtype=np.float32)
    W = rng.standard_t(3, (blocks[0] * M, blocks[1] * M)).astype(np.float32)
    if dist == "mixed":  # every third block converges slowly, its neighbours in the wave within dozens of iterations
        W[:, :] *= 0.02
        for j in range(0, blocks[1], 3):
            W[:, j * M:(j + 1) * M] = rng.standard_normal((blocks[0] * M, M), dtype=np.float32)
    return W


@pytest.mark.parametrize("M", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("tiles", ["large", "large fp32", "small"])
@pytest.mark.parametrize("dist", ["student", "mixed", "normal"])
def test_repeated_states(M, tiles, dist):
    # counts of iterations before, at and behind the distances at which states are compared (4 + 8 k, 24 k), and every
    # remainder that whole periods can leave; a last wave that is not full
    import torch

    from paper_2505_23949_amd import binding as b

    dev = torch.device("cuda:0")
    W = torch.from_numpy(_weights(M, dist, (3, 64 // M * 3 + 1))).to(dev)
    flags = {"large": b.TSENOR_FLAG_TILES_LARGE, "large fp32": b.TSENOR_FLAG_TILES_LARGE | b.TSENOR_FLAG_FP32_ITERATIONS,
             "small": b.TSENOR_FLAG_TILES_SMALL}[tiles]
    N = M // 2
    for T in (1, 5, 12, 24, 47, 48, 100, *range(300, 324, 5), 511):
        for more in (0, b.TSENOR_FLAG_COLS_FIRST) if T == 100 else (0,):
            print(f"[case] repeat {N}:{M} {tiles} {dist} T={T} flags={flags | more}", flush=True)
            got = [b.solve(W, N, M, 0.01, T, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, want_plan=True, flags=flags | more, tol=tol,
                           want_iters_done=tol > 0.0) for tol in (0.0, 1e-300)]
            torch.cuda.synchronize()
            ran = (got[1]["iters_done"] == T).view(W.shape[0] // M, -1).repeat_interleave(M, 0).repeat_interleave(M, 1)
            if flags & b.TSENOR_FLAG_FP32_ITERATIONS == 0:
                ran = torch.ones_like(ran)
            assert ran.any()
            for name in ("plan", "mask"):
                assert torch.equal(got[0][name][ran], got[1][name][ran])
