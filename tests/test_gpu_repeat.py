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


@pytest.mark.parametrize("M,shape,count", [(4, (512, 512), 2), (4, (60, 68), 3), (8, (512, 512), 2), (16, (512, 512), 2), (16, (512, 1024), 3),
                                           (32, (512, 1024), 3)])
@pytest.mark.parametrize("tol", [0.0, 1e-3])
def test_waves_alone_on_their_simd(M, shape, count, tol):
    # one matrix gives every SIMD at most one wave, a batch of them more (the second case: neither does): other exchanges
    # between the lanes, the same additions
    import torch

    from paper_2505_23949_amd import binding as b

    dev = torch.device("cuda:0")
    rng = np.random.Generator(np.random.Philox(70 + M))
    Ws = [torch.from_numpy(rng.standard_normal(shape, dtype=np.float32)).to(dev) for _ in range(count)]
    for flags in (0, b.TSENOR_FLAG_COLS_FIRST):
        print(f"[case] lone waves M={M} {shape} x {count} tol={tol} flags={flags}", flush=True)
        single = [b.solve(W, M // 2, M, 0.01, 90, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, want_plan=True, tol=tol, flags=flags) for W in Ws]
        masks = [torch.zeros(shape, dtype=torch.uint8, device=dev) for _ in Ws]
        plans = [torch.zeros(shape, dtype=torch.float64, device=dev) for _ in Ws]
        problems = [b.make_problem(W, M // 2, M, 0.01, 90, mask=m, plan_out=p, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, tol=tol, flags=flags)
                    for W, m, p in zip(Ws, masks, plans)]
        b.tsenor_mask_batched(problems, torch.empty(b.tsenor_workspace_bytes(problems), dtype=torch.uint8, device=dev))
        torch.cuda.synchronize()
        for s, m, p in zip(single, masks, plans):
            assert torch.equal(s["mask"], m)
            assert torch.equal(s["plan"], p)
