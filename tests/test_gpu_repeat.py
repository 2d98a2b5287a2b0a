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


# name: M, blocks of a matrix, matrices, flags.  Every kernel that looks for repetitions and that the counts above do not reach:
# two and more waves per SIMD, and the layouts of larger launches.
FULL = {
    "4 x 4, large tiles": (4, (257, 257), 1, "large"), "4 x 4, large tiles, fp32": (4, (257, 257), 1, "large fp32"),
    "4 x 4, lone waves of the large tiles": (4, (224, 225), 1, "large"),
    "64 x 64, fp32": (64, (33, 33), 1, "large fp32"), "64 x 64, lone waves in fp32": (64, (17, 18), 1, "large fp32"),
    "4 x 4, small tiles": (4, (130, 131), 1, "small"), "8 x 8, small tiles": (8, (65, 65), 1, "small"),
    "32 x 32, small tiles": (32, (33, 33), 1, "small"),
    "16 x 16, four to a wave": (16, (65, 65), 1, "small"), "16 x 16, four to a lone wave": (16, (43, 44), 1, "small"),
    "16 x 16, finest tiles": (16, (35, 41), 1, "small"),
    "16 x 16, the finest order": (16, (30, 31), 5, "small"), "16 x 16, the finest order, lone waves": (16, (30, 31), 3, "small"),
}


def _call(Ws, M, T, tau, flags, tol, want_plan=True):
    import torch

    from paper_2505_23949_amd import binding as b

    outs = [{"mask": torch.zeros(W.shape, dtype=torch.uint8, device=W.device),
             "plan_out": torch.zeros(W.shape, dtype=torch.float64, device=W.device) if want_plan else None,
             "iters_done_out": torch.zeros(W.numel() // M**2, dtype=torch.int32, device=W.device) if tol > 0.0 else None} for W in Ws]
    problems = [b.make_problem(W, M // 2, M, tau, T, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, flags=flags, tol=tol, **o)
                for W, o in zip(Ws, outs)]
    work = torch.empty(b.tsenor_workspace_bytes(problems), dtype=torch.uint8, device=Ws[0].device)
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    b.tsenor_mask_batched(problems, work)
    end.record()
    torch.cuda.synchronize()
    return outs, start.elapsed_time(end)


def _flag(tiles):
    from paper_2505_23949_amd import binding as b

    return {"large": b.TSENOR_FLAG_TILES_LARGE, "large fp32": b.TSENOR_FLAG_TILES_LARGE | b.TSENOR_FLAG_FP32_ITERATIONS,
            "small": b.TSENOR_FLAG_TILES_SMALL}[tiles]


@pytest.mark.parametrize("path", list(FULL))
def test_repeated_states_in_full_launches(path):
    import torch

    M, blocks, count, tiles = FULL[path]
    dev = torch.device("cuda:0")
    for dist in ("student", "mixed"):
        W = torch.from_numpy(_weights(M, dist, blocks)).to(dev)
        Ws = [W] + [W.roll(7 * k, 0).contiguous() for k in range(1, count)]
        for T in (100, 307, 511):
            print(f"[case] repeat in full launches: {path}, {dist} T={T}", flush=True)
            (got, _), (ref, _) = (_call(Ws, M, T, 0.01, _flag(tiles), tol) for tol in (0.0, 1e-300))
            for g, r in zip(got, ref):
                ran = (r["iters_done_out"] == T).view(*blocks).repeat_interleave(M, 0).repeat_interleave(M, 1)
                if "fp32" not in tiles:
                    ran = torch.ones_like(ran)
                assert ran.any()
                for name in ("mask", "plan_out"):
                    assert torch.equal(g[name][ran], r[name][ran])


@pytest.mark.parametrize("path", list(FULL))
def test_repeated_states_are_not_run(path):
    # One block everywhere, with so large an entropy weight that no entry of its plan is capped and its last bits cycle after dozens
    # of iterations: a call of 60 000 iterations takes little longer than one of 1200 (50 times as long if all of them are run).
    import torch

    M, blocks, count, tiles = FULL[path]
    dev = torch.device("cuda:0")
    W = np.tile(np.random.Generator(np.random.Philox(90 + M)).random((M, M)), blocks).astype(np.float32)
    Ws = [torch.from_numpy(W).to(dev)] * count
    print(f"[case] repeated states are not run: {path}", flush=True)
    short, long = (min(_call(Ws, M, T, 1.0, _flag(tiles), 0.0, want_plan=False)[1] for _ in range(3)) for T in (1200, 60000))
    assert long < 10 * short, (short, long)


@pytest.mark.parametrize("M,blocks,count,tiles", [(4, (224, 225), 2, "large"), (64, (17, 18), 4, "large"), (64, (17, 18), 4, "large fp32"),
                                                  (8, (40, 41), 3, "small"), (32, (21, 22), 3, "small"), (16, (30, 31), 3, "small"),
                                                  (16, (30, 31), 5, "small")])
def test_waves_alone_on_their_simd_where_states_repeat(M, blocks, count, tiles):
    # as above with weights whose states repeat, and on the large tiles; a call of its own has lone waves, the batch none (16 x 16
    # blocks: a wave each in the call; four to a lone wave, and four to a wave that shares its SIMD, in the batches)
    import torch

    W = torch.from_numpy(_weights(M, "mixed", blocks)).to("cuda:0")
    Ws = [W.roll(5 * k, 0).contiguous() for k in range(count)]
    for tol in (0.0, 1e-3):
        print(f"[case] lone waves, repeated states M={M} {blocks} x {count} {tiles} tol={tol}", flush=True)
        batch, _ = _call(Ws, M, 307, 0.01, _flag(tiles), tol)
        for X, of_batch in zip(Ws, batch):
            of_call = _call([X], M, 307, 0.01, _flag(tiles), tol)[0][0]
            for name, value in of_call.items():
                assert value is None or torch.equal(value, of_batch[name])
