"""Algorithm 2 by deferred acceptance, and the layouts of small launches it runs behind, against the oracle's sequential
selection and swaps and against each other."""
import numpy as np
import pytest

import oracle
from paper_2505_23949_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [8, 16, 32, 64])
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


@pytest.mark.parametrize("blocks", [(1, 1), (30, 59), (30, 61)])
def test_fine_tilings_of_16_wide_blocks(blocks):
    # one block, and the two sides of the line (1800 blocks) below which a block has a wave of its own
    import torch

    from paper_2505_23949_amd import binding as b

    dev = torch.device("cuda:0")
    W = np.random.Generator(np.random.Philox(5)).standard_normal((blocks[0] * 16, blocks[1] * 16), dtype=np.float32)
    for cols_first in (False, True):
        print(f"[case] fine tiles {blocks} cols_first={cols_first}", flush=True)
        res = b.solve(torch.from_numpy(W).to(dev), 7, 16, 0.01, 60, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, want_plan=True, want_stats=True,
                      flags=b.TSENOR_FLAG_COLS_FIRST if cols_first else 0)
        torch.cuda.synchronize()
        ref = oracle.mask(W, 7, 16, 0.01, 60, tau_mode=synth.TAU_REL_MATRIX_MAX, cols_first=cols_first, return_plan=True)
        # 1e-9: what the parity tests ask of a plan computed in double on both sides
        assert np.abs(res["plan"].cpu().numpy() - np.exp(ref["log_S"])).max() <= 1e-9
        assert np.array_equal(res["mask"].cpu().numpy(), ref["mask"])
        assert np.array_equal(res["stats"].cpu().numpy(), ref["stats"])


@pytest.mark.parametrize("name,options", [("early exit", {"tol": 1e-2, "T": 300}),
                                          ("early exit, columns first", {"tol": 1e-3, "T": 300, "cols_first": True}),
                                          ("bf16, column scale", {"bf16": True, "scale": True}),
                                          ("bf16, columns first, column scale", {"bf16": True, "scale": True, "cols_first": True}),
                                          ("printed swap rule", {"strict": True})])
def test_four_16_wide_blocks_per_wave(name, options):
    # the small tiles of 16 x 16 blocks, four to a wave, which serve 1800 to 62 000 blocks: 1802 blocks leave two of the last
    # wave's idle; with the early exit the blocks of a wave stop at iterations of their own
    import torch

    from paper_2505_23949_amd import binding as b

    dev, N, M, T = torch.device("cuda:0"), 7, 16, options.get("T", 60)
    rng = np.random.Generator(np.random.Philox(55))
    W = torch.from_numpy(rng.standard_normal((34 * M, 53 * M), dtype=np.float32))
    if options.get("bf16"):
        W = W.to(torch.bfloat16)
    cs = rng.lognormal(0.0, 1.0, W.shape[1]).astype(np.float32) if options.get("scale") else None
    tol, cols_first, strict = options.get("tol", 0.0), options.get("cols_first", False), options.get("strict", False)
    print(f"[case] small tiles of 16 x 16 blocks, {name}", flush=True)
    res = b.solve(W.to(dev), N, M, 0.01, T, col_scale=None if cs is None else torch.from_numpy(cs).to(dev),
                  tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, tol=tol, local_search_steps=2, want_plan=True, want_stats=True,
                  want_iters_done=True, flags=(b.TSENOR_FLAG_COLS_FIRST if cols_first else 0) | (b.TSENOR_FLAG_STRICT_PAPER if strict else 0))
    torch.cuda.synchronize()
    imp = oracle.importance(W.float().numpy(), cs)
    te = oracle.tau_eff(imp, 0.01, synth.TAU_REL_MATRIX_MAX)
    log_S, done = oracle.dykstra_adaptive(imp, N, M, te, T, tol, cols_first=cols_first)
    mask, stats = oracle.round_plan(log_S, imp, N, M, L=2, strict_paper=strict)
    if tol > 0.0:
        assert done.min() < done.max(), "the blocks should stop at different iterations"
    assert np.array_equal(res["iters_done"].cpu().numpy(), done)
    # 1e-9: what the parity tests ask of a plan computed in double on both sides
    assert np.abs(res["plan"].cpu().numpy() - np.exp(log_S)).max() <= 1e-9
    assert np.array_equal(res["mask"].cpu().numpy(), mask)
    assert np.array_equal(res["stats"].cpu().numpy(), stats)


@pytest.mark.parametrize("blocks", [(1, 1), (16, 16), (1, 257)])
def test_workgroup_per_64_wide_block(blocks):
    # one block, and the two sides of the line (257 blocks) below which a block has a workgroup of its own
    import torch

    from paper_2505_23949_amd import binding as b

    dev = torch.device("cuda:0")
    W = np.random.Generator(np.random.Philox(6)).standard_normal((blocks[0] * 64, blocks[1] * 64), dtype=np.float32)
    for cols_first, tol in ((False, 0.0), (True, 0.0), (False, 1e-2)):
        print(f"[case] team {blocks} cols_first={cols_first} tol={tol}", flush=True)
        res = b.solve(torch.from_numpy(W).to(dev), 29, 64, 0.02, 24, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, want_plan=True, want_stats=True,
                      tol=tol, want_iters_done=True, flags=b.TSENOR_FLAG_COLS_FIRST if cols_first else 0)
        torch.cuda.synchronize()
        imp = oracle.importance(W)
        te = oracle.tau_eff(imp, 0.02, synth.TAU_REL_MATRIX_MAX)
        log_S, done = oracle.dykstra_adaptive(imp, 29, 64, te, 24, tol, cols_first=cols_first)
        mask, stats = oracle.round_plan(log_S, imp, 29, 64)
        assert np.array_equal(res["iters_done"].cpu().numpy(), done)
        # 1e-9: what the parity tests ask of a plan computed in double on both sides
        assert np.abs(res["plan"].cpu().numpy() - np.exp(log_S)).max() <= 1e-9
        assert np.array_equal(res["mask"].cpu().numpy(), mask)
        assert np.array_equal(res["stats"].cpu().numpy(), stats)


@pytest.mark.parametrize("M,N", [(16, 9), (32, 21), (64, 45)])
def test_printed_swap_rule_in_a_wave_of_one_block(M, N):
    # Small launches of these sizes give a block a wave of its own, whose lanes beyond the block's rows have to agree with the
    # others on every swap.  One iteration leaves greedy selection so short that blocks take several.
    import torch

    from paper_2505_23949_amd import binding as b

    dev = torch.device("cuda:0")
    W = np.random.Generator(np.random.Philox(60 + M)).standard_normal((5 * M, 7 * M), dtype=np.float32)
    imp = oracle.importance(W)
    log_S = oracle.dykstra(imp, N, M, oracle.tau_eff(imp, 0.01, synth.TAU_REL_MATRIX_MAX), 1)
    masks = {L: oracle.round_plan(log_S, imp, N, M, L=L, strict_paper=True) for L in (2, 60)}
    longer = (masks[2][0] != masks[60][0]).reshape(5, M, 7, M).any(axis=(1, 3))
    assert longer.sum() >= 5, "several blocks should take three and more swaps"
    for L in (2, 60):
        print(f"[case] printed swap rule {N}:{M} L={L}", flush=True)
        res = b.solve(torch.from_numpy(W).to(dev), N, M, 0.01, 1, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, local_search_steps=L,
                      want_stats=True, flags=b.TSENOR_FLAG_STRICT_PAPER)
        torch.cuda.synchronize()
        assert np.array_equal(res["mask"].cpu().numpy(), masks[L][0])
        assert np.array_equal(res["stats"].cpu().numpy(), masks[L][1])


@pytest.mark.parametrize("M,N", [(4, 3), (8, 3), (16, 7), (32, 5), (64, 29)])
def test_swaps_fill_every_row_whatever_their_scores(M, N):
    # Squares of finite weights that overflow: a swap that gives up an infinite importance scores minus infinity or no number
    # at all.  Without the printed rule a valid swap is applied whatever its score, so no row or column stays short.
    import torch

    from oracle import exact
    from paper_2505_23949_amd import binding as b

    rng = np.random.Generator(np.random.Philox(700 + M))
    some = rng.standard_normal((6 * M, 7 * M), dtype=np.float32)
    some[rng.random(some.shape) < 0.6] = 3e19
    for name, W in (("all", np.full_like(some, 3e19)), ("some", some)):
        for T, flags in ((0, 0), (20, 0), (20, b.TSENOR_FLAG_TILES_LARGE)):
            print(f"[case] infinite importances: {name}, {N}:{M} T={T} flags={flags}", flush=True)
            res = b.solve(torch.from_numpy(W).to("cuda:0"), N, M, 0.01, T, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, flags=flags,
                          importance=b.TSENOR_IMPORTANCE_SQUARE, want_stats=True)
            torch.cuda.synchronize()
            assert exact.is_transposable_nm(res["mask"].cpu().numpy(), N, M)
            assert int(res["stats"][3]) == 0


OPTIONS = {"plain": {}, "columns first": {"cols_first": True}, "bf16, column scale": {"bf16": True, "scale": True},
           "early exit": {"tol": 1e-2}, "early exit, columns first, bf16": {"tol": 1e-2, "cols_first": True, "bf16": True},
           "additive term, square, previous mask": {"add": True, "prev": True}, "printed swap rule": {"strict": True}}


@pytest.mark.parametrize("options", list(OPTIONS))
@pytest.mark.parametrize("M,block_rows,block_cols,count", [(16, 30, 59, 2), (16, 9, 11, 16), (16, 1, 1, 2), (64, 11, 23, 2), (64, 2, 5, 16),
                                                           (64, 1, 1, 2)])
def test_a_batch_is_its_calls_on_every_layout(M, block_rows, block_cols, count, options):
    # 16 x 16 and 64 x 64 blocks of small matrices have a wave or a workgroup each as long as the launch is small; a fused
    # launch of several such matrices (here on both sides of its lines, 2048 and 257 blocks) takes the coarser layout, which
    # adds in the same order: every output is that of the calls of their own, bit for bit.  (1, 1): idle lanes.
    import torch

    from paper_2505_23949_amd import binding as b

    dev, o = torch.device("cuda:0"), OPTIONS[options]
    N, (rows, cols) = M // 2 - 1, (block_rows * M, block_cols * M)
    flags = (b.TSENOR_FLAG_COLS_FIRST if o.get("cols_first") else 0) | (b.TSENOR_FLAG_STRICT_PAPER if o.get("strict") else 0)
    gen = torch.Generator(device=dev).manual_seed(M + count)
    dtype = torch.bfloat16 if o.get("bf16") else torch.float32
    keep, probs, outs, singles = [], [], [], []
    print(f"[case] layouts of {count} x {block_rows * block_cols} blocks of {N}:{M}, {options}", flush=True)
    for _ in range(count):
        W, V = ((0.3 * torch.randn((rows, cols), device=dev, generator=gen)).to(dtype) for _ in range(2))
        kw = dict(tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, flags=flags, tol=o.get("tol", 0.0))
        if o.get("scale"):
            kw["col_scale"] = torch.empty(cols, device=dev).log_normal_(0.0, 1.0, generator=gen)
        if o.get("add"):
            kw.update(add=V, add_scale=0.5, importance=b.TSENOR_IMPORTANCE_SQUARE)
        if o.get("prev"):
            kw["prev_mask"] = ((torch.arange(rows, device=dev)[:, None] + torch.arange(cols, device=dev)) % M < N).to(torch.uint8)
        singles.append(b.solve(W, N, M, 0.01, 40, want_plan=True, want_stats=True, want_objective=True, want_iters_done=True, **kw))
        outs.append({k: torch.zeros_like(singles[-1][k]) for k in ("mask", "plan", "stats", "objective", "iters_done")})
        probs.append(b.make_problem(W, N, M, 0.01, 40, mask=outs[-1]["mask"], **{k + "_out": v for k, v in outs[-1].items() if k != "mask"},
                                    **kw))
        keep += [W, kw]
    work = torch.empty(b.tsenor_workspace_bytes(probs), dtype=torch.uint8, device=dev)
    b.tsenor_mask_batched(probs, work)
    if M == 64:
        keep[1]["flags"] |= b.TSENOR_FLAG_TILES_LARGE  # the coarser layout of the first matrix alone
        outs.append(b.solve(keep[0], N, M, 0.01, 40, want_plan=True, want_stats=True, want_objective=True, want_iters_done=True, **keep[1]))
        singles.append(singles[0])
    torch.cuda.synchronize()
    for out, single in zip(outs, singles):
        for k in ("mask", "plan", "stats", "objective", "iters_done"):
            assert torch.equal(out[k], single[k]), k


@pytest.mark.parametrize("T,small", [(20, True), (150, True), (151, False)])
def test_line_of_4_wide_blocks_goes_by_the_iterations(T, small):
    # 102 401 to 114 688 blocks of 4 x 4 in double run on the small tiles up to 150 iterations and on the large ones beyond: the
    # plan, whose sums the two add in different orders, is that of the one asked for by its flag, bit for bit
    import torch

    from paper_2505_23949_amd import binding as b

    dev = torch.device("cuda:0")
    W = torch.from_numpy(np.random.Generator(np.random.Philox(8)).standard_normal((4 * 317, 4 * 341), dtype=np.float32)).to(dev)
    print(f"[case] line of 4 x 4 blocks T={T}", flush=True)
    plans = [b.solve(W, 2, 4, 0.01, T, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, want_plan=True, flags=flags)["plan"]
             for flags in (0, b.TSENOR_FLAG_TILES_SMALL, b.TSENOR_FLAG_TILES_LARGE)]
    torch.cuda.synchronize()
    assert not torch.equal(plans[1], plans[2])
    assert torch.equal(plans[0], plans[1 if small else 2])
