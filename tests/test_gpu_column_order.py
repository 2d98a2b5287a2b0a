"""Matrices with a column scale, whose blocks the iterations take column by column in the order of their scales: the results are those
of the oracle, and of the same call in ABSOLUTE mode, which takes them row by row."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def _scales(kind, cols, M, rng):
    if kind == "equal":  # ties go by index
        return np.full(cols, 0.75, np.float32)
    if kind == "zeros":  # whole block columns without any importance
        return np.where(np.arange(cols) // M % 3 == 0, 0.0, rng.random(cols)).astype(np.float32)
    if kind == "descending":
        return np.linspace(3.0, 0.01, cols, dtype=np.float32)
    return rng.lognormal(0.0, 1.0, cols).astype(np.float32)


def _solve(W, scale, N, M, T, tau, mode, flags, **kw):
    import torch

    from paper_2505_23949_amd import binding as b

    got = b.solve(W, N, M, tau, T, col_scale=scale, tau_mode=mode, flags=flags, want_plan=True, want_objective=True, want_stats=True, **kw)
    torch.cuda.synchronize()
    return got


# (M, block rows, block columns, tiles): small tiles from just above the line of the rule on, large ones in both precisions; a matrix
# of two block columns, one with as many as the list holds and one with more (row by row again)
SIZES = [(8, 13, 317, "small"), (16, 2050, 2, "small"), (32, 5, 205, "small"), (8, 2, 4096, "small"), (8, 2, 4097, "small"),
         (8, 33, 994, "large"), (16, 131, 126, "large"), (32, 64, 65, "large"), (32, 91, 91, "large fp32"), (64, 33, 63, "large fp32")]


@pytest.mark.parametrize("M,br,bc,tiles", SIZES)
@pytest.mark.parametrize("kind", ["equal", "zeros", "descending", "lognormal"])
def test_blocks_by_column_scale(M, br, bc, tiles, kind):
    import torch

    from paper_2505_23949_amd import binding as b

    flags = {"small": b.TSENOR_FLAG_TILES_SMALL, "large": b.TSENOR_FLAG_TILES_LARGE,
             "large fp32": b.TSENOR_FLAG_TILES_LARGE | b.TSENOR_FLAG_FP32_ITERATIONS}[tiles]
    rng = np.random.Generator(np.random.Philox(80 + M + bc))
    rows, cols, N, T = br * M, bc * M, M // 2, 150
    wide = (0.02 * rng.standard_normal((rows, cols + 8), dtype=np.float32))
    W = torch.from_numpy(wide).to("cuda:0")[:, 3:3 + cols]  # a column range: ld is not cols, rows are not aligned
    scale = _scales(kind, cols, M, rng)
    s = torch.from_numpy(np.concatenate([[1.0], scale]).astype(np.float32)).to("cuda:0")[1:]
    imp = oracle.importance(np.ascontiguousarray(wide[:, 3:3 + cols]), scale)
    tau = 0.01
    te = oracle.tau_eff(imp, tau, oracle.TAU_REL_MATRIX_MAX)
    for more in (0, b.TSENOR_FLAG_COLS_FIRST) if kind == "lognormal" else (0,):
        print(f"[case] by column scale {N}:{M} {br}x{bc} {tiles} {kind} flags={flags | more}", flush=True)
        got = _solve(W, s, N, M, T, tau, b.TSENOR_TAU_REL_MATRIX_MAX, flags | more)
        ref = _solve(W, s, N, M, T, te, b.TSENOR_TAU_ABSOLUTE, flags | more)
        # in double a block's result does not depend on the blocks it shares its wave with but for the last iterations' rounding; in
        # fp32 the tile of a wave is formed anew for all of its blocks at once
        if "fp32" in tiles:
            assert (got["plan"] - ref["plan"]).abs().max().item() < 1e-4
            assert (got["mask"] != ref["mask"]).float().mean().item() < 1.2e-4
        else:
            assert (got["plan"] - ref["plan"]).abs().max().item() < 1e-11
            assert (got["mask"] != ref["mask"]).float().mean().item() < 2e-5
        # a few block rows against the oracle
        for r in sorted({0, br // 2, br - 1}):
            rows_of = slice(r * M, r * M + M)
            plan = np.exp(oracle.dykstra(imp[rows_of], N, M, te, T, cols_first=more != 0))
            assert np.abs(got["plan"][rows_of].cpu().numpy() - plan).max() < (1e-4 if "fp32" in tiles else 1e-9)


def test_batch_of_ordered_matrices():
    # a list of its own for every matrix of a launch, and one without a scale between them: bit for bit the separate calls
    import torch

    from paper_2505_23949_amd import binding as b

    rng = np.random.Generator(np.random.Philox(99))
    shapes, M = ((1200, 2000), (2000, 1040), (1040, 1600)), 8
    mats = []
    for k, (rows, cols) in enumerate(shapes):
        W = torch.from_numpy(rng.standard_normal((rows, cols), dtype=np.float32)).to("cuda:0")
        mats.append((W, torch.from_numpy(rng.lognormal(0.0, 1.0, cols).astype(np.float32)).to("cuda:0") if k != 1 else None))

    def problems():
        outs = [(torch.zeros(W.shape, dtype=torch.uint8, device="cuda:0"), torch.zeros(W.shape, dtype=torch.float64, device="cuda:0"))
                for W, _ in mats]
        return [b.make_problem(W, 4, M, 0.01, 120, mask=m, plan_out=p, col_scale=s, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX)
                for (W, s), (m, p) in zip(mats, outs)], outs

    print("[case] batch of ordered matrices", flush=True)
    together, outs = problems()
    b.tsenor_mask_batched(together, torch.empty(b.tsenor_workspace_bytes(together), dtype=torch.uint8, device="cuda:0"))
    apart, single = problems()
    for p in apart:
        b.tsenor_mask_ex(p, torch.empty(b.tsenor_workspace_bytes([p]), dtype=torch.uint8, device="cuda:0"))
    torch.cuda.synchronize()
    for (m, p), (ms, ps) in zip(outs, single):
        assert torch.equal(m, ms)
        assert torch.equal(p, ps)
