"""Matrices with a column scale, whose blocks the iterations take column by column in the order of their scales: plans, masks, counts and
objectives are those of the oracle on a few block rows, and those of the same call in ABSOLUTE mode, which takes them row by row, up to
what a block's last bits owe to the blocks it shares a wave with."""
import numpy as np
import pytest

import oracle
from oracle import exact

pytestmark = pytest.mark.gpu


def _scales(kind, cols, M, rng):
    if kind == "equal":  # ties go by index
        return np.full(cols, 0.75, np.float32)
    if kind == "zeros":  # whole block columns without any importance
        return np.where(np.arange(cols) // M % 3 == 0, 0.0, rng.random(cols)).astype(np.float32)
    if kind == "signed zeros":  # any bits are ordered, as integers: -0 comes before every scale
        at = np.arange(cols) // M
        return np.where(at % 5 == 0, -0.0, np.where(at % 7 == 1, 1e-40, rng.random(cols))).astype(np.float32)
    if kind == "descending":
        return np.linspace(3.0, 0.01, cols, dtype=np.float32)
    return rng.lognormal(0.0, 1.0, cols).astype(np.float32)


def _differ(got, ref, M):
    """Blocks of two masks that differ, of those in which no two entries of the oracle's plan are mathematically tied: closer than 100 times
    what the two sides agree to on a logarithm after some hundred iterations."""
    same = (exact.blocks(got, M) == exact.blocks(ref["mask"], M)).all(axis=(1, 2))
    keys = np.sort(exact.blocks(ref["log_S"], M).reshape(-1, M * M), axis=1)
    size = np.maximum(np.abs(keys[:, 1:]), np.abs(keys[:, :-1]))
    tied = ((np.diff(keys, axis=1) <= 1e-10 * np.maximum(size, 1e-3)) & (size > 0)).any(axis=1)
    return int((~same & ~tied).sum()), int((~tied).sum())


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
@pytest.mark.parametrize("kind", ["equal", "zeros", "signed zeros", "descending", "lognormal"])
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
        # The last bits of a block owe something to the blocks it shares its wave with, which are others in the two orders: in double where
        # increments begin, in fp32 where the tile of a wave is formed anew.
        fp32 = "fp32" in tiles
        differing = (got["mask"] != ref["mask"]).view(br, M, bc, M).any(3).any(1).sum().item()
        # (measured: plans within 1.1e-14 and 9e-7, every mask the same)
        apart = (got["plan"] - ref["plan"]).abs().max().item()
        assert apart < (1e-4 if fp32 else 1e-13)
        assert (got["mask"] != ref["mask"]).float().mean().item() <= (1.2e-4 if fp32 else 0.0)
        assert (got["stats"] - ref["stats"]).abs().max().item() <= M * differing
        mask = got["mask"].cpu().numpy()
        assert exact.is_transposable_nm(mask, N, M)
        objective = oracle.objective(mask, imp, M)
        assert abs(got["objective"][0].item() - objective) <= 1e-12 * objective
        # a few block rows against the oracle
        differ = compared = 0
        for r in sorted({0, br // 2, br - 1}):
            rows_of = slice(r * M, r * M + M)
            of = oracle.mask(np.ascontiguousarray(wide[rows_of, 3:3 + cols]), N, M, te, T, col_scale=scale, cols_first=more != 0,
                             return_plan=True)
            assert np.abs(got["plan"][rows_of].cpu().numpy() - np.exp(of["log_S"])).max() < (1e-4 if fp32 else 1e-9)
            d, n = _differ(mask[rows_of], of, M)
            differ, compared = differ + d, compared + n
        print(f"plans {apart:.1e} apart, blocks of another mask: {differing} in the two orders, {differ} of {compared} by the oracle", flush=True)
        assert differ <= (0.01 * compared if fp32 else 0)


@pytest.mark.parametrize("M,br,bc,tiles", [(8, 13, 317, "small"), (16, 131, 126, "large"), (32, 5, 205, "small"), (32, 64, 65, "large"),
                                           (64, 33, 63, "large"), (32, 91, 91, "large fp32")])
def test_early_exit_by_column_scale(M, br, bc, tiles):
    # a block stops by itself, so that in double everything is bit for bit what the order of the rows gives, at every block's own place
    import torch

    from paper_2505_23949_amd import binding as b

    flags = {"small": b.TSENOR_FLAG_TILES_SMALL, "large": b.TSENOR_FLAG_TILES_LARGE,
             "large fp32": b.TSENOR_FLAG_TILES_LARGE | b.TSENOR_FLAG_FP32_ITERATIONS}[tiles]
    rng = np.random.Generator(np.random.Philox(180 + M))
    N, T, tau, tol = M // 2, 150, 0.02, 1e-4
    W = 0.02 * rng.standard_normal((br * M, bc * M), dtype=np.float32)
    scale = _scales("lognormal", bc * M, M, rng)
    imp = oracle.importance(W, scale)
    te = oracle.tau_eff(imp, tau, oracle.TAU_REL_MATRIX_MAX)
    Wd, s = torch.from_numpy(W).to("cuda:0"), torch.from_numpy(scale).to("cuda:0")
    print(f"[case] early exit by column scale {N}:{M} {br}x{bc} {tiles}", flush=True)
    got = _solve(Wd, s, N, M, T, tau, b.TSENOR_TAU_REL_MATRIX_MAX, flags, tol=tol, want_iters_done=True)
    ref = _solve(Wd, s, N, M, T, te, b.TSENOR_TAU_ABSOLUTE, flags, tol=tol, want_iters_done=True)
    done = got["iters_done"].view(br, bc)
    assert (done < T).any() and done.min().item() < done.max().item()
    if "fp32" not in tiles:
        for name in ("iters_done", "plan", "mask", "stats", "objective"):
            assert torch.equal(got[name], ref[name]), name
    else:
        assert (got["iters_done"] - ref["iters_done"]).abs().max().item() <= 4 * b.TSENOR_ADAPTIVE_CHECK_EVERY
    for r in (0, br - 1):
        _, done_ref = oracle.dykstra_adaptive(imp[r * M:r * M + M], N, M, te, T, tol)
        apart = np.abs(done[r].cpu().numpy() - done_ref.reshape(-1))
        assert apart.max() <= (4 if "fp32" in tiles else 1) * b.TSENOR_ADAPTIVE_CHECK_EVERY


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
