"""The last iterations in double, done in increments: the plan is that of the log-domain oracle after T iterations."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# The factors of an iteration carry 2^-48 and an entry of the plan what its block's convergence makes of them, and the oracle's log-domain
# sums round too: up to 1e-12 with and without increments.
PLAN_ATOL = 1e-11

# the tilings whose iterations in double may end in increments
TILINGS = [(8, "large"), (16, "large"), (32, "large"), (16, "small"), (32, "small")]


def _weights(M, dist, blocks):
    rng = np.random.Generator(np.random.Philox(60 + M))
    if dist == "normal":
        return rng.standard_normal((blocks[0] * M, blocks[1] * M), dtype=np.float32)
    W = rng.standard_t(3, (blocks[0] * M, blocks[1] * M)).astype(np.float32)
    if dist == "mixed":  # waves in which one block keeps the others from their increments
        W[:, :] *= 0.02
        for j in range(0, blocks[1], 7):
            W[:, j * M:(j + 1) * M] = rng.standard_normal((blocks[0] * M, M), dtype=np.float32)
    return W


def _copies(W, M, flags):
    """How often the blocks stand beside and below each other in the call: fewer than 1800 blocks of 16 x 16 have finer tiles, which do no
    increments, than the small ones."""
    from paper_2505_23949_amd import binding as b

    return int(np.ceil((1800 * M * M / W.size) ** 0.5)) if M == 16 and flags & b.TSENOR_FLAG_TILES_SMALL else 1


def _plan(W, N, M, tau, T, flags, tol=0.0):
    """Plans (copy, rows, cols) and, with a tolerance, the iterations (copy, blocks) of all copies of the matrix."""
    import torch

    from paper_2505_23949_amd import binding as b

    k = _copies(W, M, flags)
    W_all = torch.from_numpy(np.tile(W, (k, k))).to("cuda:0")
    got = b.solve(W_all, N, M, tau, T, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, flags=flags, tol=tol, want_plan=True,
                  want_iters_done=tol > 0.0)
    torch.cuda.synchronize()

    def split(x, rows, cols):
        return x.cpu().numpy().reshape(k, rows, k, cols).transpose(0, 2, 1, 3).reshape(k * k, rows, cols)

    done = split(got["iters_done"], W.shape[0] // M, W.shape[1] // M).reshape(k * k, -1) if tol > 0.0 else None
    return split(got["plan"], *W.shape), done


@pytest.mark.parametrize("M,tiles", TILINGS)
@pytest.mark.parametrize("dist,tau", [("student", 0.01), ("student", 0.05), ("mixed", 0.02), ("normal", 0.2)])
def test_plan_after_increments(M, tiles, dist, tau):
    # before, at and behind the first windows, and every remainder of the eight increments between two looks
    from paper_2505_23949_amd import binding as b

    flags = b.TSENOR_FLAG_TILES_LARGE if tiles == "large" else b.TSENOR_FLAG_TILES_SMALL
    W = _weights(M, dist, (4, 64 // M * 2 + 1))
    te = oracle.tau_eff(np.abs(W), tau, oracle.TAU_REL_MATRIX_MAX)
    for N in (M // 2, M // 4 + 1):
        for T in (24, 25, 26, 48, 50, 73, 97, 100, *range(121, 129), 400):
            for more in (0, b.TSENOR_FLAG_COLS_FIRST) if T == 100 else (0,):
                print(f"[case] increments {N}:{M} {tiles} {dist} tau={tau} T={T} flags={flags | more}", flush=True)
                ref = np.exp(oracle.dykstra(np.abs(W), N, M, te, T, cols_first=more != 0))
                plan, _ = _plan(W, N, M, tau, T, flags | more)
                assert np.abs(plan - ref).max() < PLAN_ATOL
                same, done = _plan(W, N, M, tau, T, flags | more, 1e-300)
                assert np.array_equal(plan, same)


def _plan_80_bits(W, N, M, tau_eff, T):
    blocks = (W.shape[0] // M, M, W.shape[1] // M, M)
    K = (tau_eff * np.abs(W).astype(np.float64)).reshape(blocks).transpose(0, 2, 1, 3).reshape(-1, M, M)
    kappa = np.exp((K - K.max(2, keepdims=True)).astype(np.longdouble))
    U, V = (np.ones((len(K), M), np.longdouble) for _ in range(2))
    for _ in range(T):
        e = np.minimum(kappa * U[:, :, None] * V[:, None, :], 1)
        R = N / e.sum(2)
        V *= N / (e * R[:, :, None]).sum(1)
        U *= R
    plan = np.minimum(kappa * U[:, :, None] * V[:, None, :], 1).astype(np.float64)
    return plan.reshape(blocks[0], blocks[2], M, M).transpose(0, 2, 1, 3).reshape(W.shape)


@pytest.mark.parametrize("M,tiles", TILINGS)
@pytest.mark.parametrize("dist,tau,T", [("student", 0.02, 300), ("normal", 0.1, 300)])
def test_error_of_the_plan_after_increments(M, tiles, dist, tau, T):
    # An entry is exp((K - m) + (f + g)): a few roundings of numbers up to 1 / tau, 0.2e-15 to 1.2e-15 in these cases.  Iterations in double
    # to the end, and increments that start from their factors of 2^-48, leave 1.7e-15 to 2.3e-15.
    from paper_2505_23949_amd import binding as b

    flags = b.TSENOR_FLAG_TILES_LARGE if tiles == "large" else b.TSENOR_FLAG_TILES_SMALL
    W = _weights(M, dist, (4, 64 // M * 2 + 1))
    te = oracle.tau_eff(np.abs(W), tau, oracle.TAU_REL_MATRIX_MAX)
    print(f"[case] error of the plan {M // 2}:{M} {tiles} {dist} tau={tau}", flush=True)
    ref = _plan_80_bits(W, M // 2, M, te, T)
    plan, _ = _plan(W, M // 2, M, tau, T, flags)
    error = np.sqrt(((plan - ref) ** 2).sum() / (ref**2).sum() / len(plan))
    print(f"error {error:.3e} max {np.abs(plan - ref).max():.3e}", flush=True)
    assert error < 1.45e-15


@pytest.mark.parametrize("M,T,seed", [(8, 30000, None), (16, 30000, None), (8, 30000, 30116), (16, 10000, 10172)])
def test_increments_of_many_iterations(M, T, seed):
    # slow blocks: the increments' sum passes its bound, and the plan they act on is formed anew
    from paper_2505_23949_amd import binding as b

    N, tau = M // 2, 0.02 if seed is None else 1.0 / 60.0
    W = _weights(M, "normal", (2, 64 // M)) if seed is None else np.random.default_rng(seed).standard_normal((M, 8 * M)).astype(np.float32)
    te = oracle.tau_eff(np.abs(W), tau, oracle.TAU_REL_MATRIX_MAX)
    print(f"[case] increments of many iterations {N}:{M} T={T} seed={seed}", flush=True)
    ref = _plan_80_bits(W, N, M, te, T)
    plan, _ = _plan(W, N, M, tau, T, b.TSENOR_FLAG_TILES_LARGE)
    # (four roundings of numbers up to 60, the largest K, in the logarithm of an entry.  With sums in fp32 and factors of 2^-48 before them
    # the last two are off by 2.7e-13 and 5.6e-14, with iterations in double to the end by 1.3e-14 and 2.3e-14.)
    print(f"max error {np.abs(plan - ref).max():.3e}", flush=True)
    assert np.abs(plan - ref).max() < 4 * 60 * 2.0**-53


def test_entry_that_drifts_to_the_cap():
    # Two parts, each with a capped entry of the other's columns, and an entry of 7e-12 in one of the two corners only: the plan stands
    # still and the capped entry of that corner comes down by 2e-12 per iteration.  It is 1e-6 above the cap once the rest has
    # converged and 1.3e-11 below it at the end.
    from paper_2505_23949_amd import binding as b

    import torch

    M, N, T = 8, 3, 700000
    rng = np.random.default_rng(0)
    K = np.full((M, M), -200.0)
    for part in (slice(0, 4), slice(4, 8)):
        K[part, part] = 0.3 * rng.random((4, 4))
    K[0, 4], K[4, 0], K[1, 5] = 0.0063, 5.0, -25.7
    W = (K + 200.0).astype(np.float32)

    def above(tau):
        log_S, log_Q = oracle.dykstra(W, N, M, tau, 150, return_log_Q=True)
        return log_Q[0, 4] + log_S[0, 4] - 1.05e-6

    low, high = 1.0, 1.001
    for _ in range(50):
        mid = 0.5 * (low + high)
        low, high = (low, mid) if above(mid) > 0.0 else (mid, high)
    print("[case] entry that drifts to the cap", flush=True)
    ref = np.exp(oracle.dykstra(W, N, M, high, T))
    assert 1e-11 < 1.0 - ref[0, 4] < 2e-11
    got = b.solve(torch.from_numpy(W).to("cuda:0"), N, M, high, T, tau_mode=b.TSENOR_TAU_ABSOLUTE, flags=b.TSENOR_FLAG_TILES_LARGE,
                  want_plan=True)
    assert np.abs(got["plan"].cpu().numpy() - ref).max() < 1e-12


@pytest.mark.parametrize("M,tiles", TILINGS)
def test_tolerance_met_in_increments(M, tiles):
    # a tolerance far below where they begin, and far above the rounding of the factors: the count is the oracle's
    from paper_2505_23949_amd import binding as b

    W, N, tau, T, tol = _weights(M, "student", (3, 64 // M * 2)), M // 2, 0.05, 600, 1e-12
    te = oracle.tau_eff(np.abs(W), tau, oracle.TAU_REL_MATRIX_MAX)
    flags = b.TSENOR_FLAG_TILES_LARGE if tiles == "large" else b.TSENOR_FLAG_TILES_SMALL
    print(f"[case] tolerance met in increments {N}:{M} {tiles}", flush=True)
    log_S, done_ref = oracle.dykstra_adaptive(np.abs(W), N, M, te, T, tol)
    plan, done = _plan(W, N, M, tau, T, flags, tol)
    # (factors at the tolerance carry 4e-15 and the increments 1e-7 of themselves: one look earlier or later)
    assert np.abs(done - done_ref.reshape(-1)).max() <= b.TSENOR_ADAPTIVE_CHECK_EVERY
    assert (done < T).any()
    assert np.abs(plan - np.exp(log_S)).max() < PLAN_ATOL


@pytest.mark.parametrize("M,tiles", TILINGS)
def test_tolerance_below_the_factors_rounding(M, tiles):
    # Factors of iterations in double carry 2^-48, by which 0.1 to 0.6 of these blocks miss the smaller one to the end; the increments do
    # not, so that this also shows that they are run.  (Started from such factors they kept what these left of a constant in rows and
    # columns, and 0.1 of the blocks missed the larger one too.)
    from paper_2505_23949_amd import binding as b

    W, N, tau, T = _weights(M, "normal", (8, 256 // M)), M // 2, 0.1, 500
    flags = b.TSENOR_FLAG_TILES_LARGE if tiles == "large" else b.TSENOR_FLAG_TILES_SMALL
    for tol in (1e-300, 2.0**-52, 2.0**-50):
        print(f"[case] tolerance below the factors' rounding {N}:{M} {tiles} {tol}", flush=True)
        plan, done = _plan(W, N, M, tau, T, flags, tol)
        print(f"mean {done.mean():.1f}, to the end {(done == T).mean():.3f}", flush=True)
        # (one below 2^-53 is met by factors of exactly 1, which the increments of some blocks do not come down to: 0 to 0.16)
        assert done.mean() < 300 if tol < 2.0**-53 else (done == T).mean() < 0.04


def _seconds(W, N, M, tau, T, flags, tau_mode=1):
    import torch

    from paper_2505_23949_amd import binding as b

    p = b.make_problem(W, N, M, tau, T, mask=torch.zeros(W.shape, dtype=torch.uint8, device=W.device),
                       tau_mode=tau_mode, flags=flags)
    work = torch.empty(b.tsenor_workspace_bytes([p]), dtype=torch.uint8, device=W.device)
    best = float("inf")
    for _ in range(3):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        b.tsenor_mask_ex(p, work)
        end.record()
        torch.cuda.synchronize()
        best = min(best, start.elapsed_time(end))
    return best


def _beside_the_cap(M, rng):
    """A block that converges within dozens of iterations (K = W) to a plan whose first entry is a few 1e-7 below the cap."""
    W = rng.random((M, M)).astype(np.float32)
    low, high = 0.0, 8.0
    for _ in range(60):
        W[0, 0] = 0.5 * (low + high)
        below = 1.0 - np.exp(oracle.dykstra(W, M // 2, M, 1.0, 150)[0, 0])
        if 1e-7 < below < 7e-7:
            return W
        low, high = (low, W[0, 0]) if below < 1e-7 else (W[0, 0], high)
    raise AssertionError("no such weight")


@pytest.mark.parametrize("M,tiles", [(8, "large"), (16, "large"), (16, "small"), (32, "small")])
def test_repeated_states_beside_the_cap(M, tiles):
    # entries so near the cap that the increments are never taken up: the look for them runs an iteration now and then, and states
    # are found to repeat all the same
    import torch

    from paper_2505_23949_amd import binding as b

    # one block everywhere, eight of them in turn: their last bits run through cycles, of which all but a few have a period that the
    # kernels look for, most of them an even one
    rng = np.random.Generator(np.random.Philox(5 + M))
    flags = b.TSENOR_FLAG_TILES_LARGE if tiles == "large" else b.TSENOR_FLAG_TILES_SMALL
    found = 0
    for k in range(8):
        print(f"[case] repeated states beside the cap M={M} {tiles} {k}", flush=True)
        W = torch.from_numpy(np.tile(_beside_the_cap(M, rng), (43, 43))).to("cuda:0")
        short, long = (_seconds(W, M // 2, M, 1.0, T, flags, b.TSENOR_TAU_ABSOLUTE) for T in (1200, 60000))
        found += long < 10 * short
    assert found >= 5, found


def test_increments_end_early():
    # 32 x 32 blocks on the large tiles do not look for repeated states: 60 000 iterations are over after some thousands of steps
    import torch

    from paper_2505_23949_amd import binding as b

    W = torch.from_numpy(np.tile(np.random.Generator(np.random.Philox(7)).random((32, 32)), (33, 33)).astype(np.float32)).to("cuda:0")
    print("[case] increments end early", flush=True)
    short, long = (_seconds(W, 16, 32, 1.0, T, b.TSENOR_FLAG_TILES_LARGE) for T in (1200, 60000))
    assert long < 10 * short, (short, long)
