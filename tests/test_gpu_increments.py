"""The last iterations in double, done in increments: the plan is that of the log-domain oracle after T iterations."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# The factors of an iteration carry 2^-48 and an entry of the plan what its block's convergence makes of them: up to 1e-12 with and
# without increments (those add 2^-24 of changes below 2^-30).
PLAN_ATOL = 1e-11


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


def _plan(W, N, M, tau, T, flags, tol=0.0):
    import torch

    from paper_2505_23949_amd import binding as b

    got = b.solve(torch.from_numpy(W).to("cuda:0"), N, M, tau, T, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, flags=flags, tol=tol, want_plan=True,
                  want_iters_done=tol > 0.0)
    torch.cuda.synchronize()
    return got["plan"].cpu().numpy(), got["iters_done"].cpu().numpy() if tol > 0.0 else None


@pytest.mark.parametrize("M,tiles", [(8, "large"), (16, "large"), (32, "large"), (16, "small"), (32, "small")])
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


@pytest.mark.parametrize("M", [8, 16])
def test_increments_of_many_iterations(M):
    # slow blocks: the increments' sum passes its bound, and the plan they act on is formed anew
    from paper_2505_23949_amd import binding as b

    W, N, tau, T = _weights(M, "normal", (2, 64 // M)), M // 2, 0.02, 30000
    te = oracle.tau_eff(np.abs(W), tau, oracle.TAU_REL_MATRIX_MAX)
    print(f"[case] increments of many iterations {N}:{M}", flush=True)
    ref = np.exp(oracle.dykstra(np.abs(W), N, M, te, T))
    plan, _ = _plan(W, N, M, tau, T, b.TSENOR_FLAG_TILES_LARGE)
    assert np.abs(plan - ref).max() < 1e-9


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


@pytest.mark.parametrize("M", [8, 16, 32])
def test_tolerance_met_in_increments(M):
    # a tolerance far below where they begin, and far above the rounding of the factors: the count is the oracle's
    from paper_2505_23949_amd import binding as b

    W, N, tau, T, tol = _weights(M, "student", (3, 64 // M * 2)), M // 2, 0.05, 600, 1e-12
    te = oracle.tau_eff(np.abs(W), tau, oracle.TAU_REL_MATRIX_MAX)
    print(f"[case] tolerance met in increments {N}:{M}", flush=True)
    log_S, done_ref = oracle.dykstra_adaptive(np.abs(W), N, M, te, T, tol)
    plan, done = _plan(W, N, M, tau, T, b.TSENOR_FLAG_TILES_LARGE, tol)
    # (factors at the tolerance carry 4e-15 and the increments 1e-7 of themselves: one look earlier or later)
    assert np.abs(done.reshape(-1) - done_ref.reshape(-1)).max() <= b.TSENOR_ADAPTIVE_CHECK_EVERY
    assert (done < T).any()
    assert np.abs(plan - np.exp(log_S)).max() < PLAN_ATOL


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
        W = torch.from_numpy(np.tile(_beside_the_cap(M, rng), (33, 33))).to("cuda:0")
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
