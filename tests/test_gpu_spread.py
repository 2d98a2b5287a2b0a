"""Rows whose K spreads over nearly all of the supported 700: the plan agrees with the log-domain oracle as it does elsewhere."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

PLAN_ATOL = 1e-9  # both sides compute in double precision


def _sparse(M, blocks, seed, kind):
    """Importances of exactly 0 and 1 (weights that are zero or of one magnitude): with tau = 1 / spread a row that has both
    holds K = 0 and K = spread.  Every block has a share of ones of its own, or one in every row."""
    rng = np.random.Generator(np.random.Philox(seed))
    W = np.zeros((blocks * M, blocks * M), np.float32)
    for r in range(blocks):
        for c in range(blocks):
            if kind == "one in a row":
                block = np.eye(M, dtype=np.float32)[rng.integers(0, M, M)]
            else:
                block = (rng.random((M, M)) < rng.random()).astype(np.float32)
            W[r * M:(r + 1) * M, c * M:(c + 1) * M] = block
    return W


def _plan(W, N, M, spread, T, flags, tol=0.0):
    import torch

    from paper_2505_23949_amd import binding as b

    got = b.solve(torch.from_numpy(W).to("cuda:0"), N, M, 1.0 / spread, T, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, flags=flags, tol=tol,
                  want_plan=True)
    torch.cuda.synchronize()
    return got["plan"].cpu().numpy()


@pytest.mark.parametrize("kind", ["share of ones", "one in a row"])
@pytest.mark.parametrize("M", [4, 8, 16, 32, 64])
def test_rows_that_spread_over_the_range(M, kind):
    # after T iterations a block is far from convergence, so what its smallest entries were still shows
    from paper_2505_23949_amd import binding as b

    W = _sparse(M, 6, 10 + M, kind)
    for N in sorted({1, M // 2, M - 1}):
        for T in (20, 300):
            for spread in (650.0, 690.0):
                ref = np.exp(oracle.dykstra(W, N, M, oracle.tau_eff(W, 1.0 / spread, oracle.TAU_REL_MATRIX_MAX), T))
                for flags in (0, b.TSENOR_FLAG_TILES_LARGE, b.TSENOR_FLAG_TILES_SMALL):
                    print(f"[case] spread {N}:{M} {kind} T={T} spread={spread} flags={flags}", flush=True)
                    assert np.abs(_plan(W, N, M, spread, T, flags) - ref).max() < PLAN_ATOL


@pytest.mark.parametrize("M,blocks", [(4, 24), (8, 12), (16, 8), (32, 5)])
def test_row_scalings_beyond_a_double(M, blocks):
    # with N = M - 1 the scaling of a row with a single one passes e^710 on its way, and comes back: the kernels that keep their
    # tile (all but the large tiles of 32 x 32 and 64 x 64 blocks) follow it
    from paper_2505_23949_amd import binding as b

    W, N, T, spread = _sparse(M, blocks, 20 + M, "share of ones"), M - 1, 900, 690.0
    ref = np.exp(oracle.dykstra(W, N, M, oracle.tau_eff(W, 1.0 / spread, oracle.TAU_REL_MATRIX_MAX), T))
    for flags in (0, b.TSENOR_FLAG_TILES_SMALL) if M == 32 else (0, b.TSENOR_FLAG_TILES_LARGE, b.TSENOR_FLAG_TILES_SMALL):
        for tol in (0.0, 1e-300):
            print(f"[case] large scalings {N}:{M} flags={flags} tol={tol}", flush=True)
            assert np.abs(_plan(W, N, M, spread, T, flags, tol) - ref).max() < PLAN_ATOL
