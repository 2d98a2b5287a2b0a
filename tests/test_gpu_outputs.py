"""The outputs derived from the final mask, on buffers that allow 8-weight accesses and on ones that do not."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _at(torch, dev, shape, dtype, offset):
    """A contiguous tensor `offset` elements into a buffer that is itself 256-byte aligned."""
    n = int(np.prod(shape))
    return torch.zeros(n + offset, dtype=dtype, device=dev)[offset:].view(shape)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M", [4, 8, 16, 32])
def test_derived_outputs_at_every_alignment(M, dtype, offset):
    # offset 1: no buffer is aligned for a wide access.  The previous mask is once worse than any found one (it keeps the
    # lightest weights) and once better (the mask found under its own importance, scored against a found mask of T = 0 with
    # the printed swap rule, which may leave rows short).
    import torch

    from paper_2505_23949_amd import binding as b

    dev = torch.device("cuda:0")
    N, rows, cols = M // 2, 5 * M, 24 * M
    rng = np.random.Generator(np.random.Philox(40 + M))
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    W, V = (_at(torch, dev, (rows, cols), tdt, offset) for _ in range(2))
    W.copy_(torch.from_numpy(rng.standard_normal((rows, cols), dtype=np.float32)))
    V.copy_(torch.from_numpy(0.3 * rng.standard_normal((rows, cols), dtype=np.float32)))
    x = W.float().cpu().numpy() + np.float32(0.5) * V.float().cpu().numpy()
    imp = (np.abs(x) * np.abs(x)).astype(np.float32)
    kw = dict(add=V, add_scale=0.5, importance=b.TSENOR_IMPORTANCE_SQUARE, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX)
    good = b.solve(W, N, M, 0.01, 200, **kw)["mask"]
    for prev_better in (False, True):
        print(f"[case] outputs {M} {dtype} offset={offset} prev_better={prev_better}", flush=True)
        mask, prev, packed, pruned, plain = (_at(torch, dev, (rows, c), t, offset) for c, t in (
            (cols, torch.uint8), (cols, torch.uint8), (cols // 8, torch.uint8), (cols, tdt), (cols, torch.uint8)))
        objective = torch.zeros(2, dtype=torch.float64, device=dev)
        T, flags = (0, b.TSENOR_FLAG_STRICT_PAPER) if prev_better else (200, 0)
        prev.copy_(good if prev_better else torch.from_numpy((imp < np.median(imp)).astype(np.uint8)))
        for prev_mask, out, extra in ((None, plain, {}), (prev, mask, dict(packed_out=packed, pruned_out=pruned, objective_out=objective))):
            p = b.make_problem(W, N, M, 0.01, T, mask=out, prev_mask=prev_mask, flags=flags, **kw, **extra)
            b.tsenor_mask_ex(p, torch.empty(b.tsenor_workspace_bytes([p]), dtype=torch.uint8, device=dev))
        torch.cuda.synchronize()
        mine, theirs = (float((imp.astype(np.float64) * m.cpu().numpy()).sum()) for m in (plain, prev))
        assert (theirs > mine) == prev_better, "the case should decide as it says"
        want = (prev if prev_better else plain).cpu().numpy()
        assert np.array_equal(mask.cpu().numpy(), want)
        assert np.array_equal(packed.cpu().numpy(), np.packbits(want, axis=1, bitorder="little"))
        kept = torch.from_numpy(np.where(want != 0, x, np.float32(0))).to(tdt)
        assert torch.equal(pruned.cpu(), kept)
        # the importance terms are the same numbers on both sides; the two sums of `size` of them differ by their order
        bar = imp.size * 2.0 ** -53
        got = objective.cpu().numpy()
        assert abs(got[0] - max(mine, theirs)) <= bar * got[0] and abs(got[1] - theirs) <= bar * theirs


def test_batch_with_a_matrix_of_one_4_wide_block_column():
    # fused with matrices that ask for derived outputs, a matrix of 4 columns (plain, and with its objective) is what it is
    # in a call of its own
    import torch

    from paper_2505_23949_amd import binding as b

    dev = torch.device("cuda:0")
    rng = np.random.Generator(np.random.Philox(77))
    kw = dict(tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX)
    keep, probs, outs, singles = [], [], [], []
    for cols, want in ((4, ()), (64, ("packed", "pruned")), (4, ("objective",)), (64, ("objective",))):
        W = torch.from_numpy(rng.standard_normal((64, cols), dtype=np.float32)).to(dev)
        print(f"[case] 4-wide batch cols={cols} {want}", flush=True)
        keep.append(W)
        singles.append(b.solve(W, 2, 4, 0.01, 50, **{"want_" + k: True for k in want}, **kw))
        outs.append({k: torch.zeros_like(singles[-1][k]) for k in ("mask",) + want})
        probs.append(b.make_problem(W, 2, 4, 0.01, 50, mask=outs[-1]["mask"], **{k + "_out": outs[-1][k] for k in want}, **kw))
    b.tsenor_mask_batched(probs, torch.empty(b.tsenor_workspace_bytes(probs), dtype=torch.uint8, device=dev))
    torch.cuda.synchronize()
    for out, single in zip(outs, singles):
        for k in out:
            assert torch.equal(out[k], single[k]), k


@pytest.mark.parametrize("blocks", [(1, 1), (32, 32), (25, 41)])
def test_objective_alone_and_with_derived_outputs(blocks):
    # one block, and the two sides of the line (1024 blocks) up to which one workgroup sums the objectives and writes them:
    # the same bits whether the call also has derived outputs or not, alone or fused with the other sizes
    import torch

    import oracle
    from paper_2505_23949_amd import binding as b

    dev, N, M = torch.device("cuda:0"), 3, 8
    rng = np.random.Generator(np.random.Philox(90 + blocks[1]))
    Wf = rng.standard_normal((blocks[0] * M, blocks[1] * M), dtype=np.float32)
    W = torch.from_numpy(Wf).to(dev)
    first = torch.from_numpy((np.add.outer(np.arange(Wf.shape[0]), np.arange(Wf.shape[1])) % M < N).astype(np.uint8)).to(dev)
    print(f"[case] objective of {blocks[0] * blocks[1]} blocks", flush=True)
    kw = dict(tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, want_objective=True)
    alone, packed, safe = b.solve(W, N, M, 0.01, 30, **kw), b.solve(W, N, M, 0.01, 30, want_packed=True, **kw), \
        b.solve(W, N, M, 0.01, 30, prev_mask=first, **kw)
    small = torch.from_numpy(rng.standard_normal((M, 2 * M), dtype=np.float32)).to(dev)
    masks, sums = [torch.empty(x.shape, dtype=torch.uint8, device=dev) for x in (W, small)], torch.zeros((2, 2), dtype=torch.float64, device=dev)
    probs = [b.make_problem(x, N, M, 0.01, 30, mask=m, objective_out=o, tau_mode=b.TSENOR_TAU_REL_MATRIX_MAX, flags=b.TSENOR_FLAG_TILES_LARGE)
             for x, m, o in zip((W, small), masks, sums)]
    b.tsenor_mask_batched(probs, torch.empty(b.tsenor_workspace_bytes(probs), dtype=torch.uint8, device=dev))
    torch.cuda.synchronize()
    imp = np.abs(Wf)
    # the importance terms are the same numbers on both sides; the two sums of `size` of them differ by their order
    bar = imp.size * 2.0 ** -53
    for res, theirs in ((alone, 0.0), (packed, 0.0), (safe, oracle.objective(first.cpu().numpy(), imp, M))):
        want, got = oracle.objective(res["mask"].cpu().numpy(), imp, M), res["objective"].cpu().numpy()
        assert abs(got[0] - want) <= bar * want and abs(got[1] - theirs) <= bar * max(theirs, 1e-300)
    assert torch.equal(alone["objective"], packed["objective"])
    for x, m, o in zip((Wf, small.cpu().numpy()), masks, sums.cpu().numpy()):
        want = oracle.objective(m.cpu().numpy(), np.abs(x), M)
        assert abs(o[0] - want) <= bar * want and o[1] == 0.0
