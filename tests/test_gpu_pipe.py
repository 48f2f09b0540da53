"""The pipelined chain sweeps (dmm_pipe.h) against the one-wave chain kernels: the same
operations in the same order, so every output is the same bit for bit (tolerance 0).

One-wave references.  Half-steps: a forward that records its checkpoints
(keep_checkpoints=2).  Final pass: the frame repeated downwards until its rows are more than
the pipelines that fit the chip.  Messages by scans (T > 3): batched plans.
Label counts at the edges of the pipelined tiles and of whole-lane vectors, chains around a
chunk's length, and enough chains for several workgroups to share a CU."""
import pytest
import torch

pytestmark = pytest.mark.gpu

RESIDENT = 768 * 4  # rows that never fit at once: at most 3 workgroups of 4 rows, or 4 of one, per CU


def _instance(H, W, K, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    # quarter steps: exact ties between candidates and between labels are frequent
    cost = (torch.randint(0, 5, (H, W, K), generator=g) / 4).to(dtype).cuda()
    w_h, w_v = (torch.rand(s, generator=g).cuda() * 0.5 for s in ((H, W - 1), (H - 1, W)))
    return cost, w_h, w_v


def _equal(a, b, names):
    for name, x, y in zip(names, a, b):
        assert torch.equal(x, y), f"{name} differs"


def _compare(H, W, K, T, dtype, minorant="iterative", half=0, seed=0, gammas=(0.25, 0.25, 1.0), final=True):
    from paper_1601_06274_amd import ops
    print(f"[case] {H}x{W}x{K} T={T} {dtype} {minorant} half-steps {half}", flush=True)
    cost, w_h, w_v = _instance(H, W, K, dtype, seed)
    kw = dict(T=T, n_iters=2, n_half_steps=half, minorant=minorant, gammas=gammas)
    r = ops.solve_discrete(cost, w_h, w_v, **kw)
    ref = ops.solve_discrete(cost, w_h, w_v, keep_checkpoints=2, **kw)
    torch.cuda.synchronize()
    _equal((r.dual, r.bounds[:1]), (ref.dual, ref.bounds[:1]), ("dual", "lower bound"))
    # a plan of this frame and of a smaller one
    kw["tile"] = ops.tile_for(K)
    small = [x.contiguous() for x in (cost[: H // 2 + 1], w_h[: H // 2 + 1], w_v[: H // 2])]
    want = ops.solve_discrete(*small, **kw)
    plan = ops.BatchedPlan([dict(cost=c, w_h=h, w_v=v) for c, h, v in ((cost, w_h, w_v), small)], want_minmarg=True,
                           **kw)
    try:
        plan.run()
        torch.cuda.synchronize()
        for got, one in zip(plan.instances, (r, want)):
            _equal([got[k] for k in ("dual", "minmarg", "labels")], (one.dual, one.minmarg, one.labels),
                   ("plan dual", "plan min-marginals", "plan labels"))
            assert got["bounds"][0].item() == one.bounds[0].item()
    finally:
        plan.close()
    if final and minorant == "iterative":
        n = RESIDENT // H + 1
        many = ops.solve_discrete(cost.repeat(n, 1, 1), w_h.repeat(n, 1), torch.zeros((n * H - 1, W), device="cuda"),
                                  T=T, n_iters=0, dual=r.dual.repeat(n, 1, 1), warm_start=True)
        torch.cuda.synchronize()
        _equal((r.minmarg, r.labels), (many.minmarg[:H], many.labels[:H]), ("min-marginals", "labels"))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("K", [5, 16, 17, 32, 33, 63, 64, 65, 66, 72, 100, 127, 128, 129, 130, 132, 191, 192, 193, 196, 255, 256])
def test_label_counts(K, dtype):
    _compare(13, 22, K, 3, dtype, seed=K)


@pytest.mark.parametrize("H,W", [(1, 1), (1, 9), (9, 1), (2, 3), (3, 2), (4, 8), (5, 7), (16, 17), (31, 33), (12, 95)])
@pytest.mark.parametrize("K", [40, 128, 150])
def test_chain_lengths(H, W, K):
    _compare(H, W, K, 3, torch.float32, seed=H * W, final=False)
    _compare(H, W, K, 2, torch.float16, half=3, seed=H + W, final=W < 20)


@pytest.mark.parametrize("K", [24, 100, 192])
def test_options(K):
    _compare(11, 30, K, 1, torch.float32, final=False)
    _compare(11, 30, K, 3, torch.float16, minorant="naive")
    _compare(11, 30, K, 3, torch.float32, gammas=(1.0,), final=False)
    _compare(11, 30, K, 3, torch.float32, gammas=(0.5, 0.25, 0.25, 0.5, 1.0), final=False)


@pytest.mark.parametrize("K", [64, 128, 192, 256])
def test_many_chains(K):
    """Two and more workgroups per CU (rows and columns)."""
    _compare(600, 61, K, 3, torch.float16, seed=K)
    _compare(61, 600, K, 3, torch.float32, seed=K + 1, final=False)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("T", [4, 6, 9, 40])
@pytest.mark.parametrize("K", [17, 30, 32, 50, 64, 90, 96, 100, 126, 128, 150, 192, 212, 256])
def test_scans(K, T, dtype):
    from paper_1601_06274_amd import ops
    for H, W in ((13, 22), (530, 9)) if T == 6 else ((7, 11),):
        print(f"[case] {H}x{W}x{K} T={T} {dtype}", flush=True)
        cost, w_h, w_v = _instance(H, W, K, dtype, K + T)
        kw = dict(T=T, n_iters=2, tile=ops.tile_for(K))
        plan = ops.BatchedPlan([dict(cost=cost, w_h=w_h, w_v=w_v)], want_minmarg=True, **kw)
        try:
            plan.run()
            r = ops.solve_discrete(cost, w_h, w_v, **kw)
            torch.cuda.synchronize()
            ref = plan.instances[0]
            _equal((r.dual, r.minmarg, r.labels), [ref[k] for k in ("dual", "minmarg", "labels")],
                   ("dual", "min-marginals", "labels"))
            assert r.bounds[0].item() == ref["bounds"][0].item()
        finally:
            plan.close()
