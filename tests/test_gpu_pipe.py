"""The pipelined chain sweeps (dmm_pipe.h) against the one-wave kernels that batched plans run:
the same operations in the same order, so every output is the same bit for bit (tolerance 0).
Label counts at the edges of the pipelined tiles, chains around a chunk's length, and enough
chains for several workgroups to share a CU."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _instance(H, W, K, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    # quarter steps: exact ties between candidates and between labels are frequent
    cost = (torch.randint(0, 5, (H, W, K), generator=g) / 4).to(dtype).cuda()
    w_h, w_v = (torch.rand(s, generator=g).cuda() * 0.5 for s in ((H, W - 1), (H - 1, W)))
    return cost, w_h, w_v


def _compare(H, W, K, T, dtype, minorant="iterative", half=0, seed=0, gammas=(0.25, 0.25, 1.0)):
    from paper_1601_06274_amd import ops
    print(f"[case] {H}x{W}x{K} T={T} {dtype} {minorant} half-steps {half}", flush=True)
    g = torch.Generator().manual_seed(seed)
    # quarter steps: exact ties between candidates and between labels are frequent
    cost = (torch.randint(0, 5, (H, W, K), generator=g) / 4).to(dtype).cuda()
    w_h, w_v = (torch.rand(s, generator=g).cuda() * 0.5 for s in ((H, W - 1), (H - 1, W)))
    kw = dict(T=T, n_iters=2, n_half_steps=half, minorant=minorant, gammas=gammas, tile=ops.tile_for(K))
    plan = ops.BatchedPlan([dict(cost=cost, w_h=w_h, w_v=w_v)], want_minmarg=True, **kw)
    try:
        plan.run()
        r = ops.solve_discrete(cost, w_h, w_v, **{**kw, "tile": None})
        torch.cuda.synchronize()
        ref = plan.instances[0]
        for name in ("dual", "minmarg", "labels"):
            assert torch.equal(getattr(r, name), ref[name]), f"{name} differs"
        assert r.bounds[0].item() == ref["bounds"][0].item()
    finally:
        plan.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("K", [5, 16, 17, 32, 33, 63, 64, 65, 66, 127, 128, 129, 191, 192, 193, 255, 256])
def test_label_counts(K, dtype):
    _compare(13, 22, K, 3, dtype, seed=K)


@pytest.mark.parametrize("H,W", [(1, 1), (1, 9), (9, 1), (2, 3), (3, 2), (4, 8), (5, 7), (16, 17), (31, 33), (12, 95)])
@pytest.mark.parametrize("K", [40, 128, 150])
def test_chain_lengths(H, W, K):
    _compare(H, W, K, 3, torch.float32, seed=H * W)
    _compare(H, W, K, 2, torch.float16, half=3, seed=H + W)


@pytest.mark.parametrize("K", [24, 100, 192])
def test_options(K):
    _compare(11, 30, K, 1, torch.float32)
    _compare(11, 30, K, 3, torch.float16, minorant="naive")
    _compare(11, 30, K, 3, torch.float32, gammas=(1.0,))
    _compare(11, 30, K, 3, torch.float32, gammas=(0.5, 0.25, 0.25, 0.5, 1.0))


@pytest.mark.parametrize("K", [64, 128, 192, 256])
def test_many_chains(K):
    """Two and more workgroups per CU (rows and columns)."""
    _compare(600, 61, K, 3, torch.float16, seed=K)
    _compare(61, 600, K, 3, torch.float32, seed=K + 1)


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
            for name in ("dual", "minmarg", "labels"):
                assert torch.equal(getattr(r, name), ref[name]), f"{name} differs"
            assert r.bounds[0].item() == ref["bounds"][0].item()
        finally:
            plan.close()
