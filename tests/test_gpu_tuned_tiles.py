"""Tiles that the autotuner picks per truncation: scan messages (T > 3) round by tile, so a plan
and a single solve on the tuned tile are compared on that tile (tolerance 0)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [20, 50, 90, 100, 160])
def test_tuned_tiles_with_scans(K):
    from paper_1601_06274_amd import ops
    H, W = 60, 83
    print(f"[case] tuned tiles {H}x{W}x{K}", flush=True)
    g = torch.Generator().manual_seed(K)
    cost = (torch.randint(0, 5, (H, W, K), generator=g) / 4).half().cuda()
    w_h, w_v = (torch.rand(s, generator=g).cuda() * 0.5 for s in ((H, W - 1), (H - 1, W)))
    for T in (3, 6, 20, 6):
        tiles = ops.autotune_tiles((H, W, K), torch.float16, T=T)
        assert all(a * b >= K for a, b in tiles)
        assert tiles == ops.autotune_tiles((H, W, K), torch.float16, T=T)  # cached
        kw = dict(T=T, n_iters=2, tile=tiles)
        one = ops.solve_discrete(cost, w_h, w_v, **kw)
        ref = ops.solve_discrete(cost, w_h, w_v, keep_checkpoints=2, **kw)  # one wave per chain
        torch.cuda.synchronize()
        assert torch.equal(one.dual, ref.dual) and torch.equal(one.labels, ref.labels)
