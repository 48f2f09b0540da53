"""Batched plans of many chains on tiles that K fills, where the rule (pipe_plan_serves) leaves
the pipelines for the one-wave queue, by one family or by both: every instance bit for bit its
single-instance solve, whatever kernels either runs (tolerance 0)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("minorant", ["iterative", "naive"])
@pytest.mark.parametrize("n,H,W,K", [(60, 40, 30, 64), (30, 200, 36, 64), (30, 36, 200, 64), (160, 40, 30, 32), (90, 40, 38, 128)])
def test_many_short_chains(n, H, W, K, minorant):
    from paper_1601_06274_amd import ops
    print(f"[case] {n} frames of {H}x{W}x{K} {minorant}", flush=True)
    g = torch.Generator().manual_seed(K + n)
    insts = []
    for i in range(n):
        h, w = H + i % 3, W + i % 2
        # quarter steps: exact ties between candidates and between labels are frequent
        insts.append(dict(cost=(torch.randint(0, 5, (h, w, K), generator=g) / 4).half().cuda(),
                          w_h=torch.rand((h, w - 1), generator=g).cuda() * 0.5,
                          w_v=torch.rand((h - 1, w), generator=g).cuda() * 0.5))
    kw = dict(T=3, n_iters=2, minorant=minorant)
    plan = ops.BatchedPlan(insts, want_minmarg=True, **kw)
    try:
        for _ in range(2):
            plan.run()
            torch.cuda.synchronize()
            for i in (0, 1, n // 2, n - 1):
                one = ops.solve_discrete(insts[i]["cost"], insts[i]["w_h"], insts[i]["w_v"], **kw)
                torch.cuda.synchronize()
                got = plan.instances[i]
                for name in ("dual", "minmarg", "labels"):
                    assert torch.equal(got[name], getattr(one, name)), f"instance {i}: {name}"
                assert got["bounds"][0].item() == one.bounds[0].item()
    finally:
        plan.close()
