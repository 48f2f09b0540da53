"""The linearisation's adjoint (linearize_adjoint_kernel) where its six entries of a pixel's
labels coincide or leave the range: steps h below, at and above one label, few labels.  The
projections of the gradient against the oracle's directional derivatives, within the bound of
the other refinement gradients."""
import numpy as np
import pytest
import torch

import synth
from oracle import grad as ograd
from oracle import refine as oref

pytestmark = pytest.mark.gpu

REL = 1e-4  # FP32 gradients of FP64 arithmetic, relative to the projection's terms


@pytest.mark.parametrize("h", [0.5, 1.0, 2.0])
@pytest.mark.parametrize("K", [3, 4, 6, 9])
def test_refine_grad_steps(K, h):
    from paper_1601_06274_amd import ops
    H, W, seed = 6, 7, 11 * K
    print(f"[case] refine grad K={K} h={h}", flush=True)
    theta, w_h, w_v = synth.tiny_instance(H, W, K, seed=seed, w_max=0.5)
    dev = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda() for x in (theta, w_h, w_v)]
    th64, wh64, wv64 = (x.cpu().numpy().astype(np.float64) for x in dev)
    labels = np.random.default_rng(seed).integers(1, K - 1, (H, W))
    Gu = np.random.default_rng(seed + 7).normal(size=(H, W)).astype(np.float32)
    kw = dict(C=2.0, h=h, n_warps=2, n_iters=7)
    ws = torch.empty(ops.refine_workspace_bytes((H, W, K), keep_tape=True, **kw), dtype=torch.uint8, device="cuda")
    ops.refine_continuous(dev[0], torch.from_numpy(labels.astype(np.int32)).cuda(), dev[1], dev[2], workspace=ws,
                          keep_tape=True, **kw)
    got = ops.refine_continuous_backward(torch.from_numpy(Gu).cuda(), *dev, ws, **kw)
    torch.cuda.synchronize()
    got = [x.cpu().numpy().astype(np.float64) for x in got]
    P = oref.RefineParams(tau=float(np.float32(0.3)), sigma=float(np.float32(0.3)), **kw)
    for d in range(3):
        g = np.random.default_rng(1000 * seed + d)
        dirs = [g.normal(size=x.shape) for x in (theta, w_h, w_v)]
        _, ud = ograd.refine_continuous_jvp(th64, dirs[0], wh64, dirs[1], wv64, dirs[2], labels, P)
        ref = float((Gu.astype(np.float64) * ud).sum())
        terms = np.concatenate([(a * b).ravel() for a, b in zip(got, dirs)])
        assert abs(terms.sum() - ref) <= REL * np.abs(terms).sum()
