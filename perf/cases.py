"""Performance cases of the matching path: what a user of this library has it do.

A case is a dict of plain values; ``op`` names the public call or calls that it times:

  sad        build_cost_volume of a stereo pair
  census     build_cost_volume_census of both views of a pair
  solve      solve_discrete on a cost volume (any minorant, truncation and cost type)
  grad       solve_discrete and solve_discrete_backward (a training step's discrete stage, tapes kept)
  refine     refine_continuous_ad forward and backward
  two_view   the two-view pipeline: Census volumes, solves, refinements, left-right check
  flow_cost  build_flow_cost_volume of an image pair
  flow       solve_flow: layer projections, both layers' solves, quadratic-fit refinement
  batched    BatchedPlan over uneven instances (the plan is kept, each pass replays it)

Inputs are synthetic stereo / flow pairs (random texture, piecewise-planar disparities,
sensor noise) drawn on the GPU from the seed.
"""
import math

import torch
import torch.nn.functional as F

import paper_1601_06274_amd as dm
from paper_1601_06274_amd import autograd, ops

DEV = "cuda"
REFINE = dict(C=3.0, n_warps=5, n_iters=40)
GAMMAS = (0.25, 0.25, 1.0)


def listed():
    return [
        # the smallest solve: a thumbnail frame, FP32; latency and launch count
        {"name": "solve_thumb", "op": "solve", "W": 128, "H": 96, "K": 32, "dtype": "f32", "T": 3, "n_iters": 10,
         "minorant": "iterative"},
        # the live-camera setting: 640x480, 128 disparities, 4 dual iterations
        {"name": "solve_vga", "op": "solve", "W": 640, "H": 480, "K": 128, "dtype": "f32", "T": 3, "n_iters": 4,
         "minorant": "iterative"},
        # a driving-scene frame at the solver's default iteration count, FP16 cost
        {"name": "solve_drive", "op": "solve", "W": 1242, "H": 375, "K": 192, "dtype": "f16", "T": 3, "n_iters": 10,
         "minorant": "iterative"},
        # a crop with a label range that fits no power of two, wider truncation (scan messages)
        {"name": "solve_crop", "op": "solve", "W": 611, "H": 437, "K": 100, "dtype": "f32", "T": 6, "n_iters": 4,
         "minorant": "iterative"},
        # the hierarchical minorant on the live-camera frame
        {"name": "solve_hier", "op": "solve", "W": 640, "H": 480, "K": 128, "dtype": "f16", "T": 3, "n_iters": 4,
         "minorant": "hierarchical"},
        # the discrete stage of a training step on the driving-scene frame (largest case)
        {"name": "grad_drive", "op": "grad", "W": 1242, "H": 375, "K": 192, "dtype": "f16", "T": 3, "n_iters": 20,
         "minorant": "iterative"},
        # refinement of that frame, forward and backward
        {"name": "refine_drive", "op": "refine", "W": 1242, "H": 375, "K": 192, "dtype": "f16"},
        # the data term of that frame
        {"name": "sad_drive", "op": "sad", "W": 1242, "H": 375, "K": 192, "dtype": "f16", "window": 3},
        # the paper's data term, both views, at the frame's odd size
        {"name": "census_drive", "op": "census", "W": 1242, "H": 375, "K": 192, "dtype": "f16", "window": 5},
        # two-view stereo of a small frame, end to end
        {"name": "two_view", "op": "two_view", "W": 320, "H": 240, "K": 64, "dtype": "f16", "T": 3, "n_iters": 10},
        # optical flow: the two-dimensional data term and the pipeline on it
        {"name": "flow_vga", "op": "flow_cost", "W": 640, "H": 480, "K1": 32, "K2": 32, "dtype": "f16", "window": 3},
        # uneven instances in one plan: serving several cameras at once
        {"name": "batched", "op": "batched", "n": 6, "W": 640, "H": 360, "K": 128, "dtype": "f16", "T": 3,
         "n_iters": 4},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    op = rng.choice(["solve", "solve", "solve", "solve", "grad", "grad", "refine", "sad", "census", "two_view",
                     "flow_cost", "flow", "batched"])
    c = {"op": op, "W": _log(rng, 96, 1280), "H": _log(rng, 72, 480), "dtype": rng.choice(["f16", "f32"])}
    if op in ("flow_cost", "flow"):
        c["W"], c["H"] = _log(rng, 96, 640), _log(rng, 72, 480)
        c["K1"], c["K2"] = rng.randint(9, 32), rng.randint(9, 32)
        if op == "flow_cost":
            c["window"] = rng.choice([1, 3, 3, 5])
        else:
            c["T"], c["n_iters"] = 3, rng.choice([4, 10])
        return c
    # half of the label ranges are those that rigs are configured with, half are any
    c["K"] = rng.choice([32, 48, 64, 96, 128, 192, 256]) if rng.random() < 0.5 else _log(rng, 12, 240)
    if op in ("solve", "grad"):
        c["T"] = rng.choice([1, 2, 3, 3, 3, 3, 5, 8])
        c["n_iters"] = rng.choice([2, 4, 4, 8])
        c["minorant"] = rng.choice(["iterative"] * 6 + (["naive"] if op == "grad" else ["naive", "hierarchical"]))
    elif op == "sad":
        c["window"] = rng.choice([3, 3, 5])
    elif op == "census":
        c["window"] = rng.choice([3, 5, 5, 7])
    elif op == "two_view":
        c["W"], c["H"], c["K"] = min(c["W"], 640), min(c["H"], 360), min(c["K"], 128)
        c["T"], c["n_iters"] = 3, rng.choice([4, 10])
    elif op == "batched":
        c["W"], c["H"], c["K"] = min(c["W"], 640), min(c["H"], 360), min(c["K"], 128)
        c["n"], c["T"], c["n_iters"] = rng.randint(2, 8), 3, rng.choice([2, 4])
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) % (1 << 62))


def _texture(W, H, g):
    img = torch.rand((1, 1, H, W), generator=g, device=DEV, dtype=torch.float64)
    img = F.avg_pool2d(F.pad(img, (1, 1, 1, 1), mode="replicate"), 3, 1)[0, 0]
    return (img - img.min()) / (img.max() - img.min())


def _planes(W, H, lo, hi, slope, g):
    """Piecewise-planar field: a Voronoi partition into planes with values around U[lo, hi]."""
    n = max(4, round(W * H / 20000.0))
    cx = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * W
    cy = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * H
    d0 = lo + (hi - lo) * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    a = slope * (2 * torch.rand(n, generator=g, device=DEV, dtype=torch.float64) - 1)
    b = slope * (2 * torch.rand(n, generator=g, device=DEV, dtype=torch.float64) - 1)
    ys = torch.arange(H, device=DEV, dtype=torch.float64)[:, None, None]
    xs = torch.arange(W, device=DEV, dtype=torch.float64)[None, :, None]
    seg = ((xs - cx) ** 2 + (ys - cy) ** 2).argmin(-1)
    return d0[seg] + a[seg] * (xs[:, :, 0] - cx[seg]) + b[seg] * (ys[:, :, 0] - cy[seg])


def _noisy(img, g):
    return (img + (2.0 / 255.0) * torch.randn(img.shape, generator=g, device=DEV, dtype=torch.float64)).clamp(0, 1)


def _stereo(W, H, K, g):
    """(left, right, disparity): I_R(x', y) = I_L(x' + d(x', y), y) plus noise."""
    left = _texture(W, H, g)
    disp = _planes(W, H, 0.1 * K, 0.8 * K, 0.08, g).clamp(0, K - 1)
    src = (torch.arange(W, device=DEV, dtype=torch.float64) + disp).clamp(0, W - 1)
    x0 = src.floor().long()
    t = src - x0
    right = (1 - t) * left.gather(1, x0) + t * left.gather(1, (x0 + 1).clamp(max=W - 1))
    return left.float().contiguous(), _noisy(right, g).float().contiguous(), disp


def _flow_images(W, H, K1, K2, g):
    """I2(p) = I1(p - u(p)), |u| below a third of the label range, plus noise."""
    I1 = _texture(W, H, g)
    u1 = _planes(W, H, -K1 / 3, K1 / 3, 0.02, g)
    u2 = _planes(W, H, -K2 / 3, K2 / 3, 0.02, g)
    xs = torch.arange(W, device=DEV, dtype=torch.float64)[None, :] - u1
    ys = torch.arange(H, device=DEV, dtype=torch.float64)[:, None] - u2
    grid = torch.stack((2 * xs / max(W - 1, 1) - 1, 2 * ys / max(H - 1, 1) - 1), -1)
    I2 = F.grid_sample(I1[None, None], grid[None], padding_mode="border", align_corners=True)[0, 0]
    return I1.float().contiguous(), _noisy(I2, g).float().contiguous()


def _dtype(c):
    return torch.float16 if c["dtype"] == "f16" else torch.float32


def _batch_shapes(c):
    """Uneven instances around the case's size: each camera has its own frame and label range."""
    return [(max(32, c["W"] * (6 - i % 4) // 6), max(24, c["H"] * (5 - i % 3) // 5), max(8, c["K"] * (4 - i % 3) // 4))
            for i in range(c["n"])]


def _volume(W, H, K, dtype, g):
    left, right, disp = _stereo(W, H, K, g)
    return dm.build_cost_volume(left, right, K, dtype=dtype) + (disp,)


def prepare(case, seed):
    c, g, op = case, _gen(seed), case["op"]
    W, H, dtype = c["W"], c["H"], _dtype(c)
    if op in ("sad", "census", "two_view"):
        left, right, _ = _stereo(W, H, c["K"], g)
        return dict(case=c, left=left, right=right)
    if op == "flow_cost":
        I1, I2 = _flow_images(W, H, c["K1"], c["K2"], g)
        return dict(case=c, I1=I1, I2=I2)
    if op == "flow":
        I1, I2 = _flow_images(W, H, c["K1"], c["K2"], g)
        cost, w_h, w_v = dm.build_flow_cost_volume(I1, I2, c["K1"], c["K2"], c["K1"] // 2, c["K2"] // 2, dtype=dtype)
        return dict(case=c, cost=cost, w_h=w_h, w_v=w_v)
    if op == "batched":
        inst = []
        for w, h, k in _batch_shapes(c):
            cost, w_h, w_v, _ = _volume(w, h, k, dtype, g)
            inst.append(dict(cost=cost, w_h=w_h, w_v=w_v))
        plan = ops.BatchedPlan(inst, T=c["T"], n_iters=c["n_iters"], refine=dict(C=float(c["T"]), n_warps=5, n_iters=40),
                               want_minmarg=True)
        return dict(case=c, plan=plan)
    cost, w_h, w_v, disp = _volume(W, H, c["K"], dtype, g)
    s = dict(case=c, cost=cost, w_h=w_h, w_v=w_v)
    if op == "refine":
        s["labels"] = disp.round().clamp(0, c["K"] - 1).to(torch.int32)
        s["g_u"] = torch.randn((H, W), generator=g, device=DEV)
    if op == "grad":
        s["g_mm"] = torch.randn((H, W, c["K"]), generator=g, device=DEV)
        s["g_b"] = torch.tensor([1.0, 0.0], dtype=torch.float64, device=DEV)  # dL/dLB, dL/dE
    if op == "refine":
        for k in ("cost", "w_h", "w_v"):
            s[k].requires_grad_(True)
    return s


# ------------------------------------------------------------------ one pass
def _solve(cost, w_h, w_v, c, **kw):
    return dm.solve_discrete(cost, w_h, w_v, T=c["T"], n_iters=c["n_iters"], minorant=c.get("minorant", "iterative"),
                             **kw)


def run(state):
    s, c = state, state["case"]
    op, dtype = c["op"], _dtype(c)
    if op == "sad":
        return dm.build_cost_volume(s["left"], s["right"], c["K"], window=c["window"], dtype=dtype)
    if op == "census":
        return [dm.build_cost_volume_census(s["left"], s["right"], c["K"], window=c["window"], view=v, dtype=dtype)
                for v in ("left", "right")]
    if op == "solve":
        r = _solve(s["cost"], s["w_h"], s["w_v"], c)
        return {"minmarg": r.minmarg, "dual": r.dual, "bounds": r.bounds, "labels": r.labels}
    if op == "grad":
        # the workspace with the tapes (tens of GB on the largest frame) is kept from step to step
        r = _solve(s["cost"], s["w_h"], s["w_v"], c, keep_checkpoints=2, workspace=s.get("ws"))
        s["ws"] = r.workspace
        grads = ops.solve_discrete_backward(s["cost"], s["w_h"], s["w_v"], r.dual, r.workspace, grad_minmarg=s["g_mm"],
                                            grad_bounds=s["g_b"], T=c["T"], n_iters=c["n_iters"],
                                            minorant=c["minorant"], keep_checkpoints=2)
        return {"minmarg": r.minmarg, "dual": r.dual, "bounds": r.bounds, "labels": r.labels, "grads": grads}
    if op == "refine":
        ins = (s["cost"], s["w_h"], s["w_v"])
        u = autograd.refine_continuous_ad(s["cost"], s["labels"], s["w_h"], s["w_v"], **REFINE)
        return {"u": u, "grads": torch.autograd.grad(u, ins, s["g_u"])}
    if op == "two_view":
        out, us = {}, []
        for v in ("left", "right"):
            cost, w_h, w_v = dm.build_cost_volume_census(s["left"], s["right"], c["K"], view=v, dtype=dtype)
            r = _solve(cost, w_h, w_v, c)
            us.append(dm.refine_continuous(cost, r.labels, w_h, w_v, **REFINE))
            out[v] = {"minmarg": r.minmarg, "labels": r.labels, "u": us[-1]}
        out["checked"] = dm.lr_check(us[0], us[1])
        return out
    if op == "flow_cost":
        return dm.build_flow_cost_volume(s["I1"], s["I2"], c["K1"], c["K2"], c["K1"] // 2, c["K2"] // 2,
                                         window=c["window"], dtype=dtype)
    if op == "flow":
        r = dm.solve_flow(s["cost"], s["w_h"], s["w_v"], off1=c["K1"] // 2, off2=c["K2"] // 2, T=c["T"],
                          n_iters=c["n_iters"])
        return {"f": [r.f1, r.f2], "minmarg": [r.layer1.minmarg, r.layer2.minmarg],
                "labels": [r.layer1.labels, r.layer2.labels], "u": [r.u1, r.u2]}
    s["plan"].run()
    return [{k: d[k] for k in ("minmarg", "dual", "bounds", "labels", "u")} for d in s["plan"].instances]


# ------------------------------------------------------------------ what a pass cannot do without
def _solve_work(W, H, K, c, b):
    n, T = W * H * K, c["T"]
    naive = c.get("minorant") == "naive"
    updates = (4 if naive else 8) * c["n_iters"] + 2
    if c.get("minorant") == "hierarchical":
        updates = 2 * c["n_iters"] * (2 + 0.5 * math.log2(max(2, W)) + 3) + 2
    # per label and node: two sums, two minima, the message's window (an add and a min per
    # candidate, at most the T - 1 of an envelope scan each way) and the update
    return {"bytes": n * (b + 8.0) + W * H * 12.0, "flops": n * updates * (8.0 + 4.0 * min(T, 3))}


def work(case):
    c, op = case, case["op"]
    W, H, b = c["W"], c["H"], 2.0 if c["dtype"] == "f16" else 4.0
    px = W * H
    if op == "flow_cost":
        return {"bytes": px * (8.0 + 8.0 + b * c["K1"] * c["K2"]), "flops": px * c["K1"] * c["K2"] * 12.0}
    if op == "flow":
        w1, w2 = (_solve_work(W, H, c[k], c, b) for k in ("K1", "K2"))
        return {"bytes": px * (b * c["K1"] * c["K2"] + 8.0 + (b + 4.0) * (c["K1"] + c["K2"]) + 16.0),
                "flops": w1["flops"] + w2["flops"] + px * 2.0 * (c["K1"] * c["K2"] + 200 * 50)}
    if op == "batched":
        ws = [_solve_work(w, h, k, c, b) for w, h, k in _batch_shapes(c)]
        pxs = sum(w * h for w, h, _ in _batch_shapes(c))
        return {"bytes": sum(w["bytes"] for w in ws) + 4.0 * pxs, "flops": sum(w["flops"] for w in ws) + pxs * 200 * 50.0}
    n = px * c["K"]
    if op == "sad":
        return {"bytes": px * 16.0 + n * b, "flops": n * 12.0}
    if op == "census":
        return {"bytes": 2 * (px * 16.0 + n * b), "flops": 2 * n * 4.0}
    if op == "solve":
        return _solve_work(W, H, c["K"], c, b)
    if op == "grad":
        w = _solve_work(W, H, c["K"], c, b)
        # cost and the min-marginals' gradient in, min-marginals and the cost's gradient out;
        # the backward visits every label-node as often as the forward
        return {"bytes": n * (2 * b + 8.0) + px * 20.0, "flops": 2 * w["flops"]}
    if op == "refine":
        # the volume is read at five labels of every pixel and warp only; its gradient is dense
        return {"bytes": n * b + px * (5 * 5 * b + 4 * 7.0), "flops": px * 200 * 2 * 50.0}
    if op == "two_view":
        w = _solve_work(W, H, c["K"], c, b)
        return {"bytes": px * 32.0 + 2 * n * 4.0, "flops": 2 * (w["flops"] + n * 4.0 + px * 200 * 50.0)}
    raise ValueError(op)


# ------------------------------------------------------------------ the same in 64 bits
def _weights64(I):
    I = I.double()
    return 0.1 * torch.exp(-(I[:, 1:] - I[:, :-1]).abs() / 0.1), 0.1 * torch.exp(-(I[1:] - I[:-1]).abs() / 0.1)


def _window_mean(e, window, trunc):
    """Mean over the window, clamped to the image, of e [..., H, W], truncated."""
    H, W = e.shape[-2:]
    r = window // 2
    p = F.pad(e.reshape(-1, 1, H, W), (r, r, r, r), mode="replicate")[:, 0]
    acc = torch.zeros_like(p[:, :H, :W])
    for dy in range(window):
        for dx in range(window):
            acc += p[:, dy:dy + H, dx:dx + W]
    return (acc / (window * window)).clamp(max=trunc).reshape(e.shape)


def _sad64(L, R, K, window, trunc=0.3):
    L, R = L.double(), R.double()
    H, W = L.shape
    out = torch.empty((H, W, K), dtype=torch.float64, device=DEV)
    for d in range(K):
        e = torch.full((H, W), trunc, dtype=torch.float64, device=DEV)
        if d < W:
            e[:, d:] = (L[:, d:] - R[:, :W - d]).abs()
        out[:, :, d] = _window_mean(e, window, trunc)
    return out


def _flow_cost64(I1, I2, K1, K2, window, trunc=0.3):
    A, B = I1.double(), I2.double()
    H, W = A.shape
    out = torch.empty((H, W, K2, K1), dtype=torch.float64, device=DEV)
    pad = max(K1, K2)
    Bp = F.pad(B[None, None], (pad, pad, pad, pad), value=float("inf"))[0, 0]
    for j in range(K2):
        for i in range(K1):
            dy, dx = pad + j - K2 // 2, pad + i - K1 // 2
            b = Bp[dy:dy + H, dx:dx + W]
            e = torch.where(torch.isinf(b), torch.full_like(A, trunc), (A - b).abs())
            out[:, :, j, i] = _window_mean(e, window, trunc)
    return out


def _census64(L, R, K, window, view):
    H, W = L.shape
    r = window // 2

    def bits(I):
        p = F.pad(I[None, None], (r, r, r, r), mode="replicate")[0, 0]
        return torch.stack([p[dy:dy + H, dx:dx + W] < I for dy in range(window) for dx in range(window)
                            if dy != r or dx != r], -1)

    bl, br = bits(L), bits(R)
    n = bl.shape[-1]
    out = torch.ones((H, W, K), dtype=torch.float64, device=DEV)
    for d in range(min(K, W)):
        ham = (bl[:, d:] != br[:, :W - d]).sum(-1).double() / n
        if view == "left":
            out[:, d:, d] = ham
        else:
            out[:, :W - d, d] = ham
    return out


def _message(v, w, T):
    """min over labels a of v(a) + w min(|a - b|, T), minus min v; v [..., K], w [..., 1]."""
    K = v.shape[-1]
    vmin = v.amin(-1, keepdim=True)
    out = torch.minimum(v, vmin + w * T)
    if T > 1:
        p = F.pad(v, (T - 1, T - 1), value=float("inf"))
        for d in range(1, T):
            near = torch.minimum(p[..., T - 1 - d:T - 1 - d + K], p[..., T - 1 + d:T - 1 + d + K])
            out = torch.minimum(out, near + w * d)
    return out - vmin


def _backward_messages(r, w, T):
    R = torch.zeros_like(r)
    for j in range(r.shape[1] - 2, -1, -1):
        R[:, j] = _message(R[:, j + 1] + r[:, j + 1], w[:, j], T)
    return R


def _min_marginals(r, w, T):
    R = _backward_messages(r, w, T)
    m = torch.empty_like(r)
    carry = torch.zeros_like(r[:, 0])
    n = r.shape[1]
    for j in range(n):
        v = r[:, j] + carry
        m[:, j] = v + R[:, j]
        if j + 1 < n:
            carry = _message(v, w[:, j], T)
    return m


def _iterative(a, w, T):
    r = a.clone()
    msg = _backward_messages(r, w, T)
    n = r.shape[1]
    for s, gamma in enumerate(GAMMAS):
        carry = torch.zeros_like(r[:, 0])
        for j in (range(n) if s % 2 == 0 else range(n - 1, -1, -1)):
            m = r[:, j] + carry + msg[:, j]
            r[:, j] -= gamma * (m - m.amin(-1, keepdim=True))
            msg[:, j] = carry
            last = n - 1 if s % 2 == 0 else 0
            if j != last:
                carry = _message(r[:, j] + carry, w[:, j if s % 2 == 0 else j - 1], T)
    return a - r


def _split(s, e):
    return s + (e - s + 1) // 2 - 1


def _hierarchical(a, w, T):
    """Handshake minorant, all parts of one depth at a time."""
    n = a.shape[1]
    L, R = torch.zeros_like(a), torch.zeros_like(a)

    def passes(starts, stops, to, step):
        """Messages from node k to node k + step for k from starts until stops, all parts together."""
        t = 0
        while True:
            k = [s + step * t for s, e in zip(starts, stops) if (e - (s + step * t)) * step > 0]
            if not k:
                return
            k = torch.tensor(k, device=DEV)
            edge = k if step > 0 else k - 1
            to[:, k + step] = _message(to[:, k] + a[:, k], w[:, edge], T)
            t += 1

    if n >= 2:
        i = _split(0, n - 1)
        passes([0], [i], L, 1)
        passes([n - 1], [i + 1], R, -1)
    parts = [(0, n - 1)] if n >= 2 else []
    while parts:
        cut = [_split(s, e) for s, e in parts]
        i = torch.tensor(cut, device=DEV)
        wi = w[:, i]
        back = _message(a[:, i + 1] + R[:, i + 1], wi, T)
        fwd = _message((L[:, i] + a[:, i] + back) / 2 - back, wi, T)
        R[:, i], L[:, i + 1] = _message(-fwd, wi, T), fwd
        left = [(s, m) for (s, e), m in zip(parts, cut) if m > s]
        right = [(m + 1, e) for (s, e), m in zip(parts, cut) if e > m + 1]
        passes([m for s, m in left], [_split(s, m) + 1 for s, m in left], R, -1)
        passes([s for s, e in right], [_split(s, e) for s, e in right], L, 1)
        parts = left + right
    m = a + L + R
    return m - m.amin(-1, keepdim=True)


def _minorant(a, w, T, kind):
    w = w[:, :, None]
    if kind == "hierarchical":
        return _hierarchical(a, w, T)
    if kind == "naive":
        m = _min_marginals(a, w, T)
        return (m - m.amin(-1, keepdim=True)) / a.shape[1]
    return _iterative(a, w, T)


def _solve64(cost, w_h, w_v, T, n_iters, kind="iterative"):
    """(min-marginals, dual, [lower bound, energy], labels) of the discrete solve."""
    th, wh, wv = cost.detach().double(), w_h.detach().double(), w_v.detach().double()
    lam = torch.zeros_like(th)
    for _ in range(n_iters):
        lam = lam + _minorant(th - lam, wh, T, kind)
        lam = lam - _minorant(lam.transpose(0, 1).contiguous(), wv.T.contiguous(), T, kind).transpose(0, 1)
    m = _min_marginals(th - lam, wh[:, :, None], T)
    mm = m - m.amin(-1, keepdim=True)
    labels = mm.argmin(-1)
    bound = _optima(th - lam, wh, T).sum() + _optima(lam.transpose(0, 1).contiguous(), wv.T, T).sum()
    energy = th.gather(2, labels[:, :, None]).sum()
    energy = energy + (wh * (labels[:, 1:] - labels[:, :-1]).abs().clamp(max=T)).sum()
    energy = energy + (wv * (labels[1:] - labels[:-1]).abs().clamp(max=T)).sum()
    return mm, lam, torch.stack((bound, energy)), labels


def _optima(r, w, T):
    """Optimum of every chain, from messages that keep their constants."""
    carry = torch.zeros_like(r[:, 0])
    for j in range(r.shape[1] - 1, 0, -1):
        v = carry + r[:, j]
        carry = _message(v, w[:, j - 1, None], T) + v.amin(-1, keepdim=True)
    return (r[:, 0] + carry).amin(-1)


def _refine64(cost, labels, w_h, w_v, C=3.0, tau=None, h=1.0, n_warps=5, n_iters=40):
    """The warped primal-dual refinement (eps = 1, delta = 0); tau = sigma as the call passes them."""
    tau = float(torch.tensor(0.3, dtype=torch.float32)) if tau is None else tau
    th, wh, wv = cost.detach().double(), w_h.detach().double(), w_v.detach().double()
    H, W, K = th.shape

    def D(v):
        v = v.clamp(0, K - 1)
        k0 = v.floor().long()
        t = v - k0
        k1 = (k0 + 1).clamp(max=K - 1)
        return (1 - t) * th.gather(2, k0[:, :, None])[:, :, 0] + t * th.gather(2, k1[:, :, None])[:, :, 0]

    def conj(t, w, alpha, beta, step):
        a = t.abs()
        t = torch.where(a <= alpha * w, t, torch.maximum(alpha * w, a - beta * step) * t.sign())
        return torch.minimum(torch.maximum(t, -w), w)

    u = labels.double()
    ph, qh, pv, qv = torch.zeros_like(wh), torch.zeros_like(wh), torch.zeros_like(wv), torch.zeros_like(wv)
    for _ in range(n_warps):
        u0 = u
        sL, sR = (D(u0) - D(u0 - h)) / h, (D(u0 + h) - D(u0)) / h
        hl, hr = u0 - h >= 0, u0 + h <= K - 1
        zero = torch.zeros_like(sL)
        sL, sR = torch.where(hl, sL, torch.where(hr, sR, zero)), torch.where(hr, sR, torch.where(hl, sL, zero))
        mean = 0.5 * (sL + sR)
        bad = sL > sR
        sL, sR = torch.where(bad, mean, sL), torch.where(bad, mean, sR)
        lo, hi = (u0 - h).clamp(min=0), (u0 + h).clamp(max=K - 1)
        for _ in range(n_iters):
            yh, yv = ph - qh, pv - qv
            at = F.pad(yh, (0, 1)) - F.pad(yh, (1, 0)) + F.pad(yv, (0, 0, 0, 1)) - F.pad(yv, (0, 0, 1, 0))
            hat = u - tau * at
            new = torch.where(hat > u0 + tau * sR, hat - tau * sR, torch.where(hat < u0 + tau * sL, hat - tau * sL, u0))
            new = torch.minimum(torch.maximum(new, lo), hi)
            qh = conj(qh + tau * (u[:, :-1] - u[:, 1:]), wh, 0.0, C, tau)
            qv = conj(qv + tau * (u[:-1] - u[1:]), wv, 0.0, C, tau)
            b = 2 * new - u
            ph = conj(ph + tau * (b[:, :-1] - b[:, 1:]), wh, 1.0, 0.0, tau)
            pv = conj(pv + tau * (b[:-1] - b[1:]), wv, 1.0, 0.0, tau)
            u = new
    return u


def _steps(W, H, c):
    """Chain steps of a 64-bit solve: what its time goes with."""
    return (W + H) * 4 * c["n_iters"]


def exact(case, seed):
    c, op = case, case["op"]
    W, H = c["W"], c["H"]
    if op == "grad" and _steps(W, H, c) > 90000:
        return None  # minutes in 64 bits
    s = prepare(case, seed)
    if op == "sad":
        return [_sad64(s["left"], s["right"], c["K"], c["window"]), *_weights64(s["left"])]
    if op == "census":
        return [[_census64(s["left"], s["right"], c["K"], c["window"], v), *_weights64(s[v])] for v in ("left", "right")]
    if op == "solve":
        mm, lam, bounds, _ = _solve64(s["cost"], s["w_h"], s["w_v"], c["T"], c["n_iters"], c["minorant"])
        return {"minmarg": mm, "dual": lam, "bounds": bounds, "labels": None}
    if op == "grad":
        # the gradients follow the selections that the minima took: no independent 64-bit value at ties
        mm, lam, bounds, _ = _solve64(s["cost"], s["w_h"], s["w_v"], c["T"], c["n_iters"], c["minorant"])
        return {"minmarg": mm, "dual": lam, "bounds": bounds, "labels": None, "grads": None}
    if op == "refine":
        return {"u": _refine64(s["cost"], s["labels"], s["w_h"], s["w_v"], **REFINE), "grads": None}
    if op == "two_view":
        out = {}
        for v in ("left", "right"):
            cost = _census64(s["left"], s["right"], c["K"], 5, v).to(_dtype(c))  # as it is stored
            mm, _, _, _ = _solve64(cost, *_weights64(s[v]), c["T"], c["n_iters"])
            out[v] = {"minmarg": mm, "labels": None, "u": None}  # u starts from whole-number labels
        out["checked"] = None
        return out
    if op == "flow_cost":
        return [_flow_cost64(s["I1"], s["I2"], c["K1"], c["K2"], c["window"]), *_weights64(s["I1"])]
    if op == "flow":
        f = [s["cost"].double().amin(2), s["cost"].double().amin(3)]
        return {"f": f, "minmarg": [_solve64(x, s["w_h"], s["w_v"], c["T"], c["n_iters"])[0] for x in f],
                "labels": None, "u": None}
    out = []
    for d in s["plan"].instances:
        mm, lam, bounds, _ = _solve64(d["cost"], d["w_h"], d["w_v"], c["T"], c["n_iters"])
        out.append({"minmarg": mm, "dual": lam, "bounds": bounds, "labels": None, "u": None})
    return out
