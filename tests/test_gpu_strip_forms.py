"""Forms of the strip kernels (sad_strip.h) and the Census kernel that the other tests leave out,
bit for bit (tolerance 0): the same sums in the same order whatever kernel or vector width."""
import pytest
import torch

from test_gpu_sad_strips import _bands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("window,K", [(5, 33), (5, 64), (5, 201), (5, 256), (7, 34), (7, 99), (7, 200)])
def test_wide_windows_many_labels(window, K, dtype):
    from paper_1601_06274_amd import ops
    g = torch.Generator().manual_seed(K)
    H, W = 1203, 129  # 903 strips; the bands of 61 rows are the row kernel's
    print(f"[case] {H}x{W}x{K} window {window} {dtype}", flush=True)
    left, right = (torch.rand((H, W), generator=g).cuda() for _ in range(2))
    kw = dict(window=window, trunc=0.4, dtype=dtype)
    got = ops.build_cost_volume(left, right, K, **kw)
    want = _bands(left, right, K, **kw)
    torch.cuda.synchronize()
    for name, x, y in zip(("cost", "w_h", "w_v"), got, want):
        assert torch.equal(x, y), f"{name} differs"


@pytest.mark.parametrize("window", [1, 3, 5])
@pytest.mark.parametrize("K1,K2", [(64, 5), (31, 13), (17, 15), (48, 3), (3, 64)])
def test_flow_small_frames(K1, K2, window):
    """Frames of few strips, whose blocks take fewer labels j, against the rows of a tall frame."""
    from paper_1601_06274_amd import ops
    H, W, R = 1100, 70, window // 2
    print(f"[case] flow {K1}x{K2} window {window}", flush=True)
    g = torch.Generator().manual_seed(K1)
    I1, I2 = (torch.rand((H, W), generator=g).cuda() for _ in range(2))
    kw = dict(window=window, trunc=0.4, dtype=torch.float16)
    got = ops.build_flow_cost_volume(I1, I2, K1, K2, K1 // 2, K2 // 2, **kw)
    halo = R + K2  # the rows of both images that a row's costs reach
    for y in (0, 301, H - 9):
        a, b = max(y - halo, 0), min(y + 9 + halo, H)
        want = ops.build_flow_cost_volume(I1[a:b].contiguous(), I2[a:b].contiguous(), K1, K2, K1 // 2, K2 // 2, **kw)
        torch.cuda.synchronize()
        assert torch.equal(got[0][y:y + 9], want[0][y - a:y - a + 9]), f"cost differs at row {y}"
        assert torch.equal(got[1][y:y + 9], want[1][y - a:y - a + 9])
        assert torch.equal(got[2][y:y + 8], want[2][y - a:y - a + 8])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("offset", [1, 2, 3])
def test_unaligned_outputs(offset, dtype):
    """Volumes that start at any element: the vector width follows the pointer's alignment, and
    nothing beside the volume is written."""
    from paper_1601_06274_amd import ops
    g = torch.Generator().manual_seed(offset)

    def compare(build, shape, what):
        n = shape[0] * shape[1] * shape[2] * (shape[3] if len(shape) == 4 else 1)
        print(f"[case] {what} {shape} {dtype} offset {offset}", flush=True)
        pool = torch.full((n + 16,), 7.0, dtype=dtype, device="cuda")
        out = pool[offset:offset + n].view(shape)
        want = build(dtype=dtype)[0]
        build(cost_out=out, dtype=dtype)
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"{what} differs"
        assert (pool[:offset] == 7.0).all() and (pool[offset + n:] == 7.0).all(), f"{what}: written beside the volume"

    H, W = 905, 129
    left, right = (torch.rand((H, W), generator=g).cuda() for _ in range(2))
    for window, K in ((1, 64), (3, 64), (3, 66), (5, 32), (7, 16)):  # strips
        compare(lambda **kw: ops.build_cost_volume(left, right, K, window=window, **kw), (H, W, K), f"sad {window}")
    a, b = left[:40].contiguous(), right[:40].contiguous()
    for window in (3, 5, 7):
        for view in ("left", "right"):
            compare(lambda **kw: ops.build_cost_volume_census(a, b, 64, window=window, view=view, **kw), (40, W, 64),
                    f"census {window} {view}")
    for window in (1, 3, 5):
        compare(lambda **kw: ops.build_flow_cost_volume(a, b, 16, 9, 8, 4, window=window, **kw), (40, W, 9, 16),
                f"flow {window}")
