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
