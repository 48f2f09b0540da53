"""The pipelined sweeps on chains long enough for the loader's steady state (32 nodes and more at
one label a lane), with one, two and four chains per workgroup, against the one-wave kernels bit
for bit.  Rows of 33 to 60 nodes whose ends share a cache line with the next row's start are
loaded while that start is stored."""
import pytest
import torch

from test_gpu_pipe import _compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
@pytest.mark.parametrize("K", [5, 7, 8, 12, 15, 16, 17, 20, 31, 32, 33, 48, 63])
def test_steady_state(K, dtype):
    for H, W in ((37, 45), (34, 57), (9, 33), (50, 32), (70, 103)):
        _compare(H, W, K, 3, dtype, seed=K + W)
    _compare(41, 47, K, 3, dtype, minorant="naive", seed=K)
    _compare(47, 41, K, 2, dtype, half=3, seed=K, final=False)


@pytest.mark.parametrize("K", [5, 16, 20, 32, 61])
def test_steady_state_many_chains(K):
    """Several workgroups a CU."""
    _compare(1100, 43, K, 3, torch.float32, seed=K, final=False)
    _compare(37, 1100, K, 3, torch.float16, seed=K, final=False)
