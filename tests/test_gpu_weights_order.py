"""Compressed passes over lists in arenas around the lengths between which the weights are asked for behind the other streams,
against the same lists with buffers that lie anywhere, whose kernels ask for all at once: bit for bit.  (Lists of
17 to 32 workers against the oracle: test_gpu_dispatch_lines.py.  Longer lists of more workers against their parts: test_gpu_cache_policies.py.)"""
import pytest
import torch

from test_gpu_arenas import B, _pair  # noqa: F401  (B is the fixture)

pytestmark = pytest.mark.gpu

TILE = 1024


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("N,t,tiles", [(17, 0.5, 2048), (32, 0.3, 2048), (24, 0.5, 16384), (20, 0.3, 16384)])
def test_lists_on_either_side_of_the_lines(B, N, t, tiles, dtype):
    for more in (0, 1):
        # whole tiles, a ragged tensor in the middle, and one chunk more above the line
        sizes = [(tiles // 2 - 8) * TILE, 4 * TILE - 3, 1, (tiles - tiles // 2) * TILE + more * 4096]
        a, b, _, _, check = _pair(B, sizes, N, N - 1, t, dtype)
        for plan in (a, b):
            plan.step(1, 4, t, 0.4, 0.7)
            plan.step_global(3, 4, t, 0.7)           # without the local rule
        check("N=%d tiles=%d more=%d" % (N, tiles, more))
        a.destroy()
        b.destroy()
