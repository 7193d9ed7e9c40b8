"""GPU parity of the compressed pass on lists long enough for the launch shapes of long lists (one-wave groups up to 8
workers, workers' words behind the tile's own streams, bounded residency), beside tensors with every kind of ragged
end, with 32- and 16-bit gradients, whole and split, with and without a workgroup limit (groups that walk several tiles
and use their LDS again).  Bit for bit against the oracle: the small tensors whole, the long one at its ends and inside."""
import numpy as np
import pytest
import torch

from helpers import assert_bits_equal

pytestmark = pytest.mark.gpu

SMALL = [1, 5, 16, 255, 257, 1023, 1024, 1025, 2048 + 15, 4096, 4096 + 1024 + 3, 3 * 4096 + 256]
LONG = (1 << 24) + 4096 * 3 + 277
LR_LOCAL, LR_GLOBAL = 0.4, 0.7


@pytest.fixture(scope="module")
def B():
    from paper_2106_10796_amd import binding, build
    build.ensure_built()
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def _blocks(n):
    """What of a tensor is compared: all of a small one, both ends and an edge of a chunk inside a long one."""
    if n <= 1 << 16:
        return [(0, n)]
    mid, last = n // 2 // 4096 * 4096, n // 4096 * 4096 - 4096
    return [(0, 8192 + 48), (mid - 1024, mid + 5120), (last, n)]


def _check(B, oracle, long_n, N, rank, dtype, runs):
    sizes = SMALL[:6] + [long_n] + SMALL[6:]
    gen = torch.Generator(device="cuda").manual_seed(1000 * N + rank)
    streams = [[torch.randint(-2 ** 31, 2 ** 31, (B.packed_words(n),), dtype=torch.int32, device="cuda", generator=gen)
                for n in sizes] for _ in range(N)]
    for t in (0.5, 0.3):
        rand = lambda n, s: torch.empty(n, device="cuda").normal_(0, s, generator=gen)
        start = [dict(w_global=rand(n, 1.0), residual=rand(n, 0.5 * t), grad=rand(n, t).to(dtype)) for n in sizes]
        want = []
        for i, n in enumerate(sizes):
            parts = []
            for a, b in _blocks(n):
                cut = lambda x: x[a:b].float().cpu().numpy()
                g, r, w = cut(start[i]["grad"]), cut(start[i]["residual"]), cut(start[i]["w_global"])
                loc = np.zeros_like(w)
                words = [streams[j][i][a // 16: a // 16 + B.packed_words(b - a)].cpu().numpy().view(np.uint32).copy()
                         for j in range(N)]
                words[rank] = oracle.quantize_pack(g, r, t)
                oracle.update(w, loc, g, oracle.decode_sum(words, b - a, t), LR_LOCAL, LR_GLOBAL, N)
                parts.append((a, b, dict(residual=r, w_global=w, w_local=loc), words[rank]))
            want.append(parts)
        for limit, split in runs:
            layers = [dict(w_global=s["w_global"].clone(), residual=s["residual"].clone(), grad=s["grad"],
                           w_local=torch.full((n,), 7.0, device="cuda"), packed_self=torch.full((B.packed_words(n),), -1,
                           dtype=torch.int32, device="cuda")) for s, n in zip(start, sizes)]
            plan = B.Plan(layers, [None if j == rank else streams[j] for j in range(N)], N, rank, grad_dtype=dtype)
            plan.set_max_workgroups(limit)
            if split:
                plan.step_local(LR_LOCAL)
                plan.step_global(1, 4, t, LR_GLOBAL)
            else:
                plan.step(1, 4, t, LR_LOCAL, LR_GLOBAL)
            torch.cuda.synchronize()
            for i, n in enumerate(sizes):
                for a, b, bufs, own in want[i]:
                    what = "N=%d self=%d t=%g limit=%d split=%d n=%d [%d, %d)" % (N, rank, t, limit, split, n, a, b)
                    for key, ref in bufs.items():
                        assert_bits_equal(layers[i][key][a:b].cpu().numpy(), ref, "%s %s" % (key, what))
                    got = layers[i]["packed_self"][a // 16: a // 16 + own.size].cpu().numpy()
                    assert_bits_equal(got, own.view(np.int32), "packed_self " + what)
            plan.destroy()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("N,rank", [(2, 0), (2, 1), (5, 2), (7, 6), (8, 0), (8, 7), (9, 4), (16, 15), (20, 3)])
def test_long_and_ragged_tensors_in_one_list(B, oracle, N, rank, dtype):
    _check(B, oracle, LONG, N, rank, dtype, [(0, False), (0, True), (300, False), (4096, True)])


@pytest.mark.parametrize("N,rank,dtype", [(3, 1, torch.float32), (6, 5, torch.bfloat16), (11, 0, torch.float32),
                                          (13, 12, torch.float16)])
def test_longest_launch_shapes(B, oracle, N, rank, dtype):
    _check(B, oracle, (81 << 20) + 1024 + 9, N, rank, dtype, [(0, False), (2500, False)])
