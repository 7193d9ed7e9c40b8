"""GPU parity of compressed passes over lists whose buffers lie in arenas, which find a chunk without its tensor's
descriptor, against the same list with buffers that lie anywhere: bit for bit, for every kernel that has both forms."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2106_10796_amd import binding, build
    build.ensure_built()
    binding.lib()
    assert torch.cuda.is_available()
    return binding


KEYS = ("w_global", "w_local", "residual", "packed_self")


def _pair(B, sizes, N, rank, t, dtype, align=1024, extra=0):
    """Plans over the same values: one list in arenas (gaps filled with a sentinel), one with every buffer on its own."""
    at, total = [], 0
    for n in sizes:
        at.append(total)
        total += (n + align - 1) // align * align + extra
    gen = torch.Generator(device="cuda").manual_seed(sum(sizes) + N)
    f32 = lambda s: torch.empty(total, device="cuda").normal_(0, s, generator=gen)
    arena = dict(w_global=f32(1.0), w_local=f32(1.0), residual=f32(0.4 * t), grad=f32(t).to(dtype),
                 packed_self=torch.full((total // 16,), 77, dtype=torch.int32, device="cuda"))
    streams = [torch.randint(-2 ** 31, 2 ** 31, (total // 16,), dtype=torch.int32, device="cuda", generator=gen) for _ in range(N)]
    cut = lambda k, v: [v[o // 16: o // 16 + B.packed_words(n)] if k in ("packed_self", "peer") else v[o: o + n]
                        for o, n in zip(at, sizes)]
    parts = {k: cut(k, v) for k, v in arena.items()}
    mine = [{k: parts[k][i] for k in parts} for i in range(len(sizes))]
    ref = [{k: v.clone() for k, v in d.items()} for d in mine]
    peers = [None if j == rank else cut("peer", s) for j, s in enumerate(streams)] if N > 1 else None
    apart = None if peers is None else [None if p is None else [x.clone() for x in p] for p in peers]
    gaps = {k: torch.ones(arena[k].numel(), dtype=torch.bool, device="cuda") for k in KEYS}
    for k in KEYS:
        for x in parts[k]:
            o = x.storage_offset()
            gaps[k][o: o + x.numel()] = False
    before = {k: arena[k].clone() for k in KEYS}

    def check(where):
        torch.cuda.synchronize()
        for i in range(len(sizes)):
            for k in KEYS:
                assert torch.equal(mine[i][k].view(torch.int32), ref[i][k].view(torch.int32)), "%s: %s of tensor %d" % (where, k, i)
        for k in KEYS:
            assert torch.equal(arena[k][gaps[k]].view(torch.int32), before[k][gaps[k]].view(torch.int32)), "%s: %s between tensors" % (where, k)
    return (B.Plan(mine, peers, N, rank, grad_dtype=dtype), B.Plan(ref, apart, N, rank, grad_dtype=dtype), mine, peers, check)


RAGGED = [1, 4096, 17, 4095, 4097, 1024, 1027, 12288, 15, 16, 8191, 3 * 4096 + 1025, 64, 250]


@pytest.mark.parametrize("t", [0.5, 0.3])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("N", [1, 2, 4, 5, 8, 9, 13, 16, 17, 24, 29, 32, 33])
def test_ragged_list_in_arenas(B, N, dtype, t):
    a, b, mine, peers, check = _pair(B, RAGGED, N, N // 2, t, dtype, align=64 if N % 2 else 1024)
    for plan in (a, b):
        plan.step(1, 4, t, 0.4, 0.7)
    check("whole")
    for first, count in ((9, 5), (3, 6), (0, 3)):
        for plan in (a, b):
            plan.step_range(first, count, 2, 4, t, 0.4, 0.7)
    check("ranges")
    own = [float(x) for x in 2.0 ** np.arange(-6, len(RAGGED) - 6)]
    for plan in (a, b):
        plan.set_thresholds(own)
        plan.step(1, 4, t, 0.4, 0.7)
        plan.set_thresholds(None)
    check("thresholds of their own")
    for plan in (a, b):
        plan.set_max_workgroups(3)
        plan.step(3, 4, t, 0.4, 0.7)
        plan.set_max_workgroups(0)
    check("workgroup limit")
    B.cdsgd_step_fused_static(mine, peers, N, N // 2, 1, 4, t, 0.4, 0.7, grad_dtype=dtype)
    b.step(1, 4, t, 0.4, 0.7)
    check("static")


# lists of more than 6, 16 and 28 times 2^20 elements have launch shapes of their own, and the longest no arenas
@pytest.mark.parametrize("N,t,dtype", [(4, 0.3, torch.bfloat16), (8, 0.5, torch.float32), (16, 0.5, torch.float32),
                                       (16, 0.3, torch.float16), (12, 0.5, torch.bfloat16)])
@pytest.mark.parametrize("n", [6_400_000, 17_000_000, 29_500_000])
def test_long_lists_in_arenas(B, N, t, dtype, n):
    sizes = [n // 3 + 5, 77, n // 3 + 4097, 4096, n // 3 - 9]
    a, b, mine, peers, check = _pair(B, sizes, N, N - 1, t, dtype, extra=64)
    for plan in (a, b):
        plan.step(1, 4, t, 0.4, 0.7)
    check("whole")
    B.cdsgd_step_fused_static(mine, peers, N, N - 1, 1, 4, t, 0.4, 0.7, grad_dtype=dtype)
    b.step(1, 4, t, 0.4, 0.7)
    check("static")


# 256 tensors fit the arguments of one launch; above 32 workers that form ends at 16 M elements
@pytest.mark.parametrize("T,N,t,dtype", [(2, 3, 0.5, torch.float32), (255, 8, 0.3, torch.bfloat16), (256, 16, 0.5, torch.float16),
                                         (256, 33, 0.3, torch.float32), (257, 9, 0.5, torch.float32), (256, 64, 0.25, torch.float32)])
def test_static_lists_at_the_edge_of_one_launch(B, T, N, t, dtype):
    rng = np.random.default_rng(T + N)
    sizes = [int(x) for x in 2.0 ** rng.uniform(0, 13.5, T)]
    a, b, mine, peers, check = _pair(B, sizes, N, N // 2, t, dtype, align=64)
    B.cdsgd_step_fused_static(mine, peers, N, N // 2, 1, 4, t, 0.4, 0.7, grad_dtype=dtype)
    b.step(1, 4, t, 0.4, 0.7)
    check("static")


@pytest.mark.parametrize("n", [16 * 1024 * 1024 - 5000, 16 * 1024 * 1024 + 8192])
@pytest.mark.parametrize("N,t", [(20, 0.5), (24, 0.3), (36, 0.5), (36, 0.3)])
def test_static_list_of_many_workers(B, n, N, t):
    a, b, mine, peers, check = _pair(B, [n - 70_001, 4097, 60_000], N, 3, t, torch.bfloat16)
    B.cdsgd_step_fused_static(mine, peers, N, 3, 1, 4, t, 0.4, 0.7, grad_dtype=torch.bfloat16)
    b.step(1, 4, t, 0.4, 0.7)
    check("static")


# sparse peers of 17 to 32 workers have kernels of their own, but for long lists of 32-bit gradients
@pytest.mark.parametrize("t", [0.5, 0.3])
@pytest.mark.parametrize("N,sizes,dtype", [(17, RAGGED, torch.float32), (24, RAGGED, torch.float16), (32, RAGGED, torch.bfloat16),
                                           (20, [29_500_000, 77, 4097], torch.float32),
                                           (20, [29_500_000, 77, 4097], torch.bfloat16)])
def test_sparse_peers_equal_packed_ones(B, N, sizes, dtype, t):
    a, b, mine, peers, check = _pair(B, sizes, N, 5, t, dtype)

    def encode(stream, n):
        out = B.new_sparse(n)
        B.cdsgd_sparse_encode(stream, n, out)
        return out
    encoded = [None if p is None else [encode(x, n) for x, n in zip(p, sizes)] for p in peers]
    sparse = B.Plan(mine, encoded, N, 5, grad_dtype=dtype, peers_sparse=True)
    sparse.step(1, 4, t, 0.4, 0.7)
    b.step(1, 4, t, 0.4, 0.7)
    check("sparse")


# sparse peers: passes over more than 16 M elements (17 to 32 workers: 28 M, 16-bit gradients) have kernels of their own
@pytest.mark.parametrize("N,tiles,dtype,t", [(6, 16384, torch.float32, 0.3), (8, 16384, torch.bfloat16, 0.5), (9, 16384, torch.float16, 0.3),
                                             (16, 16384, torch.float32, 0.5), (18, 28 * 1024, torch.float16, 0.3)])
def test_sparse_peers_on_either_side_of_six_groups(B, N, tiles, dtype, t):
    for more in (0, 1):
        test_sparse_peers_equal_packed_ones(B, N, [tiles * 1024 - 4096 - 1, 4096 + more], dtype, t)


# up to 8 workers, a limit of at most half the list's tiles: a kernel of its own (56 tiles: 14 chunks)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("N,t", [(1, 0.5), (2, 0.3), (4, 0.5), (4, 0.3), (5, 0.3), (8, 0.5), (8, 0.3)])
def test_few_groups_walk_the_list(B, N, t, dtype):
    limited, b, _, _, check = _pair(B, [40 * 1024 - 3, 1, 8192 + 5], N, N // 2, t, dtype)
    for limit in (1, 3, 28, 29):
        limited.set_max_workgroups(limit)
        for plan in (limited, b):
            plan.step(1, 4, t, 0.4, 0.7)
            plan.step_global(3, 4, t, 0.7)
        check("N=%d limit=%d" % (N, limit))
