"""GPU parity of correction and warm-up passes that sum the workers' gradients in the kernel, where several gradients are asked
for at once (short lists) and where they are not: own gradient first, last, and on either side of a batch of eight, and lists
on either side of the lines, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

from helpers import assert_bits_equal

pytestmark = pytest.mark.gpu

LR_LOCAL, LR_GLOBAL, TILE = 0.4, 0.7, 1024


@pytest.fixture(scope="module")
def B():
    from paper_2106_10796_amd import binding, build
    build.ensure_built()
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def _check(B, oracle, sizes, N, rank, dtype, modes, limit=0):
    rng = np.random.default_rng(N * 100 + rank)
    # (sums of such values depend on their order)
    draw = lambda n: torch.from_numpy((rng.standard_normal(n) * 10.0 ** rng.uniform(-3, 3, n)).astype(np.float32)).to(dtype)
    grads = [[draw(n) for n in sizes] for _ in range(N)]
    dev = [[g.cuda() for g in x] for x in grads]
    w0 = [rng.standard_normal(n, dtype=np.float32) for n in sizes]
    layers = [dict(w_global=torch.from_numpy(w).cuda(), w_local=torch.zeros(n, device="cuda"), residual=torch.zeros(n, device="cuda"),
                   grad=dev[rank][i], packed_self=B.new_packed(n)) for i, (w, n) in enumerate(zip(w0, sizes))]
    idle = [B.new_packed(n) for n in sizes]
    plan = B.Plan(layers, [None if j == rank else idle for j in range(N)], N, rank, grad_dtype=dtype)
    plan.bind_full_grads([None if j == rank else dev[j] for j in range(N)])
    plan.set_max_workgroups(limit)
    host = [[g.float().numpy() for g in x] for x in grads]
    agg = [oracle.full_sum([host[j][i] for j in range(N)]) for i in range(len(sizes))]
    for mode in modes:                       # warm-up passes 0 (global), 1 (with the copy), 2 (local rule); correction
        before = [w.copy() for w in w0]
        if mode < 3:
            plan.step_warmup(mode, 2, LR_LOCAL, LR_GLOBAL)
        else:
            plan.step(0, 4, 0.5, LR_LOCAL, LR_GLOBAL)
        torch.cuda.synchronize()
        for i, n in enumerate(sizes):
            local = np.zeros(n, np.float32)
            oracle.update(w0[i], local, host[rank][i], agg[i], LR_LOCAL, LR_GLOBAL, N)
            what = "N=%d rank=%d n=%d mode=%d" % (N, rank, n, mode)
            assert_bits_equal(layers[i]["w_global"].cpu().numpy(), w0[i], "w_global " + what)
            if mode >= 1:
                assert_bits_equal(layers[i]["w_local"].cpu().numpy(), w0[i] if mode == 1 else local, "w_local " + what)
        assert any((a != b).any() for a, b in zip(before, w0))
    plan.destroy()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("N", [4, 5, 6, 7, 8, 9, 10, 16, 17, 18, 33, 64])
def test_own_gradient_at_every_place(B, oracle, N, dtype):
    for rank in sorted({0, 1, 7, 8, 9, 15, 16, N // 2, N - 2, N - 1} & set(range(N))):
        _check(B, oracle, [5, 1023, 4096 + 258], N, rank, dtype, (0, 1, 2, 3), limit=2 if rank == 1 else 0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,tiles", [(5, 768), (6, 768), (7, 1024), (16, 1024)])
def test_lists_on_either_side_of_the_lines(B, oracle, N, tiles, dtype):
    for more in (0, 1):
        _check(B, oracle, [tiles * TILE - 4096 - 3, 4096 + more], N, N - 2, dtype, (3,))
