"""GPU parity of the compressed pass's chain of adds with the own worker at every kind of place among the others: the own codes
make a row of their own between the workers' rows, and a group that walks several tiles uses the same rows again.  Bit for bit
against the oracle, sums that depend on their order."""
import numpy as np
import pytest
import torch

from helpers import ODD_TINY, assert_bits_equal

pytestmark = pytest.mark.gpu

SIZES = [3 * 1024 + 5, 4096, 17, 2 * 4096 + 1023]
LR_LOCAL, LR_GLOBAL = 0.4, 0.7


@pytest.fixture(scope="module")
def B():
    from paper_2106_10796_amd import binding, build
    build.ensure_built()
    binding.lib()
    assert torch.cuda.is_available()
    return binding


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("t", [0.3, ODD_TINY[3]])
@pytest.mark.parametrize("N", [5, 8, 9, 16, 17, 32, 33, 48, 49, 64])
def test_own_worker_at_every_kind_of_place(B, oracle, N, t, sparse):
    rng = np.random.default_rng(N)
    words = [[oracle.pack(rng.choice(4, size=n, p=[0.4, 0.3, 0.25, 0.05]).astype(np.uint8)) for n in SIZES] for _ in range(N)]
    on_gpu = lambda w, n: torch.from_numpy((oracle.sparse_encode(w, n)[0] if sparse else w).view(np.int32)).cuda()
    given = [[on_gpu(w, n) for w, n in zip(x, SIZES)] for x in words]
    for rank in sorted({0, 3, 4, 15, 16, 31, 32, 47, 48, N // 2, N - 1} & set(range(N))):
        host = [dict(w_global=rng.standard_normal(n, dtype=np.float32), w_local=np.zeros(n, np.float32),
                     residual=rng.standard_normal(n, dtype=np.float32) * np.float32(t),
                     grad=rng.standard_normal(n, dtype=np.float32) * np.float32(t)) for n in SIZES]
        layers = [dict({k: torch.from_numpy(v).cuda() for k, v in x.items()}, packed_self=B.new_packed(n)) for x, n in zip(host, SIZES)]
        plan = B.Plan(layers, [None if j == rank else given[j] for j in range(N)], N, rank, peers_sparse=sparse)
        for limit in (0, 2):
            plan.set_max_workgroups(limit)
            plan.step(1, 4, t, LR_LOCAL, LR_GLOBAL)
            torch.cuda.synchronize()
            for i, (x, n) in enumerate(zip(host, SIZES)):
                own = oracle.quantize_pack(x["grad"], x["residual"], t)
                agg = oracle.decode_sum([own if j == rank else words[j][i] for j in range(N)], n, t)
                oracle.update(x["w_global"], x["w_local"], x["grad"], agg, LR_LOCAL, LR_GLOBAL, N)
                for key, ref in (("packed_self", own.view(np.int32)), *((k, x[k]) for k in ("residual", "w_global", "w_local"))):
                    assert_bits_equal(layers[i][key].cpu().numpy(), ref, "%s N=%d self=%d n=%d limit=%d" % (key, N, rank, n, limit))
        plan.destroy()
