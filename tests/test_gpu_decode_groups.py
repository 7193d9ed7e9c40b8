"""GPU parity of decode-and-sum at the edges of its groups (4, 2 or 1 tiles of 1024 elements, by the number of workers)
and of the batches of workers it is compiled for (4, 8, 16, 32), packed and sparse streams, count and chain form and the
chain of thresholds whose half is not exact: bit for bit against the oracle, and on tensors long enough for the
chunk-wise order against the call on their parts."""
import numpy as np
import pytest
import torch

from helpers import ODD_TINY, assert_bits_equal

pytestmark = pytest.mark.gpu

SIZES = [3, 1024, 2 * 1024 - 1, 2 * 1024 + 17, 3 * 1024 + 5, 4 * 1024, 4 * 1024 + 1, 6 * 1024 + 2, 33 * 4096 + 2 * 1024 + 1]


@pytest.fixture(scope="module")
def B():
    from paper_2106_10796_amd import binding, build
    build.ensure_built()
    binding.lib()
    assert torch.cuda.is_available()
    return binding


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("t", [0.25, 0.3, *ODD_TINY])
@pytest.mark.parametrize("N", [1, 3, 4, 5, 8, 9, 16, 17, 20, 31, 32, 33, 64])
def test_decode_sum_at_group_and_batch_edges(B, oracle, N, t, sparse):
    rng = np.random.default_rng(41 * N + int(sparse))
    for n in SIZES:
        streams = [oracle.pack(rng.choice(4, size=n, p=[0.5, 0.25, 0.2, 0.05]).astype(np.uint8)) for _ in range(N)]
        if N > 2:
            streams[N // 2][:] = 0                       # a worker that sends nothing
        want = oracle.decode_sum(streams, n, t)
        if sparse:
            given = [oracle.sparse_encode(w, n, fill=0x7F7F7F7F)[0] for w in streams]
        else:
            given = [np.concatenate([np.zeros(1, np.uint32), w]) for w in streams]   # 4-byte alignment and no more
        given = [torch.from_numpy(w.view(np.int32)).cuda() for w in given]
        if not sparse:
            given = [w[1:] for w in given]
        out = torch.full((n + 16,), 9.0, device="cuda")
        (B.cdsgd_decode_sum_sparse if sparse else B.cdsgd_decode_sum)(given, out[:n], t)
        torch.cuda.synchronize()
        assert_bits_equal(out[:n].cpu().numpy(), want, "agg N=%d n=%d t=%g sparse=%d" % (N, n, t, sparse))
        assert bool((out[n:] == 9.0).all()), "written past the end: N=%d n=%d" % (N, n)


@pytest.mark.parametrize("t", [0.25, 0.3])
@pytest.mark.parametrize("N", [2, 20, 40])
def test_decode_sum_of_a_long_tensor_equals_its_parts(B, N, t):
    n = (28 << 20) + 5 * 4096 + 1024 + 77
    gen = torch.Generator(device="cuda").manual_seed(N)
    streams = [torch.randint(-2 ** 31, 2 ** 31, (B.packed_words(n),), dtype=torch.int32, device="cuda", generator=gen)
               for _ in range(N)]
    whole, part = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    B.cdsgd_decode_sum(streams, whole, t)
    step = 4096 * 517
    for a in range(0, n, step):
        b = min(n, a + step)
        B.cdsgd_decode_sum([s[a // 16: a // 16 + B.packed_words(b - a)] for s in streams], part[a:b], t)
    torch.cuda.synchronize()
    assert torch.equal(whole.view(torch.int32), part.view(torch.int32))
