"""GPU parity of decode-and-sum on either side of the sizes where the cache policy of its loads changes, and behind a ragged
end there: bit for bit against the call on parts that are short enough for the other policy."""
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


# elements x workers / 4 bytes of streams: above 28 MB (56 MB up to eight workers) they are read non-temporally
@pytest.mark.parametrize("t", [0.25, 0.3, 1.1e-38])
@pytest.mark.parametrize("N,n", [(4, 57_000_013), (7, 33_000_001), (16, 7_100_005), (17, 6_600_007), (64, 1_800_001)])
def test_decode_sum_of_many_streams_equals_its_parts(B, N, n, t):
    gen = torch.Generator(device="cuda").manual_seed(N)
    streams = [torch.randint(-2 ** 31, 2 ** 31, (B.packed_words(n),), dtype=torch.int32, device="cuda", generator=gen)
               for _ in range(N)]
    whole, part = torch.full((n + 8,), 9.0, device="cuda"), torch.zeros(n, device="cuda")
    B.cdsgd_decode_sum(streams, whole[:n], t)
    step = 4096 * 401
    for a in range(0, n, step):
        b = min(n, a + step)
        B.cdsgd_decode_sum([s[a // 16: a // 16 + B.packed_words(b - a)] for s in streams], part[a:b], t)
    torch.cuda.synchronize()
    assert torch.equal(whole[:n].view(torch.int32), part.view(torch.int32))
    assert bool((whole[n:] == 9.0).all()), "written past the end"
