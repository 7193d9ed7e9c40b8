"""GPU parity of the single-tensor calls on either side of the sizes where the cache policy of their loads and stores
changes, and of the lanes behind a ragged end there: bit for bit against the oracle (update, quantise-and-pack) and,
for decode-and-sum, against the call on parts that are short enough for the other policy, and against the oracle at the
ends.  Passes over long lists go the same way, against the pass on their parts."""
import numpy as np
import pytest
import torch

from helpers import ODD_TINY, assert_bits_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2106_10796_amd import binding, build
    build.ensure_built()
    binding.lib()
    assert torch.cuda.is_available()
    return binding


SMALL, KEEP = 7 << 20, 24 << 20


def _floats(rng, n, scale):
    return rng.standard_normal(n, dtype=np.float32) * np.float32(scale)


# (five workers' aggregates from 1.25 M to 3.2 M elements are stored non-temporally; weights of the global
# rule of more than four workers do not stay in the memory-side cache above 5 M elements, or 48 MB of streams, 64 workers and 3 M elements)
@pytest.mark.parametrize("n,N", [(1_250_000, 5), (1_250_003, 5), (3_200_000, 5), (3_200_001, 5), (SMALL, 5), (SMALL + 3, 5),
                                 (KEEP, 5), (KEEP + 1, 5), (5_000_000, 5), (5_000_001, 5),
                                 (3_000_000, 64), (3_000_003, 64)])
@pytest.mark.parametrize("mode", ["local", "global", "both"])
def test_update_at_the_edges_of_its_lengths(B, oracle, n, N, mode):
    rng = np.random.default_rng(n + len(mode))
    w, g, a = (_floats(rng, n, s) for s in (1.0, 0.1, 3.0))
    host = {"w": w, "l": np.full(n, 7.0, np.float32), "g": g if mode != "global" else None, "a": a if mode != "local" else None}
    want_w, want_l = w.copy(), (host["l"].copy() if mode != "global" else None)
    oracle.update(want_w, want_l, host["g"], host["a"], 0.05, 0.1, N)
    pad = {k: torch.full((n + 8,), 9.0, device="cuda") for k in ("w", "l")}
    for k in pad:
        pad[k][:n] = torch.from_numpy(host[k]).cuda()
    dev = {k: None if host[k] is None else torch.from_numpy(host[k]).cuda() for k in ("g", "a")}
    B.cdsgd_update(pad["w"][:n], pad["l"][:n] if mode != "global" else None, dev["g"], dev["a"], 0.05, 0.1, N)
    torch.cuda.synchronize()
    assert_bits_equal(pad["w"][:n].cpu().numpy(), want_w, "w_global")
    if mode != "global":
        assert_bits_equal(pad["l"][:n].cpu().numpy(), want_l, "w_local")
    assert all(bool((x[n:] == 9.0).all()) for x in pad.values()), "written past the end"


@pytest.mark.parametrize("n", [SMALL, SMALL + 3, KEEP, KEEP + 1])
def test_quantize_pack_at_the_edges_of_its_lengths(B, oracle, n):
    rng = np.random.default_rng(n)
    t = 0.3
    g, r = _floats(rng, n, 0.3), _floats(rng, n, 0.2)
    want_r = r.copy()
    want_p = oracle.quantize_pack(g, want_r, t)
    pad = torch.full((n + 8,), 9.0, device="cuda")
    pad[:n] = torch.from_numpy(r).cuda()
    packed = torch.full((B.packed_words(n) + 4,), 5, dtype=torch.int32, device="cuda")
    B.cdsgd_quantize_pack(torch.from_numpy(g).cuda(), pad[:n], packed[:B.packed_words(n)], t)
    torch.cuda.synchronize()
    assert_bits_equal(pad[:n].cpu().numpy(), want_r, "residual")
    assert_bits_equal(packed[:B.packed_words(n)].cpu().numpy().view(np.uint32), want_p, "packed")
    assert bool((pad[n:] == 9.0).all()) and bool((packed[B.packed_words(n):] == 5).all()), "written past the end"


# elements x workers / 4 bytes of streams: above 56 MB (100 MB above 16 workers) they are read non-temporally; aggregates from
# 1.25 M elements up to 4.5 M (4 workers), 3.2 M (16) and 1.75 M (32) are stored so, which the parts are too short for
@pytest.mark.parametrize("t", [0.25, 0.3, ODD_TINY[3]])
@pytest.mark.parametrize("N,n", [(4, 57_000_013), (7, 33_000_001), (16, 7_100_005), (17, 6_600_007), (64, 1_800_001),
                                 (1, 4_500_000), (4, 4_500_001), (8, 3_199_999), (16, 3_200_001), (32, 1_750_000), (16, 14_100_005), (17, 23_600_007), (64, 6_300_001)])
def test_decode_sum_of_many_streams_equals_its_parts(B, oracle, N, n, t):
    gen = torch.Generator(device="cuda").manual_seed(N)
    streams = [torch.randint(-2 ** 31, 2 ** 31, (B.packed_words(n),), dtype=torch.int32, device="cuda", generator=gen)
               for _ in range(N)]
    whole, part = torch.full((n + 8,), 9.0, device="cuda"), torch.zeros(n, device="cuda")
    B.cdsgd_decode_sum(streams, whole[:n], t)
    step = 4096 * 303
    for a in range(0, n, step):
        b = min(n, a + step)
        B.cdsgd_decode_sum([s[a // 16: a // 16 + B.packed_words(b - a)] for s in streams], part[a:b], t)
    torch.cuda.synchronize()
    assert torch.equal(whole[:n].view(torch.int32), part.view(torch.int32))
    assert bool((whole[n:] == 9.0).all()), "written past the end"
    for a, b in ((0, 20_000), (n // 16 * 16 - 16_000, n)):
        words = [s[a // 16: a // 16 + B.packed_words(b - a)].cpu().numpy().view(np.uint32) for s in streams]
        assert_bits_equal(whole[a:b].cpu().numpy(), oracle.decode_sum(words, b - a, t), "[%d, %d)" % (a, b))


def _list_state(B, n, N, grad, gen):
    """One tensor's buffers and its peers' streams, in tensors that parts can be cut from."""
    d = dict(device="cuda", generator=gen)
    s = {"w_global": torch.randn(n, **d), "residual": torch.rand(n, **d) - 0.5, "grad": torch.randn(n, **d).to(grad),
         "w_local": torch.zeros(n, device="cuda"),
         "packed_self": torch.zeros(B.packed_words(n), dtype=torch.int32, device="cuda")}
    peers = [torch.randint(-2 ** 31, 2 ** 31, (B.packed_words(n),), dtype=torch.int32, **d) for _ in range(N - 1)]
    return s, peers


def _run_list(B, s, peers, N, grad, a, b, call):
    words = slice(a // 16, a // 16 + B.packed_words(b - a))
    layer = {k: v[words] if k == "packed_self" else v[a:b] for k, v in s.items()}
    plan = B.Plan([layer], [None] + [[p[words]] for p in peers], N, 0, grad_dtype=grad)
    call(plan, a, b)
    torch.cuda.synchronize()
    plan.destroy()


def _whole_equals_parts(B, n, N, grad, step, call):
    gen = torch.Generator(device="cuda").manual_seed(n + N)
    whole, peers = _list_state(B, n, N, grad, gen)
    part = {k: v.clone() for k, v in whole.items()}
    _run_list(B, whole, peers, N, grad, 0, n, call)
    for a in range(0, n, step):
        _run_list(B, part, peers, N, grad, a, min(n, a + step), call)
    for k in ("w_global", "w_local", "residual", "packed_self"):
        assert torch.equal(whole[k].view(torch.int32), part[k].view(torch.int32)), k


# Above 32 workers and 112 MB of streams the workers' words are read non-temporally, and parts of 1.6 M elements are not; results
# of 9 to 16 workers are written through above 1 M elements and of 17 to 32 above 2 M, but for 32-bit chains of 9 to 16 above 48 M
# and 32-bit lists of more than 20 above 28 M.
@pytest.mark.parametrize("t", [0.25, 0.3])
@pytest.mark.parametrize("N,n,grad", [(33, 13_600_003, torch.float32), (64, 7_001_003, torch.bfloat16),
                                      (9, 17_000_013, torch.float32), (16, 51_000_001, torch.float32),
                                      (16, 51_000_001, torch.float16), (20, 29_400_003, torch.float32),
                                      (21, 29_400_003, torch.float32), (32, 29_400_003, torch.bfloat16)])
def test_compressed_pass_equals_its_parts(B, N, n, grad, t):
    _whole_equals_parts(B, n, N, grad, 4096 * 401, lambda p, a, b: p.step(1, 4, t, 0.05, 0.1))


# a correction pass of more than 4 workers writes its results through above 72 * 2^20 elements, one of 4 from 4 to 14 times 2^20;
# parts of 1.6 M elements are stored non-temporally
@pytest.mark.parametrize("N,n,grad", [(4, (14 << 20) - 4097, torch.float32), (3, (4 << 20) + 4097, torch.float16),
                                      (16, (2 << 20) + 5, torch.float32), (5, (72 << 20) + 7, torch.float32)])
def test_correction_pass_equals_its_parts(B, N, n, grad):
    gen = torch.Generator(device="cuda").manual_seed(n)
    full = [None] + [torch.randn(n, device="cuda", generator=gen).to(grad) for _ in range(N - 1)]

    def call(plan, a, b):
        plan.bind_full_grads([None if g is None else [g[a:b]] for g in full])
        plan.step(0, 4, 0.5, 0.05, 0.1)
    _whole_equals_parts(B, n, N, grad, 4096 * 397, call)
