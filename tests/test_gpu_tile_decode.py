"""GPU parity of the compressed pass at the edges of its tiles (256 and 1024 elements, chunks of 4096) and of its
batches of workers (8, 16, 32, 48), in every decode form: count form, chain form, chain form for thresholds whose half
is not exact; packed and sparse peers.  Bit for bit against the oracle: the interface fixes every sum's order."""
import numpy as np
import pytest
import torch

from helpers import ODD_TINY, assert_bits_equal

pytestmark = pytest.mark.gpu

SIZES = [1, 5, 16, 255, 257, 1023, 1024, 1025, 2048 + 15, 4096, 4096 + 1024 + 3, 2 * 4096 - 1, 3 * 4096 + 256]
TINY = ODD_TINY[2]   # about 1.37 * 2^-127: its half is not exact


@pytest.fixture(scope="module")
def B():
    from paper_2106_10796_amd import binding, build
    build.ensure_built()
    binding.lib()
    assert torch.cuda.is_available()
    return binding


def _words(oracle, rng, n):
    codes = rng.choice(4, size=n, p=[0.4, 0.3, 0.25, 0.05]).astype(np.uint8)   # the field that reads as nothing too
    return oracle.pack(np.ascontiguousarray(codes))


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("t", [0.25, 0.3, TINY])
@pytest.mark.parametrize("N", [1, 2, 4, 7, 8, 9, 15, 16, 17, 32, 33, 49, 63, 64])
def test_compressed_pass_at_tile_and_batch_edges(B, oracle, N, t, sparse):
    rng = np.random.default_rng(97 * N + int(sparse))
    self_rank = int(rng.integers(N))
    f = lambda a: torch.from_numpy(a).cuda()
    layers, want = [], []
    streams = [[_words(oracle, rng, n) for n in SIZES] for _ in range(N)]
    for i, n in enumerate(SIZES):
        g = rng.normal(0, t, n).astype(np.float32)
        r = (rng.uniform(-1, 1, n) * t).astype(np.float32)
        w = (rng.normal(0, 1, n) * (1.0 if t > 1e-30 else 64 * t)).astype(np.float32)
        layers.append(dict(w_global=f(w), w_local=f(np.full(n, 3.0, np.float32)), residual=f(r), grad=f(g),
                           packed_self=torch.full((B.packed_words(n),), -1, dtype=torch.int32, device="cuda")))
        r2, w2, l2 = r.copy(), w.copy(), np.zeros(n, np.float32)
        own = oracle.quantize_pack(g, r2, t)
        streams[self_rank][i] = own
        agg = oracle.decode_sum([streams[j][i] for j in range(N)], n, t)
        oracle.update(w2, l2, g, agg, 0.4, 0.7, N)
        want.append((r2, own, w2, l2))

    def on_gpu(words, n):
        if sparse:
            words = oracle.sparse_encode(words, n, fill=0x7F7F7F7F)[0]
        elif n % 16:
            words = words.copy()
            words[-1] |= np.uint32(0xFFFFFFFF ^ ((1 << (2 * (n % 16))) - 1))   # garbage behind the last element
        return f(words.view(np.int32))

    peers = [None if j == self_rank else [on_gpu(streams[j][i], n) for i, n in enumerate(SIZES)] for j in range(N)]
    plan = B.Plan(layers, peers if N > 1 else None, N, self_rank, peers_sparse=sparse)
    plan.step(1, 4, t, 0.4, 0.7)
    torch.cuda.synchronize()
    for i, n in enumerate(SIZES):
        for key, ref in zip(("residual", "packed_self", "w_global", "w_local"), want[i]):
            ref = ref.view(np.int32) if key == "packed_self" else ref
            assert_bits_equal(layers[i][key].cpu().numpy(), ref, "%s N=%d self=%d n=%d t=%g" % (key, N, self_rank, n, t))
        # the same streams through the single-tensor call
        full = torch.full((n + 8,), 9.0, device="cuda")
        decode = B.cdsgd_decode_sum_sparse if sparse else B.cdsgd_decode_sum
        decode([on_gpu(streams[j][i], n) for j in range(N)], full[:n], t)
        agg = oracle.decode_sum([streams[j][i] for j in range(N)], n, t)
        assert_bits_equal(full[:n].cpu().numpy(), agg, "agg N=%d n=%d t=%g" % (N, n, t))
        assert bool((full[n:] == 9.0).all())
    plan.destroy()


@pytest.mark.parametrize("sparse", [False, True])
@pytest.mark.parametrize("N", [1, 4, 9, 17, 64])
def test_own_thresholds_of_every_kind_in_one_list(B, oracle, N, sparse):
    """Thresholds whose half is not exact beside ordinary and very large ones: one kernel decodes them all."""
    rng = np.random.default_rng(7 * N + int(sparse))
    ts = [*ODD_TINY, 0.3, 0.5, 2.0 ** -125, float(np.nextafter(np.float32(2.0 ** -125), np.float32(1))), 1e30, 1e36]
    n, f = 2 * 4096 + 1027, lambda a: torch.from_numpy(a).cuda()
    layers, want, streams = [], [], []
    for t in ts:
        g, r = rng.normal(0, t, n).astype(np.float32), (rng.uniform(-1, 1, n) * t).astype(np.float32)
        w = (rng.uniform(-1, 1, n) * 64 * t).astype(np.float32)
        layers.append(dict(w_global=f(w), w_local=f(np.zeros(n, np.float32)), residual=f(r), grad=f(g), packed_self=B.new_packed(n)))
        given = [_words(oracle, rng, n) for _ in range(N)]
        r2, w2, l2 = r.copy(), w.copy(), np.zeros(n, np.float32)
        given[0] = own = oracle.quantize_pack(g, r2, t)
        oracle.update(w2, l2, g, oracle.decode_sum(given, n, t), 0.4, 0.7, N)
        want.append((r2, own, w2, l2))
        streams.append(given)
    on_gpu = lambda w: f((oracle.sparse_encode(w, n, fill=0x7F7F7F7F)[0] if sparse else w).view(np.int32))
    peers = [None] + [[on_gpu(s[j]) for s in streams] for j in range(1, N)]
    plan = B.Plan(layers, peers if N > 1 else None, N, 0, peers_sparse=sparse)
    plan.set_thresholds(ts)
    plan.step(1, 4, 0.5, 0.4, 0.7)
    torch.cuda.synchronize()
    for i, t in enumerate(ts):
        for key, ref in zip(("residual", "packed_self", "w_global", "w_local"), want[i]):
            ref = ref.view(np.int32) if key == "packed_self" else ref
            assert_bits_equal(layers[i][key].cpu().numpy(), ref, "%s N=%d t=%g" % (key, N, t))
    plan.destroy()


@pytest.mark.parametrize("t", [0.5, 0.3])
@pytest.mark.parametrize("N", [4, 8, 12])
def test_long_list_of_few_workers(B, N, t):
    """A list long enough for the one-wave groups, and for the workers' words behind the tile's own streams (more than
    2^24 elements), against the single-tensor calls."""
    n = (1 << 24) + 4096 * 3 + 277
    gen = torch.Generator(device="cuda").manual_seed(5 + N)
    rand = lambda s: torch.empty(n, device="cuda").normal_(0, s, generator=gen)
    g, r, w = rand(t), rand(0.4 * t), rand(1.0)
    streams = [torch.randint(-2 ** 31, 2 ** 31, (B.packed_words(n),), dtype=torch.int32, device="cuda", generator=gen)
               for _ in range(N)]
    layer = dict(w_global=w.clone(), w_local=torch.zeros_like(w), residual=r.clone(), grad=g,
                 packed_self=B.new_packed(n))
    plan = B.Plan([layer], [None if j == 1 else [streams[j]] for j in range(N)], N, 1)
    plan.step(1, 4, t, 0.4, 0.7)
    own, agg, wl = B.new_packed(n), torch.empty_like(w), torch.empty_like(w)
    B.cdsgd_quantize_pack(g, r, own, t)
    B.cdsgd_decode_sum([own if j == 1 else streams[j] for j in range(N)], agg, t)
    B.cdsgd_update(w, wl, g, agg, 0.4, 0.7, N)
    torch.cuda.synchronize()
    for key, ref in (("packed_self", own), ("residual", r), ("w_global", w), ("w_local", wl)):
        assert torch.equal(layer[key].view(torch.int32), ref.view(torch.int32)), "%s N=%d t=%g" % (key, N, t)
    plan.destroy()


@pytest.mark.parametrize("n", [(24 << 20) - 3, 24 << 20, (24 << 20) + 5])
def test_single_tensor_calls_at_the_kept_gradient_limit(B, n):
    """Quantise-and-pack and the update (eq. 11 alone, both rules) on the two sides of the length up to which the
    gradient's loads keep it cached, against the pass over a list of that one tensor, N = 1."""
    gen = torch.Generator(device="cuda").manual_seed(11)
    rand = lambda s: torch.empty(n, device="cuda").normal_(0, s, generator=gen)
    g, r, w = rand(0.3), rand(0.2), rand(1.0)
    layer = dict(w_global=w.clone(), w_local=torch.zeros_like(w), residual=r.clone(), grad=g, packed_self=B.new_packed(n))
    plan = B.Plan([layer], None, 1, 0)
    plan.step(1, 4, 0.3, 0.4, 0.7)
    own, agg, wl, wl2 = B.new_packed(n), torch.empty_like(w), torch.zeros_like(w), torch.zeros_like(w)
    B.cdsgd_update(w, wl, g, None, 0.4, 0.7, 1)
    B.cdsgd_quantize_pack(g, r, own, 0.3)
    B.cdsgd_decode_sum([own], agg, 0.3)
    B.cdsgd_update(w, wl2, g, agg, 0.4, 0.7, 1)
    torch.cuda.synchronize()
    for what, a, b in (("packed", layer["packed_self"], own), ("residual", layer["residual"], r), ("w_global", layer["w_global"], w),
                       ("w_local", layer["w_local"], wl), ("w_local, both rules", layer["w_local"], wl2)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32)), "%s n=%d" % (what, n)
    plan.destroy()
