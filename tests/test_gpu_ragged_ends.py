"""GPU parity of every pass at ragged ends, where loads and stores are clipped word by word at the end of a tensor: all
remainders of a quad, a word of codes, a wave, a tile and a chunk, each gradient type, against the oracle bit for bit.  What
lies between and behind the tensors has to be what it was: NaN, but for gradients and residuals values past the threshold and for streams
codes that are sent, so that one read from there would show in the codes behind a tensor's last one."""
import numpy as np
import pytest
import torch

from helpers import assert_bits_equal

pytestmark = pytest.mark.gpu

SIZES = [*range(1, 10), *range(62, 68), *range(253, 260), *range(1021, 1030), *range(4093, 4100), 4096 + 1022, 2 * 4096 + 2051]
LR_LOCAL, LR_GLOBAL, N = 0.4, 0.7, 5


@pytest.fixture(scope="module")
def B():
    from paper_2106_10796_amd import binding, build
    build.ensure_built()
    binding.lib()
    assert torch.cuda.is_available()
    return binding


class _Arena:
    """A tensor of every size in one allocation, `fill` (in packed words: all codes 01) between and behind them."""

    def __init__(self, values, dtype, fill=9.0):
        self.packed, per = dtype == torch.int32, 16 if dtype == torch.int32 else 1
        self.fill = 0x55555555 if self.packed else fill
        at, total = [], 0
        for n in SIZES:
            at.append(total // per)
            total += (n + 63) // 64 * 64 + 64
        self.all = torch.full((total // per,), self.fill, dtype=dtype, device="cuda")
        self.views = [self.all[a: a + v.size] for a, v in zip(at, values)]
        self.between = torch.ones(self.all.numel(), dtype=torch.bool, device="cuda")
        for a, v in zip(at, values):
            self.between[a: a + v.size] = False
        self.set(values)

    def set(self, values):
        for view, v in zip(self.views, values):
            view.copy_(torch.from_numpy(v.view(np.int32) if self.packed else v))

    def check(self, want, what):
        left = self.all[self.between]
        assert bool((left == self.fill).all() if self.fill == self.fill else torch.isnan(left).all()), "%s: written between tensors" % what
        for n, view, ref in zip(SIZES, self.views, want):
            assert_bits_equal((view if self.packed else view.float()).cpu().numpy(), ref.view(np.int32) if self.packed else ref, "%s of %d elements" % (what, n))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
def test_every_pass_at_ragged_ends(B, oracle, dtype):
    rng = np.random.default_rng(7)
    t, rank = 0.5, 3
    values = lambda s: [rng.standard_normal(n, dtype=np.float32) * np.float32(s) for n in SIZES]
    widened = lambda vs: [torch.from_numpy(v).to(dtype).float().numpy() for v in vs]
    host = dict(w_global=values(1.0), w_local=values(1.0), residual=values(0.2), grad=widened(values(0.5)), agg_full=values(1.0),
                packed_self=[np.zeros((n + 15) // 16, np.uint32) for n in SIZES])
    dev = {k: _Arena(v, dtype if k == "grad" else (torch.int32 if k == "packed_self" else torch.float32),
                     9.0 if k in ("grad", "residual") else float("nan")) for k, v in host.items()}
    words = [[oracle.pack(rng.integers(0, 4, n).astype(np.uint8)) for n in SIZES] for _ in range(N)]
    peers = [None if j == rank else _Arena(words[j], torch.int32).views for j in range(N)]
    grads = [host["grad"] if j == rank else widened(values(0.5)) for j in range(N)]
    bound = [None if j == rank else _Arena(grads[j], dtype).views for j in range(N)]
    layers = [{k: a.views[i] for k, a in dev.items()} for i in range(len(SIZES))]
    everywhere = range(len(SIZES))

    def check(what):
        torch.cuda.synchronize()
        for k, a in dev.items():
            a.check(host[k], "%s: %s" % (what, k))

    plan = B.Plan(layers, peers, N, rank, grad_dtype=dtype)
    for what in ("compressed", "static"):
        for i in everywhere:
            words[rank][i] = host["packed_self"][i] = oracle.quantize_pack(host["grad"][i], host["residual"][i], t)
            oracle.update(host["w_global"][i], host["w_local"][i], host["grad"][i],
                          oracle.decode_sum([w[i] for w in words], SIZES[i], t), LR_LOCAL, LR_GLOBAL, N)
        if what == "static":
            B.cdsgd_step_fused_static(layers, peers, N, rank, 1, 4, t, LR_LOCAL, LR_GLOBAL, grad_dtype=dtype)
        else:
            plan.step(1, 4, t, LR_LOCAL, LR_GLOBAL)
        check(what)
    plan.step(0, 4, t, LR_LOCAL, LR_GLOBAL)
    for i in everywhere:
        oracle.update(host["w_global"][i], host["w_local"][i], host["grad"][i], host["agg_full"][i], LR_LOCAL, LR_GLOBAL, N)
    check("correction, aggregate given")
    plan.bind_full_grads(bound)
    plan.step(0, 4, t, LR_LOCAL, LR_GLOBAL)
    for i in everywhere:
        oracle.update(host["w_global"][i], host["w_local"][i], host["grad"][i], oracle.full_sum([g[i] for g in grads]),
                      LR_LOCAL, LR_GLOBAL, N)
    check("correction, summed")
    plan.step_local(LR_LOCAL)
    for i in everywhere:
        oracle.update(host["w_global"][i], host["w_local"][i], host["grad"][i], None, LR_LOCAL, LR_GLOBAL, N)
    check("local half")
    plan.destroy()
    if dtype == torch.float32:
        for i in everywhere:
            x = layers[i]
            B.cdsgd_quantize_pack(x["grad"], x["residual"], x["packed_self"], t)
            host["packed_self"][i] = oracle.quantize_pack(host["grad"][i], host["residual"][i], t)
            words[rank][i] = host["packed_self"][i]
            B.cdsgd_decode_sum([x["packed_self"] if j == rank else peers[j][i] for j in range(N)], x["agg_full"], t)
            host["agg_full"][i] = oracle.decode_sum([w[i] for w in words], SIZES[i], t)
            B.cdsgd_update(x["w_global"], x["w_local"], x["grad"], x["agg_full"], LR_LOCAL, LR_GLOBAL, N)
            oracle.update(host["w_global"][i], host["w_local"][i], host["grad"][i], host["agg_full"][i], LR_LOCAL, LR_GLOBAL, N)
        check("calls per tensor")
