"""GPU parity of cdsgd_step_fused_static's tables, in both forms they travel in (lists in arenas, lists of buffers
that lie anywhere), one and several launches of them, against a plan on the same list: bit for bit."""
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


def _lists(B, sizes, N, rank, t, dtype, layout, seed):
    """The same layer list twice (one to step through each entry point) and the peers' streams."""
    at, total = [], 0
    for n in sizes:
        at.append(total)
        total += (n + 1023) // 1024 * 1024
    if layout == "reversed":          # arenas, but tensor 0 lies behind the others
        at = [total - o - (n + 1023) // 1024 * 1024 for o, n in zip(at, sizes)]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    f32 = lambda s: torch.empty(total, device="cuda").normal_(0, s, generator=gen)
    base = dict(w_global=f32(1.0), w_local=torch.zeros(total, device="cuda"), residual=f32(0.4 * t),
                grad=f32(t).to(dtype), agg_full=f32(t),
                packed_self=torch.zeros(total // 16, dtype=torch.int32, device="cuda"))
    streams = [torch.randint(-2 ** 31, 2 ** 31, (total // 16,), dtype=torch.int32, device="cuda", generator=gen)
               for _ in range(N)]
    cut = lambda a: [a[o: o + n] for o, n in zip(at, sizes)]
    words = lambda a: [a[o // 16: o // 16 + B.packed_words(n)] for o, n in zip(at, sizes)]
    out = []
    for _ in range(2):
        a = {k: v.clone() for k, v in base.items()}
        parts = {k: (words(v) if k == "packed_self" else cut(v)) for k, v in a.items()}
        if layout == "one_moved":     # a single buffer of a single tensor elsewhere
            parts["w_local"][-1] = torch.zeros(sizes[-1], device="cuda")
        out.append([{k: v[i] for k, v in parts.items()} for i in range(len(sizes))])
    if layout == "apart":
        out = [[{k: v.clone() for k, v in d.items()} for d in lst] for lst in out]
    peers = [None if j == rank else words(streams[j]) for j in range(N)] if N > 1 else None
    return out, peers


@pytest.mark.parametrize("layout", ["arenas", "reversed", "one_moved", "apart"])
@pytest.mark.parametrize("T,N,dtype", [(1, 4, torch.float32), (300, 8, torch.float16), (70, 1, torch.float32),
                                       (61, 17, torch.bfloat16), (20, 64, torch.float32), (1024, 3, torch.float32)])
@pytest.mark.parametrize("step", [0, 1])
def test_static_entry_equals_a_plan(B, layout, T, N, dtype, step):
    rng = np.random.default_rng(T + N)
    sizes = [int(x) for x in 2 ** rng.uniform(0, 13.5, T)]
    t, rank = 0.3, N // 2
    (mine, ref), peers = _lists(B, sizes, N, rank, t, dtype, layout, 11 * T + N)
    plan = B.Plan(ref, peers, N, rank, grad_dtype=dtype)
    plan.step(step, 4, t, 0.4, 0.7)
    B.cdsgd_step_fused_static(mine, peers, N, rank, step, 4, t, 0.4, 0.7, grad_dtype=dtype)
    torch.cuda.synchronize()
    for i in range(T):
        for key in ("w_global", "w_local", "residual", "packed_self"):
            assert torch.equal(mine[i][key].view(torch.int32), ref[i][key].view(torch.int32)), \
                "%s of tensor %d (n=%d), %s, T=%d N=%d step %d" % (key, i, sizes[i], layout, T, N, step)
    plan.destroy()
