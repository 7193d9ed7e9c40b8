"""The calls marshalled in native code: what they decline, and that both ways of marshalling do the same."""
import numpy as np
import pytest
import torch

from paper_2106_10796_amd import binding as B


@pytest.fixture(scope="module")
def native():
    from paper_2106_10796_amd import build
    build.ensure_built()
    return B._native()


def _no_stream():
    raise AssertionError("asked for a stream though an argument is not good")


def test_declines_what_is_not_plainly_good(native):
    f, w = torch.zeros(32), torch.zeros(2, dtype=torch.int32)
    for got in (native.quantize_pack(f, f, w, 0.5, _no_stream), native.quantize_pack(f, f, w, 0.5),
                native.quantize_pack(None, f, w, 0.5, _no_stream), native.decode_sum([w], f, 0.5, _no_stream),
                native.decode_sum([], f, 0.5, _no_stream), native.decode_sum(iter([w]), f, 0.5, _no_stream),
                native.decode_sum_sparse((w,), f, 0.5, _no_stream), native.update(f, f, f, None, 0.1, 0.1, 2, _no_stream),
                native.update(3, f, f, None, 0.1, 0.1, 2, _no_stream), native.sparse_encode(w, 32, w, None, _no_stream),
                native.sparse_encode(w, -1, w, None, _no_stream), native.step(None, 1, 4, 0.5, 0.1, 0.1, _no_stream),
                native.step(0, 1, 4, 1, 0.1, 0.1, _no_stream), native.step(0, 1, 4, np.float32(0.5), 0.1, 0.1, _no_stream),
                native.step(0, 1 << 70, 4, 0.5, 0.1, 0.1, _no_stream), native.step(0, 1, 1 << 40, 0.5, 0.1, 0.1, _no_stream),
                native.step(0, True, 4, 0.5, 0.1, 0.1, _no_stream), native.step_range(0, 0, 1, 1, 4, 0.5, 0.1, "x", _no_stream)):
        assert got == -1


def test_says_what_is_wrong_as_before(native):
    f, w = torch.zeros(32), torch.zeros(2, dtype=torch.int32)
    with pytest.raises(TypeError, match="grad must be a contiguous CUDA tensor"):
        B.cdsgd_quantize_pack(f, f, w, 0.5)
    with pytest.raises(TypeError, match=r"packed\[0\] must be"):
        B.cdsgd_decode_sum([w], f, 0.5)
    with pytest.raises(TypeError, match="w_global must be"):
        B.cdsgd_update(f, f, f, None, 0.1, 0.1, 2)
    with pytest.raises(TypeError, match="bind takes"):
        native.bind(1)


def test_a_failing_stream_lookup_is_raised(native, monkeypatch):
    plan = B.Plan.__new__(B.Plan)
    plan._at, plan._handle = 0, None
    monkeypatch.setattr(B, "_stream", _no_stream)
    with pytest.raises(AssertionError, match="asked for a stream"):
        plan.step(1, 4, 0.5, 0.1, 0.1)
    monkeypatch.setattr(B, "_stream", lambda: 0)
    with pytest.raises(B.CdsgdError) as e:
        plan.step(1, 4, 0.5, 0.1, 0.1)
    assert e.value.status == B.ERR_NULL


class _Declines:
    def __getattr__(self, name):
        return lambda *a: -1


@pytest.mark.gpu
@pytest.mark.parametrize("N,n", [(1, 1), (3, 4097), (64, 70001)])
def test_both_ways_do_the_same(native, monkeypatch, N, n):
    gen = torch.Generator(device="cuda").manual_seed(n)
    rnd = lambda: torch.randn(n, device="cuda", generator=gen)
    first = dict(wg=rnd(), wl=rnd(), r=rnd(), g=rnd(), agg=rnd(), p=B.new_packed(n).zero_(), s=B.new_sparse(n).zero_(),
                 c=torch.zeros(B.sparse_segments(n), dtype=torch.int32, device="cuda"))
    second = {k: v.clone() for k, v in first.items()}
    streams = [torch.randint(-2 ** 31, 2 ** 31, (B.packed_words(n),), dtype=torch.int32, device="cuda", generator=gen)
               for _ in range(N)]

    def go(d, number):
        B.cdsgd_quantize_pack(d["g"], d["r"], d["p"], number(0.3))
        B.cdsgd_sparse_encode(d["p"], n, d["s"], d["c"])
        B.cdsgd_update(d["wg"], d["wl"], d["g"], None, number(0.1), number(0.2), N)
        B.cdsgd_decode_sum(streams, d["agg"], number(0.3))
        B.cdsgd_update(d["wg"], None, None, d["agg"], number(0.1), number(0.2), N)
        B.cdsgd_decode_sum_sparse(tuple([d["s"]] * N), d["agg"], number(0.25))
        layer = dict(w_global=d["wg"], w_local=d["wl"], residual=d["r"], grad=d["g"], packed_self=d["p"])
        peers = [None] + [[s] for s in streams[1:]]
        plan, static = B.Plan([layer], peers, N, 0), B.StaticLayerList([layer], peers, N)
        plan.step(1, 4, number(0.3), number(0.1), number(0.2))
        plan.step_range(0, 1, 2, 4, number(0.3), number(0.1), number(0.2))
        static.step(0, 3, 4, number(0.3), number(0.1), number(0.2))
        torch.cuda.synchronize()
        plan.destroy()
        with pytest.raises(B.CdsgdError):
            plan.step(1, 4, 0.3, 0.1, 0.2)

    go(first, float)
    with torch.cuda.stream(torch.cuda.Stream()):
        torch.cuda.current_stream().wait_stream(torch.cuda.default_stream())
        monkeypatch.setattr(B, "_calls", _Declines())
        go(second, np.float64)
    for k in first:
        assert torch.equal(first[k].view(torch.int32), second[k].view(torch.int32)), k


@pytest.mark.gpu
def test_bad_arguments_on_the_gpu(native):
    f, w = torch.zeros(64, device="cuda"), torch.zeros(4, dtype=torch.int32, device="cuda")
    with pytest.raises(ValueError, match="residual has 32 elements"):
        B.cdsgd_quantize_pack(f, f[:32], w, 0.5)
    with pytest.raises(TypeError):
        B.cdsgd_quantize_pack(f[::2], f[:32], w[:2], 0.5)
    with pytest.raises(TypeError):
        B.cdsgd_quantize_pack(f.double(), f, w, 0.5)
    with pytest.raises(B.CdsgdError) as e:
        B.cdsgd_quantize_pack(f, f.clone(), w, -1.0)
    assert e.value.status == B.ERR_PARAM
    with pytest.raises(B.CdsgdError) as e:
        B.cdsgd_quantize_pack(f[1:33], f.clone()[:32], w[:2], 0.5)
    assert e.value.status == B.ERR_ALIGN
    with pytest.raises(B.CdsgdError) as e:
        B.cdsgd_decode_sum([w] * 65, f, 0.5)
    assert e.value.status == B.ERR_WORKERS
