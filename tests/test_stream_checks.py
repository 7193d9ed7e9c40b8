"""The checks of the peers' streams of a layer list: a stream that touches a buffer's end on either side is taken, one byte of
overlap, a stray address or a missing one refused, for every buffer, on either side of the lengths that are looked at at a time,
and what comes first by worker and tensor is what is reported.  (No GPU: the call with parameters that are refused behind these checks.)"""
import ctypes

import pytest

A, APART, N = 0x10000000, 0x1000000, 5


@pytest.fixture(scope="module")
def call():
    from paper_2106_10796_amd import binding, build
    build.ensure_built()
    L = binding.lib()

    def run(T, n, change=None, missing=None):
        """T tensors of n elements, far apart; change: {(worker, tensor): address}."""
        def base(i):
            return A + i * 16 * APART

        arr = (binding.cdsgd_tensor * T)()
        for i, t in enumerate(arr):
            t.w_global, t.w_local, t.residual, t.packed_self, t.grad = (base(i) + b * APART for b in range(5))
            t.agg_full, t.n = None, n
        rows = (ctypes.POINTER(ctypes.c_void_p) * N)()
        keep = []
        for j in range(N):
            if j in (2, missing):                            # the worker's own: no row
                continue
            keep.append((ctypes.c_void_p * T)(*[(change or {}).get((j, i), base(i) + (8 + j) * APART) for i in range(T)]))
            rows[j] = ctypes.cast(keep[-1], ctypes.POINTER(ctypes.c_void_p))
        return L.cdsgd_step_fused_static(arr, T, rows, N, 2, 0, 1, 0, 0.5, 0.1, 0.1, None)
    return run


@pytest.mark.parametrize("T,i", [(1, 0), (128, 127), (129, 128), (300, 255), (300, 256)])
@pytest.mark.parametrize("n", [1, 16, 1000])
def test_streams_at_the_ends_of_buffers(call, T, i, n):
    from paper_2106_10796_amd.binding import ERR_ALIAS, ERR_ALIGN, ERR_NULL, ERR_PARAM
    packed = 4 * ((n + 15) // 16)
    assert call(T, n) == ERR_PARAM                           # all checks passed
    for b in range(4):
        lo = A + i * 16 * APART + b * APART
        hi = lo + (packed if b == 3 else 4 * n)
        for j in (0, 4):
            assert call(T, n, {(j, i): lo - packed}) == ERR_PARAM
            assert call(T, n, {(j, i): hi}) == ERR_PARAM
            for inside in (lo - packed + 4, lo, hi - 4):
                assert call(T, n, {(j, i): inside}) == ERR_ALIAS
    for j in (0, 4):
        assert call(T, n, {(j, i): None}) == ERR_NULL
        assert call(T, n, {(j, i): A - 0x1000 + 2}) == ERR_ALIGN
    assert call(T, n, missing=4) == ERR_NULL


def test_the_first_fault_is_reported(call):
    from paper_2106_10796_amd.binding import ERR_ALIAS, ERR_ALIGN, ERR_NULL
    odd, on_w = A - 0x1000 + 2, A + 200 * 16 * APART
    assert call(300, 1000, {(3, 5): None, (1, 200): on_w}) == ERR_ALIAS
    assert call(300, 1000, {(1, 6): odd, (1, 5): None}) == ERR_NULL
    assert call(300, 1000, {(1, 200): odd, (3, 5): None}, missing=4) == ERR_ALIGN
    assert call(300, 1000, {(1, 200): on_w}, missing=0) == ERR_NULL
