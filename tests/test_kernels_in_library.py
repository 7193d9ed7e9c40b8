"""The kernels of the compressed pass that the library holds are those that a launch can reach: every combination of
workers, decode form, gradient type and launch shape that the rules of the dispatch give, and no other."""
import itertools
import re

from paper_2106_10796_amd import build

COUNT, CHAIN, TINY = 0, 1, 2
LATE, OUT, NT_WORDS, ARENA = 1, 2, 4, 8
TYPES, F32 = (0, 1, 2), (0,)
ANY = 0


def _held(name, pattern):
    build.ensure_built()
    with open(build.LIB, "rb") as fh:
        return {tuple(int(x) for x in m) for m in re.findall(name + pattern, fh.read())}


def test_passes_over_a_plan():
    want = set()

    def add(size, waves, forms, types, sparse, hows):
        want.update((size, waves, f, t, s, h) for f, t, s, h in itertools.product(forms, types, sparse, hows))
    both = (COUNT, CHAIN)
    add(8, 4, both, TYPES, (1,), (0,))
    add(16, 4, both, TYPES, (1,), (0,))
    add(32, 4, both, TYPES, (1,), (0,))
    add(ANY, 4, (COUNT, CHAIN, TINY), TYPES, (0, 1), (0,))
    add(ANY, 4, both, TYPES, (0,), (NT_WORDS,))
    add(8, 1, both, TYPES, (0,), (0, ARENA))
    add(8, 4, both, TYPES, (0,), (0, ARENA))
    add(16, 4, both, TYPES, (0,), (0, OUT, ARENA, OUT | ARENA))
    add(16, 4, (CHAIN,), TYPES, (0,), (OUT | LATE, OUT | LATE | ARENA))
    add(16, 4, (COUNT,), F32, (0,), (OUT | LATE, OUT | LATE | ARENA))
    add(16, 4, (COUNT,), TYPES, (0,), (LATE,))
    add(32, 4, both, TYPES, (0,), (0, OUT, ARENA, OUT | ARENA))
    assert _held(rb"k_fused_compressed", rb"ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb([01])ELi(\d+)E") == want


def test_passes_from_arguments():
    want = set()

    def add(size, waves, forms, types, hows):
        want.update((size, waves, f, t, h | ARENA) for f, t, h in itertools.product(forms, types, hows))
    both = (COUNT, CHAIN)
    add(8, 1, both, TYPES, (0,))
    add(8, 4, both, TYPES, (0,))
    add(16, 4, both, TYPES, (0, OUT))
    add(16, 4, (CHAIN,), TYPES, (OUT | LATE,))
    add(16, 4, (COUNT,), F32, (OUT | LATE,))
    add(32, 4, both, TYPES, (0, OUT))
    add(ANY, 4, both, TYPES, (0,))
    assert _held(rb"k_fused_arguments", rb"ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E") == want
