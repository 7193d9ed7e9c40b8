"""The kernels of the compressed pass that the library holds are those that a launch can reach: every combination of
workers, decode form, gradient type and launch shape that the rules of the dispatch give, and no other."""
import itertools
import re

from paper_2106_10796_amd import build

COUNT, CHAIN, TINY = 0, 1, 2
LATE, OUT, NT_WORDS, ARENA, SIX, FEW = 1, 2, 4, 8, 32, 64
TYPES, F32 = (0, 1, 2), (0,)
ANY = 0


def _held(name, pattern):
    build.ensure_built()
    with open(build.LIB, "rb") as fh:
        return {tuple(int(x) for x in m) for m in re.findall(name + pattern, fh.read())}


def test_passes_over_a_plan():
    want = set()

    def add(size, waves, forms, types, sparse, hows, weights_wait=(0,)):
        want.update((size, waves, *x) for x in itertools.product(forms, types, sparse, hows, weights_wait))
    both = (COUNT, CHAIN)
    add(8, 4, both, TYPES, (1,), (0,))
    add(16, 4, both, TYPES, (1,), (0,))
    add(32, 4, both, TYPES, (1,), (0,))
    add(8, 4, both, TYPES, (1,), (SIX,))
    add(16, 4, both, TYPES, (1,), (SIX,))
    add(32, 4, both, (1, 2), (1,), (SIX,))
    add(ANY, 4, (COUNT, CHAIN, TINY), TYPES, (0, 1), (0,))
    add(ANY, 4, (COUNT,), TYPES, (0,), (NT_WORDS,), (1,))
    add(ANY, 4, (CHAIN,), TYPES, (0,), (NT_WORDS,))
    add(8, 1, both, TYPES, (0,), (0, ARENA))
    add(8, 4, both, TYPES, (0,), (0, ARENA))
    add(8, 4, (COUNT,), F32, (0,), (FEW,))
    add(8, 4, (CHAIN,), TYPES, (0,), (FEW,))
    add(16, 4, both, TYPES, (0,), (0, OUT, ARENA, OUT | ARENA))
    add(16, 4, (CHAIN,), TYPES, (0,), (OUT | LATE, OUT | LATE | ARENA))
    add(16, 4, (COUNT,), F32, (0,), (OUT | LATE, OUT | LATE | ARENA))
    add(16, 4, (COUNT,), TYPES, (0,), (LATE,))
    add(32, 4, both, TYPES, (0,), (0, OUT, ARENA, OUT | ARENA))
    add(32, 4, both, TYPES, (0,), (OUT | ARENA,), (1,))
    assert _held(rb"k_fused_compressed", rb"ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb([01])ELi(\d+)ELb([01])EEE") == want


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


def _resources(name):
    """What the code object says of every kernel of that name: {mangled name: {key: number}}."""
    build.ensure_built()
    with open(build.LIB, "rb") as fh:
        text = fh.read()
    number = rb"([\x00-\x7f]|\xcc.|\xcd..)"           # msgpack's short unsigned numbers
    got = {}
    for m in re.finditer(rb"\.group_segment_fixed_size" + number + rb"(?:(?!\.group_segment_fixed_size).)*?\.name(?:\xd9.|\xda..)(_ZN\w*?"
                         + name + rb"\w*)\xbb\.private_segment_fixed_size" + number + rb"\xab\.sgpr_count" + number
                         + rb"\xb1\.sgpr_spill_count" + number, text, re.S):
        lds, _, sgprs, spilled = (int.from_bytes(x[1:] or x, "big") for x in (m[1], m[3], m[4], m[5]))
        got[m[2]] = {"lds": lds, "sgprs": sgprs, "spilled": spilled}
    return got


def _groups(kernel):
    """Groups of four waves that a compute unit's scalar registers admit: a SIMD has 800, a wave takes its own and 16 more, in sixteens."""
    return 800 // (-(-(kernel["sgprs"] + 16) // 16) * 16)


def test_scalar_registers_of_passes_over_arenas():
    """Up to 32 workers no stream pointer is kept in lanes of a vector register; six groups of 17 to 32 workers' passes fit a
    compute unit."""
    kernels = {k: v for k, v in _resources(b"k_fused_compressed").items() if re.search(rb"ILi(8|16|32)ELi\dELi\dELi\dELb0E", k)}
    arenas = {k: v for k, v in kernels.items() if re.search(rb"ELb0ELi(8|10|11)E", k)}
    assert len(arenas) > 40
    for k, v in kernels.items():
        assert v["spilled"] == 0, (k, v)
    for k, v in arenas.items():
        if b"ILi32E" in k:
            assert _groups(v) == 6, (k, v)


def test_groups_bounded_by_registers():
    """Passes of which a compute unit is to run six groups say so in registers, not in LDS, which other streams' kernels may want."""
    late = {**_resources(b"k_fused_compressedILi16ELi4ELi1ELi\\dELb0ELi(?:3|11)E"), **_resources(b"k_fused_argumentsILi16ELi4ELi1ELi\\dELi11E")}
    sparse = _resources(b"k_fused_compressedILi\\d+ELi4ELi\\dELi\\dELb1ELi32E")
    anyone = _resources(b"k_fused_compressedILi0ELi4ELi\\dELi\\dELb1ELi0E")   # any number of workers, sparse
    assert (len(late), len(sparse), len(anyone)) == (9, 16, 9)
    for k, v in {**late, **sparse, **anyone}.items():
        assert _groups(v) == 6, (k, v)


def test_no_row_without_an_own_worker():
    """The chain form's LDS of up to 16 workers holds their rows, and a spare one only where an own row is written without a test."""
    for size, rows in ((4, 4), (8, 8), (16, 16)):
        decode = _resources(b"k_decode_sumILi%dELi[12]ELb[01]ELi4E" % size)
        assert len(decode) == 6
        assert all(v["lds"] == 4 * 256 * rows for v in decode.values()), decode
    sparse = _resources(b"k_fused_compressedILi16ELi4ELi1ELi\\dELb1E")
    assert len(sparse) == 6 and all(v["lds"] == 256 * 16 for v in sparse.values()), sparse
