"""Every device function of the built library is within a branch's reach (no
GPU).  A branch holds 16 signed bits of 4-byte words, 128 KiB; beyond it the
compiler jumps through a register pair, and in a function that calls nothing
it took the pair of the return address, so that the function never came back
(the 5-clique listing at roots of out-degree 833 to 896)."""
import os
import struct

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2011_03135_amd", "libgpmhip.so")
REACH = 128 * 1024
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            start, size, id_len = struct.unpack_from("<QQQ", blob, p)
            if blob[p + 24:p + 24 + id_len].startswith(b"hip") and size:
                yield blob[at + start:at + start + size]
            p += 24 + id_len
        at = blob.find(MAGIC, at + 1)


def functions(elf):
    """(name, bytes) of the functions in a code object's symbol tables."""
    assert elf[:4] == b"\x7fELF"
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    heads = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * shentsize) for i in range(shnum)]
    for h in heads:
        if h[1] not in (2, 11):   # SHT_SYMTAB, SHT_DYNSYM
            continue
        names = heads[h[6]][4]
        for s in range(h[4], h[4] + h[5], 24):
            name, info, _, _, _, size = struct.unpack_from("<IBBHQQ", elf, s)
            if info & 15 == 2:    # STT_FUNC
                a = names + name
                yield elf[a:elf.index(b"\0", a)].decode(), size


def test_functions_within_a_branchs_reach():
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    with open(LIB, "rb") as f:
        sizes = dict(x for o in code_objects(f.read()) for x in functions(o))
    assert any("k_lg5" in n for n in sizes) and any("lgk_set" in n or "k_tc_seg" in n for n in sizes)
    assert {n: s for n, s in sizes.items() if s >= REACH} == {}
