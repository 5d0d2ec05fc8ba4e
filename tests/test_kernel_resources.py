"""Registers and scratch memory of the built kernels, read from the library's own kernel
descriptors (the metadata note of each embedded gfx950 code object); no GPU."""
import os
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1105_2791_amd", "libmodal.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def kernels(path=LIB):
    """{mangled name: metadata} of every gfx950 kernel in the library."""
    msgpack = pytest.importorskip("msgpack")
    d = open(path, "rb").read()
    out, at = {}, d.find(MAGIC)
    while at >= 0:
        o = at + 32
        for _ in range(struct.unpack_from("<Q", d, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", d, o)
            target, o = d[o + 24:o + 24 + n], o + 24 + n
            if not size or b"gfx950" not in target:
                continue
            elf = d[at + off:at + off + size]
            shoff = struct.unpack_from("<Q", elf, 0x28)[0]
            shsize, shnum = struct.unpack_from("<HH", elf, 0x3a)
            for k in range(shnum):
                sh = struct.unpack_from("<IIQQQQIIQQ", elf, shoff + k * shsize)
                if sh[1] != 7:   # SHT_NOTE
                    continue
                note = elf[sh[4]:sh[4] + sh[5]]
                nsz, dsz = struct.unpack_from("<II", note)
                desc = note[12 + (nsz + 3) // 4 * 4:][:dsz]
                for q in msgpack.unpackb(desc, raw=False)["amdhsa.kernels"]:
                    out[q[".name"]] = q
        at = d.find(MAGIC, at + 1)
    return out


@pytest.fixture(scope="module")
def built():
    if not os.path.exists(LIB):
        pytest.fail("libmodal.so is not built (run __graft_entry__.build())")
    return kernels()


def test_ring_transforms_use_no_scratch_memory(built):
    """The register-pass ring transforms hold a ring's points in registers: a pass that is
    called instead of inlined, or a spill, puts them in memory."""
    rg = {k: v for k, v in built.items() if "_rg" in k}
    assert len(rg) >= 15 and any("3008" in k for k in rg)
    assert {k: v[".private_segment_fixed_size"] for k, v in rg.items() if v[".private_segment_fixed_size"]} == {}


def test_split_synthesis_recurrence_does_not_spill(built):
    """The split synthesis that runs the recurrence itself: accumulators, lambda's words and the
    coefficients of a chunk fit its registers."""
    recur = {k: v for k, v in built.items() if "k_legendre_splitILi2ELi0E" in k or "k_legendre_splitILi3ELi0E" in k}
    assert len(recur) == 2
    assert {v[".private_segment_fixed_size"] for v in recur.values()} == {0}
