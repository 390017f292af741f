"""Registers that the compiled kernels spill, from the metadata of the code objects in libddml.so.

A change of the source around a kernel can make the compiler keep more alive than
there are registers.  Nothing fails then: the values go through scratch memory and
the kernel is slower.
"""
import os
import re
import struct
import subprocess

import pytest

msgpack = pytest.importorskip("msgpack")

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1601_04587_amd", "libddml.so")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The gfx950 ELF images of every offload bundle in the library."""
    for m in re.finditer(MAGIC, blob):
        base = m.start()
        n, = struct.unpack_from("<Q", blob, base + len(MAGIC))
        at = base + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, at)
            triple = blob[at + 24:at + 24 + idlen]
            at += 24 + idlen
            if b"gfx950" in triple and size:
                yield blob[base + off:base + off + size]


def _kernels(elf):
    """The kernels' entries of an image's AMDGPU metadata note (type 32)."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phsize, phnum = struct.unpack_from("<HH", elf, 54)
    for k in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + k * phsize)
        if kind != 4:   # PT_NOTE
            continue
        at = off
        while at < off + size:
            nlen, dlen, note = struct.unpack_from("<III", elf, at)
            data = at + 12 + (nlen + 3) // 4 * 4
            if note == 32 and elf[at + 12:at + 18] == b"AMDGPU":
                yield from msgpack.unpackb(elf[data:data + dlen], strict_map_key=False)["amdhsa.kernels"]
            at = data + (dlen + 3) // 4 * 4


@pytest.fixture(scope="module")
def spills():
    if not os.path.exists(LIB):
        pytest.skip("libddml.so is not built")
    with open(LIB, "rb") as f:
        blob = f.read()
    out = {}
    for elf in _code_objects(blob):
        for k in _kernels(elf):
            out[k[".name"]] = k[".vgpr_spill_count"]
    assert out, "no kernel metadata found"
    names = subprocess.run(["c++filt"], input="\n".join(out), capture_output=True, text=True).stdout.split("\n")
    return {n.split("(")[0].split(" ", 1)[-1]: v for n, v in zip(names, out.values())}


# The most that a kernel of the family may spill: a quarter of its 168 registers for the
# unstaged FP64 stencil, which reads links and clover data itself; the twelve components
# of one column for the 16-bit one
@pytest.mark.parametrize("kernel,most", [("k_hop_item", 42), (r"k_hop_batch<ddml::h16c", 12)])
def test_stencils_keep_their_values_in_registers(spills, kernel, most):
    found = {n: v for n, v in spills.items() if re.search(kernel, n)}
    assert found
    assert max(found.values()) <= most, found
