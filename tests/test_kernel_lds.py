"""Kernels that lay the decode tables out in LDS (carve) address them with or, which is right only
where dynamic LDS starts at address 0: they may have no static LDS.  The built library's own
kernel descriptions say how much each has."""
import glob
import os
import re
import struct

import msgpack
import pytest

from paper_1711_00244_amd import binding

CSRC = os.path.join(os.path.dirname(binding.__file__), "csrc")


def _kernels(path):
    """name -> bytes of static LDS, from the notes of the gfx950 code objects in the library."""
    data = open(path, "rb").read()
    sizes = {}
    for bundle in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        base = bundle.start()
        n, at = struct.unpack_from("<Q", data, base + 24)[0], base + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            triple = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" not in triple:
                continue
            elf = data[base + offset:base + offset + size]
            shoff, = struct.unpack_from("<Q", elf, 0x28)
            shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
            for i in range(shnum):
                kind, _, _, off, length_, = struct.unpack_from("<IQQQQ", elf, shoff + i * shentsize + 4)
                if kind != 7:                                                   # SHT_NOTE
                    continue
                namesz, descsz, what = struct.unpack_from("<III", elf, off)
                if what == 32:                                                  # the metadata note
                    desc = elf[off + 12 + (namesz + 3) // 4 * 4:][:descsz]
                    for k in msgpack.unpackb(desc)["amdhsa.kernels"]:
                        sizes[k[".name"]] = k[".group_segment_fixed_size"]
    return sizes


def _callers_of_carve():
    """Names of the kernels that call carve, themselves or through a function of the sources."""
    bodies = {}                                 # function -> (is a kernel, body), one per overload
    for f in glob.glob(os.path.join(CSRC, "*.hpp")) + glob.glob(os.path.join(CSRC, "*.hip")):
        for part in open(f).read().split("\n}\n"):
            head, brace, body = part.rpartition("\n{\n") if part.count("\n{\n") == 1 else part.partition("\n{\n")
            head = re.sub(r"//.*", "", head).split("\n\n")[-1]                   # the declaration right before the body
            m = re.search(r"(\w+)\(", re.sub(r"__launch_bounds__\(.*?\)\s+(?=void)", "", head))
            if brace and m:
                bodies.setdefault(m.group(1), []).append(("__global__" in head, body))
    reach = {"carve"}
    while True:
        more = {n for n, bs in bodies.items() if any(re.search(r"\b%s(<[^()]*>)?\(" % r, b) for _, b in bs for r in reach)} - reach
        if not more:
            break
        reach |= more
    return {n for n in reach if any(g for g, _ in bodies.get(n, []))}


@pytest.mark.skipif(not os.path.exists(binding.library_path()), reason="library not built")
def test_kernels_with_decode_tables_have_no_static_lds():
    sizes, callers = _kernels(binding.library_path()), _callers_of_carve()
    # the sources are read right: the kernels this is about are among them, and some kernel has static LDS
    assert {"decode_kernel", "decode_blocks_kernel", "fc_sparse_kernel", "fc_sparse_group_kernel", "fc_rows_kernel", "fc_mfma_kernel",
            "fc_mfma_bf16_kernel", "wide_expand_kernel", "decode_tiles_kernel"} <= callers, callers
    assert any(sizes.values())
    for name in callers:
        mine = {k: v for k, v in sizes.items() if re.search(r"\d%s[A-Z]" % name, k)}
        assert mine, name
        assert not any(mine.values()), mine
