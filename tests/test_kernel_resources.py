"""Registers of the built library's kernels, from the metadata that the compiler writes beside each (ELF note of the
gfx950 code object): the vector registers decide how many workgroups a CU holds, and spills go to memory."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

from paper_2609_03515_amd import build


def code_object(blob):
    """The gfx950 code objects inside a host library: (offset, size) entries of every offload bundle."""
    out, magic = [], b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        count, p = struct.unpack_from("<Q", blob, at + len(magic))[0], at + len(magic) + 8
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24 : p + 24 + tlen].decode()
            p += 24 + tlen
            if triple.endswith("gfx950") and size:
                out.append(blob[at + off : at + off + size])
        at = blob.find(magic, at + 1)
    return out


def metadata(elf):
    """The AMDGPU metadata note (type 32) of an ELF64 code object."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entsize, num = struct.unpack_from("<HH", elf, 58)
    for i in range(num):
        kind, _, _, off, size = struct.unpack_from("<IQQQQ", elf, shoff + i * entsize + 4)
        if kind != 7:
            continue
        p = off
        while p < off + size:
            nlen, dlen, ntype = struct.unpack_from("<III", elf, p)
            name, p = elf[p + 12 : p + 12 + nlen], p + 12 + (nlen + 3) // 4 * 4
            if ntype == 32 and name.startswith(b"AMDGPU"):
                return msgpack.unpackb(elf[p : p + dlen])
            p += (dlen + 3) // 4 * 4
    raise AssertionError("no metadata note")


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(build.LIB):
        build.build()
    with open(build.LIB, "rb") as f:
        objs = code_object(f.read())
    assert objs, "no uncompressed gfx950 code object in the library"
    found = {}
    for o in objs:
        for k in metadata(o)["amdhsa.kernels"]:
            found[k[".name"]] = k
    names = subprocess.run(["c++filt", "-p"], input="\n".join(found), text=True, capture_output=True, check=True)
    names = names.stdout.split("\n")
    return {re.sub(r"ikv::|\(anonymous namespace\)::", "", n): k for n, k in zip(names, found.values())}


def test_scorer_spills(kernels):
    """The scorer of f32 rows of 128 with one head per KV head holds 16 rows a lane and spills 84 to 130 registers (one
    slab, several, VNorm); with each wave's first units loaded ahead of the queries it had been 97 to 179 and 6% slower.
    No other scorer instance spills."""
    most = {"<float, 128, 1, false, false>": 84, "<float, 128, 1, true, false>": 91, "<float, 128, 1, true, true>": 130}
    seen = {n[len("score_lds_kernel"):]: k[".vgpr_spill_count"] for n, k in kernels.items() if n.startswith("score_lds_kernel")}
    assert set(most) <= set(seen)
    assert {n: c for n, c in seen.items() if c > most.get(n, 0)} == {}


def test_fold_registers(kernels):
    """VNorm's fold, which keeps no rows in flight, is an instance of its own with 8 waves per SIMD (64 of 512
    registers); so are the folds of few rows per layer."""
    used = {i: kernels["fold_kernel" + i][".vgpr_count"] for i in ("<0>", "<2>", "<4>")}
    assert max(used.values()) <= 64, used
