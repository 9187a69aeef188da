"""Scratch memory of the built library's kernels, from the metadata in its own code objects (no GPU needed)."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2608_01718_amd", "liblacache.so")

# bytes a lane of the kernels that keep a few registers in scratch outside their main loops, by the start of the name
ALLOWED = {"k_stage1_gemm<7>": 68, "k_simhash_bulk": 12}


def _code_objects(blob):
    """The gfx950 code objects of every offload bundle in the library."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        n, p = struct.unpack_from("<Q", blob, at + len(magic))[0], at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, p)
            ident = blob[p + 24:p + 24 + idlen]
            p += 24 + idlen
            if b"gfx950" in ident:
                yield blob[at + off:at + off + size]
        at += len(magic)


def _metadata(elf):
    """The AMDGPU metadata note (type 32) of a 64-bit ELF file."""
    assert elf[:4] == b"\x7fELF"
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        p, end = off, off + size
        while kind == 7 and p < end:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, p)
            p += 12 + (namesz + 3) // 4 * 4
            if ntype == 32:
                return msgpack.unpackb(elf[p:p + descsz], raw=False, strict_map_key=False)
            p += (descsz + 3) // 4 * 4
    raise AssertionError("no metadata note")


def _name(mangled):
    """k_name<first, ...> of a kernel lacache::k_name<...>(...), from its mangled name (integer arguments)."""
    rest = mangled.split("7lacache", 1)[1]
    digits = len(rest) - len(rest.lstrip("0123456789"))
    n = int(rest[:digits])
    name, rest = rest[digits:digits + n], rest[digits + n:]
    if not rest.startswith("I"):
        return name
    args = [a.split("E")[0][1:] for a in rest[1:].split("EEv")[0].split("L")[1:]]
    return f"{name}<{', '.join(args)}>"


def test_kernels_need_no_scratch():
    with open(LIB, "rb") as f:
        blob = f.read()
    kernels = {}
    for obj in _code_objects(blob):
        for k in _metadata(obj)["amdhsa.kernels"]:
            kernels[_name(k[".name"])] = k[".private_segment_fixed_size"]
    assert len(kernels) > 40, sorted(kernels)
    limit = lambda name: max([v for k, v in ALLOWED.items() if name.startswith(k)], default=0)  # noqa: E731
    assert {k: v for k, v in kernels.items() if v > limit(k)} == {}


def test_calibration_of_unaligned_rows_keeps_its_waves():
    """Eight waves on a SIMD (64 registers) up to 1024 columns: with fewer the loads of rows that are no whole chunks
    are waited for (72 registers: 245 us for 100k pairs of 900 bfloat16 columns, 218 us with at most 64)."""
    with open(LIB, "rb") as f:
        blob = f.read()
    registers = {_name(k[".name"]): k[".vgpr_count"] for obj in _code_objects(blob)
                 for k in _metadata(obj)["amdhsa.kernels"]}
    for name in ("k_pair_cosine<1, 0, 0>", "k_pair_cosine<2, 0, 0>"):
        assert registers[name] <= 64, (name, registers[name])
