"""Registers of the built kernels (no device needed): the metadata of the code
objects inside libpwadv.so.  A kernel that spills moves its spills through
memory on every level of its march."""
import re
import struct
import subprocess

import pytest

from paper_2301_13016_amd import binding as B

msgpack = pytest.importorskip("msgpack")
EM_AMDGPU, NT_METADATA = 224, 32


def _metadata(elf):
    """The msgpack documents of an AMDGPU code object's notes."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phsize)
        at, end = off, off + size
        while kind == 4 and at + 12 <= end:   # PT_NOTE
            nlen, dlen, ntype = struct.unpack_from("<III", elf, at)
            name = elf[at + 12:at + 12 + nlen]
            at += 12 + (nlen + 3) // 4 * 4
            if ntype == NT_METADATA and name.rstrip(b"\0") == b"AMDGPU":
                yield msgpack.unpackb(elf[at:at + dlen], strict_map_key=False)
            at += (dlen + 3) // 4 * 4


def scratch_by_kernel():
    """Demangled name -> bytes of scratch per lane of every kernel built in."""
    data = open(B.LIB_PATH, "rb").read()
    out = {}
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            for doc in _metadata(memoryview(data)[at:].tobytes()):
                for k in doc["amdhsa.kernels"]:
                    out[k[".name"]] = k[".private_segment_fixed_size"]
        at = data.find(b"\x7fELF", at + 4)
    plain = "\n".join(out).replace("DF16_", "Dh")   # _Float16, which older demanglers do not know
    names = subprocess.run(["c++filt"], input=plain, capture_output=True, text=True, check=True).stdout
    return dict(zip(names.split("\n"), out.values()))


def test_packed_kernels_do_not_spill():
    try:
        B.lib()
    except B.PWLibraryMissing:
        pytest.skip("library not built")
    packed = {}
    for name, scratch in scratch_by_kernel().items():
        m = re.search(r"pw_(forward|zfast)_kernel<([^>]*), true>", name)
        if m and m.group(1) + m.group(2):
            args = m.group(2).split(", ")
            if len(args) == (7 if m.group(1) == "forward" else 6):
                packed[m.group(0)] = (args, scratch)
    assert len(packed) > 60, "packed kernels not found in the library"
    # eight rows of FP64 do not fit any register file (a given shape only: no rule picks them)
    spilled = {n: s for n, (a, s) in packed.items() if s and (a[0], a[2]) != ("double", "8")}
    assert not spilled, spilled
