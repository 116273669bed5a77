"""What the compiler made of the kernels, from the metadata of the built library's code objects: none of them spills or keeps anything in scratch memory."""
import os
import re
import struct
import subprocess

from paper_1805_05225_amd import binding as Bn

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    """The gfx950 entries of every offload bundle in the library: magic, count, then (offset, size, name length, name) each."""
    at = data.find(BUNDLE)
    while at >= 0:
        count, p = struct.unpack_from("<Q", data, at + 24)[0], at + 32
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length] and size:
                yield data[at + off:at + off + size]
            p += 24 + length
        at = data.find(BUNDLE, at + 24)


def test_no_kernel_uses_scratch_memory(tmp_path):
    assert os.path.exists(READELF)
    kernels, bad = 0, []
    for i, code in enumerate(_code_objects(open(Bn.LIB_PATH, "rb").read())):
        path = tmp_path / ("%d.elf" % i)
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for entry in notes.split("  - .agpr_count:")[1:]:
            field = lambda name: re.search(r"\.%s:\s+(\S+)" % name, entry).group(1)
            kernels += 1
            if int(field("private_segment_fixed_size")) or int(field("vgpr_spill_count")):
                bad.append((field("name"), field("private_segment_fixed_size")))
    assert kernels > 100 and not bad, bad
