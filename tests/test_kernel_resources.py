"""CPU check of the built library's kernels: none uses scratch memory.  A
kernel that spills keeps part of its state in memory, and the persistent
sweep kernels that did have been seen to run fewer workgroups at once than the
occupancy query reports, which they rely on.  Read from the metadata that the
compiler leaves in the library's gfx950 code objects."""
import os
import re
import struct
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in triple:
                yield blob[at + offset:at + offset + size]
        at = blob.find(MAGIC, p)


def test_no_kernel_uses_scratch(tmp_path):
    from paper_1602_05716_amd import mc
    with open(mc.LIB_PATH, "rb") as f:
        blob = f.read()
    scratch = {}
    for k, obj in enumerate(_code_objects(blob)):
        path = tmp_path / ("%d.co" % k)
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for block in re.split(r"(?m)^\s+- \.a", notes)[1:]:
            name = re.search(r"\.name:\s+(_Z\S+)", block)
            if name:
                scratch[name.group(1)] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block).group(1))
    assert sum("sweep_kernel" in n for n in scratch) == 12 and len(scratch) >= 25, sorted(scratch)
    assert {n: s for n, s in scratch.items() if s} == {}
