"""No kernel of the built library keeps registers in scratch memory (host only):
a sweep that does runs up to three times slower than its memory traffic."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2102_12416_amd", "libjc.so")
READELF = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The device code objects of the bundles that the host library embeds."""
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + n]
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
            p += 24 + n
        at = data.find(MAGIC, at + 1)


@pytest.mark.skipif(not os.path.exists(READELF), reason="llvm-readelf not installed")
def test_no_kernel_uses_scratch(tmp_path):
    kernels, scratch = 0, []
    for i, obj in enumerate(code_objects(open(LIB, "rb").read())):
        path = str(tmp_path / ("%d.o" % i))
        open(path, "wb").write(obj)
        notes = subprocess.run([READELF, "--notes", path], check=True, capture_output=True, text=True).stdout
        for m in re.finditer(r"\.name:\s+(_Z\S+)\n(?:.*\n)*?\s+\.private_segment_fixed_size:\s+(\d+)", notes):
            kernels += 1
            if int(m.group(2)):
                scratch.append((m.group(1), int(m.group(2))))
    assert kernels > 100, "no device code found in %s" % LIB
    assert not scratch, "%d kernels, the first: %s" % (len(scratch), scratch[:3])
