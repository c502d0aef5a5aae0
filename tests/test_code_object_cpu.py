"""What the compiled kernels ask of the device, read from the code objects' own
metadata in libfftpl.so (no GPU needed)."""
import os
import re
import struct
import subprocess
import tempfile

import pytest

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
READELF = "/opt/rocm/llvm/bin/llvm-readelf"


def _code_objects(path):
    """The gfx950 code objects bundled in a library built by hipcc."""
    data = open(path, "rb").read()
    for m in re.finditer(MAGIC, data):
        at = m.start() + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", data, at)
            name = data[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in name and size:
                yield data[m.start() + off:m.start() + off + size]


@pytest.fixture(scope="module")
def kernels():
    """(mangled name, static LDS bytes) of every kernel of the library."""
    from paper_1312_4587_amd import build
    build.ensure_built()
    got = []
    for obj in _code_objects(build.LIB):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(obj)
            f.flush()
            notes = subprocess.run([READELF, "--notes", f.name], capture_output=True, text=True,
                                   check=True).stdout
        sizes = [int(v) for v in re.findall(r"\.group_segment_fixed_size:\s*(\d+)", notes)]
        names = re.findall(r"\.symbol:\s*'?(\w+)\.kd", notes)
        assert len(sizes) == len(names) > 0
        got += zip(names, sizes)
    return got


# the dynamic LDS begins where the static LDS ends; k_compact_mid keeps float4 lists
# 16-byte aligned in it
def test_dynamic_lds_of_the_compact_kernel_is_aligned(kernels):
    mids = [(n, s) for n, s in kernels if "k_compact_mid" in n]
    assert len(mids) >= 20
    assert [n for n, s in mids if s % 16] == []
