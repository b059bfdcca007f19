"""No kernel of the library spills registers: a contraction loop whose accumulators and fragments no longer fit goes
through scratch memory at several times its cost, with the same results.  Read from the metadata of the code objects that
this tree has built; no GPU is needed."""
import os
import re
import shutil
import struct
import subprocess
import tempfile

import pytest

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(path):
    """The gfx950 code objects in the library's offload bundles (one bundle per source file)."""
    data = open(path, "rb").read()
    pos = data.find(MAGIC)
    while pos >= 0:
        count, = struct.unpack_from("<Q", data, pos + len(MAGIC))
        at = pos + len(MAGIC) + 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            if size and b"gfx950" in data[at + 24:at + 24 + name]:
                yield data[pos + offset:pos + offset + size]
            at += 24 + name
        pos = data.find(MAGIC, pos + len(MAGIC))


def test_no_kernel_spills():
    from paper_2407_17029_amd import binding
    if not os.path.exists(READELF):
        pytest.skip("llvm-readelf is not installed")
    if not os.path.exists(binding.LIB_PATH):
        from paper_2407_17029_amd import build
        build.build_library()
    spills = {}
    for obj in _code_objects(binding.LIB_PATH):
        with tempfile.NamedTemporaryFile(suffix=".co") as f:
            f.write(obj)
            f.flush()
            notes = subprocess.run([READELF, "--notes", f.name], capture_output=True, text=True, check=True).stdout
        names = re.findall(r"\.symbol:\s+(\S+)", notes)
        counts = re.findall(r"\.vgpr_spill_count:\s+(\d+)", notes)
        assert len(names) == len(counts)
        spills.update(zip(names, map(int, counts)))
    assert any("k_qlinear" in n for n in spills) and any("k_dense" in n for n in spills)
    assert not {n: c for n, c in spills.items() if c}
