"""What the built library holds, read from the kernel descriptors that the compiler left in it: no kernel keeps registers in scratch
memory.  (The kernels fill their registers on purpose; a spill in a 16-bit epilogue costs time at the least.)"""
import os
import re
import struct
import subprocess
import tempfile

import pytest

from paper_2601_15013_amd import binding

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    at = blob.find(MAGIC)
    while at >= 0:
        n, p = struct.unpack_from("<Q", blob, at + len(MAGIC))[0], at + len(MAGIC) + 8
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + length] and size:
                yield blob[at + offset:at + offset + size]
            p += 24 + length
        at = blob.find(MAGIC, at + len(MAGIC))


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(binding.LIB_PATH):
        from paper_2601_15013_amd import build
        build.build()
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    found = {}
    with open(binding.LIB_PATH, "rb") as f:
        blob = f.read()
    for obj in code_objects(blob):
        with tempfile.NamedTemporaryFile(suffix=".co") as t:
            t.write(obj)
            t.flush()
            notes = subprocess.run([READELF, "--notes", t.name], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
            field = lambda k: re.search(r"\." + k + r":\s+(\S+)", kernel).group(1)  # noqa: E731
            found[field("name")] = {k: int(field(k)) for k in ("vgpr_spill_count", "sgpr_spill_count", "private_segment_fixed_size")}
    return found


def test_no_kernel_spills(kernels):
    assert sum("gemm_mfma_kernel" in k for k in kernels) > 50 and any("index_chain_kernel" in k for k in kernels)
    spilled = {k: v for k, v in kernels.items() if any(v.values())}
    assert not spilled, spilled
