"""Register use of the operator's kernels, read from the metadata of the code objects in the
built library: no instance of D or of the reduced operator keeps registers in scratch memory
(the set-up kernels, which run once per operator, do)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2202_07388_amd import qdw

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 code objects of a library's offload bundles."""
    at = data.find(MAGIC)
    while at >= 0:
        entry = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, entry)
            if b"gfx950" in data[entry + 24:entry + 24 + n]:
                yield data[at + off:at + off + size]
            entry += 24 + n
        at = data.find(MAGIC, at + 24)


def spills(tmp_path, pattern):
    """How many kernels of the library match, and those of them that spill registers."""
    if not os.path.exists(qdw.LIB_PATH) or not os.path.exists(READELF):
        pytest.skip("needs the built library and llvm-readelf")
    seen, spilled = 0, []
    with open(qdw.LIB_PATH, "rb") as fh:
        data = fh.read()
    for obj in code_objects(data):
        path = tmp_path / "obj"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in notes.split(".agpr_count")[1:]:
            field = lambda k: re.search(r"\.%s: +(\S+)" % k, kernel).group(1)  # noqa: E731
            if not re.search(pattern, field("symbol")):
                continue
            seen += 1
            if int(field("vgpr_spill_count")) or int(field("private_segment_fixed_size")):
                spilled.append((field("symbol"), field("vgpr_spill_count")))
    return seen, spilled


def test_operator_kernels_do_not_spill(tmp_path):
    seen, spilled = spills(tmp_path, r"\d+(dw_\w+?|schur)_kernelI")
    assert seen > 40 and not spilled, spilled


def test_block_solves_do_not_spill(tmp_path):
    """Storage in FP32 and FP16, and the reduced blocks in every type (the plain BF16 one keeps
    11 registers in memory: three waves per SIMD are faster with them than two without)."""
    seen, spilled = spills(tmp_path, r"\d+sap_mr_kernelILi[12]E|\d+sap_mr_eo_kernelI")
    assert seen == 8 and not spilled, spilled
