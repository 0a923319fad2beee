"""Registers of the built GEMM kernels, from the code objects in libmsd.so (no
GPU): a variant that spills would read and write scratch memory between its
matrix instructions, which the runtime may have to allocate in a decode call."""
import os
import re
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The GPU code objects of every offload bundle in the library."""
    at = blob.find(MAGIC)
    while at >= 0:
        n = int.from_bytes(blob[at + 24:at + 32], "little")
        p = at + 32
        for _ in range(n):
            off, size, id_len = (int.from_bytes(blob[p + 8 * i:p + 8 * i + 8], "little")
                                 for i in range(3))
            target = blob[p + 24:p + 24 + id_len]
            if b"gfx950" in target:
                yield blob[at + off:at + off + size]
            p += 24 + id_len
        at = blob.find(MAGIC, at + 24)


def test_no_gemm_kernel_spills(tmp_path):
    from paper_2505_14260_amd import msd
    if not os.path.exists(msd.LIB_PATH) or not os.path.exists(READELF):
        pytest.skip("libmsd.so not built")
    seen, spills = 0, []
    for i, obj in enumerate(code_objects(open(msd.LIB_PATH, "rb").read())):
        path = tmp_path / f"{i}.co"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True,
                               check=True).stdout
        for k in re.split(r"\n\s+- \.agpr_count", notes)[1:]:
            kernel = re.findall(r"\.symbol:\s+(\S+)", k)[0]
            if "k_gemm" not in kernel and "k_feature" not in kernel:
                continue
            seen += 1
            if int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", k).group(1)):
                spills.append(kernel)
    assert seen >= 20, seen
    assert not spills, spills
