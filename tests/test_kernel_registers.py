"""Register spills of the built kernels, from the code objects' own metadata: no GEMM
kernel keeps more than four vector registers in scratch memory (tiles of 128 x 128 in
eight wavefronts are limited to 128 registers; a second set of accumulators in them
spilled 5 to 27 and cost fp32 projections of 4096 rows and more 2 to 7 %)."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_10820_amd", "libkforcing.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _kernels(tmp_path):
    """(name, spilled vector registers) of every kernel in the library."""
    data, found, at = open(LIB, "rb").read(), [], 0
    while (at := data.find(MAGIC, at)) >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + n].decode()
            p += 24 + n
            if "gfx950" not in target:
                continue
            f = tmp_path / f"{at}.co"
            f.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
            names = re.findall(r"^    \.name: +(\S+)", notes, re.M)
            spills = re.findall(r"^    \.vgpr_spill_count: +(\d+)", notes, re.M)
            assert len(names) == len(spills)
            found += zip(names, map(int, spills))
        at += len(MAGIC)
    return found


@pytest.mark.skipif(not (os.path.exists(LIB) and os.path.exists(READELF)), reason="needs the built library and llvm-readelf")
def test_gemm_kernels_do_not_spill(tmp_path):
    kernels = _kernels(tmp_path)
    gemms = [k for k in kernels if "gemm_kernel" in k[0] or "gemm_skinny_kernel" in k[0]]
    assert len(gemms) > 100
    assert [k for k in gemms if k[1] > 4] == []
