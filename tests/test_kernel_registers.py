"""The real backward kernel keeps what it needs in registers (no GPU: read from the built library's kernel metadata).

What a kernel spills it reloads through the same queue as its global memory accesses.  With addresses of the maps' rows spilled, the
form that adds its sums of dBm and dCm with atomics waited for all of them four times at the head of every tile: 6 packed
sequences of 32768 steps, 1536 channels, N = 16, bf16 1240 us, 1042 without."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_2602_08810_amd import build

READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(path):
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        pos = at + len(MAGIC) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + n]
            pos += 24 + n
            if b"gfx950" in name and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


def _spills(tmp_path):
    """{mangled kernel name: spilled vector registers} of the library."""
    found = {}
    for i, obj in enumerate(_code_objects(build.LIB)):
        f = tmp_path / f"{i}.o"
        f.write_bytes(obj)
        text = subprocess.run([READELF, "--notes", str(f)], capture_output=True, text=True, check=True).stdout
        names = re.findall(r"\.name:\s+(_Z\S+)\s*\n(?:.*\n)*?.*\.vgpr_spill_count:\s+(\d+)", text)
        found.update((n, int(c)) for n, c in names)
    return found


@pytest.mark.skipif(not os.path.exists(READELF), reason="no llvm-readelf")
def test_backward_kernel_spills_nothing(tmp_path):
    if not os.path.exists(build.LIB):
        pytest.skip("liblrnnx.so not built (run python -m paper_2602_08810_amd.build)")
    spills = _spills(tmp_path)
    for states in (8, 16, 32):                   # e^{Delta A}: the multipliers of S6 (0) and dirac (3)
        for disc in (0, 3):
            k = {n: c for n, c in spills.items() if re.search(rf"8k_ss_bwdI.*Li{states}ELi{disc}ELb", n)}
            assert len(k) == 8, f"{len(k)} kernels of N = {states}, scheme {disc}"        # types, gate, workspace
            assert not any(k.values()), k
