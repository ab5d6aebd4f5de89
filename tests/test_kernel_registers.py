"""What the compiler made of the kernels whose loads stay in flight over their K loops: a vector register that is spilled there
comes back through memory, and the wait for it is a wait for every load in front of it."""
import os
import re
import shutil
import struct
import subprocess

import pytest

import paper_1805_04170_amd.binding as binding

READELF = shutil.which("llvm-readelf", path="/opt/rocm/llvm/bin") or shutil.which("llvm-readelf")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects():
    data = open(binding.LIB_PATH, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        (n,), pos = struct.unpack_from("<Q", data, at + len(MAGIC)), at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, pos)
            name = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


@pytest.mark.skipif(READELF is None or not os.path.exists(binding.LIB_PATH), reason="no llvm-readelf, or the library is not built")
def test_kernels_with_loads_in_flight_keep_their_values_in_registers(tmp_path):
    seen = {}
    for i, obj in enumerate(code_objects()):
        path = os.path.join(str(tmp_path), "%d.o" % i)
        with open(path, "wb") as f:
            f.write(obj)
        notes = subprocess.run([READELF, "--notes", path], capture_output=True, text=True, check=True).stdout
        for name, spilled in re.findall(r"\.symbol:\s+(\S+)\.kd.*?\.vgpr_spill_count:\s+(\d+)", notes, re.S):
            kernel = re.search(r"(gemm_bf16_(?:v2|v3|v4|v6|rows|v5(?=_kernelILi\d+ELb[01]ELb0E))|conv_gather_a[24]|conv_wgrad_split2)_kernel", name)
            if kernel:
                seen.setdefault(kernel.group(1), []).append((name, int(spilled)))
    assert len(seen) == 9
    assert not [k for ks in seen.values() for k in ks if k[1]]
