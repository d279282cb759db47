"""What the compiler gave the kernels, from the metadata of the library's code objects (CPU only): no kernel spills
registers or keeps anything in scratch memory."""
import os
import re
import struct
import subprocess

import pytest

from paper_1805_01993_amd import binding as B

READELF = "/opt/rocm/lib/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects bundled into a host library."""
    data = open(path, "rb").read()
    at = data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + length].decode()
            pos += 24 + length
            if "gfx950" in target and size:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


def test_no_kernel_uses_scratch_memory(tmp_path):
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    kernels = {}
    for i, obj in enumerate(code_objects(B.LIB_PATH)):
        path = tmp_path / f"{i}.o"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
            name = re.search(r"\.symbol:\s+'?(\S+?)\.kd", kernel).group(1)
            kernels[name] = [int(re.search(rf"\.{key}:\s+(\d+)", kernel).group(1))
                             for key in ("private_segment_fixed_size", "vgpr_spill_count", "sgpr_spill_count")]
    assert sum("k_pipeline" in name for name in kernels) >= 300
    assert any("k_map" in name for name in kernels) and any("k_node_encode" in name for name in kernels)
    assert {name: v for name, v in kernels.items() if any(v)} == {}
