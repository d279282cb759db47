"""What the compiler gave the kernels, from the metadata of the library's code objects (CPU only): no kernel spills
registers or keeps anything in scratch memory."""
import os
import re
import shutil
import struct
import subprocess

import pytest

from paper_1805_01993_amd import binding as B

READELF = "/opt/rocm/lib/llvm/bin/llvm-readelf"
CXXFILT = shutil.which("c++filt")
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


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Per kernel: bytes of scratch memory, spilled vector and scalar registers."""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    tmp_path, kernels = tmp_path_factory.mktemp("objects"), {}
    for i, obj in enumerate(code_objects(B.LIB_PATH)):
        path = tmp_path / f"{i}.o"
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for kernel in re.split(r"\n\s+- \.agpr_count:", notes)[1:]:
            name = re.search(r"\.symbol:\s+'?(\S+?)\.kd", kernel).group(1)
            kernels[name] = [int(re.search(rf"\.{key}:\s+(\d+)", kernel).group(1))
                             for key in ("private_segment_fixed_size", "vgpr_spill_count", "sgpr_spill_count")]
    return kernels


def test_no_kernel_uses_scratch_memory(kernels):
    assert sum("k_pipeline" in name for name in kernels) >= 300
    assert any("k_map" in name for name in kernels) and any("k_node_encode" in name for name in kernels)
    assert {name: v for name, v in kernels.items() if any(v)} == {}


def test_one_pass_kernels_past_the_caches_have_ends_that_occur(kernels):
    """Packs of less than 16 bytes are read past the caches only where a packet and its segments are whole cache lines:
    the last segment is whole then (end 0; the kernels for several files a batch have 1, which takes that too)."""
    if not CXXFILT:
        pytest.skip("no c++filt")
    names = subprocess.run([CXXFILT], input="\n".join(kernels), capture_output=True, text=True, check=True).stdout
    found = re.findall(r"k_pipeline<ccdc::(\w+)(?:<\w+>)?, (\d), (\d), (true|false), (\d), (true|false)>", names)
    assert len(found) == sum("k_pipeline" in name for name in kernels)
    past = [(int(vec) * (2 if algebra == "Hyb16" else 4), multi, end) for algebra, vec, _, multi, end, kept in found
            if kept == "false"]
    assert {end for size, _, end in past if size == 16} == {"0", "1", "2"}
    assert {(multi, end) for size, multi, end in past if size < 16} == {("false", "0"), ("true", "1")}
