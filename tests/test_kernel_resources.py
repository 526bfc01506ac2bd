"""The compiler's resource report of the built library, read from the metadata of its own code objects: kernels hold their data in
registers and LDS.  Scratch memory is off-chip traffic, and a value stored there right after its load waits for the load."""

import os
import re
import struct
import subprocess

import pytest

import paper_2512_11269_amd as K

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    for start in (m.start() for m in re.finditer(MAGIC, data)):
        at = start + len(MAGIC)
        (count,) = struct.unpack_from("<Q", data, at)
        at += 8
        for _ in range(count):
            offset, size, name = struct.unpack_from("<QQQ", data, at)
            if b"gfx950" in data[at + 24:at + 24 + name] and size:
                yield data[start + offset:start + offset + size]
            at += 24 + name


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """Bytes of scratch memory a lane, by kernel."""
    if not os.path.exists(READELF):
        pytest.skip("no %s" % READELF)
    K.load_library()
    path = tmp_path_factory.mktemp("code") / "object"
    found = {}
    with open(K.library_path(), "rb") as f:
        data = f.read()
    for code in _code_objects(data):
        path.write_bytes(code)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        names, sizes = re.findall(r"\.symbol:\s+(\S+)\.kd", notes), re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes)
        assert len(names) == len(sizes)
        found.update(zip(names, map(int, sizes)))
    assert len(found) > 100
    return found


@pytest.mark.parametrize("kernel", [
    r"rows_inner_product",                     # its split form too
    r"inner_product_kernel",
    r"rotate_mac_rows_kernel",
    r"rotate_finish_kernel",
    r"bconv_mfma_ntt_colsILi\dELi1ELi9E",      # one target per lane half, nine sources a half
])
def test_no_scratch_memory(scratch, kernel):
    of_kernel = {name: size for name, size in scratch.items() if re.search(r"\d" + kernel, name)}
    assert of_kernel
    assert not {name: size for name, size in of_kernel.items() if size}
